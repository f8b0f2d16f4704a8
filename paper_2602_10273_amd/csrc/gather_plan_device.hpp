// Device side of the reorder's plan (Alg. 1 "reorder KV cache by A"; App. C): a team of threads groups the moved rows of
// one resampled prompt by ancestor for the gather kernel.  In a header because several kernels run it: the plan kernel of
// smc_kv_reindex, and, when the reorder follows in the same call, whatever resampled the prompt goes on to plan it.
#pragma once
#include "weights_device.hpp"

namespace psmc {

// The plan of resampled prompt b by one team.  phase: which of the plan's two group counters this call uses.
// The caller has filled and synchronised sh.anc (ancestors within the prompt; -1: the row is left untouched), sh.cum,
// sh.done and sh.par (the rows' state before the reorder).
__device__ inline void plan_prompt(const PlanArgs& pl, int b, int phase, const Team& tm, const PromptLds& sh)
{
    const int N = pl.N, row0 = b * N;
    int32_t* const first = reinterpret_cast<int32_t*>(sh.b);       // lowest moved row that continues each ancestor
    int32_t* const group = first + pad_serial(N);                  // group number of each ancestor that has one
    int* const sh_base = reinterpret_cast<int*>(sh.red);
    // descendants of each ancestor as a bit set over the prompt's rows: in LDS where one word holds them (N <= 64)
    unsigned long long* const desc = reinterpret_cast<unsigned long long*>(sh.a);
    const bool one_word = pl.mask_words == 1;
    for (int k = tm.tid; k < N; k += tm.n) { first[k] = N; desc[k] = 0ull; }
    tm.sync();
    for (int k = tm.tid; k < N; k += tm.n) {
        const int a = sh.anc[k];
        if (a < 0 || a == k) continue;                             // a row that is its own ancestor has nothing to move
        atomicMin(&first[a], k);
        if (one_word) atomicOr(&desc[a], 1ull << k);
    }
    tm.sync();
    // leaders: first moved row (in particle order) of each distinct ancestor
    if (tm.first_wave()) {
        int n_lead = 0;
        for (int k0 = 0; k0 < N; k0 += kWave) {
            const int k = k0 + tm.tid;
            const bool lead = k < N && sh.anc[k] >= 0 && sh.anc[k] != k && first[sh.anc[k]] == k;
            const unsigned long long mk = __ballot(lead);
            if (lead) group[sh.anc[k]] = n_lead + mask_rank(mk);
            n_lead += __popcll(mk);
        }
        if (tm.tid == 0) *sh_base = n_lead ? atomicAdd(&pl.plan->n_groups[phase], n_lead) : 0;
    }
    tm.sync();
    const int base = *sh_base;
    for (int k = tm.tid; k < N; k += tm.n) {
        const int a = sh.anc[k];
        if (a < 0 || a == k || first[a] != k) continue;
        const int g = base + group[a];
        pl.grp_src[g] = row0 + a;
        pl.grp_base[g] = row0;
        // bit 0: the ancestor's live buffer, before any flip; bit 1 (only where the caller opted in and an
        // end-of-sequence token is configured): the ancestor has terminated -- its cache is never read again
        // (App. D: the absorbing state is a no-op), so its KV rows are not copied
        pl.grp_srcpar[g] = sh.par[a] | ((pl.skip_terminated && sh.done[a]) ? 2 : 0);
        if (one_word) pl.grp_mask[g] = desc[a];
        else for (int w = 0; w < pl.mask_words; ++w) pl.grp_mask[(int64_t)g * pl.mask_words + w] = 0ull;
    }
    if (!one_word) {                                               // the leaders have cleared, now every moved row adds itself
        __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt(0): the zeros precede the atomics
        tm.sync();
    }
    for (int k = tm.tid; k < N; k += tm.n) {
        const int a = sh.anc[k];
        if (a < 0 || a == k) continue;
        if (!one_word) atomicOr(&pl.grp_mask[(int64_t)(base + group[a]) * pl.mask_words + (k >> 6)], 1ull << (k & 63));
        pl.cumlogp[row0 + k] = sh.cum[a];
        pl.done[row0 + k] = sh.done[a];
        pl.parity[row0 + k] = sh.par[k] ^ 1;                       // from now on: the buffer this row is written to
    }
}

// What plan_prompt wants to find in LDS, from global memory.
__device__ inline void load_plan_state(const PlanArgs& pl, int b, const Team& tm, const PromptLds& sh)
{
    for (int k = tm.tid; k < pl.N; k += tm.n) {
        const int row = b * pl.N + k;
        sh.cum[k] = pl.cumlogp[row];
        sh.done[k] = pl.done[row];
        sh.par[k] = pl.parity[row];
    }
}

// The two group counters alternate between successive plans, and the switch happens on the device: every workgroup
// of a plan reads plan->phase first and calls this last; the one with the last ticket clears the other counter for
// the next plan and flips the phase.  No host-side state is involved, so a captured launch sequence can be replayed.
// (The read of the phase has to precede the ticket, and it has: its value chose the counter that was added to.  A device-wide
// fence here would write back and invalidate caches for nothing.)
__device__ inline void plan_finish(GatherPlan* plan, int phase, int n_workgroups)
{
    if (threadIdx.x == 0) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt(0): the phase has arrived
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");     // (for the compiler's order)
        if (__hip_atomic_fetch_add(&plan->ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_workgroups - 1) {
            plan->n_groups[phase ^ 1] = 0;
            plan->ticket = 0;
            plan->phase = phase ^ 1;
        }
    }
}

}  // namespace psmc
