// Device functions of the per-prompt weight step: normalisation, ESS (Eq. "ess") and ESS-triggered resampling
// (Alg. 1; Sec. 7 implementation details; the other schemes App. E names).  A team of threads works on one prompt: one
// wave, or all waves of a workgroup.  The functions serve both the kernels of weights.hip and the tail of the vocabulary
// pass, where the workgroup that completes a prompt goes on to resample it.
//
// The sums that decide discrete outcomes (ESS < kappa*N, cumulative weights against the resampling positions)
// are accumulated in particle order, so that they round like a plain left-to-right loop.  Such a sum is a
// chain of dependent fp64 additions of 5.6 cycles each; what made it slow was not the chain but an LDS round trip per link,
// so a wave reads sixteen terms at a time, one read ahead, and broadcasts them lane by lane inside the addition.  A copy of
// the weights, the ESS and systematic resampling of 8 prompts: 512 particles 38.4 -> 18.1 us, 1024 particles 68.4 -> 27.5
// (three launches of any size take 12).
#pragma once
#include "device_rng.hpp"
#include "smc_internal.hpp"

namespace psmc {

// Orders the LDS traffic of one wave: what any lane wrote before is visible to every lane after.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// The threads that work on one prompt: `n` threads numbered `tid`; n is 64 (one wave) or the whole workgroup.
struct Team {
    int tid, n;
    __device__ __forceinline__ void sync() const { if (n == kWave) wave_sync(); else __syncthreads(); }
    __device__ __forceinline__ bool first_wave() const { return tid < kWave; }
};

// Threads of the stand-alone kernels' teams: one wave up to 128 particles, where a workgroup of 8 waves saves nothing
// (16 prompts of 128: 12.1 against 12.6 us for three launches), the workgroup above (256 particles: 13.5 against 18.3 us).
constexpr int kTeamThreads = 512;
inline int team_threads(int N) { return N <= 128 ? kWave : kTeamThreads; }

constexpr int kSerial = 16;                            // links of a serial sum per LDS read: one row of lanes

__host__ __device__ constexpr int pad_serial(int N) { return (N + kSerial - 1) / kSerial * kSerial; }

// LDS a team needs for a prompt of N particles: arrays padded to a multiple of kSerial.
struct PromptLds {
    double* w;                                         // log-weights of the prompt
    double* a; double* b;                              // scratch
    double* red;                                       // 32 doubles
    int32_t* anc;                                      // ancestors within the prompt, where it resampled
    int32_t* done; int32_t* par;                       // (plan of the reorder only) termination flag and live buffer ...
    double* cum;                                       // ... and cumulative log p of each row
    __host__ __device__ static constexpr size_t weight_bytes(int N) { return (size_t)pad_serial(N) * (3 * 8 + 4) + 32 * 8; }
    __host__ __device__ static constexpr size_t plan_bytes(int N) { return weight_bytes(N) + (size_t)pad_serial(N) * (8 + 2 * 4); }
    __device__ __forceinline__ PromptLds(unsigned char* lds, int N)
    {
        const int n = pad_serial(N);
        w = reinterpret_cast<double*>(lds);
        a = w + n; b = a + n; red = b + n;
        anc = reinterpret_cast<int32_t*>(red + 32);
        done = anc + n; par = done + n;
        cum = reinterpret_cast<double*>(par + n);      // (an even number of ints, kSerial being even)
    }
};

// One link of a serial sum: s += x(lane N of the row of 16) * m.  With m = 1 it is the rounded addition, with m = 0 it
// leaves s as it is.  (fp64 lane broadcasts exist for the two-operand v_fmac_f64.)  The wait before the first link is the
// one a lane broadcast needs after a vector write of its source.
#define PSMC_LINK(S, X, M, N) "v_fmac_f64_dpp " S ", " X ", " M " row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void serial_links(double& s, double x, double one)
{
    asm("s_nop 1\n\t"
        PSMC_LINK("%0", "%1", "%2", 0)
        PSMC_LINK("%0", "%1", "%2", 1)
        PSMC_LINK("%0", "%1", "%2", 2)
        PSMC_LINK("%0", "%1", "%2", 3)
        PSMC_LINK("%0", "%1", "%2", 4)
        PSMC_LINK("%0", "%1", "%2", 5)
        PSMC_LINK("%0", "%1", "%2", 6)
        PSMC_LINK("%0", "%1", "%2", 7)
        PSMC_LINK("%0", "%1", "%2", 8)
        PSMC_LINK("%0", "%1", "%2", 9)
        PSMC_LINK("%0", "%1", "%2", 10)
        PSMC_LINK("%0", "%1", "%2", 11)
        PSMC_LINK("%0", "%1", "%2", 12)
        PSMC_LINK("%0", "%1", "%2", 13)
        PSMC_LINK("%0", "%1", "%2", 14)
        PSMC_LINK("%0", "%1", "%2", 15)
        : "+v"(s) : "v"(x), "v"(one));
}
__device__ __forceinline__ void serial_links(double& s, double x, const double (&m)[kSerial])
{
    asm("s_nop 1\n\t"
        PSMC_LINK("%0", "%1", "%2", 0)
        PSMC_LINK("%0", "%1", "%3", 1)
        PSMC_LINK("%0", "%1", "%4", 2)
        PSMC_LINK("%0", "%1", "%5", 3)
        PSMC_LINK("%0", "%1", "%6", 4)
        PSMC_LINK("%0", "%1", "%7", 5)
        PSMC_LINK("%0", "%1", "%8", 6)
        PSMC_LINK("%0", "%1", "%9", 7)
        PSMC_LINK("%0", "%1", "%10", 8)
        PSMC_LINK("%0", "%1", "%11", 9)
        PSMC_LINK("%0", "%1", "%12", 10)
        PSMC_LINK("%0", "%1", "%13", 11)
        PSMC_LINK("%0", "%1", "%14", 12)
        PSMC_LINK("%0", "%1", "%15", 13)
        PSMC_LINK("%0", "%1", "%16", 14)
        PSMC_LINK("%0", "%1", "%17", 15)
        : "+v"(s) : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]), "v"(m[8]), "v"(m[9]), "v"(m[10]), "v"(m[11]), "v"(m[12]), "v"(m[13]), "v"(m[14]), "v"(m[15]));
}
#undef PSMC_LINK

// Left-to-right sums of two arrays padded with zeros (adding +0 changes nothing), by one whole wave; on every lane.
// The lower rows of lanes sum the one array, the upper rows the other.
__device__ inline void serial_sums(const double* a, const double* b, int N, double& s1, double& s2)
{
    const int lane = lane_id();
    const double* const src = (lane < kWave / 2 ? a : b) + (lane & (kSerial - 1));
    double s = 0.0, x = src[0];
    for (int i = 0; i < N; i += kSerial) {
        const double next = src[i + kSerial < N ? i + kSerial : i];
        serial_links(s, x, 1.0);
        x = next;
    }
    s1 = read_lane(s, 0); s2 = read_lane(s, kWave / 2);
}

// c[j] = a[0] + ... + a[j], left to right, by one whole wave; `a` is padded with zeros, `c` has room for the padding.
// Lane l of a row takes links 0 .. l of its sixteen and so ends with c[i + l].
__device__ inline void serial_scan(const double* a, double* c, int N)
{
    const int lane = lane_id(), l = lane & (kSerial - 1);
    double m[kSerial];
#pragma unroll
    for (int n = 0; n < kSerial; ++n) m[n] = n <= l ? 1.0 : 0.0;
    double s = 0.0, x = a[l];
    for (int i = 0; i < N; i += kSerial) {
        const int next = i + kSerial < N ? i + kSerial : i;
        const double nx = a[next + l];
        serial_links(s, x, m);
        if (lane < kSerial) c[i + l] = s;
        s = __shfl(s, kSerial - 1);
        x = nx;
    }
}

// log-sum-exp of x_i and of 2 x_i over one prompt, particle order, from sh.w (written and synchronised by the caller).
// Returns on every thread of the team.  One copy of the exponential and one of the logarithm, with the terms side by side on
// the lanes: a short launch waits for its code (fp64 exp and log take about 100 instructions each).
__device__ inline void prompt_lse(const Team& tm, int N, const PromptLds& sh, double& L1, double& L2)
{
    double mx = -INFINITY;
    for (int i = tm.tid; i < N; i += tm.n) mx = fmax(mx, sh.w[i]);
    mx = wave_max_f64(mx);
    if (tm.n > kWave) {
        if ((tm.tid & (kWave - 1)) == 0) sh.red[tm.tid / kWave] = mx;
        __syncthreads();
        for (int k = 0; k < tm.n / kWave; ++k) mx = fmax(mx, sh.red[k]);
    }
    const int Np = pad_serial(N);
#pragma unroll 1
    for (int k = tm.tid; k < 2 * Np; k += tm.n) {      // sh.a, then sh.b, which follows it
        const int i = k < Np ? k : k - Np;
        const double w = i < N ? sh.w[i] : 0.0;
        const double x = exp(k < Np ? w - mx : 2.0 * w - 2.0 * mx);
        sh.a[k] = i < N ? x : 0.0;
    }
    tm.sync();
    double s1 = 0.0, s2 = 0.0;
    if (tm.first_wave()) serial_sums(sh.a, sh.b, N, s1, s2);
    if (tm.n > kWave) {
        if (tm.tid == 0) { sh.red[16] = s1; sh.red[17] = s2; }
        __syncthreads();
        s1 = sh.red[16]; s2 = sh.red[17];
    }
    const double lg = log((tm.tid & 1) ? s2 : s1);
    L1 = mx + read_lane(lg, 0);
    L2 = 2.0 * mx + read_lane(lg, 1);
    tm.sync();                                          // sh.a and sh.b are free again
}

// first j in [0, n) with C_j >= p for a non-decreasing C; n-1 if rounding leaves none
__device__ __forceinline__ int first_reaching(const double* C, int n, double p)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (C[mid] >= p) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// uniform of word i of the prompt's resampling stream (Philox domain 1, row := prompt)
__device__ __forceinline__ double resampling_uniform(uint32_t i, uint32_t b, uint32_t step, uint32_t key0, uint32_t key1)
{
    const U4 blk = philox4x32_10(i >> 2, b, step, 1u, key0, key1);
    return ((double)pick_word(blk, i & 3u) + 0.5) * 0x1p-32;
}

// Residual resampling: floor(N w_j) copies of each j in index order, the rest by inversion of the residual weights' running
// sum (uniforms u_0, u_1, ...).  sh.a holds the normalised weights.
__device__ inline void residual_ancestors(const ResampleArgs& r, int b, uint32_t step, const Team& tm, const PromptLds& sh)
{
    const int N = r.N;
    int* const sh_k = reinterpret_cast<int*>(sh.red);
    if (tm.first_wave()) {
        const int lane = tm.tid;
        int k = 0;                                      // copies placed so far (exact integers: any order of addition will do)
        for (int j0 = 0; j0 < N; j0 += kWave) {
            const int j = j0 + lane;
            int copies = 0;
            if (j < N) {
                const double nw = (double)N * sh.a[j];
                copies = (int)floor(nw);
                sh.b[j] = nw - (double)copies;
            }
            int inc = copies;
            for (int o = 1; o < kWave; o <<= 1) { const int x = __shfl_up(inc, o); if (lane >= o) inc += x; }
            for (int c = 0; c < copies; ++c) {
                const int at = k + inc - copies + c;
                if (at < N) sh.anc[at] = j;
            }
            k += read_lane(inc, kWave - 1);
        }
        if (lane == 0) *sh_k = k < N ? k : N;
    }
    tm.sync();
    const int k = *sh_k, rest = N - k, Np = pad_serial(N);
    for (int j = tm.tid; j < Np; j += tm.n) sh.a[j] = j < N && rest > 0 ? sh.b[j] / (double)rest : 0.0;
    tm.sync();
    if (rest > 0 && tm.first_wave()) serial_scan(sh.a, sh.b, N);
    tm.sync();
    for (int i = tm.tid; i < rest; i += tm.n)
        sh.anc[k + i] = first_reaching(sh.b, N, resampling_uniform((uint32_t)i, (uint32_t)b, step, r.key0, r.key1));
}

// Ancestor order 1: every distinct ancestor keeps its own slot, the other copies, in the order in which they were drawn,
// fill the free slots in increasing order.  Rewrites sh.anc.
__device__ inline void survivors_in_place(int N, const Team& tm, const PromptLds& sh)
{
    int32_t* const first = reinterpret_cast<int32_t*>(sh.a);       // lowest draw of each ancestor, N where there is none
    int32_t* const extra = reinterpret_cast<int32_t*>(sh.b);       // the further copies, in the order drawn
    for (int i = tm.tid; i < N; i += tm.n) first[i] = N;
    tm.sync();
    for (int i = tm.tid; i < N; i += tm.n) atomicMin(&first[sh.anc[i]], i);
    tm.sync();
    if (tm.first_wave()) {
        int n = 0;
        for (int i0 = 0; i0 < N; i0 += kWave) {
            const int i = i0 + tm.tid;
            const bool more = i < N && first[sh.anc[i]] != i;
            const unsigned long long mk = __ballot(more);
            if (more) extra[n + mask_rank(mk)] = sh.anc[i];
            n += __popcll(mk);
        }
        wave_sync();
        n = 0;
        for (int i0 = 0; i0 < N; i0 += kWave) {
            const int i = i0 + tm.tid;
            const bool open = i < N && first[i] == N;
            const unsigned long long mk = __ballot(open);
            if (i < N) sh.anc[i] = open ? extra[n + mask_rank(mk)] : i;
            n += __popcll(mk);
        }
    }
    tm.sync();
}

// a3 + a4 for prompt b by one team: trigger ESS < kappa*N, ancestors, weights of resampled prompts reset.  Running sums
// of the normalised weights are taken in particle order by one lane.  scheme 0 is the paper's systematic resampling
// (A_i = min{ j : C_j >= (u_0 + i)/N }); 1 stratified ((u_i + i)/N), 2 multinomial (u_i), 3 residual
// (floor(N w_j) copies, the rest multinomial on the residual weights) are the alternatives App. E names.
// sh.w holds the prompt's weights (synchronised by the caller); lw: where they live in global memory, written with 0 where
// the prompt resamples.  Returns whether it did (on every thread); sh.anc then holds the ancestors, synchronised.
__device__ inline bool resample_prompt(const ResampleArgs& r, double* __restrict__ lw, int b, uint32_t step, const Team& tm,
                                       const PromptLds& sh)
{
    const int N = r.N;
    double L1, L2;
    prompt_lse(tm, N, sh, L1, L2);
    // the normalised weights, wanted only if the prompt resamples, and the ESS in one more pass through the exponential
    const int Np = pad_serial(N);
    double ess = 0.0;
#pragma unroll 1
    for (int i = tm.tid; i < Np + 1; i += tm.n) {
        const double x = exp(i < N ? sh.w[i] - L1 : 2.0 * L1 - L2);
        if (i < Np) sh.a[i] = i < N ? x : 0.0;
        else sh.red[18] = x;
    }
    tm.sync();
    ess = sh.red[18];
    const bool fire = ess < r.kappa * (double)N;         // strict; false for NaN
    if (tm.tid == 0) {
        if (r.ess_out) r.ess_out[b] = ess;
        r.resampled[b] = fire ? 1 : 0;
        // running estimate of the normalising constant: every resampling contributes the mean unnormalised weight
        if (fire && r.logZhat) r.logZhat[b] += L1 - r.log_N;
    }
    int32_t* A = r.anc + (int64_t)b * N;
    if (!fire) {
        for (int i = tm.tid; i < N; i += tm.n) A[i] = b * N + i;
        return false;
    }
    if (r.scheme == 3) {
        residual_ancestors(r, b, step, tm, sh);
    } else {
        if (tm.first_wave()) serial_scan(sh.a, sh.b, N);
        const double u0 = resampling_uniform(0u, (uint32_t)b, step, r.key0, r.key1);
        tm.sync();
        for (int i = tm.tid; i < N; i += tm.n) {
            double p;
            if (r.scheme == 0) p = (u0 + (double)i) / (double)N;
            else {
                const double u = resampling_uniform((uint32_t)i, (uint32_t)b, step, r.key0, r.key1);
                p = r.scheme == 1 ? (u + (double)i) / (double)N : u;
            }
            sh.anc[i] = first_reaching(sh.b, N, p);
        }
    }
    tm.sync();
    if (r.order == 1) survivors_in_place(N, tm, sh);
    for (int i = tm.tid; i < N; i += tm.n) { A[i] = b * N + sh.anc[i]; lw[i] = 0.0; }
    return true;
}

// host side: the arguments of resample_prompt for a context (defined in weights.hip)
ResampleArgs resample_args(const smc_ctx* c, double* logW, int32_t* anc, int32_t* resampled, double* ess_out);

}  // namespace psmc
