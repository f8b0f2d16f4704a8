#!/usr/bin/env python3
"""Throughput of the Power-SMC per-token step on one MI355X.

One "step" is one pass of the whole hot path over one batch of synthetic logits with the KV cache resident in
HBM: smc_step_resample_reindex = smc_step_resample (boundary reweight, vocabulary pass, increment, ESS, trigger,
ancestors) -> smc_kv_reindex (KV / history / cumulative-log-p gather for the prompts that resampled), two launches below 1024 rows, three above.  Resampling fires
whenever the weights say so; how often is an observed quantity and is reported.

Prints ONE JSON line.  `value` is particle-steps/s over the timed steps.  `roofline` describes the kernel that
took the most time by the HIP events the library records on its own stream around each launch -- over the timed
steps themselves when a dense cache is bound (millisecond steps), else over a second window of as many steps right
after them (`config.kernel_events` says which); `roofline_other` the other dominant kernel.  `cpu_baseline` times the CPU
oracle on a bounded sample of the same workload, on all host cores and (in a child process) on one.

The default workload is the largest configuration (cfg4: 2048 rows of fp32 logits, 2 x 120 GB of KV cache), timed
in the regime it is defined for: the 128 steps of the exponent ramp run first, untimed, as a prologue (so the timed
steps see the weights, sums and histories the ramp leaves behind), then alpha is held at 4, resampling fires
whenever the accumulated weights say so, and the whole double-buffered cache is bound, so vocabulary pass,
resampling and gather run in the same step.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=0, help="timed steps (0: per-workload default)")
    ap.add_argument("--warmup", type=int, default=4)
    ap.add_argument("--workload", default="cfg4", choices=["cfg2", "cfg3", "cfg4", "cfg5"])
    ap.add_argument("--kv-positions", type=int, default=0,
                    help="--mode reindex: cache positions per head instead of the workload's (other row lengths)")
    ap.add_argument("--concentration", type=float, default=0.5,
                    help="--mode reindex: Dirichlet concentration of the synthetic weights the ancestors are drawn from "
                         "(smaller: fewer distinct ancestors, i.e. fewer rows read per row written)")
    ap.add_argument("--gather-variant", default="", metavar="V:G",
                    help="--mode reindex: kernel variant and workgroups per CU for smc_set_gather_tuning")
    ap.add_argument("--separate-launches", action="store_true",
                    help="smc_step and smc_resample as two calls instead of smc_step_resample (one launch for a0..a4)")
    ap.add_argument("--no-prologue", action="store_true",
                    help="skip the untimed steps through the workload's exponent ramp (the run then starts at t = 1)")
    ap.add_argument("--cpu-single-leg", action="store_true", help=argparse.SUPPRESS)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-kv", action="store_true", help="vocabulary pass + weights only (no cache bound)")
    ap.add_argument("--events-apart", action="store_true",
                    help="record the per-kernel events over a second window of steps instead of over the timed one")
    ap.add_argument("--n-split", type=int, default=0, help="slices a row is split over in the vocabulary pass (0: automatic)")
    ap.add_argument("--wg-waves", type=int, default=0, help="waves per workgroup of the vocabulary pass: 4, 8 or 16 (0: automatic)")
    ap.add_argument("--mode", default="step", choices=["step", "reindex", "attention"],
                    help="step: the whole hot path (default); reindex: the KV reorder alone, every prompt resampled "
                         "with synthetic ancestors (sorted draws from Dirichlet(0.5) weights); attention: decode "
                         "attention of every layer over the full cache (dense, or paged with --paged P)")
    ap.add_argument("--q-heads", type=int, default=0, help="query heads for --mode attention (default 7 per KV head)")
    ap.add_argument("--paged", type=int, default=0, metavar="P",
                    help="paged cache with P positions per page: the reorder copies page numbers, appends copy on write")
    ap.add_argument("--in-place", action="store_true",
                    help="ancestor order 1: surviving ancestors keep their slot, only the other copies move")
    return ap.parse_args()


def _cpu_gather_leg(w, seed, orc, np):
    """Oracle KV gather of one prompt (N rows) of a few tensors, scaled linearly to all tensors; seconds per prompt."""
    n_t = max(1, min(w.kv_tensors, int(1.5e9 // (w.N * w.kv_row_bytes))))
    rng = np.random.default_rng(seed)
    src = [rng.integers(0, 65535, size=(w.N, w.H, w.S, w.D), dtype=np.uint16) for _ in range(n_t)]
    dst = [np.empty_like(a) for a in src]
    anc = np.sort(rng.integers(0, w.N, w.N)).astype(np.int32)
    flag = np.ones(1, np.int32)
    t0 = time.perf_counter()
    for a, d in zip(src, dst):
        orc.gather_kv(a, anc, flag, w.N, w.S, d)
    return (time.perf_counter() - t0) * (w.kv_tensors / n_t), n_t


def _cpu_step_leg(w, seed, x, first_t, budget_s, orc):
    """Full-width oracle steps (vocabulary pass, ESS, resampling) on the rows of x until budget_s seconds of CPU work
    have been timed (at least 2 steps); seconds per step."""
    B = x[0].shape[0] // w.N
    o = orc.OracleSMC(B, w.N, w.V, first_t + 4096, w.kappa, seed, w.dtype)
    t0 = time.perf_counter()
    n_steps = 0
    while n_steps < 2 or (time.perf_counter() - t0 < budget_s and n_steps < 4000):
        t = first_t + n_steps
        o.step(x[n_steps % len(x)], t, w.alpha_at(t), w.alpha_at(t - 1), -1.0)
        o.resample(t)
        n_steps += 1
    return (time.perf_counter() - t0) / n_steps, n_steps


def _as_oracle_input(t, w):
    import numpy as np
    import torch
    t = t.cpu()
    return t.view(torch.int16).numpy().view(np.uint16) if w.dtype == "bf16" else t.numpy()


def cpu_single_leg(args):
    """Child process (OMP_NUM_THREADS=1 set by the parent before the oracle's library loads): the oracle on ONE core,
    on a few prompts of the same recipe.  Prints one JSON line; touches no GPU."""
    import numpy as np
    from oracle import reference as orc
    from paper_2602_10273_amd import synth
    w = synth.WORKLOADS[args.workload]
    sub = synth.scaled(w, B=max(1, 32 // w.N))
    x = [_as_oracle_input(synth.logits_torch(sub, 1000 + i, args.seed, device="cpu"), w) for i in range(2)]
    import ctypes
    ctypes.CDLL("libgomp.so.1").omp_set_num_threads(1)      # the OpenMP runtime the oracle links: one thread from here on
    first_t = w.ramp + 1
    t_step, n_steps = _cpu_step_leg(w, args.seed, x, first_t, 6.0, orc)
    t_gather, n_t = _cpu_gather_leg(w, args.seed, orc, np)
    print(json.dumps({"threads": orc.threads(), "rows": sub.R, "steps": n_steps, "step_s": t_step,
                      "gather_prompt_s": t_gather, "gather_tensors": n_t}))


def cpu_baseline(w, seed, gpu_resample_frac, ring, first_t, args):
    """The oracle as it stands, on the host cores: full-width steps on all rows of the same logits the GPU saw, plus
    the KV gather of one prompt's rows scaled to the number of prompts that resample per step.  A second leg runs
    the same oracle on one core in a child process (on a few prompts, scaled to all rows)."""
    import subprocess
    import numpy as np
    from oracle import reference as orc

    threads = orc.threads()
    x = [_as_oracle_input(ring[i], w) for i in range(min(2, len(ring)))]
    t_step, n_steps = _cpu_step_leg(w, seed, x, first_t, 10.0, orc)
    t_gather_prompt, n_t = _cpu_gather_leg(w, seed, orc, np)
    t_total = t_step + t_gather_prompt * gpu_resample_frac * w.B
    out = {
        "value": w.R / t_total, "unit": "particle-steps/s", "cores": threads, "kind": "oracle",
        "sample": (f"{n_steps} full-width steps (vocabulary pass + ESS + resampling) on all {w.R} rows, t >= {first_t}; KV "
                   f"gather of one prompt ({w.N} rows x {n_t} of {w.kv_tensors} tensors) scaled to all tensors and to the "
                   f"{gpu_resample_frac * w.B:.2f} prompts/step that resampled on the GPU"),
        "step_s": t_step, "gather_prompt_s": t_gather_prompt,
    }
    env = dict(os.environ, OMP_NUM_THREADS="1")
    cmd = [sys.executable, os.path.abspath(__file__), "--cpu-single-leg", "--workload", args.workload, "--seed", str(seed)]
    try:
        r = subprocess.run(cmd, env=env, capture_output=True, text=True, timeout=240, check=True)
        leg = json.loads(r.stdout.strip().splitlines()[-1])
        t1 = leg["step_s"] * (w.R / leg["rows"]) + leg["gather_prompt_s"] * gpu_resample_frac * w.B
        out["single_core"] = {
            "value": w.R / t1, "unit": "particle-steps/s", "cores": leg["threads"], "kind": "oracle",
            "sample": (f"{leg['steps']} full-width steps on {leg['rows']} rows scaled to {w.R}; KV gather of one prompt "
                       f"({leg['gather_tensors']} of {w.kv_tensors} tensors) scaled as above; child process, OpenMP limited to one thread"),
            "step_s_scaled": leg["step_s"] * (w.R / leg["rows"]), "gather_prompt_s": leg["gather_prompt_s"],
        }
    except (subprocess.SubprocessError, ValueError, KeyError, IndexError) as e:
        out["single_core"] = {"error": repr(e)[:200]}
    return out


def measured_ceilings(smc, torch, dev):
    """Plain streaming kernels of the library on a 4 GiB buffer: the device's own ceilings for four read:write mixes."""
    nbytes = 4 << 30
    buf = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream().cuda_stream
    out = {name: smc.smc_hbm_probe(kind, buf, nbytes, stream)
           for kind, name in enumerate(("read", "write", "copy_1r1w", "fanout_1r3w"))}
    del buf
    return out


def check_rows_after_reorder(s, w, anc_before, torch, np, n_rows=6):
    """One more reorder with the ancestors `anc_before`, then sampled destination rows of the first, a middle and the
    last tensor are compared byte for byte with their ancestors' rows as they were before it (moved rows of both
    parities and a row that stayed).  Raises on any mismatch: a timed cache that was never checked proves nothing."""
    _, _, par0 = s.state()
    anc = anc_before.cpu().numpy()
    moved = np.nonzero(anc != np.arange(w.R))[0]
    stay = np.nonzero(anc == np.arange(w.R))[0]
    pick = []
    for p in (0, 1):                                   # destination rows whose ancestors lived in buffer A / buffer B
        cand = moved[par0[anc[moved]] == p]
        pick += list(cand[:: max(1, len(cand) // (n_rows // 2))][: n_rows // 2])
    pick += list(stay[:1])
    tensors = sorted({0, w.kv_tensors // 2, w.kv_tensors - 1})
    want = {}
    for ten in tensors:
        for k in pick:
            a = int(anc[k])
            src = s.kvB[ten] if par0[a] else s.kvA[ten]
            want[(ten, int(k))] = src[a].clone()
    flag = torch.ones(w.B, dtype=torch.int32, device="cuda")
    s.reindex(w.S, 4, anc_before, flag)
    _, _, par1 = s.state()
    for (ten, k), ref in want.items():
        dst = s.kvB[ten] if par1[k] else s.kvA[ten]
        if not torch.equal(dst[k].view(torch.int16), ref.view(torch.int16)):
            raise RuntimeError(f"reorder check failed: tensor {ten}, row {k} differs from its ancestor {int(anc[k])}")
    assert all(par1[k] != par0[k] for k in pick[:-1] if anc[k] != k)


def reindex_only(args, w, K, W, smc, synth, Session, np, torch):
    """The KV reorder alone at the workload's full cache: K launches with distinct synthetic ancestor vectors."""
    if args.kv_positions:
        w = synth.scaled(w, S=args.kv_positions)
    s = Session(w.B, w.N, w.V, 8, w.dtype, w.kappa, args.seed, kv_geom=(w.kv_tensors, w.H, w.S, w.D))
    if args.gather_variant:
        v, g_ = (int(x) for x in args.gather_variant.split(":"))
        smc.smc_set_gather_tuning(s.ctx, g_, v)
    g = torch.Generator(device="cuda"); g.manual_seed(args.seed + 12345)
    for t in s.kvA:
        t.normal_(generator=g)
    ancs = [synth.ancestors_numpy(w, args.seed + i, args.concentration) for i in range(W + K)]
    d_anc = [torch.as_tensor(a).cuda() for a in ancs]
    flag = torch.ones(w.B, dtype=torch.int32, device="cuda")
    for i in range(W):
        s.reindex(w.S, 4, d_anc[i], flag)
    torch.cuda.synchronize()
    smc.smc_profile_enable(s.ctx, 1)
    t0 = time.perf_counter()
    for i in range(W, W + K):
        s.reindex(w.S, 4, d_anc[i], flag)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_gather, n_gather = smc.smc_profile_read(s.ctx, 1)
    smc.smc_profile_enable(s.ctx, 0)
    check_rows_after_reorder(s, w, d_anc[W + K - 1], torch, np)
    ident = np.arange(w.R)
    rows_written = rows_read = 0
    for a in ancs[W:]:
        moved = a != ident
        rows_written += int(moved.sum())
        rows_read += sum(len(np.unique(a[b * w.N:(b + 1) * w.N][moved[b * w.N:(b + 1) * w.N]])) for b in range(w.B))
    total_bytes = float(rows_written + rows_read) * w.kv_row_bytes * w.kv_tensors
    gbps = total_bytes / (ms_gather * 1e-3) / 1e9
    s.close()
    del s
    torch.cuda.empty_cache()
    out = {
        "metric": "particle-steps/s (KV reindex only), 1 MI355X",
        "value": w.R * K / elapsed, "unit": "particle-steps/s", "n_gpus": 1, "steps": K, "warmup": W,
        "ms_per_step": elapsed / K * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u8", "data": "synthetic",
        "config": {"workload": w.name, "mode": "reindex", "B": w.B, "N": w.N,
                   "kv": f"{w.layers}x2 tensors [{w.R},{w.H},{w.S},{w.D}] bf16 x2 buffers", "valid_len": w.S,
                   "ancestors": f"sorted draws from Dirichlet({args.concentration}) weights, every prompt resampled",
                   "rows_read_per_row_written": rows_read / max(rows_written, 1)},
        "roofline": {"kernel": "gather_kernel", "bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": gbps / HBM_PEAK_GBPS, "traffic": None, "launches": int(n_gather),
                     "avg_launch_ms": ms_gather / max(n_gather, 1), "algorithmic_bytes_per_launch": total_bytes / max(n_gather, 1)},
    }
    out["measured_ceilings_GBps"] = measured_ceilings(smc, torch, "cuda")
    print(json.dumps(out))


def attention_only(args, w, K, W, smc, synth, Session, np, torch):
    """Decode attention of all layers over the workload's full cache: one step = one call per layer."""
    P = args.paged
    s = Session(w.B, w.N, w.V, 8, w.dtype, w.kappa, args.seed, kv_geom=(w.kv_tensors, w.H, w.S, w.D), with_hist=False,
                page_len=P, len0=w.S)
    g = torch.Generator(device="cuda"); g.manual_seed(args.seed + 12345)
    for t in (s.pools if P else s.kvA):
        t.normal_(generator=g)
    if not P:                                           # rows in both buffers, as after a few reorders
        flag = torch.ones(w.B, dtype=torch.int32, device="cuda")
        for i in range(2):
            s.reindex(w.S, 0, torch.as_tensor(synth.ancestors_numpy(w, args.seed + i)).cuda(), flag)
    Hq = args.q_heads or 7 * w.H
    q = torch.randn((w.R, Hq, w.D), device="cuda", generator=g).to(torch.bfloat16)
    scale = float(w.D) ** -0.5

    def one_step():
        for layer in range(w.layers):
            s.attention(2 * layer, 2 * layer + 1, q, w.S, scale)

    for _ in range(W):
        one_step()
    torch.cuda.synchronize()
    smc.smc_profile_enable(s.ctx, 1)
    t0 = time.perf_counter()
    for _ in range(K):
        one_step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms, n = smc.smc_profile_read(s.ctx, 3)
    smc.smc_profile_enable(s.ctx, 0)
    bytes_per_call = 2.0 * w.R * w.H * w.S * w.D * 2            # K and V of one layer, every position read once
    gbps = bytes_per_call * n / (ms * 1e-3) / 1e9
    s.close()
    del s
    torch.cuda.empty_cache()
    out = {
        "metric": "particle-steps/s (decode attention of all layers only), 1 MI355X",
        "value": w.R * K / elapsed, "unit": "particle-steps/s", "n_gpus": 1, "steps": K, "warmup": W,
        "ms_per_step": elapsed / K * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": w.name, "mode": "attention", "rows": w.R, "kv_heads": w.H, "q_heads": Hq, "head_dim": w.D,
                   "positions": w.S, "layers": w.layers, "cache": f"paged, {P} positions per page" if P else "dense, double-buffered rows"},
        "roofline": {"kernel": "attn_decode_kernel", "bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": gbps / HBM_PEAK_GBPS, "traffic": None, "launches": int(n), "avg_launch_ms": ms / max(n, 1),
                     "algorithmic_bytes_per_launch": bytes_per_call},
    }
    try:
        ratio = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic_ratio.json"))).get(args.workload, {}).get("attn_decode_kernel")
        if ratio and not P:
            out["roofline"]["traffic"] = ratio * bytes_per_call
            out["roofline"]["traffic_source"] = "profiles/hbm_traffic_ratio.json x algorithmic bytes of this run"
    except OSError:
        pass
    out["measured_ceilings_GBps"] = measured_ceilings(smc, torch, "cuda")
    print(json.dumps(out))


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py: this build measures one GPU only (the path shards by prompt with no communication); "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)
    if args.cpu_single_leg:
        return cpu_single_leg(args)
    import numpy as np
    import torch
    from paper_2602_10273_amd import binding as smc
    from paper_2602_10273_amd import synth
    from paper_2602_10273_amd.harness import Session

    w = synth.WORKLOADS[args.workload]
    K = args.steps or {"cfg2": 48, "cfg3": 16, "cfg4": 24, "cfg5": 16}[args.workload]
    W = args.warmup
    if args.mode == "reindex":
        torch.cuda.set_device(0)
        return reindex_only(args, w, K, min(W, 2), smc, synth, Session, np, torch)
    if args.mode == "attention":
        torch.cuda.set_device(0)
        return attention_only(args, w, K, min(W, 2), smc, synth, Session, np, torch)
    dev = "cuda"
    torch.cuda.set_device(0)
    # untimed prologue: the steps of the exponent ramp where the workload has one (cfg4: t = 1..128), so that the timed
    # steps run at the held exponent (the integer-exponent instantiation of the vocabulary pass) on the state a real
    # run has there
    prologue = 0 if args.no_prologue else w.ramp
    first_t = 1
    T_max = (prologue + W + 2 * K + 8 + 3) // 4 * 4

    kv_geom = None if args.no_kv else (w.kv_tensors, w.H, w.S, w.D)
    P = 0 if args.no_kv else args.paged
    len0 = max(0, w.S - (prologue + W + 2 * K) - 1)           # paged runs: the cache is this full when the run starts
    kv_note = None
    s = None
    try:
        s = Session(w.B, w.N, w.V, T_max, w.dtype, w.kappa, args.seed, kv_geom=kv_geom, page_len=P, len0=len0)
    except torch.OutOfMemoryError:
        if args.workload != "cfg4" or args.no_kv:
            raise
    if s is None:
        # the 2 x 120 GB cache did not fit beside whatever else holds device memory: the next largest configuration
        import gc
        gc.collect()
        torch.cuda.empty_cache()
        args.workload = "cfg3"
        w = synth.WORKLOADS["cfg3"]
        kv_note = "cfg4's 246 GB allocation failed on this box; fell back to cfg3"
        prologue = 0
        kv_geom = (w.kv_tensors, w.H, w.S, w.D)
        len0 = max(0, w.S - (prologue + W + 2 * K) - 1)
        s = Session(w.B, w.N, w.V, T_max, w.dtype, w.kappa, args.seed, kv_geom=kv_geom, page_len=P, len0=len0)
    if args.n_split or args.wg_waves:
        smc.smc_set_tuning(s.ctx, args.n_split, 0, args.wg_waves)
    if args.in_place:
        smc.smc_set_ancestor_order(s.ctx, 1)
    if args.gather_variant:
        v, g_ = (int(x) for x in args.gather_variant.split(":"))
        smc.smc_set_gather_tuning(s.ctx, g_, v)
    if not args.no_kv:
        g = torch.Generator(device=dev); g.manual_seed(args.seed + 12345)
        for t in (s.pools if P else s.kvA):
            t.normal_(generator=g)
    n_ring = 4 if w.dtype == "f32" else 16       # distinct logits buffers: more bytes than the 256 MB last-level cache
    # Each buffer holds kExtraRows more i.i.d. rows than the workload has, and the window of R rows a step reads slides
    # by one row every n_ring steps: no particle slot meets the same logits row twice within n_ring * (kExtraRows + 1)
    # steps.  (Re-using a buffer unshifted would hit the same rows with the same increments every n_ring steps, which
    # is not the recipe's fresh draw per step: the weights would degenerate differently.)
    kExtraRows = 256
    w_gen = synth.scaled(w, B=w.B + (kExtraRows + w.N - 1) // w.N)
    ring = [synth.logits_torch(w_gen, i, args.seed) for i in range(n_ring)]
    torch.cuda.synchronize()

    def logits_of(t):
        shift = ((t - 1) // n_ring) % (kExtraRows + 1)
        return ring[t % n_ring][shift:shift + w.R]

    step_no = [first_t - 1]

    # Paged cache: the reorder after token t and the preparation of the next position are one call (and one launch
    # less) unless --separate-launches asks for the two calls; the first position is prepared before the first step.
    paged_fused = bool(P) and not args.separate_launches
    if paged_fused:
        s.prepare_append(len0)

    def prepare(t):
        if P and not paged_fused:
            s.prepare_append(len0 + (t - first_t))  # the decoder would now write this position and emit logits

    def reorder(t):
        if paged_fused:
            s.paged_reindex_prepare(t, len0 + (t - first_t) + 1)
        elif P:
            s.paged_reindex(t)
        else:
            s.reindex(w.S, t)

    def one_step():
        step_no[0] += 1
        t = step_no[0]
        prepare(t)
        if args.separate_launches:
            s.step(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), -1.0)
            s.resample(t)
        elif P:     # a0..a4 in one launch: the wave that completes a prompt's last row resamples the prompt
            s.step_resample(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), -1.0)
        else:       # a0..a5 in one call: two launches below 1024 rows, three above
            s.step_resample_reindex(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), w.S)
            return
        reorder(t)

    n_pro_resampled = 0
    for _ in range(prologue):
        one_step()
        n_pro_resampled += s.resampled          # device tensor: no synchronisation inside the prologue
    for _ in range(W):
        one_step()
    torch.cuda.synchronize()
    t_first_timed = step_no[0] + 1
    anc_log = torch.zeros((K, w.R), dtype=torch.int32, device=dev)
    flag_log = torch.zeros((K, w.B), dtype=torch.int32, device=dev)

    def logged_step(i):                                   # one_step() + what the step resampled (two small device copies)
        step_no[0] += 1
        t = step_no[0]
        prepare(t)
        if args.separate_launches:
            s.step(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), -1.0)
            s.resample(t)
        elif P:
            s.step_resample(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), -1.0)
        else:
            s.step_resample_reindex(logits_of(t), t, w.alpha_at(t), w.alpha_at(t - 1), w.S)
            anc_log[i].copy_(s.anc); flag_log[i].copy_(s.resampled)
            return
        anc_log[i].copy_(s.anc); flag_log[i].copy_(s.resampled)
        reorder(t)

    # Millisecond steps (a dense cache bound): the per-kernel HIP events are recorded over the timed region itself, so
    # that the kernel times and the step time describe the same steps -- which prompts resample, and with them the
    # bytes gathered, differ from step to step.  The events (and the log of what resampled) cost a few microseconds per
    # launch; where a step is tens of microseconds (no cache, or the paged cache) the timed region runs bare and the
    # events are recorded over a second window of the same length right after it.
    events_in_timed = (not args.no_kv) and not P and not args.events_apart
    if events_in_timed:
        smc.smc_profile_enable(s.ctx, 1)
        torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(K):
        if events_in_timed:
            logged_step(i)
        else:
            one_step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    if not events_in_timed:
        smc.smc_profile_enable(s.ctx, 1)
        for i in range(K):
            logged_step(i)
    first_logged = step_no[0] - K + 1
    ms_vocab, n_vocab = smc.smc_profile_read(s.ctx, 0)
    ms_gather, n_gather = smc.smc_profile_read(s.ctx, 2 if P else 1)
    smc.smc_profile_enable(s.ctx, 0)
    anc_h = anc_log.cpu().numpy().reshape(K, w.B, w.N)
    flag_h = flag_log.cpu().numpy()
    esz = 2 if w.dtype == "bf16" else 4
    vocab_bytes = float(w.R) * w.V * esz                              # per launch: every logit read once
    # per resampled prompt: rows whose ancestor is another row are written once; their distinct ancestors are read once
    local = anc_h - (np.arange(w.B)[None, :, None] * w.N)
    moved = (local != np.arange(w.N)[None, None, :]) & (flag_h[:, :, None] != 0)
    rows_written = int(moved.sum())
    rows_read = sum(len(np.unique(local[i, b][moved[i, b]])) for i in range(K) for b in range(w.B))
    gather_bytes_total = float(rows_written + rows_read) * w.kv_row_bytes * w.kv_tensors
    if P:
        # an append at offset o = pos % P copies o positions (read + write) for every sharer of a page but one: the
        # rows of the prompts that resampled at the previous step, minus their distinct ancestors
        gather_bytes_total = 0.0
        pos_bytes = w.kv_row_bytes // w.S
        # (with reorder and preparation in one call, step i prepares the position after its own and the sharers are
        # those its own resampling made)
        for i in range(0 if paged_fused else 1, K):
            o = (len0 + first_logged - first_t + i + (1 if paged_fused else 0)) % P
            src = i if paged_fused else i - 1
            needy = sum(w.N - len(np.unique(local[src, b])) for b in range(w.B) if flag_h[src, b])
            gather_bytes_total += 2.0 * needy * o * pos_bytes * w.kv_tensors
    resample_frac = float(flag_h.mean())

    def roof(name, total_bytes, ms, launches):
        if launches == 0 or ms <= 0:
            return {"kernel": name, "bound": "hbm", "achieved": 0.0, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                    "frac": 0.0, "traffic": None, "launches": int(launches)}
        gbps = total_bytes / (ms * 1e-3) / 1e9
        return {"kernel": name, "bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                "frac": gbps / HBM_PEAK_GBPS, "traffic": None, "launches": int(launches),
                "avg_launch_ms": ms / launches, "algorithmic_bytes_per_launch": total_bytes / launches}

    # HBM traffic per launch is not a counter of this run: rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this same
    # command (calibrated on a copy of known size) gave traffic as a multiple of the algorithmic bytes; that committed
    # ratio is applied to this run's algorithmic bytes and labelled as derived.
    ratios = {}
    try:
        ratios = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic_ratio.json"))).get(args.workload, {})
    except OSError:
        pass

    r_vocab = roof("vocab_pass_kernel", vocab_bytes * n_vocab, ms_vocab, n_vocab)
    r_gather = roof("paged_copy_kernel" if P else "gather_kernel", gather_bytes_total, ms_gather,
                    n_gather if not args.no_kv else 0)
    for r in (r_vocab, r_gather):
        if r["kernel"] in ratios and r.get("algorithmic_bytes_per_launch"):
            r["traffic"] = ratios[r["kernel"]] * r["algorithmic_bytes_per_launch"]
            r["traffic_source"] = ("derived, not measured in this run: the FETCH_SIZE+WRITE_SIZE / algorithmic-bytes ratio "
                                   "in profiles/hbm_traffic_ratio.json x the algorithmic bytes of this run")
    dominant, other = (r_gather, r_vocab) if ms_gather >= ms_vocab else (r_vocab, r_gather)

    out = {
        "metric": "particle-steps/s (SMC step + KV reindex), 1 MI355X",
        "value": w.R * K / elapsed, "unit": "particle-steps/s", "n_gpus": 1, "steps": K, "warmup": W,
        "ms_per_step": elapsed / K * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": w.dtype, "data": "synthetic",
        "config": {"workload": w.name, "B": w.B, "N": w.N, "V": w.V, "logits_dtype": w.dtype, "alpha": w.alpha,
                   "prologue_steps": prologue, "first_timed_step": t_first_timed,
                   "alpha_timed": [w.alpha_at(t_first_timed), w.alpha_at(t_first_timed + K - 1)],
                   "kernel_events": "recorded over the timed steps" if events_in_timed
                                    else f"recorded over the {K} steps after the timed ones",
                   "prologue_resampled_prompt_fraction": (float(n_pro_resampled.sum()) / (prologue * w.B)) if prologue else None,
                   "kappa": w.kappa, "ancestor_order": "survivors-in-place" if args.in_place else "as-drawn", "kv": None if args.no_kv else (f"{w.layers}x2 paged pools [{w.B}x{s.Q},{w.H},{P},{w.D}] bf16, {len0} positions filled at start"
                                                 if P else f"{w.layers}x2 tensors [{w.R},{w.H},{w.S},{w.D}] bf16 x2 buffers"),
                   "valid_len": w.S, "resampled_prompt_fraction": resample_frac,
                   "rows_read_per_row_written": rows_read / max(rows_written, 1),
                   "launches_per_step": (3 if paged_fused else 5) if P else (4 if args.separate_launches else 2 if w.R < 1024 and args.wg_waves != 4 else 3),
                   "logits_ring": f"{n_ring} buffers of {w_gen.R} rows, window of {w.R} rows sliding one row per {n_ring} steps"},
        "roofline": dominant, "roofline_other": other,
    }
    if kv_note:
        out["config"]["note"] = kv_note
    s.close()
    del s
    torch.cuda.empty_cache()
    # the device's own ceilings (plain streaming kernels) as a second, measured denominator
    out["measured_ceilings_GBps"] = measured_ceilings(smc, torch, dev)
    out["device_copy_GBps"] = out["measured_ceilings_GBps"]["copy_1r1w"]
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, args.seed, resample_frac if not args.no_kv else 0.0, [r[:w.R] for r in ring], t_first_timed, args)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
