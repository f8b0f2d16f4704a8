"""Performance cases: the calls a decoder makes of this library, over the sizes it makes them at.

A decode loop with particles makes, per token, a vocabulary step (with or without the resampling and the reorder in the
same call), a reorder of its dense cache or of its page tables, and -- per layer -- a store of the new keys and values
and an attention over the cache.  The cases are these calls one by one, and two whole generations.  Every case is a dict
of plain values; `prepare` makes on the GPU what the caller has in hand, `run` is one pass through the public calls.
"""
import math

import numpy as np
import torch

from paper_2602_10273_amd import binding as smc
from paper_2602_10273_amd.harness import Session

DEV = "cuda"


# ---- cases ----------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest step: the enumerable toy model (four particles, eight tokens); what counts is latency
        dict(name="step_tiny_1x4_f32", kind="step", call="full", B=1, N=4, V=8, dtype="f32", values="gauss", alpha=4.0,
             alpha_prev=4.0, tau=-1.0, kappa=0.5, T=8, eos=False, masked=False),
        # one user: one prompt, 64 particles, a 152k vocabulary
        dict(name="step_1x64_bf16", kind="step", call="step_resample", B=1, N=64, V=152064, dtype="bf16",
             values="gauss_boost", alpha=4.0, alpha_prev=4.0, tau=-1.0, kappa=0.5, T=512, eos=False, masked=False),
        # a served batch: 16 prompts of 8 particles
        dict(name="step_16x8_bf16", kind="step", call="step_resample", B=16, N=8, V=152064, dtype="bf16",
             values="gauss_boost", alpha=4.0, alpha_prev=4.0, tau=-1.0, kappa=0.5, T=512, eos=False, masked=False),
        # odd sizes: a ragged vocabulary with masked ids, a proposal temperature off 1/alpha, a stage boundary, terminated rows
        dict(name="step_12x10_bf16_ragged", kind="step", call="full", B=12, N=10, V=50257, dtype="bf16",
             values="gauss_boost", alpha=2.5, alpha_prev=2.4, tau=0.7, kappa=0.5, T=256, eos=True, masked=True),
        # the largest step: 64 prompts of 32 particles, fp32 heavy-tailed logits, inside the exponent ramp
        dict(name="step_64x32_f32_ramp", kind="step", call="full", B=64, N=32, V=152064, dtype="f32", values="student_t",
             alpha=2.5, alpha_prev=2.4765625, tau=-1.0, kappa=0.5, T=256, eos=False, masked=False),
        # the same batch with bf16 logits through the entry point that owns no workspace
        dict(name="step_64x32_bf16_noalloc", kind="step", call="noalloc", B=64, N=32, V=152064, dtype="bf16",
             values="gauss_boost", alpha=4.0, alpha_prev=4.0, tau=-1.0, kappa=0.5, T=256, eos=False, masked=False),
        # ESS and resampling of the caller's own weights, many particles
        dict(name="weights_8x512", kind="weights", B=8, N=512, kappa=0.5, spread=2.0, scheme=0, order=0),
        # the dense reorder of a 28-layer cache, every prompt resampled, a prefix that is not the whole capacity
        dict(name="reorder_16x8_28_layers", kind="reorder", B=16, N=8, layers=28, H=4, S=1024, D=128, valid=1000, T=512,
             t=437, share=1.0),
        # decode attention of one layer over the dense cache, 7 query heads per KV head
        dict(name="attention_16x8_dense", kind="attention", B=16, N=8, H=4, G=7, S=2048, D=128, length=2031, page=0),
        # ... and over pages of 16 positions, one user, an odd length
        dict(name="attention_1x64_paged", kind="attention", B=1, N=64, H=8, G=4, S=2048, D=128, length=1337, page=16),
        # a whole generation of 24 tokens, four layers, paged cache: every call of the loop
        dict(name="generate_16x8_paged", kind="generate", B=16, N=8, V=152064, dtype="bf16", values="gauss_boost",
             alpha=4.0, ramp=0, kappa=0.5, layers=4, H=4, G=7, S=1024, D=128, page=16, len0=700, tokens=24, eos=False),
        # a short one with a small vocabulary, dense cache, exponent ramp and an end-of-sequence token: latency-bound
        dict(name="generate_2x16_dense", kind="generate", B=2, N=16, V=32000, dtype="f32", values="gauss_boost",
             alpha=4.0, ramp=16, kappa=0.5, layers=2, H=2, G=2, S=256, D=64, page=0, len0=90, tokens=32, eos=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "weights", "reorder", "attention", "attention", "generate"])
    if kind == "step":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        esz = 2 if dtype == "bf16" else 4
        while True:
            B, N, V = _log(rng, 1, 64), _log(rng, 1, 128), _log(rng, 8, 160000)
            if 64 <= B * N * V * esz <= 1.25e9 and B * N <= 4096:
                break
        call = rng.choice(["full", "step_resample", "noalloc"])
        ints = rng.random() < 0.5
        alpha = float(rng.choice([2, 3, 4, 6])) if ints else round(rng.uniform(1.1, 6.0), 3)
        return dict(kind="step", call=call, B=B, N=N, V=V, dtype=dtype,
                    values="gauss" if V < 64 else rng.choice(["gauss_boost", "gauss_boost", "student_t"]), alpha=alpha,
                    alpha_prev=alpha if ints else round(max(1.0, alpha - 0.1), 3),
                    tau=round(rng.uniform(0.3, 1.2), 3) if rng.random() < 0.25 else -1.0, kappa=rng.choice([0.3, 0.5, 0.7]),
                    T=4 * _log(rng, 2, 128), eos=bool(V >= 64 and rng.random() < 0.3),
                    masked=bool(V >= 64 and rng.random() < 0.3))
    if kind == "weights":
        return dict(kind="weights", B=_log(rng, 1, 64), N=_log(rng, 4, 1024), kappa=rng.choice([0.3, 0.5, 0.7]),
                    spread=round(rng.uniform(0.5, 3.0), 2), scheme=rng.choice([0, 0, 0, 1, 2, 3]), order=rng.choice([0, 0, 1]))
    if kind == "reorder":
        while True:
            B, N, layers = _log(rng, 1, 64), _log(rng, 4, 64), _log(rng, 1, 28)
            H, S, D = rng.choice([2, 4, 8]), _log(rng, 60, 4000), rng.choice([64, 128])
            if B * N * layers * 2 * H * S * D * 2 <= 7.4e9:
                break
        T = 4 * _log(rng, 8, 512)
        return dict(kind="reorder", B=B, N=N, layers=layers, H=H, S=S, D=D, valid=rng.randint(max(1, S // 2), S), T=T,
                    t=rng.randint(1, T), share=rng.choice([1.0, 1.0, 0.3]))
    if kind == "attention":
        while True:
            B, N, H, S, D = _log(rng, 1, 64), _log(rng, 4, 64), rng.choice([2, 4, 8]), _log(rng, 60, 4000), rng.choice([64, 128])
            if B * N * H * S * D * 4 <= 2.2e9:
                break
        return dict(kind="attention", B=B, N=N, H=H, G=rng.choice([1, 4, 7, 8]), S=S, D=D,
                    length=rng.randint(max(1, S // 3), S), page=rng.choice([0, 0, 16, 16, 24]))
    while True:
        B, N, V, layers = _log(rng, 1, 16), _log(rng, 4, 64), _log(rng, 1000, 152064), rng.choice([1, 2, 4])
        if B * N <= 128 and B * N * V <= 2e7:
            break
    dtype = rng.choice(["bf16", "f32"])
    tokens = rng.randint(8, 24)
    len0 = _log(rng, 20, 700)
    return dict(kind="generate", B=B, N=N, V=V, dtype=dtype, values="gauss_boost", alpha=4.0, ramp=rng.choice([0, 8]),
                kappa=0.5, layers=layers, H=rng.choice([2, 4]), G=rng.choice([2, 7]), S=len0 + tokens + rng.randint(0, 200),
                D=rng.choice([64, 128]), page=rng.choice([0, 16, 16]), len0=len0, tokens=tokens, eos=rng.random() < 0.3)


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _logits(c, seed, salt=0):
    """[R, V] logits as the head gives them; rows start 16 bytes apart, so a ragged vocabulary leaves a gap."""
    R, V = c["B"] * c["N"], c["V"]
    per = 8 if c["dtype"] == "bf16" else 4
    stride = (V + per - 1) // per * per
    out = torch.empty((R, stride), device=DEV, dtype=torch.bfloat16 if c["dtype"] == "bf16" else torch.float32)
    g = _gen(seed, salt)
    for lo in range(0, R, 512):
        n = min(512, R - lo)
        x = torch.randn((n, stride), generator=g, device=DEV)
        if c["values"] == "gauss":
            x *= 2.0
        elif c["values"] == "gauss_boost":                  # 20 plausible continuations over a Gaussian floor
            x *= 3.0
            at = torch.randint(0, V, (n, min(20, V)), generator=g, device=DEV)
            x.scatter_add_(1, at, torch.full(at.shape, 8.0, device=DEV))
        else:                                               # Student-t, three degrees of freedom
            chi2 = sum(torch.randn((n, stride), generator=g, device=DEV).square_() for _ in range(3))
            x *= torch.rsqrt(chi2 / 3.0) * 3.0
        if c.get("masked"):                                 # ids a grammar does not allow
            x.masked_fill_(torch.rand((n, stride), generator=g, device=DEV) < 0.2, -math.inf)
        out[lo:lo + n] = x.to(out.dtype)
    return out


def _done_rows(c):
    r = np.arange(c["B"] * c["N"])
    return (r % 5 == 4).astype(np.int32) if c.get("eos") else np.zeros(r.size, np.int32)


def _ancestors(c, seed):
    """Sorted draws from a moderately degenerate weight vector per prompt, and which prompts resample."""
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 777])
    B, N = c["B"], c["N"]
    anc = np.arange(B * N, dtype=np.int32)
    flag = (rng.random(B) < c.get("share", 1.0)).astype(np.int32)
    flag[rng.integers(0, B)] = 1
    for b in range(B):
        p = rng.dirichlet(np.full(N, 0.5))
        d = b * N + np.sort(rng.choice(N, size=N, p=p))
        if flag[b]:
            anc[b * N:(b + 1) * N] = d
    return anc, flag


def _normal(shape, g):
    return torch.empty(shape, device=DEV, dtype=torch.bfloat16).normal_(generator=g)


class _Context:
    """A context over buffers the caller keeps (what a program that drives the C interface itself holds)."""

    def __init__(self, cfg):
        self.cfg = cfg
        self.bytes = smc.smc_workspace_bytes(cfg)
        self.memory = torch.empty(self.bytes + 256, dtype=torch.uint8, device=DEV)
        self.ctx = None

    def open(self):
        at = (self.memory.data_ptr() + 255) & ~255
        self.ctx = smc.smc_init(self.cfg, at, self.bytes, torch.cuda.current_stream().cuda_stream)
        return self.ctx

    def close(self):
        if self.ctx is not None:
            smc.smc_destroy(self.ctx)
            self.ctx = None

    def __del__(self):
        self.close()


def prepare(case, seed):
    return {"step": _prepare_step, "weights": _prepare_weights, "reorder": _prepare_reorder,
            "attention": _prepare_attention, "generate": _prepare_generate}[case["kind"]](dict(case), int(seed))


def run(state):
    return {"step": _run_step, "weights": _run_weights, "reorder": _run_reorder, "attention": _run_attention,
            "generate": _run_generate}[state["c"]["kind"]](state)


# ---- a step over the vocabulary ---------------------------------------------------------------------------------------
def _prepare_step(c, seed):
    R = c["B"] * c["N"]
    eos = 3 if c["eos"] else -1
    st = {"c": c, "t": 0, "x": _logits(c, seed)}
    if c["call"] == "noalloc":
        st["cfg"] = smc.make_config(c["B"], c["N"], c["V"], c["T"], c["dtype"], c["kappa"], seed, eos_id=eos)
        st["logW"] = torch.zeros(R, dtype=torch.float64, device=DEV)
        st["cumlogp"] = torch.zeros(R, dtype=torch.float64, device=DEV)
        st["done"] = torch.as_tensor(_done_rows(c)).to(DEV)
        st["tokens"] = torch.zeros(R, dtype=torch.int32, device=DEV)
        return st
    s = st["s"] = Session(c["B"], c["N"], c["V"], c["T"], c["dtype"], c["kappa"], seed, eos_id=eos)
    if c["eos"]:
        s.set_done(_done_rows(c))
    return st


def _run_step(st):
    c = st["c"]
    t = st["t"] = st["t"] % c["T"] + 1
    if c["call"] == "noalloc":
        smc.smc_step_noalloc(st["cfg"], torch.cuda.current_stream().cuda_stream, st["x"], st["x"].stride(0), t, c["alpha"],
                             c["alpha_prev"], c["tau"], st["logW"], st["cumlogp"], st["done"], st["tokens"])
        return {k: st[k] for k in ("tokens", "logW", "cumlogp", "done")}
    s = st["s"]
    if c["call"] == "full":
        s.step_resample_reindex(st["x"], t, c["alpha"], c["alpha_prev"], 0, c["tau"])
    else:
        s.step_resample(st["x"], t, c["alpha"], c["alpha_prev"], c["tau"])
    return {"tokens": s.tokens, "anc": s.anc, "resampled": s.resampled, "ess": s.ess, "histA": s.histA, "histB": s.histB}


# ---- weights --------------------------------------------------------------------------------------------------------
def _prepare_weights(c, seed):
    R = c["B"] * c["N"]
    s = Session(c["B"], c["N"], 8, 8, "f32", c["kappa"], seed, with_hist=False)
    smc.smc_set_resampler(s.ctx, c["scheme"])
    smc.smc_set_ancestor_order(s.ctx, c["order"])
    w = torch.randn(R, generator=_gen(seed, 5), device=DEV, dtype=torch.float64) * c["spread"]
    return {"c": c, "s": s, "t": 0, "from": w, "logW": torch.empty_like(w)}


def _run_weights(st):
    s = st["s"]
    t = st["t"] = st["t"] % 8 + 1
    st["logW"].copy_(st["from"])                            # the call resets the weights of prompts that resample
    smc.smc_ess_from(s.ctx, st["logW"], s.ess, s.lognormw)
    smc.smc_resample_from(s.ctx, st["logW"], t, s.anc, s.resampled, None)
    return {"ess": s.ess, "lognormw": s.lognormw, "anc": s.anc, "resampled": s.resampled, "logW": st["logW"]}


# ---- the dense reorder ------------------------------------------------------------------------------------------------
def _prepare_reorder(c, seed):
    R, n = c["B"] * c["N"], c["layers"]
    st = {"c": c}
    cfg = smc.make_config(c["B"], c["N"], 8, c["T"], "bf16", 0.5, seed, 2 * n, c["H"], c["S"], c["D"], 2)
    st["context"] = _Context(cfg)
    ctx = st["context"].open()
    g = _gen(seed, 9)
    shape = (n, R, c["H"], c["S"], c["D"])
    st["kA"], st["vA"] = _normal(shape, g), _normal(shape, g)
    st["kB"], st["vB"] = (torch.zeros(shape, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    st["histA"] = torch.randint(0, 1000, (R, c["T"]), generator=g, device=DEV, dtype=torch.int32)
    st["histB"] = torch.zeros_like(st["histA"])
    pairs = [t for i in range(n) for t in (st["kA"][i], st["vA"][i])], [t for i in range(n) for t in (st["kB"][i], st["vB"][i])]
    smc.smc_kv_bind(ctx, pairs[0], pairs[1], st["histA"], st["histB"])
    anc, flag = _ancestors(c, seed)
    st["anc"], st["flag"] = torch.as_tensor(anc).to(DEV), torch.as_tensor(flag).to(DEV)
    return st


def _run_reorder(st):
    smc.smc_kv_reindex(st["context"].ctx, st["anc"], st["flag"], st["c"]["valid"], st["c"]["t"])
    return {k: st[k] for k in ("kA", "vA", "kB", "vB", "histA", "histB")}


# ---- attention --------------------------------------------------------------------------------------------------------
def _attention_inputs(c, seed):
    """Keys and values per row (dense) or per page, and the queries."""
    R, g = c["B"] * c["N"], _gen(seed, 21)
    if c["page"]:
        pages = R * ((c["S"] + c["page"] - 1) // c["page"])
        shape = (pages, c["H"], c["page"], c["D"])
    else:
        shape = (R, c["H"], c["S"], c["D"])
    return _normal(shape, g), _normal(shape, g), _normal((R, c["H"] * c["G"], c["D"]), g)


def _prepare_attention(c, seed):
    k, v, q = _attention_inputs(c, seed)
    anc, flag = _ancestors(c, seed)
    anc, flag = torch.as_tensor(anc).to(DEV), torch.as_tensor(flag).to(DEV)
    if c["page"]:
        s = Session(c["B"], c["N"], 8, 8, "bf16", 0.5, seed, kv_geom=(2, c["H"], c["S"], c["D"]), with_hist=False,
                    page_len=c["page"], len0=c["length"])
        s.pools[0].copy_(k)
        s.pools[1].copy_(v)
        s.paged_reindex(0, anc, flag)                       # descendants share their ancestor's pages
    else:
        s = Session(c["B"], c["N"], 8, 8, "bf16", 0.5, seed, kv=[k, v], with_hist=False)
        s.reindex(c["length"], 0, anc, flag)                # some rows live in the second buffer
    return {"c": c, "s": s, "q": q}


def _run_attention(st):
    c = st["c"]
    return st["s"].attention(0, 1, st["q"], c["length"], c["D"] ** -0.5)


# ---- a whole generation -----------------------------------------------------------------------------------------------
def _prepare_generate(c, seed):
    R, n = c["B"] * c["N"], c["layers"]
    st = {"c": c}
    T = (c["tokens"] + 3) // 4 * 4
    cfg = smc.make_config(c["B"], c["N"], c["V"], T, c["dtype"], c["kappa"], seed, 2 * n, c["H"], c["S"], c["D"], 2,
                          eos_id=3 if c["eos"] else -1)
    st["context"] = _Context(cfg)
    g = _gen(seed, 31)
    st["x"] = [_logits(c, seed, 100 + i) for i in range(4)]
    st["new"] = _normal((4, n, 2, R, c["H"], c["D"]), g)    # keys and values of a new position, per layer
    st["q"] = _normal((4, n, R, c["H"] * c["G"], c["D"]), g)
    i32 = dict(dtype=torch.int32, device=DEV)
    st["histA"], st["histB"] = torch.zeros((R, T), **i32), torch.zeros((R, T), **i32)
    st["tokens"], st["anc"], st["slot"] = (torch.zeros(R, **i32) for _ in range(3))
    st["resampled"], st["choice"] = (torch.zeros(c["B"], **i32) for _ in range(2))
    st["ess"] = torch.zeros(c["B"], dtype=torch.float64, device=DEV)
    st["out"] = torch.zeros((n, R, c["H"] * c["G"], c["D"]), device=DEV)
    st["awork_bytes"] = smc.smc_attn_workspace_bytes(cfg, c["H"] * c["G"])
    st["awork"] = torch.empty(st["awork_bytes"], dtype=torch.uint8, device=DEV)
    if c["page"]:
        pages = R * ((c["S"] + c["page"] - 1) // c["page"])
        st["pools"] = [_normal((pages, c["H"], c["page"], c["D"]), g) for _ in range(2 * n)]
        st["paged_bytes"] = smc.smc_paged_workspace_bytes(cfg, c["page"])
        st["paged"] = torch.empty(st["paged_bytes"] + 256, dtype=torch.uint8, device=DEV)
    else:
        st["kvA"] = [_normal((R, c["H"], c["S"], c["D"]), g) for _ in range(2 * n)]
        st["kvB"] = [torch.zeros_like(t) for t in st["kvA"]]
    return st


def _alpha(c, t):
    return c["alpha"] if c["ramp"] <= 0 else 1.0 + (c["alpha"] - 1.0) * min(t, c["ramp"]) / c["ramp"]


def _run_generate(st):
    c, R = st["c"], st["c"]["B"] * st["c"]["N"]
    ctx = st["context"].open()
    paged, row, Hq, scale = c["page"] > 0, c["H"] * c["D"], c["H"] * c["G"], c["D"] ** -0.5
    if paged:
        smc.smc_kv_bind(ctx, [], [], st["histA"], st["histB"])
        smc.smc_paged_bind(ctx, st["pools"], c["page"], (st["paged"].data_ptr() + 255) & ~255, st["paged_bytes"], c["len0"])
        smc.smc_paged_prepare_append(ctx, c["len0"], st["slot"])
    else:
        smc.smc_kv_bind(ctx, st["kvA"], st["kvB"], st["histA"], st["histB"])
    for i in range(c["tokens"]):
        pos, t, j = c["len0"] + i, i + 1, i % 4
        for l in range(c["layers"]):
            smc.smc_kv_append(ctx, 2 * l, 2 * l + 1, st["new"][j, l, 0], row, st["new"][j, l, 1], row, pos)
            smc.smc_attn_decode(ctx, 2 * l, 2 * l + 1, st["q"][j, l], Hq, pos + 1, scale, st["awork"], st["awork_bytes"],
                                st["out"][l])
        x = st["x"][j]
        a, before = _alpha(c, t), _alpha(c, t - 1)
        if paged:
            smc.smc_step_resample(ctx, x, x.stride(0), t, a, before, -1.0, st["tokens"], st["anc"], st["resampled"], st["ess"])
            if i + 1 < c["tokens"]:
                smc.smc_paged_reindex_prepare(ctx, st["anc"], st["resampled"], t, pos + 1, st["slot"])
            else:
                smc.smc_paged_reindex(ctx, st["anc"], st["resampled"], t)
        else:
            smc.smc_step_resample_reindex(ctx, x, x.stride(0), t, a, before, -1.0, pos + 1, st["tokens"], st["anc"],
                                          st["resampled"], st["ess"])
    smc.smc_final_draw(ctx, c["tokens"], st["choice"])
    logW, cum = np.empty(R), np.empty(R)
    smc.smc_get_state(ctx, logW, cum)
    st["context"].close()
    out = {k: st[k] for k in ("histA", "histB", "choice", "ess", "slot", "out")}
    out["logW"], out["cumlogp"] = logW, cum
    out["cache"] = st["pools"] if paged else st["kvA"] + st["kvB"]
    return out


# ---- what a pass cannot do without --------------------------------------------------------------------------------------
def work(case):
    c = case
    R = c["B"] * c["N"]
    if c["kind"] == "step":
        live = R - int(_done_rows(c).sum())
        return {"bytes": live * c["V"] * (2 if c["dtype"] == "bf16" else 4) + 40 * R, "flops": 6 * live * c["V"]}
    if c["kind"] == "weights":
        return {"bytes": 28 * R + 12 * c["B"], "flops": 40 * R}
    if c["kind"] == "reorder":
        anc, _ = _ancestors(c, 1)
        moved = np.nonzero(anc != np.arange(R))[0]
        rows = len(moved) + len(set(anc[moved].tolist()))
        return {"bytes": rows * (2 * c["layers"] * c["H"] * c["valid"] * c["D"] * 2 + 4 * c["t"]) + 8 * R, "flops": 0}
    if c["kind"] == "attention":
        return _attention_work(R, c, c["length"])
    per = [_attention_work(R, c, c["len0"] + i + 1) for i in range(c["tokens"])]
    logits = R * c["V"] * (2 if c["dtype"] == "bf16" else 4)
    append = 2 * c["layers"] * R * c["H"] * c["D"] * 4
    return {"bytes": c["tokens"] * (logits + append) + c["layers"] * sum(p["bytes"] for p in per),
            "flops": c["tokens"] * 6 * R * c["V"] + c["layers"] * sum(p["flops"] for p in per)}


def _attention_work(R, c, length):
    Hq = c["H"] * c["G"]
    return {"bytes": R * (2 * c["H"] * length * c["D"] * 2 + Hq * c["D"] * 6), "flops": 4 * R * Hq * length * c["D"]}


def tolerance(case):
    """Moved bytes are the same bytes.  Log weights and what follows from them are 32-bit sums over the vocabulary
    (measured 2e-7 off the 64-bit value), the weight arithmetic itself is 64-bit (2e-15), attention carries its weights in
    two 16-bit parts (4e-6); each about four times that, for other sizes and values.  A draw may differ where two keys tie
    in 32 bits."""
    k = case["kind"]
    if k == "reorder":
        return "exact"
    if k == "weights":
        return {"rel": 1e-13, "max": 1e-11, "differ": 1e-3}
    if k == "attention":
        return {"rel": 2e-5, "max": 2e-4}
    if k == "generate":
        return {"rel": 2e-5, "max": 2e-4, "differ": 1e-3}
    return {"rel": 1e-6, "max": 4e-5, "differ": 1e-3}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors that hold 32-bit words; the four output words."""
    mask = 0xFFFFFFFF
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57             # wraps modulo 2^64, the bits are what counts
        c0, c1, c2, c3 = (((b >> 32) & mask) ^ c1 ^ k0, b & mask, ((a >> 32) & mask) ^ c3 ^ k1, a & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _gumbel(rows, V, step, seed):
    blocks = (V + 3) // 4
    c0 = torch.arange(blocks, device=DEV, dtype=torch.int64).expand(rows.numel(), blocks)
    c1 = rows[:, None].expand_as(c0)
    zero = torch.zeros_like(c0)
    w = torch.stack(_philox(c0, c1, zero + step, zero, seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF), dim=2)
    w = w.reshape(rows.numel(), 4 * blocks)[:, :V]
    low = w < 0x80000000
    e = torch.where(low, -torch.log((w.double() + 0.5) * 2.0 ** -32), -torch.log1p(-(((0xFFFFFFFF - w).double() + 0.5) * 2.0 ** -32)))
    return -torch.log(e)


def _exact_step(c, seed):
    R, V = c["B"] * c["N"], c["V"]
    x = _logits(c, seed)
    beta = c["alpha"] if c["tau"] <= 0 else 1.0 / c["tau"]
    delta = torch.zeros(R, dtype=torch.float64, device=DEV)
    logp = torch.zeros_like(delta)
    done = torch.as_tensor(_done_rows(c)).to(DEV) != 0
    chunk = max(1, min(R, int(2e7) // V + 1))
    for lo in range(0, R, chunk):
        rows = torch.arange(lo, min(R, lo + chunk), device=DEV)
        l = x[rows, :V].double()
        z1, zb = torch.logsumexp(l, 1), torch.logsumexp(beta * l, 1)
        y = (beta * l + _gumbel(rows, V, 1, seed)).argmax(1)
        ly = l.gather(1, y[:, None])[:, 0]
        logp[rows] = ly - z1
        delta[rows] = c["alpha"] * (ly - z1) - (beta * ly - zb)
    delta.masked_fill_(done, 0.0)
    logp.masked_fill_(done, 0.0)
    if c["call"] == "noalloc":
        return {"tokens": None, "logW": delta, "cumlogp": logp, "done": None}
    w = delta.view(c["B"], c["N"])
    ess = torch.exp(2.0 * torch.logsumexp(w, 1) - torch.logsumexp(2.0 * w, 1))
    return {"tokens": None, "anc": None, "resampled": None, "ess": ess, "histA": None, "histB": None}


def _exact_attention(c, seed):
    k, v, q = _attention_inputs(c, seed)
    anc, _ = _ancestors(c, seed)
    R, H, G, D, n = c["B"] * c["N"], c["H"], c["G"], c["D"], c["length"]
    out = torch.empty((R, H * G, D), dtype=torch.float64, device=DEV)
    j = torch.arange(n, device=DEV)
    for r in range(R):
        a = int(anc[r])
        if c["page"]:                                       # page j of row i of prompt b is number b*Q + j*N + i
            b, i = divmod(a, c["N"])
            page = b * c["N"] * ((c["S"] + c["page"] - 1) // c["page"]) + j // c["page"] * c["N"] + i
            kr, vr = (t[page, :, j % c["page"]].transpose(0, 1).double() for t in (k, v))
        else:
            kr, vr = k[a, :, :n].double(), v[a, :, :n].double()
        qr = q[r].double().view(H, G, 1, D)
        p = torch.softmax((qr * kr[:, None]).sum(-1) * D ** -0.5, -1)
        out[r] = (p[..., None] * vr[:, None]).sum(2).view(H * G, D)
    return out


def exact(case, seed):
    if case["kind"] == "step":
        return _exact_step(case, int(seed))
    if case["kind"] == "attention":
        return _exact_attention(case, int(seed))
    if case["kind"] == "weights":
        w = (torch.randn(case["B"] * case["N"], generator=_gen(seed, 5), device=DEV, dtype=torch.float64)
             * case["spread"]).view(case["B"], case["N"])
        l1, l2 = torch.logsumexp(w, 1), torch.logsumexp(2.0 * w, 1)
        ess = torch.exp(2.0 * l1 - l2)
        after = torch.where((ess < case["kappa"] * case["N"])[:, None], torch.zeros_like(w), w)
        return {"ess": ess, "lognormw": (w - l1[:, None]).reshape(-1), "anc": None, "resampled": None, "logW": after.reshape(-1)}
    return None
