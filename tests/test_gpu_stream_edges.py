"""The vocabulary pass where its stream leaves the ordinary path: a maximum that rises by little or by far in the middle of a
batch, rows that begin masked, sums whose terms fall below the cut, slices that end inside a batch, flat rows that overflow
the ring -- against the CPU oracle, with the tolerances of the component tests."""
import numpy as np
import pytest

from paper_2602_10273_amd import synth
from tests.test_gpu_components import check_step

pytestmark = pytest.mark.gpu


def _rows(kind, R, V, rng):
    x = rng.standard_normal((R, V)).astype(np.float32)
    i = np.arange(V)
    if kind == "rising":                                    # a new maximum in every batch
        x += 0.002 * i
    elif kind == "stairs":                                  # jumps of 30 and of 300, at a place of its own in each row
        for r in range(R):
            at = np.sort(rng.integers(0, V, 3))
            x[r, at[0]:] += 30.0
            x[r, at[1]:] += 30.0
            x[r, at[2]:] += 300.0
    elif kind == "spike":                                   # one entry far above the rest, anywhere
        x[np.arange(R), rng.integers(0, V, R)] += 300.0
    elif kind == "masked_start":
        for r in range(R):
            x[r, :rng.integers(1, V - 1)] = -np.inf
    elif kind == "deep":                                    # the bulk lies beyond the cut of both sums
        x *= 20.0
    return x


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind", ["rising", "stairs", "spike", "masked_start", "deep", "flat"])
def test_running_maximum_and_cut(dtype, kind):
    rng = np.random.default_rng(len(kind))
    # (a fractional exponent times a large bf16 logit is beyond the fp32 constant beta*log2e: integers there)
    third, fourth = (8.0, 3.0) if kind in ("stairs", "spike", "deep") else (7.5, 40.0)
    for V, alpha, n_split, waves in ((40961, 4.0, 0, 0), (33000, 1.0, 1, 4), (70001, third, 3, 8), (8192, fourth, 0, 16)):
        w = synth.scaled(synth.WORKLOADS["cfg2"], B=2, N=3, V=V, dtype=dtype, S=16, layers=1)
        x = _rows(kind, w.R, V, rng)
        if kind == "flat":
            x *= 0.01
        x = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
        check_step(w, 5, 2, alpha, alpha, -1.0, n_split=n_split, wg_waves=waves, logits=x, stride_pad=(-V) % 8 + 8)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("waves", [4, 8, 16])
def test_slices_that_end_inside_a_batch(dtype, waves):
    """Slice lengths round one, two and three batches of the stream, and a last vector of every length."""
    per = 8 if dtype == "bf16" else 4
    batch = waves * 64 * 4 * per
    for V in [batch - per, batch - 1, batch, batch + 1, 2 * batch - 3, 2 * batch, 2 * batch + 64 * per + 1, 3 * batch + 5]:
        w = synth.scaled(synth.WORKLOADS["cfg2"], B=1, N=2, V=V, dtype=dtype, S=16, layers=1)
        check_step(w, V, 1, 4.0, 4.0, -1.0, n_split=1, wg_waves=waves, stride_pad=(-V) % per + per)
        check_step(w, V, 1, 2.5, 2.4, 0.8, n_split=2, wg_waves=waves, stride_pad=(-V) % per + per)


@pytest.mark.parametrize("B,N,V,dtype,eos,order,waves", [
    (1, 1, 4096, "f32", -1, 0, 0), (1, 4, 8, "f32", -1, 0, 0), (256, 1, 2056, "bf16", -1, 0, 0), (2, 128, 9000, "bf16", -1, 1, 0),
    (257, 1, 1000, "f32", 7, 0, 0), (2, 129, 4104, "bf16", 7, 0, 0), (1, 300, 3000, "f32", -1, 0, 0), (1, 1023, 1032, "bf16", -1, 1, 0),
    (1, 1024, 1032, "bf16", -1, 0, 0), (5, 8, 40000, "bf16", 3, 0, 8), (5, 8, 40000, "bf16", 3, 0, 4), (3, 40, 70000, "f32", -1, 0, 16)])
def test_one_call_equals_the_separate_calls_at_every_launch_shape(B, N, V, dtype, eos, order, waves):
    """Rows round the sizes where the launch shape changes, prompts of one row to a thousand: the step with resampling and
    plan folded in against smc_step, smc_resample and smc_kv_reindex, bit for bit, histories and cache included."""
    import torch
    from paper_2602_10273_amd import binding as smc
    from paper_2602_10273_amd.harness import Session
    kw = dict(kv_geom=(2, 1, 8, 16), eos_id=eos)
    one, sep = (Session(B, N, V, 8, dtype, 0.9, 5, **kw) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(N)
    for s in (one, sep):
        smc.smc_set_ancestor_order(s.ctx, order)
        smc.smc_set_tuning(s.ctx, 0, 0, waves)
    for a, b in zip(one.kvA, sep.kvA):
        a.normal_(generator=g)
        b.copy_(a)
    stride = (V + 7) // 8 * 8
    for t in range(1, 6):
        x = (torch.randn((B * N, stride), generator=g, device="cuda") * 3).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        one.step_resample_reindex(x, t, 2.0, 2.0, 5)
        sep.step(x, t, 2.0, 2.0)
        sep.resample(t)
        sep.reindex(5, t)
        for k in ("tokens", "anc", "resampled"):
            assert torch.equal(getattr(one, k), getattr(sep, k)), (t, k)
        assert torch.equal(one.ess.view(torch.int64), sep.ess.view(torch.int64)), t
        for a, b in zip(one.state(), sep.state()):
            assert np.array_equal(a, b), t
        assert np.array_equal(one.done(), sep.done())
        assert np.array_equal(one.live_hist(), sep.live_hist())
        assert np.array_equal(one.live_kv(1)[:, :, :5], sep.live_kv(1)[:, :, :5])
        assert np.allclose(one.log_Zhat(), sep.log_Zhat(), rtol=0, atol=1e-12)
    one.close()
    sep.close()
