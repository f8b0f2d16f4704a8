"""The per-prompt weight kernels at the sizes where their teams change (one wave / a workgroup), where the padded rows of the
serial sums end, and where the descendants' bit set takes a second word, against the CPU oracle: ancestors, flags and moved
state bit for bit, ESS to 1e-9 N as elsewhere."""
import numpy as np
import pytest
import torch

from oracle import reference as orc
from paper_2602_10273_amd import binding as smc
from paper_2602_10273_amd.harness import Session

pytestmark = pytest.mark.gpu
SIZES = (1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 200, 511, 513, 1023, 1024)


@pytest.mark.parametrize("scheme", ["systematic", "stratified", "multinomial", "residual"])
@pytest.mark.parametrize("order", [0, 1])
def test_resampling_at_the_edges_of_the_teams(scheme, order):
    rng = np.random.default_rng(11)
    for N in SIZES:
        B = 3
        s = Session(B, N, 64, 8, "f32", 1.0, seed=91, with_hist=False)
        smc.smc_set_resampler(s.ctx, orc.SCHEMES[scheme])
        smc.smc_set_ancestor_order(s.ctx, order)
        logW = rng.standard_normal(B * N) * 1.5
        logW[:N] = rng.standard_normal(N) * 8.0
        if N > 2:
            logW[N:N + N // 2] = -np.inf                        # half of a prompt without weight
        d = torch.as_tensor(logW).cuda()
        smc.smc_ess_from(s.ctx, d, s.ess, s.lognormw)
        e_ref, lnw_ref = orc.ess(logW, B, N)
        assert np.abs(s.ess.cpu().numpy() - e_ref).max() < 1e-9 * N, N
        fin = np.isfinite(lnw_ref)
        assert np.abs(s.lognormw.cpu().numpy()[fin] - lnw_ref[fin]).max() < 1e-12, N
        smc.smc_resample_from(s.ctx, d, 4, s.anc, s.resampled, s.ess)
        anc_ref, flag_ref, _, lw_ref = orc.resample(logW, B, N, 1.0, 91, 4, scheme, in_place=bool(order))
        assert np.array_equal(s.resampled.cpu().numpy(), flag_ref), N
        assert np.array_equal(s.anc.cpu().numpy(), anc_ref), N
        assert np.array_equal(d.cpu().numpy(), lw_ref), N
        s.set_state(logW=logW)
        s.final_draw(5)
        assert np.array_equal(s.choice.cpu().numpy(), orc.final_draw(logW, B, N, 91, 5)), N
        s.close()


@pytest.mark.parametrize("sorted_", [True, False])
def test_reorder_plan_at_the_edges_of_the_teams(sorted_):
    rng = np.random.default_rng(12)
    for N in SIZES:
        B, T = 3, 16
        s = Session(B, N, 64, T, "f32", 0.5, 0)
        o = orc.OracleSMC(B, N, 64, T, 0.5, 0, "f32")
        hist = rng.integers(0, 64, (B * N, T)).astype(np.int32)
        cum = rng.standard_normal(B * N)
        s.histA.copy_(torch.as_tensor(hist))
        s.set_state(np.zeros(B * N), cum)
        o.hist[:], o.cumlogp[:] = hist, cum
        for _ in range(3):
            anc = np.concatenate([b * N + (np.sort if sorted_ else np.asarray)(rng.integers(0, N, N)) for b in range(B)]).astype(np.int32)
            flag = np.array([1, 0, 1], np.int32)
            anc[N:2 * N] = np.arange(N, 2 * N)
            o.reindex(anc, flag, 0, T)
            s.reindex(0, T, torch.as_tensor(anc).cuda(), torch.as_tensor(flag).cuda())
            assert np.array_equal(s.live_hist(), o.hist), N
            assert np.array_equal(s.state()[1], o.cumlogp), N
        s.close()
