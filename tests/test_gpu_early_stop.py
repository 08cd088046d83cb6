"""The host stops enqueueing a restart cycle once the device has reported it done. With use_graph the
whole cycle is captured and replayed instead, by the same kernels: iterations, residual history and
solution agree bit for bit, wherever the cycle ends: within the first steps, at its last step, in the
middle, in the partial cycle that a step budget leaves after replays (enqueued directly), and not at all."""
import numpy as np
import pytest
import torch

from test_gpu_batch_solve import system
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def case(seed, diag):
    """A system above the size that one workgroup takes; diag sets how many steps it needs."""
    nb, L, nf = 4, 4, 700
    rng = np.random.default_rng(seed)
    K, nbr, _ = system(rng, nb, L, nf)
    K[:, 0] += (diag - 4) * np.eye(nb)
    K64 = torch.as_tensor(np.nan_to_num(K)).cuda()
    d = dict(ne=2, nf=nf, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L)
    return d, K64, torch.as_tensor(nbr).cuda(), torch.as_tensor(rng.standard_normal(nf * nb)).cuda()


@pytest.mark.parametrize("orth", ["cgs2", "dcgs2", "cgs", "mgs"])
@pytest.mark.parametrize("prec", ["bj", "none", "bj_poly"])
def test_early_stop_equals_whole_cycles(orth, prec):
    from paper_2512_13619_amd import hdg
    ctx = hdg.Context(0)

    def solve(data, **kw):
        d, K, nbr, b = data
        x = torch.zeros_like(b)
        st = ctx.gmres_solve(d, K, None, nbr, b, x, orth=orth, prec=prec, poly_degree=4, poly_v0=b, hist_len=600, **kw)
        return st, x

    easy, hard = case(41, 3.0), case(43, 0.14)
    n = solve(easy, rtol=1e-10, restart=30)[0]["iters"]
    m = solve(hard, rtol=1e-10, restart=60, max_iters=400)[0]["iters"]
    say("early stop", orth, prec, n, m)
    assert 1 < n <= 12 < m
    runs = [(easy, dict(rtol=1e-2, restart=30)), (easy, dict(rtol=1e-10, restart=n)), (easy, dict(rtol=1e-10, restart=50)),
            (hard, dict(rtol=1e-10, restart=7, max_iters=400)), (hard, dict(rtol=1e-15, restart=7, max_iters=17)),
            (hard, dict(rtol=1e-10, restart=60, max_iters=400, time_phases=True))]
    for data, kw in runs:
        a, xa = solve(data, **kw)
        b, xb = solve(data, **dict(kw, use_graph=True, time_phases=False))
        assert (a["iters"], a["cycles"], a["status"]) == (b["iters"], b["cycles"], b["status"]), (kw, a["iters"], b["iters"])
        assert np.array_equal(a["hist"], b["hist"]) and torch.equal(xa, xb), kw
        if kw.get("time_phases"):
            assert a["iters"] <= a["n_timed"] <= a["iters"] + a["cycles"]
