"""hdg_gmres_solve at the sizes where a whole restart cycle runs in one workgroup: up to 16 thread groups
a row, one, and two rows a thread; neighbour tables in LDS or not; restarts past 64 columns; and sizes
just past its limits, where the general path runs. Against scipy's sparse direct solve.

The systems are those of the batched test (4 I plus blocks of row sum below 1.5, condition number under
3), solved to 1e-12 in the residual: 1e-11 of the solution's largest entry."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
import torch

from test_gpu_batch_solve import system
from test_gpu_parity import relerr, say

pytestmark = pytest.mark.gpu

# block edge, faces of an element, faces
SIZES = [(1, 3, 1), (2, 4, 9), (3, 4, 85), (8, 4, 65), (5, 3, 204), (2, 4, 512), (1, 3, 1025), (1, 3, 2048), (1, 3, 2049),
         (12, 4, 60), (12, 4, 90)]


@pytest.mark.parametrize("kw", [dict(restart=50), dict(restart=3, use_graph=True), dict(restart=200, orth="cgs"),
                                dict(restart=30, prec="none"), dict(restart=20, precision="mixed", time_phases=True)],
                         ids=["cgs2", "short_graph", "cgs_200", "none", "mixed_timed"])
def test_small_solve_matches_direct(kw):
    from paper_2512_13619_amd import hdg
    rng = np.random.default_rng(23)
    ctx = hdg.Context(0)
    for nb, L, nf in SIZES:
        K, nbr, A = system(rng, nb, L, nf)
        b = rng.standard_normal(nf * nb)
        want = spla.spsolve(A, b)
        d = dict(ne=2, nf=nf, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L)
        K64 = torch.as_tensor(K).cuda()
        x = torch.zeros(nf * nb, dtype=torch.float64, device="cuda")
        st = ctx.gmres_solve(d, K64, K64.float(), torch.as_tensor(nbr).cuda(), torch.as_tensor(b).cuda(), x, rtol=1e-12,
                             max_iters=600, hist_len=700, **kw)
        err = relerr(x.cpu().numpy(), want)
        say("small solve", kw, (nb, L, nf), st["iters"], st["cycles"], err)
        assert st["converged"] and err < 1e-11, (nb, L, nf, st["iters"], err)
        assert len(st["hist"]) == st["iters"] + st["cycles"] + 1
        assert st["n_timed"] == (st["iters"] if kw.get("time_phases") else 0)


def test_small_solve_budget_guess_and_nonfinite():
    """A step budget inside a cycle, a converged initial guess, and a NaN in the matrix."""
    from paper_2512_13619_amd import hdg
    rng = np.random.default_rng(29)
    nb, L, nf = 3, 4, 60
    K, nbr, A = system(rng, nb, L, nf)
    b = rng.standard_normal(nf * nb)
    d = dict(ne=2, nf=nf, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L)
    ctx = hdg.Context(0)
    K64, nd, bd = torch.as_tensor(K).cuda(), torch.as_tensor(nbr).cuda(), torch.as_tensor(b).cuda()
    x = torch.zeros(nf * nb, dtype=torch.float64, device="cuda")
    st = ctx.gmres_solve(d, K64, None, nd, bd, x, rtol=1e-14, max_iters=5)
    assert not st["converged"] and st["iters"] == 5
    x.copy_(torch.as_tensor(spla.spsolve(A, b)))
    st = ctx.gmres_solve(d, K64, None, nd, bd, x, rtol=1e-10)
    assert st["converged"] and st["iters"] == 0
    K64[7, 1, 0, 0] = float("nan")
    with pytest.raises(hdg.HdgError):
        ctx.gmres_solve(d, K64, None, nd, bd, x, rtol=1e-10)
