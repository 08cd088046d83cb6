"""hdg_gmres_solve_batch on seeded block systems at the sizes where its kernels change path: 8, 16
and 32 threads a face, faces with more entries than are loaded ahead, instances of one reduction
chunk and of more chunks than a wave adds at once, restarts past 64 columns, and the options
(CGS, no preconditioner, graph replay). Every instance against scipy's sparse direct solve.

The systems are 4 I plus blocks whose row sums stay below 1.5 (condition number under 3), solved to
1e-12 in the residual: the solutions agree to 1e-11 of their largest entry. Empty slots hold NaN:
they are never used."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla
import torch

from test_gpu_parity import relerr, say

pytestmark = pytest.mark.gpu

# npf (the block edge, one component), nlfe, faces
INSTANCES = [(1, 3, 7), (2, 4, 33), (3, 4, 11003), (4, 3, 129), (5, 4, 300), (5, 3, 64), (8, 4, 65), (7, 4, 40)]


def system(rng, nb, L, nf):
    S = 2 * L - 1
    nbr = np.full((nf, S), -1, np.int32)
    nbr[:, 0] = np.arange(nf)
    for s in range(1, S):
        nbr[:, s] = (np.arange(nf) + s * s) % nf
    K = rng.uniform(-1, 1, (nf, S, nb, nb)) / (S * nb)
    K[:, 0] += 4 * np.eye(nb)
    edge = rng.uniform(size=nf) < 0.3              # boundary faces: one element's slots only
    nbr[edge, L:] = -1
    rows, cols, vals = [], [], []
    for s in range(S):
        f = np.nonzero(nbr[:, s] >= 0)[0]
        r, c = np.meshgrid(np.arange(nb), np.arange(nb), indexing="ij")
        rows.append((f[:, None, None] * nb + r).ravel())
        cols.append((nbr[f, s][:, None, None] * nb + c).ravel())
        vals.append(K[f, s].transpose(0, 2, 1).ravel())      # K is column-major
    A = sp.csc_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols))), shape=(nf * nb, nf * nb))
    K[edge, L:] = np.nan
    return K, nbr, A


@pytest.mark.parametrize("kw", [dict(restart=30), dict(restart=70, orth="cgs"), dict(restart=9, prec="none"),
                                dict(restart=30, precision="mixed"), dict(restart=12, use_graph=True)],
                         ids=["cgs2", "cgs_70", "none", "mixed", "graph"])
def test_batch_solve_matches_direct(kw):
    from paper_2512_13619_amd import hdg
    rng = np.random.default_rng(17)
    ctx = hdg.Context(0)
    dims = [dict(ne=2, nf=nf, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L) for nb, L, nf in INSTANCES]
    bt = hdg.Batch(ctx, dims)
    K, nbr, r, ref = [], [], [], []
    for nb, L, nf in INSTANCES:
        k, n, A = system(rng, nb, L, nf)
        b = rng.standard_normal(nf * nb)
        K.append(k.ravel()), nbr.append(n.ravel()), r.append(b), ref.append(spla.spsolve(A, b))
    dev = lambda v: torch.as_tensor(np.concatenate(v)).cuda()
    K64 = dev(K)
    x = torch.zeros(bt.total("vec"), dtype=torch.float64, device="cuda")
    for again in range(2):
        x.zero_()
        st, stats = bt.gmres_solve(K64, K64.float(), dev(nbr), dev(r), x, max_iters=400, rtol=1e-12, **kw)
        torch.cuda.synchronize()
        assert st == 0, stats
    off = bt.offsets("vec")
    for i, want in enumerate(ref):
        err = relerr(x[off[i]:off[i + 1]].cpu().numpy(), want)
        say("batch solve", kw, INSTANCES[i], stats[i]["iters"], err)
        assert err < 1e-11, (INSTANCES[i], err)
