"""hdg_condense_batch and hdg_recover_batch on seeded random element blocks with one, two and three
components in one, two and three dimensions, mixed in one batch: products with W by 16x16 tiles with every remainder
(where large elements have most of the work) and by entries, fewer and more than threads (where small ones
have), and row interchanges at every pivot (E is near a scaled permutation). Against the oracle's dense solve of the whole local system.

Every entry is a sum of at most 150 products with O(1) data and an elimination of at most 48 unknowns with a
condition number below 10: rounding below 150 * 48 * 10 eps / 10 = 2e-12 of the array's largest entry; 1e-11."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import relerr, say

pytestmark = pytest.mark.gpu

# D, M, P, PF, L
SHAPES = [(1, 1, 3, 1, 2), (1, 4, 4, 1, 2), (1, 8, 5, 1, 2), (2, 1, 4, 2, 4), (2, 1, 9, 3, 4), (2, 1, 16, 4, 4),
          (2, 1, 25, 5, 4), (2, 2, 6, 3, 3), (2, 3, 4, 2, 4), (2, 2, 9, 3, 4), (2, 3, 16, 2, 4), (3, 1, 8, 4, 5), (3, 2, 4, 3, 4),
          (3, 1, 17, 8, 4)]


@pytest.mark.parametrize("small,large", [(3, 3), (300, 1), (2, 0)])
def test_random_blocks_match_oracle(small, large):
    """small, large: elements of each shape of up to 24 rows, and of each larger one"""
    from paper_2512_13619_amd import hdg
    ctx = hdg.Context(0)
    rng = np.random.default_rng(small)
    dims, blks, shapes = [], [], []
    for D, M, P, PF, L in SHAPES:
        ne = small if M * P + L * M * PF <= 24 else large
        if ne == 0:
            continue
        shapes.append((D, M, P, PF, L))
        nu, nq, nt = M * P, M * D * P, L * M * PF
        r = lambda *s: rng.uniform(-1, 1, (ne,) + s) / 4
        b = dict(Minv=np.eye(P) + r(P, P) / P, Bd=r(D, P, P), Cd=r(D, P, L * PF), D=r(nu, nq) / nq, E=r(nu, nu) / nu, F=r(nu, nt),
                 G=r(nt, nq) / nq, H=r(nt, nu), J=r(nt, nt), ru=r(nu), rt=r(nt))
        b["E"] += 2 * np.eye(nu)[rng.permutation(nu)]
        blks.append(b)
        dims.append(dict(ne=ne, nf=ne * L, ncomp=M, dim=D, npe=P, npf=PF, nlfe=L))
    bt = hdg.Batch(ctx, dims)
    dev = lambda name: torch.as_tensor(np.concatenate([b[name].ravel() for b in blks])).cuda()
    blk = {k: dev(k) for k in blks[0]}
    z = lambda k: torch.full((bt.total(k),), float("nan"), dtype=torch.float64, device="cuda")
    Kbar, rbar, local, du, dq = (z(k) for k in ("Kbar", "rbar", "local", "du", "dq"))
    bt.condense(blk, Kbar, rbar, local)
    e2fs = [rng.permutation(d["nf"]).astype(np.int32).reshape(d["ne"], -1) for d in dims]
    xs = [rng.standard_normal(d["nf"] * d["ncomp"] * d["npf"]) for d in dims]
    cat = lambda a: torch.as_tensor(np.concatenate([v.ravel() for v in a])).cuda()
    bt.recover(local, blk["Minv"], blk["Bd"], blk["Cd"], cat(e2fs), cat(xs), du, dq)
    for i, (d, b) in enumerate(zip(dims, blks)):
        Kb, rb = oracle.condense.condense(b, d)
        wq, wu = oracle.condense.recover(b, xs[i], e2fs[i], d)
        for k, t, want in (("Kbar", Kbar, Kb), ("rbar", rbar, rb), ("du", du, wu), ("dq", dq, wq)):
            o = bt.offsets(k)
            err = relerr(t[o[i]:o[i + 1]].cpu().numpy(), np.ravel(want))
            say("batch condense", shapes[i], k, err)
            assert err < 1e-11, (shapes[i], k, err)
