"""hdg_asm_setup on seeded random element blocks at the edges where its kernels change path: rows filled by 16,
32 or 64 lanes (fewer than 16, 32 or more unknowns), the factorisations by size, and above 192 unknowns the
inverse taken from the solve. Against numpy's inverse of the enriched element blocks (diagonal blocks those
of the assembled matrix). The blocks are 4 I plus entries below 2/n: condition below 3, and an inverse of n
unknowns is accurate to about 10 n eps: 6e-13 at 285; 1e-11."""
import numpy as np
import pytest
import torch

from test_gpu_parity import relerr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,L", [(1, 3), (5, 3), (4, 4), (31, 2), (10, 3), (8, 4), (13, 5), (48, 4), (57, 5)])
def test_inverses_match_numpy(nb, L):
    from paper_2512_13619_amd import hdg
    rng = np.random.default_rng([nb, L])
    ne, nt, S = 3, nb * L, 2 * L - 1
    nf = ne * L
    e2f = rng.permutation(nf).astype(np.int32).reshape(ne, L)
    Kbar = rng.uniform(-1, 1, (ne, nt, nt)) / nt
    K = rng.uniform(-1, 1, (nf, S, nb, nb)) / nt
    K[:, 0] += 4 * np.eye(nb)
    d = dict(ne=ne, nf=nf, ncomp=1, dim=3, npe=3, npf=nb, nlfe=L)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    inv = torch.full((ne * nt * nt,), float("nan"), dtype=torch.float64, device="cuda")
    inv32 = torch.full((ne * nt * nt,), float("nan"), dtype=torch.float32, device="cuda")
    hdg.Context(0).asm_setup(d, dev(Kbar), dev(K), dev(e2f), inv, inv32)
    got = inv.cpu().numpy().reshape(ne, L, L, nb, nb)          # [e][l][l'][col][row]
    for e in range(ne):
        P = Kbar[e].copy()
        for l in range(L):
            P[l * nb:(l + 1) * nb, l * nb:(l + 1) * nb] = K[e2f[e, l], 0].T
        err = relerr(got[e].transpose(0, 3, 1, 2).reshape(nt, nt), np.linalg.inv(P))
        say("asm shapes", nb, L, e, err)
        assert err < 1e-11
    assert torch.equal(inv32, inv.float())
