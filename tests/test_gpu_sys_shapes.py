"""hdg_element_blocks_sys on seeded random geometry at the sizes where its kernels change path:
one or two tiles of basis functions (P <= 16 or not), remainders of the 16-entry tiles and of the
four-point steps, tables resident in LDS or staged in chunks, a face's values in LDS or read from
memory, an element shared by several blocks (small meshes) or not, and both phase orders.

The tables are rows of non-negative weights that sum to 1 (so states at the points stay physical)
and the inverse mass matrix is given (kept mass). Tolerance: every output is a sum of at most
about 1300 products of such weights with O(1) data, whose rounding is bounded by 1300 eps = 3e-13
of the sum of magnitudes; 1e-12 of the array's largest entry."""
import numpy as np
import pytest
import torch

import oracle.elements_sys as OS
from oracle.elements import mass_and_q_operators

from test_gpu_parity import relerr, say

pytestmark = pytest.mark.gpu

# M, P, PF, L, nqv, nqf, ne
SHAPES = {
    "one_tile_small": (5, 4, 3, 4, 5, 3, 1),
    "one_tile": (5, 10, 6, 4, 9, 7, 3),
    "tile_edge_16": (3, 16, 16, 6, 4, 4, 2),
    "tile_edge_17": (5, 17, 17, 4, 6, 5, 2),
    "three_tiles": (5, 33, 9, 4, 7, 6, 1),
    "staged_tables": (3, 64, 16, 6, 37, 9, 1),
    "face_from_memory": (3, 20, 10, 4, 2, 300, 1),
    "both_phase_orders": (3, 8, 4, 6, 8, 4, 600),
}


def weights(rng, *shape):
    w = rng.uniform(0.1, 1.0, shape)
    return w / w.sum(-1, keepdims=True)


def draw(name):
    M, P, PF, L, nqv, nqf, ne = SHAPES[name]
    rng = np.random.default_rng(list(SHAPES[name]))
    nf = ne * L
    g = dict(wdet=rng.uniform(0.5, 1.0, (ne, nqv)) / nqv, dphix=rng.standard_normal((ne, nqv, P, 3)),
             phi=weights(rng, nqv, P), phif=weights(rng, ne, L, nqf, P), psi=weights(rng, nqf, PF),
             ndA=rng.standard_normal((ne, L, nqf, 3)) / nqf, dA=rng.uniform(0.5, 1.0, (ne, L, nqf)) / nqf,
             src=rng.standard_normal((ne, nqv, M)), uD=rng.standard_normal((ne, L, nqf, M)),
             bnd=(rng.uniform(size=(ne, L)) < 0.4).astype(np.int32), nqv=nqv, nqf=nqf)
    if M == 5:
        m = dict(kind="navier_stokes", tau=3.0, Re=100.0, Pr=0.72, gamma=1.4)
        base = np.array([1.0, 1.0, 0.1, -0.1, 6.0])
    else:
        m = dict(kind="elasticity", tau=1.0, lam=0.6, mu=0.4)
        base = np.zeros(3)
    u = base[None, :, None] + 0.1 * rng.standard_normal((ne, M, P))
    uh = base[None, :, None] + 0.1 * rng.standard_normal((nf, M, PF))
    minv = np.eye(P) + 0.1 * rng.standard_normal((ne, P, P)) / P
    up = u + 0.1 * rng.standard_normal(u.shape)
    e2f = np.arange(nf, dtype=np.int32).reshape(ne, L)
    d = dict(ne=ne, nf=nf, ncomp=M, dim=3, npe=P, npf=PF, nlfe=L)
    return d, g, m, u, uh, up, minv, e2f


@pytest.mark.parametrize("name", list(SHAPES))
def test_random_geometry_matches_oracle(name):
    from paper_2512_13619_amd import hdg
    d, g, m, u, uh, up, minv, e2f = draw(name)
    say("sys shapes", name, d)
    ne, M, P, PF, L = (d[k] for k in ("ne", "ncomp", "npe", "npf", "nlfe"))
    c = 2.5
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    gd = {k: (dev(v) if isinstance(v, np.ndarray) else v) for k, v in g.items()}
    nu, nq, nt = M * P, 3 * M * P, L * M * PF
    z = lambda *s: torch.full((ne,) + s, np.nan, dtype=torch.float64, device="cuda")
    out = dict(Minv=dev(minv), D=z(nu, nq), E=z(nu, nu), F=z(nu, nt), G=z(nt, nq), H=z(nt, nu), J=z(nt, nt), ru=z(nu),
               rt=z(nt), q=z(nq), Bd=z(3, P, P), Cd=z(3, P, L * PF))
    ctx = hdg.Context(0)
    args = (d, gd, m, dev(e2f), dev(u), dev(uh), out)
    tt = dict(c=c, u_prev=dev(up))
    ctx.element_blocks_sys(*args, keep_mass=True, time_term=tt)
    got = {k: v.cpu().numpy() for k, v in out.items()}
    res = dict(Minv=out["Minv"], ru=z(nu), rt=z(nt))
    ctx.element_blocks_sys(*args[:-1], res, keep_mass=True, residual_only=True, time_term=tt)
    assert torch.equal(res["ru"], out["ru"]) and torch.equal(res["rt"], out["rt"])
    for e in sorted({0, min(255, ne - 1), min(256, ne - 1), ne - 1}):
        uh_el = uh[e2f[e]]
        _, Bd, Cd = mass_and_q_operators(g, e)
        q = np.zeros((M, 3, P))
        for a in range(M):
            for x in range(3):
                q[a, x] = -minv[e] @ (Bd[x] @ u[e, a] + Cd[x] @ uh_el[:, a].reshape(-1))
        assert relerr(got["q"][e].reshape(q.shape), q) < 1e-12, (name, e, "q")
        _, Ru, Rt = OS.residual(g, m, e, q, u[e], uh_el, (c, up[e], None))
        for k, want in (("ru", -Ru), ("rt", -Rt)):
            assert relerr(got[k][e], want.reshape(-1)) < 1e-12, (name, e, k)
        for k, want in zip("DEFGHJ", OS.jacobian(g, m, e, q, u[e], uh_el, c)):
            err = relerr(got[k][e], want)
            assert err < 1e-12, (name, e, k, err)
