"""hdg_element_blocks on seeded random geometry at the sizes where its kernel changes path: one wave
or four per element (P <= 16 or not), remainders of the 16-entry tiles and of the four-point steps,
one, two and three dimensions, with and without a time term and a kept inverse mass matrix.

The tables are rows of non-negative weights that sum to 1, the mass matrices well conditioned (at
least as many points as basis functions, or given). Tolerance as for the M-component kernels: sums
of at most 200 products with O(1) data, 1e-12 of the array's largest entry; 1e-11 where the inverse
of a mass matrix of condition up to 1e2 enters."""
import numpy as np
import pytest
import torch

import oracle.elements as OE

from test_gpu_parity import relerr, say
from test_gpu_sys_shapes import weights

pytestmark = pytest.mark.gpu

# D, P, PF, L, nqv, nqf, ne, keep, c
SHAPES = {
    "line": (1, 3, 1, 2, 5, 1, 3, True, 0.0),
    "one_wave": (2, 4, 2, 4, 9, 3, 5, False, 2.5),
    "tile_edge_16": (2, 16, 4, 4, 33, 5, 2, True, 0.0),
    "tile_edge_17": (2, 17, 5, 3, 34, 6, 2, True, 2.5),
    "quad_p4": (2, 25, 5, 4, 50, 6, 2, False, 0.0),
    "solid": (3, 20, 17, 4, 30, 19, 2, True, 2.5),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_random_geometry_matches_oracle(name):
    from paper_2512_13619_amd import hdg
    D, P, PF, L, nqv, nqf, ne, keep, c = SHAPES[name]
    rng = np.random.default_rng([D, P, PF, L, nqv])
    say("element shapes", name)
    nf, nt, nq = ne * L, L * PF, D * P
    phi = np.eye(nqv, P) + 0.2 * weights(rng, nqv, P)      # mass matrix near the identity
    g = dict(wdet=rng.uniform(0.5, 1.0, (ne, nqv)), dphix=rng.standard_normal((ne, nqv, P, D)), phi=phi,
             phif=weights(rng, ne, L, nqf, P), psi=weights(rng, nqf, PF), ndA=rng.standard_normal((ne, L, nqf, D)) / nqf,
             dA=rng.uniform(0.5, 1.0, (ne, L, nqf)) / nqf, src=rng.standard_normal((ne, nqv)),
             uD=rng.standard_normal((ne, L, nqf)), bnd=(rng.uniform(size=(ne, L)) < 0.4).astype(np.int32),
             nqv=nqv, nqf=nqf)
    m = dict(nu=0.3, tau=1.5, beta=[0.7, -0.2, 0.4][:D], gamma=[0.1, 1.0, -0.5][:D])
    mo = dict(m, beta=np.array(m["beta"]), gamma=np.array(m["gamma"]))
    u, uh, up, rx = (rng.standard_normal(s) for s in ((ne, P), (nf, PF), (ne, P), (ne, P)))
    minv = np.eye(P) + 0.1 * rng.standard_normal((ne, P, P)) / P
    e2f = np.arange(nf, dtype=np.int32).reshape(ne, L)
    d = dict(ne=ne, nf=nf, ncomp=1, dim=D, npe=P, npf=PF, nlfe=L)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    gd = {k: (dev(v) if isinstance(v, np.ndarray) else v) for k, v in g.items()}
    z = lambda *s: torch.full((ne,) + s, np.nan, dtype=torch.float64, device="cuda")
    out = dict(Minv=dev(minv) if keep else z(P, P), Bd=z(D, P, P), Cd=z(D, P, nt), D=z(P, nq), E=z(P, P), F=z(P, nt),
               G=z(nt, nq), H=z(nt, P), J=z(nt, nt), ru=z(P), rt=z(nt), q=z(nq))
    tt = dict(c=c, u_prev=dev(up), r_extra=dev(rx)) if c else None
    ctx = hdg.Context(0)
    args = (d, gd, m, dev(e2f), dev(u), dev(uh))
    ctx.element_blocks(*args, out, keep_mass=keep, time_term=tt)
    res = dict(Minv=out["Minv"], ru=z(P), rt=z(nt))
    ctx.element_blocks(*args, res, keep_mass=True, residual_only=True, time_term=tt)
    assert torch.equal(res["ru"], out["ru"]) and torch.equal(res["rt"], out["rt"])
    tol = 1e-12 if keep else 1e-11
    for e in range(ne):
        uh_el = uh[e2f[e]]
        Mm, Bd, Cd = OE.mass_and_q_operators(g, e)
        mi = minv[e] if keep else np.linalg.inv(Mm)
        q = np.stack([-mi @ (Bd[x] @ u[e] + Cd[x] @ uh_el.ravel()) for x in range(D)])
        _, Ru, Rt = OE.residual(g, mo, e, q, u[e], uh_el, (c, up[e], rx[e]) if c else None)
        want = dict(zip("DEFGHJ", OE.jacobian(g, mo, e, q, u[e], uh_el, c)), ru=-Ru, rt=-Rt, q=q)
        if not keep:
            want.update(Minv=mi, Bd=Bd, Cd=Cd)
        for k, w in want.items():
            err = relerr(out[k][e].cpu().numpy().ravel(), np.ravel(w))
            assert err < tol, (name, e, k, err)
