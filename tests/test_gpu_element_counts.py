"""The element kernels share an element's tiles out over one, two or four waves, by the LDS it needs and the
size of the mesh. How many does not change a result: the same elements give the same arrays, bit for bit,
alone, in a mesh of some hundred and in one of thousands (where each count of waves is taken), with and
without kept mass matrices; the values themselves are checked in test_gpu_element_shapes.py."""
import numpy as np
import pytest
import torch

from test_gpu_parity import say
from test_gpu_sys_shapes import weights

pytestmark = pytest.mark.gpu

# D, P, PF, L, nqv, nqf: about 0.6, 3, 12, 19, 41 and 54 KB of LDS
SHAPES = {"line_p1": (1, 2, 1, 2, 3, 1), "quad_p1": (2, 4, 2, 4, 9, 3), "tri_p3": (2, 10, 4, 3, 25, 5),
          "hex_p1": (3, 8, 4, 6, 27, 9), "tet_p2": (3, 10, 6, 4, 64, 16), "tet_p3": (3, 20, 10, 4, 45, 14)}
NAMES = dict(Minv="P P", Bd="D P P", Cd="D P T", D="P Q", E="P P", F="P T", G="T Q", H="T P", J="T T", ru="P", rt="T", q="Q")


def draw(name, few):
    D, P, PF, L, nqv, nqf = SHAPES[name]
    rng = np.random.default_rng([D, P, nqv])
    phi = 0.2 * weights(rng, nqv, P)
    phi[np.arange(min(nqv, P)), np.arange(min(nqv, P))] += 1
    g = dict(wdet=rng.uniform(0.5, 1.0, (few, nqv)), dphix=rng.standard_normal((few, nqv, P, D)), phi=phi,
             phif=weights(rng, few, L, nqf, P), psi=weights(rng, nqf, PF), ndA=rng.standard_normal((few, L, nqf, D)) / nqf,
             dA=rng.uniform(0.5, 1.0, (few, L, nqf)) / nqf, src=rng.standard_normal((few, nqv)),
             uD=rng.standard_normal((few, L, nqf)), bnd=(rng.uniform(size=(few, L)) < 0.4).astype(np.int32))
    state = dict(u=rng.standard_normal((few, P)), uh=rng.standard_normal((few * L, PF)), up=rng.standard_normal((few, P)))
    return g, state


@pytest.mark.parametrize("name", list(SHAPES))
def test_number_of_waves_does_not_change_results(name):
    from paper_2512_13619_amd import hdg
    D, P, PF, L, nqv, nqf = SHAPES[name]
    few = 3
    g, s = draw(name, few)
    m = dict(nu=0.3, tau=1.5, beta=[0.7, -0.2, 0.4][:D], gamma=[0.1, 1.0, -0.5][:D])
    size = dict(P=P, D=D, T=L * PF, Q=D * P)
    ctx = hdg.Context(0)
    first = None
    for copies in (1, 500, 2000):
        say("element counts", name, few * copies)
        dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
        rep = lambda a: dev(a).repeat(copies, *[1] * (np.ndim(a) - 1))
        geom = {k: (dev(v) if k in ("phi", "psi") else rep(v)) for k, v in g.items()} | dict(nqv=nqv, nqf=nqf)
        ne = few * copies
        d = dict(ne=ne, nf=ne * L, ncomp=1, dim=D, npe=P, npf=PF, nlfe=L)
        e2f = torch.arange(ne * L, dtype=torch.int32, device="cuda")
        u, uh, up = rep(s["u"]), rep(s["uh"]), rep(s["up"])
        out = {k: torch.full([ne] + [size[c] for c in v.split()], float("nan"), dtype=torch.float64, device="cuda")
               for k, v in NAMES.items()}
        tt = dict(c=2.5, u_prev=up)
        ctx.element_blocks(d, geom, m, e2f, u, uh, out, time_term=tt)
        kept = {k: v.clone() for k, v in out.items()}
        ctx.element_blocks(d, geom, m, e2f, u, uh, kept, time_term=tt, keep_mass=True)
        res = dict(Minv=out["Minv"], ru=torch.zeros_like(out["ru"]), rt=torch.zeros_like(out["rt"]))
        ctx.element_blocks(d, geom, m, e2f, u, uh, res, time_term=tt, keep_mass=True, residual_only=True)
        first = first or {k: v[:few].clone() for k, v in out.items()}
        for k, v in out.items():
            assert not torch.isnan(v).any(), k
            assert torch.equal(v[:few], first[k]) and torch.equal(v[-few:], first[k]), (k, ne)
            assert torch.equal(kept[k], v), (k, ne)
        assert torch.equal(res["ru"], out["ru"]) and torch.equal(res["rt"], out["rt"]), ne
