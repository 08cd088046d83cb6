"""hdg_element_blocks_batch in one, two and three dimensions, mixed in one batch, at the sizes of
test_gpu_element_shapes.py and in batches large enough for each count of waves an element: every instance
against hdg_element_blocks on it alone (which that file checks against the oracle). Both sum in the same
order; contraction may differ, so the tolerances of that file are kept: 1e-12 of the array's largest entry
with kept mass matrices, 1e-11 where they are formed."""
import numpy as np
import pytest
import torch

from test_gpu_element_counts import NAMES
from test_gpu_parity import say
from test_gpu_sys_shapes import weights

pytestmark = pytest.mark.gpu

# D, P, PF, L, nqv, nqf, elements
LINE, PAIR, SOLID = (1, 3, 1, 2, 5, 1), (2, 4, 2, 4, 9, 3), (3, 20, 8, 4, 30, 9)
BATCHES = {"mixed_dimensions": [LINE + (3,), PAIR + (5,), (2, 16, 4, 4, 33, 5, 2), (2, 17, 5, 3, 34, 6, 2), (2, 25, 5, 4, 50, 6, 2), SOLID + (2,)],
           "one_wave": [LINE + (2000,), PAIR + (1500,), LINE + (1,)], "two_waves": [LINE + (900,), (3, 8, 4, 6, 27, 9, 1300)],
           "four_waves": [SOLID + (700,), LINE + (1200,)]}


def instance(seed, D, P, PF, L, nqv, nqf, ne):
    rng = np.random.default_rng([seed, D, P, ne])
    phi = 0.2 * weights(rng, nqv, P)
    phi[np.arange(min(nqv, P)), np.arange(min(nqv, P))] += 1
    g = dict(wdet=rng.uniform(0.5, 1.0, (ne, nqv)), dphix=rng.standard_normal((ne, nqv, P, D)), phi=phi,
             phif=weights(rng, ne, L, nqf, P), psi=weights(rng, nqf, PF), ndA=rng.standard_normal((ne, L, nqf, D)) / nqf,
             dA=rng.uniform(0.5, 1.0, (ne, L, nqf)) / nqf, src=rng.standard_normal((ne, nqv)),
             uD=rng.standard_normal((ne, L, nqf)), bnd=(rng.uniform(size=(ne, L)) < 0.4).astype(np.int32))
    m = dict(nu=0.1 + 0.2 * seed, tau=1.5, beta=[0.7, -0.2, 0.4][:D], gamma=[0.1, 1.0, -0.5][:D])
    d = dict(ne=ne, nf=ne * L, ncomp=1, dim=D, npe=P, npf=PF, nlfe=L)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    s = {k: dev(v) for k, v in dict(u=rng.standard_normal((ne, P)), uh=rng.standard_normal((ne * L, PF)),
                                    up=rng.standard_normal((ne, P)), rx=rng.standard_normal((ne, P)),
                                    e2f=rng.permutation(ne * L).astype(np.int32)).items()}
    return d, {k: dev(v) for k, v in g.items()}, m, s, 0.0 if seed % 2 else 2.5


@pytest.mark.parametrize("name", list(BATCHES))
def test_batched_elements_match_single(name):
    from paper_2512_13619_amd import hdg
    say("batch elements", name)
    insts = [instance(i, *k) for i, k in enumerate(BATCHES[name])]
    qv, qf = [k[4] for k in BATCHES[name]], [k[5] for k in BATCHES[name]]
    ctx = hdg.Context(0)
    bt = hdg.Batch(ctx, [d for d, *_ in insts])
    cat = lambda arrs: torch.cat([a.reshape(-1) for a in arrs])
    geom = {k: cat([g[k] for _, g, *_ in insts]) for k in insts[0][1]}
    e2f, u, uh, up, rx = (cat([s[k] for _, _, _, s, _ in insts]) for k in ("e2f", "u", "uh", "up", "rx"))
    arr = {"q": "dq"}
    for keep, residual in ((False, False), (True, False), (True, True)):
        out = {k: torch.full((bt.total(arr.get(k, k)),), float("nan"), dtype=torch.float64, device="cuda") for k in NAMES}
        if keep:
            out["Minv"].copy_(minv)
        bt.element_blocks(qv, qf, geom, [m for _, _, m, _, _ in insts], e2f, u, uh, out, residual_only=residual,
                          c=[c for *_, c in insts], u_prev=up, keep_mass=keep, r_extra=rx)
        minv = out["Minv"]
        for i, (d, g, m, s, c) in enumerate(insts):
            D, P, PF, L, nqv, nqf, ne = BATCHES[name][i]
            size = dict(P=P, D=D, T=L * PF, Q=D * P)
            z = lambda k: torch.full([ne] + [size[v] for v in NAMES[k].split()], float("nan"), dtype=torch.float64, device="cuda")
            want = {k: z(k) for k in NAMES}
            off = lambda k: slice(*bt.offsets(arr.get(k, k))[i:i + 2])
            if keep:
                want["Minv"].copy_(out["Minv"][off("Minv")].view_as(want["Minv"]))
            # a steady instance of the batch takes r_extra too
            ctx.element_blocks(d, dict(g, nqv=nqv, nqf=nqf), m, s["e2f"], s["u"], s["uh"], want, keep_mass=keep,
                               residual_only=residual, time_term=dict(c=c, u_prev=s["up"], r_extra=s["rx"]))
            for k in ("ru", "rt", "q") if residual else [k for k in NAMES if not (keep and k in ("Bd", "Cd"))]:
                a, b = out[k][off(k)], want[k].view(-1)
                err = float((a - b).abs().max() / b.abs().max())
                assert err < (1e-12 if keep else 1e-11), (name, i, k, keep, residual, err)
