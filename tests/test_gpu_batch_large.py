"""Large instances in a batch: the Gram-Schmidt sweeps of an instance above the size where its partial sums
are added up by a kernel of their own, beside instances below it, and a cost per unknown that does not grow
with the instance. The systems are those of test_gpu_long_cycles.py, formed on the GPU; solved to 1e-11 in the
residual, which is recomputed here in float64."""
import torch

import numpy as np
import pytest

from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def system(seed, nb, L, nf, diag):
    g = torch.Generator(device="cuda").manual_seed(seed)
    S = 2 * L - 1
    f = torch.arange(nf, device="cuda")
    nbr = torch.stack([(f + s * s) % nf for s in range(S)], 1).int().contiguous()
    K = (2 * torch.rand(nf, S, nb, nb, generator=g, dtype=torch.float64, device="cuda") - 1) / (S * nb)
    K[:, 0] += diag * torch.eye(nb, dtype=torch.float64, device="cuda")
    return K, nbr, torch.randn(nf * nb, generator=g, dtype=torch.float64, device="cuda")


def times(K, nbr, x):
    """K x, blocks column-major."""
    nf, S, nb, _ = K.shape
    xb = x.view(nf, nb)
    y = torch.zeros_like(xb)
    for s in range(S):
        y += (K[:, s].transpose(1, 2) * xb[nbr[:, s].long()][:, None, :]).sum(2)
    return y.view(-1)


@pytest.mark.parametrize("kw", [dict(restart=200), dict(restart=70, orth="cgs"), dict(restart=90, use_graph=True, prec="none")],
                         ids=["cgs2", "cgs", "graph"])
def test_large_beside_small(kw):
    from paper_2512_13619_amd import hdg
    # 256, 16 and 64 chunks: the first is above the bound from 33 columns on, the last from 129
    shapes = [(4, 4, 32768), (2, 4, 4096), (4, 4, 8192)]
    data = [system(60 + i, *s, 1.2 / np.sqrt(3 * (2 * s[1] - 1) * s[0])) for i, s in enumerate(shapes)]
    ctx = hdg.Context(0)
    bt = hdg.Batch(ctx, [dict(ne=2, nf=nf, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L) for nb, L, nf in shapes])
    K, nbr, b = (torch.cat([d[k].reshape(-1) for d in data]) for k in range(3))
    x = torch.zeros_like(b)
    st, stats = bt.gmres_solve(K, None, nbr, b, x, max_iters=600, rtol=1e-11, **kw)
    off = bt.offsets("vec")
    for i, (k, n, r) in enumerate(data):
        err = float(torch.linalg.norm(r - times(k, n, x[off[i]:off[i + 1]])) / torch.linalg.norm(r))
        say("large batch", kw, shapes[i], stats[i]["iters"], stats[i]["cycles"], err)
        assert stats[i]["converged"] and err < 1.1e-11, shapes[i]
        assert stats[i]["iters"] > 64 and stats[i]["cycles"] <= -(-stats[i]["iters"] // kw["restart"]) + 1
    assert st == 0


def test_one_large_instance_costs_no_more_than_many():
    """4,000,000 unknowns in one instance and in 64: with every block adding up all of its instance's partial sums
    one takes more than twice the time of many."""
    from paper_2512_13619_amd import hdg
    ctx = hdg.Context(0)
    nb, L, total = 4, 4, 1000000
    best = {}
    for n in (1, 64):
        parts = [system(70, nb, L, total // n, 0.2) for _ in range(n)]
        K, nbr, b = (torch.cat([p[k].reshape(-1) for p in parts]) for k in range(3))
        bt = hdg.Batch(ctx, [dict(ne=2, nf=total // n, ncomp=1, dim=2, npe=3, npf=nb, nlfe=L)] * n)
        best[n] = np.inf
        for _ in range(4):
            x = torch.zeros_like(b)
            torch.cuda.synchronize()
            _, stats = bt.gmres_solve(K, None, nbr, b, x, restart=30, max_iters=30, rtol=1e-300)
            best[n] = min(best[n], stats[0]["t_total"])
        bt.close()
    say("one and many", {n: f"{1e3 * t:.1f} ms" for n, t in best.items()})
    assert best[1] < 1.4 * best[64]
