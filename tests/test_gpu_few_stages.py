"""2-D grids of 2^16 cells and more: super-steps of at most four stages and one or
two sub-steps are cut into regions of their own.  The same bits as the one-stage
launches, with every kind of edge, on both sides of that size and of four stages."""
import numpy as np
import pytest

import oracle
from helpers import lib_desc, oracle_grid
from paper_1702_05487_amd import inputs
from test_gpu_flat import both

pytestmark = pytest.mark.gpu

P, O, F = 0, 1, 2
CASES = [((255, 256), (P, P), 1, 0, 2.5, "fp64"), ((256, 256), (P, P), 1, 1, 2.5, "mixed"), ((300, 260), (O, P), 0, 0, 0.0, "fp64"),
         ((517, 131), (F, O), 1, 2, 1.7, "mixed"), ((3, 30000), (P, F), 0, 1, 0.0, "mixed"), ((70000, 1), (F, P), 1, 1, 2.5, "fp64"),
         ((1030, 2051), (O, P), 1, 2, 1.7, "mixed"), ((2051, 1030), (F, O), 0, 0, 1.7, "mixed")]   # s learned before the first group


@pytest.mark.parametrize("k", range(len(CASES)), ids=["%dx%d" % c[0] for c in CASES])
def test_few_stages(k):
    import torch
    from paper_1702_05487_amd import rkl
    n, edges, lim, sat, law, precision = CASES[k]
    print("few stages", n, edges, precision, flush=True)
    n += (1,)
    rng = np.random.default_rng(500 + k)
    T = 1.0 + 0.3 * rng.random(n[::-1])
    b = inputs.unit_vectors(rng.standard_normal((3,) + n[::-1]))
    p = dict(inputs.BASE, limiter=lim, saturation=sat, phi=0.02, kappa_exp=law, kperp_ratio=0.05, boundary=edges + (0,))
    h = (0.03, 0.04, 1.0)
    gh = {d: tuple(1.0 + 0.3 * rng.random(oracle.ghost_shape(n, d)) for _ in range(2)) for d in range(2) if edges[d] == F}
    c = (n, h, 2, p, precision, 3, T, b, gh)
    g = oracle_grid(n, h, 2, p)
    g.ghosts = gh
    dtp = oracle.dt_par(g, T)
    for s in (2, 3, 4, 5):
        dt = inputs.midpoint_ratio(s) * dtp
        calls = [lambda L: L.plan.superstep(L.T, L.b, dt)]
        for cap in (s, 4, 5):
            if cap >= s:
                calls.append(lambda L, cap=cap: L.plan.superstep_async(L.T, L.b, dt, cap))
        out = []
        for call in calls:
            (r, got), (r1, one) = both(c, "rkl2", call)
            assert r == r1 and np.array_equal(got, one), s
            out.append(got)
        if not gh and n[0] * n[1] <= 1 << 21:   # the most rkl_superstep_noalloc takes
            Td = torch.from_numpy(T).to("cuda:0")
            rkl.superstep_noalloc(lib_desc(n, h, 2, p), Td, torch.from_numpy(b).to("cuda:0", torch.float32 if precision == "mixed" else torch.float64),
                                  dt, s, None, precision=precision)
            out.append(Td.cpu().numpy())
        assert all(np.array_equal(o, out[0]) for o in out), s
        (r, got), (r1, one) = both(c, "rkl1", lambda L: L.plan.superstep(L.T, L.b, ((s - 1.5) ** 2 + s - 1.5) / 2 * dtp))
        assert r == r1 == s - 1 and np.array_equal(got, one), s
    for q in (1, 2, 3, 4, 5):
        (r, got), (r1, one) = both(c, "rkl2", lambda L: L.plan.subcycle(L.T, L.b, (q - 0.3) * dtp))
        assert r == r1 == q and np.array_equal(got, one), q
