"""The calls that wait for a word from the GPU return while their launch ends.
What comes next on another stream must find them over: rkl_dt_par, and
rkl_subcycle and rkl_aag with nothing to do, have nothing left to store or to
read (the state of the grid, the caller's T) once they return."""
import numpy as np
import pytest

from helpers import lib_desc
from paper_1702_05487_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [((400, 1, 1), 1), ((64, 50, 1), 2), ((24, 18, 14), 3), ((150, 127, 30), 3)]


@pytest.mark.parametrize("k", range(len(SIZES)), ids=["%dx%dx%d" % n for n, _ in SIZES])
def test_next_call_on_another_stream(k):
    import torch
    from paper_1702_05487_amd import rkl
    n, ndim = SIZES[k]
    print("read-back", n, flush=True)
    rng = np.random.default_rng(k)
    T0 = torch.from_numpy(1.0 + 0.2 * rng.random(n[::-1])).to("cuda:0")
    hot = 3.0 * T0
    b = torch.from_numpy(inputs.unit_vectors(rng.standard_normal((3,) + n[::-1]))).to("cuda:0")
    plan = rkl.Plan([lib_desc(n, (0.03, 0.04, 0.05), ndim, dict(inputs.SPITZER_MC_SAT, phi=0.05))])
    dt = inputs.midpoint_ratio(6) * plan.dt_par(T0)
    want = T0.clone()
    assert plan.superstep(want, b, dt) == 6
    state = plan.query()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    W, X = T0.clone(), hot.clone()
    torch.cuda.synchronize()
    reads = [lambda: plan.dt_par(X), lambda: plan.subcycle(X, b, 0.0), lambda: plan.aag(X, b, 0.0, 0.1)]
    for i in range(60):
        with torch.cuda.stream(one):
            reads[i % 3]()
        with torch.cuda.stream(two):
            X.fill_(float("nan"))          # no longer read
            assert plan.superstep(W, b, dt) == 6
            assert plan.query() == state   # not that of the first call
            assert torch.equal(W, want), i
            W.copy_(T0)
            X.copy_(hot)
            torch.cuda.synchronize()
    plan.close()
