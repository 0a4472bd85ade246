"""z-chunk lengths of the 3-D stage kernels on grids wide enough to keep them.

A launch shortens its z-chunks while the grid would leave CUs idle, so
narrow grids run chunks of one or two planes whatever their depth.  Here a
plane holds 512 tiles of 32 x 8 cells, which fills the GPU, and a chunk is as
long as the variant allows: the depths give every remainder of the six-fold
plane loop in one chunk, and chunks of unequal work at 33 and 65 planes.

  - depths to 14: against the oracle, FP64 rel-L1 <= 1e-12, mixed <= 1e-5
    (the bars of the other super-step tests), the same stage count;
  - every depth: the same bits with chunks of at most 16, 32 and 64 planes,
    and from rkl_superstep_async.

Grids of about 130 cells a side march too (smaller ones run in blocks of
16 x 4 x 4 cells): with ragged sides, every kind of z and x edge and every
saturation form against the oracle, and chained super-steps, whose last stage
keeps the extrema, against separate calls.
"""
import numpy as np
import pytest

import oracle
from helpers import lib_desc, oracle_grid, rel_l1
from paper_1702_05487_amd import inputs

pytestmark = pytest.mark.gpu

H = (0.03, 0.04, 0.05)


@pytest.mark.parametrize("depth", (1, 2, 3, 4, 5, 6, 7, 9, 14, 33, 65))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_long_chunks(precision, depth):
    import torch
    from paper_1702_05487_amd import rkl
    print("z-chunk", precision, depth, flush=True)
    n = (512, 256, depth)
    rng = np.random.default_rng(2000 + depth)
    T = 1.0 + 0.2 * rng.random((depth, 256, 512))
    b = inputs.unit_vectors(rng.standard_normal((3, depth, 256, 512)))
    p = dict(inputs.SPITZER_MC_SAT, phi=0.003)
    g = oracle_grid(n, H, 3, p)
    dt = inputs.midpoint_ratio(4) * oracle.dt_par(g, T)
    bd = torch.from_numpy(b).to("cuda:0", torch.float32 if precision == "mixed" else torch.float64)
    got = {}
    for v in (6, 0, 1, 3):
        plan = rkl.Plan([lib_desc(n, H, 3, p)], precision=precision, variant=v)
        Td = torch.from_numpy(T).to("cuda:0")
        assert plan.superstep(Td, bd, dt) == 4
        Ta = torch.from_numpy(T).to("cuda:0")
        plan.superstep_async(Ta, bd, dt, 5)
        assert torch.equal(Td, Ta), v
        plan.close()
        got[v] = Td.cpu().numpy()
        assert np.array_equal(got[v], got[6]), v
    if depth <= 14:
        oracle.set_threads(16)
        ref, s, _ = oracle.superstep(g, T, bd.double().cpu().numpy(), dt)
        oracle.set_threads(1)
        assert s == 4
        assert rel_l1(got[6], ref) <= (1e-12 if precision == "fp64" else 1e-5)


@pytest.mark.parametrize("edges,lim,sat,law,precision", [
    ((0, 0, 0), 1, 1, 2.5, "fp64"), ((1, 0, 1), 0, 2, 0.0, "mixed"), ((0, 1, 1), 1, 0, 1.7, "fp64"),
    ((1, 1, 0), 1, 2, 2.5, "mixed"),
])
def test_marched_ragged(edges, lim, sat, law, precision):
    import torch
    from paper_1702_05487_amd import rkl
    print("marched", edges, lim, sat, law, precision, flush=True)
    n = (131, 126, 129)
    rng = np.random.default_rng(77)
    T = 1.0 + 0.2 * rng.random(n[::-1])
    b = inputs.unit_vectors(rng.standard_normal((3,) + n[::-1]))
    p = dict(inputs.BASE, limiter=lim, saturation=sat, phi=0.01, kappa_exp=law, kperp_ratio=0.02, boundary=edges)
    g = oracle_grid(n, H, 3, p)
    dt = inputs.midpoint_ratio(4) * oracle.dt_par(g, T)
    bd = torch.from_numpy(b).to("cuda:0", torch.float32 if precision == "mixed" else torch.float64)
    plan = rkl.Plan([lib_desc(n, H, 3, p)], precision=precision)
    Td = torch.from_numpy(T).to("cuda:0")
    assert plan.superstep(Td, bd, dt) == 4
    oracle.set_threads(16)
    ref, s, _ = oracle.superstep(g, T, bd.double().cpu().numpy(), dt)
    oracle.set_threads(1)
    assert s == 4
    assert rel_l1(Td.cpu().numpy(), ref) <= (1e-12 if precision == "fp64" else 1e-5)
    many = torch.from_numpy(T).to("cuda:0")
    plan.supersteps_async(many, bd, dt, 3, 6)
    for _ in range(2):
        plan.superstep(Td, bd, dt)
    assert torch.equal(Td, many)
    plan.close()


@pytest.mark.parametrize("edges,lim,sat,law", [
    ((0, 0, 0), 1, 1, 2.5), ((1, 0, 1), 0, 2, 2.5), ((0, 1, 1), 1, 1, 0.0), ((1, 1, 0), 0, 1, 1.7),
])
@pytest.mark.parametrize("depth", (1, 2, 5, 7, 13))
def test_three_waves(depth, edges, lim, sat, law):
    """The saturated FP64 kernel reads the own cell back from LDS and loads one
    plane ahead on the 32 x 8 and 16 x 16 tiles; the 64 x 4 tile (variants 2, 3
    and 7) keeps it in registers and loads two ahead: the same bits on ragged
    sides, and the oracle's values.  512 tiles, so that every depth marches."""
    import torch
    from paper_1702_05487_amd import rkl
    print("three waves", depth, edges, lim, sat, law, flush=True)
    n = (500, 251, depth)
    rng = np.random.default_rng(50 + depth)
    T = 1.0 + 0.2 * rng.random(n[::-1])
    b = inputs.unit_vectors(rng.standard_normal((3,) + n[::-1]))
    p = dict(inputs.BASE, limiter=lim, saturation=sat, phi=0.01, kappa_exp=law, kperp_ratio=0.02, boundary=edges)
    g = oracle_grid(n, H, 3, p)
    dt = inputs.midpoint_ratio(4) * oracle.dt_par(g, T)
    bd = torch.from_numpy(b).to("cuda:0")
    got = []
    for v in range(8):
        plan = rkl.Plan([lib_desc(n, H, 3, p)], precision="fp64", variant=v)
        Td = torch.from_numpy(T).to("cuda:0")
        assert plan.superstep(Td, bd, dt) == 4
        plan.close()
        got.append(Td.cpu().numpy())
        assert np.array_equal(got[v], got[0]), v
    oracle.set_threads(16)
    ref, s, _ = oracle.superstep(g, T, b, dt)
    oracle.set_threads(1)
    assert s == 4
    assert rel_l1(got[0], ref) <= 1e-12


@pytest.mark.parametrize("depth", (171, 172))
def test_cached_and_streamed(depth):
    """Mixed grids up to 352 MiB of stage fields keep the pointwise fields in
    the caches, larger ones stream them past: 172 planes of 212 x 212 cells are
    the first beyond.  Both, and all one-stage variants, have the fused
    kernel's bits."""
    import torch
    from paper_1702_05487_amd import rkl
    print("cached", depth, flush=True)
    n = (212, 212, depth)
    assert (48 * n[0] * n[1] * n[2] <= 352 << 20) == (depth == 171)
    rng = np.random.default_rng(9)
    T = 1.0 + 0.2 * rng.random(n[::-1])
    b = torch.from_numpy(inputs.unit_vectors(rng.standard_normal((3,) + n[::-1]))).to("cuda:0", torch.float32)
    p = dict(inputs.SPITZER_MC_SAT, phi=0.003)
    dt = inputs.midpoint_ratio(5) * oracle.dt_par(oracle_grid(n, H, 3, p), T)
    got = []
    for v in (8, 0, 2, 4, 6):
        plan = rkl.Plan([lib_desc(n, H, 3, p)], precision="mixed", variant=v)
        Td = torch.from_numpy(T).to("cuda:0")
        assert plan.superstep(Td, b, dt) == 5
        plan.close()
        got.append(Td)
        assert torch.equal(Td, got[0]), v
