"""Which kernel a call launches, with how many workgroups, on the stand-in
runtime of fake_hip.py: the variants launch the tiles and chunks that
rkl_variant_info names, the default the form that measured fastest."""
import fake_hip

SIZES = "((37, 11, 70), (48, 40, 36), (20, 20, 20), (5, 3, 1), (500, 251, 13), (100, 90, 200))"


def test_a_variant_runs_its_own_tile_and_chunk(tmp_path):
    """every variant but 0, whatever the grid; a small 3-D grid must not end up in
    the block kernel unless the variant is left to the library"""
    fake_hip.run(tmp_path, r'''
up = lambda a, b: -(-a // b)
seen = set()
for n in %s:
    for prec in (0, 1):
        for v in range(1, rkl.rkl_variant_count()):
            x, y, z, fuse = rkl.rkl_variant_info(v)
            if fuse != 1:
                continue
            plan = rkl.rkl_plan([desc(n)], precision=prec, variant=v)
            for call in (lambda: rkl.rkl_superstep(plan, 0, T, b, 1e-3, None), lambda: rkl.rkl_flux_div(plan, 0, T, b, out, None),
                         lambda: rkl.rkl_subcycle(plan, 0, T, b, 2.5, 9, None),
                         lambda: rkl.rkl_supersteps_async(plan, 0, T, b, 1e-3, 2, 4, None, None)):
                hip.fake_reset()
                call()
                got = {l[:2] for l in launches() if "finalize" not in l[0] and "reduce" not in l[0]}
                want = up(n[0], x) * up(n[1], y) * up(n[2], z)
                assert got and all("stage_kernel" in k and (", %%d, %%d, " %% (x, y)) in k and g == want for k, g in got), (n, v, got, want)
            seen.add((x, y, z))
            rkl.rkl_destroy(plan)
assert len(seen) == 8, seen
''' % SIZES)


def test_zeroed_options_give_the_default(tmp_path):
    fake_hip.run(tmp_path, r'''
for n, ndim in [(m, 3) for m in %s] + [((64, 64, 1), 2), ((400, 1, 1), 1)]:
    got = []
    for v in (-1, 0):
        plan = rkl.rkl_plan([desc(n, ndim)], variant=v)
        hip.fake_reset()
        rkl.rkl_superstep(plan, 0, T, b, 1e-3, None)
        got.append(launches())
        rkl.rkl_destroy(plan)
    assert got[0] == got[1], n
''' % SIZES)


def test_autotune_times_each_form_once(tmp_path):
    """variants that launch the same kernels on a grid are one candidate"""
    fake_hip.run(tmp_path, r'''
for n, ndim, edges, prec in (((20, 20, 1), 2, (0, 0, 0), 0), ((20, 20, 20), 3, (0, 0, 0), 0), ((37, 11, 40), 3, (0, 1, 0), 0),
                             ((20, 20, 20), 3, (0, 0, 0), 1), ((24, 24, 24), 3, (2, 0, 0), 0)):
    plan = rkl.rkl_plan([desc(n, ndim, edges=edges)], precision=prec)
    for ax in range(3):
        if edges[ax] == 2:
            rkl.rkl_set_ghosts(plan, 0, ax, T, T)
    forms = set()
    for v in range(rkl.rkl_variant_count()):
        try:
            rkl.rkl_set_variant(plan, v)
        except rkl.RklError:
            continue                       # fused variants: mixed, periodic 3-D grids
        put("s", 9)
        hip.fake_reset()
        rkl.rkl_superstep(plan, 0, T, b, 1e-3, None)
        forms.add(tuple(launches()))
    starts = sum("finalize" in l[0] or ndim == 2 for l in min(forms, key=len))   # of one super-step
    assert starts == 1
    hip.fake_reset()
    best, ms = rkl.rkl_autotune(plan, 0, T, b, 1e-3, 2, None)
    got = sum("finalize" in l[0] or ndim == 2 for l in launches())
    assert got == 3 * len(forms), (n, got, len(forms))     # one untimed and two timed each
    assert best == 0 or ndim == 3
    rkl.rkl_destroy(plan)
''')


def test_default_form(tmp_path):
    """sizes at which one form measured at least 10 % faster than the other
    (us a stage, march / blocks)"""
    fake_hip.run(tmp_path, r'''
FP64, MIXED = 0, 1
MC, SAT, POW = dict(sat=0), dict(sat=1), dict(sat=2, law=1.7)
CASES = [  # size, precision, physics, blocks
    ((24, 24, 24), FP64, MC, True), ((24, 24, 24), MIXED, POW, True),          # 7.2 / 5.4, 8.2 / 6.6
    ((64, 64, 64), FP64, SAT, True), ((64, 64, 64), MIXED, MC, True),          # 11.2 / 9.4, 8.7 / 7.2
    ((104, 104, 104), FP64, MC, True), ((112, 112, 112), FP64, MC, True),      # 28.7 / 24.9, 35.0 / 28.8
    ((128, 128, 128), FP64, MC, False), ((144, 144, 144), MIXED, SAT, False),  # 35.7 / 41.9, 35.7 / 43.0
    ((160, 160, 160), FP64, SAT, False), ((192, 192, 192), MIXED, MC, False),  # 76.4 / 85.2, 68.1 / 95.4
    ((128, 128, 128), FP64, POW, True), ((256, 256, 256), FP64, POW, True),    # 124 / 90, 915 / 654
    ((256, 256, 256), MIXED, POW, False), ((384, 384, 384), FP64, POW, True),  # 307 / 386, 3181 / 2190
    ((512, 512, 1), FP64, MC, False), ((512, 512, 1), FP64, POW, False),       # 14.1 / 21.2, 35.7 / 43.7
    ((512, 512, 4), FP64, MC, True), ((512, 512, 4), FP64, POW, True),         # 25.6 / 22.2, 80.7 / 44.6
    ((512, 512, 6), MIXED, SAT, False), ((65, 65, 300), FP64, SAT, True),      # 24.7 / 29.6, 50.7 / 34.4
    ((1000, 1000, 5), FP64, SAT, False), ((8, 8, 512), MIXED, SAT, True),      # 102 / 162, 7.0 / 5.2
]
for n, prec, phys, blocks in CASES:
    plan = rkl.rkl_plan([desc(n, **phys)], precision=prec)
    hip.fake_reset()
    rkl.rkl_superstep(plan, 0, T, b, 1e-3, None)
    got = any("block_kernel" in l[0] for l in launches())
    assert got == blocks, (n, prec, phys)
    rkl.rkl_destroy(plan)
''')


def test_persistent_batches_keep_the_chunk_of_the_policy(tmp_path):
    """the per-stage launches shorten the chunks of a small batch, the persistent
    launch does not; switching back and forth gives each its own tiles"""
    fake_hip.run(tmp_path, r'''
sizes = (ctypes.c_size_t * 4096).in_dll(hip, "fake_alloc")
grids = [desc((32, 32, 64)) for _ in range(12)]
for prec in (0, 1):
    for policy in range(rkl.rkl_batch_policy_count()):
        tz = rkl.rkl_batch_policy_info(policy)[1]
        plan = rkl.rkl_plan(grids, precision=prec)
        lib.rkl_set_batch_policy(plan, policy)

        def items(mode):
            put("allocs", 0)
            assert lib.rkl_set_batch_mode(plan, mode) == 0
            return sizes[1] // 8           # the second allocation is the list of (grid, tile) pairs
        first = items(1)
        assert first %% (12 * (-(-64 // tz))) == 0 and first // (12 * (-(-64 // tz))) <= 8, (policy, first)
        hip.fake_reset()
        assert items(0) > first and items(1) == first
        rkl.rkl_destroy(plan)
'''.replace("%%", "%"))


def test_plan_of_many_grids_is_quick(tmp_path):
    """host time of rkl_plan, a grid of a batch: 1.1 us before launches were fitted
    to grids, 0.6 us now; fitting every variant to every grid took 3.4 us"""
    fake_hip.run(tmp_path, r'''
import random, time
r = random.Random(1)
for ndim in (3, 2):
    grids = [desc((r.randint(16, 64), r.randint(16, 64), r.randint(16, 64) if ndim == 3 else 1), ndim) for _ in range(2000)]
    best = 1e9
    for _ in range(15):
        t = time.perf_counter()
        plan = rkl.rkl_plan(grids, smax=32)
        best = min(best, time.perf_counter() - t)
        rkl.rkl_destroy(plan)
    assert best <= 2000 * 2e-6, (ndim, best)
''')


def test_extrema_of_a_batch_fit(tmp_path):
    """the room for the last stage's extrema covers every variant's launch, also
    where it is bounded instead of fitted (more than 16 grids)"""
    fake_hip.run(tmp_path, r'''
import random
sizes = (ctypes.c_size_t * 4096).in_dll(hip, "fake_alloc")
r = random.Random(2)
for k in range(12):
    ns = [tuple(r.choice((1, 2, 5, 17, 33, 64, 130, 200)) for _ in range(3)) for _ in range(17)]
    for prec in (0, 1):
        put("allocs", 0)
        plan = rkl.rkl_plan([desc(n, law=(2.5, 1.7)[k % 2]) for n in ns], precision=prec)
        room = sizes[4]                       # Ya, Yb, tau M(Y0), coefficients, then the small one
        for v in list(range(8)) + [16]:
            rkl.rkl_set_variant(plan, v)
            for g in range(17):
                hip.fake_reset()
                rkl.rkl_supersteps_async(plan, g, T, b, 1e-3, 2, 3, None, None)
                most = max(l[1] for l in launches() if "stage_kernel" in l[0] or "block_kernel" in l[0])
                assert 24 * most <= room - 24 * 1024, (ns[g], v, most, room)
        rkl.rkl_destroy(plan)
''', 300)


def test_few_stages_of_a_large_2d_grid(tmp_path):
    """one sub-step takes one launch (and a copy), two take two; a super-step of few
    stages takes regions that reach fewer cells around their tiles"""
    fake_hip.run(tmp_path, r'''
plan = rkl.rkl_plan([desc((1000, 1000, 1), 2, sat=2, law=1.7)], precision=1)
flat = lambda: [l for l in launches() if "flat_kernel" in l[0]]
for q in (1, 2):
    hip.fake_reset()
    assert rkl.rkl_subcycle(plan, 0, T, b, q - 0.5, 9, None) == q
    assert len(flat()) == q, flat()
plan = rkl.rkl_plan([desc((2048, 2048, 1), 2, lim=0, law=0.0)], precision=1)
cells = {}
for cap in (3, 20):
    hip.fake_reset()
    rkl.rkl_superstep_async(plan, 0, T, b, 1e-3, cap, None, None)
    cells[cap] = flat()[0][1] * flat()[0][2] / 2048.0 ** 2      # computed, borders included
assert cells[3] < 1.45 < 1.6 < cells[20], cells
''')


def test_few_stages_of_a_large_mixed_pow_grid(tmp_path):
    """kappa ~ T^1.7 in mixed precision: rkl_superstep learns s before it cuts a large
    2-D grid, so that few stages get regions of their own in every group (a super-step
    of three stages took 4 to 10 % longer than with one stage a launch)"""
    fake_hip.run(tmp_path, r'''
for n in ((1500, 1400, 1), (4096, 4096, 1)):
    for prec, law in ((1, 1.7), (1, 2.5), (0, 1.7)):
        plan = rkl.rkl_plan([desc(n, 2, law=law)], precision=prec)
        for s in (3, 4, 5, 20):
            put("s", s)
            hip.fake_reset()
            assert rkl.rkl_superstep(plan, 0, T, b, 1e-3, None) == s
            flat = [l[1:] for l in launches() if "flat_kernel" in l[0]]
            assert any("finalize" in l[0] for l in launches()) == (prec == 1 and law == 1.7)
            if prec == 1 and law == 1.7:
                assert len(set(flat)) == 1 and len(flat) >= 2, (n, s, flat)
        rkl.rkl_destroy(plan)
''')
