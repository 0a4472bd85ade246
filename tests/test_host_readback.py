"""The calls that wait for a word from the GPU (rkl_superstep, rkl_dt_par,
rkl_subcycle, rkl_aag), on the stand-in runtime of fake_hip.py: what they leave
behind when they fail, and how they wait."""
import fake_hip


def test_a_failed_call_leaves_nothing_pending(tmp_path):
    """A launch fails behind the one that stores s and dt_par: the call returns
    only after the stream has drained, so that neither the store reaches a later
    call nor a launch still reads fields that the caller may free."""
    fake_hip.run(tmp_path, r'''
for n, ndim in (((20, 20, 20), 3), ((200, 200, 200), 3), ((200, 200, 1), 2), ((400, 1, 1), 1)):
    plan = rkl.rkl_plan([desc(n, ndim)])
    for call in (lambda: rkl.rkl_superstep(plan, 0, T, b, 1e-3, None), lambda: rkl.rkl_dt_par(plan, 0, T, None)):
        put("pending", 1)
        put("queries", 0)
        put("s", 3)
        hip.fake_reset()
        call()
        last = hip.fake_count()
        for k in range(last):
            put("fail_at", k)
            put("s", 7)
            put("dt_par", 0.25)
            hip.fake_reset()
            try:
                call()
                raise SystemExit("launch %d of %s failed unnoticed" % (k, n))
            except rkl.RklError as e:
                assert e.status == rkl.RKL_EDEVICE, e
            assert get("unfinished") == 0, (n, k, get("unfinished"))
            put("fail_at", -1)
            put("s", 4)
            put("dt_par", 0.5)
            hip.fake_reset()
            r = call()
            assert r in (4, 0.5), (n, k, r)
    rkl.rkl_destroy(plan)
''')


def test_a_refused_stage_count_leaves_nothing_pending(tmp_path):
    """RKL_ESTAGES: the stages enqueued before s was known do nothing, but they
    have been given T and b"""
    fake_hip.run(tmp_path, r'''
for n, ndim in (((20, 20, 20), 3), ((200, 200, 200), 3), ((200, 200, 1), 2)):
    plan = rkl.rkl_plan([desc(n, ndim)], smax=8)
    put("s", 9)
    try:
        rkl.rkl_superstep(plan, 0, T, b, 1e-3, None)
        raise SystemExit("accepted")
    except rkl.RklError as e:
        assert e.status == rkl.RKL_ESTAGES
    assert get("unfinished") == 0, n
    rkl.rkl_destroy(plan)
''')


def test_a_long_wait_sleeps_where_the_process_asked_for_it(tmp_path):
    """hipDeviceScheduleBlockingSync (4): behind a stream that stays busy the
    wait goes to hipStreamSynchronize instead of asking over and over"""
    fake_hip.run(tmp_path, r'''
put("flags", 4)
put("pending", 1)
put("queries", -1)
put("query_limit", 50)
for n, ndim in (((20, 20, 20), 3), ((200, 200, 1), 2)):
    plan = rkl.rkl_plan([desc(n, ndim)])
    before = get("syncs")
    assert rkl.rkl_superstep(plan, 0, T, b, 1e-3, None) == 3
    assert rkl.rkl_dt_par(plan, 0, T, None) == 1.0
    assert get("syncs") == before + 2
    rkl.rkl_destroy(plan)
''')


def test_calls_with_nothing_to_do_leave_nothing_pending(tmp_path):
    """rkl_subcycle and rkl_aag that enqueue no sub-step, and those refused"""
    fake_hip.run(tmp_path, r'''
plan = rkl.rkl_plan([desc((20, 20, 20))])
put("pending", 1)
for dtp, dt, status in ((1.0, 0.0, 0), (float("inf"), 1.0, 0), (1e-9, 1.0, rkl.RKL_ESTAGES)):
    put("dt_par", dtp)
    for call in (lambda: rkl.rkl_subcycle(plan, 0, T, b, dt, 10, None), lambda: rkl.rkl_aag(plan, 0, T, b, dt, 0.1, 10, None)):
        try:
            assert call() == 0 and status == 0
        except rkl.RklError as e:
            assert e.status == status
        assert get("unfinished") == 0, (dtp, dt)
''')
