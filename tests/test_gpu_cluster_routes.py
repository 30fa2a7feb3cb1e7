"""Which solver runs when clusters are the choice: one kernel form per launch at
the sizes where the form changes, and what takes over where clusters cannot
run.  Every result is the tiled solve's, bit for bit."""
import sys
import time

import numpy as np
import pytest

import cnfgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hm = pytest.importorskip("paper_2402_03640_amd")


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.lib()
    yield
    torch.cuda.synchronize()


def _bits(t):
    return t.cpu().numpy().view(np.uint32) if t.dtype == torch.float32 else t.cpu().numpy()


def _same(a, b):
    np.testing.assert_array_equal(a.restart_best, b.restart_best)
    np.testing.assert_array_equal(a.restart_step, b.restart_step)
    np.testing.assert_array_equal(a.best_assignment, b.best_assignment)
    np.testing.assert_array_equal(_bits(a.x_final), _bits(b.x_final))
    # the loss totals are FP64 sums in different orders over the same terms
    np.testing.assert_allclose(a.restart_loss, b.restart_loss, rtol=1e-12, atol=0)


def _cnf(n, k=3, ratio=4.0, seed=None):
    return hm.load_cnf(n, cnfgen.uniform_kcnf(n, int(n * ratio), k, seed=n + k if seed is None else seed))


# 31000 variables: t fits LDS with 16 workgroups per restart and not with 32
@pytest.mark.parametrize("n,R", [(31000, 1), (31000, 8), (31000, 9), (31000, 17), (31744, 2), (31745, 2)])
def test_form_change_single(n, R):
    cnf = _cnf(n)
    kw = dict(steps=70, restarts=R, eval_every=9, seed=2, lr=1e-2, want_x=True)
    a, b = hm.solve(cnf, schedule=hm.CLUSTER, **kw), hm.solve(cnf, schedule=1, **kw)
    assert a.schedule == hm.CLUSTER and b.schedule & 0xFF == 1
    _same(a, b)
    cnf.free()


# (variables, restarts) of a batch's instances whose form depended on the
# restarts that share a launch
FORM_BATCHES = [[(31000, 1)] * 9, [(31000, 1)] * 12, [(31000, 5)] * 2, [(40000, 1)] * 8 + [(31000, 1)],
                [(31000, 1), (33000, 4), (36000, 3), (45000, 2), (31500, 1), (30000, 2)]]


@pytest.mark.parametrize("batch", range(len(FORM_BATCHES)))
@pytest.mark.parametrize("schedule", [0, hm.CLUSTER])
def test_form_change_batch(batch, schedule):
    insts = FORM_BATCHES[batch]
    cnfs = [_cnf(n, seed=j) for j, (n, _) in enumerate(insts)]
    N = len(insts)
    kw = dict(steps=[70 + j for j in range(N)], restarts=[r for _, r in insts], seeds=list(range(3, 3 + N)))
    outs = hm.solve_batch(cnfs, schedule=schedule, eval_every=9, lr=1e-2, want_x=True, **kw)
    for j, (cnf, out) in enumerate(zip(cnfs, outs)):
        one = hm.solve(cnf, schedule=1, steps=kw["steps"][j], restarts=kw["restarts"][j], seed=kw["seeds"][j],
                       eval_every=9, lr=1e-2, want_x=True)
        _say(f"batch {batch} schedule {schedule} instance {j} {insts[j]}: schedule {out.schedule}, best {out.best_cost}")
        assert out.status == 0 and out.schedule == hm.CLUSTER
        _same(out, one)
        cnf.free()


def _solve_into(cnf, x, **kw):
    """hm.solve with x_T written over the start point `x` (a [n][R] tensor)."""
    import ctypes as C

    from paper_2402_03640_amd import _lib
    d = dict(steps=300, restarts=x.shape[1], eval_every=10, seed=0, optimizer=hm.ADAM, lr=1e-2, beta1=0.9, beta2=0.999,
             eps=1e-8, loss_mode=hm.LOSS_UNSAT, schedule=0, use_graph=True, time_limit_s=0.0, x0=x, stream=None,
             autotune=False)
    d.update(kw)
    p = _lib._params(cnf, **d)
    res = _lib.SolveResult()
    best = np.zeros(d["restarts"], dtype=np.int64)
    res.restart_best = best.ctypes.data
    res.x_final = x.data_ptr()
    _lib._check(_lib.lib().hms_solve(cnf.handle, C.byref(p), C.byref(res)))
    return res.schedule, best


def test_outputs_over_inputs_take_what_is_next_best():
    """A start point that receives x_T rules clusters out: small instances run
    on the resident solver, larger ones on the schedule that was timed."""
    for n, tuned in ((1000, False), (6000, True)):
        cnf = _cnf(n, ratio=4.2)
        x0 = torch.from_numpy(cnfgen.random_x(n, 2, seed=3)).cuda()
        kw = dict(steps=300, restarts=2, eval_every=10, lr=1e-2)
        ref = hm.solve(cnf, x0=x0, want_x=True, schedule=1, **kw)
        other = hm.RESIDENT
        if tuned:
            assert hm.tune(cnf, restarts=2)[0] == hm.CLUSTER
            other = hm.solve(cnf, time_limit_s=100.0, x0=x0, **kw).schedule
            assert other not in (hm.CLUSTER, hm.RESIDENT)
        assert hm.solve(cnf, x0=x0, autotune=False, **kw).schedule == hm.CLUSTER
        x = x0.clone()
        schedule, best = _solve_into(cnf, x)
        _say(f"n={n}: schedule {schedule} over the start point")
        assert schedule == other
        np.testing.assert_array_equal(best, ref.restart_best)
        np.testing.assert_array_equal(_bits(x), _bits(ref.x_final))
        cnf.free()


def test_time_limited_solve_leaves_the_timed_choice():
    """A solve that clusters cannot take (a time limit) uses the schedule timed
    next to them; it does not time again and put it in their place."""
    cnf = _cnf(8000, ratio=4.2)
    kw = dict(steps=300, restarts=9, eval_every=10)
    assert hm.tune(cnf, restarts=9)[0] == hm.CLUSTER
    a = hm.solve(cnf, time_limit_s=100.0, **kw)
    assert a.schedule != hm.CLUSTER
    assert hm.solve(cnf, **kw).schedule == hm.CLUSTER
    assert hm.solve(cnf, time_limit_s=100.0, **kw).schedule == a.schedule


def _beside(work, run):
    """run() while another thread repeats work(stream); stops it afterwards."""
    import threading
    errors, stop, turns = [], threading.Event(), []

    def loop():
        try:
            torch.cuda.set_device(0)
            st = torch.cuda.Stream()
            while not stop.is_set():
                work(st)
                turns.append(1)
        except BaseException as e:  # reported below, on the test's thread
            errors.append(repr(e))

    th = threading.Thread(target=loop)
    th.start()
    time.sleep(0.1)
    try:
        return run()
    finally:
        stop.set()
        th.join()
        _say("turns of the other thread:", len(turns))
        assert not errors, errors


def test_small_instances_beside_a_cluster_solve():
    """While another thread's solve holds the clusters, small instances take
    the resident solver, alone and in a batch."""
    big = _cnf(20000, ratio=4.2)
    small = [_cnf(1000 + 300 * j, ratio=4.2) for j in range(3)]
    kw = dict(steps=300, restarts=2, eval_every=10, lr=1e-2, want_x=True)
    ref = [hm.solve(c, schedule=1, seed=j, **kw) for j, c in enumerate(small)]
    ran = []

    def work(st):  # clusters, unless one of the small solves holds them at its start
        hm.solve(big, steps=15000, restarts=8, eval_every=50, autotune=False, stream=st)

    def run():
        st = torch.cuda.Stream()
        for _ in range(4):
            outs = [hm.solve(c, seed=j, stream=st, autotune=False, **kw) for j, c in enumerate(small)]
            outs += hm.solve_batch(small, seeds=[0, 1, 2], stream=st, **kw)
            for j, out in enumerate(outs):
                ran.append(out.schedule)
                _same(out, ref[j % 3])

    _beside(work, run)
    _say("schedules:", sorted(ran))
    assert set(ran) <= {hm.CLUSTER, hm.RESIDENT}


def test_clusters_that_do_not_fill():
    """Other work holds CUs of every XCD for longer than a cluster waits to
    fill: the registration is voided and the solve runs elsewhere."""
    other = _cnf(2500, ratio=4.2, seed=1)
    inst = [_cnf(2500, ratio=4.2, seed=2), _cnf(9000, ratio=4.2, seed=3)]
    kw = dict(steps=300, restarts=1, eval_every=10, lr=1e-2)
    ref = [hm.solve(c, schedule=1, seed=j, **kw) for j, c in enumerate(inst)]
    streams = [torch.cuda.Stream() for _ in range(4)]

    seconds = []

    def solves(st):
        t0 = time.perf_counter()
        outs = [hm.solve(c, schedule=hm.CLUSTER, seed=j, stream=st, **kw) for j, c in enumerate(inst)]
        seconds.append(time.perf_counter() - t0)
        return outs

    def hold(stream, steps=60000):  # 64 workgroups, eight on each XCD; too much LDS for a cluster's beside them
        r = hm.solve(other, steps=steps, restarts=64, eval_every=50, schedule=hm.RESIDENT, stream=stream)
        assert r.schedule == hm.RESIDENT

    for st in streams:
        assert [o.schedule for o in solves(st)] == [hm.CLUSTER] * 2
    hold(streams[0], 10)
    # a stream that shares a hardware queue with the other work runs behind it, the others beside it
    turns = _beside(hold, lambda: [solves(st) for st in streams])
    _say("schedules:", [[o.schedule for o in outs] for outs in turns])
    for outs in turns:
        for out, one in zip(outs, ref):
            np.testing.assert_array_equal(out.restart_best, one.restart_best)
            np.testing.assert_array_equal(out.restart_step, one.restart_step)
            np.testing.assert_array_equal(out.best_assignment, one.best_assignment)
            np.testing.assert_allclose(out.restart_loss, one.restart_loss, rtol=1e-12, atol=0)
    # each of the two waits no longer than the solve would take (2 ms here), well under a whole 20 ms
    _say("seconds:", seconds)
    assert min(seconds[-4:]) < 0.03
    voided = [outs for outs in turns if all(o.schedule != hm.CLUSTER for o in outs)]
    assert voided and all(outs[0].schedule == hm.RESIDENT and outs[1].schedule != hm.RESIDENT for outs in voided)


def test_few_steps_on_a_timed_handle():
    """A solve too short to make up for building the records takes the schedule
    timed next to clusters, also by the size class's timing."""
    n, R = 60000, 8
    lits = cnfgen.uniform_kcnf(n, int(4.2 * n), 3, seed=1)
    cnf, twin = hm.load_cnf(n, lits), hm.load_cnf(n, lits)
    assert hm.tune(cnf, restarts=R)[0] == hm.CLUSTER
    kw = dict(restarts=R, eval_every=10, lr=1e-2, seed=2, want_x=True)
    other = hm.solve(cnf, steps=100, time_limit_s=100.0, **kw).schedule
    for c in (cnf, twin):
        a, b = hm.solve(c, steps=1, **kw), hm.solve(c, steps=1, schedule=hm.CLUSTER, **kw)
        assert a.schedule == other and b.schedule == hm.CLUSTER
        _same(a, b)
        assert hm.solve(c, steps=100, **kw).schedule == hm.CLUSTER


def test_timing_beside_another_cluster_solve():
    """Timing waits for the clusters that another thread holds: the time is a
    step's, and clusters stay the timed choice."""
    big, cnf = _cnf(20000, ratio=4.2), _cnf(7000, ratio=4.2)
    alone = hm.time_kernels(cnf, restarts=5, iters=20, schedule=hm.CLUSTER)[2]

    def work(st):
        hm.solve(big, steps=3000, restarts=8, eval_every=50, autotune=False, stream=st)

    def run():
        st = torch.cuda.Stream()
        times = [hm.time_kernels(cnf, restarts=5, iters=20, schedule=hm.CLUSTER, stream=st)[2] for _ in range(5)]
        return times, hm.tune(cnf, restarts=5, stream=st)[0]

    times, code = _beside(work, run)
    _say("ms per step:", alone, times, "timed choice", code)
    assert all(0 < t < 1 for t in times)  # 1 ms: some hundred times a step's time
    assert code == hm.CLUSTER


def test_timing_many_iterations():
    """More iterations than a cluster solve has steps for are timed over fewer."""
    cnf = _cnf(130, ratio=4.2)
    assert 0 < hm.time_kernels(cnf, iters=100000, schedule=hm.CLUSTER)[2] < 1


def test_kernel_times_of_the_automatic_schedule():
    """hms_time_kernels with schedule 0 times the forward and the backward
    kernels, whatever the step count and also on a handle timed to clusters."""
    import ctypes as C

    from paper_2402_03640_amd import _lib
    cnf = _cnf(20000, ratio=4.2)
    f, b, st = C.c_double(), C.c_double(), C.c_double()
    p = _lib._params(cnf, 1000, 4, 50, 0, hm.ADAM, 1e-4, 0.9, 0.999, 1e-8, hm.LOSS_UNSAT, 0, False, 0.0, None, None,
                     False)
    for tuned in (False, True):
        if tuned:
            assert hm.tune(cnf, restarts=4)[0] == hm.CLUSTER
        _lib._check(_lib.lib().hms_time_kernels(cnf.handle, C.byref(p), 20, C.byref(f), C.byref(b), C.byref(st)))
        _say("ms:", f.value, b.value, st.value)
        assert f.value > 0 and b.value > 0 and st.value > 0
    assert hm.time_kernels(cnf, restarts=4, schedule=hm.CLUSTER)[:2] == (0.0, 0.0)


# (variables, clauses, literals, restarts, entry of the schedule table): the
# untimed choice on either side of its size limits
UNTIMED = [(20000, 86000, 3, 8, 39), (50000, 215000, 3, 8, 5), (20000, 86000, 3, 18, 35), (26000, 110000, 3, 18, 10),
           (12000, 50000, 3, 17, 6), (20000, 86000, 3, 17, 10), (20000, 86000, 3, 34, 35), (26000, 110000, 3, 34, 10),
           (50000, 215000, 3, 33, 14), (50000, 215000, 3, 36, 34)]


@pytest.mark.parametrize("n,m,k,R,entry", UNTIMED)
def test_untimed_schedule_of_several_restarts(n, m, k, R, entry):
    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, m, k, seed=1))
    # an optimizer that no other test times a schedule for (a size class shares its timing)
    kw = dict(steps=3, restarts=R, eval_every=2, lr=1e-2, optimizer=hm.SGD, want_x=True)
    a, b = hm.solve(cnf, autotune=False, **kw), hm.solve(cnf, schedule=1, **kw)
    assert a.schedule & 0xFF == entry
    _same(a, b)
    cnf.free()


# (variables, literals, clauses per variable, restarts, counting period, whether clusters are the untimed choice)
PERIODS = [(28000, 3, 4.3, 44, 1, True), (28000, 3, 4.3, 64, 1, False), (28000, 3, 4.3, 64, 2, True),
           (20000, 3, 4.3, 256, 1, True), (20000, 4, 5.0, 32, 1, True), (20000, 4, 5.0, 64, 1, False),
           (20000, 4, 5.0, 64, 2, True), (22000, 5, 4.0, 129, 1, False), (34000, 3, 4.2, 17, 1, False),
           (34000, 3, 4.2, 17, 4, True), (34000, 3, 4.2, 33, 4, False), (34000, 3, 4.2, 33, 16, True),
           (3000, 4, 5.0, 128, 1, True), (3000, 4, 5.0, 129, 1, False), (3000, 4, 5.0, 129, 4, True),
           (1000, 3, 4.3, 64, 1, True), (1000, 3, 4.3, 65, 1, False), (1000, 3, 4.3, 65, 2, True),
           (1200, 3, 4.3, 65, 1, True)]


@pytest.mark.parametrize("n,k,ratio,R,K,clusters", PERIODS)
def test_untimed_choice_by_counting_period(n, k, ratio, R, K, clusters):
    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, int(n * ratio), k, seed=1))
    assert cnf.info["n_heavy"] == 0
    out = hm.solve(cnf, steps=256, restarts=R, eval_every=K, optimizer=hm.SGD, autotune=False)
    assert (out.schedule == hm.CLUSTER) == clusters
    cnf.free()


def test_watched_solves_and_the_timed_choice():
    """A time limit or a cancel flag keeps a solve off the one-launch solvers, but
    not later solves of the handle: not when it is the first and times the
    schedules, nor where the resident solver is next to clusters."""
    cnf = _cnf(8000, ratio=4.2, seed=9)
    kw = dict(steps=300, restarts=7, eval_every=10)
    first = hm.solve(cnf, cancel=hm.CancelFlag(), **kw)
    assert first.schedule not in (hm.CLUSTER, hm.RESIDENT)
    assert hm.solve(cnf, **kw).schedule == hm.CLUSTER
    assert hm.solve(cnf, time_limit_s=100.0, **kw).schedule == first.schedule
    small = _cnf(2400, ratio=4.2, seed=9)
    kw = dict(steps=300, restarts=13, eval_every=1)
    best = hm.tune(small, restarts=13)[0]
    first = hm.solve(small, time_limit_s=100.0, **kw)
    assert first.schedule not in (hm.CLUSTER, hm.RESIDENT)
    assert hm.solve(small, **kw).schedule == best
    assert hm.solve(small, time_limit_s=100.0, **kw).schedule == first.schedule
    assert best in (hm.CLUSTER, hm.RESIDENT)


def test_more_restarts_than_memory_is_an_error():
    """A restart count that nothing can hold is refused at once, not listed on the
    host first."""
    import ctypes as C

    from paper_2402_03640_amd import _lib
    cnf = _cnf(9000, ratio=4.2)
    p = _lib._params(cnf, 300, 1 << 30, 50, 0, hm.SGD, 1e-2, 0.9, 0.999, 1e-8, hm.LOSS_UNSAT, 0, False, 0.0, None, None,
                     False)
    res = _lib.SolveResult()
    t0 = time.perf_counter()
    with pytest.raises(hm.HipMsatError):
        _lib._check(_lib.lib().hms_solve(cnf.handle, C.byref(p), C.byref(res)))
    assert time.perf_counter() - t0 < 10
    assert hm.solve(cnf, steps=300, eval_every=50, optimizer=hm.SGD, autotune=False).schedule == hm.CLUSTER
