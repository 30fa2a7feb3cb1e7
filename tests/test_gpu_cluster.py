"""The cluster solver (whole loop in several workgroups of one XCD per
restart, exchanged through its L2): bit for bit the tiled kernels' solve, at
the sizes where its layout can go wrong."""
import sys
import threading

import numpy as np
import pytest

import cnfgen
import oracle as O

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


def _ragged(n, m, seed, kmax=5, spread=None):
    """Clauses of 0 to kmax literals with repeats and complementary pairs;
    `spread` limits the variables used (the rest stay in no clause)."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(m):
        k = int(rng.integers(0, kmax + 1))
        v = rng.integers(1, (spread or n) + 1, size=k)
        out.append([int(x) for x in v * np.where(rng.random(k) < 0.5, -1, 1)])
    return cnfgen.from_clauses(out)


# tile and list edges: 65 and 129 variables (one row in the last tile), lists
# of 7 to 17 records (a record block holds 8), one workgroup more than tiles
# allow; 1, 8, 9, 17, 33, 65 restarts (workgroups per restart 32 down to 4,
# and a second launch); 4096 and 4097 variables (t exchanged in words that carry
# their step, and behind flags), one tile per wavefront and several
CASES = [("uniform", 65, 300, 3, 1), ("uniform", 129, 520, 3, 9), ("uniform", 1000, 4200, 3, 17),
         ("uniform", 640, 2752, 4, 8), ("uniform", 300, 4000, 5, 33), ("mixed", 1000, 4200, 4, 65),
         ("uniform", 5000, 21500, 3, 2), ("two", 2000, 5000, 2, 3), ("ragged", 700, 3000, 5, 5),
         ("ragged3", 2500, 9000, 3, 4), ("sparse", 4000, 3000, 4, 2), ("uniform", 20000, 86000, 3, 64),
         ("uniform", 30000, 129000, 3, 18), ("uniform", 4096, 17600, 3, 1), ("uniform", 4097, 17600, 3, 1),
         ("mixed", 2050, 8600, 4, 16), ("uniform", 8200, 35000, 3, 9),
         # only the roundings in LDS: the first size past the 15-bit slots, ragged lists and clauses with
         # fewer literals than the record holds, fewer workgroups per restart, the largest number of tiles
         ("uniform", 32767, 120000, 3, 1), ("ragged", 40000, 170000, 5, 3), ("two", 50000, 90000, 2, 9),
         ("mixed", 36000, 150000, 4, 17), ("uniform", 34000, 200000, 5, 2), ("uniform", 63488, 200000, 3, 1)]


def _formula(kind, n, m, k, seed):
    if kind == "uniform":
        return cnfgen.uniform_kcnf(n, m, k, seed=seed)
    if kind == "two":
        return cnfgen.mixed_kcnf(n, m, seed=seed, ks=(1, 2))
    if kind == "mixed":
        return cnfgen.mixed_kcnf(n, m, seed=seed)
    if kind == "sparse":  # most variables in no clause
        return _ragged(n, m, seed, kmax=k, spread=n // 5)
    return _ragged(n, m, seed, kmax=k)


@pytest.mark.parametrize("kind,n,m,k,R", CASES)
@pytest.mark.parametrize("weighted", [False, True])
def test_cluster_equals_tiled(kind, n, m, k, R, weighted):
    if weighted and R == 64:
        pytest.skip("covered by the smaller cases")
    lits = _formula(kind, n, m, k, seed=n + k)
    w = None
    if weighted:
        rng = np.random.default_rng(n)
        w = rng.integers(1, 40, size=m).astype(np.int64)
        w[rng.integers(0, m, size=5)] = 5000  # hard clauses
    cnf = hm.load_cnf(n, lits, weights=w)
    assert cnf.info["n_heavy"] == 0
    kw = dict(steps=45, restarts=R, eval_every=7, seed=11, lr=1e-2, want_x=True)
    a = hm.solve(cnf, schedule=hm.CLUSTER, **kw)
    b = hm.solve(cnf, schedule=1, **kw)
    _say(f"{kind} n={n} m={m} R={R} weighted={weighted}: best {a.best_cost} (tiled {b.best_cost})")
    assert a.schedule == hm.CLUSTER and b.schedule & 0xFF == 1
    _same(a, b)
    cnf.free()


@pytest.mark.parametrize("kw", [dict(steps=0, eval_every=3), dict(steps=1, eval_every=1),
                                dict(steps=30, eval_every=1), dict(steps=30, eval_every=100),
                                dict(steps=25, eval_every=4, optimizer=hm.SGD, lr=0.3)])
def test_cluster_step_counts_and_optimizers(kw):
    """No step, one, counting every step or only at the end, plain gradient
    descent; x0 with the rounding's edge values (zeros of either sign,
    subnormals, large magnitudes, infinities)."""
    n, m, R = 400, 1700, 3
    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, m, 3, seed=5))
    x0 = torch.from_numpy(cnfgen.random_x(n, R, seed=3, specials=True)).cuda()
    kw = dict(dict(restarts=R, lr=1e-2, want_x=True, x0=x0, trace_cap=9), **kw)
    a, b = hm.solve(cnf, schedule=hm.CLUSTER, **kw), hm.solve(cnf, schedule=1, **kw)
    assert a.schedule == hm.CLUSTER
    _same(a, b)
    assert a.trace.shape == b.trace.shape
    np.testing.assert_array_equal(a.trace["step"], b.trace["step"])
    np.testing.assert_array_equal(a.trace["cost"], b.trace["cost"])
    np.testing.assert_allclose(a.trace["loss"], b.trace["loss"], rtol=1e-12)


@pytest.mark.parametrize("opt", [hm.ADAM, hm.SGD])
def test_cluster_resume_and_state(opt):
    """A solve cut in two, the pieces on different solvers: state, best and
    x_T as one uninterrupted tiled solve; variables in no clause keep theirs."""
    n, m, R = 900, 2600, 5
    cnf = hm.load_cnf(n, _ragged(n, m, 8, kmax=3, spread=700))
    kw = dict(restarts=R, eval_every=10, seed=3, lr=1e-2, optimizer=opt, want_state=True, want_x=True)
    full = hm.solve(cnf, steps=80, schedule=2, **kw)
    kw.pop("seed")
    for s1, s2 in ((hm.CLUSTER, 2), (2, hm.CLUSTER), (hm.CLUSTER, hm.CLUSTER)):
        a = hm.solve(cnf, steps=30, schedule=s1, seed=3, **kw)
        b = hm.solve(cnf, steps=50, schedule=s2, resume=a.state, **kw)
        _same(full, b)
        for key in ("x", "m", "v", "best_assignment"):
            ta, tb = getattr(full.state, key), getattr(b.state, key)
            assert (ta is None) == (tb is None)
            if ta is not None:
                np.testing.assert_array_equal(_bits(ta), _bits(tb), err_msg=key)
        np.testing.assert_array_equal(full.state.best, b.state.best)
        assert b.state.step == 80


def test_cluster_step_matches_oracle():
    """One step from x0 away from 0: counts equal the oracle's and the step is
    within the rounding of an FP32 update (as for the tiled schedules)."""
    n, m, R = 3000, 12900, 9
    lits = cnfgen.uniform_kcnf(n, m, 3, seed=4)
    rng = np.random.default_rng(6)
    x0 = (rng.uniform(0.05, 1.0, (n, R)) * np.where(rng.random((n, R)) < 0.5, -1, 1)).astype(np.float32)
    cnf = hm.load_cnf(n, lits)
    a = hm.solve(cnf, steps=1, restarts=R, eval_every=1, x0=torch.from_numpy(x0).cuda(), lr=0.2, optimizer=hm.SGD,
                 want_x=True, schedule=hm.CLUSTER)
    ro = O.OracleCNF(n, lits).solve(steps=1, restarts=R, eval_every=1, x0=x0, lr=0.2, optimizer=O.SGD, want_x=True)
    np.testing.assert_array_equal(a.restart_best, ro["restart_best"])
    d_g = a.x_final.cpu().numpy().astype(np.float64) - x0
    d_o = ro["x"].reshape(n, R) - x0
    assert np.all(np.abs(d_g - d_o) <= 1e-5 * np.abs(d_o) + 2e-7 * np.abs(x0) + 1e-12)


def test_cluster_choice_and_refusals():
    """Solves of 64 steps or more take it by themselves; what it cannot run is
    refused when asked for by id and runs on other schedules otherwise."""
    n, m = 6000, 25800
    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, m, 3, seed=2))
    assert hm.solve(cnf, steps=64, eval_every=10, autotune=False).schedule == hm.CLUSTER
    assert hm.solve(cnf, steps=63, eval_every=10, autotune=False).schedule != hm.CLUSTER
    assert hm.solve(cnf, steps=64, eval_every=10, loss_mode=hm.LOSS_ALL, autotune=False).schedule != hm.CLUSTER
    assert hm.solve(cnf, steps=64, eval_every=10, time_limit_s=100.0, autotune=False).schedule != hm.CLUSTER
    assert hm.solve(cnf, steps=64, eval_every=10, cancel=hm.CancelFlag(), autotune=False).schedule != hm.CLUSTER
    for kw in (dict(loss_mode=hm.LOSS_ALL), dict(time_limit_s=10.0), dict(steps=(1 << 20) + 1)):
        with pytest.raises(hm.HipMsatError):
            hm.solve(cnf, **dict(dict(steps=4, schedule=hm.CLUSTER), **kw))
    heavy = hm.load_cnf(3000, cnfgen.structured_cnf(3000, 15000, seed=4))  # split rows
    long = hm.load_cnf(500, cnfgen.uniform_kcnf(500, 300, 6, seed=4))      # six literals
    wide = hm.load_cnf(63489, cnfgen.uniform_kcnf(63489, 400000, 3, seed=4))  # more variables than the widest form
    big = hm.load_cnf(500, cnfgen.uniform_kcnf(500, 2000, 3, seed=4), weights=np.full(2000, 1 << 22, np.int64))
    for c in (heavy, long, wide, big):
        with pytest.raises(hm.HipMsatError):
            hm.solve(c, steps=4, schedule=hm.CLUSTER)
        assert hm.solve(c, steps=70, eval_every=10, autotune=False).schedule != hm.CLUSTER


def test_cluster_concurrent_threads():
    """Solves on several threads at once: one holds the device's clusters, the
    others take tiled kernels; every result is the one it gets alone."""
    inst = [(2000 + 900 * i, cnfgen.uniform_kcnf(2000 + 900 * i, 9000 + 4000 * i, 3, seed=i)) for i in range(4)]
    cnfs = [hm.load_cnf(n, lits) for n, lits in inst]
    kw = dict(steps=150, restarts=3, eval_every=10, seed=3, lr=1e-2, want_x=True, autotune=False)
    solo = [hm.solve(c, schedule=1, **kw) for c in cnfs]
    errors, ran = [], []

    def run(i):
        try:
            torch.cuda.set_device(0)
            st = torch.cuda.Stream()
            for _ in range(4):
                r = hm.solve(cnfs[i], stream=st, **kw)
                ran.append(r.schedule)
                _same(r, solo[i])
        except BaseException as e:  # reported below, on the test's thread
            errors.append(f"instance {i}: {e!r}")

    th = [threading.Thread(target=run, args=(i,)) for i in range(len(cnfs))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    _say("schedules:", sorted(ran))
    assert not errors, errors
    assert hm.CLUSTER in ran


# (kind, n, k, restarts) of the batch's instances: one form and one kernel
# (words, flags), several kernels' sizes in one form, several forms, more
# restarts than one launch holds, and instances that run elsewhere
BATCHES = [
    [("uniform", 600 + 150 * i, 3, 1 + i % 3) for i in range(5)],
    [("uniform", n, 3, 1) for n in (5000, 9000, 12000)],
    [("uniform", n, 3, R) for n, R in ((20000, 1), (15500, 1), (16700, 2), (900, 4), (26000, 1), (5000, 1))],
    [("uniform", 3000, 3, 1), ("mixed", 2000, 4, 2), ("uniform", 700, 4, 3), ("uniform", 1500, 5, 1),
     ("mixed", 5000, 4, 1), ("two", 9000, 2, 1)],
    [("uniform", 20000, 3, 70), ("uniform", 8000, 3, 90)],
    [("uniform", 140000, 3, 1), ("uniform", 18000, 3, 1), ("uniform", 150, 3, 2), ("uniform", 21000, 3, 1),
     ("uniform", 33000, 3, 2), ("uniform", 41000, 3, 1)],
]


@pytest.mark.parametrize("batch", range(len(BATCHES)))
@pytest.mark.parametrize("schedule", [0, hm.CLUSTER])
def test_cluster_batch_equals_single(batch, schedule):
    """A batch's cluster solves share launches: each result is the tiled
    solve's bit for bit, with its own steps, period, rate and optimizer."""
    insts = BATCHES[batch]
    cnfs, w = [], None
    for j, (kind, n, k, R) in enumerate(insts):
        m = int(n * {2: 2.0, 3: 4.2, 4: 6.0, 5: 12.0}[k])
        if batch == 3 and j in (0, 4):
            w = np.random.default_rng(j).integers(1, 30, size=m).astype(np.int64)
        cnfs.append(hm.load_cnf(n, _formula(kind, n, m, k, seed=n), weights=w))
        w = None
    N = len(insts)
    kw = dict(steps=[256 + 3 * j for j in range(N)], restarts=[i[3] for i in insts], eval_every=[1 + 6 * j for j in range(N)],
              seeds=list(range(5, 5 + N)), lr=[1e-2 / (1 + j) for j in range(N)],
              optimizer=[hm.SGD if j == 1 else hm.ADAM for j in range(N)])
    outs = hm.solve_batch(cnfs, schedule=schedule, want_x=True, **kw)
    for j, (cnf, out) in enumerate(zip(cnfs, outs)):
        one = hm.solve(cnf, schedule=1, want_x=True, seed=kw["seeds"][j],
                       **{key: kw[key][j] for key in ("steps", "restarts", "eval_every", "lr", "optimizer")})
        _say(f"batch {batch} schedule {schedule} instance {j} {insts[j]}: schedule {out.schedule}, best {out.best_cost}")
        assert out.status == 0
        _same(out, one)
        big = insts[j][1] > 63488
        assert out.schedule != hm.CLUSTER if big else out.schedule == hm.CLUSTER or insts[j][1] < 3000
        cnf.free()
