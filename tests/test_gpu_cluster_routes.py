"""Which solver runs when clusters are the choice: one kernel form per launch at
the sizes where the form changes, and what takes over where clusters cannot
run.  Every result is the tiled solve's, bit for bit."""
import sys

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
