"""The evaluation's two routes, one launch with a workgroup per point (small
instances) and the tiled passes: points and gradients go straight between the
caller's arrays, so alignment, overlap and variables in no clause matter."""
import sys

import numpy as np
import pytest

import cnfgen
import oracle as O
from _helpers import assert_eval_parity, w_abs_matrix

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hm = pytest.importorskip("paper_2402_03640_amd")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hm.lib()
    yield
    torch.cuda.synchronize()


# (n, m, k, variables used, R): one tile, a workgroup of four wavefronts and of
# sixteen, just below and above the small route's 2^16 nonzeros; restart counts
# of every schedule rule (up to 8, multiples of four to 16 and beyond, even, odd)
CASES = [(3, 5, 2, 3, 1), (60, 250, 3, 50, 7), (300, 900, 3, 300, 64), (5000, 21845, 3, 4000, 3),
         (5000, 21900, 3, 4000, 8), (6000, 25000, 3, 5000, 12), (6000, 25000, 3, 5000, 16), (6000, 25000, 3, 5500, 20),
         (6000, 25000, 3, 6000, 17), (6000, 25000, 3, 6000, 18)]


def _inst(n, m, k, used):
    lits = cnfgen.uniform_kcnf(used, m, k, seed=n + m)  # variables past `used` are in no clause
    return lits, hm.load_cnf(n, lits)


@pytest.mark.parametrize("n,m,k,used,R", CASES)
@pytest.mark.parametrize("mode", [hm.LOSS_UNSAT, hm.LOSS_ALL])
def test_eval_alignment_and_overlap(n, m, k, used, R, mode):
    lits, cnf = _inst(n, m, k, used)
    x = cnfgen.random_x(n, R, seed=7, lo=-2, hi=2, specials=True)
    xt = torch.from_numpy(x).cuda()
    loss, g, u = hm.eval_relaxed(cnf, xt, loss_mode=mode)
    assert_eval_parity(O.OracleCNF(n, lits), w_abs_matrix(n, lits), x, loss, g.cpu().numpy(), u, mode)
    ref = g.cpu().numpy().view(np.uint32)
    # points and gradients four bytes off a 16-byte boundary
    b1, b2 = torch.zeros(n * R + 1, device="cuda"), torch.full((n * R + 1,), 9.0, device="cuda")
    xo, go = b1[1:].view(n, R), b2[1:].view(n, R)
    xo.copy_(xt)
    l2, g2, u2 = hm.eval_relaxed(cnf, xo, loss_mode=mode, grad_out=go)
    np.testing.assert_array_equal(g2.cpu().numpy().view(np.uint32), ref)
    np.testing.assert_array_equal(u2, u)
    np.testing.assert_array_equal(l2, loss)
    assert float(b2[0]) == 9.0
    # gradients over the points themselves, and over all but the first
    same = xt.clone()
    hm.eval_relaxed(cnf, same, loss_mode=mode, grad_out=same)
    np.testing.assert_array_equal(same.cpu().numpy().view(np.uint32), ref)
    buf = torch.zeros(n * R + 1, device="cuda")
    src, dst = buf[:-1].view(n, R), buf[1:].view(n, R)
    src.copy_(xt)
    hm.eval_relaxed(cnf, src, loss_mode=mode, grad_out=dst)
    np.testing.assert_array_equal(dst.cpu().numpy().view(np.uint32), ref)
    # without the gradient
    l3, none, u3 = hm.eval_relaxed(cnf, xt, loss_mode=mode, want_grad=False)
    assert none is None
    np.testing.assert_array_equal(u3, u)
    np.testing.assert_array_equal(l3, loss)


@pytest.mark.parametrize("R", [1, 4, 16, 33])
def test_autograd_gradient_equals_eval(R):
    """The saved-adjoint and the recomputing backward give the evaluation's
    gradient bit for bit; variables in no clause get scale * 0."""
    from paper_2402_03640_amd.autograd import maxsat_loss
    n, m, used = 4000, 16000, 3500
    _, cnf = _inst(n, m, 3, used)
    x = torch.from_numpy(cnfgen.random_x(n, R, seed=1)).cuda()
    _, g, _ = hm.eval_relaxed(cnf, x)
    for checkpoint in (False, True):
        xt = x.clone().requires_grad_(True)
        loss, _ = maxsat_loss(cnf, xt, checkpoint=checkpoint)
        loss.sum().backward()
        np.testing.assert_array_equal(xt.grad.cpu().numpy().view(np.uint32), g.cpu().numpy().view(np.uint32))
        xt.grad = None
        loss, _ = maxsat_loss(cnf, xt, checkpoint=checkpoint)
        (loss * float("inf")).sum().backward()
        assert torch.isnan(xt.grad[used + 1:]).all()


def test_results_with_more_points_than_the_pinned_memory():
    """More points than one piece of pinned host memory holds (512) are copied
    back instead: same values as point by point."""
    n, m, R = 40, 170, 515
    _, cnf = _inst(n, m, 3, n)
    x = torch.from_numpy(cnfgen.random_x(n, R, seed=2)).cuda()
    loss, g, u = hm.eval_relaxed(cnf, x)
    for r in (0, 511, 514):
        l1, g1, u1 = hm.eval_relaxed(cnf, x[:, r].contiguous())
        assert u1[0] == u[r]
        np.testing.assert_allclose(l1[0], loss[r], rtol=1e-13)
        np.testing.assert_array_equal(g1.cpu().numpy().view(np.uint32).ravel(),
                                      g[:, r].contiguous().cpu().numpy().view(np.uint32))


# more points than the pinned memory holds (512); the last sizes of the one-launch route and the first past it (6 or,
# up to 512 points, 12 times 2^16 values of x; 256 tiles of clauses); no clause at all
NOALLOC = [(40, 170, 512), (40, 170, 513), (128, 200, 3072), (128, 200, 3073), (640, 2700, 614), (640, 2700, 615),
           (1536, 6450, 512), (1537, 6450, 512), (3900, 16384, 3), (3900, 16385, 3), (40, 0, 515),
           # the fixed workspace holds them only with fewer restarts per group
           (40000, 176000, 34), (40000, 176000, 33)]


@pytest.mark.parametrize("n,m,R", NOALLOC)
@pytest.mark.parametrize("mode", [hm.LOSS_UNSAT, hm.LOSS_ALL])
def test_noalloc_equals_eval_bitwise(n, m, R, mode):
    """With and without allocation: the same loss, gradient and counts, bit for
    bit, with results in pinned memory or copied; each output may be left out."""
    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, m, 3, seed=n + m) if m else np.zeros(0, np.int32))
    x = torch.from_numpy(cnfgen.random_x(n, R, seed=4, lo=-2, hi=2)).cuda()
    loss, g, u = hm.eval_relaxed(cnf, x, loss_mode=mode)
    dl = torch.full((R,), -1.0, dtype=torch.float64, device="cuda")
    du = torch.full((R,), -1, dtype=torch.int64, device="cuda")
    dg = torch.full((n, R), 9.0, device="cuda")
    hm.eval_relaxed_noalloc(cnf, x, loss_out=dl, grad_out=dg, unsat_out=du, loss_mode=mode)
    np.testing.assert_array_equal(dl.cpu().numpy().view(np.uint64), loss.view(np.uint64))
    np.testing.assert_array_equal(du.cpu().numpy(), u)
    np.testing.assert_array_equal(dg.cpu().numpy().view(np.uint32), g.cpu().numpy().view(np.uint32))
    l2, none, u2 = hm.eval_relaxed(cnf, x, loss_mode=mode, want_grad=False)
    assert none is None
    np.testing.assert_array_equal(l2.view(np.uint64), loss.view(np.uint64))
    np.testing.assert_array_equal(u2, u)
    dg.fill_(9.0)
    hm.eval_relaxed_noalloc(cnf, x, grad_out=dg, loss_mode=mode)
    np.testing.assert_array_equal(dg.cpu().numpy().view(np.uint32), g.cpu().numpy().view(np.uint32))
