"""Device memory of the differentiable forward and backward: the clause
adjoints are in the caller's buffer, not in the workspace a second time."""
import ctypes as C

import pytest

import cnfgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hm = pytest.importorskip("paper_2402_03640_amd")

USED_MEM_HIGH = 8  # hipMemPoolAttrUsedMemHigh


def _high(pool, call):
    """Most bytes in use in the library's memory pool during the call."""
    L = hm.lib()
    torch.cuda.synchronize()
    v = C.c_uint64(0)
    assert L.hipMemPoolSetAttribute(pool, USED_MEM_HIGH, C.byref(v)) == 0
    call()
    torch.cuda.synchronize()
    assert L.hipMemPoolGetAttribute(pool, USED_MEM_HIGH, C.byref(v)) == 0
    return v.value


@pytest.mark.parametrize("n,m,k,R", [(20000, 86000, 3, 33), (20000, 86000, 3, 64), (12000, 60000, 5, 5)])
def test_adjoint_is_not_laid_out_twice(n, m, k, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_03640_amd.autograd import adjoint_bytes, maxsat_loss

    cnf = hm.load_cnf(n, cnfgen.uniform_kcnf(n, m, k, seed=n + R))
    pool = C.c_void_p()
    L = hm.lib()
    L.hipMemPoolSetAttribute.argtypes = L.hipMemPoolGetAttribute.argtypes = [C.c_void_p, C.c_int, C.c_void_p]
    assert L.hipDeviceGetDefaultMemPool(C.byref(pool), torch.cuda.current_device()) == 0
    gen = torch.Generator(device="cuda").manual_seed(R)
    x = (torch.rand(n, R, device="cuda", generator=gen) * 2 - 1).requires_grad_(True)
    out = {}

    def forward(checkpoint):
        out["loss"] = maxsat_loss(cnf, x, checkpoint=checkpoint)[0].sum()

    def backward():
        x.grad = None
        out["loss"].backward()

    adj = adjoint_bytes(cnf, R)
    high = {}
    for checkpoint in (False, True):
        high[checkpoint] = (_high(pool, lambda: forward(checkpoint)), _high(pool, backward))
        out[checkpoint] = x.grad.clone()
    # without the checkpoint both passes do without the adjoints that they need with it
    # (a quarter of them for what the pool may round a block up by)
    for kept, made in zip(high[False], high[True]):
        assert 0 < kept <= made - 0.75 * adj
    assert torch.equal(out[False], out[True])
