"""A device array shorter than its LP needs is refused, not read past its end.

The array is an allocation of its own of 800 bytes; the LP claims 3200 bytes of it,
so that even a read past its end would stay in the allocation's page.
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")  # before libpsl, whose HIP runtime is then torch's
psl = pytest.importorskip("paper_2609_16182_amd.psl")

M, LEN = 100, 4  # 400 entries: 1600 bytes of columns, 3200 of values


@pytest.fixture
def short():
    hip = psl._hiprt()
    q = C.c_void_p()
    hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    hip.hipFree.argtypes = [C.c_void_p]
    assert hip.hipMalloc(C.byref(q), 800) == 0
    yield q
    hip.hipGetLastError()  # of the refused copy
    assert hip.hipFree(q) == 0


def lp_struct(keep):
    ci = np.arange(M * LEN) % LEN
    lp = dict(m=M, n=M * LEN, row_ptr=np.arange(0, M * LEN + 1, LEN, dtype=np.int32), col_idx=ci.astype(np.int32),
              val=np.ones(M * LEN), lhs=np.full(M, -np.inf), rhs=np.full(M, 9.0), lb=np.zeros(M * LEN),
              ub=np.ones(M * LEN), c=np.ones(M * LEN))
    dev = {k: torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v for k, v in lp.items()}
    torch.cuda.synchronize()
    return psl.make_lp(dev, keep)


@pytest.mark.parametrize("field", ["val", "lb", "ub", "c", "col_idx"])
def test_short_array_is_refused(short, field):
    keep = []
    lp = lp_struct(keep)
    setattr(lp, field, short.value)
    with pytest.raises(psl.PslError) as e:
        psl.psl_presolve_create(lp, psl.make_settings())
    assert e.value.status == psl.PSL_ERR_DEVICE


def test_reload_with_a_short_array_then_a_whole_one(short):
    keep = []
    good = lp_struct(keep)
    h = psl.psl_presolve_create(good, psl.make_settings())
    bad = lp_struct(keep)
    bad.val = short.value
    with pytest.raises(psl.PslError) as e:
        psl.psl_presolve_reload(h, bad)
    assert e.value.status == psl.PSL_ERR_DEVICE
    psl._hiprt().hipGetLastError()
    psl.psl_presolve_reload(h, good)
    assert psl.psl_presolve_run(h)[0] is not None
    psl.psl_presolve_free(h)
