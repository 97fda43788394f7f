"""Ingest of LPs with many columns and few entries."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")  # before libpsl, whose HIP runtime is then torch's
psl = pytest.importorskip("paper_2609_16182_amd.psl")


def lp_of(m, n, length=8, seed=0):
    """m rows of `length` entries at any columns; all columns boxed."""
    rng = np.random.default_rng(seed)
    ci = (rng.integers(0, n, (m, 1)) + np.arange(length) * (n // length)) % n
    ci.sort(axis=1)
    return dict(m=m, n=n, row_ptr=(np.arange(m + 1) * length).astype(np.int32), col_idx=ci.reshape(-1).astype(np.int32),
                val=rng.choice([-2.0, -1.0, 1.0, 3.0], m * length), lhs=np.full(m, -np.inf), rhs=np.full(m, 9.0),
                lb=np.zeros(n), ub=1.0 + rng.integers(0, 9, n), c=rng.integers(-3, 4, n).astype(float), obj_offset=0.0)


def on_gpu(lp):
    d = {k: torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v for k, v in lp.items()}
    d["nnz"] = len(lp["val"])
    torch.cuda.synchronize()
    return d


def ingest_ms(lp):
    d = on_gpu(lp)
    p = psl.Presolver(d)
    ms = []
    for _ in range(6):
        p.reload(d)
        p.run()
        ms.append(p.stats["ms_ingest"])
    p.close()
    return min(ms)


def test_few_entries_take_no_longer_than_many():
    """The work over the columns is spread over the chip, not over as many
    workgroups as the entries give: 2000 entries and 8e6 columns are ingested no
    slower than 4e6 entries and as many columns."""
    few, many = ingest_ms(lp_of(250, 8_000_000)), ingest_ms(lp_of(500_000, 8_000_000))
    assert few <= many, (few, many)


@pytest.mark.parametrize("m,n", [(1, 100_000), (250, 2047 * 2048), (250, 2048 * 2048 - 1), (250, 2048 * 2048 + 4096)])
def test_many_columns(m, n):
    """Column starts at the edges of the launch's workgroups (2048 of 2048)."""
    lp = lp_of(m, n, seed=n)
    out, p = psl.presolve(lp)
    p.close()
    assert_same(out, O.presolve(lp), f"{m} x {n}")


@pytest.mark.parametrize("at", [1, 2047, 2048, 5000])
@pytest.mark.parametrize("what", ["column", "order", "value"])
def test_lowest_invalid_entry_is_named(at, what):
    """Of two invalid entries the message names the lower one, in full."""
    lp = lp_of(1000, 1000, length=7)
    for p in (at, 6001):
        if what == "column":
            lp["col_idx"][p] = 1000
        elif what == "order":
            assert p % 7  # not a row's first entry
            lp["col_idx"][p] = lp["col_idx"][p - 1]
        else:
            lp["val"][p] = np.inf
    with pytest.raises(psl.PslError) as e:
        psl.presolve(lp)
    assert e.value.status == psl.PSL_ERR_INVALID
    assert f"(first at index {at})" in str(e.value)
