"""LPs with far more rows than rows with entries.

Up to 500000 nonzeros a sweep tests each row itself, and up to 4e6 rounds are
queued ahead with grids of all rows; both only where the rows are not many more
than the entries. Parity on both sides of the limits on the rows, and the time of an
LP that only the limit on the rows keeps off a path against one that the limit on the
nonzeros keeps off it.
"""
import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")  # before libpsl, whose HIP runtime is then torch's
psl = pytest.importorskip("paper_2609_16182_amd.psl")


def lp_of(m, full, length, n, seed=0):
    """m rows, `full` of them with entries (at random places), met by a point."""
    rng = np.random.default_rng(seed)
    lens = np.zeros(m, np.int64)
    lens[rng.choice(m, full, replace=False)] = length
    rp = np.concatenate([[0], np.cumsum(lens)])
    ci = ((rng.integers(0, n, (full, 1)) + np.arange(length) * (n // length)) % n)
    ci.sort(axis=1)
    val = rng.choice([-2.0, -1.0, 1.0, 3.0], full * length)
    lb = np.where(rng.random(n) < 0.3, -np.inf, -1.0 * rng.integers(0, 5, n))
    ub = 1.0 + rng.integers(0, 9, n)
    x0 = np.floor(np.maximum(lb, -3.0) + rng.random(n) * (ub - np.maximum(lb, -3.0)))
    act = np.zeros(m)
    act[lens > 0] = (val.reshape(full, length) * x0[ci]).sum(1)
    return dict(m=m, n=n, row_ptr=rp.astype(np.int32), col_idx=ci.reshape(-1).astype(np.int32), val=val,
                lhs=np.where(rng.random(m) < 0.5, -np.inf, act - rng.integers(0, 9, m)), rhs=act + rng.integers(0, 9, m),
                lb=lb, ub=ub, c=np.where(np.isinf(lb), 0.0, rng.integers(-3, 4, n)), obj_offset=0.0)


@pytest.mark.parametrize("m,full", [(700_000, 5000), (700_001, 5000), (3_000_000, 70_000), (3_000_001, 70_000)])
@pytest.mark.parametrize("options", [{}, dict(enable_free_singletons=1, enable_dual_fix=1)])
def test_parity_at_the_limits(m, full, options):
    lp = lp_of(m, full, 8, 3 * full // 2, seed=m)
    out, p = psl.presolve(lp, **options)
    p.close()
    assert_same(out, O.presolve(lp, **options), f"{m} rows {options}")


def run_ms(lp):
    d = {k: torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v for k, v in lp.items()}
    d["nnz"] = len(lp["val"])
    torch.cuda.synchronize()
    p = psl.Presolver(d, max_outer=1)
    ms = []
    for _ in range(7):
        p.reload(d)
        p.run()
        ms.append(p.stats["ms_total"])
    rounds = p.stats["rounds"]
    p.close()
    return min(ms), rounds


@pytest.mark.parametrize("m,few,many", [(4_000_000, 60_000, 64_000), (30_000_000, 490_000, 510_000)])
def test_no_slower_than_with_more_entries(m, few, many):
    """8 entries in 60000 or 490000 rows are below a limit on the nonzeros, a few
    percent more are beyond it. Per round the smaller LP takes no longer than the
    larger one (15% for what two runs differ by)."""
    a, ra = run_ms(lp_of(m, few, 8, 3 * few // 2))
    b, rb = run_ms(lp_of(m, many, 8, 3 * few // 2))
    assert a / ra <= 1.15 * b / rb, (a, ra, b, rb)
