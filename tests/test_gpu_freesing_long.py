"""Free singletons of many long rows: more chunks of claiming and leaving rows than
the launches over their lists have workgroups."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

psl = pytest.importorskip("paper_2609_16182_amd.psl")


def lp_of(m, n, length, cost, seed=0):
    """m rows of `length` entries over n shared boxed columns, each with a free
    column of its own (a share `cost` of these with a cost)."""
    rng = np.random.default_rng(seed)
    ci = (rng.integers(0, n, (m, 1)) + rng.integers(1, n // length + 1, (m, 1)) * np.arange(length)) % n
    ci.sort(axis=1)
    ci = np.concatenate([ci, n + np.arange(m)[:, None]], 1)
    val = rng.choice([-2.0, -1.0, 1.0, 3.0], ci.shape)
    N = n + m
    lb, ub = np.concatenate([np.zeros(n), np.full(m, -np.inf)]), np.concatenate([rng.integers(1, 9, n), np.full(m, np.inf)])
    c = np.concatenate([rng.integers(-3, 4, n), (rng.random(m) < cost) * rng.integers(1, 4, m)]).astype(float)
    return dict(m=m, n=N, row_ptr=(np.arange(m + 1) * ci.shape[1]).astype(np.int32),
                col_idx=ci.reshape(-1).astype(np.int32), val=val.reshape(-1), lhs=np.full(m, -4.0),
                rhs=rng.integers(0, 9, m).astype(float), lb=lb, ub=ub, c=c, obj_offset=0.0)


@pytest.mark.parametrize("m,length", [(255, 40), (257, 40), (1023, 33), (1025, 40), (3000, 64), (700, 600)])
@pytest.mark.parametrize("cost", [0.0, 0.5, 1.0])
def test_many_long_rows(m, length, cost):
    lp = lp_of(m, 40 * m + 700, length, cost, seed=m)
    out, p = psl.presolve(lp, enable_free_singletons=1)
    ref = O.presolve(lp, enable_free_singletons=1)
    p.close()
    assert_same(out, ref, f"{m} rows of {length}, cost {cost}")
    assert (ref.records["type"] == O.REC["FREE_SINGLETON"]).sum() >= 25
