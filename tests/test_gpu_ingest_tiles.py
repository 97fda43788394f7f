"""The ingest's launches at the edges of their tiles, and what they report.

Rows are listed in tiles of 1024, positions in tiles of 2048 whose rows are
found by search; runs of empty rows, long rows over many tiles and invalid
entries in any tile are compared with the CPU oracle bit for bit.
"""
import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")  # before libpsl, whose HIP runtime is then torch's
psl = pytest.importorskip("paper_2609_16182_amd.psl")


def lp_of_lengths(lengths, n, seed=0):
    rng = np.random.default_rng(seed)
    lengths = np.minimum(np.asarray(lengths, np.int64), n)
    m, nnz = len(lengths), int(lengths.sum())
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    start = (rng.integers(0, n, m) % np.maximum(1, n - lengths + 1))
    ci = (np.arange(nnz) - np.repeat(rp[:-1], lengths) + np.repeat(start, lengths)).astype(np.int32)
    lhs = np.where(rng.random(m) < 0.5, -np.inf, -50.0 - lengths)
    return dict(m=m, n=n, row_ptr=rp, col_idx=ci, val=rng.choice([-2.0, -1.0, 1.0, 3.0], nnz), lhs=lhs,
                rhs=60.0 + lengths, lb=np.where(rng.random(n) < 0.3, -np.inf, -1.0 * rng.integers(0, 5, n)),
                ub=1.0 + rng.integers(0, 9, n), c=rng.integers(-3, 4, n).astype(float), obj_offset=0.0)


def lengths_of(kind):
    rng = np.random.default_rng(7)
    if kind == "one tile":
        return [1] * 2047 + [1]
    if kind == "a tile and one":
        return [3] * 683
    if kind == "rows across tiles":
        return rng.integers(1, 700, 300)
    if kind == "a long row":
        return [5, 0, 9000, 0, 0, 4, 2048, 1]
    if kind == "empty rows between":
        x = np.zeros(120000, np.int64)
        x[[0, 60000, 119999]] = 3  # one tile, 120000 rows: searched per position
        return x
    if kind == "empty rows at the ends":
        return [0] * 3000 + [4] * 1500 + [0] * 3000
    return [0] * 1025  # no entries


@pytest.mark.parametrize("mem", ["host", "device"])
@pytest.mark.parametrize("kind", ["one tile", "a tile and one", "rows across tiles", "a long row",
                                  "empty rows between", "empty rows at the ends", "no entries"])
def test_tiles(kind, mem):
    lp = lp_of_lengths(lengths_of(kind), 9500)
    if mem == "device":
        dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() if isinstance(v, np.ndarray) else v
               for k, v in lp.items()}
        torch.cuda.synchronize()
        out, p = psl.presolve(dev)
    else:
        out, p = psl.presolve(lp)
    p.close()
    assert_same(out, O.presolve(lp), f"{kind} {mem}")


@pytest.mark.parametrize("at", [0, 2047, 2048, 5000])
@pytest.mark.parametrize("what", ["column", "order", "value"])
def test_first_invalid_entry(at, what):
    """The lowest invalid position is reported, whichever tile sees it first."""
    lp = lp_of_lengths([7] * 1000, 1000)
    for p in (at, 6001):
        if what == "column":
            lp["col_idx"][p] = 1000
        elif what == "order" and p % 7:
            lp["col_idx"][p] = lp["col_idx"][p - 1]
        else:
            lp["val"][p] = np.nan
    with pytest.raises(psl.PslError) as e:
        psl.presolve(lp)
    assert str(at) in str(e.value)


@pytest.mark.parametrize("m,n", [(2047, 2049), (2048, 2048), (4096, 63), (64, 4097)])
def test_reduced_problem_tiles(m, n):
    """Kept rows, columns and entries are ranked in tiles of 2048, 64 to a word."""
    rng = np.random.default_rng(m)
    lp = lp_of_lengths(rng.integers(0, 5, m), n, seed=n)
    fixed = rng.random(n) < 0.3
    lp["ub"] = np.where(fixed & np.isfinite(lp["lb"]), lp["lb"], lp["ub"])
    out, p = psl.presolve(lp, max_rounds=1, max_outer=1)
    p.close()
    assert_same(out, O.presolve(lp, max_rounds=1, max_outer=1), f"{m} x {n}")
