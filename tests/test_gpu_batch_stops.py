"""Batches whose members stop in the middle of the rounds.

An LP found infeasible by one of its rows still has every row of that round
swept, whatever the order in which the rows run: its records are those it has
alone. The stopping members have thousands of rows over all bins, most of which
leave or tighten a bound in the round that finds the LP infeasible; the batches
lie on both sides of the 500000 nonzeros up to which a sweep tests each row
itself. Every member is compared bit for bit with the CPU oracle.
"""
import functools

import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

psl = pytest.importorskip("paper_2609_16182_amd.psl")

INF = np.inf
# Rows of each length: every bin, and rows of several chunks. The many rows of 17
# entries, four to a workgroup, are several times what the chip holds at once.
SHORT = ((3, 1500), (7, 1000), (14, 600), (17, 18000), (200, 100), (400, 20))
LONG = SHORT + ((2500, 4),)
SMALL = ((3, 300), (7, 200), (14, 100), (17, 900), (200, 10), (400, 2))


@functools.lru_cache(maxsize=None)
def member(seed, rows, stop=0, at="first"):
    """Boxed columns, rows of the given lengths that a point meets: 60% redundant,
    the others tighten. stop = 1 adds a row that cannot be met; 2 a row that
    cannot once two rows of one entry have raised its columns' bounds. `at`: that
    row's place."""
    rng = np.random.default_rng(seed)
    n = 3000
    lens = np.repeat([k for k, _ in rows], [c for _, c in rows])
    rng.shuffle(lens)
    ub = rng.integers(1, 10, n).astype(float)
    x0 = np.floor(ub * rng.random(n))
    r = []  # (columns, coefficients, lhs, rhs)
    for k in lens:
        j = (rng.integers(n) + rng.integers(1, n // k + 1) * np.arange(k)) % n
        j.sort()
        a = rng.choice([-2.0, -1.0, 1.0, 2.0], k)
        lo, up = np.minimum(a, 0) @ ub[j], np.maximum(a, 0) @ ub[j]
        side = max(a @ x0[j], np.floor(lo + rng.uniform(0.1, 0.9) * (up - lo)))
        r.append((j, a, -INF, up + 1.0 if rng.random() < 0.6 else side))
    if stop:
        j, one = np.array([0, 1]), np.ones(2)
        ub[:2] = 9.0
        bad = [(j, one, 100.0, INF)] if stop == 1 else [(j, one, -INF, 8.0)]
        if stop == 2:
            r[len(r) // 2:len(r) // 2] = [(j[:1], one[:1], 5.0, INF), (j[1:], one[:1], 5.0, INF)]
        r = bad + r if at == "first" else r + bad
    return dict(m=len(r), n=n, row_ptr=np.concatenate([[0], np.cumsum([len(x[0]) for x in r])]).astype(np.int32),
                col_idx=np.concatenate([x[0] for x in r]).astype(np.int32), val=np.concatenate([x[1] for x in r]),
                lhs=np.array([x[2] for x in r]), rhs=np.array([x[3] for x in r], float), lb=np.zeros(n), ub=ub,
                c=rng.integers(-3, 4, n).astype(float), obj_offset=0.0)


def check(lps, label, **settings):
    refs = [O.presolve(lp, **settings) for lp in lps]
    b = psl.Batch(lps, **settings)
    for rep in range(3):  # the order in which workgroups run differs from run to run
        if rep:
            b.reload(lps)
        names = b.run()
        for k, ref in enumerate(refs):
            got = {"result_name": names[k], "records": b.records(k),
                   "reduced": b.reduced(k) if names[k] in ("REDUCED", "UNCHANGED") else None}
            assert_same(got, ref, f"{label} LP {k} run {rep}")
            st = b.lp_stats(k)
            assert st["rounds"] == ref.rounds and st["records"] == len(ref.records)
        assert b.stats["records"] == sum(len(ref.records) for ref in refs)
    b.close()
    return names


@pytest.mark.parametrize("at", ["first", "last"])
@pytest.mark.parametrize("stop", [1, 2])
@pytest.mark.parametrize("rows", [SHORT, LONG], ids=["short", "long"])
@pytest.mark.parametrize("side", ["direct", "selected"])
def test_infeasible_members(side, rows, stop, at):
    lps = [member(1, rows, stop, at), member(2, SMALL), member(3, SMALL, 3 - stop, at)]
    if side == "selected":
        lps += [member(4, SHORT, stop, at)]
    nnz = sum(len(lp["val"]) for lp in lps)
    assert nnz < 500000 if side == "direct" else nnz > 500000, nnz
    names = check(lps, f"{side} {stop} {at}")
    assert names[:3] == ["INFEASIBLE", "REDUCED", "INFEASIBLE"]


@pytest.mark.parametrize("stop", [1, 2])
def test_infeasible_members_with_options(stop):
    lps = [member(1, LONG, stop), member(2, SMALL), member(3, SMALL, stop, "last")]
    check(lps, f"options {stop}", enable_dual_fix=1, enable_free_singletons=1, enable_forcing_rows=1)


def few_rows(seed):
    """An LP of one to three rows over a few columns; a third of them cannot be met."""
    rng = np.random.default_rng(seed)
    m, n = 1 + seed % 3, 4
    return dict(m=m, n=n, row_ptr=np.arange(0, 3 * m + 1, 3).astype(np.int32),
                col_idx=np.concatenate([np.sort(rng.choice(n, 3, replace=False)) for _ in range(m)]).astype(np.int32),
                val=rng.choice([-1.0, 1.0, 2.0], 3 * m), lhs=np.where(rng.random(m) < 0.3, 9.0, -INF),
                rhs=np.full(m, 9.0), lb=np.zeros(n), ub=rng.integers(1, 6, n).astype(float), c=np.ones(n),
                obj_offset=0.0)


@pytest.mark.parametrize("K", [255, 257, 2047, 2048, 2049, 4097])
def test_many_lps(K):
    """The control goes over the LPs in steps of 2048, 256 at a time."""
    lps = [few_rows(s) for s in range(K)]
    refs = [O.presolve(lp) for lp in lps]
    b = psl.Batch(lps)
    names = b.run()
    assert names == [ref.result_name for ref in refs]
    assert "INFEASIBLE" in names[K - 200:] and "REDUCED" in names[K - 200:]
    for k, ref in enumerate(refs):
        assert b.lp_stats(k)["rounds"] == ref.rounds, k
    for k in list(range(8)) + list(range(max(0, K - 8), K)):
        got = {"result_name": names[k], "records": b.records(k),
               "reduced": b.reduced(k) if names[k] in ("REDUCED", "UNCHANGED") else None}
        assert_same(got, refs[k], f"LP {k} of {K}")
    b.close()


@pytest.mark.parametrize("rows,direct", [(96000, True), (98000, False)])
def test_both_lists_are_reached(rows, direct):
    """The LPs of the two-sided test of the rounds lie on either side."""
    from tests.test_gpu_round_units import lp_of

    nnz = len(lp_of(rows, 100000, seed=1)["val"])
    assert nnz < 500000 if direct else nnz > 500000
