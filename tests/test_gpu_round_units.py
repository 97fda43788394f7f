"""Rounds queued ahead of the host: tile edges, unit boundaries, full record stacks.

The decisions count records per tile of 1024 rows or columns and per 64 tiles,
the selection takes rows in tiles of 1024, and up to 8 rounds are queued before
the host reads the results. Sizes and round limits on both sides of these edges
are compared bit for bit with the CPU oracle (exact: every output is defined to
the last bit).
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_16182_amd import lpgen
from tests.parity_util import assert_same

pytestmark = pytest.mark.gpu

psl = pytest.importorskip("paper_2609_16182_amd.psl")


def lp_of(m, n, seed=0):
    """m rows of 2 to 9 entries over n columns, some of every planted kind."""
    k = m // 40
    return lpgen.make_lp(m, n, seed=seed, row_len=(2, 9), singleton=k, empty=k, doubleton=k, duplicate=k,
                         fixed_cols=n // 40)


def gpu(lp, **kw):
    out, p = psl.presolve(lp, **kw)
    p.close()
    return out


@pytest.mark.parametrize("m,n", [(1, 12), (1023, 1025), (1024, 1024), (1025, 2047), (2049, 1023), (4097, 6000),
                                 (65535, 65537), (65537, 65536), (66561, 131073)])
def test_tile_edges(m, n):
    lp = lp_of(m, n, seed=m)
    assert_same(gpu(lp), O.presolve(lp), f"{m} x {n}")


@pytest.mark.parametrize("rounds", [1, 2, 7, 8, 9, 16, 17])
def test_unit_boundaries(rounds):
    lp = lpgen.large(seed=3, scale=2e-4)
    assert_same(gpu(lp, max_rounds=rounds, enable_free_singletons=1),
                O.presolve(lp, max_rounds=rounds, enable_free_singletons=1), f"max_rounds {rounds}")


@pytest.mark.parametrize("slack", [0, 1, 5000])
def test_record_stack_stops_a_unit(slack):
    """A stack of one round's records and a little more: the queued rounds stop
    when the next might not fit, the host empties it, the rounds go on."""
    lp = lp_of(3000, 4500, seed=7)
    need = lp["m"] + 3 * lp["n"] + 16
    got = gpu(lp, device_records=need + slack)
    assert_same(got, O.presolve(lp), f"slack {slack}")
    assert got["stats"]["record_flushes"] >= 1


@pytest.mark.parametrize("rounds", [3, 8, 16])
def test_batch_lps_end_in_different_rounds(rounds):
    lps = [lp_of(1 + 257 * i, 12 + 300 * i, seed=i) for i in range(9)] + [lpgen.tiny(s) for s in range(7)]
    b = psl.Batch(lps, max_rounds=rounds)
    names = b.run()
    for k, lp in enumerate(lps):
        got = {"result_name": names[k], "records": b.records(k),
               "reduced": b.reduced(k) if names[k] in ("REDUCED", "UNCHANGED") else None}
        ref = O.presolve(lp, max_rounds=rounds)
        assert_same(got, ref, f"LP {k}")
        assert b.lp_stats(k)["rounds"] == ref.rounds
    b.close()
    assert np.isfinite(b.stats["ms_sweep"]) and b.stats["ms_sweep"] >= 0


@pytest.mark.parametrize("length,block", [(4, 64), (8, 32), (16, 16), (60, 4), (250, 1)])
@pytest.mark.parametrize("off", [-1, 0, 1])
def test_row_block_edges(length, block, off):
    """One row block to a workgroup: rows of one bin, one less and one more
    than whole blocks of it."""
    lp = lpgen.make_lp(max(1, 3 * block + off), 400, seed=length, row_len=(max(1, length - 1), length))
    assert_same(gpu(lp, max_rounds=4), O.presolve(lp, max_rounds=4), f"{lp['m']} rows of {length}")


@pytest.mark.parametrize("rows", [96000, 98000])
def test_direct_and_selected_lists(rows):
    """On both sides of the 500000 nonzeros up to which a sweep tests each row."""
    lp = lp_of(rows, 100000, seed=1)
    assert_same(gpu(lp), O.presolve(lp), f"{rows} rows, {len(lp['val'])} nonzeros")


def with_long_column(m, entries, seed):
    """lp_of plus one column in the first `entries` rows, its bounds far out:
    every one of them may tighten it."""
    lp = lp_of(m, m, seed)
    rng = np.random.default_rng(seed)
    rp, n = lp["row_ptr"], lp["n"]
    at = rp[1:entries + 1]  # behind each row's last entry
    lp["col_idx"] = np.insert(lp["col_idx"], at, n).astype(lp["col_idx"].dtype)
    lp["val"] = np.insert(lp["val"], at, rng.choice([-2.0, -1.0, 1.0, 2.0], entries))
    lp["row_ptr"] = (rp + np.minimum(np.arange(m + 1), entries)).astype(rp.dtype)
    for k, v in (("lb", -1e4), ("ub", 1e4), ("c", 1.0)):
        lp[k] = np.append(lp[k], v)
    lp["n"] = n + 1
    return lp


@pytest.mark.parametrize("entries", [4095, 4096, 4097, 6000])
def test_long_column_accumulators(entries):
    """With columns of more than 4096 entries a candidate looks at its
    accumulator before the atomic."""
    lp = with_long_column(6000, entries, seed=5)
    assert_same(gpu(lp), O.presolve(lp), f"{entries} entries")


@pytest.mark.parametrize("m", [255, 257, 16384, 16385, 33000])
def test_free_singleton_tiles(m):
    """Eliminations are counted in tiles of 256 rows, 64 tiles to a sum."""
    lp = lp_of(m, m + m // 4, seed=m)
    assert_same(gpu(lp, enable_free_singletons=1), O.presolve(lp, enable_free_singletons=1), f"{m} rows")
