"""PSL_TRACE: a line on stderr for every propagation round."""
import re

import pytest

from oracle import oracle as O
from paper_2609_16182_amd import lpgen

pytestmark = pytest.mark.gpu

psl = pytest.importorskip("paper_2609_16182_amd.psl")

LINE = re.compile(r"\[psl\] round (\d+): swept rows (\d+) nnz (\d+), records (\d+), rows removed (\d+), "
                  r"bounds made finite (\d+), LPs propagating (\d+)\n")


def lines_of(monkeypatch, capfd, make):
    monkeypatch.setenv("PSL_TRACE", "1")
    b = make()
    capfd.readouterr()
    b.run()
    return b, [tuple(int(x) for x in m.groups()) for m in LINE.finditer(capfd.readouterr().err)]


@pytest.mark.parametrize("options", [{}, dict(enable_free_singletons=1)])
def test_a_line_for_each_round(monkeypatch, capfd, options):
    lp = lpgen.large(seed=3, scale=2e-4)
    p, lines = lines_of(monkeypatch, capfd, lambda: psl.Presolver(lp, **options))
    ref = O.presolve(lp, **options)
    assert p.stats["records"] == len(ref.records)
    per_round = {}
    for r in ref.records["round"]:
        per_round[int(r)] = per_round.get(int(r), 0) + 1
    assert len(lines) == p.stats["sweep_launches"] and len(set(x[0] for x in lines)) == len(lines)
    for no, rows, nnz, records, removed, fin, going in lines:
        assert records == per_round.get(no, 0), no
        assert going == (records > 0)
    assert lines[0][1:3] == (lp["m"], len(lp["val"]))
    p.close()


def test_lps_still_propagating(monkeypatch, capfd):
    lps = [lpgen.batch_member(i, m=150 + 50 * i) for i in range(5)]
    b, lines = lines_of(monkeypatch, capfd, lambda: psl.Batch(lps))
    refs = [O.presolve(lp) for lp in lps]
    first = {}  # of the first cycle: the LPs that recorded something in the round
    for no, rows, nnz, records, removed, fin, going in lines:
        first.setdefault(no, (records, going))
    for no in range(1, 4):
        changed = [int((ref.records["round"] == no).sum()) for ref in refs]
        assert first[no] == (sum(changed), sum(x > 0 for x in changed)), no
    b.close()
