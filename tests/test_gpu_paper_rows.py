"""The sorted backward's rows by level: the finest learnable level two or more
below the grid (the row is then a level that does not go out), one below it, and
the grid itself, at the coarsest grids and at the finest that the sorted path
takes, with triangles cut by wave boundaries and ones of a few fragments.
Oracle and tolerances are those of the levels' backward."""
import pytest

from . import test_gpu_paper as paper

pytestmark = pytest.mark.gpu

CASES = [
    dict(seed=61, T=40, R=1, Rmin=0, Rtop=0, sizes=[(33, 47)], from_log=False),
    dict(seed=62, T=7, R=4, Rmin=1, Rtop=2, sizes=[(120, 90), (31, 77)], from_log=True),
    dict(seed=63, T=500, R=5, Rmin=0, Rtop=2, sizes=[(64, 50)], from_log=False),
    dict(seed=64, T=200, R=5, Rmin=3, Rtop=5, sizes=[(90, 70)], from_log=True),
    dict(seed=65, T=3, R=5, Rmin=4, Rtop=4, sizes=[(128, 128)], from_log=False),
    dict(seed=66, T=60, R=0, Rmin=0, Rtop=0, sizes=[(40, 30)], from_log=False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"R{c['R']}L{c['Rmin']}-{c['Rtop']}")
def test_levels_rows_match_oracle(case):
    paper.test_paper_levels_backward_matches_oracle(case)
