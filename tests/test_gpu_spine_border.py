"""Traces on both sides of 2,560 scan tiles of 4,096 words.  Up to there the
blocks of the down sweep compose what comes before them and count a one-level
tree's root; beyond, the prefixes come from the spine (one block, or chunks over
several where the records of four 16-state monitors make more than two passes)
and the root from a launch of its own.  Every instance, node, count, verdict and
timeline entry against the oracle."""
import pytest

from paper_1411_2239_amd import workloads as W

from _util import prop_workload
from test_gpu_parent_events import _check as check_parents
from test_gpu_parent_events import parent_workload
from test_gpu_parity import _check
from test_gpu_timeline import _run_events

pytestmark = pytest.mark.gpu

BORDER = 2560 * 4096


@pytest.mark.parametrize("n", [BORDER, BORDER + 1])
@pytest.mark.parametrize("levels,keys", [(1, [300_000]), (2, [300, 4000])])
def test_both_sides(n, levels, keys):
    _check(prop_workload(n, levels, keys, seed=levels, n_props=2))


def test_wide_monitors_spread_spine():
    # four monitors of 9-10 states: 80-byte records, chunks of 1,024 tiles
    big = [W.BATCH_FORMULAS[i] for i in (6, 8, 9, 12)]
    _check(prop_workload(BORDER + 4097, 2, [300, 4000], seed=91, n_props=4, formulas=big))


def test_parent_events_after_a_spine():
    check_parents(parent_workload(BORDER + 70_001, 2, [3000, 200], seed=92, n_props=2))


def test_timeline_after_a_spine():
    _run_events(prop_workload(BORDER + 12_345, 1, [100_000], seed=93, n_props=3,
                              formulas=["G(a -> X b)", "F(a & X F a)", "G a | (b U c)"]))
