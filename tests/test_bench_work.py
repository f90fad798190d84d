"""The benchmark prices the kernels by what they have to move."""
import pytest

bench = pytest.importorskip("bench")
from paper_2310_06650_amd import synth  # noqa: E402


def test_assembly_is_not_priced_by_sums_that_are_not_stored():
    """The period-split map-reduce stores R and Q of overloaded rows alone, and a flag
    per row and contingency block for the others: 64 more blocks cost eight bytes a
    branch and period.  The branch-stacked form stores both for every row."""
    c = synth.config_case("c2")
    TL = c.n_period * c.n_branch
    dims = dict(ctg_split=1, nKb=9, nLb=4)
    amount = lambda **k: bench.kernel_work(c, {**dims, **k})["k_ctg_asm"][1]  # noqa: E731
    assert amount(nKb=73) - amount() == 8 * TL
    assert amount(ctg_split=0, nKb=73) - amount(ctg_split=0) == 64 * 16 * TL
    # and by the device terms: eight doubles a generator and period
    assert amount() >= 8 * 8 * c.n_period * c.n_gen


def test_update_of_a_small_grid_is_both_kernels_work():
    c = synth.config_case("c1")
    assert c.n_branch <= bench.UPDATE_MAX_BRANCH
    w = bench.kernel_work(c, dict(ctg_split=1, nKb=1, nLb=1))
    ends = 8 * 4 * c.n_period * c.n_branch  # written by one, read by the other
    assert w["k_update"][1] == w["k_adjoint"][1] + w["k_final"][1] - 2 * ends
