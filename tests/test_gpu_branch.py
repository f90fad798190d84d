"""The branch penalty where its binding side or its root is delicate."""
import numpy as np
import pytest

from oracle import objective as ob
from tests._cases import tiny_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qg():
    from paper_2310_06650_amd import qg as _qg
    return _qg


def line(bch):
    """One line of g = 1, b = -1 between two buses, over its rating at any
    voltages used here."""
    return tiny_case(2, [0], [1], [0.5], [0], T=1, br_r=[0.5], br_bch=np.array([bch]),
                     br_smax=np.array([0.1]))


def evaluate(qg, c, v):
    import torch
    x = np.concatenate([v, np.zeros(2), [0.5, 0.1, 0.05, 0.9]])
    prob = qg.Problem(c)
    t, g = prob.eval_grad(prob.new_vector(x), 1e-2)
    torch.cuda.synchronize()
    t, g = dict(zip(qg.TERM_NAMES, t.cpu().numpy())), g.cpu().numpy()
    prob.close()
    return x, t, g


def test_side_is_chosen_by_the_rounded_roots(qg):
    """At v = (1, 1.75), no angle and this charging the to side's |S|^2 is one
    unit above the from side's however the squares and products are fused, and
    both roots are the same number: the from side binds (its derivative in the
    voltages differs from the other side's by more than a tenth)."""
    charge = 1.0 - float.fromhex("0x1.4babe8c1a9212p-1")
    c = line(2.0 * charge)
    v = np.array([1.0, 1.75])
    model = ob.make_model(c)
    fl = ob.branch_flows(model, v[None], np.zeros((1, 2)))
    sf2, st2 = (fl["pf"] ** 2 + fl["qf"] ** 2).item(), (fl["pt"] ** 2 + fl["qt"] ** 2).item()
    assert st2 > sf2 and np.sqrt(st2) == np.sqrt(sf2)
    x, t, g = evaluate(qg, c, v)
    tr, gr = ob.evaluate(model, x, 1e-2, 1.0, 1.0)
    assert abs(t["br"] - tr["br"]) <= 1e-9 * tr["br"]
    assert np.abs(g - gr).max() <= 1e-9 * np.abs(gr).max()


def test_overflowing_flow_is_not_within_its_rating(qg):
    """A flow whose square overflows does not count as one inside the rating."""
    t = evaluate(qg, line(0.1), np.array([1e100, 1.0]))[1]
    assert not np.isfinite(t["br"])
