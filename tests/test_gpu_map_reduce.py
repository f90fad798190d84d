"""The row-compacted contingency map-reduce at the edges of its blocks: one
contingency block with one used lane up to a second one with one, branch
counts around a 64-branch group, more groups than slices, one period; every
precision of the factors, with and without the bound-based skip, and a
screened set around a contingency block."""
import numpy as np
import pytest

from oracle import objective as ob
from paper_2310_06650_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qg():
    from paper_2310_06650_amd import qg as _qg
    return _qg


def evaluate(prob, x):
    import torch
    t, g = prob.eval_grad(prob.new_vector(x), 1e-2, 0.9, 0.8)
    torch.cuda.synchronize()
    return t.cpu().numpy(), g.cpu().numpy()


def close(c, qg, t, g, ref, tol):
    tr, gr = ref
    for name, v in zip(qg.TERM_NAMES, t):
        assert abs(v - tr[name]) <= tol * max(abs(tr[name]), 1e-300), name
    for sl in c.block_slices():
        assert np.abs(g[sl] - gr[sl]).max() <= tol * np.abs(gr[sl]).max()


# (buses, branches, periods, contingencies); the bounds per precision are
# those of the full-size parity and precision tests
@pytest.mark.parametrize("shape", [(40, 63, 1, 1), (40, 64, 3, 63), (45, 65, 2, 64),
                                   (80, 128, 5, 65), (90, 150, 4, None), (500, 1100, 2, 129)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp32", 1e-5), ("bf16", 1e-3)])
def test_edges_match_oracle_with_and_without_skip(qg, shape, prec, tol):
    n, nb, T, k = shape
    flag = {"fp64": 0, "fp32": qg.QG_FLAG_CTG_FP32, "bf16": qg.QG_FLAG_CTG_BF16}[prec]
    c = synth.make_case(seed=900 + n + nb, n_bus=n, n_branch=nb, n_gen=max(2, n // 7), n_period=T,
                        n_ctg=k, mesh=1.0)
    x = synth.random_point(c, 5, spread=0.3)
    m = ob.make_model(c)
    ref = ob.evaluate(m, x, 1e-2, 0.9, 0.8)
    got = []
    for extra in (0, qg.QG_FLAG_CTG_NO_SKIP):
        prob = qg.Problem(c, flags=flag | extra)
        assert prob.dims["ctg_split"] == 1
        got.append(evaluate(prob, x))
        prob.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    close(c, qg, *got[0], ref, tol)
    K = c.n_ctg
    if K > 64:  # a set of one lane more than a contingency block
        A = np.sort(np.random.default_rng(7).choice(K, size=min(65, K - 1), replace=False))
        prob = qg.Problem(c, flags=flag)
        prob.set_screening(top_frac=len(A) / K)
        prob.set_active_contingencies(A)
        t, g = evaluate(prob, x)
        prob.close()
        close(c, qg, t, g, ob.evaluate(m, x, 1e-2, 0.9, 0.8, active=A), tol)


def test_split_tile_names_change_nothing(qg):
    """Wavefronts and periods of a period-split tile name it; the launch follows
    from lt alone, whether given or left to the library: bitwise equal results of
    a grid for which eight tiles are the default of one name and not of another."""
    c = synth.make_case(seed=3, n_bus=2000, n_branch=2800, n_gen=300, n_period=48, n_ctg=None,
                        tree="prufer", mesh=3.0)
    x = synth.random_point(c, 17, spread=0.05)
    prob = qg.Problem(c)
    for lt in ("", "x8"):
        got = []
        for name in ("s4x4", "s8x8", "s1x4"):
            prob.set_tile(name + lt)
            got.append((prob.dims["ctg_lt"],) + evaluate(prob, x))
        if lt == "":
            assert len({g[0] for g in got}) > 1  # the defaults do differ
        for g in got[1:]:
            assert np.array_equal(got[0][1], g[1]) and np.array_equal(got[0][2], g[2]), lt
    prob.close()
