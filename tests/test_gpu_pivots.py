"""Pivots at the ends of their range in the factorization of G: one that is not
positive, in the first and later 16-wide blocks of it (status and stage,
untouched neighbours; after the last pivot of a problem, the unit pivot in its
place leaves numbers), and FP32 pivots so large that their reciprocal is subnormal."""
import numpy as np
import pytest

from oracle import kkt, riccati
from paper_1510_03110_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-10


def _rs():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    return torch, rs


@pytest.mark.parametrize("nx,nu,precision,factored", [(4, 2, 0, False), (20, 10, 0, False), (16, 8, 0, False),
                                                      (32, 16, 0, False), (32, 32, 0, True), (48, 33, 0, True),
                                                      (64, 32, 0, True), (64, 64, 0, True), (128, 64, 0, True),
                                                      (100, 80, 0, True), (20, 40, 0, True)])
def test_failed_pivot(nx, nu, precision, factored):
    """Q_w of stage 0 (the last one factored) with one negative entry: first
    entry, last entry and the first of the second block; as one leaf and as
    three with master levels above them.  As one leaf with the last entry bad
    nothing is eliminated after the unit pivot, and the results stay finite."""
    torch, rs = _rs()
    N = 12
    for j, Ns in [(j, Ns) for j in sorted({0, min(16, nu - 1), nu - 1}) for Ns in (4, 16)]:
        probs = [W.g2(nx, nu, N, seed=7 * nx + i) for i in range(3)]
        probs[1]["Qw"] = probs[1]["Qw"].copy()
        probs[1]["Qw"][0, j, j] = -1e3
        bt = rs.Batch({k: [p[k] for p in probs] for k in probs[0]}, precision=precision, Ns=Ns, branch=3,
                      factored=factored, rank_reveal=Ns * nu < nx)
        if factored:
            bt.factor()
            st = bt.status().tolist()
            bt.solve_factored()
        else:
            bt.solve()
            torch.cuda.synchronize()
            st = bt.status().tolist()
        torch.cuda.synchronize()
        assert st[0] == [0, -1] and st[2] == [0, -1]
        assert st[1] == [rs.RS_ERR_NOT_SPD, 0]
        for i in (0, 2):
            assert kkt.rel_error(bt.result(i), riccati.solve(probs[i])) <= TOL
        bad = bt.result(1)
        assert Ns < N or j < nu - 1 or all(np.isfinite(bad[k]).all() for k in ("x", "w", "lam"))
        bt.close()


@pytest.mark.parametrize("nx,nu", [(16, 8), (32, 16), (48, 20), (64, 32), (128, 64)])
def test_fp32_pivots_near_the_largest_number(nx, nu):
    """Weights of 0.5e38 to 2e38, so that G's pivots lie above 2^126 but within
    FP32: the minimiser does not depend on the scale, and mixed precision
    reaches it."""
    torch, rs = _rs()
    prob = W.g1_invariant(nx, nu, 20, 3)
    prob["A"], prob["B"] = 0.3 * prob["A"], 0.05 * prob["B"]
    ref = riccati.solve(W.materialize(prob))
    for k in ("Qx", "Qw", "QxN", "lx", "lw", "lN"):
        prob[k] = prob[k] * 1e38
    bt = rs.Batch({k: [prob[k]] for k in prob if k != "Qxw"}, precision=rs.RS_MIXED_FP32, Ns=5, branch=3,
                  rank_reveal=5 * nu < nx)
    bt.solve()
    torch.cuda.synchronize()
    assert bt.status()[0, 0] == 0
    sol = bt.result(0)
    for k in ("x", "w"):
        assert np.abs(sol[k] - ref[k]).max() <= TOL * np.abs(ref[k]).max()
    bt.close()
