"""Accuracy of the reductions of mixed plans, on data whose FP32 leaf
factorization is exact, so that the first solve of a mixed plan is as accurate
as an FP64 one and its first correction shows any rounding added to it."""
import numpy as np
import pytest

from paper_1510_03110_amd import workloads as W  # noqa: F401  (imports the package)

pytestmark = pytest.mark.gpu


def _rs():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    return torch, rs


def _first_correction(prob, **opt):
    """Size of the first correction relative to the solution."""
    torch, rs = _rs()
    bt = rs.Batch({k: [prob[k]] for k in prob}, max_refine=1, tol=1e-30, **opt)
    bt.solve()
    torch.cuda.synchronize()
    assert bt.status()[0, 0] in (0, rs.RS_ERR_NOT_CONVERGED)
    dz = float(bt.refine_stats()[0][4])
    bt.close()
    return dz


def _sums_of_inputs(n, m, Ns, leaves, seed):
    """A = I, Q_x = 0, Q_w = I and no cross term: every leaf reduces to
    P = 0, V = I and Q_w_hat = sum_t B_t B_t'.  Its last stage has B = 2^12 I
    (2^24 on the diagonal), the others B = 1/2 everywhere: m terms of 1/4 an
    element and stage, which FP32 adds to 2^24 without error once they are
    summed (m / 4 is even), and loses one by one.  The leaf with the terminal
    has B = 0."""
    rng = np.random.default_rng(seed)
    N = Ns * leaves
    B = np.full((N, n, m), 0.5)
    B[Ns - 1::Ns] = 4096.0 * np.eye(n, m)
    B[-Ns:] = 0.0
    eye = np.eye(n)
    return dict(Qx=np.zeros((N, n, n)), Qw=np.tile(np.eye(m), (N, 1, 1)), Qxw=np.zeros((N, n, m)),
                A=np.tile(eye, (N, 1, 1)), B=B, a=rng.standard_normal((N, n)), lx=rng.standard_normal((N, n)),
                lw=rng.standard_normal((N, m)), c=np.zeros(N), QxN=eye, lN=rng.standard_normal(n),
                cN=np.float64(0.0), x0=rng.standard_normal(n))


@pytest.mark.parametrize("n,m,precision", [(8, 8, 1), (16, 16, 1), (32, 32, 1), (48, 48, 1), (64, 64, 1), (80, 80, 1),
                                           (128, 128, 1), (80, 80, 2), (128, 128, 2)])
def test_reduced_input_weight_is_summed_once_a_stage(n, m, precision):
    """Q_w_hat is exact in FP32 (products formed apart, added once).  Bound:
    its condition number is 2^24 (1 + 32 n m / 2^26), so the FP64 master levels
    give 2^24 2^-53 n = n 2e-9 < 1e-6 for n <= 128.  Terms lost one by one
    change Q_w_hat by 32 m / 4 on every element, m n / 2^21 of its norm (3e-5 at
    n = m = 8)."""
    dz = _first_correction(_sums_of_inputs(n, m, 33, 3, n), precision=precision, Ns=33, branch=2)
    assert dz <= 1e-6, "first correction %.2e" % dz


@pytest.mark.parametrize("n,m", [(8, 3), (16, 8), (20, 10), (32, 16), (48, 8), (64, 16)])
def test_rank_revealing_factor_keeps_64_bits(n, m):
    """One-stage leaves of small whole numbers with Q_w = I, Q_xw = 0 (P = 0
    before them, so K = 0, L = I, V = A' and Q_w_hat = B B', all exact in
    FP32) and Q_xN = 0.  The pivoted factor of B B' holds its remaining rows
    in 64 bits, as the master levels do.  Bound: a 64th of one rounding to
    FP32 (2^-24 / 64); FP64 roundings leave about 1e-13, a factor held in 32
    bits 5e-11 and more."""
    rng = np.random.default_rng(n)
    N = 24
    ints = lambda *s: rng.integers(-3, 4, s).astype(float)  # noqa: E731
    prob = dict(Qx=np.tile(4.0 * np.eye(n), (N, 1, 1)), Qw=np.tile(np.eye(m), (N, 1, 1)), Qxw=np.zeros((N, n, m)),
                A=ints(N, n, n) * (rng.random((N, n, n)) < 2.0 / n) / 4, B=ints(N, n, m), a=ints(N, n),
                lx=ints(N, n), lw=ints(N, m), c=np.zeros(N), QxN=np.zeros((n, n)), lN=ints(n),
                cN=np.float64(0.0), x0=ints(n))
    dz = _first_correction(prob, precision=1, Ns=1, branch=3, rank_reveal=True)
    assert dz <= 2.0 ** -30, "first correction %.2e" % dz
