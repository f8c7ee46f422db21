"""GPU parity of the right-hand-side sweeps of the stored factorization with
many leaves, where they take another form (v two stages behind, one wavefront a
leaf or work item): leaves of one to three stages, master items of two to four,
at the edges of the size classes, against the serial FP64 oracle.  Tolerance:
the repository's bar of 1e-10 relative per block."""
import pytest

from oracle import kkt, riccati
from paper_1510_03110_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,nu,N,Ns,b,count", [
    (16, 16, 19, 1, 3, 15),       # 285 leaves of one stage
    (13, 7, 27, 2, 2, 20),
    (32, 16, 39, 3, 4, 21),       # 273 leaves
    (32, 16, 40, 2, 4, 53),       # 1060 leaves, one wavefront each
    (32, 32, 35, 1, 2, 30),       # 1050 leaves of one stage
    (24, 12, 47, 3, 3, 18),
    (32, 16, 22, 3, 2, 4),        # 32 leaves, up to 128 work items: two wavefronts an item
    (64, 32, 25, 2, 3, 20),
    (33, 40, 11, 1, 4, 27),       # more inputs than states
])
def test_sweeps_with_many_leaves(nx, nu, N, Ns, b, count, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    # (leaves with as many inputs as states in all: their reduced weight may be
    # singular in FP32)
    probs = [W.with_costs(W.g2(nx, nu, N - i % 3, seed=nx * 100 + nu + i), seed=i) for i in range(count)]
    bt = rs.Batch({k: [p[k] for p in probs] for k in probs[0]}, precision=precision, Ns=Ns, branch=b, factored=True,
                  rank_reveal=Ns * nu <= nx)
    bt.factor()
    bt.solve_factored()
    torch.cuda.synchronize()
    assert (bt.status()[:, 0] == 0).all()
    for i, p in enumerate(probs):
        sol, ref = bt.result(i), riccati.solve(p)
        assert kkt.rel_error(sol, ref) <= TOL
        assert abs(sol["obj"] - ref["obj"]) <= 1e-9 * max(1.0, abs(ref["obj"]))
    bt.close()
