"""GPU parity of the column-owner stored factorization (n_x <= 64, run-time
sizes padded to 16-wide tiles) at the edges of its tiles, against the serial
FP64 oracle: one below, at and one above a multiple of 16, the smallest and
the largest sizes, a single input, as many inputs as states (where Y and X lie
over A and B), single-leaf instances and short last leaves.  Tolerance: the
repository's bar of 1e-10 relative per block."""
import pytest

from oracle import kkt, riccati
from paper_1510_03110_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,nu,N,Ns", [(5, 3, 37, 8), (15, 15, 40, 4), (17, 16, 33, 8), (17, 17, 26, 6), (33, 1, 60, 70),
                                        (33, 32, 41, 8), (47, 33, 30, 6), (49, 7, 50, 16), (63, 31, 43, 8),
                                        (64, 33, 29, 7), (64, 48, 20, 5), (64, 64, 21, 4), (50, 25, 12, 16)])
def test_column_owner_shapes(nx, nu, N, Ns, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    prob = W.with_costs(W.g2(nx, nu, N, seed=nx * 100 + nu), seed=N)
    bt = rs.Batch({k: [prob[k]] for k in prob}, precision=precision, Ns=Ns, branch=2, factored=True)
    bt.factor()
    bt.solve_factored()
    torch.cuda.synchronize()
    assert bt.status()[0].tolist() == [0, -1]
    sol, ref = bt.result(0), riccati.solve(prob)
    assert kkt.rel_error(sol, ref) <= TOL
    assert abs(sol["obj"] - ref["obj"]) <= 1e-9 * max(1.0, abs(ref["obj"]))
    bt.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,nu,N,Ns,b", [(65, 1, 12, 16, 2), (65, 65, 9, 3, 2), (80, 64, 14, 4, 2), (113, 17, 20, 10, 2),
                                          (127, 128, 7, 2, 2), (128, 49, 13, 5, 3), (20, 100, 9, 3, 2)])
def test_wide_stage_shapes(nx, nu, N, Ns, b, precision):
    """Stages of more than 64 states (column blocks of 128, left operands in
    panels), at both sizes of the factorization of G in LDS (up to 64 and up to
    128 inputs), at the edges of their tiles and panels, with fewer row tiles
    than waves, a single leaf, and its use with more than 64 inputs on few
    states.  Bar as above."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    prob = W.with_costs(W.g2(nx, nu, N, seed=nx * 100 + nu), seed=N)
    bt = rs.Batch({k: [prob[k]] for k in prob}, precision=precision, Ns=Ns, branch=b, factored=True)
    bt.factor()
    bt.solve_factored()
    torch.cuda.synchronize()
    assert bt.status()[0].tolist() == [0, -1]
    sol, ref = bt.result(0), riccati.solve(prob)
    assert kkt.rel_error(sol, ref) <= TOL
    assert abs(sol["obj"] - ref["obj"]) <= 1e-9 * max(1.0, abs(ref["obj"]))
    bt.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,nu,N,Ns,b", [(3, 7, 7, 1, 2), (8, 4, 9, 4, 3), (16, 32, 11, 2, 2), (31, 33, 8, 2, 4), (33, 64, 10, 3, 2),
                                          (64, 64, 5, 2, 2)])
def test_prefetched_sweeps_at_short_lengths(nx, nu, N, Ns, b, precision):
    """The right-hand-side sweeps, whose matrices come through registers one
    stage ahead, at leaf and master lengths of one to four stages, at the
    edges of their size classes, with more inputs than states, and without
    the optional vectors a, lx, lw and c.  Bar as above."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    prob = W.with_costs(W.g2(nx, nu, N, seed=nx * 100 + nu + 7), seed=N)
    for drop in ((), ("a", "lx", "lw", "c")):
        data = {k: [prob[k]] for k in prob if k not in drop}
        data["N"] = [N]
        ref = riccati.solve({**prob, **{k: 0.0 * prob[k] for k in drop}})
        bt = rs.Batch(data, precision=precision, Ns=Ns, branch=b, factored=True)
        bt.factor()
        bt.solve_factored()
        torch.cuda.synchronize()
        assert bt.status()[0].tolist() == [0, -1]
        sol = bt.result(0)
        assert kkt.rel_error(sol, ref) <= TOL
        assert abs(sol["obj"] - ref["obj"]) <= 1e-9 * max(1.0, abs(ref["obj"]))
        bt.close()


def test_noalloc_takes_the_plans_it_counts_in():
    """Shapes below the full tiles keep V and L_t in their fused leaf records,
    which rs_batch_solve_noalloc does not count: a plan whose workspace is
    beyond the 64 MiB only by them is taken (and gives the workspace call's
    results bit for bit), one beyond it without them is refused."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    prob = W.g1_invariant(8, 4, 40000, seed=3)
    bt = rs.Batch({k: [prob[k]] for k in prob}, Ns=32, branch=8)
    assert bt.work_bytes > rs.RS_NOALLOC_SCRATCH_BYTES
    bt.solve()
    torch.cuda.synchronize()
    assert bt.status()[0].tolist() == [0, -1]
    ref = bt.x[0].clone(), bt.w[0].clone(), bt.lam[0].clone(), bt.obj.clone()
    for t in (bt.x[0], bt.w[0], bt.lam[0], bt.obj):
        t.zero_()
    rs.rs_batch_solve_noalloc(bt.plan, bt.probs, bt.stream_ptr(), bt.info.data_ptr())
    torch.cuda.synchronize()
    assert bt.status()[0].tolist() == [0, -1]
    for a, b in zip(ref, (bt.x[0], bt.w[0], bt.lam[0], bt.obj)):
        assert torch.equal(a, b)
    bt.close()
    plan = rs.rs_plan_create([(8, 4, 70000)], Ns=32, branch=8)
    with pytest.raises(rs.RsError) as e:
        rs.rs_batch_solve_noalloc(plan, (rs.rs_problem * 1)())
    assert e.value.status == rs.RS_ERR_NOMEM
    rs.rs_plan_destroy(plan)


@pytest.mark.parametrize("precision,factored", [(0, False), (0, True), (1, False)])
def test_many_leaves_run_longest_first(precision, factored):
    """Plans of more leaves than workgroups that start together take them by
    length: horizons below, at and above whole leaves, every leaf once (its
    instance equals the oracle's, bar as above)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_03110_amd import rs
    Ns = [1 + (7 * i) % 23 for i in range(150)]
    probs = [W.with_costs(W.g2(6, 3, N, seed=900 + i), seed=i) for i, N in enumerate(Ns)]
    bt = rs.Batch({k: [p[k] for p in probs] for k in probs[0]}, precision=precision, Ns=4, branch=4, factored=factored)
    assert len(rs.rs_plan_export(bt.plan, 0)) > 256
    if factored:
        bt.factor()
        bt.solve_factored()
    else:
        bt.solve()
    torch.cuda.synchronize()
    assert (bt.status()[:, 0] == 0).all()
    for i in range(150):
        assert kkt.rel_error(bt.result(i), riccati.solve(probs[i])) <= TOL
    bt.close()
