"""Performance cases of the parallel Riccati solver: the Newton-step (KKT)
solves that programs built on this library run, through its public entry
points (``rs_plan_create*``, ``rs_batch_solve``, ``rs_factor`` / ``rs_solve``,
``rs_plan_ring_update``), with everything resident in device memory.

A case is a batch of ``count`` problems P(N) of one shape (nx, nu) whose
horizons are spread over [Nmin, N]:

* ``call`` "solve": one ``rs_batch_solve`` of the whole batch;
  "factor": one interior-point iteration's linear algebra, ``rs_factor`` and
  two ``rs_solve`` (affine predictor, then the corrector's input cost);
  "window": one request of a receding-horizon serving loop: the window table
  is updated (``rs_plan_ring_update``) and solved with the interior leaves'
  factorization kept from the request before, the stage data in records.
* ``precision`` "fp64" or "mixed" (FP32 leaf factorization, refined in FP64 to
  a relative KKT residual of 1e-10).  BF16 products are not listed: they are
  measured slower than both others at every shape that offers them.
* ``data`` "dense": time-varying A_t, dense Q_x, cross term; "invariant": A and
  B given once, diagonal weights per stage, no cross term; "varying_A": A_t
  per stage, everything else given once.
"""
import ctypes
import math
import random

import torch

from paper_1510_03110_amd import rs

DEVICE = "cuda"
F64 = dict(dtype=torch.float64, device=DEVICE)


def _case(call, nx, nu, N, count, Ns, branch, precision="fp64", data="dense", Nmin=0):
    return dict(call=call, precision=precision, data=data, nx=nx, nu=nu, N=N, Nmin=Nmin or N, count=count, Ns=Ns,
                branch=branch)


def listed():
    return [
        # the smallest configuration, one problem: launches and latency alone
        dict(_case("solve", 4, 2, 64, 1, 4, 2, data="invariant"), name="step_nx4_N64"),
        # one Newton step of a mid-size estimator, no matrix-core shape
        dict(_case("solve", 20, 10, 1024, 1, 8, 4), name="step_nx20_N1024"),
        # the headline problem as a single step: latency of the tree
        dict(_case("solve", 32, 16, 1024, 1, 16, 4), name="step_nx32_N1024"),
        # the headline problem as a batch: throughput, FP64 and mixed
        dict(_case("solve", 32, 16, 1024, 512, 512, 8), name="batch_nx32"),
        dict(_case("solve", 32, 16, 1024, 256, 512, 8, precision="mixed"), name="batch_nx32_mixed"),
        # many independent problems of uneven horizons, time-invariant dynamics
        dict(_case("solve", 16, 8, 2048, 1024, 256, 8, data="invariant", Nmin=32), name="batch_nx16_ragged"),
        # stages too large for a register- and LDS-resident working set
        dict(_case("solve", 64, 32, 1024, 64, 64, 8), name="batch_nx64"),
        dict(_case("solve", 64, 32, 1024, 32, 64, 8, precision="mixed"), name="batch_nx64_mixed"),
        # one long problem of the largest blocks
        dict(_case("solve", 128, 64, 16384, 1, 64, 8, data="varying_A"), name="long_nx128"),
        # the linear algebra of an interior-point iteration on one problem
        dict(_case("factor", 32, 16, 1000, 1, 32, 8), name="interior_point_nx32"),
        # one launch of a serving lane: sessions of one shape, uneven horizons
        dict(_case("window", 64, 32, 4096, 16, 32, 8, Nmin=64), name="window_nx64"),
        dict(_case("window", 8, 4, 4096, 16, 32, 8, Nmin=64), name="window_nx8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: small shapes, matrix-core shapes (single
    steps to batches, both precisions, factor and solve), uneven horizons,
    large blocks of any size, serving windows."""
    kind = rng.choice(("small", "tile", "tile", "ragged", "large", "factor", "window"))
    branch = rng.choice((2, 3, 4, 8))
    if kind == "small":
        nx, nu = rng.choice(((2, 1), (3, 2), (4, 2), (6, 3), (8, 4), (20, 10)))
        N = _log_int(rng, 16, 2048)
        return _case("solve", nx, nu, N, min(_log_int(rng, 1, 64), max(1, 16384 // N)), rng.choice((4, 8, 16, 32)),
                     branch, data=rng.choice(("dense", "invariant")))
    if kind == "tile":
        nx, nu = rng.choice(((16, 16), (16, 8), (16, 5), (32, 16), (32, 16), (32, 8), (32, 32)))
        count = _log_int(rng, 1, 256)
        Ns = rng.choice((16, 24, 32)) if count <= 8 else rng.choice((64, 128, 200, 512))
        return _case("solve", nx, nu, _log_int(rng, 64, 1024), count, Ns, branch,
                     precision=rng.choice(("fp64", "fp64", "mixed")), data=rng.choice(("dense", "invariant")))
    if kind == "ragged":
        nx, nu = rng.choice(((16, 8), (16, 16), (32, 16)))
        return _case("solve", nx, nu, _log_int(rng, 256, 2048), _log_int(rng, 16, 256), rng.choice((128, 256, 512)),
                     8, precision=rng.choice(("fp64", "mixed")), data="invariant", Nmin=32)
    if kind == "large":
        nx = _log_int(rng, 33, 128)
        nu = max(8, nx * rng.choice((2, 3, 4)) // 8)
        N = _log_int(rng, 128, 4096)
        count = max(1, min(_log_int(rng, 1, 64), int(1.5e9 / (N * nx ** 2.6))))
        return _case("solve", nx, nu, N, count, rng.choice((32, 48, 64)), rng.choice((4, 8)),
                     precision=rng.choice(("fp64", "fp64", "mixed")), data=rng.choice(("dense", "varying_A")))
    if kind == "factor":
        nx, nu = rng.choice(((16, 16), (32, 16), (32, 8), (8, 4), (64, 32)))
        return _case("factor", nx, nu, _log_int(rng, 64, 1024), _log_int(rng, 1, 8), rng.choice((16, 32)),
                     rng.choice((4, 8)), precision=rng.choice(("fp64", "mixed")))
    nx, nu = rng.choice(((8, 4), (32, 16), (64, 32)))
    return _case("window", nx, nu, _log_int(rng, 256, 4096), _log_int(rng, 1, 16), 32, 8, Nmin=64)


def _horizons(case):
    lo, hi, n = case["Nmin"], case["N"], case["count"]
    if n == 1:
        return [hi]
    # evenly spread over [lo, hi], in a fixed mixed order
    step = next(s for s in range(n * 5 // 8 + 1, 2 * n + 2) if math.gcd(s, n) == 1)
    return [lo + (hi - lo) * ((i * step + n - 1) % n) // (n - 1) for i in range(n)]


# ------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Stage arrays over all stages of the batch, one after another (or one
    block per problem where the data are time-invariant)."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 1009 + 17)
    n, m, count = case["nx"], case["nu"], case["count"]
    Ns = _horizons(case)
    S = sum(Ns)
    randn = lambda *s: torch.randn(s, generator=gen, **F64)  # noqa: E731
    weight = lambda *s: torch.rand(s, generator=gen, **F64) * 1.5 + 0.5  # noqa: E731
    A0 = randn(count, n, n)
    A0 *= (0.95 / torch.linalg.eigvals(A0.cpu()).abs().amax(dim=-1).to(DEVICE))[:, None, None]
    d = dict(horizons=Ns, a=randn(S, n), lx=randn(S, n), lw=randn(S, m), c=randn(S), lN=randn(count, n),
             cN=randn(count), x0=randn(count, n))
    if case["data"] != "invariant":
        d["A"] = torch.empty((S, n, n), **F64)
        at = 0
        for i, N in enumerate(Ns):
            torch.randn((N, n, n), generator=gen, out=d["A"][at:at + N])
            d["A"][at:at + N].mul_(0.05).add_(A0[i])
            at += N
    if case["data"] == "dense":
        d["B"] = randn(S, n, m).div_(math.sqrt(n))
        d["Qx"] = torch.empty((S, n, n), **F64)
        step = max(1, (1 << 24) // (n * n))
        for s in range(0, S, step):
            M = randn(min(step, S - s), n, n)
            d["Qx"][s:s + step] = torch.matmul(M, M.transpose(1, 2).contiguous())
        d["Qx"].diagonal(dim1=1, dim2=2).add_(0.1)
        d["Qw"] = torch.diag_embed(weight(S, m))
        # |Qxw|_F = 0.1 keeps the stage Hessian positive definite (Qx >= 0.1, Qw >= 0.5)
        d["Qxw"] = randn(S, n, m)
        d["Qxw"].mul_(0.1 / torch.linalg.vector_norm(d["Qxw"], dim=(1, 2), keepdim=True))
        M = randn(count, n, n)
        d["QxN"] = torch.matmul(M, M.transpose(1, 2).contiguous())
        d["QxN"].diagonal(dim1=1, dim2=2).add_(0.1)
    else:
        per = S if case["data"] == "invariant" else count
        if case["data"] == "invariant":
            d["A"] = A0
        d["B"] = randn(count, n, m)
        d["Qx"] = torch.diag_embed(weight(per, n))
        d["Qw"] = torch.diag_embed(weight(per, m))
        d["QxN"] = torch.diag_embed(weight(count, n))
    if case["call"] == "factor":
        d["lw2"] = randn(S, m)       # the corrector's input cost
    return d


# -------------------------------------------------------------------- cases
_STAGE = ("Qx", "Qw", "Qxw", "A", "B", "a", "lx", "lw", "c")


class _State:
    def __del__(self):
        if getattr(self, "plan", None):
            rs.rs_plan_destroy(self.plan)


def prepare(case, seed):
    n, m, count = case["nx"], case["nu"], case["count"]
    st = _State()
    st.call, st.d = case["call"], _inputs(case, seed)
    d, Ns = st.d, st.d["horizons"]
    S = sum(Ns)
    size = dict(Qx=n * n, Qw=m * m, Qxw=n * m, A=n * n, B=n * m, a=n, lx=n, lw=m, c=1)
    st.x, st.w, st.lam = (torch.zeros((S + count, n), **F64), torch.zeros((S, m), **F64),
                          torch.zeros((S + count, n), **F64))
    st.obj, st.info = torch.zeros(count, **F64), torch.zeros((count, 2), dtype=torch.int32, device=DEVICE)
    if st.call == "window":
        # stage records, as a session's ring holds them
        st.rec = torch.cat([d[k].reshape(S, -1) for k in _STAGE], dim=1)
        for k in _STAGE:
            d.pop(k)
    st.probs = (rs.rs_problem * count)()
    at = 0
    for i, N in enumerate(Ns):
        p = st.probs[i]
        p.nx, p.nu, p.N = n, m, N
        if st.call == "window":
            off, E = 0, st.rec.shape[1]
            for k in _STAGE:
                setattr(p, k, st.rec.data_ptr() + 8 * (at * E + off))
                setattr(p, "s" + k, E)
                off += size[k]
        else:
            for k in _STAGE:
                if k not in d:
                    continue
                per_stage = d[k].shape[0] == S
                setattr(p, k, d[k].data_ptr() + 8 * size[k] * (at if per_stage else i))
                setattr(p, "s" + k, size[k] if per_stage else 0)
        for k, sz in (("QxN", n * n), ("lN", n), ("cN", 1), ("x0", n)):
            setattr(p, k, d[k].data_ptr() + 8 * sz * i)
        p.x, p.lam = st.x.data_ptr() + 8 * n * (at + i), st.lam.data_ptr() + 8 * n * (at + i)
        p.w, p.obj = st.w.data_ptr() + 8 * m * at, st.obj.data_ptr() + 8 * i
        at += N
    prec = rs.RS_MIXED_FP32 if case["precision"] == "mixed" else rs.RS_FP64
    if st.call == "window":
        start = 5 * case["Ns"] + 11          # a window between two leaf boundaries
        rows = [(n, m, N, case["Ns"], case["branch"], start, 0, 0) for N in Ns]
        st.plan = rs.rs_plan_create_ring(rows, precision=prec)
        st.dims = [r[:6] + rs.ring_current_leaves(start, r[2], r[3]) for r in rows]
    else:
        st.plan = rs.rs_plan_create([(n, m, N) for N in Ns], precision=prec, Ns=case["Ns"], branch=case["branch"],
                                    flags=rs.RS_PLAN_FACTORED if st.call == "factor" else 0)
    st.bytes = rs.rs_plan_workspace_size(st.plan)
    st.work = torch.empty(st.bytes + 256, dtype=torch.uint8, device=DEVICE)
    st.work_ptr = (st.work.data_ptr() + 255) // 256 * 256
    if st.call == "window":
        _call(rs.rs_batch_solve, st)         # the request before: leaves its factorization
    if st.call == "factor":
        st.lw1, st.w_aff = d["lw"].clone(), torch.zeros_like(st.w)
    return st


def _call(fn, st):
    fn(st.plan, st.probs, st.work_ptr, st.bytes, torch.cuda.current_stream().cuda_stream, st.info.data_ptr())


def run(st):
    out = {}
    if st.call == "factor":
        st.d["lw"].copy_(st.lw1)
        _call(rs.rs_factor, st)
        _call(rs.rs_solve, st)
        st.w_aff.copy_(st.w)
        st.d["lw"].copy_(st.d["lw2"])
        _call(rs.rs_solve, st)
        out["w_aff"] = st.w_aff
    else:
        if st.call == "window":
            rs.rs_plan_ring_update(st.plan, st.dims)
        _call(rs.rs_batch_solve, st)
    out.update(x=st.x, w=st.w, lam=st.lam, obj=st.obj, info=st.info)
    return out


def work(case):
    n, m, count = case["nx"], case["nu"], case["count"]
    S = sum(_horizons(case))
    out = 2 * n + m
    vec = 2 * n + m + 1
    stage = {"dense": 2 * n * n + 2 * n * m + m * m, "varying_A": n * n, "invariant": n * n + m * m}[case["data"]]
    # symmetric results counted once: P [A B], [A B]'P [A B], the factorization
    # of G, L^{-1} H', the update of P and the feedback; then the vector lines
    factor = 3 * n ** 3 + 5 * n * n * m + 3 * n * m * m + m ** 3 / 3
    solve = 8 * n * n + 8 * n * m + 2 * m * m
    factored = S
    if case["call"] == "window":
        # the stages outside the kept leaves are factored again; of the kept
        # ones A, B and the stage vectors are read
        start, Ns = 5 * case["Ns"] + 11, case["Ns"]
        factored = sum(N - Ns * (hi - lo) for N in _horizons(case) for lo, hi in
                       [rs.ring_current_leaves(start, N, Ns)])
        read = factored * stage + (S - factored) * (n * n + n * m)
    else:
        read = S * stage
    bytes_ = 8 * (read + S * (vec + out) + count * (n * n + 2 * n + 2))
    flops = factored * factor + S * solve
    if case["call"] == "factor":
        bytes_ += 8 * S * 3 * m
        flops += S * solve
    return dict(bytes=bytes_, flops=flops)


# --------------------------------------------------- the same answer, plainly
def exact(case, seed):
    """The serial Riccati recursion over the whole batch, one stage at a time
    from the end, in FP64 (plain torch)."""
    d = _inputs(case, seed)
    n, m, count = case["nx"], case["nu"], case["count"]
    Ns = torch.tensor(d["horizons"])
    S = int(Ns.sum())
    order = torch.argsort(Ns, descending=True, stable=True)      # problems still running are a prefix
    N = Ns[order]
    first = (torch.cumsum(Ns, 0) - Ns)[order]
    inst, at, N = order.to(DEVICE), first.to(DEVICE), N.to(DEVICE)
    live = [int((Ns > k).sum()) for k in range(int(Ns.max()))]

    def stage(key, idx, c):
        v = d.get(key)
        return None if v is None else v[idx] if v.shape[0] == S else v[inst[:c]]

    K, kv = torch.empty((S, m, n), **F64), torch.empty((S, m), **F64)
    Ps, Psis = torch.empty((S, n, n), **F64), torch.empty((S, n), **F64)

    def backward(lw):
        P, Psi = d["QxN"][inst], -d["lN"][inst]
        for k, c in enumerate(live):
            idx = at[:c] + N[:c] - 1 - k
            P, Psi = P[:c], Psi[:c]
            A, B = stage("A", idx, c), stage("B", idx, c)
            AB = torch.cat([A, B], dim=2)
            W = torch.matmul(P, AB)
            M = torch.matmul(AB.transpose(1, 2).contiguous(), W)
            F, H, G = M[:, :n, :n] + stage("Qx", idx, c), M[:, :n, n:], M[:, n:, n:] + stage("Qw", idx, c)
            Qxw = stage("Qxw", idx, c)
            H = H if Qxw is None else H + Qxw
            Ht = H.transpose(1, 2).contiguous()
            p = Psi - torch.matmul(P, d["a"][idx].unsqueeze(2)).squeeze(2)
            g = torch.matmul(AB.transpose(1, 2).contiguous(), p.unsqueeze(2)).squeeze(2)
            gx, gw = g[:, :n] - d["lx"][idx], g[:, n:] - lw[idx]
            L = torch.linalg.cholesky_ex((G + G.transpose(1, 2)) / 2)[0]
            KK = torch.cholesky_solve(torch.cat([-Ht, gw.unsqueeze(2)], dim=2), L)
            K[idx], kv[idx] = KK[:, :, :n], KK[:, :, n]
            Psi = gx - torch.matmul(H, KK[:, :, n:]).squeeze(2)
            P = F + torch.matmul(H, KK[:, :, :n].contiguous())
            P = (P + P.transpose(1, 2)) / 2
            Ps[idx], Psis[idx] = P, Psi

    x, w, lam = torch.empty((S + count, n), **F64), torch.empty((S, m), **F64), torch.empty((S + count, n), **F64)
    mv = lambda M, v: torch.matmul(M, v.unsqueeze(2)).squeeze(2)  # noqa: E731

    def forward():
        xt = d["x0"][inst]
        for k, c in enumerate(live):
            xt, idx = xt[:c], at[:c] + k
            wt = mv(K[idx], xt) + kv[idx]
            row = idx + inst[:c]
            x[row], w[idx] = xt, wt
            lam[row] = mv(Ps[idx], xt) - Psis[idx]
            xt = mv(stage("A", idx, c), xt) + mv(stage("B", idx, c), wt) + d["a"][idx]
            done = c if k + 1 == len(live) else live[k + 1]
            if done < c or k + 1 == len(live):
                lo = 0 if k + 1 == len(live) else done
                end, i = row[lo:] + 1, inst[lo:c]
                x[end] = xt[lo:]
                lam[end] = mv(d["QxN"][i], xt[lo:]) + d["lN"][i]

    out = {}
    backward(d["lw"])
    forward()
    lw = d["lw"]
    if case["call"] == "factor":
        out["w_aff"] = w.clone()
        lw = d["lw2"]
        backward(lw)
        forward()
    # the optimal value, stage by stage
    owner = torch.repeat_interleave(torch.arange(count), Ns).to(DEVICE)
    xs = x[torch.arange(S, device=DEVICE) + owner]
    every = torch.arange(S, device=DEVICE)
    pick = lambda key: d[key][every] if d[key].shape[0] == S else d[key][owner]  # noqa: E731
    cost = 0.5 * (xs * mv(pick("Qx"), xs)).sum(1) + 0.5 * (w * mv(pick("Qw"), w)).sum(1) + d["c"]
    cost += (xs * d["lx"]).sum(1) + (w * lw).sum(1)
    if "Qxw" in d:
        cost += (xs * mv(d["Qxw"], w)).sum(1)
    xN = x[torch.cumsum(Ns, 0).to(DEVICE) + torch.arange(count, device=DEVICE)]
    obj = 0.5 * (xN * mv(d["QxN"], xN)).sum(1) + (xN * d["lN"]).sum(1) + d["cN"]
    obj = obj.index_add(0, owner, cost)
    out.update(x=x, w=w, lam=lam, obj=obj, info=None)
    return out
