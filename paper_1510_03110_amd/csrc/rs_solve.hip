// Right-hand-side pass over the master levels for RS_PLAN_REFACTOR_DOWN (the
// down pass that factors every master subproblem again from its parent's
// message, kept for comparison), on the matrix-core shapes.  Everything else
// of the factor / solve split runs on the prefetching sweeps (rs_vsweep.hip).
//
// With the stored factors (P_t, L^{-1} and L^{-T} with G_{t+1} = L L', K and,
// for Alg. 4, V_t) the vector lines of Alg. 2-4 and the forward recursion of
// Alg. 3 are matrix-vector products only:
//
//   P a   with P = P_{t+1}           pt  = Psi_{t+1} - P a
//   g_w   = B' pt - l_w             z   = L^{-1} g_w         k = L^{-T} z
//   Psi_t = A' pt + K' g_w - l_x     (K' g_w = -H' G^{-1} g_w, Alg. 2)
//   cbar_t = cbar_{t+1} + 1/2 a'Pa - Psi_{t+1}'a + c - 1/2 z'z
//   Alg. 4:  v += V_{t+1}' (a + B k)
//   Alg. 3:  w = K x + k,  x_{t+1} = A x + B w + a
//
// A master subproblem is one wavefront; all operands of a stage are loaded
// into registers before the first product of the stage.
//   kv_tree       work queue over the master levels (vector part of Alg. 5,
//                 top solve, Alg. 6 down to level 1)
#include <hip/hip_runtime.h>

#include "rs_launch.hpp"
#include "rs_vec.hpp"

namespace rs {
namespace sv {

// LDS vectors of one work unit.
template <int NX, int NU>
struct VSmem {
    double Psi[NX], pt[NX], av[NX], d[NX], x[NX];
    double gw[NU], z[NU], kk[NU], wv[NU];
    double v[NX];
};

// Where a backward stage's operands live.  Stored factors are of type TR
// (double, or float for mixed-precision leaves); a P_{t+1} that comes from
// the problem or a parent's message is FP64 (Pn64).
template <class TR>
struct VSrc {
    const TR *Pn;          // P_{t+1}, symmetric
    const double *Pn64;    // used when Pn is null; both null = 0 (Alg. 4 preliminary terminal)
    const TR *Vn;          // V_{t+1}; nullptr = identity (Alg. 4 only)
    const TR *Li, *LT;     // L^{-1}, L^{-T}, row-major NU x NU
    const TR *K;           // NU x NX row-major
    const double *A, *B;   // dynamics (B: NX x NU row-major)
    const double *a, *lx, *lw;
    double c;
};

// One backward stage of the vector recursion.  Psi, cbar (and v for RED) are
// the running state; Psi_t and k_{t+1} are returned in LDS (S.Psi, S.kk) and
// handed to emit(Psi_i, k_i) from lanes i < NX / i < NU.
template <int NX, int NU, bool RED, bool WANTK, class TR, class Emit>
__device__ __forceinline__ void vstage(VSmem<NX, NU> &S, const VSrc<TR> &q, double &cbar, Emit emit) {
    const int l = lane();
    Op<NX, NX> oP, oA, oV;
    Op<NU, NX> oB;
    Op<NU, NU> oLT, oLi;
    Op<NX, NU> oK;
    if (q.Pn)
        oP.template load<false>(q.Pn, NX);
    else
        oP.template load<false>(q.Pn64, NX);
    oB.template load<false>(q.B, NU);
    oLT.template load<false>(q.LT, NU);
    oA.template load<false>(q.A, NX);
    oK.template load<false>(q.K, NX);
    if constexpr (RED || WANTK) oLi.template load<false>(q.Li, NU);
    if constexpr (RED) {
        if (q.Vn) oV.template load<false>(q.Vn, NX);
    }
    const double av = (l < NX && q.a) ? q.a[l] : 0.0;
    const double lx = (l < NX && q.lx) ? q.lx[l] : 0.0;
    const double lw = (l < NU && q.lw) ? q.lw[l] : 0.0;
    if (l < NX) S.av[l] = av;
    wsync();
    // P a, pt, cbar += 1/2 a'Pa - Psi'a + c
    {
        const double pa = oP.apply(S.av);
        double part = 0.0;
        if (l < NX) {
            S.pt[l] = S.Psi[l] - pa;
            part = av * (0.5 * pa - S.Psi[l]);
        }
        cbar += wave_sum(part) + q.c;
    }
    wsync();
    {
        const double g = oB.apply(S.pt) - lw;
        if (l < NU) S.gw[l] = g;
    }
    wsync();
    {
        const double z = oLT.apply(S.gw);                        // L^{-1} g_w
        const double psi = oA.apply(S.pt) + oK.apply(S.gw) - lx;  // Psi_t
        if (l < NU) S.z[l] = z;
        cbar -= 0.5 * wave_sum(l < NU ? z * z : 0.0);
        if (l < NX) S.Psi[l] = psi;
    }
    wsync();
    if constexpr (RED || WANTK) {
        const double k = oLi.apply(S.z);                         // L^{-T} z
        if (l < NU) S.kk[l] = k;
        emit(l < NX ? S.Psi[l] : 0.0, k);
        wsync();
    } else {
        emit(l < NX ? S.Psi[l] : 0.0, 0.0);
    }
    if constexpr (RED) {
        RowOp<NX, NU> rB;      // B again, as contiguous rows (read from cache)
        rB.load(q.B, NU);
        rB.apply(S.kk, [&](int r, double bk) { S.d[r] = S.av[r] + bk; });   // a + B k
        wsync();
        const double dd = l < NX ? S.d[l] : 0.0;
        const double inc = q.Vn ? oV.apply(S.d) : dd;
        if (l < NX) S.v[l] += inc;
        wsync();
    }
}

// One forward stage (Alg. 3): w = K x + k, x_{t+1} = A x + a + B w and, for
// leaves, lam_t = P_t x - Psi_t.  Operands as in VSrc (ROW-read here).
template <int NX, int NU, bool LAM, class TR>
__device__ __forceinline__ void fstage(VSmem<NX, NU> &S, const TR *K, const double *kvec, const double *A,
                                       const double *B, const double *a, const TR *P, const double *Psi,
                                       double &lam_out, double &w_out) {
    const int l = lane();
    Op<NU, NX> oK;
    Op<NX, NX> oA, oP;
    Op<NX, NU> oB;
    oK.template load<true>(K, NX);
    oA.template load<true>(A, NX);
    oB.template load<true>(B, NU);
    if constexpr (LAM) oP.template load<false>(P, NX);
    const double kk = l < NU ? kvec[l] : 0.0;
    const double av = (l < NX && a) ? a[l] : 0.0;
    const double psi = (LAM && l < NX) ? Psi[l] : 0.0;
    const double w = oK.apply(S.x) + kk;
    const double ax = oA.apply(S.x) + av;
    if constexpr (LAM) lam_out = oP.apply(S.x) - psi;
    if (l < NU) S.wv[l] = w;
    w_out = w;
    wsync();
    const double xn = ax + oB.apply(S.wv);
    wsync();
    if (l < NX) S.x[l] = xn;
    wsync();
}

// 1/2 x'Px - Psi'x + cbar (value of the cost to go at x).
template <int NX, int NU, class TP>
__device__ __forceinline__ double cost_to_go(const VSmem<NX, NU> &S, const TP *P, double cbar) {
    const int l = lane();
    Op<NX, NX> oP;
    oP.template load<false>(P, NX);
    const double px = oP.apply(S.x);
    const double part = l < NX ? S.x[l] * (0.5 * px - S.Psi[l]) : 0.0;
    return wave_sum(part) + cbar;
}

__device__ __forceinline__ TreeItem load_item(const TreeItem *tab, int i) {
    const TreeItem r = tab[i];
    TreeItem u;
    u.kind = uni(r.kind);
    u.inst = uni(r.inst);
    u.level = uni(r.level);
    u.first = uni(r.first);
    u.count = uni(r.count);
    u.last = uni(r.last);
    u.term_slot = uni(r.term_slot);
    u.out_slot = uni(r.out_slot);
    u.dep_first = uni(r.dep_first);
    u.dep_count = uni(r.dep_count);
    return u;
}

template <int NX>
__device__ __forceinline__ VSrc<double> slot_src(const double *sl) {
    const SlotLayout L{NX};
    VSrc<double> q;
    q.Pn = nullptr;
    q.Pn64 = nullptr;
    q.Vn = nullptr;
    q.A = sl + L.A();
    q.B = sl + L.Qw();
    q.a = sl + L.a();
    q.lx = sl + L.lx();
    q.lw = nullptr;
    q.c = sl[L.c()];
    return q;
}

// -------------------------------------------------------------- the tree
template <int NX>
__global__ void __launch_bounds__(WT) kv_tree(GroupArgs g) {
    __shared__ VSmem<NX, NX> S;
    __shared__ int s_item;
    const int l = lane();
    const SlotLayout SL{NX};
    double *slots = uni_ptr(g.slots);
    auto slot = [&](int s) { return slots + (int64_t)s * SL.size(); };
    if (pass_idle(g)) return;
    for (;;) {
        if (l == 0) s_item = atomicAdd(g.queue, 1);
        wsync();
        const int idx = uni(s_item);
        wsync();
        if (idx >= g.nitems) break;
        const TreeItem it = load_item(g.items, idx);
        if (l == 0) {
            for (int d = 0; d < it.dep_count; ++d) {
                int spins = 0;
                while (__hip_atomic_load(&g.flags[it.dep_first + d], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) !=
                       g.epoch) {
                    __builtin_amdgcn_s_sleep(4);
                    if (++spins > SPIN_LIMIT) {
                        int32_t *inf = g.info + 2 * it.inst;
                        atomicCAS(inf, 0, 6);
                        atomicCAS(inf + 1, -1, -2);
                        break;
                    }
                }
            }
        }
        wsync();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int count = it.count;
        if (skip_inst(g, it.inst)) {
            // converged: nothing to do (its dependents belong to the same instance)
        } else if (it.kind == ITEM_UP || it.kind == ITEM_UP_LAST) {
            const bool red = it.kind == ITEM_UP;
            const double *term = red ? nullptr : slot(it.term_slot);
            if (l < NX) {
                S.Psi[l] = red ? 0.0 : -term[SL.lx() + l];
                S.v[l] = 0.0;
            }
            double cbar = red ? 0.0 : term[SL.c()];
            wsync();
            for (int s = count - 1; s >= 0; --s) {
                double *sl = slot(it.first + s);
                VSrc<double> q = slot_src<NX>(sl);
                const double *sn = slot(it.first + s + 1);
                const bool end = s + 1 == count;
                q.Li = sl + SL.uL();
                q.LT = sl + SL.uLT();
                q.K = sl + SL.uK();
                auto keep = [](double, double) {};
                if (red) {
                    q.Pn = end ? nullptr : sn + SL.uP();
                    q.Vn = end ? nullptr : sn + SL.uV();
                    vstage<NX, NX, true, false>(S, q, cbar, keep);
                } else {
                    q.Pn = end ? term + SL.Qx() : sn + SL.uP();
                    q.Vn = nullptr;
                    vstage<NX, NX, false, true>(S, q, cbar, keep);
                }
            }
            double *out = slot(it.out_slot);
            if (l < NX) {
                if (red) out[SL.a() + l] = S.v[l];
                out[SL.lx() + l] = -S.Psi[l];
            }
            if (l == 0) out[SL.c()] = cbar;
        } else {
            const bool top = it.kind == ITEM_TOP;
            const Prob p = load_prob(g.probs, it.inst);
            const double *msg = top ? nullptr : slot(it.out_slot);
            const double *term = it.last ? slot(it.term_slot) : nullptr;
            if (l < NX) {
                S.Psi[l] = term ? -term[SL.lx() + l] : msg[SL.Psi() + l];
                S.x[l] = top ? p.x0[l] : msg[SL.xh() + l];
            }
            double cbar = term ? term[SL.c()] : msg[SL.cb()];
            wsync();
            for (int s = count - 1; s >= 0; --s) {
                double *sl = slot(it.first + s);
                // message to child s: cost to go at the end of master stage s
                if (l < NX) sl[SL.Psi() + l] = S.Psi[l];
                if (l == 0) sl[SL.cb()] = cbar;
                VSrc<double> q = slot_src<NX>(sl);
                q.Pn = sl + SL.P();
                q.Vn = nullptr;
                q.Li = sl + SL.dL();
                q.LT = sl + SL.dLT();
                q.K = sl + SL.K();
                vstage<NX, NX, false, true>(S, q, cbar, [&](double, double k) {
                    if (l < NX) sl[SL.k() + l] = k;
                });
            }
            if (top && p.obj) {
                const double v = cost_to_go<NX, NX>(S, slot(it.term_slot) + SL.P(), cbar);
                if (l == 0) p.obj[0] = v;
            }
            wsync();
            for (int s = 0; s < count; ++s) {
                double *sl = slot(it.first + s);
                if (l < NX) sl[SL.xh() + l] = S.x[l];
                double lam, w;
                fstage<NX, NX, false, double>(S, sl + SL.K(), sl + SL.k(), sl + SL.A(), sl + SL.Qw(), sl + SL.a(),
                                              nullptr, nullptr, lam, w);
            }
            if (it.last && l < NX) slot(it.term_slot)[SL.xh() + l] = S.x[l];
        }
        __threadfence();
        wsync();
        if (l == 0) __hip_atomic_store(&g.flags[idx], g.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        wsync();
    }
}

template <class TR>
hipError_t launch_up(const GroupArgs &g, int, hipStream_t st) {
    return sweep_leaf(g, sizeof(TR) == 4, false, st);
}
template <int NX>
hipError_t launch_tree(const GroupArgs &g, int grid, hipStream_t st) {
    if (g.superpose) return sweep_tree(g, grid, st);
    hipLaunchKernelGGL((kv_tree<NX>), dim3(grid), dim3(WT), 0, st, g);
    return hipGetLastError();
}
template <class TR>
hipError_t launch_down(const GroupArgs &g, int, hipStream_t st) {
    return sweep_leaf(g, sizeof(TR) == 4, true, st);
}

}  // namespace sv

// which: 0 leaf up, 1 tree, 2 leaf down; fp32: the leaf records are FP32.
Launcher vector_solve(int nx, int nu, int which, bool fp32) {
#define RS_VEC(a, b)                                                                   \
    if (nx == a && nu == b) {                                                          \
        if (which == 1) return &sv::launch_tree<a>;                                    \
        if (which == 0) return fp32 ? &sv::launch_up<float> : &sv::launch_up<double>;  \
        return fp32 ? &sv::launch_down<float> : &sv::launch_down<double>;              \
    }
    RS_VEC(16, 16)
    RS_VEC(32, 16)
    RS_VEC(32, 32)
#undef RS_VEC
    return nullptr;
}

}  // namespace rs
