// Fused FP64 solve (factor and right-hand side in one pass, no stored
// factorization) for n_x <= 32 on the column-owner engine (rs_col.hpp):
//   kf_leaf   one workgroup per leaf.  Up: Alg. 4, or elimination with the true
//             terminal; down: elimination with the true terminal and Alg. 3
//   kf_tree   work queue over the master levels: Alg. 5 up, the top solve, and
//             Alg. 6 down to level 1
// Shapes of full tiles (n_x and n_u multiples of 16) keep K, k, P, Psi, V and
// L_t of every stage of the up pass, and everything below the top is a forward
// sweep on them by superposition (fused_leaf_forward for the leaves; whole-
// problem leaves go through kf_leaf).  The others (run-time sizes, n_x = 4, 8,
// 20, ...) are eliminated again with the parent's P and Psi, keeping K, k, P and
// Psi of that pass: there the superposition's w = K x + k + L_t lam_N, whose
// L_t does not know the terminal, would pass the rounding of lam_N on undamped
// (2 times the error of elimination on average, 10 times with small state
// weights and unstable dynamics; it would take 69 us instead of 81 for one
// problem of 4 x 2, N = 64, and 275 instead of 380 for 20 x 10, N = 1024).
// Sizes below the tiles are padded on load, as are the inputs of instances with
// fewer inputs than their group's tile (g.data_nu).
//
// Bound: the dependent chain of a stage; on large batches the workgroups that
// share a CU fill one another's waits, and the records' bytes are next.  FP64,
// the whole solve before (a four-wave tile engine with every product through
// LDS for full tiles, vector-unit kernels below them that factored the master
// levels twice) and now: one problem of N = 1024, 32 x 16 505 -> 250 us and
// 20 x 10 862 -> 380 us; 4 x 2, N = 64 129 -> 81 us; 512 problems of 32 x 16,
// N = 1024 13.6 -> 10.1 ms (leaves 10.2 -> 6.8 ms); 1024 of 16 x 8, N in [32,
// 2048] 14.9 -> 7.0 ms (padding on load instead of padded copies: 1.3 ms).
#include <hip/hip_runtime.h>

#include "rs_col.hpp"
#include "rs_launch.hpp"
#include "rs_vsweep.hpp"

namespace rs {
namespace cw {

// Sizes: all of the tile's (FULL), the tile's with each instance's own number
// of inputs in the data (DATA), or run-time (ANY).
enum { FULL = 0, DATA = 1, ANY = 2 };

template <int NXT, int NUT, int SZ, int SX = 4, int SU = 4>
__global__ void __launch_bounds__(128 * NXT, NXT == 1 ? 4 : NUT == 1 ? 3 : 2) kf_leaf(GroupArgs g, int down) {
    using SM = Smem<double, NXT, NUT, SX, SU>;
    constexpr int W = 2 * NXT;
    constexpr bool EX = SZ != ANY, EXD = SZ == FULL;
    __shared__ SM S;
    __shared__ vs::Smem<SM::RX, SM::RU, W> F;
    const LeafItem it = load_leaf_u(g.leaves, my_leaf(g));
    const bool top = (it.flags & LEAF_TOP) != 0, last = (it.flags & LEAF_LAST) != 0;
    if ((down ? EX && !top : top) || inst_skipped(g.probs, it.inst)) return;
    const DevProb p = load_prob(g.probs, it.inst);
    const int n = EX ? SM::RX : g.nx, m = EX ? SM::RU : g.nu, md = SZ == DATA ? p.nu : m, tid = threadIdx.x;
    const SlotLayout SL{n};
    double *out = g.slots + (int64_t)it.slot * SL.size();
    double *base = static_cast<double *>(g.leaf_scratch) + it.scratch;
    const int len = leaf_rec_len(n, m);
    const StageWalk wk = prob_walk(p, it.t0 + it.len - 1);
    auto no_pre = [](int, int, int) {};
    auto rec = [&](int s) {
        double *K = base + (int64_t)s * len, *P = K + m * n + m, *V = P + n * n + n;
        return Rec<double>{P, K, V, V + n * n, nullptr, nullptr, P + n * n, K + m * n};
    };
    const Ln<double> L;
    const int w = wave(), col = 16 * (w < NXT ? w : w - NXT) + L.c;
    const bool own = L.q == 0 && col < n;            // owner lane of entry col
    Cols<double, NXT> C;
    Vec y{};
    if (!down && !last) {
        set_P(S, n, [](int) { return 0.0; });
        pass<true, EX, EXD, true, EX>(S, C, n, m, md, wk, it.len, g.info, it.inst, it.t0, 2, no_pre, rec, y);
        store_V_transposed<SX>(C, out + SL.A(), n);
        copy_P(S, out + SL.Qx(), n);
        if (!g.ident) store_Q<SX>(C, out + SL.Qw(), n);
        if (own && w >= NXT) out[SL.a() + col] = y.v;
    } else if (!down || top || !last) {
        // from the true terminal: the parent's message, or the problem's own
        // (whose records, kept by the up pass, also serve the down pass)
        const double *P0 = last ? p.QxN : out + SL.P();
        set_P(S, n, [&](int e) { return P0[e]; });
        if (w < NXT && col < n) y.psi = !last ? out[SL.Psi() + col] : p.lN ? -p.lN[col] : 0.0;
        pass<false, EX, EXD, true>(S, C, n, m, md, wk, it.len, g.info, it.inst, it.t0, 2, no_pre, rec, y);
        if (!down) copy_P(S, out + SL.Qx(), n);
    }
    if (!down || top) {
        const double c = total(S, y.cb + vs::sum_c(p.c ? p.c + (int64_t)it.t0 * p.sc : nullptr, p.sc, it.len)) +
                         ((last && p.cN) ? p.cN[0] : 0.0);
        if (!down) {
            if (own && w < NXT) out[SL.lx() + col] = -y.psi;
            if (tid == 0) out[SL.c()] = c;
            if (g.ident && !last) {
                store_Q<SX>(C, S.A, n);              // A is dead: Q_w_hat, row-major
                rank_reveal_rows<SM::RX>(S.A, n, unit_roundoff<double>(), out + SL.Qw(), nullptr);
            }
            return;
        }
        if (p.obj) {
            // whole problem: optimal value 1/2 x0'P_0 x0 - Psi_0'x0 + cbar_0
            for (int e = tid; e < SM::RX; e += SM::NTH) F.x[e] = e < n ? p.x0[e] : 0.0;
            __syncthreads();
            double px = 0.0;
            if (w < NXT) {
#pragma unroll
                for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                    for (int r = 0; r < SX; ++r) px += ldN<SM::RX>(L, S.P, kt, w, r) * F.x[16 * kt + L.row(r)];
                px = q_sum(px);
            }
            const double o = total(S, (own && w < NXT) ? F.x[col] * (0.5 * px - y.psi) : 0.0);
            if (tid == 0) p.obj[0] = o + c;
        }
    }
    // ---- Alg. 3
    const double *x0 = top ? p.x0 : out + SL.xh();
    for (int e = tid; e < SM::RX; e += SM::NTH) F.x[e] = e < n ? x0[e] : 0.0;
    __threadfence_block();                   // the records are read back by other lanes
    __syncthreads();
    const int64_t t0 = it.t0;
    vs::forward<SM::RX, SM::RU, W, EX, EXD, double>(
        F, n, m, md, it.len, vs::FusedStages{sv::load_prob(g.probs, it.inst), it.t0, n, m, base}, false,
        [&](int s) { return p.x + (t0 + s) * n; }, [&](int s) { return p.w + (t0 + s) * md; },
        [&](int s) { return p.lam + (t0 + s) * n; });
    if (!last) return;
    const int64_t t = t0 + it.len;
    const double q = vs::sym_apply<SM::RX, SM::RU, W>(p.QxN, F.x, n);
    typedef vs::Mat<double, SM::RX, SM::RX, W> MA;
    const int i = MA::out_row();
    if (MA::lead_row() && i < n) {
        p.lam[t * n + i] = q + (p.lN ? p.lN[i] : 0.0);          // lam_N = QxN x_N + lN
        p.x[t * n + i] = F.x[i];
    }
}

// EX: full tiles.
template <int NXT, bool EX, int SX = 4>
__global__ void __launch_bounds__(128 * NXT, 2) kf_tree(GroupArgs g) {
    using SM = Smem<double, NXT, NXT, SX, SX>;
    constexpr int W = 2 * NXT, NM = SM::RX;
    __shared__ SM S;
    __shared__ vs::Smem<NM, NM, W> F;
    __shared__ int s_item;
    const int n = EX ? NM : g.nx, tid = threadIdx.x;
    const SlotLayout SL{n};
    double *slots = g.slots;
    auto slot = [&](int s) { return slots + (int64_t)s * SL.size(); };
    typedef vs::Mat<double, NM, NM, W> MA;
    for (;;) {
        if (tid == 0) s_item = atomicAdd(g.queue, 1);
        __syncthreads();
        const int idx = uni(s_item);
        __syncthreads();
        if (idx >= g.nitems) break;
        const TreeItem it = load_item_u(g.items, idx);
        wait_deps(g, it);
        const StageWalk wk = slot_walk(slot(it.first + it.count - 1), n, g.ident);
        auto no_pre = [](int, int, int) {};
        auto c_sum = [&] { return vs::sum_c(slot(it.first) + SL.c(), SL.size(), it.count); };
        const Ln<double> L;
        const int w = wave(), col = 16 * (w < NXT ? w : w - NXT) + L.c;
        const bool own = L.q == 0 && col < n;
        const int ir = MA::out_row();
        const bool ownr = MA::lead_row() && ir < n;
        auto none = [](int) { return (double *)nullptr; };
        // forward with the K and k of the item's stages, x to the children
        auto solve = [&] {
            auto st = [&](int s) {
                vs::Stage<double> q = vs::SlotStages{slots, it.first, n, false}(s);
                q.P = nullptr;
                return q;
            };
            vs::forward<NM, NM, W, EX, EX, double>(F, n, n, n, it.count, st, false,
                                                   [&](int s) { return slot(it.first + s) + SL.xh(); }, none, none);
        };
        const bool last = it.last != 0;
        Cols<double, NXT> C;
        Vec y{};
        if (inst_skipped(g.probs, it.inst)) {
            // excluded instance: only its completion flag is published
        } else if (it.kind == ITEM_UP) {
            set_P(S, n, [](int) { return 0.0; });
            pass<true, EX, EX, true, EX>(S, C, n, n, n, wk, it.count, g.info, it.inst, -1, 3, no_pre, [&](int s) {
                double *d = slot(it.first + s);
                return Rec<double>{d + SL.uP(), d + SL.uK(), d + SL.uV(), d + SL.dL(), nullptr, nullptr, d + SL.Psi(),
                                   d + SL.k()};
            }, y);
            double *out = slot(it.out_slot);
            store_V_transposed<SX>(C, out + SL.A(), n);
            copy_P(S, out + SL.Qx(), n);
            if (!g.ident) store_Q<SX>(C, out + SL.Qw(), n);
            const double c = total(S, y.cb + c_sum());
            if (own) out[(w < NXT ? SL.lx() : SL.a()) + col] = w < NXT ? -y.psi : y.v;
            if (tid == 0) out[SL.c()] = c;
            if (g.ident) {
                store_Q<SX>(C, S.A, n);
                rank_reveal_rows<SM::RX>(S.A, n, unit_roundoff<double>(), out + SL.Qw(), nullptr);
            }
        } else if (it.kind != ITEM_DOWN || (!EX && !last)) {
            // Alg. 1-2 from the true terminal: the level's own, or the
            // parent's message.  The level's last item keeps its up records
            // (full tiles); the others keep K and k and send P and Psi to
            // their children.
            const bool top = it.kind == ITEM_TOP, upl = it.kind == ITEM_UP_LAST, msgs = !EX || top;
            double *end = slot(it.kind == ITEM_DOWN ? it.out_slot : it.term_slot);
            const double *P0 = end + (it.kind == ITEM_DOWN ? SL.P() : SL.Qx());
            set_P(S, n, [&](int e) { return P0[e]; });
            if (w < NXT && col < n) y.psi = it.kind == ITEM_DOWN ? end[SL.Psi() + col] : -end[SL.lx() + col];
            if (msgs) {
                double *d = slot(it.first + it.count - 1);
                __syncthreads();
                copy_P(S, d + SL.P(), n);
                if (own && w < NXT) d[SL.Psi() + col] = y.psi;
            }
            pass<false, EX, EX, true>(S, C, n, n, n, wk, it.count, g.info, it.inst, -1, 3, no_pre, [&](int s) {
                double *d = slot(it.first + s);
                if (!msgs)
                    return Rec<double>{d + SL.uP(), d + SL.uK(), nullptr, nullptr, nullptr, nullptr, d + SL.Psi(),
                                       d + SL.k()};
                double *c = slot(it.first + (s > 0 ? s - 1 : 0));
                return Rec<double>{s > 0 ? c + SL.P() : nullptr, d + SL.K(), nullptr, nullptr, nullptr, nullptr,
                                   s > 0 ? c + SL.Psi() : nullptr, d + SL.k()};
            }, y);
            double c = 0.0;
            if (top || upl) c = total(S, y.cb + c_sum()) + end[SL.c()];
            if (upl) {
                double *out = slot(it.out_slot);
                copy_P(S, out + SL.Qx(), n);
                if (own && w < NXT) out[SL.lx() + col] = -y.psi;
                if (tid == 0) out[SL.c()] = c;
            } else {
                const DevProb p = load_prob(g.probs, it.inst);
                const double *x0 = top ? p.x0 : end + SL.xh();
                for (int e = tid; e < NM; e += SM::NTH) F.x[e] = e < n ? x0[e] : 0.0;
                __threadfence_block();       // K, k and the messages are read back by other lanes
                __syncthreads();
                if (top && p.obj) {
                    double px = 0.0;
                    if (w < NXT) {
#pragma unroll
                        for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                            for (int r = 0; r < SX; ++r) px += ldN<NM>(L, S.P, kt, w, r) * F.x[16 * kt + L.row(r)];
                        px = q_sum(px);
                    }
                    const double o = total(S, (own && w < NXT) ? F.x[col] * (0.5 * px - y.psi) : 0.0);
                    if (tid == 0) p.obj[0] = o + c;
                }
                solve();
                if (top && ownr) end[SL.xh() + ir] = F.x[ir];
                if constexpr (EX) {
                    // terminal costate of child s, lam_{s+1} = P_{s+1} x_{s+1} -
                    // Psi_{s+1}, from the cost to go sent to it and the initial
                    // state of the next child (of the terminal node for the last)
                    __threadfence_block();
                    __syncthreads();
                    for (int s = 0; s < it.count; ++s) {
                        double *d = slot(it.first + s);
                        const double *xn = (s + 1 < it.count ? slot(it.first + s + 1) : end) + SL.xh();
                        for (int e = tid; e < n; e += SM::NTH) F.x[e] = xn[e];
                        sv::wsync();
                        const double l = vs::sym_apply<NM, NM, W>(d + SL.P(), F.x, n);
                        if (ownr) d[SL.lamN() + ir] = l - d[SL.Psi() + ir];
                        sv::wsync();
                    }
                }
            }
        } else if constexpr (!EX) {
            // the level's last item: solved on the K and k of its up pass,
            // which started from the same terminal
            const double *msg = slot(it.out_slot);
            for (int e = tid; e < NM; e += SM::NTH) F.x[e] = e < n ? msg[SL.xh() + e] : 0.0;
            __syncthreads();
            solve();
            if (ownr) slot(it.term_slot)[SL.xh() + ir] = F.x[ir];
        } else {
            // down pass below the top (Alg. 6, k >= 1) on the up records:
            // child s receives x_s and its terminal costate lam_{s+1}
            const double *msg = slot(it.out_slot);
            for (int e = tid; e < NM; e += SM::NTH) {
                F.x[e] = e < n ? msg[SL.xh() + e] : 0.0;
                F.lamN[e] = (!last && e < n) ? msg[SL.lamN() + e] : 0.0;
            }
            __syncthreads();
            vs::forward<NM, NM, W, EX, EX, double>(
                F, n, n, n, it.count, vs::SlotStages{slots, it.first, n, true}, !last,
                [&](int s) { return slot(it.first + s) + SL.xh(); }, none,
                [&](int s) { return s > 0 ? slot(it.first + s - 1) + SL.lamN() : (double *)nullptr; });
            // the last child ends where the item does: at lam_N, or for the
            // last item at the terminal node, lam = P_term x - Psi_term
            double *lend = slot(it.first + it.count - 1) + SL.lamN();
            if (last) {
                double *term = slot(it.term_slot);
                const double l = vs::sym_apply<NM, NM, W>(term + SL.Qx(), F.x, n);
                if (ownr) {
                    lend[ir] = l + term[SL.lx() + ir];
                    term[SL.xh() + ir] = F.x[ir];
                }
            } else if (ownr) {
                lend[ir] = F.lamN[ir];
            }
        }
        publish(g, idx);
    }
}

// Superposition on the records of the up pass, or elimination with the true
// terminal (see above).
bool full_tiles(const GroupArgs &g) { return g.nx % 16 == 0 && g.nu % 16 == 0; }

template <int A, int B>
hipError_t fused_leaf(const GroupArgs &g, int down, hipStream_t st) {
    const dim3 grid(g.nleaves), block(128 * A);
    if constexpr (A == 1) {
        // one or two slices of the tile
        if (g.nx <= 4 && g.nu <= 4) {
            hipLaunchKernelGGL((kf_leaf<A, B, ANY, 1, 1>), grid, block, 0, st, g, down);
            return hipGetLastError();
        }
        if (g.nx <= 8 && g.nu <= 4) {
            hipLaunchKernelGGL((kf_leaf<A, B, ANY, 2, 1>), grid, block, 0, st, g, down);
            return hipGetLastError();
        }
    }
    if (!full_tiles(g))
        hipLaunchKernelGGL((kf_leaf<A, B, ANY>), grid, block, 0, st, g, down);
    else if (g.data_nu)
        hipLaunchKernelGGL((kf_leaf<A, B, DATA>), grid, block, 0, st, g, down);
    else
        hipLaunchKernelGGL((kf_leaf<A, B, FULL>), grid, block, 0, st, g, down);
    return hipGetLastError();
}
hipError_t fused_leaf_any(const GroupArgs &g, int down, hipStream_t st) {
    if (g.nx <= 16) return fused_leaf<1, 1>(g, down, st);
    if (g.nu <= 16) return fused_leaf<2, 1>(g, down, st);
    return fused_leaf<2, 2>(g, down, st);
}

hipError_t launch_up(const GroupArgs &g, int, hipStream_t st) {
    return g.ntop == g.nleaves ? hipSuccess : fused_leaf_any(g, 0, st);
}
hipError_t launch_tree(const GroupArgs &g, int grid, hipStream_t st) {
    const dim3 gd(grid);
    if (full_tiles(g) && g.nx == 16)
        hipLaunchKernelGGL((kf_tree<1, true>), gd, dim3(128), 0, st, g);
    else if (full_tiles(g))
        hipLaunchKernelGGL((kf_tree<2, true>), gd, dim3(256), 0, st, g);
    else if (g.nx <= 4)
        hipLaunchKernelGGL((kf_tree<1, false, 1>), gd, dim3(128), 0, st, g);
    else if (g.nx <= 8)
        hipLaunchKernelGGL((kf_tree<1, false, 2>), gd, dim3(128), 0, st, g);
    else if (g.nx <= 16)
        hipLaunchKernelGGL((kf_tree<1, false>), gd, dim3(128), 0, st, g);
    else
        hipLaunchKernelGGL((kf_tree<2, false>), gd, dim3(256), 0, st, g);
    return hipGetLastError();
}
hipError_t launch_down(const GroupArgs &g, int, hipStream_t st) {
    if (!full_tiles(g)) return fused_leaf_any(g, 1, st);
    if (g.ntop > 0) {
        const hipError_t e = fused_leaf_any(g, 1, st);
        if (e != hipSuccess || g.ntop == g.nleaves) return e;
    }
    return fused_leaf_forward(g, st);
}

}  // namespace cw

Launcher fused_solve(int nx, int nu, int which) {
    if (nx > 32 || !mid_shape(nx, nu)) return nullptr;
    return which == 0 ? &cw::launch_up : which == 1 ? &cw::launch_tree : &cw::launch_down;
}

}  // namespace rs
