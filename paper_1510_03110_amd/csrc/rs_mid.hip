// Stored factorization up to n_x = 64 (n_u <= n_x in tiles of 16): the
// column-owner stage engine (rs_col.hpp), with run-time sizes or sizes that
// fill the tiles, in place of the global-memory workspace
// of the large-block kernels.  Same records, slots and work tables, so the
// vector passes of the large-block family solve on them.
//
// Bound: the dependent chain of a stage (G, its Cholesky factorization, Y, P)
// on one workgroup per CU at n_x = 64 (123 KB of LDS), then the matrix cores.
// (64, 32), FP64, 1024 leaves of 64 stages: 23 us a stage, 38 TFLOP/s (98 us
// with every operand read through the L2); a 64 x 64 master stage takes about
// 55 us (161 us); 8 x 4 stages (one tile, two wavefronts) 4 us (13.6 us).
//   kc_leaf   one workgroup per leaf: Alg. 4 or the last-leaf elimination (up),
//             Alg. 1 with the true terminal on whole-problem leaves (down)
//   kc_tree   work queue over the master levels
#include <hip/hip_runtime.h>

#include "rs_col.hpp"
#include "rs_launch.hpp"

namespace rs {
namespace cw {

// One workgroup per leaf.  Up (down = 0): leaves of multi-leaf instances;
// down (down = 1): whole-problem leaves, the only ones that need the
// factorization with the true terminal (the others are solved from their up
// records).
template <class T, int NXT, int NUT, bool EX, int SX = 4, int SU = 4>
__global__ void __launch_bounds__(128 * NXT, 2) kc_leaf(GroupArgs g, int down) {
    using SM = Smem<T, NXT, NUT, SX, SU>;
    __shared__ SM S;
    const LeafItem it = load_leaf_u(g.leaves, my_leaf(g));
    if (((it.flags & LEAF_TOP) != 0) != (down != 0) || inst_skipped(g.probs, it.inst)) return;
    const int n = EX ? SM::RX : g.nx, m = EX ? SM::RU : g.nu, tid = threadIdx.x;
    const SlotLayout SL{n};
    const LeafRec R{n, m};
    double *out = g.slots + (int64_t)it.slot * SL.size();
    if (it.flags & LEAF_REUSE) {
        // stored factorization current (receding-horizon plans): only its
        // cached M1 goes to this call's slot
        const double *c = g.m1cache + (int64_t)it.m1 * 3 * n * n;
        for (int e = tid; e < 3 * n * n; e += SM::NTH) out[e] = c[e];
        return;
    }
    const DevProb p = load_prob(g.probs, it.inst);
    double *cache = (g.m1cache && it.m1 >= 0) ? g.m1cache + (int64_t)it.m1 * 3 * n * n : nullptr;
    T *base = reinterpret_cast<T *>(g.fstore) + g.rec_stage(it.scratch) * (int64_t)R.per_stage();
    const StageWalk wk = prob_walk(p, it.t0 + it.len - 1);
    auto no_pre = [](int, int, int) {};
    Cols<T, NXT> C;
    Vec y{};
    if (!(it.flags & LEAF_LAST)) {
        set_P(S, n, [](int) { return 0.0; });
        pass<true, EX, EX, false>(S, C, n, m, m, wk, it.len, g.info, it.inst, it.t0, 2, no_pre, [&](int s) {
            T *d = base + (int64_t)s * R.per_stage();
            return Rec<T>{d + R.P(), d + R.K(), d + R.V(), d + R.Lt(), d + R.L(), d + R.LT(), nullptr, nullptr};
        }, y);
        store_V_transposed<SX>(C, out + SL.A(), n);
        copy_P(S, out + SL.Qx(), n);
        if (!g.ident) store_Q<SX>(C, out + SL.Qw(), n);
        if (cache) {
            store_V_transposed<SX>(C, cache + SL.A(), n);
            copy_P(S, cache + SL.Qx(), n);
            if (!g.ident) store_Q<SX>(C, cache + SL.Qw(), n);
        }
        if (g.ident) {
            store_Q<SX>(C, S.A, n);              // A is dead: Q_w_hat, row-major
            rank_reveal_rows<SM::RX>(S.A, n, unit_roundoff<T>(), out + SL.Qw(), cache ? cache + SL.Qw() : nullptr);
        }
    } else {
        if (down) base += R.up();
        set_P(S, n, [&](int e) { return p.QxN[e]; });
        pass<false, EX, EX, false>(S, C, n, m, m, wk, it.len, g.info, it.inst, it.t0, 2, no_pre, [&](int s) {
            T *d = base + (int64_t)s * R.per_stage();
            return Rec<T>{d + R.P(), d + R.K(), nullptr, nullptr, d + R.L(), d + R.LT(), nullptr, nullptr};
        }, y);
        if (!down) copy_P(S, out + SL.Qx(), n);
    }
}

#ifndef RS_MID_FP32
template <int NXT, bool EX, int SX = 4>
__global__ void __launch_bounds__(128 * NXT, 2) kc_tree(GroupArgs g) {
    using SM = Smem<double, NXT, NXT, SX, SX>;
    __shared__ SM S;
    __shared__ int s_item;
    const int n = EX ? SM::RX : g.nx, tid = threadIdx.x;
    const SlotLayout SL{n};
    double *slots = g.slots;
    auto slot = [&](int s) { return slots + (int64_t)s * SL.size(); };
    for (;;) {
        if (tid == 0) s_item = atomicAdd(g.queue, 1);
        __syncthreads();
        const int idx = uni(s_item);
        __syncthreads();
        if (idx >= g.nitems) break;
        const TreeItem it = load_item_u(g.items, idx);
        wait_deps(g, it);
        const StageWalk wk = slot_walk(slot(it.first + it.count - 1), n, g.ident);
        Cols<double, NXT> C;
        Vec y{};
        if (inst_skipped(g.probs, it.inst)) {
            // excluded instance: only its completion flag is published
        } else if (it.kind == ITEM_UP) {
            set_P(S, n, [](int) { return 0.0; });
            pass<true, EX, EX, false>(S, C, n, n, n, wk, it.count, g.info, it.inst, -1, 3, [](int, int, int) {}, [&](int s) {
                double *d = slot(it.first + s);
                return Rec<double>{d + SL.uP(), d + SL.uK(), d + SL.uV(), g.superpose ? d + SL.dL() : nullptr,
                                   d + SL.uL(), d + SL.uLT(), nullptr, nullptr};
            }, y);
            double *out = slot(it.out_slot);
            store_V_transposed<SX>(C, out + SL.A(), n);
            copy_P(S, out + SL.Qx(), n);
            if (!g.ident) {
                store_Q<SX>(C, out + SL.Qw(), n);
            } else {
                store_Q<SX>(C, S.A, n);
                rank_reveal_rows<SM::RX>(S.A, n, unit_roundoff<double>(), out + SL.Qw(), nullptr);
            }
        } else if (it.kind == ITEM_DOWN && g.superpose) {
            // solved by the vector pass from the up records: nothing to factor
        } else {
            // Alg. 1 on the master stages from the true terminal (a level's
            // last item, up records) or from the parent's message (down
            // records; top, and below it without superposition)
            const bool upl = it.kind == ITEM_UP_LAST;
            const double *msg = it.kind == ITEM_DOWN ? slot(it.out_slot) : nullptr;
            double *term = it.last ? slot(it.term_slot) : nullptr;
            const double *P0 = term ? term + SL.Qx() : msg + SL.P();
            set_P(S, n, [&](int e) { return P0[e]; });
            pass<false, EX, EX, false>(S, C, n, n, n, wk, it.count, g.info, it.inst, -1, 3,
                            [&](int s, int t0, int t1) {      // M2 for child s: P at the end of master stage s
                                if (!upl) copy_P(S, slot(it.first + s) + SL.P(), n, t0, t1);
                            },
                            [&](int s) {
                                double *d = slot(it.first + s);
                                return upl ? Rec<double>{d + SL.uP(), d + SL.uK(), nullptr, nullptr, d + SL.uL(),
                                                         d + SL.uLT(), nullptr, nullptr}
                                           : Rec<double>{nullptr, d + SL.K(), nullptr, nullptr, d + SL.dL(),
                                                         d + SL.dLT(), nullptr, nullptr};
                            }, y);
            // a level's last item: its reduced terminal; the top: P_0, for the optimal value
            double *d = upl ? slot(it.out_slot) + SL.Qx() : it.kind == ITEM_TOP ? term + SL.P() : nullptr;
            if (d) copy_P(S, d, n);
        }
        publish(g, idx);
    }
}
#endif

inline int tiles(int d) { return (d + 15) / 16; }

// Sizes that fill the tiles have an instance without bounds checks: n_x of 16, 32
// and 64, the shapes that the workloads use; 48 states, and in FP32 64 with more
// than 32 inputs, run on the checked one (not measured against each other).
template <class T, int A, int B>
hipError_t leaf(const GroupArgs &g, hipStream_t st, int down) {
    const dim3 grid(g.nleaves), block(128 * A);
    if constexpr (A != 3 && (sizeof(T) == 8 || A < 4 || B < 3)) {
        if (g.nx == 16 * A && g.nu == 16 * B) {
            hipLaunchKernelGGL((kc_leaf<T, A, B, true>), grid, block, 0, st, g, down);
            return hipGetLastError();
        }
    }
    if constexpr (A == 1 && sizeof(T) == 8) {
        // one or two slices of the tile
        if (g.nx <= 4 && g.nu <= 4)
            hipLaunchKernelGGL((kc_leaf<T, A, B, false, 1, 1>), grid, block, 0, st, g, down);
        else if (g.nx <= 8 && g.nu <= 4)
            hipLaunchKernelGGL((kc_leaf<T, A, B, false, 2, 1>), grid, block, 0, st, g, down);
        else
            hipLaunchKernelGGL((kc_leaf<T, A, B, false>), grid, block, 0, st, g, down);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((kc_leaf<T, A, B, false>), grid, block, 0, st, g, down);
    return hipGetLastError();
}

template <class T>
hipError_t leaf_any(const GroupArgs &g, hipStream_t st, int down) {
    switch (10 * tiles(g.nx) + tiles(g.nu)) {
    case 11: return leaf<T, 1, 1>(g, st, down);
    case 21: return leaf<T, 2, 1>(g, st, down);
    case 22: return leaf<T, 2, 2>(g, st, down);
    case 31: return leaf<T, 3, 1>(g, st, down);
    case 32: return leaf<T, 3, 2>(g, st, down);
    case 33: return leaf<T, 3, 3>(g, st, down);
    case 41: return leaf<T, 4, 1>(g, st, down);
    case 42: return leaf<T, 4, 2>(g, st, down);
    case 43: return leaf<T, 4, 3>(g, st, down);
    case 44: return leaf<T, 4, 4>(g, st, down);
    }
    return hipErrorInvalidValue;
}

#ifndef RS_MID_FP32
template <int A>
hipError_t tree(const GroupArgs &g, int grid, hipStream_t st) {
    if constexpr (A == 1) {
        if (g.nx <= 4) {
            hipLaunchKernelGGL((kc_tree<A, false, 1>), dim3(grid), dim3(128 * A), 0, st, g);
            return hipGetLastError();
        }
        if (g.nx <= 8) {
            hipLaunchKernelGGL((kc_tree<A, false, 2>), dim3(grid), dim3(128 * A), 0, st, g);
            return hipGetLastError();
        }
    }
    if (g.nx == 16 * A)
        hipLaunchKernelGGL((kc_tree<A, true>), dim3(grid), dim3(128 * A), 0, st, g);
    else
        hipLaunchKernelGGL((kc_tree<A, false>), dim3(grid), dim3(128 * A), 0, st, g);
    return hipGetLastError();
}
#endif

}  // namespace cw

// Leaves of one element type; the source is compiled once per type.
#ifdef RS_MID_FP32
hipError_t mid_leaf_f32(const GroupArgs &g, bool down, hipStream_t st) {
    return cw::leaf_any<float>(g, st, down ? 1 : 0);
}
#else
hipError_t mid_leaf_f64(const GroupArgs &g, bool down, hipStream_t st) {
    return cw::leaf_any<double>(g, st, down ? 1 : 0);
}

hipError_t mid_tree(const GroupArgs &g, int grid, hipStream_t st) {
    switch (cw::tiles(g.nx)) {
    case 1: return cw::tree<1>(g, grid, st);
    case 2: return cw::tree<2>(g, grid, st);
    case 3: return cw::tree<3>(g, grid, st);
    default: return cw::tree<4>(g, grid, st);
    }
}

// Stored factorization on the column-owner engine; which: 0 leaf up, 1 tree,
// 2 leaf down; fp32: leaf passes in FP32 (the tree is FP64 in both).
Launcher mfma_factor(int nx, int nu, int which, bool fp32) {
    if (!((nx == 16 && nu == 16) || (nx == 32 && nu == 16) || (nx == 32 && nu == 32))) return nullptr;
    if (which == 1) return [](const GroupArgs &g, int grid, hipStream_t st) { return mid_tree(g, grid, st); };
    if (which == 0)
        return fp32 ? [](const GroupArgs &g, int, hipStream_t st) { return mid_leaf_f32(g, false, st); }
                    : [](const GroupArgs &g, int, hipStream_t st) { return mid_leaf_f64(g, false, st); };
    return fp32 ? [](const GroupArgs &g, int, hipStream_t st) { return g.ntop ? mid_leaf_f32(g, true, st) : hipSuccess; }
                : [](const GroupArgs &g, int, hipStream_t st) { return g.ntop ? mid_leaf_f64(g, true, st) : hipSuccess; };
}

#endif

}  // namespace rs
