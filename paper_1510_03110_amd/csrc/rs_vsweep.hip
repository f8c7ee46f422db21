// Right-hand-side passes of the stored factorization for n_x, n_u <= 64 on the
// prefetching sweeps (rs_vsweep.hpp), and the leaf solve of the fused path.
//   ks_leaf_up / ks_tree / ks_leaf_down
// Measured in FP64 (one product after another, then this form): 64 x 32,
// windows of 16 sessions with 33 k stages: leaf up 2.09 -> 1.11 ms, tree
// 1.14 -> 0.89 ms, leaf down 2.46 -> 0.96 ms (4.8 GB, 4.9 TB/s: the memory is
// the bound); 64 problems of N = 1024: 2.81 -> 1.76 and 3.28 -> 1.71 ms
// (5.5 TB/s); 8 x 4 windows: 0.47 -> 0.11, 0.46 -> 0.14 and 0.39 -> 0.08 ms
// (latency: 1.7 us a stage).
#include <hip/hip_runtime.h>

#include "rs_launch.hpp"
#include "rs_vsweep.hpp"

namespace rs {
namespace vs {

// ------------------------------------------------------------------ leaves
// Stages of a leaf; `down` selects the down records (whole-problem leaves).
template <class TR>
struct LeafStages {
    sv::Prob p;
    int t0, n, m;
    const TR *rec;
    double *vec;
    __device__ Stage<TR> operator()(int s) const {
        const LeafRec R{n, m};
        const int64_t t = t0 + s;
        const TR *r = rec + (int64_t)s * R.per_stage();
        double *q = vec + (int64_t)s * R.vec();
        return Stage<TR>{r + R.P(), r + R.V(), r + R.L(), r + R.LT(), r + R.K(), r + R.Lt(), p.A + t * p.sA,
                         p.B + t * p.sB, p.a ? p.a + t * p.sa : nullptr, p.lx ? p.lx + t * p.slx : nullptr,
                         p.lw ? p.lw + t * p.slw : nullptr, q, q + n};
    }
};

template <class TR>
__device__ __forceinline__ LeafStages<TR> leaf_stages(const GroupArgs &g, const sv::Prob &p, const LeafItem &it, int n,
                                                      int m, bool down) {
    const LeafRec R{n, m};
    const int64_t s0 = g.rec_stage(it.scratch);
    const TR *rec = reinterpret_cast<const TR *>(g.fstore) + s0 * (int64_t)R.per_stage() + (down ? R.up() : 0);
    return LeafStages<TR>{p, it.t0, n, m, rec, g.fvec + s0 * (int64_t)R.vec()};
}

// LT: the form of v (see backward).
template <int NM, int MM, int W, bool EX, bool LT, class TR>
__global__ void __launch_bounds__(64 * W) ks_leaf_up(GroupArgs g) {
    __shared__ Smem<NM, MM, W> S;
    if (sv::pass_idle(g)) return;
    const LeafItem it = sv::load_leaf(g.leaves, my_leaf(g));
    if ((it.flags & LEAF_TOP) || sv::skip_inst(g, it.inst)) return;
    const int n = EX ? NM : g.nx, m = EX ? MM : g.nu;
    const sv::Prob p = sv::load_prob(g.probs, it.inst);
    const SlotLayout SL{n};
    double *out = g.slots + (int64_t)it.slot * SL.size();
    const bool last = (it.flags & LEAF_LAST) != 0;
    typedef Mat<double, NM, NM, W> MA;
    const int i = MA::out_col();
    const bool own = MA::lead_col() && i < n;
    double psi = (last && p.lN && i < n) ? -p.lN[i] : 0.0, v = 0.0, cb;
    const auto st = leaf_stages<TR>(g, p, it, n, m, false);
    if (!last) {
        cb = backward<NM, MM, W, true, LT, TR>(S, n, m, it.len, st, nullptr, psi, v);
        if (own) out[SL.a() + i] = v;
    } else {
        cb = backward<NM, MM, W, false, false, TR>(S, n, m, it.len, st, p.QxN, psi, v);
    }
    cb += block_sum(S, sum_c(p.c ? p.c + (int64_t)it.t0 * p.sc : nullptr, p.sc, it.len));
    if (own) out[SL.lx() + i] = -psi;
    if (threadIdx.x == 0) out[SL.c()] = cb + ((last && p.cN) ? p.cN[0] : 0.0);
}

template <int NM, int MM, int W, bool EX, class TR>
__global__ void __launch_bounds__(64 * W) ks_leaf_down(GroupArgs g) {
    __shared__ Smem<NM, MM, W> S;
    if (sv::pass_idle(g)) return;
    const LeafItem it = sv::load_leaf(g.leaves, my_leaf(g));
    if (sv::skip_inst(g, it.inst)) return;
    const int n = EX ? NM : g.nx, m = EX ? MM : g.nu;
    const sv::Prob p = sv::load_prob(g.probs, it.inst);
    const SlotLayout SL{n};
    const bool top = (it.flags & LEAF_TOP) != 0, last = (it.flags & LEAF_LAST) != 0;
    const double *msg = top ? nullptr : g.slots + (int64_t)it.slot * SL.size();
    const auto st = leaf_stages<TR>(g, p, it, n, m, top);
    typedef Mat<double, NM, NM, W> MA;
    const int i = MA::out_row();
    const bool own = MA::lead_row() && i < n;
    if (top) {
        // whole-problem leaf: vector part of Alg. 1-2 with the true terminal
        // on the down records first
        const int ic = MA::out_col();
        double psi = (p.lN && ic < n) ? -p.lN[ic] : 0.0, v = 0.0;
        double cb = backward<NM, MM, W, false, false, TR>(S, n, m, it.len, st, p.QxN, psi, v);
        cb += block_sum(S, sum_c(p.c ? p.c + (int64_t)it.t0 * p.sc : nullptr, p.sc, it.len));
        if (p.obj) {
            // optimal value 1/2 x0'P_0 x0 - Psi_0'x0 + cbar_0
            for (int e = threadIdx.x; e < NM; e += 64 * W) S.x[e] = e < n ? p.x0[e] : 0.0;
            wsync();
            Mat<TR, NM, NM, W> mp;
            mp.load_col(st(0).P, n, n, n);
            const double px = mp.col(S.x);
            const double part = (MA::lead_col() && ic < n) ? S.x[ic] * (0.5 * px - psi) : 0.0;
            const double o = block_sum(S, part);
            if (threadIdx.x == 0) p.obj[0] = o + cb + (p.cN ? p.cN[0] : 0.0);
        }
        __threadfence_block();      // Psi and k are read back by other lanes
    }
    const bool lterms = !last;
    for (int e = threadIdx.x; e < NM; e += 64 * W) {
        S.x[e] = e < n ? (top ? p.x0[e] : msg[SL.xh() + e]) : 0.0;
        // terminal costate lam_N sent by the master level, or formed from its
        // cost to go and the next leaf's initial state
        S.lamN[e] = (lterms && e < n) ? (g.superpose ? msg[SL.lamN() + e] : msg[SL.size() + SL.xh() + e]) : 0.0;
    }
    __syncthreads();
    if (lterms && !g.superpose) {
        const double l = sym_apply<NM, MM, W>(msg + SL.P(), S.lamN, n);
        wsync();
        if (own) S.lamN[i] = l - msg[SL.Psi() + i];
        wsync();
    }
    const int64_t t0 = it.t0;
    forward<NM, MM, W, EX, EX, TR>(S, n, m, m, it.len, st, lterms, [&](int s) { return p.x + (t0 + s) * n; },
                           [&](int s) { return p.w + (t0 + s) * m; }, [&](int s) { return p.lam + (t0 + s) * n; });
    if (last) {
        const int64_t t = t0 + it.len;
        const double q = sym_apply<NM, MM, W>(p.QxN, S.x, n);
        if (own) {
            p.lam[t * n + i] = q + (p.lN ? p.lN[i] : 0.0);         // lam_N = QxN x_N + lN
            p.x[t * n + i] = S.x[i];
        }
    }
}

// Leaf solve of the fused path from the records of the fused leaf reduction
// (shapes of full tiles); whole-problem leaves are solved by the fused leaf
// kernel itself.  MD: the data width is the instance's own (padded inputs).
template <int NM, int MM, int W, bool MD>
__global__ void __launch_bounds__(64 * W) ks_leaf_fwd(GroupArgs g) {
    __shared__ Smem<NM, MM, W> S;
    const LeafItem it = sv::load_leaf(g.leaves, my_leaf(g));
    if ((it.flags & LEAF_TOP) || sv::skip_inst(g, it.inst)) return;
    const int n = NM, m = MM, md = MD ? uni(g.probs[it.inst].nu) : m;
    const sv::Prob p = sv::load_prob(g.probs, it.inst);
    const SlotLayout SL{n};
    const bool last = (it.flags & LEAF_LAST) != 0;
    const double *msg = g.slots + (int64_t)it.slot * SL.size();
    typedef Mat<double, NM, NM, W> MA;
    const int i = MA::out_row();
    for (int e = threadIdx.x; e < NM; e += 64 * W) {
        S.x[e] = e < n ? msg[SL.xh() + e] : 0.0;
        S.lamN[e] = (last || e >= n) ? 0.0 : msg[SL.lamN() + e];
    }
    __syncthreads();
    const FusedStages st{p, it.t0, n, m, static_cast<double *>(g.leaf_scratch) + it.scratch};
    const int64_t t0 = it.t0;
    forward<NM, MM, W, true, !MD, double>(
        S, n, m, md, it.len, st, !last, [&](int s) { return p.x + (t0 + s) * n; },
        [&](int s) { return p.w + (t0 + s) * md; }, [&](int s) { return p.lam + (t0 + s) * n; });
    if (last) {
        const int64_t t = t0 + it.len;
        const double q = sym_apply<NM, MM, W>(p.QxN, S.x, n);
        if (MA::lead_row() && i < n) {
            p.lam[t * n + i] = q + (p.lN ? p.lN[i] : 0.0);         // lam_N = QxN x_N + lN
            p.x[t * n + i] = S.x[i];
        }
    }
}

// -------------------------------------------------------------- the tree
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

// Master levels with the superposition down pass (g.superpose).
template <int NM, int W, bool EX>
__global__ void __launch_bounds__(64 * W) ks_tree(GroupArgs g) {
    __shared__ Smem<NM, NM, W> S;
    __shared__ int s_item;
    if (sv::pass_idle(g)) return;
    const int n = EX ? NM : g.nx, tid = threadIdx.x;
    const SlotLayout SL{n};
    double *slots = sv::uni_ptr(g.slots);
    auto slot = [&](int s) { return slots + (int64_t)s * SL.size(); };
    typedef Mat<double, NM, NM, W> MA;
    for (;;) {
        if (tid == 0) s_item = atomicAdd(g.queue, 1);
        __syncthreads();
        const int idx = uni(s_item);
        __syncthreads();
        if (idx >= g.nitems) break;
        const TreeItem it = load_item(g.items, idx);
        if (tid == 0) {
            for (int d = 0; d < it.dep_count; ++d) {
                int spins = 0;
                while (__hip_atomic_load(&g.flags[it.dep_first + d], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) !=
                       g.epoch) {
                    __builtin_amdgcn_s_sleep(2);
                    if (++spins > sv::SPIN_LIMIT) {
                        int32_t *inf = g.info + 2 * it.inst;
                        atomicCAS(inf, 0, 6);
                        atomicCAS(inf + 1, -1, -2);
                        break;
                    }
                }
            }
        }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int count = it.count;
        const int ic = MA::out_col(), ir = MA::out_row();
        const bool ownc = MA::lead_col() && ic < n, ownr = MA::lead_row() && ir < n;
        if (sv::skip_inst(g, it.inst)) {
            // converged or excluded: nothing to do (its dependents belong to the same instance)
        } else if (it.kind == ITEM_UP) {
            double psi = 0.0, v = 0.0;
            // the constants of the item's master stages, one per slot
            const double cs = sum_c(slot(it.first) + SL.c(), SL.size(), count);
            double cb = backward<NM, NM, W, true, true, double>(S, n, n, count, SlotStages{slots, it.first, n, true},
                                                                nullptr, psi, v);
            cb += block_sum(S, cs);
            double *out = slot(it.out_slot);
            if (ownc) {
                out[SL.a() + ic] = v;
                out[SL.lx() + ic] = -psi;
            }
            if (tid == 0) out[SL.c()] = cb;
        } else if (it.kind == ITEM_UP_LAST || it.kind == ITEM_TOP) {
            // Alg. 1-2 from the level's true terminal (on the up records of
            // its last item; at the top on the down records)
            const bool top = it.kind == ITEM_TOP;
            double *term = slot(it.term_slot);
            double psi = ic < n ? -term[SL.lx() + ic] : 0.0, v = 0.0;
            if (top && ownc) slot(it.first + count - 1)[SL.Psi() + ic] = psi;
            const SlotStages st{slots, it.first, n, !top};
            const double cs = sum_c(slot(it.first) + SL.c(), SL.size(), count), ct = term[SL.c()];
            const sv::Prob p = sv::load_prob(g.probs, it.inst);
            double px = 0.0;
            if (top) {
                // P_0 x_0, for the optimal value, ahead of the chain
                for (int e = tid; e < NM; e += 64 * W) S.x[e] = e < n ? p.x0[e] : 0.0;
                wsync();
                if (p.obj) {
                    Mat<double, NM, NM, W> mp;
                    mp.load_col(term + SL.P(), n, n, n);
                    px = mp.col(S.x);
                }
            }
            double cb = backward<NM, NM, W, false, true, double>(S, n, n, count, st, term + SL.Qx(), psi, v);
            cb += block_sum(S, cs) + ct;
            if (!top) {
                double *out = slot(it.out_slot);
                if (ownc) out[SL.lx() + ic] = -psi;
                if (tid == 0) out[SL.c()] = cb;
            } else {
                __threadfence_block();      // Psi and k are read back by other lanes
                __syncthreads();
                if (p.obj) {
                    const double o = block_sum(S, ownc ? S.x[ic] * (0.5 * px - psi) : 0.0);
                    if (tid == 0) p.obj[0] = o + cb;
                }
                // terminal costate of child s, lam_{s+1} = P_{s+1} x_{s+1} -
                // Psi_{s+1}, from the cost to go sent to it and the initial
                // state of the next child (of the terminal node for the last):
                // what the sweep has at stage s + 1 anyway
                forward<NM, NM, W, EX, EX, double>(
                    S, n, n, n, count, st, false, [&](int s) { return slot(it.first + s) + SL.xh(); },
                    [](int) { return (double *)nullptr; },
                    [&](int s) { return s > 0 ? slot(it.first + s - 1) + SL.lamN() : (double *)nullptr; });
                double *sl = slot(it.first + count - 1);
                const double l = sym_apply<NM, NM, W>(sl + SL.P(), S.x, n);
                if (ownr) {
                    term[SL.xh() + ir] = S.x[ir];
                    sl[SL.lamN() + ir] = l - sl[SL.Psi() + ir];
                }
            }
        } else {
            // down pass below the top (Alg. 6, k >= 1): child s receives x_s
            // and its terminal costate lam_{s+1}
            const bool last = it.last != 0;
            const double *msg = slot(it.out_slot);
            for (int e = tid; e < NM; e += 64 * W) {
                S.x[e] = e < n ? msg[SL.xh() + e] : 0.0;
                S.lamN[e] = (!last && e < n) ? msg[SL.lamN() + e] : 0.0;
            }
            __syncthreads();
            const SlotStages st{slots, it.first, n, true};
            forward<NM, NM, W, EX, EX, double>(S, n, n, n, count, st, !last, [&](int s) { return slot(it.first + s) + SL.xh(); },
                                       [](int) { return (double *)nullptr; },
                                       [&](int s) { return s > 0 ? slot(it.first + s - 1) + SL.lamN() : (double *)nullptr; });
            // the last child ends where the item does: at lam_N, or for the
            // last item at the terminal node, lam = P_term x - Psi_term
            double *lend = slot(it.first + count - 1) + SL.lamN();
            if (last) {
                double *term = slot(it.term_slot);
                const double l = sym_apply<NM, NM, W>(term + SL.Qx(), S.x, n);
                if (ownr) {
                    lend[ir] = l + term[SL.lx() + ir];
                    term[SL.xh() + ir] = S.x[ir];
                }
            } else if (ownr) {
                lend[ir] = S.lamN[ir];
            }
        }
        __threadfence();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(&g.flags[idx], g.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
}

// ------------------------------------------------------------- launchers
// Wavefronts per unit: one at n <= 16 (no workgroup barrier to wait at), four
// at n <= 32, eight at n <= 64, so that an n x n matrix takes 4, 4 and 8
// registers (doubles) a thread.  Sizes that fill them have an instance
// without bounds checks.
// Backward sweeps of 32 states, full sizes, with more leaves than four a CU: one
// wavefront each, without barriers and with longer runs of a matrix to a load,
// since the memory is then the bound and not the chain of a leaf (32 x 16, FP64:
// 2048 leaves of 64 stages 790 -> 730 us, 4000 1.41 -> 1.32 ms; at 256 leaves of 32
// stages four wavefronts take 78 us and one 112).
// The reductions take v by L_t'g, which ends sooner (32 x 16, FP64: 64 leaves of 16
// stages 37 us and 40 the other way; 8 x 4, 6400 leaves of 16 116 and 126), and by
// V'(a + B k) where the memory is the bound: full sizes, in FP64 more leaves than
// one a CU (16 x 16, 4096 leaves of 64 stages 705 and 650 us; 32 x 16, 512 of 128
// 431 and 425).  An FP32 L_t has half the bytes: there above four a CU (16 x 16,
// 8000 of 64 stages 247 and 224 us; 32 x 16, 512 of 128 113 and 117).
template <int NM, int MM, int W, class TR>
hipError_t leaf_of(const GroupArgs &g, bool down, hipStream_t st) {
    const dim3 grid(g.nleaves), block(64 * W);
    const bool ex = g.nx == NM && g.nu == MM;
    if (down && ex)
        hipLaunchKernelGGL((ks_leaf_down<NM, MM, W, true, TR>), grid, block, 0, st, g);
    else if (down)
        hipLaunchKernelGGL((ks_leaf_down<NM, MM, W, false, TR>), grid, block, 0, st, g);
    else if (ex && NM == 32 && g.nleaves > 1024)
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, NM == 32 ? 1 : W, true, false, TR>), grid, dim3(64), 0, st, g);
    else if (ex && g.nleaves > (sizeof(TR) == 8 ? 256 : 1024))
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, W, true, false, TR>), grid, block, 0, st, g);
    else if (ex)
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, W, true, true, TR>), grid, block, 0, st, g);
    else
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, W, false, true, TR>), grid, block, 0, st, g);
    return hipGetLastError();
}
template <class TR>
hipError_t leaf(const GroupArgs &g, bool down, hipStream_t st) {
    const int n = g.nx, m = g.nu;
    if (n <= 16 && m <= 16) return leaf_of<16, 16, 1, TR>(g, down, st);
    if (n <= 32 && m <= 16) return leaf_of<32, 16, 4, TR>(g, down, st);
    if (n <= 32 && m <= 32) return leaf_of<32, 32, 4, TR>(g, down, st);
    if (m <= 32) return leaf_of<64, 32, 8, TR>(g, down, st);
    return leaf_of<64, 64, 8, TR>(g, down, st);
}
template <int NM, int MM, int W>
hipError_t fwd_of(const GroupArgs &g, hipStream_t st) {
    const dim3 grid(g.nleaves), block(64 * W);
    if (g.data_nu)
        hipLaunchKernelGGL((ks_leaf_fwd<NM, MM, W, true>), grid, block, 0, st, g);
    else
        hipLaunchKernelGGL((ks_leaf_fwd<NM, MM, W, false>), grid, block, 0, st, g);
    return hipGetLastError();
}
template <int NM, int W>
hipError_t tree_of(const GroupArgs &g, int grid, hipStream_t st) {
    if (g.nx == NM)
        hipLaunchKernelGGL((ks_tree<NM, W, true>), dim3(grid), dim3(64 * W), 0, st, g);
    else
        hipLaunchKernelGGL((ks_tree<NM, W, false>), dim3(grid), dim3(64 * W), 0, st, g);
    return hipGetLastError();
}

}  // namespace vs

hipError_t sweep_leaf(const GroupArgs &g, bool fp32, bool down, hipStream_t st) {
    return fp32 ? vs::leaf<float>(g, down, st) : vs::leaf<double>(g, down, st);
}

hipError_t fused_leaf_forward(const GroupArgs &g, hipStream_t st) {
    if (g.nx <= 16 && g.nu <= 16) return vs::fwd_of<16, 16, 1>(g, st);
    if (g.nu <= 16) return vs::fwd_of<32, 16, 4>(g, st);
    return vs::fwd_of<32, 32, 4>(g, st);
}

// Up to 32 states one wavefront per work item, so that four items a CU are at
// work at once; trees of few items two, for the chain of each (32 states, FP64: 41
// items 83 us with one, 69 with two, 72 with four; 1152 items 347, 444 and 467 us).
hipError_t sweep_tree(const GroupArgs &g, int grid, hipStream_t st) {
    if (g.nx <= 16) return vs::tree_of<16, 1>(g, grid, st);
    if (g.nx <= 32 && g.nitems <= 128) return vs::tree_of<32, 2>(g, grid, st);
    if (g.nx <= 32) return vs::tree_of<32, 1>(g, grid, st);
    return vs::tree_of<64, 8>(g, grid, st);
}

}  // namespace rs
