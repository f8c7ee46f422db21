// Right-hand-side passes of the stored factorization for n_x, n_u <= 64: the
// vector lines of Alg. 2-4 and the forward recursion (Alg. 3) as sweeps whose
// matrices come through registers one stage ahead.
//
// Backward (leaf and master reductions and eliminations), with the stored
// P_{t+1}, V_{t+1}, L^{-1}, L^{-T}, K and L_t = -G^{-1} B'V_{t+1}:
//   pt = Psi - P a;  g = B'pt - l_w;  Psi_t = A'pt - l_x + K'g
//   z = L^{-1} g,  k = L^{-T} z;  cbar += 1/2 a'Pa - Psi'a + c - 1/2 z'z
//   Alg. 4: v += V'a - L_t'g    (= V'(a + B k), since G k = g)
// Forward:
//   w = K x + k_0 + L_t lam_N,  lam = P x - Psi_0 + V lam_N,  x+ = A x + a + B w
// (k_0, Psi_0 of the reduction and lam_N sent by the parent; the last item of
// a level and whole-problem leaves hold final records, without the lam_N
// terms).
//
// Only two products of a stage depend on one another (g, then Psi; w, then
// x+): the others use what is already there, so a stage takes two workgroup
// barriers.  Every product is spread over the W wavefronts so that each
// output is summed inside one wavefront, and a matrix's registers are loaded
// with the next stage's as soon as they have been used: a stage costs about
// one memory latency or its share of the bandwidth, where one product after
// another, each loading its own operands, cost seven.
//   ks_leaf_up / ks_tree / ks_leaf_down
// Measured in FP64 (one product after another, then this form): 64 x 32,
// windows of 16 sessions with 33 k stages: leaf up 2.09 -> 1.16 ms, tree
// 1.14 -> 0.85 ms, leaf down 2.46 -> 1.01 ms (4.8 GB, 4.7 TB/s: the memory is
// the bound); 64 problems of N = 1024: 2.81 -> 1.85 and 3.28 -> 1.75 ms
// (5.4 TB/s); 8 x 4 windows: 0.47 -> 0.11, 0.46 -> 0.14 and 0.39 -> 0.08 ms
// (latency: 1.7 us a stage).
#include <hip/hip_runtime.h>

#include "rs_launch.hpp"
#include "rs_vec.hpp"

namespace rs {
namespace vs {

using sv::lane;
using sv::uni;
using sv::wsync;

// Global-memory accesses through address space 1: pointers that come out of a
// descriptor are generic, and a generic access also counts as an LDS access,
// so that every wait for LDS would wait for the loads in flight.
template <class U>
__device__ __forceinline__ U gl(const U *p) {
    return *(const __attribute__((address_space(1))) U *)p;
}
template <class U>
__device__ __forceinline__ void gs(U *p, U v) {
    *(__attribute__((address_space(1))) U *)p = v;
}

__device__ __forceinline__ int wave() { return uni((int)(threadIdx.x >> 6)); }

// Sum over the lanes that differ in bit log2(B) of their index; every lane
// receives it.  Rows of 16 are exchanged with the row and half-wave swaps.
template <int B>
__device__ __forceinline__ double xor_sum(double v) {
    if constexpr (B == 32 || B == 16) {
        const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
        const auto l = B == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                               : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = B == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                               : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    } else if constexpr (B == 8) {
        return v + sv::dpp_move<0x128>(v);          // row_ror:8
    } else {
        return v + __shfl_xor(v, B, 64);
    }
}

// Matrix operand of y = op(M) x with OUT outputs and IN inputs over W
// wavefronts: wave w owns the outputs OPW w .. OPW w + OPW - 1, LPO lanes
// each, and lane part p takes the inputs p, p + LPO, ...
//   column form  y_i = sum_k M[k ld + i] x_k: output l % OPW, part l / OPW
//   row form     y_i = sum_k M[i ld + k] x_k: output l / LPO, part l % LPO
// (consecutive lanes on consecutive words in both).  The elements stay in the
// type they are stored in until they are used, so that a load in flight is
// not waited for early.
template <class U, int OUT, int IN, int W>
struct Mat {
    static constexpr int OPW = OUT / W, LPO = 64 / OPW, NQ = IN / LPO;
    static_assert(OUT % W == 0 && 64 % OPW == 0 && IN % LPO == 0, "whole lanes");
    U m[NQ];
    __device__ static int out_col() { return OPW * wave() + lane() % OPW; }
    __device__ static int out_row() { return OPW * wave() + lane() / LPO; }
    __device__ static bool lead_col() { return lane() < OPW; }
    __device__ static bool lead_row() { return lane() % LPO == 0; }

    __device__ __forceinline__ void load_col(const U *M, int ld, int outs, int ins) {
        const int i = out_col(), p = lane() / OPW;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = p + LPO * q;
            m[q] = (i < outs && k < ins) ? gl(M + (uint32_t)(k * ld + i)) : U(0);
        }
    }
    __device__ __forceinline__ void load_row(const U *M, int ld, int outs, int ins) {
        const int i = out_row(), p = lane() % LPO;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = p + LPO * q;
            m[q] = (i < outs && k < ins) ? gl(M + (uint32_t)(i * ld + k)) : U(0);
        }
    }
    // lane parts of the sums over a vector in LDS (IN entries, zero-padded)
    __device__ __forceinline__ double part_col(const double *x) const {
        const int p = lane() / OPW;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) s += (double)m[q] * x[p + LPO * q];
        return s;
    }
    __device__ __forceinline__ double part_row(const double *x) const {
        const int p = lane() % LPO;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) s += (double)m[q] * x[p + LPO * q];
        return s;
    }
    __device__ static __forceinline__ double sum_col(double s) {
        if constexpr (OPW <= 1) s = xor_sum<1>(s);
        if constexpr (OPW <= 2) s = xor_sum<2>(s);
        if constexpr (OPW <= 4) s = xor_sum<4>(s);
        if constexpr (OPW <= 8) s = xor_sum<8>(s);
        if constexpr (OPW <= 16) s = xor_sum<16>(s);
        return xor_sum<32>(s);
    }
    __device__ static __forceinline__ double sum_row(double s) { return sv::group_sum<LPO>(s); }
    __device__ __forceinline__ double col(const double *x) const { return sum_col(part_col(x)); }
};

template <int NM, int MM, int W>
struct Smem {
    double av[2][NM], pt[NM], x[NM], lamN[NM];
    double gw[MM], z[MM];
    double red[W];
};

// Operands of a stage; TR: type of the stored factors.
template <class TR>
struct Stage {
    const TR *P, *V, *Li, *LT, *K, *Lt;    // record of this stage (P, V: after it)
    const double *A, *B, *a, *lx, *lw;     // a, lx, lw may be null (zero)
    double *Psi, *k;                       // Psi_t and k_{t+1} of the sweep (written or read)
};

template <int NM, int MM, int W>
__device__ __forceinline__ double block_sum(Smem<NM, MM, W> &S, double v) {
    v = sv::wave_sum(v);
    if (W == 1) return v;
    wsync();
    if (lane() == 0) S.red[wave()] = v;
    wsync();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += S.red[w];
    wsync();
    return s;
}

// Backward sweep.  psi: Psi of the end in the lanes of the column form
// (replicated over the parts); P0: P of the end (nullptr: zero).  RED: Alg. 4
// (V = I at the end); v_0 is returned in v.  st(s): the stage's operands;
// per stage Psi_t goes to st(s).Psi and k_{t+1} to st(s).k (null: not kept).
// Returns the sum of the terms of cbar other than the constants c in every
// lane; psi ends as Psi_0.
template <int NM, int MM, int W, bool RED, class TR, class St>
__device__ __forceinline__ double backward(Smem<NM, MM, W> &S, int n, int m, int count, St st, const double *P0,
                                           double &psi, double &v) {
    typedef Mat<TR, NM, NM, W> MNN;       // P, V' (records)
    typedef Mat<double, NM, NM, W> MA;
    typedef Mat<double, MM, NM, W> MB;
    typedef Mat<TR, MM, MM, W> MMM;
    typedef Mat<TR, NM, MM, W> MNM;
    const int i = MA::out_col(), jj = MB::out_col();
    const bool own = MA::lead_col() && i < n, ownm = MB::lead_col() && jj < m;
    MNN mP, mV;
    MA mA;
    MB mB;
    MMM mL, mLT;
    MNM mK, mLt;
    // entry i (jj) of a stage's vectors, zero in the padding
    auto at = [&](const double *q) { return (q && i < n) ? gl(q + (uint32_t)i) : 0.0; };
    auto atm = [&](const double *q) { return (q && jj < m) ? gl(q + (uint32_t)jj) : 0.0; };
    auto load1 = [&](const Stage<TR> &q) {
        mA.load_col(q.A, n, n, n);
        mB.load_col(q.B, m, m, n);
    };
    auto load2 = [&](const Stage<TR> &q) {
        mLT.load_col(q.LT, m, m, m);
        mK.load_col(q.K, n, n, m);
        if (RED) mLt.load_col(q.Lt, n, n, m);
    };
    double acc = 0.0;
    v = 0.0;
    count = uni(count);
    Stage<TR> cur = st(count - 1);
    load1(cur);
    load2(cur);
    double lx = at(cur.lx), lw = atm(cur.lw), a0 = at(cur.a);
    double a1 = 0.0, a2 = 0.0;            // a of the next stage and of the one after it
    if (count > 1) {
        mP.load_col(cur.P, n, n, n);
        a1 = at(st(count - 2).a);
    }
    if (count > 2) a2 = at(st(count - 3).a);
    mL.load_col(cur.Li, m, m, m);
    for (int e = threadIdx.x; e < NM; e += 64 * W) S.av[0][e] = S.av[1][e] = S.pt[e] = 0.0;
    for (int e = threadIdx.x; e < MM; e += 64 * W) S.gw[e] = S.z[e] = 0.0;
    wsync();
    if (own) {
        S.av[(count - 1) & 1][i] = a0;
        S.av[count & 1][i] = a1;
    }
    wsync();
    {
        double pa = 0.0;
        if (P0) {
            MA m0;
            m0.load_col(P0, n, n, n);
            pa = m0.col(S.av[(count - 1) & 1]);
        }
        if (own) {
            S.pt[i] = psi - pa;
            acc += a0 * (0.5 * pa - psi);
        }
    }
    wsync();
    double *kout = nullptr;               // where the k of the stage before goes
    for (int s = count - 1; s >= 0; --s) {
        // ---- g = B'pt - l_w, A'pt - l_x; off the chain: P a of the next
        //      stage, V'a of this one, k of the one before
        const Stage<TR> nxt = s > 0 ? st(s - 1) : Stage<TR>{};
        const double g = mB.col(S.pt) - lw;
        const double y = mA.col(S.pt) - lx;
        if (ownm) S.gw[jj] = g;
        if (s > 0) {
            load1(nxt);
            lw = atm(nxt.lw);
            lx = at(nxt.lx);
        }
        if (kout) {
            const double k = mL.col(S.z);
            if (ownm) gs(kout + jj, k);
            mL.load_col(cur.Li, m, m, m);
        }
        double pa = 0.0;
        if (s > 0) {
            pa = mP.col(S.av[(s - 1) & 1]);
            if (s > 1) mP.load_col(nxt.P, n, n, n);
        }
        if (RED) {
            v += s + 1 < count ? mV.col(S.av[s & 1]) : a0;
            if (s > 0) mV.load_col(cur.V, n, n, n);
        }
        wsync();
        // ---- z = L^{-1} g, Psi_t = A'pt - l_x + K'g, v -= L_t'g
        const double z = mLT.col(S.gw);
        psi = y + mK.col(S.gw);
        if (RED) v -= mLt.col(S.gw);
        if (ownm) {
            S.z[jj] = z;
            acc -= 0.5 * z * z;
        }
        if (own) {
            if (cur.Psi) gs(cur.Psi + i, psi);
            if (s > 0) {
                S.pt[i] = psi - pa;
                acc += S.av[(s - 1) & 1][i] * (0.5 * pa - psi);
            }
            if (s > 1) S.av[s & 1][i] = a2;
        }
        kout = cur.k;
        if (s > 0) {
            load2(nxt);
            if (s > 2) a2 = at(st(s - 3).a);
            cur = nxt;
        }
        wsync();
    }
    if (kout) {
        const double k = mL.col(S.z);
        if (ownm) gs(kout + jj, k);
    }
    wsync();
    return block_sum(S, acc);
}

// Sum of the constants c of `count` stages (c: first one, stride sc).
__device__ __forceinline__ double sum_c(const double *c, int64_t sc, int count) {
    double s = 0.0;
    if (c)
        for (int t = threadIdx.x; t < count; t += (int)blockDim.x) s += gl(c + (int64_t)t * sc);
    return s;
}

// Forward sweep from the x in S.x (zero-padded); lterms: with the lam_N in
// S.lamN.  P may be null (no lam).  xo, wo, lo: where x_s, w_s and lam_s of
// stage s go (null: not wanted).  Ends with x of the end in S.x.
template <int NM, int MM, int W, class TR, class St, class Xo, class Wo, class Lo>
__device__ __forceinline__ void forward(Smem<NM, MM, W> &S, int n, int m, int count, St st, bool lterms, Xo xo, Wo wo,
                                        Lo lo) {
    typedef Mat<TR, NM, NM, W> MNN;
    typedef Mat<double, NM, NM, W> MA;
    typedef Mat<double, NM, MM, W> MB;
    typedef Mat<TR, MM, NM, W> MK;
    const int i = MA::out_row(), jj = MK::out_row();
    const bool own = MA::lead_row() && i < n, ownm = MK::lead_row() && jj < m;
    MNN mP, mV;
    MA mA;
    MB mB;
    MK mK, mLt;
    double kk = 0.0, a = 0.0, ps = 0.0;
    count = uni(count);
    auto load1 = [&](const Stage<TR> &q) {
        mK.load_row(q.K, n, m, n);
        mA.load_row(q.A, n, n, n);
        if (lterms) mLt.load_row(q.Lt, n, m, n);
        if (q.P) mP.load_row(q.P, n, n, n);
        if (lterms && q.P) mV.load_row(q.V, n, n, n);
        kk = ownm ? gl(q.k + jj) : 0.0;
        a = (own && q.a) ? gl(q.a + (uint32_t)i) : 0.0;
        ps = (own && q.P) ? gl(q.Psi + i) : 0.0;
    };
    Stage<TR> cur = st(0);
    load1(cur);
    mB.load_row(cur.B, m, n, m);
    for (int e = threadIdx.x; e < MM; e += 64 * W) S.gw[e] = 0.0;
    wsync();
    for (int s = 0; s < count; ++s) {
        const bool more = s + 1 < count;
        const Stage<TR> nxt = more ? st(s + 1) : Stage<TR>{};
        double w = mK.part_row(S.x), lam = 0.0;
        if (lterms) w += mLt.part_row(S.lamN);
        w = MK::sum_row(w) + kk;
        if (ownm) S.gw[jj] = w;
        const double y = MA::sum_row(mA.part_row(S.x)) + a;
        if (cur.P) {
            lam = mP.part_row(S.x);
            if (lterms) lam += mV.part_row(S.lamN);
            lam = MNN::sum_row(lam) - ps;
        }
        const double xi = own ? S.x[i] : 0.0;
        if (more) load1(nxt);
        if (own) {
            double *px = xo(s), *pl = lo(s);
            if (px) gs(px + i, xi);
            if (pl) gs(pl + i, lam);
        }
        if (ownm) {
            double *pw = wo(s);
            if (pw) gs(pw + jj, w);
        }
        wsync();
        const double xn = y + MB::sum_row(mB.part_row(S.gw));
        if (more) mB.load_row(nxt.B, m, n, m);
        if (own) S.x[i] = xn;
        cur = nxt;
        wsync();
    }
}

// y_i = (M x)_i for a symmetric n x n M (row form), in the lead lane of i.
template <int NM, int MM, int W>
__device__ __forceinline__ double sym_apply(const double *M, const double *x, int n) {
    Mat<double, NM, NM, W> m;
    m.load_row(M, n, n, n);
    return Mat<double, NM, NM, W>::sum_row(m.part_row(x));
}

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

template <int NM, int MM, int W, bool EX, class TR>
__global__ void __launch_bounds__(64 * W) ks_leaf_up(GroupArgs g) {
    __shared__ Smem<NM, MM, W> S;
    if (sv::pass_idle(g)) return;
    const LeafItem it = sv::load_leaf(g.leaves, blockIdx.x);
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
        cb = backward<NM, MM, W, true, TR>(S, n, m, it.len, st, nullptr, psi, v);
        if (own) out[SL.a() + i] = v;
    } else {
        cb = backward<NM, MM, W, false, TR>(S, n, m, it.len, st, p.QxN, psi, v);
    }
    cb += block_sum(S, sum_c(p.c ? p.c + (int64_t)it.t0 * p.sc : nullptr, p.sc, it.len));
    if (own) out[SL.lx() + i] = -psi;
    if (threadIdx.x == 0) out[SL.c()] = cb + ((last && p.cN) ? p.cN[0] : 0.0);
}

template <int NM, int MM, int W, bool EX, class TR>
__global__ void __launch_bounds__(64 * W) ks_leaf_down(GroupArgs g) {
    __shared__ Smem<NM, MM, W> S;
    if (sv::pass_idle(g)) return;
    const LeafItem it = sv::load_leaf(g.leaves, blockIdx.x);
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
        double cb = backward<NM, MM, W, false, TR>(S, n, m, it.len, st, p.QxN, psi, v);
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
    forward<NM, MM, W, TR>(S, n, m, it.len, st, lterms, [&](int s) { return p.x + (t0 + s) * n; },
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

// -------------------------------------------------------------- the tree
// Master stages read from their slots; up: the factors of the up pass
// (P and V after the stage are those records), else of the down pass, whose P
// is the message P_{s+1} kept in the stage's own slot.
struct SlotStages {
    double *slots;
    int first, n;
    bool up;
    __device__ double *slot(int s) const { return slots + (int64_t)(first + s) * SlotLayout{n}.size(); }
    __device__ Stage<double> operator()(int s) const {
        const SlotLayout L{n};
        double *d = slot(s);
        if (up)
            return Stage<double>{d + L.uP(), d + L.uV(), d + L.uL(), d + L.uLT(), d + L.uK(), d + L.dL(), d + L.A(),
                                 d + L.Qw(), d + L.a(), d + L.lx(), nullptr, d + L.Psi(), d + L.k()};
        // P after stage s of the down pass is the message of stage s - 1 (not
        // asked for at s = 0)
        return Stage<double>{s > 0 ? slot(s - 1) + L.P() : nullptr, nullptr, d + L.dL(), d + L.dLT(), d + L.K(), nullptr,
                             d + L.A(), d + L.Qw(), d + L.a(), d + L.lx(), nullptr,
                             s > 0 ? slot(s - 1) + L.Psi() : nullptr, d + L.k()};
    }
};

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
        // the constants of the item's master stages, one per slot
        auto c_sum = [&] { return block_sum(S, sum_c(slot(it.first) + SL.c(), SL.size(), count)); };
        if (sv::skip_inst(g, it.inst)) {
            // converged or excluded: nothing to do (its dependents belong to the same instance)
        } else if (it.kind == ITEM_UP) {
            double psi = 0.0, v = 0.0;
            double cb = backward<NM, NM, W, true, double>(S, n, n, count, SlotStages{slots, it.first, n, true}, nullptr,
                                                          psi, v);
            cb += c_sum();
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
            const double *P0 = term + SL.Qx();
            double cb = backward<NM, NM, W, false, double>(S, n, n, count, st, P0, psi, v);
            cb += c_sum() + term[SL.c()];
            if (!top) {
                double *out = slot(it.out_slot);
                if (ownc) out[SL.lx() + ic] = -psi;
                if (tid == 0) out[SL.c()] = cb;
            } else {
                const sv::Prob p = sv::load_prob(g.probs, it.inst);
                for (int e = tid; e < NM; e += 64 * W) S.x[e] = e < n ? p.x0[e] : 0.0;
                __threadfence_block();      // Psi and k are read back by other lanes
                __syncthreads();
                if (p.obj) {
                    Mat<double, NM, NM, W> mp;
                    mp.load_col(term + SL.P(), n, n, n);
                    const double px = mp.col(S.x);
                    const double o = block_sum(S, ownc ? S.x[ic] * (0.5 * px - psi) : 0.0);
                    if (tid == 0) p.obj[0] = o + cb;
                }
                auto none = [](int) { return (double *)nullptr; };
                auto fst = [&](int s) {
                    Stage<double> q = st(s);
                    q.P = nullptr;
                    return q;
                };
                forward<NM, NM, W, double>(S, n, n, count, fst, false, [&](int s) { return slot(it.first + s) + SL.xh(); },
                                           none, none);
                if (ownr) term[SL.xh() + ir] = S.x[ir];
                // terminal costate of child s, lam_{s+1} = P_{s+1} x_{s+1} -
                // Psi_{s+1}, from the cost to go sent to it and the initial
                // state of the next child (of the terminal node for the last)
                __threadfence_block();
                __syncthreads();
                for (int s = 0; s < count; ++s) {
                    double *sl = slot(it.first + s);
                    const double *xn = (s + 1 < count ? slot(it.first + s + 1) : term) + SL.xh();
                    for (int e = tid; e < n; e += 64 * W) S.x[e] = xn[e];
                    wsync();
                    const double l = sym_apply<NM, NM, W>(sl + SL.P(), S.x, n);
                    if (ownr) sl[SL.lamN() + ir] = l - sl[SL.Psi() + ir];
                    wsync();
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
            forward<NM, NM, W, double>(S, n, n, count, st, !last, [&](int s) { return slot(it.first + s) + SL.xh(); },
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
template <int NM, int MM, int W, class TR>
hipError_t leaf_of(const GroupArgs &g, bool down, hipStream_t st) {
    const dim3 grid(g.nleaves), block(64 * W);
    const bool ex = g.nx == NM && g.nu == MM;
    if (down && ex)
        hipLaunchKernelGGL((ks_leaf_down<NM, MM, W, true, TR>), grid, block, 0, st, g);
    else if (down)
        hipLaunchKernelGGL((ks_leaf_down<NM, MM, W, false, TR>), grid, block, 0, st, g);
    else if (ex)
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, W, true, TR>), grid, block, 0, st, g);
    else
        hipLaunchKernelGGL((ks_leaf_up<NM, MM, W, false, TR>), grid, block, 0, st, g);
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

hipError_t sweep_tree(const GroupArgs &g, int grid, hipStream_t st) {
    if (g.nx <= 16) return vs::tree_of<16, 1>(g, grid, st);
    if (g.nx <= 32) return vs::tree_of<32, 4>(g, grid, st);
    return vs::tree_of<64, 8>(g, grid, st);
}

}  // namespace rs
