// The vector lines of Alg. 2-4 and the forward recursion (Alg. 3) for
// n_x, n_u <= 64 as sweeps whose matrices come through registers one stage
// ahead.
//
// Backward (leaf and master reductions and eliminations), with the stored
// P_{t+1}, V_{t+1}, L^{-1}, L^{-T}, K and L_t = -G^{-1} B'V_{t+1}:
//   pt = Psi - P a;  g = B'pt - l_w;  Psi_t = A'pt - l_x + K'g
//   z = L^{-1} g,  k = L^{-T} z;  cbar += 1/2 a'Pa - Psi'a + c - 1/2 z'z
//   Alg. 4: v += V'(a + B k), or V'a - L_t'g (the same, since G k = g)
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
#pragma once
#include "rs_vec.hpp"

namespace rs {
namespace vs {

using sv::gl;
using sv::gs;
using sv::lane;
using sv::uni;
using sv::wsync;
using sv::xor_sum;

__device__ __forceinline__ int wave() { return uni((int)(threadIdx.x >> 6)); }

// Matrix operand of y = op(M) x with OUT outputs and IN inputs over W
// wavefronts: wave w owns the outputs OPW w .. OPW w + OPW - 1, LPO lanes
// each, and lane part p takes the inputs p, p + LPO, ...
//   column form  y_i = sum_k M[k ld + i] x_k: output l % OPW, part l / OPW
//   row form     y_i = sum_k M[i ld + k] x_k: output l / LPO, part l % LPO
// (consecutive lanes on consecutive words in both).  The elements stay in the
// type they are stored in until they are used, so that a load in flight is
// not waited for early.  PAIR (full sizes): the row form takes two consecutive
// inputs per load, 2 p, 2 p + 1, then 2 LPO further on, so that the lanes of
// an output cover whole cache lines.
template <class U, int OUT, int IN, int W, bool PAIR = false>
struct Mat {
    static constexpr int OPW = OUT / W, LPO = 64 / OPW, NQ = IN / LPO;
    static constexpr bool PR = PAIR && NQ % 2 == 0;
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
    // FULL: outs and ins fill the matrix (else guarded loads, in the same order)
    template <bool FULL = PAIR>
    __device__ __forceinline__ void load_row(const U *M, int ld, int outs, int ins) {
        const int i = out_row(), p = lane() % LPO;
        if constexpr (PR && FULL) {
            typedef U two __attribute__((ext_vector_type(2), aligned(sizeof(U))));   // element alignment only
#pragma unroll
            for (int q = 0; q < NQ / 2; ++q) {
                const two v = gl(reinterpret_cast<const two *>(M + (uint32_t)(i * ld + 2 * p + 2 * LPO * q)));
                m[2 * q] = v[0];
                m[2 * q + 1] = v[1];
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = PR ? 2 * p + 2 * LPO * (q / 2) + (q & 1) : p + LPO * q;
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
        for (int q = 0; q < NQ; ++q)
            s += (double)m[q] * x[PR ? 2 * p + 2 * LPO * (q / 2) + (q & 1) : p + LPO * q];
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
    alignas(16) double av[2][NM], pt[NM], x[NM], lamN[NM];
    alignas(16) double gw[MM], z[MM], kk[MM], u[NM];
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
// (V = I at the end); v_0 is returned in v.  LT: v by L_t'g; else by V'(a + B k),
// which needs k and so runs two stages behind, but reads B again (from the
// cache) instead of L_t: a seventh fewer bytes where the memory is the bound, and
// 2 to 3 us more at the end of a sweep.  st(s): the stage's operands;
// per stage Psi_t goes to st(s).Psi and k_{t+1} to st(s).k (null: not kept).
// Returns the sum of the terms of cbar other than the constants c in every
// lane; psi ends as Psi_0.
template <int NM, int MM, int W, bool RED, bool LT, class TR, class St>
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
    typedef Mat<double, NM, MM, W> MBR;   // B by rows
    constexpr bool VB = RED && !LT;
    MBR mBr;                              // B and a of the stage whose k comes next
    double ar = 0.0;
    const TR *pV = nullptr, *pVn = nullptr;     // V after the stage before that one, and after that one
    const int ir = MBR::out_row();
    const bool ownr = MBR::lead_row() && ir < n;
    auto load_Br = [&](const Stage<TR> &q) {
        mBr.template load_row<false>(q.B, m, n, m);
        ar = (ownr && q.a) ? gl(q.a + (uint32_t)ir) : 0.0;
    };
    auto add_v = [&](bool ident) { v += ident ? (i < n ? S.u[i] : 0.0) : mV.col(S.u); };
    auto put_u = [&] {
        const double u = MBR::sum_row(mBr.part_row(S.kk)) + ar;
        if (ownr) S.u[ir] = u;
    };
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
        if (RED && LT) mLt.load_col(q.Lt, n, n, m);
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
    for (int e = threadIdx.x; e < MM; e += 64 * W) S.gw[e] = S.z[e] = S.kk[e] = 0.0;
    if (VB)
        for (int e = threadIdx.x; e < NM; e += 64 * W) S.u[e] = 0.0;
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
            if (VB && ownm) S.kk[jj] = k;
            mL.load_col(cur.Li, m, m, m);
        }
        if (VB && s + 2 < count) {
            add_v(s + 3 == count);
            mV.load_col(pV, n, n, n);
        }
        double pa = 0.0;
        if (s > 0) {
            pa = mP.col(S.av[(s - 1) & 1]);
            if (s > 1) mP.load_col(nxt.P, n, n, n);
        }
        if (RED && LT) {
            v += s + 1 < count ? mV.col(S.av[s & 1]) : a0;
            if (s > 0) mV.load_col(cur.V, n, n, n);
        }
        wsync();
        // ---- z = L^{-1} g, Psi_t = A'pt - l_x + K'g, v -= L_t'g
        const double z = mLT.col(S.gw);
        psi = y + mK.col(S.gw);
        if (RED && LT) v -= mLt.col(S.gw);
        if (VB) {
            if (s + 1 < count) {
                put_u();
                pV = pVn;
            }
            pVn = cur.V;
            load_Br(cur);
        }
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
        if (VB && ownm) S.kk[jj] = k;
    }
    if (VB && count > 1) {
        add_v(count == 2);
        mV.load_col(pV, n, n, n);
    }
    wsync();
    if (VB) {
        put_u();
        wsync();
        add_v(count == 1);
    }
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
// stage s go (null: not wanted).  The records have m inputs, the problem data
// and w md <= m (the others are padding, and zero).  Ends with x of the end in
// S.x.
template <int NM, int MM, int W, bool EX, bool EXD, class TR, class St, class Xo, class Wo, class Lo>
__device__ __forceinline__ void forward(Smem<NM, MM, W> &S, int n, int m, int md, int count, St st, bool lterms, Xo xo,
                                        Wo wo, Lo lo) {
    typedef Mat<TR, NM, NM, W, EX> MNN;
    typedef Mat<double, NM, NM, W, EX> MA;
    typedef Mat<double, NM, MM, W, EX> MB;
    typedef Mat<TR, MM, NM, W, EX> MK;
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
    mB.template load_row<EXD>(cur.B, md, n, md);
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
        if (ownm && jj < md) {
            double *pw = wo(s);
            if (pw) gs(pw + jj, w);
        }
        wsync();
        const double xn = y + MB::sum_row(mB.part_row(S.gw));
        if (more) mB.template load_row<EXD>(nxt.B, md, n, md);
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

// Leaf solve of the fused path: the records of the fused leaf reduction (leaf
// scratch, FP64 per stage)
//   K (m n) | k (m) | P (n n) | Psi (n) | V (n n) | L_t (m n)
// with lam_N from the master level, or (V and L_t not looked at) those of an
// elimination with the true terminal.
struct FusedStages {
    sv::Prob p;
    int t0, n, m;
    double *rec;
    __device__ Stage<double> operator()(int s) const {
        const int64_t t = t0 + s;
        double *r = rec + (int64_t)s * leaf_rec_len(n, m);
        double *P = r + m * n + m, *V = P + n * n + n;
        return Stage<double>{P, V, nullptr, nullptr, r, V + n * n, p.A + t * p.sA, p.B + t * p.sB,
                             p.a ? p.a + t * p.sa : nullptr, nullptr, nullptr, P + n * n, r + m * n};
    }
};

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

}  // namespace vs
}  // namespace rs
