// Column-owner form of the per-stage Riccati recursion (Alg. 1-2 and Alg. 4)
// for n_x <= 64 and n_u <= n_x (in tiles of 16), in FP64 or FP32: the matrix
// lines alone (stored factorization), or with the right-hand-side lines (VEC,
// fused solve, FP64).
//
// A workgroup of 2 NXT wavefronts (NXT = n_x / 16 rounded up) owns one
// subproblem.  Wave j < NXT owns the 16-wide column block j of A, F, H', Y,
// K and P; wave NXT + j (Alg. 4) owns column block j of V, A'V, B'V, X, L_t
// and Q_w_hat.  The 16x16x4 matrix instructions leave a result tile in the
// register layout in which a tile enters the next product as its right-hand
// operand (element (k, j) in lane j + 16 (k mod 4) for FP64; for FP32 the
// inner index is only permuted, the same way in both operands), so a column
// block passes through the whole chain of a stage in its owner's registers:
//
//   W(:,j) = P A(:,j)   F(:,j) = Qx + A'W(:,j)   H'(:,j) = Qxw' + B'W(:,j)
//   Y(:,j) = L^{-1} H'(:,j)   K(:,j) = -L^{-T} Y(:,j)   P(:,j) = F - Y'Y(:,j)
//   A'V(:,j)  B'V(:,j)  X(:,j) = L^{-1} B'V(:,j)   L_t(:,j) = -L^{-T} X(:,j)
//   V(:,j) = A'V - Y'X(:,j)   Q_w_hat(:,j) += X'X(:,j)
//
// Only left-hand operands (P, A, B, L^{-1}, Y, X) live in LDS; V and Q_w_hat
// never leave their owner's registers.  G = Qw + B'PB is formed by the owners of
// A's columns (a column block of B each, its inner tiles split over two or more
// waves where there are fewer of them) and factored by the last wave while the
// others form W, F, H', A'V and the last stage's part of Q_w_hat.  (In that
// order, with the loads counted, a stage of 32 states and 16 inputs alone on its
// CU went from 13.6 to 11.0 k cycles.)  P, F and Q_w_hat are formed on the lower
// tiles and mirrored, so they are exactly symmetric.  Four workgroup barriers a
// stage; the next stage's A and B wait in registers.
//
// The vector lines ride on the same registers: the owner of a column block
// also owns those entries of Psi, v and g_x, whose products with a column
// block are sums over its own lanes (P a, A'pt, V'a, Y'z, X'z), and the owner
// of the last column block forms z = L^{-1} g_w and k = L^{-T} z from the operands it
// reads for Y and K anyway.
//
// Sizes that are not multiples of 16 are padded with zeros on load (an
// identity in the padded block of Q_w), which decouples the padding.
#pragma once
#include "rs_mfma.hpp"
#include "rs_vec.hpp"

namespace rs {
namespace cw {

using mf::lane;
using mf::MT;
using mf::v4_t;
using mf::wave;
using mf::wave_fence;
using mf::zero4;
typedef mf::d4 d4;

// A lane's place in the operand and result layouts: c = lane % 16, q = lane /
// 16; element r of a result tile is in row(r).  Taken afresh in every stage
// through an opaque copy: the addresses formed from it are cheap, and the
// compiler would otherwise hoist all of them out of the stage loop and spill.
template <class T>
struct Ln {
    int c, q;
    __device__ __forceinline__ Ln() {
        int l = lane();
        asm volatile("" : "+v"(l));
        c = l & 15;
        q = l >> 4;
    }
    __device__ __forceinline__ int row(int r) const { return sizeof(T) == 8 ? q + 4 * r : 4 * q + r; }
};

// LDS position of element (k, i) of a matrix with row pitch PT: the column is
// permuted within its tile by an exclusive-or with the row, so that the 16
// lanes of an operand read fall on distinct banks whether they run along a
// row or down a column.
template <int PT>
__device__ __forceinline__ int at(int k, int i) {
    return k * PT + (i ^ (k & 15));
}

// Left-hand operand tile of a product, one matrix-instruction slice r at a
// time: the element of row 16 ti + lane % 16 and inner index 16 kt + row(r).
// N: M[k][i] (the transposed view of a row-major matrix, or a symmetric one);
// it also reads a right-hand operand column block straight from LDS.
// R: M[i][k].
template <int PT, class T>
__device__ __forceinline__ T ldN(const Ln<T> &L, const T *M, int kt, int ti, int r) {
    const int row = L.row(r);
    return M[row * PT + (L.c ^ row) + 16 * kt * PT + 16 * ti];
}
template <int PT, class T>
__device__ __forceinline__ T ldR(const Ln<T> &L, const T *M, int ti, int kt, int r) {
    return M[L.c * PT + (L.c ^ L.row(r)) + 16 * ti * PT + 16 * kt];
}

// Keeps the operand reads of one tile product from being moved across the
// products before it: the compiler would otherwise issue the reads of a whole
// phase at once and spill.  Up to two tiles a side there is room for them.
template <int PITCH>
__device__ __forceinline__ void tile_fence() {
    if (PITCH > 32) __builtin_amdgcn_sched_barrier(0);
}

// acc += sum over inner tiles k0 <= kt < KT of (N view of M)(ti, kt) b[kt], NS
// slices each.
// The next inner tile's operands are read while this one's are multiplied.
template <int PT, int KT, int NS, class T>
__device__ __forceinline__ v4_t<T> mulN(const Ln<T> &L, v4_t<T> acc, const T *M, int ti, const v4_t<T> *b, int k0 = 0) {
    tile_fence<(PT > 16 * KT ? PT : 16 * KT)>();
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
        if (kt < k0) continue;
        T a[4];
#pragma unroll
        for (int r = 0; r < NS; ++r) a[r] = ldN<PT>(L, M, kt, ti, r);
#pragma unroll
        for (int r = 0; r < NS; ++r) acc = MT<T>::mfma(a[r], b[kt][r], acc);
    }
    tile_fence<(PT > 16 * KT ? PT : 16 * KT)>();
    return acc;
}

// Tile (ti, tj) of C written at LDS (row, column) and, for a lower tile of a
// symmetric result, also mirrored (the diagonal tile's upper half is the
// mirror of its lower half).
template <int PT, int NS, class T>
__device__ __forceinline__ void put(const Ln<T> &L, T *M, int ti, int tj, v4_t<T> v) {
#pragma unroll
    for (int r = 0; r < NS; ++r) M[at<PT>(16 * ti + L.row(r), 16 * tj + L.c)] = v[r];
}
template <int PT, int NS, class T>
__device__ __forceinline__ void put_sym(const Ln<T> &L, T *M, int ti, int tj, v4_t<T> v) {
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const int i = 16 * ti + L.row(r), j = 16 * tj + L.c;
        if (ti != tj || i >= j) {
            M[at<PT>(i, j)] = v[r];
            M[at<PT>(j, i)] = v[r];
        }
    }
}

__device__ __forceinline__ double rcp_est(double d) { return __builtin_amdgcn_rcp(d); }
__device__ __forceinline__ float rcp_est(float d) { return __builtin_amdgcn_rcpf(d); }
// A pivot whose reciprocal is neither subnormal nor infinite (the hardware's
// estimate flushes those).
__device__ __forceinline__ bool plain_pivot(double d) { return d >= 0x1p-1021 && d <= 0x1p+1021; }
__device__ __forceinline__ bool plain_pivot(float d) { return d >= 0x1p-125f && d <= 0x1p+125f; }

// Value of lane 16 H + i in the lanes i of all four rows of 16: two swaps
// between rows (the pairs of rows, then the halves of the wave).
template <int H>
__device__ __forceinline__ unsigned row_to_all(unsigned v) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const unsigned u = p[H & 1];
    const auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return q[H >> 1];
}
template <int H>
__device__ __forceinline__ double row_to_all(double v) {
    return __hiloint2double((int)row_to_all<H>((unsigned)__double2hiint(v)),
                            (int)row_to_all<H>((unsigned)__double2loint(v)));
}
template <int H>
__device__ __forceinline__ float row_to_all(float v) {
    return __uint_as_float(row_to_all<H>(__float_as_uint(v)));
}

// Value of lane N of this lane's row of 16 (every lane has a source: the old
// value of the destination is not used).
template <int N>
__device__ __forceinline__ double row16(double v) {
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(__double_as_longlong(v), 0x150 + N, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float row16(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xF, 0xF, true));
}
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Step K of the in-place elimination below: column K of the block becomes
// column K of L_u^{-1}.  The lanes that hold column K (row group H = K / 4)
// form the multipliers from the pivot, which reaches them by DPP, and hand
// them to the other groups by row swaps, so that no step waits for LDS or for
// a scalar register.  a / d from the hardware's estimate r of 1 / d:
// a r (1 + e + e^2) with e = 1 - d r (e^3 is below the rounding).  The pivots
// stay on the diagonal: they are checked, and their square roots taken, at
// the end (see chol_block_any for the blocks that fail the check).
template <int K, class T>
__device__ __forceinline__ void elim_step(T (&a)[4], int i, int h, int steps) {
    if constexpr (K % 4 == 0 && K > 0) {
        if (K >= steps) return;                       // padding: unit pivots, nothing to eliminate
    }
    constexpr int H = K >> 2, kc = K & 3;
    T pr[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) pr[c] = row16<K>(a[c]);     // row K; pr[kc] in row group H: the pivot
    const T r = rcp_est(pr[kc]), e = fma_t(-pr[kc], r, T(1)), f = -a[kc] * r;
    const T nm = row_to_all<H>(i > K ? fma_t(f, fma_t(e, e, e), f) : T(0));    // rows above the pivot keep their values
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const T t = fma_t(nm, pr[c], a[c]);
        a[c] = (c == kc && h == H && i > K) ? nm : t;
    }
    if constexpr (K + 1 < 16) elim_step<K + 1>(a, i, h, steps);
}

// Reciprocal square root of a pivot, or of the unit pivot that takes the place of
// one that is not positive or not finite (fail is set).
template <class T>
__device__ __forceinline__ T pivot_rsq(T d, int &fail) {
    if (!(d > T(0)) || !__builtin_isfinite(d)) {
        fail = 1;
        d = T(1);
    }
    T s = mf::rsq_est(d);
    s = s * (T(1.5) - T(0.5) * d * s * s);
    return s * (T(1.5) - T(0.5) * d * s * s);
}

// chol_block for a block with a pivot that is not plain: one step after another
// through the pivots' square roots, in LDS (so that it needs few registers), a
// failed factorization going on with unit pivots, and so with numbers.
template <int PU, int GS, class T>
__device__ __forceinline__ int chol_block_any(T *G, int kb, int steps) {
    int l = lane();
    asm volatile("" : "+v"(l));
    const int i = l & 15, j0 = 4 * (l >> 4), o = 16 * kb;
    int fail = 0;
    if (GS > 1) {
#pragma unroll 1
        for (int c = 0; c < 4; ++c) {
            T v = G[at<PU>(o + i, o + j0 + c)];
#pragma unroll 1
            for (int g = 1; g < GS; ++g) v += G[g * PU * PU + at<PU>(o + i, o + j0 + c)];
            G[at<PU>(o + i, o + j0 + c)] = v;
        }
    }
#pragma unroll 1
    for (int K = 0; K < steps && K < 16; ++K) {
        wave_fence();
        const T s = pivot_rsq(G[at<PU>(o + K, o + K)], fail);
        const T nm = i > K ? -(G[at<PU>(o + i, o + K)] * s) * s : T(0);
        wave_fence();
#pragma unroll 1
        for (int j = j0; j < j0 + 4; ++j) {
            T &e = G[at<PU>(o + i, o + j)];
            const T t = fma_t(nm, G[at<PU>(o + K, o + j)], e);
            if (i > K) e = j == K ? nm : t;
        }
    }
    wave_fence();
    int none = 0;
    const T is = pivot_rsq(G[at<PU>(o + i, o + i)], none);
    wave_fence();
#pragma unroll 1
    for (int j = j0; j < j0 + 4; ++j) {
        T &e = G[at<PU>(o + i, o + j)];
        e = j < i ? e * is : j == i ? is : T(0);
    }
    return fail;
}

// Inverse Cholesky factor of the 16 x 16 diagonal block kb of G, in place
// (upper half zero), by one wavefront: Gaussian elimination without pivoting
// in place (lane i + 16 h holds columns 4 h .. 4 h + 3 of row i) turns the
// block into D L_u' on and above the diagonal and L_u^{-1} below it, with
// G = L_u D L_u', so that L^{-1} = D^{-1/2} L_u^{-1}: the same factorization
// and forward substitution as the textbook sweep, in the 256 elements of the
// block itself.  `steps`: rows that are not padding.  (On [G | I], with twice
// the elements, a square root in every step and the pivot through scalar
// registers, a block took 5 to 6 k cycles; in place with the column through
// LDS 4.2 k; here 3.0 k.)
template <int PU, int GS = 1, class T>
__device__ __forceinline__ int chol_block(T *G, int kb, int steps) {
    int l = lane();
    asm volatile("" : "+v"(l));          // lane constants are not kept across stages
    const int i = l & 15, h = l >> 4;
    T a[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        a[c] = G[at<PU>(16 * kb + i, 16 * kb + 4 * h + c)];
#pragma unroll
        for (int g = 1; g < GS; ++g) a[c] += G[g * PU * PU + at<PU>(16 * kb + i, 16 * kb + 4 * h + c)];
    }
    elim_step<0>(a, i, h, steps);
    const T p01 = (i & 1) ? a[1] : a[0], p23 = (i & 1) ? a[3] : a[2];
    const T piv = __shfl((i & 2) ? p23 : p01, 16 * (i >> 2) + i, 64);        // row i's pivot, from row group i / 4
    if (__any(i < steps && !plain_pivot(piv))) return chol_block_any<PU, GS>(G, kb, steps);
    T is = mf::rsq_est(piv);
    is = is * (T(1.5) - T(0.5) * piv * is * is);
    is = is * (T(1.5) - T(0.5) * piv * is * is);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int j = 4 * h + c;
        G[at<PU>(16 * kb + i, 16 * kb + j)] = j < i ? a[c] * is : j == i ? is : T(0);
    }
    return 0;
}

// Cholesky factorization and inverse of the NB x NB blocks of G (lower part
// and full diagonal blocks given; m rows, the rest identity), by one
// wavefront, in place: on return the lower blocks hold L^{-1} (the diagonal
// ones with a zero upper half), the upper ones the off-diagonal blocks of L'.
// Right-looking over 16-wide blocks: L_kk^{-1}, L_ik' = L_kk^{-1} G_ik',
// G_ij -= L_ik L_jk'; then block row by block row of the inverse,
// X_ij = -X_ii sum_k L_ik X_kj.  Returns nonzero if a pivot failed.  GS: G is
// the sum of so many matrices, one after the other.
template <class T, int NB, int GS>
__device__ __forceinline__ int chol_inv(const Ln<T> &L, T *G, int m) {
    constexpr int PU = 16 * NB;
    int fail = 0;
    if constexpr (NB > 1 && GS > 1) {
#pragma unroll 4
        for (int e = lane(); e < PU * PU; e += 64) {
            T v = G[e];
#pragma unroll
            for (int g = 1; g < GS; ++g) v += G[g * PU * PU + e];
            G[e] = v;
        }
        wave_fence();
    }
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
        fail |= chol_block<PU, NB == 1 ? GS : 1>(G, kb, m - 16 * kb);
        if constexpr (NB == 1) return fail;
        wave_fence();
        // L_ik' into the upper block (k, i)
        v4_t<T> u[NB];
#pragma unroll
        for (int ib = kb + 1; ib < NB; ++ib) {
            v4_t<T> acc = zero4<T>();
#pragma unroll
            for (int r = 0; r < 4; ++r)          // G_ik' (k, i) = G[i][k]
                acc = MT<T>::mfma(ldR<PU>(L, G, kb, kb, r), ldR<PU>(L, G, ib, kb, r), acc);
            u[ib] = acc;
            put<PU, 4>(L, G, kb, ib, acc);
        }
        wave_fence();
#pragma unroll
        for (int jb = kb + 1; jb < NB; ++jb)
#pragma unroll
            for (int ib = jb; ib < NB; ++ib) {
                v4_t<T> acc = zero4<T>();
#pragma unroll
                for (int r = 0; r < 4; ++r) acc = MT<T>::mfma(ldN<PU>(L, G, kb, ib, r), u[jb][r], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = at<PU>(16 * ib + L.row(r), 16 * jb + L.c);
                    G[e] -= acc[r];
                }
            }
        wave_fence();
    }
#pragma unroll
    for (int ib = 1; ib < NB; ++ib) {
#pragma unroll
        for (int jb = 0; jb < ib; ++jb) {
            v4_t<T> s = zero4<T>();
#pragma unroll
            for (int kb = jb; kb < ib; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s = MT<T>::mfma(ldN<PU>(L, G, kb, ib, r), ldN<PU>(L, G, kb, jb, r), s);
            v4_t<T> x = zero4<T>();
#pragma unroll
            for (int r = 0; r < 4; ++r) x = MT<T>::mfma(ldR<PU>(L, G, ib, ib, r), s[r], x);
            put<PU, 4>(L, G, ib, jb, v4_t<T>{-x[0], -x[1], -x[2], -x[3]});
        }
        wave_fence();
    }
    return fail;
}

// LDS of one workgroup.  Y and X lie over A and B (dead once W, F, H', A'V
// and B'V are formed) where they do not fit beside them; the next stage's A
// and B are then written after one more barrier.
//
// SX, SU: row slices in use of a tile of states and of inputs.  A slice is the
// rows that one matrix instruction takes as inner indices (4 in FP64: rows
// 4 r .. 4 r + 3), so shapes of up to 4 or 8 states need one or two of the
// four (one tile, FP64); rows beyond them are neither written nor read.
template <class T, int NXT, int NUT, int SX_ = 4, int SU_ = 4>
struct Smem {
    typedef T elem;
    static constexpr int SX = SX_, SU = SU_;
    static_assert((SX == 4 && SU == 4) || (NXT == 1 && sizeof(T) == 8), "slices of one FP64 tile");
    static constexpr int RX = 16 * NXT, RU = 16 * NUT, NTH = 128 * NXT;
    static constexpr size_t apart = sizeof(T) * (2 * RX * RX + RX * RU + RU * RU + 2 * RU * RX);
    static constexpr bool OVER = apart > 159 * 1024;
    // Waves per column block of G (each takes NUT of the inner tiles of B'W_B
    // where fewer than half of the owners of A's columns would have one).
    static constexpr int GS = (NUT < NXT && NXT % NUT == 0) ? NXT / NUT : 1;
    static constexpr int WT = GS > 1 ? NUT : NXT;       // row tiles of W_B per wave
    T P[RX * RX], A[RX * RX], B[RX * RU], G[GS * RU * RU];
    T YX[OVER ? 1 : 2 * RU * RX];
    double av[RX], pt[RX], gw[RU], z[RU];      // VEC
    double red[2 * NXT];
    int bad;
    __device__ T *Y() { return OVER ? A : YX; }
    __device__ T *X() { return OVER ? B : YX + (OVER ? 0 : RU * RX); }
};

// Column blocks that outlive a stage (Alg. 4): V(:, j) and the lower tiles
// of Q_w_hat(:, j) of wave NXT + j.
template <class T, int NXT>
struct Cols {
    v4_t<T> V[NXT], Q[NXT];
};

// Where the factors of a stage go (row-major; nullptr: not kept; K and, with
// VEC, L_t always are), and Psi_t and k_{t+1} (VEC).
template <class T>
struct Rec {
    T *P, *K, *V, *Lt, *L, *LT;
    double *Psi, *k;
};
// Running right-hand side of a pass (VEC) in its owners' lanes: entry 16 j +
// lane % 16 of Psi (waves j) and of v (waves NXT + j), and this lane's part of
// cbar (without the constants c).
struct Vec {
    double psi, v, cb;
};

// Sum over the four lanes that hold one column of a result tile.
__device__ __forceinline__ double q_sum(double v) { return sv::xor_sum<32>(sv::xor_sum<16>(v)); }

// Accesses to global memory in the stage loops go through buffer descriptors:
// a load beyond the array gives zero and a store beyond it is dropped, so
// bounds, absent arrays and the last stage need no branch.  Without branches
// around them the number of accesses in flight is known wherever a loaded
// value is used, and a wait for it does not also wait for the record stores
// and the next loads issued since (stores and loads share one counter; with
// branches the waits of a stage were for an empty counter).
constexpr uint32_t BEYOND = 0x40000000u;      // a byte offset outside every array
typedef __amdgpu_buffer_rsrc_t Buf;
// `count` elements from p (uniform), none if p is null or !on.
template <class U>
__device__ __forceinline__ Buf buf(const U *p, int count, bool on = true) {
    void *q = const_cast<double *>(uni_ptr(reinterpret_cast<const double *>(p)));
    return __builtin_amdgcn_make_buffer_rsrc(q, 0, q && on ? count * (int)sizeof(U) : 0, 0x00020000);
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// byte: this lane's offset, the bounded part; sbyte: a uniform offset on top
// (full tiles, where nothing is out of bounds: it takes no vector register).
__device__ __forceinline__ double buf_ld(Buf b, uint32_t byte, uint32_t sbyte = 0) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, (int)byte, (int)sbyte, 0));
}
template <class T>
__device__ __forceinline__ T buf_get(Buf b, uint32_t byte) {
    if constexpr (sizeof(T) == 8)
        return buf_ld(b, byte);
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, (int)byte, 0, 0));
}
__device__ __forceinline__ void buf_st(Buf b, uint32_t byte, double v, uint32_t sbyte = 0) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, (int)byte, (int)sbyte, 0);
}
__device__ __forceinline__ void buf_st(Buf b, uint32_t byte, float v, uint32_t sbyte = 0) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), b, (int)byte, (int)sbyte, 0);
}
// Drains this wave's global accesses.
__device__ __forceinline__ void drain() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// 16x16 tile of problem data (n1 x n2 in all, rows of length ld) in the result
// layout; zeros outside (identity where ONE).  TR: the array holds the
// transpose.
template <bool EX, bool TR, bool ONE, int NS, class T>
__device__ __forceinline__ d4 load_tile(const Ln<T> &L, Buf M, int ld, int ti, int tj, int n1, int n2) {
    d4 v{0.0, 0.0, 0.0, 0.0};
    const int j = 16 * tj + L.c;
    const bool in = EX || TR || j < n2;        // the other index is bounded by the array's length
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const int i = 16 * ti + L.row(r);
        if (EX) {
            const int si = 16 * ti + L.row(r) - L.row(0), sj = 16 * tj;
            v[r] = buf_ld(M, 8u * (uint32_t)(TR ? L.c * ld + L.row(0) : L.row(0) * ld + L.c),
                          8u * (uint32_t)(TR ? sj * ld + si : si * ld + sj));
            continue;
        }
        const uint32_t e = 8u * (uint32_t)(TR ? j * ld + i : i * ld + j);
        v[r] = buf_ld(M, (TR ? i < n1 : in) ? e : BEYOND);
        if (ONE && !EX) v[r] = (i == j && i >= n1) ? 1.0 : v[r];
    }
    return v;
}
template <class T>
__device__ __forceinline__ v4_t<T> as_t(d4 v) {
    return v4_t<T>{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
}

// Result tile (ti, tj) to global memory (rows of length ld, n2 columns in use).
template <bool EX, int NS, class T>
__device__ __forceinline__ void store_tile(const Ln<T> &L, Buf M, int ld, int ti, int tj, int n2, v4_t<T> v) {
    const int j = 16 * tj + L.c;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        constexpr uint32_t B = sizeof(T);
        if (EX)
            buf_st(M, B * (uint32_t)(L.row(0) * ld + L.c), v[r],
                   B * (uint32_t)((16 * ti + L.row(r) - L.row(0)) * ld + 16 * tj));
        else
            buf_st(M, j < n2 ? B * (uint32_t)((16 * ti + L.row(r)) * ld + j) : BEYOND, v[r]);
    }
}

// P (n x n) from LDS to global memory, row by row, by the threads
// t0 <= threadIdx.x < t1.
template <class SM, class U>
__device__ __forceinline__ void copy_P(const SM &S, U *dst, int n, int t0 = 0, int t1 = SM::NTH) {
    int t = (int)threadIdx.x - t0;
    const int nt = t1 - t0;
    if (t < 0 || t >= nt) return;
    asm volatile("" : "+v"(t));
#pragma unroll 4
    for (int e = t; e < SM::RX * SM::RX; e += nt) {
        const int i = e / SM::RX, j = e % SM::RX;
        if (i < n && j < n) dst[(uint32_t)(i * n + j)] = (U)S.P[at<SM::RX>(i, j)];
    }
}
// The same by NT threads (t their index) inside a stage loop, where it may be
// switched off without a branch.
template <bool EX, int NT, class SM, class U>
__device__ __forceinline__ void put_P(const SM &S, U *dst, int n, int t, bool on) {
    constexpr int RX = SM::RX, W = (4 * SM::SX < 16 && RX == 16) ? 4 * SM::SX : RX;    // rows and columns in use
    const Buf b = buf(dst, n * n, on);
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int q = 0; q < (W * W + NT - 1) / NT; ++q) {
        const int e = t + q * NT, i = e / W, j = e % W;
        const uint32_t o = (uint32_t)sizeof(U) * (uint32_t)(i * n + j);
        const bool all = W * W % NT == 0;
        const U v = (U)S.P[at<RX>(all || i < W ? i : 0, j)];
        if (EX && all)
            buf_st(b, (uint32_t)sizeof(U) * (uint32_t)t, v, (uint32_t)sizeof(U) * (uint32_t)(q * NT));
        else
            buf_st(b, (EX || j < n) && (all || i < W) ? o : BEYOND, v);
    }
}

// Start of a pass: P from an element function (rows and columns < n).
template <class SM, class F>
__device__ __forceinline__ void set_P(SM &S, int n, F f) {
    typedef typename SM::elem T;
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
#pragma unroll 4
    for (int e = t; e < SM::RX * SM::RX; e += SM::NTH) {
        const int i = e / SM::RX, j = e % SM::RX;
        S.P[at<SM::RX>(i, j)] = (i < n && j < n) ? (T)f(i * n + j) : T(0);
    }
}

// L^{-1} and L^{-T} (m x m, dense) from LDS to their records, by NT threads (t
// their index).
template <bool EX, int NT, class SM, class T>
__device__ __forceinline__ void put_L(const SM &S, T *L, T *LT, int m, int t) {
    constexpr int RU = SM::RU, W = (4 * SM::SU < 16 && RU == 16) ? 4 * SM::SU : RU;
    const Buf b = buf(L, m * m), bt = buf(LT, m * m);
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int q = 0; q < (W * W + NT - 1) / NT; ++q) {
        const int e = t + q * NT, i = e / W, k = e % W;
        const bool in = (EX || k < m) && (W * W % NT == 0 || e < W * W);
        const uint32_t o = in ? (uint32_t)sizeof(T) * (uint32_t)(i * m + k) : BEYOND;
        const int is = W * W % NT == 0 || i < W ? i : 0;
        buf_st(b, o, k <= i ? S.G[at<RU>(is, k)] : T(0));
        buf_st(bt, o, i <= k ? S.G[at<RU>(k, is)] : T(0));
    }
}

// Y = L^{-1} H' or X = L^{-1} B'V of one column block, in place and to LDS.
// L^{-1} is lower triangular: row tile ti takes the inner tiles <= ti, so the
// block is replaced from its last tile up.  Z: also z = L^{-1} gw (to zv).
template <int RU, int RX, int NUT, int NS, bool Z = false, class T>
__device__ __forceinline__ void apply_Linv(const Ln<T> &L, const T *G, v4_t<T> *R2, T *D, int j,
                                           const double *gw = nullptr, double *zv = nullptr, double *zz = nullptr) {
#pragma unroll
    for (int ti = NUT - 1; ti >= 0; --ti) {
        tile_fence<RX>();
        v4_t<T> acc = zero4<T>();
        double z = 0.0;
#pragma unroll
        for (int kt = 0; kt <= ti; ++kt)
#pragma unroll
            for (int r = 0; r < NS; ++r) {
                const T a = ldR<RU>(L, G, ti, kt, r);
                acc = MT<T>::mfma(a, R2[kt][r], acc);
                if constexpr (Z) z += (double)a * gw[16 * kt + L.row(r)];
            }
        R2[ti] = acc;
        put<RX, NS>(L, D, ti, j, acc);
        if constexpr (Z) {
            z = q_sum(z);
            if (L.q == 0 && (NS == 4 || L.c < 4 * NS)) {
                zv[16 * ti + L.c] = z;
                *zz -= 0.5 * z * z;
            }
        }
    }
}

// K = -L^{-T} Y or L_t = -L^{-T} X of one column block, to its record.  Z:
// also k = L^{-T} z.
template <bool EX, int RU, int RX, int NUT, int NS, bool Z = false, class T>
__device__ __forceinline__ void store_feedback(const Ln<T> &L, const T *G, const v4_t<T> *R2, T *D, int j, int n, int m,
                                               const double *zv = nullptr, double *k = nullptr) {
    const Buf bd = buf(D, n * m), bk = buf(k, m);
#pragma unroll
    for (int ti = 0; ti < NUT; ++ti) {
        tile_fence<RX>();
        v4_t<T> acc = zero4<T>();
        double s = 0.0;
#pragma unroll
        for (int kt = ti; kt < NUT; ++kt)
#pragma unroll
            for (int r = 0; r < NS; ++r) {
                const T a = ldN<RU>(L, G, kt, ti, r);
                acc = MT<T>::mfma(a, R2[kt][r], acc);
                if constexpr (Z) s += (double)a * zv[16 * kt + L.row(r)];
            }
        store_tile<EX, NS>(L, bd, n, ti, j, n, v4_t<T>{-acc[0], -acc[1], -acc[2], -acc[3]});
        if constexpr (Z) {
            s = q_sum(s);
            buf_st(bk, 8u * (uint32_t)(16 * ti + L.c), s);       // (the four lanes of a column hold the same sum)
        }
    }
}

// The inputs a wave that owns a column block of A adds to its products, loaded
// one stage ahead: G's during W, F's and H''s with one tile as soon as this
// stage's are in use (EARLY), otherwise when this stage's P has left their
// registers.
template <int NXT, int NUT>
struct QTiles {
    static constexpr bool EARLY = NXT == 1;
    d4 g[NUT], f[NXT], h[NUT];
    double lx, lw;
};

// Stage loop of the waves that own a column block of A (w < NXT).
template <bool RED, bool EX, bool EXD, bool VEC, bool KEEP, class T, int NXT, int NUT, int SX, int SU, class Pre, class RecOf>
__device__ __forceinline__ void loop_P(Smem<T, NXT, NUT, SX, SU> &S, int n, int m, int md, StageWalk wk, int count, int32_t *info, int inst,
                                       int stage_base, int fail_code, Pre pre, RecOf rec, Vec &y) {
    using SM = Smem<T, NXT, NUT, SX, SU>;
    using QT = QTiles<NXT, NUT>;
    constexpr int RX = SM::RX, RU = SM::RU, GS = SM::GS, WT = SM::WT;
    const int j = wave();
    const bool zs = j == NXT - 1;           // owner of z and k (with the fewest tiles of F and P)
    QT q;
    auto load_g = [&](const Ln<T> &L, const StageSrc &src, bool on) {
#pragma unroll
        for (int ti = 0; ti < NUT; ++ti)
            q.g[ti] = load_tile<EXD, false, true, SU>(L, buf(src.Qw, md * md, on && j <= ti), md, ti, j, md, md);
        if constexpr (VEC) q.lw = buf_ld(buf(src.lw, md, on), 8u * (uint32_t)(16 * j + L.c));
    };
    auto load_f = [&](const Ln<T> &L, const StageSrc &src, bool on) {
        const Buf bh = buf(src.Qxw, n * md, on);
#pragma unroll
        for (int ti = 0; ti < NUT; ++ti) q.h[ti] = load_tile<EXD, true, false, SU>(L, bh, md, ti, j, md, n);
#pragma unroll
        for (int ti = 0; ti < NXT; ++ti)
            q.f[ti] = load_tile<EX, false, false, SX>(L, buf(src.Qx, n * n, on && ti >= j), n, ti, j, n, n);
        if constexpr (VEC) q.lx = buf_ld(buf(src.lx, n, on), 8u * (uint32_t)(16 * j + L.c));
    };
    {
        const Ln<T> L;
        load_g(L, wk.s, true);
        load_f(L, wk.s, true);
        drain();
    }
    lds_sync();
    for (int s = count - 1; s >= 0; --s) {
        const Ln<T> L;
        double pa = 0.0;
        if constexpr (VEC) {
            // ---- pt = Psi - P a, cbar += 1/2 a'Pa - Psi'a
#pragma unroll
            for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                for (int r = 0; r < SX; ++r) pa += ldN<RX>(L, S.P, kt, j, r) * S.av[16 * kt + L.row(r)];
            pa = q_sum(pa);
            if (L.q == 0) {
                S.pt[16 * j + L.c] = y.psi - pa;
                y.cb += S.av[16 * j + L.c] * (0.5 * pa - y.psi);
            }
        }
        // ---- G = Qw + B'PB: column block jb by GS waves, each with its row
        // tiles of W_B = P B
        if (j < GS * NUT) {
            const int jb = GS > 1 ? j % NUT : j, h = GS > 1 ? j / NUT : 0;
            v4_t<T> b[NXT], wb[WT];
#pragma unroll
            for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                for (int r = 0; r < SX; ++r) b[kt][r] = ldN<RU>(L, S.B, kt, jb, r);
#pragma unroll
            for (int ti = 0; ti < WT; ++ti) wb[ti] = mulN<RX, NXT, SX>(L, zero4<T>(), S.P, h * WT + ti, b);
#pragma unroll
            for (int ti = 0; ti < NUT; ++ti)
                if (ti >= jb)
                    put_sym<RU, SU>(L, S.G + h * RU * RU, ti, jb,
                                    mulN<RU, WT, SX>(L, h == 0 ? as_t<T>(q.g[ti]) : zero4<T>(),
                                                     S.B + 16 * WT * h * RU, ti, wb));
        }
        lds_sync();
        // ---- W, F, H', g_x, g_w (the last wave of the workgroup factors G)
        v4_t<T> R1[NXT], R2[NUT];
        double gx = 0.0;
        if (s > 0) wk.back();           // the next stage
        {
            v4_t<T> a[NXT], wa[NXT];
#pragma unroll
            for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                for (int r = 0; r < SX; ++r) a[kt][r] = ldN<RX>(L, S.A, kt, j, r);
            if constexpr (VEC) {
#pragma unroll
                for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                    for (int r = 0; r < SX; ++r) gx += a[kt][r] * S.pt[16 * kt + L.row(r)];
                gx = q_sum(gx) - q.lx;
                if (j < NUT) {
                    double g = 0.0;
#pragma unroll
                    for (int kt = 0; kt < NXT; ++kt)
#pragma unroll
                        for (int r = 0; r < SX; ++r) g += ldN<RU>(L, S.B, kt, j, r) * S.pt[16 * kt + L.row(r)];
                    g = q_sum(g) - q.lw;
                    if (L.q == 0) S.gw[16 * j + L.c] = g;
                }
            }
            load_g(L, wk.s, s > 0);
#pragma unroll
            for (int ti = 0; ti < NXT; ++ti) wa[ti] = mulN<RX, NXT, SX>(L, zero4<T>(), S.P, ti, a);
#pragma unroll
            for (int ti = 0; ti < NUT; ++ti) R2[ti] = mulN<RU, NXT, SX>(L, as_t<T>(q.h[ti]), S.B, ti, wa);
#pragma unroll
            for (int ti = 0; ti < NXT; ++ti)
                if (ti >= j) R1[ti] = mulN<RX, NXT, SX>(L, as_t<T>(q.f[ti]), S.A, ti, wa);
        }
        if (QT::EARLY) load_f(L, wk.s, s > 0);
        if constexpr (NXT == 1) {
            // the record of P_{s+1}, still in LDS (the other wave factors G)
            pre(s, 0, 64);
            if (KEEP) put_P<EX, 64>(S, rec(s + 1 < count ? s + 1 : s).P, n, threadIdx.x, s + 1 < count);
        }
        lds_sync();
        if (threadIdx.x == 0 && S.bad) {
            record_failure(info, inst, fail_code, stage_base < 0 ? -1 : stage_base + s);
            S.bad = 0;
        }
        if (VEC && zs)
            apply_Linv<RU, RX, NUT, SU, VEC>(L, S.G, R2, S.Y(), j, S.gw, S.z, &y.cb);
        else
            apply_Linv<RU, RX, NUT, SU>(L, S.G, R2, S.Y(), j);
        lds_sync();
        // ---- P = F - Y'Y, K = -L^{-T} Y, Psi = g_x - Y'z, k = L^{-T} z
        const Rec<T> out = rec(s);
#pragma unroll
        for (int ti = 0; ti < NXT; ++ti)
            if (ti >= j) {
                const v4_t<T> acc = mulN<RX, NUT, SU>(L, zero4<T>(), S.Y(), ti, R2);
                put_sym<RX, SX>(L, S.P, ti, j,
                            v4_t<T>{R1[ti][0] - acc[0], R1[ti][1] - acc[1], R1[ti][2] - acc[2], R1[ti][3] - acc[3]});
            }
        if (!QT::EARLY) load_f(L, wk.s, s > 0);
        if constexpr (VEC) {
            double yz = 0.0;
#pragma unroll
            for (int ti = 0; ti < NUT; ++ti)
#pragma unroll
                for (int r = 0; r < SU; ++r) yz += R2[ti][r] * S.z[16 * ti + L.row(r)];
            y.psi = gx - q_sum(yz);
            if (KEEP) buf_st(buf(out.Psi, n), 8u * (uint32_t)(16 * j + L.c), y.psi);
        }
        if (KEEP) store_feedback<EX, RU, RX, NUT, SU, VEC>(L, S.G, R2, out.K, j, n, m, S.z, zs ? out.k : nullptr);
        if (RED && !VEC) put_L<EX, 64 * NXT>(S, out.L, out.LT, m, threadIdx.x);
        lds_sync();
        if (SM::OVER) lds_sync();
    }
}

// Stage loop of the waves NXT + j: A and B of the next stage are loaded into
// their registers, the last of them (CH) factors G, and for Alg. 4 they own the
// column blocks of V and Q_w_hat.
template <bool CH, bool RED, bool EX, bool EXD, bool VEC, bool KEEP, class T, int NXT, int NUT, int SX, int SU, class Pre, class RecOf>
__device__ __forceinline__ void loop_V(Smem<T, NXT, NUT, SX, SU> &S, Cols<T, NXT> &C, int n, int m, int md, StageWalk wk, int count, Pre pre,
                                       RecOf rec, Vec &y) {
    using SM = Smem<T, NXT, NUT, SX, SU>;
    constexpr int RX = SM::RX, RU = SM::RU, NTV = 64 * NXT;
    constexpr int NA = RX * RX / NTV, NB = RX * RU / NTV;
    static_assert(RX * RX % NTV == 0 && RX * RU % NTV == 0, "whole rounds");
    const int j = wave() - NXT;
    double pa[NA], pb[NB], pv = 0.0;
    auto fetch = [&](const StageSrc &src, bool on) {
        int tv = (int)threadIdx.x - NTV;
        asm volatile("" : "+v"(tv));
        const Buf ba = buf(src.A, n * n, on), bb = buf(src.B, n * md, on);
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int e = tv + q * NTV, i = e / RX, k = e % RX;
            pa[q] = EX ? buf_ld(ba, 8u * (uint32_t)tv, 8u * (uint32_t)(q * NTV))
                       : buf_ld(ba, k < n ? 8u * (uint32_t)(i * n + k) : BEYOND);
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int e = tv + q * NTV, i = e / RU, k = e % RU;
            pb[q] = EXD ? buf_ld(bb, 8u * (uint32_t)tv, 8u * (uint32_t)(q * NTV))
                        : buf_ld(bb, k < md ? 8u * (uint32_t)(i * md + k) : BEYOND);
        }
        if constexpr (VEC) pv = buf_ld(buf(src.a, n, on), 8u * (uint32_t)tv);
    };
    auto commit = [&]() {
        int tv = (int)threadIdx.x - NTV;
        asm volatile("" : "+v"(tv));
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int e = tv + q * NTV;
            S.A[at<RX>(e / RX, e % RX)] = (T)pa[q];
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int e = tv + q * NTV;
            S.B[at<RU>(e / RU, e % RU)] = (T)pb[q];
        }
        if (VEC && tv < RX) S.av[tv] = pv;
    };
    if (RED) {
        const Ln<T> L;
#pragma unroll
        for (int ti = 0; ti < NXT; ++ti) {
            C.Q[ti] = zero4<T>();
#pragma unroll
            for (int r = 0; r < SX; ++r)
                C.V[ti][r] = (16 * ti + L.row(r) == 16 * j + L.c) ? T(1) : T(0);
        }
    }
    // What is not on the chain of a stage is left to the waves that wait for
    // the factor of G: A'V, and Q_w_hat += X'X of the stage before (X keeps its
    // place in LDS unless that is B's).
    constexpr bool QD = RED && !CH && !SM::OVER;
    // The product is summed by itself and added once: with the running sum as
    // the matrix instructions' addend every inner step rounds at its size, and
    // the FP32 reductions lost a factor of 2 to 6 of their accuracy (mixed
    // plans took one more correction; 64 problems of 64 x 32 in FP64 run 1 %
    // longer this way).
    auto add_Q = [&](const Ln<T> &L, const v4_t<T> *X) {
#pragma unroll
        for (int ti = 0; ti < NXT; ++ti)
            if (ti >= j) C.Q[ti] += mulN<RX, NUT, SU>(L, zero4<T>(), S.X(), ti, X);
    };
    auto add_Q_late = [&](const Ln<T> &L) {
        v4_t<T> X[NUT];
#pragma unroll
        for (int kt = 0; kt < NUT; ++kt)
#pragma unroll
            for (int r = 0; r < SU; ++r) X[kt][r] = ldN<RX>(L, S.X(), kt, j, r);
        add_Q(L, X);
    };
    fetch(wk.s, true);
    commit();
    lds_sync();
    for (int s = count - 1; s >= 0; --s) {
        const Ln<T> L;
        v4_t<T> R1[NXT], R2[NUT];
        auto mul_A = [&] {
#pragma unroll
            for (int ti = 0; ti < NXT; ++ti) R1[ti] = mulN<RX, NXT, SX>(L, zero4<T>(), S.A, ti, C.V);
        };
        if (s > 0) wk.back();
        if (NXT == 1) fetch(wk.s, s > 0);
        if (RED) {
            if constexpr (VEC) {
                double va = 0.0;
#pragma unroll
                for (int ti = 0; ti < NXT; ++ti)
#pragma unroll
                    for (int r = 0; r < SX; ++r) va += C.V[ti][r] * S.av[16 * ti + L.row(r)];
                y.v += q_sum(va);
            }
#pragma unroll
            for (int ti = 0; ti < NUT; ++ti) R2[ti] = mulN<RU, NXT, SX>(L, zero4<T>(), S.B, ti, C.V);
            if (CH) mul_A();
        }
        lds_sync();
        if constexpr (CH) {
            const int f = chol_inv<T, NUT, SM::GS>(L, S.G, md);
            if (f && lane() == 0) S.bad = 1;
            tile_fence<RX>();
            if (NXT > 1) fetch(wk.s, s > 0);
        } else {
            if (QD && s + 1 < count) add_Q_late(L);
            if (RED) mul_A();
            tile_fence<RX>();
            if (NXT > 1) fetch(wk.s, s > 0);
            // the record of P_{s+1}, still in LDS
            pre(s, NTV, 2 * NTV - 64);
            if (KEEP) put_P<EX, NTV - 64>(S, rec(s + 1 < count ? s + 1 : s).P, n, (int)threadIdx.x - NTV, s + 1 < count);
        }
        lds_sync();
        const Rec<T> out = rec(s);
        if (RED) apply_Linv<RU, RX, NUT, SU>(L, S.G, R2, S.X(), j);
        lds_sync();
        if (RED) {
            const Buf bv = buf(out.V, n * n);
            // ---- V = A'V - Y'X, Q_w_hat += X'X, L_t = -L^{-T} X, v += X'z
#pragma unroll
            for (int ti = 0; ti < NXT; ++ti) {
                const v4_t<T> acc = mulN<RX, NUT, SU>(L, zero4<T>(), S.Y(), ti, R2);
#pragma unroll
                for (int r = 0; r < SX; ++r) C.V[ti][r] = R1[ti][r] - acc[r];
                if (KEEP) store_tile<EX, SX>(L, bv, n, ti, j, n, C.V[ti]);
            }
            if (!QD) add_Q(L, R2);
            if constexpr (VEC) {
                double xz = 0.0;
#pragma unroll
                for (int ti = 0; ti < NUT; ++ti)
#pragma unroll
                    for (int r = 0; r < SU; ++r) xz += R2[ti][r] * S.z[16 * ti + L.row(r)];
                y.v += q_sum(xz);
            }
            if (KEEP && (VEC || out.Lt)) store_feedback<EX, RU, RX, NUT, SU>(L, S.G, R2, out.Lt, j, n, m);
        } else if (!VEC) {
            put_L<EX, NTV>(S, out.L, out.LT, m, (int)threadIdx.x - NTV);
        }
        if (!SM::OVER) commit();                 // A and B are dead since the factorization
        lds_sync();
        if (SM::OVER) {
            commit();
            lds_sync();
        }
    }
    if (QD) add_Q_late(Ln<T>());
}

// Backward pass over `count` >= 1 stages (local s = count-1 .. 0).  P_{count}
// in S.P (written by the caller; the pass starts with a barrier); RED: Alg. 4
// from V = I, Q_w_hat = 0, result in C.  wk: the data of stage count-1; pre(s, t0, t1)
// is called by the threads [t0, t1) before stage s and may read P_{s+1} from
// S.P; rec(s): where its factors go, with n and m their sizes (EX: n = 16 NXT
// and m = 16 NUT exactly).  The problem data have md <= m inputs (EXD: 16 NUT),
// the others being padding.
// VEC: with the right-hand side, y holding Psi_{count} on entry.  KEEP: the
// factors go to their records (else rec is not used).
// The three kinds of waves run loops of their own (with the same barriers), so
// that neither carries the other's registers.
template <bool RED, bool EX, bool EXD, bool VEC, bool KEEP = true, class T, int NXT, int NUT, int SX, int SU, class Pre,
          class RecOf>
__device__ __forceinline__ void pass(Smem<T, NXT, NUT, SX, SU> &S, Cols<T, NXT> &C, int n_, int m_, int md_, StageWalk wk, int count,
                                     int32_t *info, int inst, int stage_base, int fail_code, Pre pre, RecOf rec, Vec &y) {
    using SM = Smem<T, NXT, NUT, SX, SU>;
    constexpr int RX = SM::RX, RU = SM::RU, NTH = SM::NTH;
    static_assert(NUT <= NXT, "one column block of B per owner of A");
    static_assert(!VEC || !SM::OVER, "the vector lines read Y's place in LDS");
    const int n = EX ? RX : n_, m = EX ? RU : m_, md = EXD ? RU : md_;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    count = uni(count);
    if (tid == 0) S.bad = 0;
    if (wave() < NXT)
        loop_P<RED, EX, EXD, VEC, KEEP>(S, n, m, md, wk, count, info, inst, stage_base, fail_code, pre, rec, y);
    else if (wave() == 2 * NXT - 1)
        loop_V<true, RED, EX, EXD, VEC, KEEP>(S, C, n, m, md, wk, count, pre, rec, y);
    else if constexpr (NXT > 1)
        loop_V<false, RED, EX, EXD, VEC, KEEP>(S, C, n, m, md, wk, count, pre, rec, y);
    lds_sync();
    if constexpr (KEEP) {
        T *p = rec(0).P;
        if (p) copy_P(S, p, n);
    }
}

// Sum of v over the workgroup, in thread 0's wave (every thread calls).
template <class SM>
__device__ __forceinline__ double total(SM &S, double v) {
    v = sv::wave_sum(v);
    if (lane() == 0) S.red[wave()] = v;
    lds_sync();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < SM::NTH / 64; ++w) s += S.red[w];
    lds_sync();
    return s;
}

// V_0' and Q_w_hat (symmetric) from their owners' registers to row-major
// n x n places.
template <int NS, class T, int NXT, class U>
__device__ __forceinline__ void store_V_transposed(const Cols<T, NXT> &C, U *dst, int n) {
    const int j = wave() - NXT;
    if (j < 0) return;
    const Ln<T> L;
#pragma unroll
    for (int ti = 0; ti < NXT; ++ti)
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            const int i = 16 * ti + L.row(r), k = 16 * j + L.c;
            if (i < n && k < n) dst[(uint32_t)(k * n + i)] = (U)C.V[ti][r];
        }
}
template <int NS, class T, int NXT, class U>
__device__ __forceinline__ void store_Q(const Cols<T, NXT> &C, U *dst, int n) {
    const int j = wave() - NXT;
    if (j < 0) return;
    const Ln<T> L;
#pragma unroll
    for (int ti = 0; ti < NXT; ++ti) {
        if (ti < j) continue;
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            const int i = 16 * ti + L.row(r), k = 16 * j + L.c;
            if (i < n && k < n && i >= k) {
                dst[(uint32_t)(i * n + k)] = (U)C.Q[ti][r];
                dst[(uint32_t)(k * n + i)] = (U)C.Q[ti][r];
            }
        }
    }
}

// ------------------------------------------------------------ work tables
constexpr int SPIN_LIMIT = 1 << 26;

__device__ __forceinline__ LeafItem load_leaf_u(const LeafItem *tab, int i) {
    const LeafItem r = tab[i];
    LeafItem u;
    u.inst = uni(r.inst);
    u.t0 = uni(r.t0);
    u.len = uni(r.len);
    u.flags = uni(r.flags);
    u.slot = uni(r.slot);
    u.m1 = uni(r.m1);
    u.scratch = uni64(r.scratch);
    return u;
}
__device__ __forceinline__ TreeItem load_item_u(const TreeItem *tab, int i) {
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

// Waits (thread 0) until the items this one depends on carry the current
// epoch; a bounded wait records a failure instead of hanging.
__device__ __forceinline__ void wait_deps(const GroupArgs &g, const TreeItem &it) {
    if (threadIdx.x == 0) {
        for (int d = 0; d < it.dep_count; ++d) {
            int spins = 0;
            while (__hip_atomic_load(&g.flags[it.dep_first + d], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) !=
                   g.epoch) {
                __builtin_amdgcn_s_sleep(2);
                if (++spins > SPIN_LIMIT) {
                    record_failure(g.info, it.inst, 6, -2);
                    break;
                }
            }
        }
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

__device__ __forceinline__ void publish(const GroupArgs &g, int idx) {
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&g.flags[idx], g.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
}

}  // namespace cw
}  // namespace rs
