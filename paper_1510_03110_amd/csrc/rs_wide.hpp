// Per-stage Riccati recursion for 64 < n_x <= 128 on column owners (matrix
// lines of Alg. 1 and Alg. 4, FP64 or FP32), one workgroup of eight wavefronts
// per subproblem.
//
// What bounds it: a stage of 128 states and 64 inputs is 3000 16 x 16 x 16
// products, 81 us on the matrix cores of one CU.  With every product read from
// and written to a workspace (one product after another) a stage moved 4.3 MB;
// the workspaces of 256 units exceed every cache, so that traffic, not the
// matrix cores, set the time (366 us a stage with 256 units at work; 187 us in
// this form).  Here wave j owns column block j of W, F, H', Y, K, P and of A'V,
// B'V, X, L_t, V, Q_w_hat, which pass from one product to the next in its
// registers (the layout in which a product leaves is the one in which it enters
// the next as right-hand operand), and only left-hand operands come through
// LDS: panels of 16 rows of P, A, B, L, Y and X, shared by the eight waves, the
// next one in flight while one is multiplied.  P and V are kept in the records
// that the solve needs anyway.
#pragma once
#include "rs_col.hpp"

namespace rs {
namespace wd {

using cw::BEYOND;
using cw::Buf;
using cw::buf;
using cw::buf_get;
using cw::buf_st;
using cw::Ln;
using mf::MT;
using mf::v4_t;
using mf::wave;
using mf::zero4;

constexpr int NT = 8, NTHR = 64 * NT;            // column blocks of 128, threads
// Row pitch of a panel: rows of 144 elements, so that the two rows of a
// half-wave's operand read fall on different banks.
constexpr int PITCH = 16 * NT + 16, PANEL = 16 * PITCH;
// LDS elements: two pairs of panels, or G while it is factored.
template <int NUT>
constexpr int lds_elems() {
    return 4 * PANEL > 256 * NUT * NUT ? 4 * PANEL : 256 * NUT * NUT;
}

// Keeps the operand reads of a product, and the accesses of a tile, in their
// place: moved up in numbers they spill the column blocks.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

// A matrix whose rows are streamed: `rows` x `cols`, row length ld.
template <class U>
struct Mat {
    const U *p;
    int rows, cols, ld;
};

// body(kt, P0, P1) for the panels kt of 16 rows of M0 and M1 (same number of
// rows; M1.p null: none), from LDS.  pre(kt) issues what body(kt) wants loaded
// and adv() takes it over from there once it has arrived.  The loop is rolled:
// unrolled, with its register arrays indexed by kt, a stage is 200 KB of code,
// and a panel spent as long on instruction fetches as on its products.
template <class T, class U0, class U1, class Pre, class Adv, class Body>
__device__ __forceinline__ void sweep(T *sm, Mat<U0> M0, Mat<U1> M1, bool two, Pre pre, Adv adv, Body body) {
    constexpr int E = 16 * 16 * NT / NTHR;
    const Buf b0 = buf(M0.p, (M0.rows - 1) * M0.ld + M0.cols), b1 = buf(M1.p, (M1.rows - 1) * M1.ld + M1.cols);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int col = tid & 127, row = tid >> 7;
    U0 r0[E];
    U1 r1[E];
    auto fetch = [&](int kt) {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int k = 16 * kt + row + 4 * u;
            r0[u] = buf_get<U0>(b0, k < M0.rows && col < M0.cols ? (uint32_t)sizeof(U0) * (uint32_t)(k * M0.ld + col) : BEYOND);
        }
        if (two)
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int k = 16 * kt + row + 4 * u;
                r1[u] = buf_get<U1>(b1, k < M1.rows && col < M1.cols ? (uint32_t)sizeof(U1) * (uint32_t)(k * M1.ld + col) : BEYOND);
            }
        pre(kt);
    };
    const int nk = (M0.rows + 15) >> 4;
    fetch(0);
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
        T *P0 = sm + 2 * PANEL * (kt & 1), *P1 = P0 + PANEL;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            P0[(row + 4 * u) * PITCH + col] = (T)r0[u];
            if (two) P1[(row + 4 * u) * PITCH + col] = (T)r1[u];
        }
        adv();
        lds_sync();           // the panel is complete, and the other pair is free
        if (kt + 1 < nk) fetch(kt + 1);
        body(kt, P0, P1);
        fence();
    }
    lds_sync();
}

// The first of N column tiles, which goes to the end.
template <int N, class V>
__device__ __forceinline__ V rotate(V (&v)[N]) {
    const V f = v[0];
#pragma unroll
    for (int t = 0; t + 1 < N; ++t) v[t] = v[t + 1];
    v[N - 1] = f;
    return f;
}

// acc[t] += (tile t0 + t of the panel)' b for lo <= t < hi (uniform).  The
// operands of the next tile are read before this one is multiplied (in the
// order of the source, the reads of a tile waited behind the products of its
// own first half: the matrix cores idled for twice the LDS latency a tile).
template <int N, class T>
__device__ __forceinline__ void mul(const Ln<T> &L, v4_t<T> (&acc)[N], const T *P, int t0, v4_t<T> b, int lo, int hi) {
    const T *q = P + L.row(0) * PITCH + 16 * t0 + L.c;
    T a[2][4];
    auto read = [&](int t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) a[t & 1][r] = q[(L.row(r) - L.row(0)) * PITCH + 16 * t];
    };
    read(0);
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if (t + 1 < N) read(t + 1);
        fence();
        if (t >= lo && t < hi) {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t] = MT<T>::mfma(a[t & 1][r], b[r], acc[t]);
        }
        fence();
    }
}
template <class T>
__device__ __forceinline__ v4_t<T> neg(v4_t<T> v) {
    return v4_t<T>{-v[0], -v[1], -v[2], -v[3]};
}

// Tile (ti, tj) of M (n1 x n2, row length ld) in the result layout, zeros
// outside; TR: the array holds the transpose; ONE: identity outside.
template <bool TR, bool ONE, class T, class U>
__device__ __forceinline__ v4_t<T> tile(const Ln<T> &L, const U *M, int ld, int ti, int tj, int n1, int n2, bool on = true) {
    const Buf b = buf(M, TR ? (n2 - 1) * ld + n1 : (n1 - 1) * ld + n2, on);
    v4_t<T> v;
    const int j = 16 * tj + L.c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + L.row(r);
        v[r] = (T)buf_get<U>(b, i < n1 && j < n2 ? (uint32_t)sizeof(U) * (uint32_t)(TR ? j * ld + i : i * ld + j) : BEYOND);
        if (ONE) v[r] = (i == j && i >= n1) ? T(1) : v[r];
    }
    return v;
}
// Result tile (ti, tj) to M (n1 x n2, row length ld).
template <class T>
__device__ __forceinline__ void store(const Ln<T> &L, Buf b, int ld, int ti, int tj, int n1, int n2, v4_t<T> v) {
    const int j = 16 * tj + L.c;
    fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + L.row(r);
        buf_st(b, i < n1 && j < n2 ? (uint32_t)sizeof(T) * (uint32_t)(i * ld + j) : BEYOND, v[r]);
    }
}
// Lower tile of a symmetric result, and (both) its mirror image.
template <class T>
__device__ __forceinline__ void store_sym(const Ln<T> &L, Buf b, int n, int ti, int tj, v4_t<T> v, bool both) {
    const int j = 16 * tj + L.c;
    fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + L.row(r);
        const bool in = i < n && i >= j;
        buf_st(b, in ? (uint32_t)sizeof(T) * (uint32_t)(i * n + j) : BEYOND, v[r]);
        if (both) buf_st(b, in ? (uint32_t)sizeof(T) * (uint32_t)(j * n + i) : BEYOND, v[r]);
    }
}

// Places of a subproblem in the unit's workspace: P and V hold P_{count} and V
// on entry and are set to where the pass left P_0 and V_0; Q (n x n; lower
// part while the pass runs), Y and X (m x n).
template <class T>
struct Work {
    T *P, *V, *Q, *Y, *X;
};
// Where the factors of a stage go (row-major; P and V null: not kept, Lt null:
// not formed).
template <class T>
struct Rec {
    T *P, *K, *V, *Lt, *L, *LT;
};

// One stage.  src: its data; chol(G, m, L, LT): factors the m x m matrix in
// LDS at pitch 16 NUT, writes L^{-1} and L^{-T}, ends with a workgroup barrier.
template <bool RED, int NUT, class T, class Chol>
__device__ __forceinline__ void stage(T *sm, Work<T> &S, const StageSrc &src, int n, int m, const Rec<T> &out,
                                      bool last, Chol chol) {
    constexpr int PU = 16 * NUT, WT = NUT == NT ? NT : NT * NUT / NT;      // row tiles of W_B per wave
    const int j = wave(), nt = (n + 15) >> 4, mt = (m + 15) >> 4;
    const Mat<T> none{nullptr, 1, 0, 0};
    const Mat<double> A{src.A, n, n, n}, B{src.B, n, m, m};
    const Mat<T> P{S.P, n, n, n};
    auto no_pre = [](int) {};
    auto no_adv = [] {};
    // ---- W = P A and, for G = Qw + B'PB (column block c by NT / NUT waves),
    // each wave's WT row tiles of W_B = P B: one sweep over P where the
    // registers hold both
    constexpr bool ONE = NUT < NT;
    v4_t<T> w[NT];
    {
        const Ln<T> L;
        const int c = j % NUT, h = j / NUT;
        v4_t<T> wb[WT], g[NUT], a, an, b, bn;
#pragma unroll
        for (int t = 0; t < WT; ++t) wb[t] = zero4<T>();
        if (ONE)
#pragma unroll
            for (int t = 0; t < NT; ++t) w[t] = zero4<T>();
        sweep(sm, P, none, false,
              [&](int kt) {
                  bn = tile<false, false, T>(L, src.B, m, kt, c, n, m);
                  if (ONE) an = tile<false, false, T>(L, src.A, n, kt, j, n, n);
              },
              [&] {
                  b = bn;
                  a = an;
              },
              [&](int, const T *P0, const T *) {
                  mul(L, wb, P0, h * WT, b, 0, c < mt ? nt - h * WT : 0);
                  if (ONE) mul(L, w, P0, 0, a, 0, nt);
              });
#pragma unroll
        for (int t = 0; t < NUT; ++t) g[t] = tile<false, true, T>(L, src.Qw, m, t, c, m, m, h == 0 && t >= c);
        if (h != 0)
#pragma unroll
            for (int t = 0; t < NUT; ++t) g[t] = zero4<T>();
        sweep(sm, B, none, false, no_pre, no_adv, [&](int kt, const T *P0, const T *) {
            if (kt / WT == h) {
                const v4_t<T> b = rotate(wb);
                mul(L, g, P0, 0, b, c, mt);
            }
        });
        if (h == 0)
#pragma unroll
            for (int t = 0; t < NUT; ++t)
                if (t >= c) cw::put_sym<PU, 4>(L, sm, t, c, g[t]);
        lds_sync();
        if constexpr (NUT < NT) {
            static_assert(2 * NUT == NT, "two waves per column block of G");
            if (h == 1)
#pragma unroll
                for (int t = 0; t < NUT; ++t)
                    if (t >= c) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) g[t][r] += sm[cw::at<PU>(16 * t + L.row(r), 16 * c + L.c)];
                        cw::put_sym<PU, 4>(L, sm, t, c, g[t]);
                    }
            lds_sync();
        }
        chol(sm, m, out.L, out.LT);
    }
    const Mat<T> LI{out.L, m, m, m}, LT{out.LT, m, m, m}, Y{S.Y, m, n, n}, X{S.X, m, n, n};
    // k -= L^{-T} y, in a sweep of its own
    auto feedback = [&](v4_t<T>(&k)[NUT], v4_t<T>(&y)[NUT], const Ln<T> &L) {
        sweep(sm, LI, none, false, no_pre, no_adv, [&](int kt, const T *P0, const T *) {
            const v4_t<T> b = neg<T>(rotate(y));
            mul(L, k, P0, 0, b, 0, kt + 1);
        });
    };
    {
        const Ln<T> L;
        v4_t<T> F[NT], H[NUT];
        {
            if constexpr (!ONE) {
                v4_t<T> a, an;
#pragma unroll
                for (int t = 0; t < NT; ++t) w[t] = zero4<T>();
                sweep(sm, P, none, false, [&](int kt) { an = tile<false, false, T>(L, src.A, n, kt, j, n, n); },
                      [&] { a = an; },
                      [&](int, const T *P0, const T *) {
                          mul(L, w, P0, 0, a, 0, nt);
                      });
            }
            // ---- F = Qx + A'W (lower tiles), H' = Qxw' + B'W
#pragma unroll
            for (int t = 0; t < NT; ++t) F[t] = tile<false, false, T>(L, src.Qx, n, t, j, n, n, t >= j);
#pragma unroll
            for (int t = 0; t < NUT; ++t) H[t] = tile<true, false, T>(L, src.Qxw, m, t, j, m, n);
            sweep(sm, A, B, true, no_pre, no_adv, [&](int, const T *P0, const T *P1) {
                const v4_t<T> b = rotate(w);
                mul(L, H, P1, 0, b, 0, mt);
                mul(L, F, P0, 0, b, j, nt);
            });
        }
        // ---- Y = L^{-1} H'
        v4_t<T> y[NUT];
#pragma unroll
        for (int t = 0; t < NUT; ++t) y[t] = zero4<T>();
        sweep(sm, LT, none, false, no_pre, no_adv, [&](int kt, const T *P0, const T *) {
            const v4_t<T> b = rotate(H);
            mul(L, y, P0, 0, b, kt, mt);
        });
        const Buf by = buf(S.Y, m * n);
#pragma unroll
        for (int t = 0; t < NUT; ++t) store(L, by, n, t, j, m, n, y[t]);
        __syncthreads();
        // ---- P = F - Y'Y, K = -L^{-T} Y
        v4_t<T> k[NUT];
        if (ONE)
#pragma unroll
            for (int t = 0; t < NUT; ++t) k[t] = zero4<T>();
        sweep(sm, Y, LI, ONE, no_pre, no_adv, [&](int kt, const T *P0, const T *P1) {
            const v4_t<T> b = neg<T>(rotate(y));
            if (ONE) mul(L, k, P1, 0, b, 0, kt + 1);
            mul(L, F, P0, 0, b, j, nt);
        });
        T *dst = out.P ? out.P : S.P;
        const Buf bp = buf(dst, n * n), bk = buf(out.K, m * n);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t >= j) store_sym(L, bp, n, t, j, F[t], true);
        if constexpr (!ONE) {
            for (int t = mt; t < NUT; ++t) rotate(y);      // back in order
#pragma unroll
            for (int t = 0; t < NUT; ++t) k[t] = zero4<T>();
            feedback(k, y, L);
        }
#pragma unroll
        for (int t = 0; t < NUT; ++t) store(L, bk, n, t, j, m, n, k[t]);
        S.P = dst;
    }
    if constexpr (RED) {
        const Ln<T> L;
        v4_t<T> av[NT], x[NUT];
        {
            v4_t<T> bv[NUT], v, vn;
#pragma unroll
            for (int t = 0; t < NT; ++t) av[t] = zero4<T>();
#pragma unroll
            for (int t = 0; t < NUT; ++t) bv[t] = zero4<T>();
            sweep(sm, A, B, true, [&](int kt) { vn = tile<false, false, T>(L, S.V, n, kt, j, n, n); }, [&] { v = vn; },
                  [&](int, const T *P0, const T *P1) {
                      mul(L, bv, P1, 0, v, 0, mt);
                      mul(L, av, P0, 0, v, 0, nt);
                  });
            // ---- X = L^{-1} B'V
#pragma unroll
            for (int t = 0; t < NUT; ++t) x[t] = zero4<T>();
            sweep(sm, LT, none, false, no_pre, no_adv, [&](int kt, const T *P0, const T *) {
                const v4_t<T> b = rotate(bv);
                mul(L, x, P0, 0, b, kt, mt);
            });
        }
        const Buf bx = buf(S.X, m * n);
#pragma unroll
        for (int t = 0; t < NUT; ++t) store(L, bx, n, t, j, m, n, x[t]);
        __syncthreads();
        // ---- V = A'V - Y'X, L_t = -L^{-T} X
        {
            v4_t<T> l[NUT];
            if (ONE)
#pragma unroll
                for (int t = 0; t < NUT; ++t) l[t] = zero4<T>();
            sweep(sm, Y, LI, ONE && out.Lt, no_pre, no_adv, [&](int kt, const T *P0, const T *P1) {
                const v4_t<T> b = neg<T>(rotate(x));
                if (ONE && out.Lt) mul(L, l, P1, 0, b, 0, kt + 1);
                mul(L, av, P0, 0, b, 0, nt);
            });
            T *dst = out.V ? out.V : S.V;
            const Buf bv = buf(dst, n * n);
#pragma unroll
            for (int t = 0; t < NT; ++t) store(L, bv, n, t, j, n, n, av[t]);
            S.V = dst;
            for (int t = mt; t < NUT; ++t) rotate(x);      // back in order
            if (!ONE && out.Lt) {
#pragma unroll
                for (int t = 0; t < NUT; ++t) l[t] = zero4<T>();
                feedback(l, x, L);
                for (int t = mt; t < NUT; ++t) rotate(x);
            }
            const Buf bl = buf(out.Lt, m * n);
            if (out.Lt)
#pragma unroll
                for (int t = 0; t < NUT; ++t) store(L, bl, n, t, j, m, n, l[t]);
        }
        // ---- Q_w_hat += X'X (lower tiles; the whole matrix after the last):
        // the product by itself, added once (see add_Q in rs_col.hpp)
#pragma unroll
        for (int t = 0; t < NT; ++t) av[t] = zero4<T>();
        sweep(sm, X, none, false, no_pre, no_adv, [&](int, const T *P0, const T *) {
            const v4_t<T> b = rotate(x);
            mul(L, av, P0, 0, b, j, nt);
        });
#pragma unroll
        for (int t = 0; t < NT; ++t) av[t] += tile<false, false, T>(L, S.Q, n, t, j, n, n, t >= j);
        const Buf bq = buf(S.Q, n * n);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t >= j) store_sym(L, bq, n, t, j, av[t], last);
    }
    __syncthreads();
}

}  // namespace wd
}  // namespace rs
