// Device-side building blocks of the parallel Riccati solver for gfx950:
// wave-uniform loads of descriptors and stage pointers, LDS-only barriers,
// the rank-revealing form of a reduced subproblem and failure reports.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rs_types.hpp"

namespace rs {

// ------------------------------------------------------------------ scalars
// Wave-uniform copy of an integer that is the same in every lane.  Loop
// bounds and branch conditions around barriers go through this so that the
// compiler sees uniform control flow and keeps every barrier in lock-step.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Instance excluded from this call (its descriptor carries PROB_SKIP).
__device__ __forceinline__ bool inst_skipped(const DevProb *probs, int inst) {
    return (uni(probs[inst].flags) & PROB_SKIP) != 0;
}

// Workgroup barrier that orders LDS only.  __syncthreads() also orders
// global memory, which makes every wave wait for all of its outstanding
// global loads and stores (the next stage's prefetch, the records just
// written) at each barrier; the passes only exchange data through LDS
// between their phases, so their barriers leave global traffic in flight.
__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Load through a global-address-space pointer.  Problem data are reached
// through pointers read from descriptors, which the compiler would access
// with flat instructions; flat loads also count as LDS operations, so every
// LDS wait before a barrier would then wait for them too.  Global loads
// leave the prefetched data in flight across the barriers.
template <class T>
__device__ __forceinline__ T gload(const T *p) {
    typedef const __attribute__((address_space(1))) T *gptr;
    return *(gptr)(p);
}

// ------------------------------------------------------------ stage data
// Pointers to one stage's data in global memory (FP64).  Leaves point into
// the caller's problem arrays; master stages point into slots, where
// Q_xw = 0, l_w = 0 and B = Q_w = Q_w_hat (Theorem 1 with the T-transform).
struct StageSrc {
    const double *Qx, *Qw, *Qxw, *A, *B, *a, *lx, *lw;
    double c;
    const double *cp;      // where c is read from (nullptr: c = 0), for prefetching passes
};

// Problem descriptor copied once into wave-uniform registers.  Reading it
// through the global-memory reference at every stage would re-issue a chain of
// dependent loads (the compiler cannot prove the descriptor unchanged across
// the kernel's own global stores).
__device__ __forceinline__ const double *uni_ptr(const double *q) {
    const uint64_t v = (uint64_t)q;
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)(v & 0xffffffffu)), hi = (uint32_t)uni((int)(uint32_t)(v >> 32));
    return (const double *)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)((uint64_t)v & 0xffffffffu)),
                   hi = (uint32_t)uni((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ DevProb load_prob(const DevProb *tab, int i) {
    const DevProb r = tab[i];
    DevProb u;
    u.Qx = uni_ptr(r.Qx);
    u.Qw = uni_ptr(r.Qw);
    u.Qxw = uni_ptr(r.Qxw);
    u.A = uni_ptr(r.A);
    u.B = uni_ptr(r.B);
    u.QxN = uni_ptr(r.QxN);
    u.x0 = uni_ptr(r.x0);
    u.a = uni_ptr(r.a);
    u.lx = uni_ptr(r.lx);
    u.lw = uni_ptr(r.lw);
    u.c = uni_ptr(r.c);
    u.lN = uni_ptr(r.lN);
    u.cN = uni_ptr(r.cN);
    u.x = const_cast<double *>(uni_ptr(r.x));
    u.w = const_cast<double *>(uni_ptr(r.w));
    u.lam = const_cast<double *>(uni_ptr(r.lam));
    u.obj = const_cast<double *>(uni_ptr(r.obj));
    u.sQx = uni64(r.sQx);
    u.sQw = uni64(r.sQw);
    u.sQxw = uni64(r.sQxw);
    u.sA = uni64(r.sA);
    u.sB = uni64(r.sB);
    u.sa = uni64(r.sa);
    u.slx = uni64(r.slx);
    u.slw = uni64(r.slw);
    u.sc = uni64(r.sc);
    u.nx = uni(r.nx);
    u.nu = uni(r.nu);
    u.N = uni(r.N);
    u.flags = uni(r.flags);
    return u;
}

__device__ __forceinline__ StageSrc prob_stage(const DevProb &p, int t) {
    StageSrc s;
    s.Qx = p.Qx + (int64_t)t * p.sQx;
    s.Qw = p.Qw + (int64_t)t * p.sQw;
    s.Qxw = p.Qxw ? p.Qxw + (int64_t)t * p.sQxw : nullptr;
    s.A = p.A + (int64_t)t * p.sA;
    s.B = p.B + (int64_t)t * p.sB;
    s.a = p.a ? p.a + (int64_t)t * p.sa : nullptr;
    s.lx = p.lx ? p.lx + (int64_t)t * p.slx : nullptr;
    s.lw = p.lw ? p.lw + (int64_t)t * p.slw : nullptr;
    s.cp = p.c ? p.c + (int64_t)t * p.sc : nullptr;
    s.c = s.cp ? gload(s.cp) : 0.0;
    return s;
}

// A master stage (Sec. 4.3, eq. red_mpc_problem) read from the M1 message
// in its slot: B = Q_w = Q_w_hat (the form of eq. Qh_Bh_alternative_def), or,
// with `ident` (an n x n identity), B = the rank-revealing factor written in
// the Q_w_hat place and Q_w = I (see rank_reveal).
__device__ __forceinline__ StageSrc slot_stage(const double *slot, int n, const double *ident) {
    const SlotLayout L{n};
    StageSrc s;
    s.Qx = slot + L.Qx();
    s.Qw = ident ? ident : slot + L.Qw();
    s.Qxw = nullptr;
    s.A = slot + L.A();
    s.B = slot + L.Qw();
    s.a = slot + L.a();
    s.lx = slot + L.lx();
    s.lw = nullptr;
    s.cp = slot + L.c();
    s.c = *s.cp;
    return s;
}

// The stages of a pass from its last one backwards: one subtraction per
// pointer and stage (formed from the stage index, the addresses cost some
// hundred scalar instructions a stage in every wave, on the chain of the small
// shapes).
struct StageWalk {
    StageSrc s;
    int64_t dQx, dQw, dQxw, dA, dB, da, dlx, dlw;     // elements per stage (0 for absent arrays)
    __device__ __forceinline__ void back() {
        s.Qx -= dQx;
        s.Qw -= dQw;
        s.Qxw -= dQxw;
        s.A -= dA;
        s.B -= dB;
        s.a -= da;
        s.lx -= dlx;
        s.lw -= dlw;
    }
};
__device__ __forceinline__ StageWalk prob_walk(const DevProb &p, int last) {
    return StageWalk{prob_stage(p, last), p.sQx, p.sQw, p.Qxw ? p.sQxw : 0, p.sA, p.sB, p.a ? p.sa : 0,
                     p.lx ? p.slx : 0, p.lw ? p.slw : 0};
}
__device__ __forceinline__ StageWalk slot_walk(const double *last, int n, const double *ident) {
    const int64_t d = SlotLayout{n}.size();
    return StageWalk{slot_stage(last, n, ident), d, ident ? 0 : d, 0, d, d, d, d, 0};
}

// Rank-revealing form of a reduced subproblem (Sec. 4.2, eqs. Bh_def and
// Gh_Hh_def).  The reduction (Alg. 4) leaves M = S Qbar^{-1} S' in `M`
// (n x n, row-major, positive semidefinite of rank n_uo = rank(S')).  This
// factors it by Cholesky with diagonal pivoting, M ~= B B' with column c of
// B the c-th pivot column, and stops once the largest remaining diagonal
// entry is at most n eps max_i M_ii (the usual stopping rule of pivoted
// Cholesky; the remaining Schur complement, positive semidefinite, is then
// below that bound entrywise).  Columns from the rank on are zero.
// A master stage with input matrix B and input weight I has
// B I^{-1} B' = M, as does the stage of the U_1 basis
// (B_hat Q_w_hat^{-1} B_hat' = S Qbar^{-1} S'); a master stage enters the
// master problem only through that product (minimising its input cost for a
// given state step), so both master problems have the same states and
// costates, and G = I + B'PB of the stage is positive definite even when
// N_s n_u < n_x or the subinterval's inputs leave state directions
// unreached.  Zero columns are inputs that move nothing and stay 0.
// B goes to out (and cache if given), row-major n x n; M is overwritten.
// Every thread of the workgroup calls; thread i owns row i
// (n <= blockDim.x, n <= 128, at most 16 wavefronts).
template <class T>
__device__ __attribute__((noinline)) void rank_reveal(T *M, int n, double eps, double *out, double *cache) {
    __shared__ double s_val[2][16];
    __shared__ int s_idx[2][16];
    const int tid = threadIdx.x, nw = (int)(blockDim.x + 63) >> 6, w = tid >> 6, l = tid & 63;
    const bool own = tid < n;
    uint64_t done0 = 0, done1 = 0;            // pivots taken (the same in every thread)
    auto done = [&](int i) { return (((i < 64) ? (done0 >> i) : (done1 >> (i - 64))) & 1) != 0; };
    auto put = [&](int i, int c, double v) {
        out[i * n + c] = v;
        if (cache) cache[i * n + c] = v;
    };
    double tol = 0.0;
    int c = 0;
    __syncthreads();
    for (; c < n; ++c) {
        // largest remaining diagonal entry; ties go to the smaller index
        double v = (own && !done(tid)) ? (double)M[tid * n + tid] : -1.0;
        int p = tid;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double v2 = __shfl_xor(v, o, 64);
            const int p2 = __shfl_xor(p, o, 64);
            if (v2 > v || (v2 == v && p2 < p)) {
                v = v2;
                p = p2;
            }
        }
        if (l == 0) {
            s_val[c & 1][w] = v;
            s_idx[c & 1][w] = p;
        }
        __syncthreads();
        v = s_val[c & 1][0];
        p = s_idx[c & 1][0];
        for (int u = 1; u < nw; ++u) {
            const double v2 = s_val[c & 1][u];
            const int p2 = s_idx[c & 1][u];
            if (v2 > v || (v2 == v && p2 < p)) {
                v = v2;
                p = p2;
            }
        }
        if (c == 0) tol = (double)n * eps * v;
        if (!(v > tol)) break;                // rank reached (also an all-zero M)
        const double s = 1.0 / sqrt(v);
        if (own) {
            if (done(tid)) {
                put(tid, c, 0.0);
            } else if (tid == p) {
                put(tid, c, v * s);
            } else {
                const double li = (double)M[tid * n + p] * s;
                put(tid, c, li);
                for (int k = 0; k < n; ++k)
                    if (k != p && !done(k)) M[tid * n + k] = (T)((double)M[tid * n + k] - li * ((double)M[p * n + k] * s));
            }
        }
        if (p < 64)
            done0 |= 1ull << p;
        else
            done1 |= 1ull << (p - 64);
        __syncthreads();
    }
    if (own)
        for (int cc = c; cc < n; ++cc) put(tid, cc, 0.0);
}

// The same factorization for n <= NM <= 64 (NM known at compile time): four
// threads hold a row of the remaining Schur complement in registers, in 64
// bits whatever T, a quarter of it each; the pivot column goes through a short
// LDS vector, and M is only read.  A dependent chain of n pivots; 32 states of
// rank 32 take 34 us (one thread a row 68 us, and so many registers that other
// workgroups find no room; rows in LDS at pitch n, where they collide, 150 us).
// Out of line, it takes no register from the stage loops.  At least 4 NM
// threads.
template <int NM, class T>
__device__ __attribute__((noinline)) void rank_reveal_rows(const T *M, int n, double eps, double *out,
                                                           double *cache) {
    static_assert(NM % 16 == 0 && NM <= 64, "whole wavefronts of rows");
    constexpr int C = NM / 4, NW = NM / 16;   // columns of a thread, wavefronts that hold rows
    __shared__ double s_val[NW], s_l[NM];
    __shared__ int s_idx[NW];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, i = tid % NM, q = tid / NM;
    const bool own = w < NW && i < n;
    auto put = [&](int c, double v) {
        out[i * n + c] = v;
        if (cache) cache[i * n + c] = v;
    };
    double r[C];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C; ++k) r[k] = (own && C * q + k < n) ? (double)M[i * n + C * q + k] : 0.0;
    // element k of this thread's quarter
    auto pick = [&](int k) {
        double d = 0.0;
#pragma unroll
        for (int e = 0; e < C; ++e) d = (e == k) ? r[e] : d;
        return d;
    };
    uint64_t done = 0;                        // pivots taken (the same in every thread)
    double tol = 0.0;
    int c = 0;
    for (; c < n; ++c) {
        const bool live = own && !((done >> i) & 1);
        double v = (live && q == i / C) ? pick(i % C) : -1.0;
        int p = i;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double v2 = __shfl_xor(v, o, 64);
            const int p2 = __shfl_xor(p, o, 64);
            if (v2 > v || (v2 == v && p2 < p)) {
                v = v2;
                p = p2;
            }
        }
        if (l == 0 && w < NW) {
            s_val[w] = v;
            s_idx[w] = p;
        }
        __syncthreads();
        v = s_val[0];
        p = s_idx[0];
#pragma unroll
        for (int u = 1; u < NW; ++u) {
            const double v2 = s_val[u];
            const int p2 = s_idx[u];
            if (v2 > v || (v2 == v && p2 < p)) {
                v = v2;
                p = p2;
            }
        }
        if (c == 0) tol = (double)n * eps * v;
        if (!(v > tol)) break;                // rank reached (also an all-zero M)
        const double s = 1.0 / sqrt(v);
        if (w < NW && q == p / C) {
            const double li = (live && i != p) ? pick(p % C) * s : 0.0;
            if (own) put(c, !live ? 0.0 : (i == p ? v * s : li));
            s_l[i] = li;                      // 0 for the pivot row and rows already taken
        }
        __syncthreads();
        if (live && i != p) {
            const double li = s_l[i];
#pragma unroll
            for (int k = 0; k < C; ++k) r[k] -= li * s_l[C * q + k];
        }
        done |= 1ull << p;
    }
    if (own && q == 0)
        for (int cc = c; cc < n; ++cc) put(cc, 0.0);
}

template <class T>
__device__ __forceinline__ constexpr double unit_roundoff() {
    return sizeof(T) == 4 ? 1.1920928955078125e-07 : 2.220446049250313e-16;
}

// First failure of an instance wins; master-level failures carry stage -1.
__device__ __forceinline__ void record_failure(int32_t *info, int inst, int code, int stage) {
    if (stage < 0) stage = -1;
    if (info) {
        if (atomicCAS(&info[2 * inst], 0, code) == 0) info[2 * inst + 1] = stage;
    }
}

}  // namespace rs
