// Host-visible launch interface between the C ABI and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rs_types.hpp"

namespace rs {

// Leaf scratch of the fused solve per stage as rs_batch_solve_noalloc counts
// it: below the full tiles without the room for V and L_t, which those shapes
// do not use, so that the plans it takes are the same with and without it.
constexpr int scratch_counted(int nx, int nu) {
    return (nx % 16 == 0 && nu % 16 == 0) ? leaf_rec_len(nx, nu) : nu * nx + nu + nx * nx + nx;
}

typedef hipError_t (*Launcher)(const GroupArgs &, int grid, hipStream_t);

// Kernel kinds, also the index of the per-kind timers of a plan.
enum KernelKind {
    KK_INIT = 0,
    KK_LEAF_UP = 1, KK_TREE = 2, KK_LEAF_DOWN = 3,          // fused solve
    KK_F_LEAF_UP = 4, KK_F_TREE = 5, KK_F_LEAF_DOWN = 6,    // rs_factor
    KK_S_LEAF_UP = 7, KK_S_TREE = 8, KK_S_LEAF_DOWN = 9,    // rs_solve
    KK_RESIDUAL = 10, KK_UPDATE = 11, KK_CHECK = 12,        // mixed-precision refinement
    KK_REPORT = 13,                                         // K norm of the report
    KK_COUNT = 16
};

struct ShapeEntry {
    int nx, nu;
    bool large;              // no fused kernels: the FP64 solve runs on the stored factorization
    bool lb;                 // the stored factorization uses the large-block kernels (global workspace)
    Launcher fp64[3];        // fused: leaf up, tree, leaf down
    Launcher factor[3][3];   // stored factorization [fp64, fp32, bf16-product leaves][pass] (nullptr: none)
    Launcher vsolve[2][3];   // right-hand-side passes on the stored factorization
    Launcher refine[2];      // FP64 residual, refinement update
    int scratch_per_stage;
};

Launcher fused_solve(int nx, int nu, int which);         // fused FP64 solve (rs_fused.hip), n_x <= 32
hipError_t fused_leaf_forward(const GroupArgs &g, hipStream_t st);   // its leaf solve on the leaf records
Launcher mfma_factor(int nx, int nu, int which, bool fp32);
Launcher vector_solve(int nx, int nu, int which, bool fp32);
Launcher refine_kernel(int nx, int nu, int which);       // 0 residual, 1 update
// mode 0 also clears active[0 .. nactive); mode 1 counts the instances still
// iterating into *active.
hipError_t launch_refine_check(const InstInfo *tab, int count, const double *part, double *stats, int32_t *conv,
                               int32_t *info, const DevProb *probs, int mode, double tol, int32_t *active,
                               int nactive, int with_knorm, hipStream_t st);
// Finite-input check (RS_PLAN_CHECK_INPUTS): per leaf, the smallest
// offending place per instance into first[] (preset to INT32_MAX), then
// RS_ERR_ARG and the place in the status words.
hipError_t launch_scan(const GroupArgs &g, int32_t *first, hipStream_t st);
hipError_t launch_scan_mark(int count, const int32_t *first, int32_t *info, hipStream_t st);
// KKT-matrix infinity norm of each leaf's rows (PART_KN of the leaf parts).
hipError_t launch_knorm(const GroupArgs &g, hipStream_t st);
// rs_info records (40 bytes each) from the statistics (or nullptr) and the
// status words.
hipError_t launch_report(int count, const double *stats, const int32_t *info, int refined, void *out,
                         hipStream_t st);

// Large-block family (any n_x, n_u up to 128): stored factorization with a
// per-workgroup workspace of large_unit_bytes.
constexpr int LB_LEAF_UNITS = 2048, LB_TREE_UNITS = 256;
bool large_shape(int nx, int nu);
size_t large_unit_bytes(int nx, int nu);
Launcher large_factor(int which, bool fp32, bool bf16 = false);
Launcher large_vector(int which, bool fp32);
Launcher large_refine(int which);
// Stored factorization on the column-owner engine (rs_mid.hip): n_x <= 64 and
// no more 16-wide tiles of inputs than of states; the larger shapes, and those
// with more inputs than states, need the global-memory workspace.
inline bool mid_shape(int nx, int nu) { return nx <= 64 && (nu + 15) / 16 <= (nx + 15) / 16; }
hipError_t mid_leaf_f64(const GroupArgs &g, bool down, hipStream_t st);
hipError_t mid_leaf_f32(const GroupArgs &g, bool down, hipStream_t st);
hipError_t mid_tree(const GroupArgs &g, int grid, hipStream_t st);      // n_x <= 64
// Right-hand-side sweeps with register prefetch (rs_vsweep.hip), n_x, n_u <= 64
// (the tree: superposition down pass only).
inline bool sweep_shape(int nx, int nu) { return nx <= 64 && nu <= 64; }
hipError_t sweep_leaf(const GroupArgs &g, bool fp32, bool down, hipStream_t st);
hipError_t sweep_tree(const GroupArgs &g, int grid, hipStream_t st);

const ShapeEntry *find_shape(int nx, int nu);

// Device scratch of rs_batch_solve_noalloc (rs_static.hip): its device
// address on the current device (taken once per device), and its size (twice
// what the call counts: a plan's leaf scratch is less than twice its counted
// one, see scratch_counted).
constexpr size_t STATIC_SCRATCH_BYTES = size_t(128) << 20;
void *static_scratch(size_t *bytes);
hipError_t launch_init(int32_t *info, int count, int32_t *queues, int nq, hipStream_t st);
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st);
// padded copies of the inputs of npad instances (back = false), or their w
// copied back to the caller (back = true)
hipError_t launch_pad(const PadArgs *args, int npad, bool back, hipStream_t st);

}  // namespace rs
