// Small common kernels and the table of shapes.
//   k_init       clears per-instance status words and the tree work queues
//   k_fill_i32   fills the tree's completion flags
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>

#include "rs_launch.hpp"

namespace rs {

__global__ void k_init(int32_t *info, int count, int32_t *queues, int nq) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) {
        info[2 * i] = 0;
        info[2 * i + 1] = -1;
    }
    if (i < nq) queues[i] = 0;
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------- launchers
hipError_t launch_init(int32_t *info, int count, int32_t *queues, int nq, hipStream_t st) {
    const int n = count > nq ? count : nq;
    hipLaunchKernelGGL(k_init, dim3((n + 255) / 256), dim3(256), 0, st, info, count, queues, nq);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

const ShapeEntry *find_shape(int nx, int nu) {
    static ShapeEntry table[64];
    static int n = 0;
    static bool init = false;
    if (!init) {
        auto add = [&](int a, int b) {
            ShapeEntry e;
            e.nx = a;
            e.nu = b;
            e.large = false;
            e.lb = false;
            for (int k = 0; k < 3; ++k) e.fp64[k] = fused_solve(a, b, k);
            for (int f = 0; f < 2; ++f)
                for (int k = 0; k < 3; ++k) {
                    e.factor[f][k] = mfma_factor(a, b, k, f == 1);
                    e.vsolve[f][k] = vector_solve(a, b, k, f == 1);
                }
            for (int k = 0; k < 3; ++k) e.factor[2][k] = nullptr;
            e.refine[0] = refine_kernel(a, b, 0);
            e.refine[1] = refine_kernel(a, b, 1);
            // no full-tile form of the stored factorization: the run-time
            // sized kernels serve it (and mixed precision)
            e.lb = !e.factor[0][0] && large_shape(a, b);
            if (e.lb) {
                for (int f = 0; f < 2; ++f)
                    for (int k = 0; k < 3; ++k) {
                        e.factor[f][k] = large_factor(k, f == 1);
                        e.vsolve[f][k] = large_vector(k, f == 1);
                    }
                for (int k = 0; k < 3; ++k) e.factor[2][k] = large_factor(k, true, true);
                e.refine[0] = large_refine(0);
                e.refine[1] = large_refine(1);
            }
            e.scratch_per_stage = leaf_rec_len(a, b);
            table[n++] = e;
        };
        // the shapes with a fused solve, the sizes of the workloads; every other
        // one runs on the stored factorization (the fused kernels' run-time sizes
        // would take any n_u <= n_x <= 32; not measured beyond this list)
        const int shapes[][2] = {{1, 1}, {2, 1}, {2, 2}, {3, 2}, {4, 2}, {4, 4}, {6, 3}, {8, 4}, {16, 8}, {20, 10},
                                 {16, 16}, {32, 16}, {32, 32}};
        for (const auto &m : shapes) add(m[0], m[1]);
        init = true;
    }
    for (int i = 0; i < n; ++i)
        if (table[i].nx == nx && table[i].nu == nu) return &table[i];
    // large-block family: any other shape up to 128 (entries made on first use)
    if (!large_shape(nx, nu)) return nullptr;
    static std::mutex mu;
    static std::map<std::pair<int, int>, ShapeEntry> large;
    std::lock_guard<std::mutex> lock(mu);
    auto it = large.find({nx, nu});
    if (it != large.end()) return &it->second;
    ShapeEntry e;
    e.nx = nx;
    e.nu = nu;
    e.large = true;
    e.lb = true;
    for (int k = 0; k < 3; ++k) {
        e.fp64[k] = nullptr;
        for (int f = 0; f < 2; ++f) {
            e.factor[f][k] = large_factor(k, f == 1);
            e.vsolve[f][k] = large_vector(k, f == 1);
        }
        e.factor[2][k] = large_factor(k, true, true);
    }
    e.refine[0] = large_refine(0);
    e.refine[1] = large_refine(1);
    e.scratch_per_stage = 1;      // leaf stage index = scratch offset
    return &large.emplace(std::make_pair(nx, nu), e).first->second;
}

}  // namespace rs
