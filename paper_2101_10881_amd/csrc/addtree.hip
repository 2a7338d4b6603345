// addtree.hip -- the addition stage: every output's pairwise tree (Section 5,
// the addition kernel) in one or two launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/mdpe.h"
#include "md.hpp"
#include "plan.hpp"
#include "runtime.hpp"

namespace mdpe {

constexpr int kAddThreads = 256;
constexpr int kAddCoefs = 16;                        // coefficients of a workgroup
constexpr int kAddRuns = kAddThreads / kAddCoefs;    // runs of leaves of a workgroup

// A workgroup sums parts blockIdx.x, + gridDim.x, .. of a pass at the 16
// coefficients of blockIdx.y: thread (run, c) the subtree of its run of E
// leaves in registers, then the runs' subtrees meet in LDS, level by level in
// the tree's own pairs (later element + earlier one, an odd one carried), so
// every sum is that of the level-by-level additions.  Bound by the latency of
// a pass at these sizes: one launch per level (each ~4.7 us, bound by its
// boundary) took 35-77 us for 8 to 13 levels, a pass takes 4 to 13 us (38 at ten
// doubles, d = 152 and 1821 leaves).  Each leaf is read once and each part
// written once, where a launch per level reads two series and writes one per
// addition.
template <int M, bool CX>
__global__ __launch_bounds__(kAddThreads) void add_tree_kernel(double *__restrict__ A, const int *__restrict__ leaves,
                                                               const AddChunk *__restrict__ chunks, long parts,
                                                               double *__restrict__ value, double *__restrict__ grad,
                                                               int n, int d) {
    constexpr int W = kCoef<M, CX>;
    constexpr int E = add_run(W);
    __shared__ double part[W][kAddThreads];
    const int tid = (int)threadIdx.x;
    const int c = (int)blockIdx.y * kAddCoefs + tid % kAddCoefs;
    const int run = tid / kAddCoefs, f = run * E;
    const long S = (long)(d + 1) * W, at = (long)min(c, d) * W;
    for (long b = blockIdx.x; b < parts; b += gridDim.x) {
        const AddChunk ch = chunks[b];
        double v[E][W];
        if (f < ch.count) {
            long off[E];
#pragma unroll
            for (int e = 0; e < E; ++e) off[e] = (long)leaves[ch.first + min(f + e, ch.count - 1)] * S + at;
#pragma unroll
            for (int e = 0; e < E; ++e)
#pragma unroll
                for (int l = 0; l < W; ++l) v[e][l] = A[off[e] + l];
        }
#pragma unroll
        for (int s = 1; s < E; s *= 2)
#pragma unroll
            for (int p = 0; p < E; p += 2 * s)
                if (f + p + s < ch.count) {
                    double z[W];
                    coef_add<M, CX>(v[p + s], v[p], z);
#pragma unroll
                    for (int l = 0; l < W; ++l) v[p][l] = z[l];
                }
        const int runs = (ch.count + E - 1) / E;
        for (int s = 1; s < runs; s *= 2) {
            if (run % (2 * s) == s && run < runs) {
#pragma unroll
                for (int l = 0; l < W; ++l) part[l][tid] = v[0][l];
            }
            __syncthreads();
            if (run % (2 * s) == 0 && run + s < runs) {
                double later[W], z[W];
#pragma unroll
                for (int l = 0; l < W; ++l) later[l] = part[l][tid + s * kAddCoefs];
                coef_add<M, CX>(later, v[0], z);
#pragma unroll
                for (int l = 0; l < W; ++l) v[0][l] = z[l];
            }
        }
        if (run == 0 && c <= d) {
            if (ch.out < 0) {
                double *to = A + (long)leaves[ch.first + ch.count - 1] * S + at;
#pragma unroll
                for (int l = 0; l < W; ++l) to[l] = v[0][l];
            } else {
                const int d1 = d + 1;
#pragma unroll
                for (int l = 0; l < W; ++l) {
                    const double x = ch.count > 0 ? v[0][l] : 0.0;  // an absent variable's derivative
                    if (ch.out == 0)
                        value[(long)l * d1 + c] = x;
                    else
                        grad[((long)l * n + (ch.out - 1)) * d1 + c] = x;
                }
            }
        }
        if (b + gridDim.x < parts) __syncthreads();  // the next part reuses `part`
    }
}

static_assert(kAddRuns * add_run(1) == add_pass_leaves(1), "a part's leaves");

template <int M, bool CX>
static void launch(const mdpe_plan *pl, int p, double *A, double *value, double *grad, hipStream_t st) {
    const unsigned cblocks = (unsigned)((pl->P.d + kAddCoefs) / kAddCoefs);
    const long parts = pl->add_pass[p + 1] - pl->add_pass[p];
    const unsigned grid = (unsigned)std::min(parts, 1L << 22);  // 2^30 work-items in x
    hipLaunchKernelGGL((add_tree_kernel<M, CX>), dim3(grid, cblocks), dim3(kAddThreads), 0, st, A, pl->d_leaves,
                       pl->d_chunks + pl->add_pass[p], parts, value, grad, pl->P.n, pl->P.d);
}

int launch_add_pass(const mdpe_plan *pl, int p, double *A, double *value, double *grad, hipStream_t st) {
#define CASE(m)                                              \
    case m:                                                  \
        if (pl->P.complex_series())                          \
            launch<m, true>(pl, p, A, value, grad, st);      \
        else                                                 \
            launch<m, false>(pl, p, A, value, grad, st);     \
        break;
    switch (pl->P.m) {
        CASE(1)
        CASE(2)
        CASE(3)
        CASE(4)
        CASE(5)
        CASE(8)
        CASE(10)
        default: set_last_error("unsupported m"); return MDPE_EUNSUPPORTED;
    }
#undef CASE
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_error(std::string("add_tree_kernel: ") + hipGetErrorString(e));
        return MDPE_EDEVICE;
    }
    return MDPE_OK;
}

}  // namespace mdpe
