// block.hip -- per-layer launches of the blocked convolutions (conv_block.hpp).
#include <hip/hip_runtime.h>

#include "../../include/mdpe.h"
#include "conv_block.hpp"
#include "runtime.hpp"

namespace mdpe {

// WPB wavefronts per workgroup (1 or 4), each with its own group of J jobs in
// its own LDS region; Q wavefronts share each group (Q > 1: J = 1).  LONE: for
// launches of at most one wavefront per SIMD (one_per_simd).
template <int M, bool CORR, bool CX, int R, int U, int WPB, bool LONE = false>
__global__ __launch_bounds__(64 * WPB) void conv_block_kernel(double *__restrict__ A, const int4 *__restrict__ jobs,
                                                              int njobs, int d, int J, const int *__restrict__ chains,
                                                              int stride, int its, int group_bytes, int Q) {
    extern __shared__ double lds[];
    if constexpr (LONE) one_per_simd();
    const int wave = WPB == 1 ? 0 : (int)(threadIdx.x >> 6);
    const int wv = blockIdx.x * WPB + wave;
    const int g = Q == 1 ? wv : wv / Q;
    const int part = wv - g * Q;
    const int lane = threadIdx.x & 63;
    const int g0 = min(g * J, njobs), jn = min(J, njobs - g0);
    const int4 job = lane < jn ? jobs[g0 + lane] : make_int4(0, 0, 0, 0);
    conv_block_group<M, CORR, CX, R, U>(A, job, jn, J, d,
                                     (double *)((char *)lds + wave * group_bytes), chains, stride, its, lane,
                                     part * 64 + lane);
}

// Every convolution layer of a plan in one launch (Plan::fused_*): workgroup c
// runs component c layer by layer, each wavefront J of the layer's jobs at a
// time, with a workgroup barrier after every layer; the barrier makes the
// layer's stores visible to the whole workgroup, and operands are read with
// vector loads only.  Every wavefront runs the same rounds.
template <int M, bool CX, int U, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void conv_fused_block_kernel(double *__restrict__ A,
                                                                      const int4 *__restrict__ jobs,
                                                                      const int *__restrict__ off, int nl, int d, int J,
                                                                      const int *__restrict__ chains, int stride,
                                                                      int its, int group_bytes) {
    extern __shared__ double lds[];
    const int waves = (int)(blockDim.x >> 6), wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    const int *o = off + (long)blockIdx.x * (nl + 1);
    double *mine = (double *)((char *)lds + wave * group_bytes);
    // this wavefront's next jobs are loaded a round ahead
    int L = 0, r = o[0] + wave * J;
    auto jobs_left = [&](int at, int end) { return max(0, min(J, end - at)); };
    int jn = jobs_left(r, o[1]);
    int4 job = lane < jn ? jobs[r + lane] : make_int4(0, 0, 0, 0);
    while (L < nl) {
        // every wavefront of the workgroup moves on by the same rule
        const int end = o[L + 1];
        const bool layer_ends = r - wave * J + waves * J >= end;
        const int L2 = layer_ends ? L + 1 : L, r2 = layer_ends ? end + wave * J : r + waves * J;
        const int jn2 = L2 < nl ? jobs_left(r2, o[L2 + 1]) : 0;
        const int4 job2 = lane < jn2 ? jobs[r2 + lane] : make_int4(0, 0, 0, 0);
        conv_block_group<M, false, CX, 1, U>(A, job, jn, J, d, mine, chains, stride, its, lane, lane);
        if (layer_ends) __syncthreads();
        L = L2;
        r = r2;
        jn = jn2;
        job = job2;
    }
}

namespace {

int fail(int code, const std::string &msg) {
    set_last_error(msg);
    return code;
}

template <int M, bool CORR, bool CX, int R, int U>
int launch_r(const mdpe_plan *pl, double *A, const int4 *jobs, int nj, hipStream_t st) {
    const Plan &P = pl->P;
    const LaneSchedule &ls = P.blocks;
    const int J = ls.jobs_per_group, Q = ls.waves_per_job;
    const size_t bytes = (size_t)(block_group_bytes(P.d + 1, kCoef<M, CX>, U, J) + 15) / 16 * 16;
    static std::atomic<bool> attr_set[kMaxDevices];
    const int dv = pl->device >= 0 && pl->device < kMaxDevices ? pl->device : 0;
    if (!attr_set[dv].load()) {
        hipError_t e = hipFuncSetAttribute((const void *)conv_block_kernel<M, CORR, CX, R, U, 1>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLdsBytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)conv_block_kernel<M, CORR, CX, R, U, 1, true>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLdsBytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)conv_block_kernel<M, CORR, CX, R, U, 4>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLdsBytes);
        if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        attr_set[dv].store(true);
    }
    const long waves = ((long)nj + J - 1) / J * Q;
    if (waves > 0x7fffffffL) return fail(MDPE_EUNSUPPORTED, "too many wavefronts in one layer");
    const int simds = simd_count(pl->device);
    if (waves <= 3L * simds && waves > simds && 4 * bytes <= (size_t)kMaxLdsBytes)
        hipLaunchKernelGGL((conv_block_kernel<M, CORR, CX, R, U, 4>), dim3((unsigned)((waves + 3) / 4)), dim3(256),
                           4 * bytes, st, A, jobs, nj, P.d, J, pl->d_blocks, ls.stride, ls.steps, (int)bytes, Q);
    else if (lone_launch(pl->most_waves, waves, simds))
        hipLaunchKernelGGL((conv_block_kernel<M, CORR, CX, R, U, 1, true>), dim3((unsigned)waves), dim3(64), bytes, st, A,
                           jobs, nj, P.d, J, pl->d_blocks, ls.stride, ls.steps, (int)bytes, Q);
    else
        hipLaunchKernelGGL((conv_block_kernel<M, CORR, CX, R, U, 1>), dim3((unsigned)waves), dim3(64), bytes, st, A, jobs,
                           nj, P.d, J, pl->d_blocks, ls.stride, ls.steps, (int)bytes, Q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("conv_block_kernel: ") + hipGetErrorString(e));
    return MDPE_OK;
}

template <int M, bool CX, int U, int WAVES>
int launch_fused_w(const mdpe_plan *pl, double *A, hipStream_t st) {
    constexpr int W = kCoef<M, CX>;
    const Plan &P = pl->P;
    const LaneSchedule &ls = P.fused_blocks;
    const int J = ls.jobs_per_group, waves = P.fused_block_waves;
    const size_t bytes = (size_t)(block_group_bytes(P.d + 1, W, U, J) + 15) / 16 * 16;
    static std::atomic<bool> attr_set[kMaxDevices];
    const int dv = pl->device >= 0 && pl->device < kMaxDevices ? pl->device : 0;
    if (!attr_set[dv].load()) {
        const hipError_t e = hipFuncSetAttribute((const void *)conv_fused_block_kernel<M, CX, U, WAVES>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLdsBytes);
        if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        attr_set[dv].store(true);
    }
    hipLaunchKernelGGL((conv_fused_block_kernel<M, CX, U, WAVES>), dim3((unsigned)P.fused_components), dim3(64 * waves),
                       waves * bytes, st, A, pl->d_fconv, pl->d_foff, P.n_layers(), P.d, J, pl->d_fblocks, ls.stride,
                       ls.steps, (int)bytes);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("conv_fused_block_kernel: ") + hipGetErrorString(e));
    return MDPE_OK;
}

template <int M, bool CX, int U>
int launch_fused_u(const mdpe_plan *pl, double *A, hipStream_t st) {
    if (pl->P.fused_block_waves == 1) return launch_fused_w<M, CX, U, 1>(pl, A, st);
    return launch_fused_w<M, CX, U, 4>(pl, A, st);
}

template <int M, bool CX>
int launch_fused_m(const mdpe_plan *pl, double *A, hipStream_t st) {
    if constexpr (kCoef<M, CX> <= 5) {
        if (block_terms_of(pl->P.w, pl->P.d) == 4) return launch_fused_u<M, CX, 4>(pl, A, st);
        if constexpr (kCoef<M, CX> > 2) return launch_fused_u<M, CX, 2>(pl, A, st);
    }
    return fail(MDPE_EUNSUPPORTED, "no fused blocked convolution of this width");
}

template <int M>
int launch_fused_f(const mdpe_plan *pl, double *A, hipStream_t st) {
    return pl->P.complex_series() ? launch_fused_m<M, true>(pl, A, st) : launch_fused_m<M, false>(pl, A, st);
}

template <int M, bool CORR, bool CX>
int launch_m(const mdpe_plan *pl, double *A, const int4 *jobs, int nj, hipStream_t st) {
    constexpr int W = kCoef<M, CX>;
    const int ru = 10 * pl->P.block_r + pl->P.block_u;
    if constexpr (W == 1)
        if (ru == 44) return launch_r<M, CORR, CX, 4, 4>(pl, A, jobs, nj, st);
    if constexpr (W <= 5)
        if (ru == 14) return launch_r<M, CORR, CX, 1, 4>(pl, A, jobs, nj, st);
    if constexpr (W > 2)
        if (ru == 12) return launch_r<M, CORR, CX, 1, 2>(pl, A, jobs, nj, st);
    return fail(MDPE_EUNSUPPORTED, "no blocked convolution of this width");
}

template <int M>
int launch_f(const mdpe_plan *pl, bool corr, double *A, const int4 *jobs, int nj, hipStream_t st) {
    if (corr) return launch_m<M, true, false>(pl, A, jobs, nj, st);
    return pl->P.complex_series() ? launch_m<M, false, true>(pl, A, jobs, nj, st)
                                  : launch_m<M, false, false>(pl, A, jobs, nj, st);
}

}  // namespace

int launch_block_fused(const mdpe_plan *pl, double *A, hipStream_t st) {
    switch (pl->P.m) {
        case 1: return launch_fused_f<1>(pl, A, st);
        case 2: return launch_fused_f<2>(pl, A, st);
        case 3: return launch_fused_f<3>(pl, A, st);
        case 4: return launch_fused_f<4>(pl, A, st);
        case 5: return launch_fused_f<5>(pl, A, st);
        default: return fail(MDPE_EUNSUPPORTED, "no fused blocked convolution of this width");
    }
}

int launch_block_layer(const mdpe_plan *pl, bool corr, double *A, const int4 *jobs, int nj, hipStream_t st) {
    if (nj == 0) return MDPE_OK;
    switch (pl->P.m) {
        case 1: return launch_f<1>(pl, corr, A, jobs, nj, st);
        case 2: return launch_f<2>(pl, corr, A, jobs, nj, st);
        case 3: return launch_f<3>(pl, corr, A, jobs, nj, st);
        case 4: return launch_f<4>(pl, corr, A, jobs, nj, st);
        case 5: return launch_f<5>(pl, corr, A, jobs, nj, st);
        case 8: return launch_f<8>(pl, corr, A, jobs, nj, st);
        case 10: return launch_f<10>(pl, corr, A, jobs, nj, st);
        default: return fail(MDPE_EUNSUPPORTED, "unsupported m");
    }
}

}  // namespace mdpe
