// chain.hip -- the chain launch by blocks of R coefficients (Plan::pipe_*).
#include <hip/hip_runtime.h>

#include "../../include/mdpe.h"
#include "conv_block.hpp"
#include "runtime.hpp"

namespace mdpe {

// A workgroup barrier that orders LDS accesses only: the LDS stores and reads
// issued before it complete before any wavefront passes it, while global loads
// in flight (second operands) and global stores (read by later launches only)
// are not waited for.
__device__ __forceinline__ void chain_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Workgroup c runs chain c: products where each job's first operand is the
// previous job's output and its second a series no job of the launch writes.
// Its lanes follow the chain's schedule `codes`: rows of (job << 16) | b for
// block b (coefficients R*b .. R*b+R-1) of the chain's job-th product, b + 1
// iterations of R terms (R = 1: U terms, b / U + 1 iterations); (kIdleJob << 16) | (g-1) for g idle iterations; -1
// after the last.  Each coefficient is one lane's sequential sum in the
// specified order, so every bit is that of the per-layer launches.  Job j's
// first operand sits in LDS slot j mod B: job 0's is staged from A, every later
// job's is stored there block by block by the job before it, beside its store
// to A.  Block i of a product is final after its own i + 1 iterations and the
// next product reads its first operand in increasing i, so consecutive
// products overlap.  A workgroup barrier on LDS after every `window`
// iterations orders those stores and reads: iteration t reads block t + 1 of
// its item's first operand (the first iteration's, the item before or the
// prologue) and stores a finished block at its end, and the host checks the
// schedule against exactly that (check_chain_schedule over blocks).
template <int M, bool CX, int R, int U, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void conv_chain_block_kernel(double *__restrict__ A,
                                                                      const int4 *__restrict__ jobs,
                                                                      const ChainComp *__restrict__ comps,
                                                                      const int *__restrict__ codes, int d, int B,
                                                                      int window) {
    constexpr int W = kCoef<M, CX>, W8 = 8 * W;
    extern __shared__ double lds[];
    const ChainComp cc = comps[blockIdx.x];
    const unsigned S8 = (unsigned)((d + 1) * W8);
    const unsigned slot = 8u * chain_slot_doubles(d + 1, W, U);
    // the B slots, one more that takes the last job's blocks, the offsets
    BlockJob *jd = (BlockJob *)at_byte(lds, (unsigned)(B + 1) * slot);
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    {
        const int4 t0 = jobs[cc.first];
        const double *xs = at_byte(A, (unsigned)t0.x * S8);
        for (int q = tid; q < (d + 1) * W; q += nt) lds[q] = xs[q];
        for (int j = tid; j < cc.len; j += nt) {
            const int4 t = jobs[cc.first + j];
            jd[j] = BlockJob{(unsigned)(j % B) * slot, (unsigned)t.y * S8, (unsigned)t.z * S8,
                             (unsigned)(j + 1 < cc.len ? (j + 1) % B : B) * slot};
        }
    }
    // codes four ahead of the lane, as in conv_block_group
    const int *cp = codes + cc.code_off + (long)tid * cc.stride;
    auto next_code = [&]() {
        const int c = *cp;
        cp += c >= 0 ? 1 : 0;
        return c;
    };
    const int c0 = next_code(), c1 = next_code();
    int c2 = next_code(), c3 = next_code();
    __syncthreads();

    auto job_of = [&](int c) { return c >= 0 && (c >> 16) != kIdleJob ? c >> 16 : 0; };
    auto item = [&](int c, const BlockJob &jb) {
        BlockItem t;
        const bool live = c >= 0 && (c >> 16) != kIdleJob;
        const int low = c & 0xffff, b = live ? low : 0;
        const unsigned up = (unsigned)(b * R * W8);
        t.k0 = R * b;
        t.rem = c < 0 ? 1 : live && R == 1 ? (low + U) / U : low + 1;
        t.step = live ? U * W8 : 0;
        t.s = jb.y + up;
        t.b = jb.x;
        t.out = live ? jb.z + up : kNoStore;
        t.next = jb.next + up;
        return t;
    };
    unsigned sp, bp;
    // (R = 1 goes down from the item's coefficient with the terms)
    auto load_s = [&](int r) { return at_byte(A, sp + (unsigned)((R == 1 ? -r : r) * W8)); };
    auto load_b = [&](int r) { return at_byte(lds, bp + (unsigned)(r * W8)); };
    BlockItem t0 = item(c0, jd[job_of(c0)]), t1 = item(c1, jd[job_of(c1)]);
    BlockJob j2 = jd[job_of(c2)];
    sp = t0.s;
    bp = t0.b;
    double cur[U][W], x[U][W];
#pragma unroll
    for (int r = 0; r < U; ++r) {
        load_coef<W>(load_s(r), cur[r]);
        load_coef<W>(load_b(r), x[r]);
    }
    Vec<R> acc[W];
#pragma unroll
    for (int l = 0; l < W; ++l)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[l].v[r] = 0.0;
    bool first = true;
    int until_barrier = window;
    for (int s = 0; s < cc.steps; ++s) {
        const bool last = t0.rem == 1;
        sp = last ? t1.s : sp - (unsigned)t0.step;
        bp = last ? t1.b : bp + (unsigned)t0.step;
        const int over = R == 1 && U > 1 && last ? U - 1 - t0.k0 % U : 0;
        block_terms<M, CX, false, R, U>(cur, x, acc, first, last, over, load_s, load_b);
        --t0.rem;
        first = last;
        if (last) {
            if (t0.out != kNoStore) {
                double *o = at_byte(A, t0.out), *n = at_byte(lds, t0.next);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r == 0 || t0.k0 + r <= d) {
#pragma unroll
                        for (int l = 0; l < W; ++l) {
                            o[r * W + l] = acc[l].v[r];
                            n[r * W + l] = acc[l].v[r];
                        }
                    }
            }
            t0 = t1;
            t1 = item(c2, j2);
            j2 = jd[job_of(c3)];
            c2 = c3;
            c3 = next_code();
        }
        if (--until_barrier == 0) {
            chain_barrier();
            until_barrier = window;
        }
    }
}

namespace {

int fail(int code, const std::string &msg) {
    set_last_error(msg);
    return code;
}

template <int M, bool CX, int R, int U, int WAVES>
int launch_w(const mdpe_plan *pl, double *A, hipStream_t st) {
    const Plan &P = pl->P;
    const size_t lds = (size_t)chain_lds_bytes(P.d + 1, kCoef<M, CX>, U, P.pipe_ring, P.pipe_layers);
    if (lds > (size_t)kMaxLdsBytes) return fail(MDPE_EUNSUPPORTED, "chain launch: LDS beyond one workgroup's");
    static std::atomic<bool> attr_set[kMaxDevices];
    const int dv = pl->device >= 0 && pl->device < kMaxDevices ? pl->device : 0;
    if (!attr_set[dv].load()) {
        const hipError_t e = hipFuncSetAttribute((const void *)conv_chain_block_kernel<M, CX, R, U, WAVES>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLdsBytes);
        if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        attr_set[dv].store(true);
    }
    hipLaunchKernelGGL((conv_chain_block_kernel<M, CX, R, U, WAVES>), dim3((unsigned)P.pipe_comps.size()),
                       dim3(64 * P.pipe_waves), lds, st, A, pl->d_pjobs, pl->d_pcomps, pl->d_pcodes, P.d, P.pipe_ring,
                       P.pipe_window);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MDPE_EDEVICE, std::string("conv_chain_block_kernel: ") + hipGetErrorString(e));
    return MDPE_OK;
}

template <int M, bool CX, int R, int U>
int launch_r(const mdpe_plan *pl, double *A, hipStream_t st) {
    const int w = pl->P.pipe_waves;
    if (w <= 4) return launch_w<M, CX, R, U, 4>(pl, A, st);
    if (w <= 8) return launch_w<M, CX, R, U, 8>(pl, A, st);
    if constexpr (kCoef<M, CX> * U <= 10)  // (128 VGPRs: wider ones would spill)
        if (w <= 16) return launch_w<M, CX, R, U, 16>(pl, A, st);
    return fail(MDPE_EUNSUPPORTED, "chain launch: too many wavefronts per chain");
}

template <int M, bool CX>
int launch_m(const mdpe_plan *pl, double *A, hipStream_t st) {
    constexpr int W = kCoef<M, CX>;
    const int ru = 10 * pl->P.pipe_r + pl->P.pipe_u;
    if constexpr (W <= 2)
        if (ru == 44) return launch_r<M, CX, 4, 4>(pl, A, st);
    if constexpr (W <= 5)
        if (ru == 22) return launch_r<M, CX, 2, 2>(pl, A, st);
    if constexpr (W <= 10)
        if (ru == 12) return launch_r<M, CX, 1, 2>(pl, A, st);
    if (ru == 11) return launch_r<M, CX, 1, 1>(pl, A, st);
    return fail(MDPE_EUNSUPPORTED, "no blocked chain launch of this width");
}

}  // namespace

int launch_block_chain(const mdpe_plan *pl, double *A, hipStream_t st) {
    const bool cx = pl->P.complex_series();
#define CASE(m) \
    case m: return cx ? launch_m<m, true>(pl, A, st) : launch_m<m, false>(pl, A, st);
    switch (pl->P.m) {
        CASE(1)
        CASE(2)
        CASE(3)
        CASE(4)
        CASE(5)
        CASE(8)
        CASE(10)
        default: return fail(MDPE_EUNSUPPORTED, "unsupported m");
    }
#undef CASE
}

}  // namespace mdpe
