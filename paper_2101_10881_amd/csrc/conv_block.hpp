// conv_block.hpp -- one wavefront's group of convolutions (or correlations),
// several terms per iteration.
//
// A lane computes one item at a time: R consecutive output coefficients R*b ..
// R*b+R-1 of a job, U terms of each per iteration, every coefficient one
// lane's sum in the specified order, term 0 first.  The operands are
//   convolution  z_k = sum_i x_i y_{k-i}           shared x_i,  sliding y_{k-i}
//   correlation  z_{d-k} = sum_i x_{d-k+i} y_i     shared y_i,  sliding x_{d-(k-i)}
//
// R = 1: one coefficient, U terms an iteration: the products of an iteration
// are independent of each other and of the sum, and the address updates, the
// test for the item's end and the item switch are paid once per U terms.
// R = U > 1: step i of the R coefficients needs the one shared coefficient i
// and the R sliding coefficients k-i, of which R - 1 were in registers at step
// i - 1; a tile of R x R multiply-adds reads R coefficients of each operand
// (one sliding block, going down from block b; after the last one the next
// item's top block) instead of R*R.
//
// The last iteration of an item holds terms i > k, which are computed and
// dropped.  What a lane needs of its next item (operand and output addresses,
// iterations) is in registers before the switch: a switch waits for no memory.
#pragma once

#include <hip/hip_runtime.h>

#include "md.hpp"
#include "plan.hpp"

namespace mdpe {

template <int W>
__device__ __forceinline__ void load_coef(const double *p, double (&v)[W]) {
#pragma unroll
    for (int l = 0; l < W; ++l) v[l] = p[l];
}

// Workspace and LDS addresses are 32-bit byte offsets from a wavefront-uniform
// base (the blocked kernels run on workspaces below 4 GiB): one instruction
// per address step, and a lane's state is a few registers.
__device__ __forceinline__ const double *at_byte(const double *base, unsigned off) {
    return (const double *)((const char *)base + off);
}
__device__ __forceinline__ double *at_byte(double *base, unsigned off) { return (double *)((char *)base + off); }

constexpr unsigned kNoStore = 0xffffffffu;  // `out` of an item whose sum is not stored

// A job's offsets: first operand, second operand, output, and (chain launch)
// the next job's first operand.
struct BlockJob {
    unsigned x, y, z, next;
};

// What a lane needs of an item: offsets of its first sliding and shared
// coefficients, of its first output coefficient, of that coefficient in the
// next job's first operand (chain launch), iterations, first coefficient.
struct BlockItem {
    unsigned s, b, out, next;
    int rem, k0, step;  // step: bytes an iteration moves the operands by (0: idle)
};

// One tile: R terms of R coefficients' sums.  cur and low hold the sliding
// block and the one below it, x the shared block (the next iteration's on
// return: load_b(i) reads its coefficient i).
template <int M, bool CX, bool CORR, int R, int W, class LoadB>
__device__ __forceinline__ void tile_terms(const double (&cur)[R][W], const double (&low)[R][W], double (&x)[R][W],
                                           Vec<R> (&acc)[W], bool first, bool last, LoadB load_b) {
    static_assert(W == kCoef<M, CX>, "doubles per coefficient");
#pragma unroll
    for (int i = 0; i < R; ++i) {
        // row i: shared coefficient i0 + i times the sliding ones k0 + r - i0 - i
        Vec<R> sl[W], p[W], t[W];
#pragma unroll
        for (int l = 0; l < W; ++l)
#pragma unroll
            for (int r = 0; r < R; ++r)
                sl[l].v[r] = r >= i ? cur[r >= i ? r - i : 0][l] : low[r >= i ? 0 : R + r - i][l];
        if constexpr (CORR)
            coef_mul<M, CX>(sl, x[i], p);
        else
            coef_mul<M, CX>(x[i], sl, p);
        load_coef<W>(load_b(i), x[i]);
        coef_add<M, CX>(acc, p, t);
        // keeps the compiler from moving a dropped term's arithmetic into a
        // branch of its own, where it would run without the other sums beside
        // it
#pragma unroll
        for (int l = 0; l < W; ++l)
#pragma unroll
            for (int r = 0; r < i; ++r) asm volatile("" : "+v"(t[l].v[r]));
#pragma unroll
        for (int l = 0; l < W; ++l)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (i == 0)
                    acc[l].v[r] = first ? p[l].v[r] : t[l].v[r];
                else if (r < i)
                    acc[l].v[r] = last ? acc[l].v[r] : t[l].v[r];
                else
                    acc[l].v[r] = t[l].v[r];
            }
    }
}

// One iteration of R coefficients' sums.  cur and x hold its operands on
// entry, the next iteration's on return (load_s / load_b(r) read coefficient r
// of the next sliding / shared block); over: terms dropped at the end of the
// item (R = 1; 0 unless last).
template <int M, bool CX, bool CORR, int R, int U, int W, class LoadS, class LoadB>
__device__ __forceinline__ void block_terms(double (&cur)[U][W], double (&x)[U][W], Vec<R> (&acc)[W], bool first,
                                            bool last, int over, LoadS load_s, LoadB load_b) {
    static_assert(W == kCoef<M, CX>, "doubles per coefficient");
    if constexpr (R == 1) {
        double p[U][W];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (CORR)
                coef_mul<M, CX>(cur[u], x[u], p[u]);
            else
                coef_mul<M, CX>(x[u], cur[u], p[u]);
            load_coef<W>(load_s(u), cur[u]);
            load_coef<W>(load_b(u), x[u]);
        }
        double a[W], t[W];
#pragma unroll
        for (int l = 0; l < W; ++l) a[l] = acc[l].v[0];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            coef_add<M, CX>(a, p[u], t);
            const bool keep = u > 0 && over >= U - u;
#pragma unroll
            for (int l = 0; l < W; ++l) {
                if (u > 0) asm volatile("" : "+v"(t[l]));  // (a select, not a branch around the sum)
                a[l] = u == 0 ? (first ? p[0][l] : t[l]) : (keep ? a[l] : t[l]);
            }
        }
#pragma unroll
        for (int l = 0; l < W; ++l) acc[l].v[0] = a[l];
    } else {
        double low[U][W];
#pragma unroll
        for (int r = 0; r < U; ++r) load_coef<W>(load_s(r), low[r]);
        tile_terms<M, CX, CORR, R, W>(cur, low, x, acc, first, last, load_b);
#pragma unroll
        for (int r = 0; r < U; ++r)
#pragma unroll
            for (int l = 0; l < W; ++l) cur[r][l] = low[r][l];
    }
}

// Descriptors (lane j holds job j's), then the staged operands of the jn jobs as
// one flat range with several loads in flight per lane: the first operand, which
// may be the job's own output, and for coefficients of at most two doubles the
// second too.
template <int M, bool CORR, bool CX, int U>
__device__ __forceinline__ void block_stage(const double *__restrict__ A, int4 job, int jn, int J, int d, double *lds,
                                            int lane) {
    constexpr int W = kCoef<M, CX>;
    constexpr bool YL = stages_second_operand(W);
    const int S = (d + 1) * W, SX = block_series_stride(d + 1, W);
    double *X = lds + block_front_pad(W, U), *Y = X + (long)J * SX;
    BlockJob *jd = (BlockJob *)(lds + block_jobs_offset(d + 1, W, U, J));
    if (lane < jn) {
        const unsigned S8 = (unsigned)S * 8u;
        jd[lane] = BlockJob{(unsigned)job.x * S8, (unsigned)job.y * S8, (unsigned)job.z * S8, 0u};
    }
    __syncthreads();
    const int total = jn * S;
    const int sj = 64 / S, sq = 64 - sj * S;
    int j = lane / S, q = lane - j * S;
    constexpr int kLoads = YL ? 4 : 8;
    for (int g = lane; g < total; g += 64 * kLoads) {
        double vx[kLoads], vy[kLoads];
        int at[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            at[u] = -1;
            if (g + 64 * u < total) {
                const BlockJob &o = jd[j];
                at[u] = j * SX + q;
                vx[u] = *at_byte(A, o.x + 8u * (unsigned)q);
                if (YL) vy[u] = *at_byte(A, o.y + 8u * (unsigned)q);
            }
            j += sj;
            q += sq;
            if (q >= S) {
                q -= S;
                ++j;
            }
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u)
            if (at[u] >= 0) {
                X[at[u]] = vx[u];
                if (YL) Y[at[u]] = vy[u];
            }
    }
    __syncthreads();
}

// One wavefront's group: jn <= J <= 64 jobs (lane j holds job j's {t1, t2, t3}, so
// that a caller with several groups can load the next one's early), the lanes'
// items from the schedule `chains` (code (job << 16) | item, -1 after a row's
// last), `its` iterations.
// lds: block_group_bytes(d + 1, W, U, J).  Ends with the wavefront's stores
// issued.  Reads past a series only enter terms or coefficients that are
// dropped: in LDS up to one block past either end of an operand (padded); in
// global memory at most U - 1 coefficients before (convolution, R = 1) or past
// (R > 1, reverse pass) the second operand's slot, inside the workspace (the host
// checks that: reads_inside).
template <int M, bool CORR, bool CX, int R, int U>
__device__ __forceinline__ void conv_block_group(double *__restrict__ A, int4 job, int jn, int J, int d, double *lds,
                                                 const int *__restrict__ chains, int stride, int its, int lane,
                                                 int row) {
    constexpr int W = kCoef<M, CX>, W8 = 8 * W;
    static_assert(R == 1 || R == U, "one coefficient, or square tiles");
    constexpr bool YL = stages_second_operand(W);
    const int SX = block_series_stride(d + 1, W);
    const unsigned X = 8u * block_front_pad(W, U), Y = X + 8u * (unsigned)(J * SX);  // bytes in lds; Y used when YL
    const BlockJob *jd = (const BlockJob *)(lds + block_jobs_offset(d + 1, W, U, J));

    // the lane's codes, four ahead: an item's code, then its job's offsets,
    // then its addresses are in registers before the lane reaches it, so the
    // switch to it waits for no memory (the list pointer stops on the
    // terminator)
    const int *cp = chains + (long)row * stride;
    auto next_code = [&]() {
        const int c = *cp;
        cp += c >= 0 ? 1 : 0;
        return c;
    };
    const int c0 = next_code(), c1 = next_code();
    int c2 = next_code(), c3 = next_code();

    block_stage<M, CORR, CX, U>(A, job, jn, J, d, lds, lane);
    if (jn <= 0) return;  // a wavefront past the last group (after the workgroup barriers)

    auto job_of = [&](int c) { return c >= 0 && (c >> 16) < jn ? c >> 16 : 0; };
    auto item = [&](int c, const BlockJob &jb) {
        BlockItem t;
        const bool live = c >= 0 && (c >> 16) < jn;
        const int j = live ? c >> 16 : 0, b = live ? c & 0xffff : 0;
        t.k0 = R * b;
        t.rem = R == 1 ? (b + U) / U : b + 1;
        const unsigned up = (unsigned)(t.k0 * W8), down = (unsigned)((d - t.k0) * W8);
        const unsigned xl = X + 8u * (unsigned)(j * SX), yl = Y + 8u * (unsigned)(j * SX);
        if (CORR) {
            t.s = xl + down;
            t.b = YL ? yl : jb.y;
            t.out = live ? jb.z + down : kNoStore;
        } else {
            t.s = (YL ? yl : jb.y) + up;
            t.b = xl;
            t.out = live ? jb.z + up : kNoStore;
        }
        return t;
    };
    // coefficient e of a sliding block: R = 1 goes down from the item's
    // coefficient with the terms, R > 1 up over its coefficients
    constexpr int kDir = (R == 1 ? -1 : 1) * (CORR ? -1 : 1);
    unsigned sp, bp;
    auto load_s = [&](int r) { return at_byte(CORR || YL ? lds : A, sp + (unsigned)(r * kDir * W8)); };
    auto load_b = [&](int r) { return at_byte(CORR && !YL ? A : lds, bp + (unsigned)(r * W8)); };

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
    for (int s = 0; s < its; ++s) {
        const bool last = t0.rem == 1;
        sp = last ? t1.s : sp + (unsigned)(CORR ? U * W8 : -U * W8);
        bp = last ? t1.b : bp + (unsigned)(U * W8);
        const int over = R == 1 && U > 1 && last ? U - 1 - t0.k0 % U : 0;
        block_terms<M, CX, CORR, R, U>(cur, x, acc, first, last, over, load_s, load_b);
        --t0.rem;
        first = last;
        if (last) {
            if (t0.out != kNoStore) {
                double *o = at_byte(A, t0.out);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r == 0 || t0.k0 + r <= d) {
#pragma unroll
                        for (int l = 0; l < W; ++l) o[(CORR ? -r : r) * W + l] = acc[l].v[r];
                    }
            }
            t0 = t1;
            t1 = item(c2, j2);
            j2 = jd[job_of(c3)];
            c2 = c3;
            c3 = next_code();
        }
    }
}

}  // namespace mdpe
