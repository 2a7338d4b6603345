// batch.hip -- many polynomials in one persistent launch.
//
// Every instance keeps its own plan (Section 5 job lists), workspace and
// buffers.  The batch turns all instances' stages -- staging, each
// convolution layer, each addition level, gathering -- into tasks: a task is
// a chunk of one stage of one instance, sized to carry enough work to hide
// its signalling.  The tasks form one queue, ordered by pipeline depth, so a
// task only ever depends on earlier tasks.
//
// A task costs 32 ns (convolution) to 100 ns (addition) of the launch in fences
// and the claim, whatever it does (measured with more and smaller tasks).  So, at
// two to five doubles per coefficient, convolutions run by blocks (conv_block.hpp)
// and, where a queue holds at least kSetComponents independent components, a task
// is a set of whole components, every layer of them, and no wait lies between the
// layers; additions run by passes over whole output lists, the last into the
// user's buffers, instead of a stage per level and a gather.  128 mixed instances
// (2 and 4 doubles, d = 8 to 128): 12.3 -> 7.9 ms, 512: 32.8 -> 27.
//
// Instances are spread over one queue per XCD (the MI355X has 8 XCDs, each
// with its own L2), balancing estimated cost; all tasks of an instance sit in
// one queue, except for an instance costing more than an eighth of the batch
// (a batch of one), whose tasks are dealt over all queues in turn.  Each
// queue is ordered by pipeline depth.  One persistent kernel of one-wavefront
// workgroups (equal numbers per SIMD: two, or three for many tasks, by blocks,
// else as many as are resident) reads the XCD it runs on from the XCC_ID
// hardware register and claims tasks of that XCD's queue with an atomic counter, so an
// instance's data stays near one L2.  A task of stage s of instance p waits
// until p's completion counter reaches the number of p's tasks in stages
// before s (agent-scope acquire), runs, then increments the counter
// (agent-scope release).  The fences are agent-scope because narrower ones
// are not enough: an L1-only invalidation on acquire and a plain store wait
// on release gave wrong results; they also make a dealt instance's results
// visible across XCDs.  No deadlock: a task depends only on tasks of smaller
// depth, and every queue is claimed in depth order by running wavefronts (each
// XCD has resident ones), so an unfinished task of the smallest depth is
// either running with all its inputs done or is reached by its queue once the
// claimed tasks before it, of the same depth, finish.
// A bounded spin turns any unexpected wait into an error flag, not a hang.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../../include/mdpe.h"
#include "conv_block.hpp"
#include "conv_core.hpp"
#include "plan.hpp"
#include "runtime.hpp"

namespace mdpe {

struct BatchInst {
    double *A;
    const double *coeff;
    const double *z;
    double *value;
    double *grad;
    const int4 *conv;  // in launch order, or by set of components (goff)
    const int *goff;   // component sets: group g spans conv[goff[g] .. goff[g + 1])
    const int2 *add;
    const AddChunk *chunks;  // addition passes (blocked batches): parts of the output lists
    const int *leaves;
    const int2 *stage;
    const int *out;  // kSummed: written by an addition task
    const int *chains;
    int stride, steps, J;
    int simple;  // deal coefficients to lanes in turn (see conv_group)
    int m, d, n, N;
};

struct BatchTask {
    int inst;
    int kind;   // 0 stage, 1 conv, 2 add, 3 gather
    int need;   // wait until the instance's completion counter reaches this
    int count;  // conv: jobs; others: items (coefficients)
    long first; // conv: first job; add: first (pair, coefficient) item; stage/gather: first item
    // conv: a set of whole components, run group by group (groups > 0); add, by
    // passes: `groups` (part, coefficient) items from item `group` (groups > 0)
    int group, groups;
};

constexpr int kSpinLimit = 1 << 22;
constexpr int kQueues = 8;  // one task queue per XCD
constexpr int kSummed = -2;
constexpr int kSetComponents = 256;  // resident wavefronts of an XCD (32 CUs x 8)
constexpr double kSetOverLayers = 1.4;

// the XCD (XCC) this wavefront runs on
__device__ __forceinline__ int xcd_id() { return (int)(__builtin_amdgcn_s_getreg(20 | (15 << 11)) & (kQueues - 1)); }

// Terms an iteration of the blocked convolutions takes at width w (four against
// two at three doubles 1.05 times as fast, 64 instances at d = 50; at four
// doubles 0.98 to 1.02, so two there).
__host__ __device__ constexpr int batch_terms(int w) { return w <= 3 ? 4 : 2; }

// An addition task by passes: each lane sums one part of an output's list (up to
// add_pass_leaves leaves) at one coefficient, E elements at a time with their
// loads in flight together, in the pairs of the tree (an element's sum stands in
// its last leaf's slot, as the level-by-level additions leave it; a lane reads
// back only what it stored itself).  A launch stage per tree level cost a
// release, an acquire and a memory latency per level and addition.
template <int M>
__device__ void add_parts(const BatchTask &T, const BatchInst &I, int lane) {
    constexpr int E = M <= 4 ? 8 : 4;
    const int d1 = I.d + 1;
    const long S = (long)d1 * M;
    for (int it = lane; it < T.groups; it += 64) {
        const int q = T.group + it;
        const int b = q / d1, c = q - b * d1;
        const AddChunk ch = I.chunks[b];
        if (ch.count < 2) continue;  // (one leaf or none: the gather's, or already in place)
        const int *leaves = I.leaves + ch.first;
        double *A = I.A + (long)c * M;
        for (int len = ch.count, step = 1; len > 1; len = (len + E - 1) / E, step *= E) {
            for (int r = 0; r < len; r += E) {
                // element i's sum stands in the slot of leaf min((i + 1) * step, count) - 1
                double v[E][M];
                long off[E];
#pragma unroll
                for (int e = 0; e < E; ++e)
                    off[e] = (long)leaves[min((min(r + e, len - 1) + 1) * step, ch.count) - 1] * S;
#pragma unroll
                for (int e = 0; e < E; ++e)
#pragma unroll
                    for (int l = 0; l < M; ++l) v[e][l] = A[off[e] + l];
#pragma unroll
                for (int s = 1; s < E; s *= 2)
#pragma unroll
                    for (int p = 0; p < E; p += 2 * s)
                        if (r + p + s < len) {
                            double z[M];
                            md_add<M>(v[p + s], v[p], z);
#pragma unroll
                            for (int l = 0; l < M; ++l) v[p][l] = z[l];
                        }
                if (len <= E && ch.out >= 0) {
#pragma unroll
                    for (int l = 0; l < M; ++l) {
                        if (ch.out == 0)
                            I.value[(long)l * d1 + c] = v[0][l];
                        else
                            I.grad[((long)l * I.n + (ch.out - 1)) * d1 + c] = v[0][l];
                    }
                } else {
#pragma unroll
                    for (int l = 0; l < M; ++l) A[off[E - 1] + l] = v[0][l];
                }
            }
        }
    }
}

template <int M, bool BLK>
__device__ void run_task(const BatchTask &T, const BatchInst &I, double *lds, int lane) {
    const int d1 = I.d + 1;
    const int kind = __builtin_amdgcn_readfirstlane(T.kind);
    if (kind == 1) {
        if constexpr (BLK) {
            // a set's groups one after the other (the barrier orders a group's
            // stores before the next one's loads), or a run of one layer's jobs
            const int groups = T.groups > 0 ? T.groups : (T.count + I.J - 1) / I.J;
            auto range = [&](int g, long &a, int &jn) {
                a = T.first + (long)g * I.J;
                jn = min(I.J, T.count - g * I.J);
                if (T.groups > 0) {
                    a = I.goff[T.group + g];
                    jn = I.goff[T.group + g + 1] - (int)a;
                }
            };
            long a;
            int jn;
            range(0, a, jn);
            int4 job = lane < jn ? I.conv[a + lane] : make_int4(0, 0, 0, 0);
            for (int g = 0; g < groups; ++g) {
                // the next group's jobs load while this one's run
                int jn2 = 0;
                int4 job2 = make_int4(0, 0, 0, 0);
                if (g + 1 < groups) {
                    range(g + 1, a, jn2);
                    if (lane < jn2) job2 = I.conv[a + lane];
                }
                conv_block_group<M, false, false, 1, batch_terms(M)>(I.A, job, __builtin_amdgcn_readfirstlane(jn), I.J,
                                                                     I.d, lds, I.chains, I.stride, I.steps, lane, lane);
                __syncthreads();
                jn = jn2;
                job = job2;
            }
        } else {
            for (int g = 0; g < T.count; g += I.J) {
                // chain codes loaded every step: 1.4% faster here (512 mixed
                // instances) than at chain starts
                conv_group<M, false, false, false, true>(I.A, I.conv + T.first + g, min(I.J, T.count - g), I.J, I.d,
                                                         lds, I.chains, I.stride, I.steps, lane, lane, I.simple != 0);
                __syncthreads();
            }
        }
    } else {
        // item T.first + q, q = lane, lane + 64, ...: series e, coefficient c.
        // One 64-bit division per lane and task; each iteration then adds
        // (64 / d1, 64 % d1) with a carry.
        if (BLK && kind == 2 && T.groups > 0) {
            add_parts<M>(T, I, lane);
            return;
        }
        const long f = T.first + lane;
        long e = f / d1;
        int c = (int)(f - e * d1);
        const int qe = 64 / d1, qc = 64 - qe * d1;
        if (BLK && kind == 0) {
            // four items' loads in flight per lane
            for (int q = lane; q < T.count; q += 256) {
                double v[4][M];
                double *to[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (q + 64 * u < T.count) {
                        const int2 en = I.stage[e];
                        const bool co = en.y <= I.N;
                        const double *src = co ? I.coeff + (long)en.y * d1 + c : I.z + (long)(en.y - I.N - 1) * d1 + c;
                        const long plane = (long)(co ? I.N + 1 : I.n) * d1;
#pragma unroll
                        for (int l = 0; l < M; ++l) v[u][l] = src[l * plane];
                        to[u] = I.A + ((long)en.x * d1 + c) * M;
                    }
                    e += qe;
                    c += qc;
                    if (c >= d1) {
                        c -= d1;
                        ++e;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (q + 64 * u < T.count) {
#pragma unroll
                        for (int l = 0; l < M; ++l) to[u][l] = v[u][l];
                    }
            }
            return;
        }
        for (int q = lane; q < T.count; q += 64) {
            if (kind == 0)
                stage_item(I.A, I.coeff, I.z, I.stage[e], c, I.N, I.n, I.d, M);
            else if (kind == 2)
                add_item<M>(I.A, I.add[e], c, I.d);
            else if (const int slot = I.out[e]; slot != kSummed)
                gather_item(I.A, I.value, I.grad, slot, (int)e, c, I.n, I.d, M);
            e += qe;
            c += qc;
            if (c >= d1) {
                c -= d1;
                ++e;
            }
        }
    }
}

__global__ __launch_bounds__(64) void batch_reset_kernel(int *ctl, int n) {
    for (int i = threadIdx.x; i < n; i += 64) ctl[i] = 0;
}

// ctl[q] = next task of queue q, ctl[kQueues] = error flag,
// ctl[kQueues + 1 + p] = completion counter of instance p.
// qinfo[q] = first task of queue q, qinfo[kQueues + q] = its task count.
// Up to quad double the kernel asks for six resident wavefronts per SIMD
// (at most 80 VGPRs, no spills), the occupancy its register use allowed
// before the convolution loop kept operand addresses per lane.
// BLK: every instance's convolutions run by blocks (conv_block.hpp).
template <int M1, int M2, bool BLK>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(BLK ? 4 : M2 <= 4 ? 6 : 1))) void batch_kernel(const BatchTask *__restrict__ tasks, const int *__restrict__ qinfo,
                                                   const BatchInst *__restrict__ insts, int *ctl) {
    extern __shared__ double lds[];
    const int lane = threadIdx.x;
    const int q = xcd_id();
    const int qbase = qinfo[q], qcount = qinfo[kQueues + q];
    int *next = ctl + q, *err = ctl + kQueues, *done = ctl + kQueues + 1;
    // Every value that steers control flow is made wave-uniform (scalar), so
    // the task loop is one scalar loop, never a per-lane divergent one.
    for (;;) {
        int t = 0;
        if (lane == 0) t = atomicAdd(next, 1);
        t = __builtin_amdgcn_readfirstlane(__shfl(t, 0));
        if (t >= qcount) break;
        const BatchTask T = tasks[qbase + t];
        const int inst = __builtin_amdgcn_readfirstlane(T.inst);
        const int need = __builtin_amdgcn_readfirstlane(T.need);
        if (need > 0) {
            // poll without invalidating caches, then one acquire fence
            int spins = 0, ok = 1;
            for (;;) {
                const int v = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(done + inst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (v >= need) break;
                const int e = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (e || ++spins > kSpinLimit) {
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(32);  // ~2000 cycles: little polling traffic, small against a task
            }
            if (!ok) {
                if (lane == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        const BatchInst I = insts[inst];
        if (__builtin_amdgcn_readfirstlane(I.m) == M1)
            run_task<M1, BLK>(T, I, lds, lane);
        else
            run_task<M2, BLK>(T, I, lds, lane);
        // release: the fence waits for this wavefront's stores and writes the
        // L2 back; then lane 0 moves the instance's completion counter
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (lane == 0) __hip_atomic_fetch_add(done + inst, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace mdpe

// ------------------------------------------------------------------ runtime

namespace {

int bfail(int code, const std::string &msg) {
    mdpe::set_last_error(msg);
    return code;
}

#define BHIP(call)                                                                                 \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) return bfail(MDPE_EDEVICE, std::string(#call ": ") + hipGetErrorString(e_)); \
    } while (0)

}  // namespace

struct mdpe_batch {
    int device = -1;
    int count = 0;
    std::vector<mdpe::BatchInst> insts;
    std::vector<mdpe::BatchTask> tasks;
    mdpe::BatchInst *d_insts = nullptr;
    mdpe::BatchTask *d_tasks = nullptr;
    int *d_qinfo = nullptr;
    int *d_ctl = nullptr;
    std::vector<int> qinfo;      // [2 * kQueues]: first task, task count per queue
    std::vector<int> inst_queue; // queue of each instance, -1: dealt over all queues
    std::vector<int> task_queue; // queue of each task, in task order
    std::vector<int *> d_chains;
    // instances run by component sets: their jobs set by set, layer by layer, and the groups
    std::vector<std::vector<int4>> set_jobs;
    std::vector<std::vector<int>> set_groups;
    int4 *d_set_jobs = nullptr;
    int *d_set_groups = nullptr;
    std::vector<int> outs;  // blocked batches: every instance's output slots, kSummed where a list has additions
    int *d_outs = nullptr;
    size_t lds = 0;
    int grid = 0;
    bool grid_fixed = false;
    int m1 = 0, m2 = 0;
    bool blocks = false;  // convolutions by blocks
    bool buffers_set = false;
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    hipStream_t cap = nullptr;
    std::vector<int> stage_tasks;  // tasks per kind, for batch_info
    // eval_and_diff_batch: instance p's workspace starts ws_off[p] bytes into
    // the caller's one workspace of ws_bytes; pointer tables are staged in a
    // ring of pinned host buffers, each reused once its copy has run
    std::vector<int64_t> ws_off;
    int64_t ws_bytes = 0;
    static constexpr int kRing = 4;
    mdpe::BatchInst *ring[kRing] = {};
    hipEvent_t ring_ev[kRing] = {};
    bool ring_used[kRing] = {};
    int ring_next = 0;
};

namespace {

void free_batch(mdpe_batch *b) {
    if (!b) return;
    if (b->device < 0) {
        delete b;
        return;
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(b->device);
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (int r = 0; r < mdpe_batch::kRing; ++r) {
        if (b->ring_ev[r]) {
            (void)hipEventSynchronize(b->ring_ev[r]);
            (void)hipEventDestroy(b->ring_ev[r]);
        }
        if (b->ring[r]) (void)hipHostFree(b->ring[r]);
    }
    (void)hipFree(b->d_insts);
    (void)hipFree(b->d_tasks);
    (void)hipFree(b->d_qinfo);
    (void)hipFree(b->d_ctl);
    for (auto p : b->d_chains) (void)hipFree(p);
    (void)hipFree(b->d_set_jobs);
    (void)hipFree(b->d_set_groups);
    (void)hipFree(b->d_outs);
    if (prev >= 0 && b->device >= 0) (void)hipSetDevice(prev);
    delete b;
}

// Kernel attributes and the persistent grid (resident one-wavefront
// workgroups), resolved once, outside any stream capture.
template <int M1, int M2, bool BLK>
int prepare_batch(mdpe_batch *b) {
    // the LDS limit is a per-device function attribute: raise it once per device
    static std::atomic<bool> attr[kMaxDevices];
    const int dv = b->device >= 0 && b->device < kMaxDevices ? b->device : 0;
    if (b->lds > 65536 && !attr[dv].load()) {
        BHIP(hipFuncSetAttribute((const void *)mdpe::batch_kernel<M1, M2, BLK>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)mdpe::kMaxLdsBytes));
        attr[dv].store(true);
    }
    if (b->grid == 0) {
        int per_cu = 0, cus = 0;
        BHIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)mdpe::batch_kernel<M1, M2, BLK>, 64,
                                                          b->lds));
        BHIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device));
        // every XCD needs resident wavefronts to drain its queue; a CU's four
        // SIMDs get equal numbers (17 resident per CU put five on one SIMD,
        // whose tasks ran slowest: 16 measured 0.6% faster on the mixed batch)
        if (per_cu > 4) per_cu -= per_cu % 4;
        // Blocked convolutions keep a SIMD busy with few wavefronts, and with
        // fewer of them every task, and so the launch's last ones, end sooner.
        // Two and three per SIMD by convolution tasks (ms; four: three or worse):
        // two and four doubles 14687 7.08, 7.77, 28518 12.3, 12.6, 41154 18.1, 17.5,
        // 60987 26.2, 24.7; three 19212 5.40, 5.51, 27067 7.50, 7.46, 37609 10.2, 10.1;
        // five 14124 3.10, 3.30, 21203 4.57, 4.58, 30663 6.70, 6.62; four, of 4 to 12
        // variables, 16731 25.4, 25.6, 32612 49.8, 47.6.
        if (BLK) per_cu = std::min(per_cu, b->stage_tasks[1] >= 30000 ? 12 : 8);
        b->grid = std::max(1, per_cu) * cus;
    }
    return MDPE_OK;
}

template <int M1, int M2, bool BLK>
int launch_batch(mdpe_batch *b, hipStream_t st, bool prepare_only) {
    int rc = prepare_batch<M1, M2, BLK>(b);
    if (rc || prepare_only) return rc;
    hipLaunchKernelGGL(mdpe::batch_reset_kernel, dim3(1), dim3(64), 0, st, b->d_ctl, b->count + mdpe::kQueues + 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return bfail(MDPE_EDEVICE, std::string("batch_reset_kernel: ") + hipGetErrorString(e));
    hipLaunchKernelGGL((mdpe::batch_kernel<M1, M2, BLK>), dim3(b->grid), dim3(64), b->lds, st, b->d_tasks, b->d_qinfo,
                       b->d_insts, b->d_ctl);
    e = hipGetLastError();
    if (e != hipSuccess) return bfail(MDPE_EDEVICE, std::string("batch_kernel: ") + hipGetErrorString(e));
    return MDPE_OK;
}

int launch_any(mdpe_batch *b, hipStream_t st, bool prepare_only = false) {
#define MS(a, c) (b->m1 == (a) && b->m2 == (c))
    if (b->blocks) {
        if (MS(2, 2)) return launch_batch<2, 2, true>(b, st, prepare_only);
        if (MS(3, 3)) return launch_batch<3, 3, true>(b, st, prepare_only);
        if (MS(4, 4)) return launch_batch<4, 4, true>(b, st, prepare_only);
        if (MS(5, 5)) return launch_batch<5, 5, true>(b, st, prepare_only);
        if (MS(2, 4)) return launch_batch<2, 4, true>(b, st, prepare_only);
    }
    if (MS(1, 1)) return launch_batch<1, 1, false>(b, st, prepare_only);
    if (MS(2, 2)) return launch_batch<2, 2, false>(b, st, prepare_only);
    if (MS(3, 3)) return launch_batch<3, 3, false>(b, st, prepare_only);
    if (MS(4, 4)) return launch_batch<4, 4, false>(b, st, prepare_only);
    if (MS(5, 5)) return launch_batch<5, 5, false>(b, st, prepare_only);
    if (MS(8, 8)) return launch_batch<8, 8, false>(b, st, prepare_only);
    if (MS(10, 10)) return launch_batch<10, 10, false>(b, st, prepare_only);
    if (MS(2, 4)) return launch_batch<2, 4, false>(b, st, prepare_only);
#undef MS
    return bfail(MDPE_EUNSUPPORTED, "batch precisions must be all equal, or {2, 4}");
}

// ------------------------------------------------------- the tune cache --
// The autotuner writes JSON: {"<arch>": {"tiles": [{"m": .., "d": ..,
// "jobs_per_group": .., "groups_per_task": .., "add_items_per_task": ..}, ...],
// other keys ...}, ...}.  A small reader for exactly that much JSON.
struct JVal {
    enum Kind { kNull, kBool, kNum, kStr, kArr, kObj } kind = kNull;
    double num = 0;
    std::string str;
    std::vector<JVal> arr;
    std::vector<std::pair<std::string, JVal>> obj;
    const JVal *get(const std::string &k) const {
        for (auto &kv : obj)
            if (kv.first == k) return &kv.second;
        return nullptr;
    }
};

struct JReader {
    const char *p, *e;
    void ws() {
        while (p < e && (*p == ' ' || *p == '\n' || *p == '\r' || *p == '\t')) ++p;
    }
    bool lit(const char *w) {
        const size_t n = std::strlen(w);
        if ((size_t)(e - p) < n || std::strncmp(p, w, n) != 0) return false;
        p += n;
        return true;
    }
    bool string(std::string &out) {
        if (p >= e || *p != '"') return false;
        for (++p; p < e && *p != '"'; ++p) {
            if (*p == '\\') {
                if (++p >= e) return false;
                out.push_back(*p == 'n' ? '\n' : *p == 't' ? '\t' : *p);  // \uXXXX is not expected in a tune cache
            } else {
                out.push_back(*p);
            }
        }
        if (p >= e) return false;
        ++p;
        return true;
    }
    bool value(JVal &v, int depth) {
        if (depth > 32) return false;
        ws();
        if (p >= e) return false;
        if (*p == '{') {
            v.kind = JVal::kObj;
            ++p;
            ws();
            if (p < e && *p == '}') return ++p, true;
            for (;;) {
                ws();
                std::string k;
                if (!string(k)) return false;
                ws();
                if (p >= e || *p++ != ':') return false;
                JVal x;
                if (!value(x, depth + 1)) return false;
                v.obj.emplace_back(std::move(k), std::move(x));
                ws();
                if (p < e && *p == ',') { ++p; continue; }
                if (p < e && *p == '}') return ++p, true;
                return false;
            }
        }
        if (*p == '[') {
            v.kind = JVal::kArr;
            ++p;
            ws();
            if (p < e && *p == ']') return ++p, true;
            for (;;) {
                JVal x;
                if (!value(x, depth + 1)) return false;
                v.arr.push_back(std::move(x));
                ws();
                if (p < e && *p == ',') { ++p; continue; }
                if (p < e && *p == ']') return ++p, true;
                return false;
            }
        }
        if (*p == '"') {
            v.kind = JVal::kStr;
            return string(v.str);
        }
        if (lit("true") || lit("false")) return v.kind = JVal::kBool, true;
        if (lit("null")) return true;
        char *end = nullptr;
        std::string num(p, (size_t)std::min<ptrdiff_t>(e - p, 64));
        v.num = std::strtod(num.c_str(), &end);
        if (end == num.c_str()) return false;
        v.kind = JVal::kNum;
        p += end - num.c_str();
        return true;
    }
};

// Tiles for `arch` from the cache file at `path`; an absent arch key gives
// no tiles (the defaults).  Returns "" or an error message.
std::string read_tune_cache(const char *path, const std::string &arch, std::vector<mdpe_batch_tile> &tiles) {
    FILE *f = std::fopen(path, "rb");
    if (!f) return std::string("cannot read the tune cache ") + path;
    std::string text;
    char buf[4096];
    size_t got;
    while ((got = std::fread(buf, 1, sizeof buf, f)) > 0) {
        text.append(buf, got);
        if (text.size() > (16u << 20)) break;
    }
    std::fclose(f);
    JVal root;
    JReader r{text.data(), text.data() + text.size()};
    if (!r.value(root, 0) || root.kind != JVal::kObj) return std::string("tune cache ") + path + ": not a JSON object";
    const JVal *dev = root.get(arch);
    if (!dev) return "";
    const JVal *list = dev->kind == JVal::kObj ? dev->get("tiles") : nullptr;
    if (!list || list->kind != JVal::kArr) return std::string("tune cache ") + path + ": no tile list for " + arch;
    for (const JVal &t : list->arr) {
        auto field = [&](const char *k, bool need, int32_t &out) {
            const JVal *x = t.kind == JVal::kObj ? t.get(k) : nullptr;
            if (!x) return !need;
            if (x->kind != JVal::kNum || x->num < 0 || x->num > 1e9 || x->num != (double)(int64_t)x->num) return false;
            out = (int32_t)x->num;
            return true;
        };
        mdpe_batch_tile tile{0, 0, 0, 0, 0, 0};
        if (!field("m", true, tile.m) || !field("d", true, tile.d) || !field("jobs_per_group", false, tile.jobs_per_group) ||
            !field("groups_per_task", false, tile.groups_per_task) ||
            !field("add_items_per_task", false, tile.add_items_per_task) || !field("deal", false, tile.deal) ||
            tile.deal > 2)
            return std::string("tune cache ") + path + ": a tile needs integer m, d and tile fields (deal 0, 1 or 2)";
        tiles.push_back(tile);
    }
    return "";
}

// the device's architecture name without feature suffixes ("gfx950")
std::string device_arch(int device) {
    hipDeviceProp_t prop;
    if (device < 0 || hipGetDeviceProperties(&prop, device) != hipSuccess) return "gfx950";
    std::string a = prop.gcnArchName;
    const size_t c = a.find(':');
    return c == std::string::npos ? a : a.substr(0, c);
}

// capture [reset, persistent kernel] once on a private stream, replay on `stream`
int launch_graph_on(mdpe_batch *b, hipStream_t stream) {
    int rc = MDPE_OK;
    if (!b->exec) {
        if (!b->cap) BHIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
        rc = launch_any(b, b->cap, true);  // attributes and grid, outside the capture
        if (!rc) {
            BHIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
            rc = launch_any(b, b->cap);
            hipGraph_t g = nullptr;
            hipError_t e = hipStreamEndCapture(b->cap, &g);
            if (!rc && e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
            if (!rc) {
                b->graph = g;
                e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
                if (e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
            } else if (g) {
                (void)hipGraphDestroy(g);
            }
        }
    }
    if (!rc) {
        hipError_t e = hipGraphLaunch(b->exec, stream);
        if (e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("hipGraphLaunch: ") + hipGetErrorString(e));
    }
    return rc;
}

}  // namespace

// The batch's queue and device arrays; on failure the caller frees it.
static int make_batch(mdpe_batch *B, const mdpe_plan *const *plans, int count, const mdpe_batch_tile *tiles, int ntiles) {
    B->count = count;
    std::vector<int> ms;
    for (int p = 0; p < count; ++p) {
        if (!plans[p]) return bfail(MDPE_EINVAL, "NULL plan in the batch");
        const mdpe::Plan *P = &plans[p]->P;
        int dev = plans[p]->device;
        if (p == 0) B->device = dev;
        if (dev != B->device) return bfail(MDPE_EINVAL, "plans on different devices (or host-only mixed in)");
        if (P->complex_series()) return bfail(MDPE_EUNSUPPORTED, "batches hold real series only (MDPE_COMPLEX plan)");
        if (!P->scale.empty()) return bfail(MDPE_EUNSUPPORTED, "batches hold multilinear polynomials only (exponents)");
        if (P->streamed) return bfail(MDPE_EUNSUPPORTED, "batches stage operands in LDS (streamed-operand plan)");
        if (std::find(ms.begin(), ms.end(), P->m) == ms.end()) ms.push_back(P->m);
    }
    std::sort(ms.begin(), ms.end());
    if (ms.size() == 1) {
        B->m1 = B->m2 = ms[0];
    } else if (ms.size() == 2 && ms[0] == 2 && ms[1] == 4) {
        B->m1 = 2;
        B->m2 = 4;
    } else {
        return bfail(MDPE_EUNSUPPORTED, "batch precisions must be all equal, or {2, 4}");
    }
    auto tile_for = [&](int m, int d) {
        mdpe_batch_tile t{m, d, 0, 0, 0, 0};
        for (int q = 0; q < ntiles; ++q)
            if (tiles[q].m == m && tiles[q].d == d) t = tiles[q];
        if (t.jobs_per_group <= 0) t.jobs_per_group = mdpe::choose_jobs_per_group(d, m);
        return t;
    };
    // Convolutions by blocks at two to five doubles per coefficient, where
    // every instance meets what the blocked kernel needs (32-bit offsets;
    // second operands read from global memory not at the workspace's start;
    // a group's padded operands in LDS, its descriptors one per lane)
    B->blocks = ms[0] >= 2 && ms.back() <= 5;
    for (int p = 0; p < count && B->blocks; ++p) {
        const mdpe::Plan &P = plans[p]->P;
        const int J = tile_for(P.m, P.d).jobs_per_group;
        B->blocks = J <= mdpe::kLanes && mdpe::block_group_bytes(P.d + 1, P.m, mdpe::batch_terms(P.m), J) <=
                        mdpe::kMaxLdsBytes &&
                    mdpe::small_workspace(P) &&
                    (mdpe::stages_second_operand(P.m) || mdpe::reads_inside(P, P.conv, mdpe::batch_terms(P.m) - 1, 0));
    }
    // schedules per (d, J, terms an iteration)
    std::map<std::array<int, 3>, int> sched_index;
    std::vector<mdpe::LaneSchedule> scheds;
    // tasks with their depth and an instance cost for ordering
    struct Tmp {
        int queue;
        int depth;
        double cost;
        int order;
        mdpe::BatchTask t;
    };
    // estimated cost per instance (multiply-adds x limbs^2), then longest-first
    // assignment of instances to the XCD queues
    std::vector<double> icost(count);
    for (int p = 0; p < count; ++p) {
        const mdpe::Plan &P = plans[p]->P;
        const double d1 = P.d + 1;
        icost[p] = ((double)P.conv.size() * d1 * (d1 + 1) / 2 + (double)P.add.size() * d1) * P.m * P.m + d1;
    }
    std::vector<int> order_p(count);
    for (int p = 0; p < count; ++p) order_p[p] = p;
    std::stable_sort(order_p.begin(), order_p.end(), [&](int a, int c) { return icost[a] > icost[c]; });
    // An instance costing more than one queue's fair share (a batch of one, or
    // a few large instances) has its tasks dealt over all queues in turn, so it
    // runs on every XCD; the others keep one queue each, near one L2.
    double total = 0;
    for (double c : icost) total += c;
    std::vector<double> qload(mdpe::kQueues, 0.0);
    B->inst_queue.assign(count, 0);
    for (int p : order_p)
        if (icost[p] > total / mdpe::kQueues) {
            B->inst_queue[p] = -1;
            for (auto &l : qload) l += icost[p] / mdpe::kQueues;
        }
    for (int p : order_p) {
        if (B->inst_queue[p] < 0) continue;
        int best = 0;
        for (int q = 1; q < mdpe::kQueues; ++q)
            if (qload[q] < qload[best]) best = q;
        qload[best] += icost[p];
        B->inst_queue[p] = best;
    }
    // Each instance's convolution layers: the plan's, or, coefficient by coefficient,
    // of one made for the chain launch its jobs at their earliest layers (16
    // instances of 211 monomials of 1 to 12 variables, d = 37: eight doubles 11.19 ->
    // 9.47 ms, one 1.08 -> 1.07; by blocks one way or the other: sets of ragged
    // instances 0.90 of the time at four doubles, deep instances dealt over the
    // queues 1.06, 96 mixed ones of 4 to 20 variables 1.08).
    std::vector<std::vector<std::array<int32_t, 3>>> own_conv(count);
    std::vector<std::vector<int64_t>> own_off(count);
    for (int p = 0; p < count; ++p)
        if (!B->blocks && plans[p]->P.pipe_layers > 0 &&
            !mdpe::earliest_layers(plans[p]->P, own_conv[p], own_off[p])) {
            own_conv[p].clear();
            own_off[p].clear();
        }
    auto conv_of = [&](int p) -> const std::vector<std::array<int32_t, 3>> & {
        return own_off[p].empty() ? plans[p]->P.conv : own_conv[p];
    };
    auto off_of = [&](int p) -> const std::vector<int64_t> & {
        return own_off[p].empty() ? plans[p]->P.conv_off : own_off[p];
    };
    // Convolutions by component sets where a queue has a component for every
    // resident wavefront of its XCD (32 CUs x 8): a task then runs whole
    // components (monomials), its groups one after the other on one wavefront,
    // and no convolution waits for another task -- one stage instead of a
    // layer's after layer's, each with its release, acquire and idle
    // wavefronts, and the longest tasks first.  Smaller batches keep a stage per
    // layer: a component's products in sequence would be their critical path.
    std::vector<std::vector<int32_t>> comp(count);
    std::vector<int32_t> comps(count, 0);
    std::vector<long> queue_comps(mdpe::kQueues, 0);
    for (int p = 0; p < count && B->blocks; ++p) {
        if (B->inst_queue[p] < 0) continue;
        comps[p] = mdpe::job_components(plans[p]->P, comp[p]);
        queue_comps[B->inst_queue[p]] += comps[p];
    }
    // each instance's lane schedule, and each queue's convolution time: groups x
    // steps x the cost of a step (a component set's below, in the same unit)
    std::vector<int> sched_of(count);
    std::vector<double> queue_time(mdpe::kQueues, 0.0);
    auto step_cost = [&](const mdpe::Plan &P) { return mdpe::batch_terms(P.m) * P.m * P.m + 10.0; };
    for (int p = 0; p < count; ++p) {
        const mdpe::Plan &P = plans[p]->P;
        const int J = tile_for(P.m, P.d).jobs_per_group;
        const std::array<int, 3> key{P.d, J, B->blocks ? mdpe::batch_terms(P.m) : 0};
        if (!sched_index.count(key)) {
            sched_index[key] = (int)scheds.size();
            scheds.push_back(B->blocks ? mdpe::make_block_schedule(P.d, 1, mdpe::batch_terms(P.m), J, 1)
                                       : mdpe::make_lane_schedule(P.d, J));
        }
        sched_of[p] = sched_index[key];
        const auto &off = off_of(p);
        double groups = 0;
        for (size_t L = 1; L < off.size(); ++L) groups += (double)((off[L] - off[L - 1] + J - 1) / J);
        const double t = groups * scheds[sched_of[p]].steps * step_cost(P);
        if (B->inst_queue[p] >= 0)
            queue_time[B->inst_queue[p]] += t;
        else
            for (double &x : queue_time) x += t / mdpe::kQueues;
    }
    B->set_jobs.resize(count);
    B->set_groups.resize(count);
    std::vector<Tmp> tmp;
    B->insts.resize(count);
    // one workspace for all instances: each instance's part 256-byte aligned
    B->ws_off.resize(count);
    for (int p = 0; p < count; ++p) {
        const mdpe::Plan &P = plans[p]->P;
        B->ws_off[p] = B->ws_bytes;
        const int64_t bytes = P.n_series * (int64_t)(P.d + 1) * P.w * (int64_t)sizeof(double);
        B->ws_bytes += (bytes + 255) / 256 * 256;
    }
    size_t lds = 0;
    for (int p = 0; p < count; ++p) {
        const mdpe::Plan &P = plans[p]->P;
        const mdpe_batch_tile t = tile_for(P.m, P.d);
        const int J = t.jobs_per_group;
        const mdpe::LaneSchedule &S = scheds[sched_of[p]];
        const int terms = S.steps * (B->blocks ? mdpe::batch_terms(P.m) : 1);
        // a dealt instance finds its parallelism inside its own layers: one
        // group of jobs per task, small addition tasks
        const bool dealt = B->inst_queue[p] < 0;
        const int G = dealt ? 1 : t.groups_per_task > 0 ? t.groups_per_task : std::max(1, (256 + terms - 1) / terms);
        const long items_per_task = dealt ? 1024 : t.add_items_per_task > 0 ? t.add_items_per_task : 4096;
        lds = std::max(lds, (size_t)(B->blocks ? mdpe::block_group_bytes(P.d + 1, P.m, mdpe::batch_terms(P.m), J)
                                               : mdpe::group_lds_bytes(P.d + 1, mdpe::lds_doubles_per_coef(P.m), J)));
        if (lds > (size_t)mdpe::kMaxLdsBytes)
            return bfail(MDPE_EUNSUPPORTED, "a tile's jobs_per_group needs more LDS than one workgroup has");
        mdpe::BatchInst &I = B->insts[p];
        std::memset(&I, 0, sizeof(I));
        I.conv = plans[p]->d_conv;
        I.add = plans[p]->d_add;
        I.chunks = plans[p]->d_chunks;
        I.leaves = plans[p]->d_leaves;
        I.stage = plans[p]->d_stage;
        I.out = plans[p]->d_out;
        I.stride = S.stride;
        I.steps = S.steps;
        I.J = J;
        I.simple = P.m > 2 ? 0 : t.deal == 1 ? 0 : t.deal == 2 ? 1 : mdpe::prefer_simple_dealing(P.d, J, P.m, S.steps) ? 1 : 0;
        I.m = P.m;
        I.d = P.d;
        I.n = P.n;
        I.N = P.N;
        const int d1 = P.d + 1;
        const double cost = icost[p];
        const int queue = B->inst_queue[p];
        int depth = 0, done_before = 0, order = 0;
        auto emit = [&](int kind, long first, int cnt, int need) {
            const int q = queue >= 0 ? queue : (p + order) % mdpe::kQueues;
            tmp.push_back({q, depth, cost, order++, {p, kind, need, cnt, first, 0, 0}});
        };
        auto items = [&](int kind, long total) {
            int n = 0;
            for (long f = 0; f < total; f += items_per_task, ++n)
                emit(kind, f, (int)std::min(items_per_task, total - f), done_before);
            return n;
        };
        // stage
        done_before += items(0, (long)P.stage.size() * d1);
        ++depth;
        const auto &conv = conv_of(p);
        const auto &off = off_of(p);
        bool by_sets = !dealt && comps[p] > 0 && queue_comps[queue] >= mdpe::kSetComponents;
        if (by_sets) {
            // 2J components per set, so that a layer's jobs fill groups of J (a
            // tile may ask for more work per task), but two sets per wavefront
            // of the XCD
            const double per_comp = (double)conv.size() / comps[p];
            int cps = std::max(2 * J, (int)((double)t.groups_per_task * J / per_comp));
            cps = (int)std::max(1L, std::min((long)cps, queue_comps[queue] / (2 * mdpe::kSetComponents)));
            const int sets = (comps[p] + cps - 1) / cps, nl = (int)off.size() - 1;
            // components of like size in one set (a set's layers then fill their
            // groups: 0.97 to 0.99 of the places taken instead of 0.87 to 0.94),
            // the largest in the first
            {
                std::vector<int32_t> size(comps[p], 0), rank(comps[p]), order(comps[p]);
                for (int32_t c : comp[p]) ++size[c];
                for (int32_t c = 0; c < comps[p]; ++c) order[c] = c;
                std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t c) { return size[a] > size[c]; });
                for (int32_t r = 0; r < comps[p]; ++r) rank[order[r]] = r;
                for (int32_t &c : comp[p]) c = rank[c];
            }
            // counting sort by (set, layer)
            std::vector<int> at((size_t)sets * nl + 1, 0);
            for (int L = 1; L <= nl; ++L)
                for (int64_t j = off[L - 1]; j < off[L]; ++j) at[(size_t)(comp[p][j] / cps) * nl + L]++;
            for (size_t q = 1; q < at.size(); ++q) at[q] += at[q - 1];
            auto set_groups = [&](int s) {
                int g = 0;
                for (int L = 0; L < nl; ++L) g += (at[(size_t)s * nl + L + 1] - at[(size_t)s * nl + L] + J - 1) / J;
                return g;
            };
            // A set is a chain of dependent groups on one wavefront.  Where the
            // largest takes longer than the queue's work spread over the XCD's
            // wavefronts, and much longer than the layers one after the other
            // (with a task's groups each), the instance keeps a stage per layer.
            // Largest set against that work and against the layers, then time by
            // sets and by layers (ms): sets kept at 1.4 and 1.3 times 3.1, 3.8 (16
            // mixed instances), 2.5 and 1.3 times 4.4, 5.2 (32), 2.1 and 0.2 times
            // 1.0, 2.7 (16 of 211 monomials of 1 to 12 variables, four doubles);
            // layers kept at 3.9 and 2.7 times 2.3, 1.4, 7.2 and 2.5 times 6.4, 3.5,
            // 91 and 1.5 times 3.3, 2.4, 61 and 2.9 times 23.6, 9.1 (16 instances of
            // four monomials of 50 to 60 variables, d = 128, beside 120 small ones).
            long layered = 0;
            for (int L = 1; L <= nl; ++L)
                layered += std::min<long>(G, (off[L] - off[L - 1] + J - 1) / J);
            const double step = S.steps * step_cost(P), longest = set_groups(0) * step;
            by_sets = longest <= std::max(queue_time[queue] / mdpe::kSetComponents, mdpe::kSetOverLayers * layered * step);
            if (by_sets) {
                std::vector<int> to(at.begin(), at.end() - 1);
                auto &jobs = B->set_jobs[p];
                jobs.resize(conv.size());
                for (int L = 1; L <= nl; ++L)
                    for (int64_t j = off[L - 1]; j < off[L]; ++j)
                        jobs[to[(size_t)(comp[p][j] / cps) * nl + L - 1]++] =
                            make_int4(conv[j][0], conv[j][1], conv[j][2], 0);
                auto &groups = B->set_groups[p];
                for (int s = 0; s < sets; ++s) {
                    const int first = at[(size_t)s * nl], last = at[(size_t)(s + 1) * nl];
                    emit(1, first, last - first, done_before);
                    mdpe::BatchTask &T = tmp.back().t;
                    T.group = (int)groups.size();
                    T.groups = set_groups(s);
                    tmp.back().cost = T.groups * step;
                    for (int L = 0; L < nl; ++L)
                        for (int j = at[(size_t)s * nl + L]; j < at[(size_t)s * nl + L + 1]; j += J) groups.push_back(j);
                }
                groups.push_back((int)jobs.size());
                done_before += sets;
                ++depth;
            }
        }
        if (!by_sets && !own_off[p].empty())
            for (const auto &t : conv) B->set_jobs[p].push_back(make_int4(t[0], t[1], t[2], 0));
        for (int L = 1; !by_sets && L < (int)off.size(); ++L, ++depth) {
            const long a = off[L - 1], z = off[L];
            int n = 0;
            for (long f = a; f < z; f += (long)G * J, ++n) emit(1, f, (int)std::min((long)G * J, z - f), done_before);
            done_before += n;
        }
        // additions by passes over parts of the lists (plan's chunks), a task for
        // about add_items_per_task additions of coefficients
        const mdpe::AddPasses passes = B->blocks ? mdpe::make_add_passes(P, mdpe::add_pass_leaves(P.w)) : mdpe::AddPasses();
        const bool by_passes = B->blocks && (long)passes.chunks.size() * d1 < INT32_MAX;
        if (by_passes) {
            long done = 0;  // additions in the tasks so far: a task's `first` and `count` number them
            for (size_t q = 0; q + 1 < passes.off.size(); ++q) {
                const long lo = passes.off[q], hi = passes.off[q + 1];
                long adds = 0;
                for (long b = lo; b < hi; ++b) adds += std::max(0, passes.chunks[b].count - 1);
                if (adds == 0) continue;
                const long want = t.add_items_per_task > 0 ? t.add_items_per_task : 16384;
                const long per = std::max(64L, std::min(65536L, want * (hi - lo) / adds / 64 * 64));
                int n = 0;
                for (long f = lo * d1; f < hi * d1; f += per, ++n) {
                    const long e = std::min(f + per, hi * d1);
                    long cnt = 0;
                    for (long b = f / d1; b * d1 < e; ++b)
                        cnt += (std::min(e, (b + 1) * d1) - std::max(f, b * d1)) * std::max(0, passes.chunks[b].count - 1);
                    emit(2, done, (int)cnt, done_before);
                    tmp.back().t.group = (int)f;
                    tmp.back().t.groups = (int)(e - f);
                    done += cnt;
                }
                done_before += n;
                ++depth;
            }
        }
        if (B->blocks)
            for (size_t o = 0; o < P.out_slots.size(); ++o)
                B->outs.push_back(by_passes && P.list_off[o + 1] - P.list_off[o] >= 2 ? mdpe::kSummed : P.out_slots[o]);
        for (int r = 1; !by_passes && r <= P.n_levels(); ++r, ++depth) {
            const long a = P.add_off[r - 1] * d1, z = P.add_off[r] * d1;
            int n = 0;
            for (long f = a; f < z; f += items_per_task, ++n)
                emit(2, f, (int)std::min(items_per_task, z - f), done_before);
            done_before += n;
        }
        done_before += items(3, (long)(1 + P.n) * d1);
    }
    std::stable_sort(tmp.begin(), tmp.end(), [](const Tmp &a, const Tmp &b) {
        if (a.queue != b.queue) return a.queue < b.queue;
        if (a.depth != b.depth) return a.depth < b.depth;
        if (a.cost != b.cost) return a.cost > b.cost;
        if (a.t.inst != b.t.inst) return a.t.inst < b.t.inst;
        return a.order < b.order;
    });
    B->qinfo.assign(2 * mdpe::kQueues, 0);
    for (size_t q = 0; q < tmp.size(); ++q) {
        B->tasks.push_back(tmp[q].t);
        B->task_queue.push_back(tmp[q].queue);
        B->qinfo[mdpe::kQueues + tmp[q].queue]++;
    }
    for (int q = 1; q < mdpe::kQueues; ++q) B->qinfo[q] = B->qinfo[q - 1] + B->qinfo[mdpe::kQueues + q - 1];
    B->lds = lds;
    B->stage_tasks.assign(4, 0);
    for (auto &t : B->tasks) B->stage_tasks[t.kind]++;
    if (B->device < 0) return MDPE_OK;  // host-only batch: for inspecting the queue
    // device arrays
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(B->device));
    int rc = MDPE_OK;
    auto alloc_copy = [&](void **dst, const void *src, size_t bytes) -> int {
        BHIP(hipMalloc(dst, bytes ? bytes : 16));
        if (bytes) BHIP(hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice));
        return MDPE_OK;
    };
    for (auto &S : scheds) {
        int *dc = nullptr;
        if ((rc = alloc_copy((void **)&dc, S.chains.data(), S.chains.size() * sizeof(int)))) break;
        B->d_chains.push_back(dc);
    }
    if (!rc) {
        std::vector<int4> jobs;
        std::vector<int> groups;
        for (int p = 0; p < count; ++p) {
            jobs.insert(jobs.end(), B->set_jobs[p].begin(), B->set_jobs[p].end());
            groups.insert(groups.end(), B->set_groups[p].begin(), B->set_groups[p].end());
        }
        if (!jobs.empty() && !(rc = alloc_copy((void **)&B->d_set_jobs, jobs.data(), jobs.size() * sizeof(int4))))
            rc = alloc_copy((void **)&B->d_set_groups, groups.data(), groups.size() * sizeof(int));
    }
    if (!rc && B->blocks) rc = alloc_copy((void **)&B->d_outs, B->outs.data(), B->outs.size() * sizeof(int));
    if (!rc) {
        size_t jobs_at = 0, groups_at = 0, outs_at = 0;
        for (int p = 0; p < count; ++p) {
            const mdpe::Plan &P = plans[p]->P;
            if (B->blocks) {
                B->insts[p].out = B->d_outs + outs_at;
                outs_at += P.out_slots.size();
            }
            if (!B->set_jobs[p].empty()) {
                B->insts[p].conv = B->d_set_jobs + jobs_at;
                B->insts[p].goff = B->d_set_groups + groups_at;
                jobs_at += B->set_jobs[p].size();
                groups_at += B->set_groups[p].size();
            }
            B->insts[p].chains = B->d_chains[sched_of[p]];
        }
        if (!(rc = alloc_copy((void **)&B->d_tasks, B->tasks.data(), B->tasks.size() * sizeof(mdpe::BatchTask))) &&
            !(rc = alloc_copy((void **)&B->d_qinfo, B->qinfo.data(), B->qinfo.size() * sizeof(int))))
            if (!(rc = alloc_copy((void **)&B->d_insts, B->insts.data(), B->insts.size() * sizeof(mdpe::BatchInst)))) {
                // control words: zeroed by the reset kernel before every launch
                hipError_t e = hipMalloc((void **)&B->d_ctl, sizeof(int) * (size_t)(count + mdpe::kQueues + 1));
                if (e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("hipMalloc: ") + hipGetErrorString(e));
            }
    }
    for (int r = 0; !rc && r < mdpe_batch::kRing; ++r) {
        hipError_t e = hipHostMalloc((void **)&B->ring[r], sizeof(mdpe::BatchInst) * (size_t)count, hipHostMallocDefault);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&B->ring_ev[r], hipEventDisableTiming);
        if (e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("pinned pointer tables: ") + hipGetErrorString(e));
    }
    if (prev >= 0) (void)hipSetDevice(prev);
    return rc;
}

extern "C" {

int plan_batch(const mdpe_plan *const *plans, int count, const char *tune_cache, mdpe_batch **out) {
    if (!plans || !out || count <= 0) return bfail(MDPE_EINVAL, "plans, count > 0 and out are required");
    *out = nullptr;
    std::vector<mdpe_batch_tile> tiles;
    if (tune_cache && *tune_cache) {
        if (!plans[0]) return bfail(MDPE_EINVAL, "NULL plan in the batch");
        std::string err;
        try {
            err = read_tune_cache(tune_cache, device_arch(plans[0]->device), tiles);
        } catch (const std::bad_alloc &) {
            return bfail(MDPE_ENOMEM, "host allocation failed while reading the tune cache");
        }
        if (!err.empty()) return bfail(MDPE_EINVAL, err);
    }
    return plan_batch_tiles(plans, count, tiles.data(), (int)tiles.size(), out);
}

int plan_batch_tiles(const mdpe_plan *const *plans, int count, const mdpe_batch_tile *tiles, int ntiles,
                     mdpe_batch **out) {
    if (!plans || !out || count <= 0) return bfail(MDPE_EINVAL, "plans, count > 0 and out are required");
    if (ntiles < 0 || (ntiles > 0 && !tiles)) return bfail(MDPE_EINVAL, "bad tiles");
    for (int q = 0; q < ntiles; ++q)
        if (tiles[q].deal < 0 || tiles[q].deal > 2) return bfail(MDPE_EINVAL, "a tile's deal must be 0, 1 or 2");
    *out = nullptr;
    std::unique_ptr<mdpe_batch> B(new (std::nothrow) mdpe_batch());
    if (!B) return bfail(MDPE_ENOMEM, "host allocation failed");
    int rc;
    try {
        rc = make_batch(B.get(), plans, count, tiles, ntiles);
    } catch (const std::bad_alloc &) {
        rc = bfail(MDPE_ENOMEM, "host allocation failed while planning the batch");
    }
    if (rc) {
        std::string keep = mdpe::get_last_error();
        free_batch(B.release());
        mdpe::set_last_error(keep);
        return rc;
    }
    *out = B.release();
    return MDPE_OK;
}

int batch_info(const mdpe_batch *b, mdpe_batch_info *o) {
    if (!b || !o) return bfail(MDPE_EINVAL, "batch and out are required");
    o->count = b->count;
    o->n_tasks = (int64_t)b->tasks.size();
    o->n_conv_tasks = b->stage_tasks[1];
    o->n_add_tasks = b->stage_tasks[2];
    o->lds_bytes = (int64_t)b->lds;
    o->grid = b->grid;
    o->m1 = b->m1;
    o->m2 = b->m2;
    o->workspace_bytes = b->ws_bytes;
    return MDPE_OK;
}

int batch_tasks(const mdpe_batch *b, int32_t *rows) {
    if (!b || !rows) return bfail(MDPE_EINVAL, "batch and rows are required");
    for (size_t q = 0; q < b->tasks.size(); ++q) {
        const auto &t = b->tasks[q];
        rows[6 * q] = t.inst;
        rows[6 * q + 1] = t.kind;
        rows[6 * q + 2] = t.need;
        rows[6 * q + 3] = t.count;
        rows[6 * q + 4] = (int32_t)t.first;
        rows[6 * q + 5] = b->task_queue[q];
    }
    return MDPE_OK;
}

int batch_set_buffers(mdpe_batch *b, const double *const *coeff, const double *const *z, double *const *value,
                      double *const *grad, void *const *workspace) {
    if (!b || !coeff || !z || !value || !grad || !workspace) return bfail(MDPE_EINVAL, "NULL argument");
    if (b->device < 0) return bfail(MDPE_EINVAL, "host-only batch");
    for (int p = 0; p < b->count; ++p) {
        if (!coeff[p] || !z[p] || !value[p] || !grad[p] || !workspace[p])
            return bfail(MDPE_EINVAL, "NULL buffer for instance " + std::to_string(p));
        if (((uintptr_t)workspace[p]) % 256) return bfail(MDPE_EINVAL, "workspace must be 256-byte aligned");
        b->insts[p].A = (double *)workspace[p];
        b->insts[p].coeff = coeff[p];
        b->insts[p].z = z[p];
        b->insts[p].value = value[p];
        b->insts[p].grad = grad[p];
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(b->device));
    hipError_t e = hipMemcpy(b->d_insts, b->insts.data(), b->insts.size() * sizeof(mdpe::BatchInst),
                             hipMemcpyHostToDevice);
    if (prev >= 0) (void)hipSetDevice(prev);
    if (e != hipSuccess) return bfail(MDPE_EDEVICE, std::string("hipMemcpy: ") + hipGetErrorString(e));
    b->buffers_set = true;
    return MDPE_OK;
}

int batch_launch(mdpe_batch *b, void *stream) {
    if (!b) return bfail(MDPE_EINVAL, "batch is NULL");
    if (!b->buffers_set) return bfail(MDPE_EINVAL, "call batch_set_buffers first");
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(b->device));
    int rc = launch_any(b, (hipStream_t)stream);
    if (prev >= 0) (void)hipSetDevice(prev);
    return rc;
}

int batch_launch_graph(mdpe_batch *b, void *stream) {
    if (!b) return bfail(MDPE_EINVAL, "batch is NULL");
    if (!b->buffers_set) return bfail(MDPE_EINVAL, "call batch_set_buffers first");
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(b->device));
    int rc = launch_graph_on(b, (hipStream_t)stream);
    if (prev >= 0) (void)hipSetDevice(prev);
    return rc;
}

int eval_and_diff_batch(mdpe_batch *b, const double *const *coeff, const double *const *z, double *const *value,
                        double *const *grad, void *workspace, void *stream) {
    if (!b || !coeff || !z || !value || !grad || !workspace) return bfail(MDPE_EINVAL, "NULL argument");
    if (b->device < 0) return bfail(MDPE_EINVAL, "host-only batch");
    if (((uintptr_t)workspace) % 256) return bfail(MDPE_EINVAL, "workspace must be 256-byte aligned");
    bool changed = !b->buffers_set;
    for (int p = 0; p < b->count; ++p) {
        if (!coeff[p] || !z[p] || !value[p] || !grad[p])
            return bfail(MDPE_EINVAL, "NULL buffer for instance " + std::to_string(p));
    }
    for (int p = 0; p < b->count; ++p) {
        mdpe::BatchInst &I = b->insts[p];
        double *A = (double *)((char *)workspace + b->ws_off[p]);
        changed |= I.A != A || I.coeff != coeff[p] || I.z != z[p] || I.value != value[p] || I.grad != grad[p];
        I.A = A;
        I.coeff = coeff[p];
        I.z = z[p];
        I.value = value[p];
        I.grad = grad[p];
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(b->device));
    hipStream_t st = (hipStream_t)stream;
    int rc = MDPE_OK;
    if (changed) {
        // stream-ordered rebinding: the table goes through a pinned buffer
        // whose previous copy (kRing rebinds ago) has run by now, unless the
        // caller is more than kRing rebinds ahead of the device
        const int r = b->ring_next;
        b->ring_next = (r + 1) % mdpe_batch::kRing;
        hipError_t e = b->ring_used[r] ? hipEventSynchronize(b->ring_ev[r]) : hipSuccess;
        if (e == hipSuccess) {
            std::memcpy(b->ring[r], b->insts.data(), sizeof(mdpe::BatchInst) * (size_t)b->count);
            e = hipMemcpyAsync(b->d_insts, b->ring[r], sizeof(mdpe::BatchInst) * (size_t)b->count,
                               hipMemcpyHostToDevice, st);
        }
        if (e == hipSuccess) e = hipEventRecord(b->ring_ev[r], st);
        if (e != hipSuccess) rc = bfail(MDPE_EDEVICE, std::string("binding the pointer table: ") + hipGetErrorString(e));
        b->ring_used[r] = true;
        b->buffers_set = !rc;
    }
    if (!rc) rc = launch_graph_on(b, st);
    if (prev >= 0) (void)hipSetDevice(prev);
    return rc;
}

int batch_status(mdpe_batch *b) {
    if (!b) return bfail(MDPE_EINVAL, "batch is NULL");
    if (b->device < 0) return bfail(MDPE_EINVAL, "host-only batch");
    int flags[mdpe::kQueues + 1] = {0};
    int prev = -1;
    (void)hipGetDevice(&prev);
    BHIP(hipSetDevice(b->device));
    BHIP(hipDeviceSynchronize());
    hipError_t e = hipMemcpy(flags, b->d_ctl, sizeof(flags), hipMemcpyDeviceToHost);
    if (prev >= 0) (void)hipSetDevice(prev);
    if (e != hipSuccess) return bfail(MDPE_EDEVICE, std::string("hipMemcpy: ") + hipGetErrorString(e));
    if (flags[mdpe::kQueues]) return bfail(MDPE_EDEVICE, "batch watchdog: a task waited too long for its inputs");
    for (int q = 0; q < mdpe::kQueues; ++q)
        if (flags[q] < b->qinfo[mdpe::kQueues + q])
            return bfail(MDPE_EDEVICE, "batch queue " + std::to_string(q) + " was not drained (no wavefront ran on its XCD)");
    return MDPE_OK;
}

int batch_set_grid(mdpe_batch *b, int grid) {
    if (!b || grid < 0) return bfail(MDPE_EINVAL, "batch is NULL or grid < 0");
    if (b->exec) return bfail(MDPE_EINVAL, "the batch's graph is already captured");
    b->grid = grid;  // 0: resident capacity, resolved at the next launch
    b->grid_fixed = grid > 0;
    return MDPE_OK;
}

void batch_destroy(mdpe_batch *b) { free_batch(b); }

}  // extern "C"
