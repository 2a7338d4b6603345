// plan.hpp -- host-side data staging (Section 5 of the paper): series slots,
// convolution triplets per layer, addition pairs per level, output slots,
// hazard check and the lane schedule of the convolution kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <cstdint>
#include <string>
#include <vector>

namespace mdpe {

constexpr int kLanes = 64;             // one wavefront per convolution workgroup
constexpr int64_t kScratchBytes = 64ll << 20;  // workspace of the allocation-free entry
constexpr int kMaxLdsBytes = 163840;   // LDS one gfx950 workgroup may allocate
constexpr int kLdsBudget = 65536;      // LDS a workgroup aims to stay under (>= 2 per CU)
constexpr int kMaxExponent = 64;

struct LaneSchedule {
    int jobs_per_group = 1;            // J: convolution jobs staged per workgroup
    int waves_per_job = 1;             // Q: wavefronts sharing one job's coefficients (J = 1 when Q > 1)
    int steps = 0;                     // multiply-add steps of the busiest lane
    int stride = 0;                    // entries per lane in `chains`
    // chains[row*stride + s]: (job << 16) | k for the s-th output coefficient
    // schedule row `row` computes, -1 after its last one; row q*64 + lane is
    // lane `lane` of the q-th of the Q wavefronts of a group.
    std::vector<int32_t> chains;
};

// The convolution kernel stages both operands of a job in LDS when a
// coefficient is at most two doubles (short steps: the second operand's
// latency from L2 would dominate), else only the first.  Doubles of LDS per
// coefficient of a job:
__host__ __device__ constexpr bool stages_second_operand(int w) { return w <= 2; }
__host__ __device__ constexpr int lds_doubles_per_coef(int w) { return stages_second_operand(w) ? 2 * w : w; }

// A job's three series as offsets (in doubles) into A: first operand, second
// operand, output.  Kept in LDS, so that a lane starting a chain finds its
// operands' addresses with one LDS read and an add.
struct JobOffsets {
    long x, y, z, unused;
};

// LDS layout of one wavefront's group: X[J][d+1][W] doubles (the first
// operands), Y[J][d+1][W] (the second operands, only when
// stages_second_operand(W)), then the J JobOffsets (16-byte aligned).
// `doubles_per_coef` is lds_doubles_per_coef(W), or 0 for streamed operands.
__host__ __device__ inline long conv_lds_jobs_offset(long xdoubles) { return (xdoubles * 8 + 15) / 16 * 16; }
__host__ __device__ inline long group_lds_bytes(long d1, int doubles_per_coef, int J) {
    return conv_lds_jobs_offset((long)J * d1 * doubles_per_coef) + (long)J * (long)sizeof(JobOffsets);
}

// LDS layout of one wavefront's group of the blocked convolution (blocks of R
// coefficients per lane, conv_block.hpp): a front pad, X[J] series, Y[J]
// series (only when stages_second_operand(W)), an end pad of one block, then
// the J JobOffsets.  The pads hold what a top block reads past an operand.  A
// job's series start 2 doubles past a multiple of 32 (the 64 LDS banks), so
// that lanes of different jobs at one coefficient read different banks.
__host__ __device__ constexpr int block_front_pad(int w, int U) { return (U * w + 1) / 2 * 2; }
__host__ __device__ inline int block_series_stride(int d1, int w) { return (d1 * w + 31) / 32 * 32 + 2; }
__host__ __device__ inline long block_jobs_offset(int d1, int w, int U, int J) {  // in doubles
    return 2L * block_front_pad(w, U) + (long)J * (stages_second_operand(w) ? 2 : 1) * block_series_stride(d1, w);
}
__host__ __device__ inline long block_group_bytes(int d1, int w, int U, int J) {
    return block_jobs_offset(d1, w, U, J) * 8 + (long)J * 16;  // BlockJob
}

// LDS doubles of one first operand of the blocked chain launch: whole blocks.
__host__ __device__ constexpr int chain_slot_doubles(int d1, int w, int R) {
    return ((d1 + R - 1) / R * R * w + 1) / 2 * 2;
}
// LDS of a chain: B slots, one for the last job's blocks, the jobs' offsets.
__host__ __device__ constexpr long chain_lds_bytes(int d1, int w, int R, int B, int jobs) {
    return (B + 1L) * chain_slot_doubles(d1, w, R) * 8 + 16L * jobs;
}

constexpr uint32_t kKeepMonomialValues = 1u;
constexpr uint32_t kComplex = 2u;          // complex series: real limbs, then imaginary limbs
constexpr uint32_t kStreamOperands = 4u;   // read both convolution operands from global memory
constexpr uint32_t kStageOperands = 8u;    // stage them in LDS (no automatic streaming)
constexpr uint32_t kAsapLayers = 16u;      // every convolution at its earliest layer (no balancing)
constexpr uint32_t kFusedLayers = 32u;     // all convolution layers in one launch, per independent component
constexpr uint32_t kLayerLaunches = 64u;   // one launch per convolution layer (no automatic fusing)
constexpr uint32_t kChainLaunch = 128u;    // first-operand chains in one pipelined launch (see Plan::pipe_*)
constexpr uint32_t kNoChainLaunch = 256u;  // never the chain launch (the plan chooses the rest)
constexpr uint32_t kSingleLaunch = 512u;   // the whole evaluation in one launch of one workgroup
constexpr uint32_t kWideOffsets = 2048u;   // the kernels of workspaces of 4 GiB and more, whatever the size

// Chain launch: the code of an idle stretch in a lane's entry list (job field)
constexpr int32_t kIdleJob = 0x7FFF;    // codes stay positive; chain jobs are numbered below it
constexpr int kMaxChainLength = 2048;      // jobs of one chain (their descriptors sit in LDS)

// One chain of the chain launch: its jobs pipe_jobs[first .. first+len), its
// lane schedule at pipe_codes[code_off], `stride` entries per row, `steps`
// steps (a multiple of the barrier window).
struct ChainComp {
    int32_t first, len, code_off, stride, steps, pad0, pad1, pad2;
};

struct Plan {
    int n = 0, N = 0, d = 0, m = 0;
    int w = 0;                         // doubles per coefficient: m, or 2m for complex series
    uint32_t flags = 0;
    int64_t n_series = 0;
    // convolution jobs {t1, t2, t3} in launch order; layer L spans
    // conv[conv_off[L-1] .. conv_off[L])
    std::vector<std::array<int32_t, 3>> conv;
    std::vector<int64_t> conv_off;
    // addition jobs {t1, t2}: A[t2] += A[t1]; level r spans add[add_off[r-1] .. add_off[r])
    std::vector<std::array<int32_t, 2>> add;
    std::vector<int64_t> add_off;
    std::vector<int32_t> out_slots;    // [1+n]: value slot, then d/dz_i slot or -1
    // staging copies {slot, source}: source s < N+1 is coeff series s, else z series s-N-1
    std::vector<std::array<int32_t, 2>> stage;
    // general exponents: scale jobs {src, dst, e}, A[dst] := e * A[src] per
    // coefficient, run after the last convolution layer, before the additions
    std::vector<std::array<int32_t, 3>> scale;
    LaneSchedule lanes;
    // blocked convolutions (staged operands): the lane schedule of blocks of
    // block_r coefficients that the per-layer launches and the reverse pass
    // run (block_r = 0: the schedule `lanes`, coefficient by coefficient)
    int block_r = 0, block_u = 0;
    LaneSchedule blocks;
    // addition trees: the slots of each output's list (the value's, then each
    // derivative's) in tree order; list o spans list_slots[list_off[o] .. list_off[o+1])
    std::vector<int32_t> list_slots;
    std::vector<int64_t> list_off;
    // reverse pass (flags & kKeepMonomialValues): one layer of correlation jobs
    // {t1 = ybar slot, t2 = M_k or gradient slot, t3 = output slot}
    int32_t ybar_slot = -1;
    std::vector<std::array<int32_t, 3>> corr;
    std::vector<int32_t> coeff_bar_slots;   // [N+1]: ybar slot, then abar_k slots
    std::vector<int32_t> z_bar_slots;       // [n]: zbar_i slot or -1 (absent variable)

    bool complex_series() const { return (flags & kComplex) != 0; }
    // streamed operands: chosen when a job's operands would not fit in LDS, or
    // asked for; then no convolution writes its own first operand
    bool streamed = false;
    // staged coefficients of at most two doubles: deal coefficients to lanes
    // in turn instead of following the lane schedule (when estimated faster)
    bool simple = false;
    // jobs with slack moved to later layers to fill whole rounds of the SIMDs
    bool balanced = false;
    // fused layers (kFusedLayers, staged operands): the convolutions split into
    // independent components (no slot written by a job of one is read or
    // written by a job of another); fused_conv holds them by component, then
    // layer, and component c's layer L (1-based) spans
    // fused_conv[fused_off[c * (n_layers + 1) + L - 1] .. fused_off[c * (n_layers + 1) + L]).
    // One workgroup of fused_waves wavefronts runs a component, one job per
    // wavefront at a time, with the one-job lane schedule fused_lanes.
    std::vector<std::array<int32_t, 3>> fused_conv;
    std::vector<int32_t> fused_off;
    int32_t fused_components = 0;
    int32_t fused_waves = 0;
    LaneSchedule fused_lanes;
    bool fused_simple = false;
    // the fused launch by blocks: wavefronts of a workgroup (0: by coefficients) and the schedule
    int32_t fused_block_waves = 0;
    LaneSchedule fused_blocks;
    // Chain launch (kChainLaunch, or chosen by the cost model): chains of
    // convolutions where each job's first operand is the previous job's
    // output and its second a staged input series (p2's forward and backward
    // products).  Coefficient i of a product is final once its own i+1 terms
    // are summed, and the next product of the chain reads its first operand
    // in increasing i, so consecutive jobs of a chain overlap.  Layer
    // L <= pipe_layers holds the jobs at position L of their chain; one
    // launch runs them all, one workgroup of pipe_waves wavefronts per chain,
    // with a workgroup barrier every pipe_window steps; the layers after
    // pipe_layers launch one by one.
    // pipe_jobs: the chain jobs {t1, t2, t3}, chain after chain, in chain order;
    // pipe_comps: one per chain;
    // pipe_codes: per schedule (chains of one length share one), 64 *
    // pipe_waves rows of `stride` entries: (job << 16) | k for coefficient k
    // of the chain's job-th product (k+1 steps), or (kIdleJob << 16) | (g-1)
    // for g idle steps, then -1.
    // pipe_ring: LDS slots of first operands per chain (job j's in slot j mod pipe_ring).
    int pipe_layers = 0;
    // pipe_r > 0: by blocks of pipe_r coefficients, pipe_u terms an iteration
    // (chain.hip), block codes and iterations in place of coefficient codes and
    // steps.
    int pipe_waves = 0, pipe_window = 0, pipe_ring = 0, pipe_r = 0, pipe_u = 0;
    std::vector<std::array<int32_t, 3>> pipe_jobs;
    std::vector<ChainComp> pipe_comps;
    std::vector<int32_t> pipe_codes;
    // Single launch (kSingleLaunch, or chosen by the cost model for plans so
    // small that kernel boundaries dominate): one workgroup of single_waves
    // wavefronts runs staging, every convolution layer (single_lanes.jobs_per_group
    // jobs per wavefront and round), the scale stage, every addition level
    // and the gather, with a workgroup barrier after each.
    bool single = false;
    int single_waves = 0;
    LaneSchedule single_lanes;
    bool single_simple = false;
    int n_layers() const { return (int)conv_off.size() - 1; }
    int n_levels() const { return (int)add_off.size() - 1; }
};

// Returns "" on success, else a message; *unsupported distinguishes limits
// of this implementation from invalid input.
// exps: NULL (every exponent one) or [sum nvars] exponents in 1..kMaxExponent.
std::string build_plan(int n, int N, int d, int m, const int32_t *nvars, const int32_t *vars, const int32_t *exps,
                       uint32_t flags, Plan &out, bool *unsupported);

LaneSchedule make_lane_schedule(int d, int jobs_per_group, int waves_per_job = 1);
// The blocked convolution's schedule: items of R coefficients, U terms an
// iteration (R = 1, or R = U), `steps` in iterations.
LaneSchedule make_block_schedule(int d, int R, int U, int J, int Q);
LaneSchedule make_paired_schedule(int d, int waves_per_job);
// Streamed operands: wavefronts per job for degree d, and whether the paired
// schedule is used (large d, where first-fit would be slow to build).
int stream_waves_per_job(int d, bool *paired);
// Whether a group of J jobs of degree d with w doubles per coefficient is
// estimated faster dealt to the lanes in turn than by the lane schedule.
bool prefer_simple_dealing(int d, int J, int w, int schedule_steps);
// Steps of a group of J jobs of degree d dealt to the lanes of Q wavefronts in
// turn (the slowest wavefront's).
int dealt_steps(int d, int J, int Q = 1);
int choose_jobs_per_group(int d, int w);
// Leaves of one workgroup's part of an addition pass: 16 runs of the leaves that a
// thread sums in registers.
__host__ __device__ constexpr int add_run(int w) { return w <= 8 ? 8 : 4; }
constexpr int add_pass_leaves(int w) { return 16 * add_run(w); }
// One workgroup's part of an addition pass: the leaves
// leaves[first .. first+count) of one output's list.  out >= 0: the list's last
// pass, the sum is output `out` (0 = value, 1+i = d/dz_i); else the sum goes to
// the slot of the part's last leaf.
struct AddChunk {
    int32_t first, count, out, pad;
};
struct AddPasses {
    std::vector<int32_t> leaves;
    std::vector<AddChunk> chunks;
    std::vector<int64_t> off;  // pass p spans chunks[off[p] .. off[p+1])
};
// The pairwise trees of every output list cut into passes of parts of at most
// `cover` (a power of two) leaves: level r of a tree pairs whole runs of 2^r
// leaves, so a part's own tree is a subtree, its result stands where the
// level-by-level additions leave it, in its last leaf's slot, and the next
// pass runs over those slots.
AddPasses make_add_passes(const Plan &P, int cover);
// The independent component of every convolution job; returns their number.
int32_t job_components(const Plan &P, std::vector<int32_t> &comp);
// The convolutions of a chain launch's plan at their earliest layers, for an
// executor that runs layers: the plan's own put every chain's q-th product in layer
// q and all other products after the chains.  False where that order is not safe.
bool earliest_layers(const Plan &P, std::vector<std::array<int32_t, 3>> &conv, std::vector<int64_t> &off);
// What the blocked kernels need of a plan: 32-bit byte offsets into its
// workspace, and that `before` and `past` coefficients before and past every
// job's second operand lie inside it.
int block_terms_of(int w, int d);
// Wavefronts of the largest convolution launch of a plan run layer by layer (0:
// none is); more than any round where the SIMDs are uneven anyway: from eight doubles
// per coefficient on, and behind a chain launch that leaves them so.
long most_waves(const Plan &P);
bool lone_at(int w);
long most_after_chains(long largest, int chain_waves);
// Whether a launch of `waves` one-wavefront workgroups, in a plan whose largest has
// `most`, takes one wavefront per SIMD by register count (md.hpp, one_per_simd).
bool lone_launch(long most, long waves, int simds);
bool small_offsets(int64_t n_series, int64_t series_doubles);
bool small_workspace(const Plan &P);
bool reads_inside(const Plan &P, const std::vector<std::array<int32_t, 3>> &jobs, int before, int past);
// The rules every plan meets (Section 5: the jobs of one layer are
// independent): a job reads only slots written at an earlier stage (inputs,
// an earlier layer or level); no two jobs of a stage write one slot, and no
// job reads a slot another job of its stage writes; a convolution never
// writes its second operand, nor its first when operands are streamed or a
// job spans several wavefronts; output slots are written.  Returns "" or
// what is violated, naming the stage.
std::string check_hazards(const Plan &P);

// Chain launch schedule for one chain of L jobs of degree d on W wavefronts
// with a workgroup barrier every S steps and first operands in B LDS slots:
// codes (64W rows of *stride entries, the encoding of Plan::pipe_codes).
// Returns the steps (an even multiple of S).
// With U > 1 a coefficient's terms are taken U an iteration: coefficient k
// takes k / U + 1 iterations and reads x_i one iteration before its i / U-th.
int make_chain_schedule(int L, int d, int W, int S, int B, std::vector<int32_t> &codes, int *stride, int U = 1);
// Checks a chain schedule against the kernel's timing: every coefficient of
// every job exactly once, within `steps`; the first operand of step t is read
// from LDS in iteration t-1 (the prologue, iteration -1, for step 0), a
// coefficient's result is stored in the iteration of its last step, and a
// barrier follows every iteration s with (s+1) % S == 0.  Every read of a
// job's first operand must come after the barrier that follows the store of
// that coefficient by the previous job, and before the barrier that precedes
// its overwriting (B slots later).  Returns "" or what is wrong.
std::string check_chain_schedule(int L, int d, int W, int S, int B, int steps, const int32_t *codes, int stride,
                                 int U = 1);

}  // namespace mdpe
