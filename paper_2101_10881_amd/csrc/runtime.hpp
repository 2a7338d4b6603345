// runtime.hpp -- the plan object behind the C ABI and the per-thread error
// message, shared by the per-layer runtime (kernels.hip) and the batched
// executor (batch.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <string>
#include <vector>

#include "plan.hpp"

// devices whose per-device state (kernel attributes, SIMD counts) is cached
constexpr int kMaxDevices = 64;

struct mdpe_plan {
    mdpe::Plan P;
    int device = -1;
    void *d_arena = nullptr;   // the one device allocation that holds the arrays below
    int4 *d_conv = nullptr;
    int2 *d_add = nullptr;
    int2 *d_stage = nullptr;
    int *d_out = nullptr;
    int *d_chains = nullptr;
    int4 *d_corr = nullptr;
    int *d_cbar = nullptr;
    int *d_zbar = nullptr;
    int *d_ybar = nullptr;
    int4 *d_scale = nullptr;
    int4 *d_fconv = nullptr;   // fused layers: jobs by component, then layer
    int *d_foff = nullptr;     // fused layers: per-component layer offsets
    int *d_fchains = nullptr;  // fused layers: the one-job lane schedule
    int4 *d_pjobs = nullptr;   // chain launch: jobs chain after chain
    mdpe::ChainComp *d_pcomps = nullptr;  // chain launch: one per chain
    int *d_pcodes = nullptr;   // chain launch: lane schedules
    int *d_coff = nullptr;     // single launch: convolution layer offsets (int32)
    int *d_aoff = nullptr;     // single launch: addition level offsets (int32)
    int *d_blocks = nullptr;   // blocked convolutions: their lane schedule
    int *d_fblocks = nullptr;  // fused blocked convolutions: their lane schedule
    int *d_leaves = nullptr;   // addition passes: list slots
    mdpe::AddChunk *d_chunks = nullptr;  // addition passes: workgroups' parts
    long most_waves = 0;       // mdpe::most_waves(P)
    std::vector<int64_t> add_pass;       // pass p spans d_chunks[add_pass[p] .. add_pass[p+1])
    int *d_schains = nullptr;  // single launch: the lane schedule of its job groups
};

// launchers of the other translation units (each returns an MDPE_* status and
// leaves its message for last_error_string)
namespace mdpe {
// One layer of jobs as blocked convolutions (block_r > 0) on `st`.
int launch_block_layer(const mdpe_plan *pl, bool corr, double *A, const int4 *jobs, int nj, hipStream_t st);
// Every layer in one launch as blocked convolutions (fused_block_waves > 0).
int launch_block_fused(const mdpe_plan *pl, double *A, hipStream_t st);
// The chain launch by blocks (pipe_r > 0).
int launch_block_chain(const mdpe_plan *pl, double *A, hipStream_t st);
// Pass p of the plan's addition trees; the last pass of a list writes the
// caller's value or gradient.
int launch_add_pass(const mdpe_plan *pl, int p, double *A, double *value, double *grad, hipStream_t st);
int simd_count(int device);
}  // namespace mdpe

namespace mdpe {
void set_last_error(const std::string &msg);
const std::string &get_last_error();
}  // namespace mdpe
