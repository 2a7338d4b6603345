// plan.cpp -- the data staging algorithm of Section 5 of the paper.
//
// Slots (one slot = one series of d+1 coefficients; slot s starts at
// s*(d+1) in the paper's array A, Fig. 1):
//   a_0 = 0, a_k = k (k = 1..N), z_i = N + i (i = 1..n),
//   f_{k,j} = 1+N+n + alpha_k + j-1,
//   b_{k,j} = 1+N+n + alpha_{N+1} + beta_k + j-1,
//   c_{k,j} = 1+N+n + alpha_{N+1} + beta_{N+1} + gamma_k + j-1,
// with alpha, beta, gamma the prefix sums of n_l, max(1, n_l-2), max(0, n_l-2)
// (Section 5; the slot count is e/(d+1) of eq. (6)).
//
// Convolution jobs per monomial (Section 3, statement list and eq. (2);
// Section 5, steps 1-7) with the readings: forward chain by z_{i_j};
// c_j = f_j * b_{n-2-j} at layer max(j, n-2-j)+1; b_{n-2} := b_{n-2} * a and
// c_{n-2} = f_{n-2} * z_{i_n} at layer n-1; n = 2: b_1 = z_{i_2} * a; n = 1:
// the derivative is a_k itself, copied into its b slot at staging time.
//
// Addition jobs: per output list a pairwise tree, adjacent pairs with the odd
// element carried, the later element updated (Section 5, the addition
// recursion, read through the worked example after eq. (5)).
//
// General exponents (Section 3): a table of powers z_i^p := z_i^{p-1} * z_i,
// the common factor a_k * prod z^(e-1) in front of the monomial's jobs, and a
// scale stage (A[dst] := e * A[src]) for the partial derivatives.  Streamed
// operands (degrees beyond one workgroup's LDS, or estimated faster): no job
// writes its own first operand, and a job may span several wavefronts.
#include "plan.hpp"

#include <cmath>
#include <limits>

#include <algorithm>
#include <numeric>
#include <unordered_map>

namespace mdpe {

static bool supported_m(int m) { return m == 1 || m == 2 || m == 3 || m == 4 || m == 5 || m == 8 || m == 10; }

int choose_jobs_per_group(int d, int w) {
    // Enough jobs per wavefront that the average lane load, J(d+1)(d+2)/2/64,
    // covers the longest output coefficient (d+1 multiply-adds); within the
    // LDS budget.
    int need = (2 * kLanes + (d + 2) - 1) / (d + 2);
    need = std::max(1, std::min(need, kLanes));
    long per_job = (long)(d + 1) * lds_doubles_per_coef(w) * 8;
    long cap = std::max(1L, (long)kLdsBudget / per_job);
    return (int)std::max(1L, std::min((long)need, cap));
}

// J jobs of `lengths.size()` items each (item k takes lengths[k] steps,
// nondecreasing in k) over the lanes of Q wavefronts.
static LaneSchedule pack_items(const std::vector<int> &lengths, int J, int Q) {
    // Assign the items (output coefficients: coefficient k costs k+1
    // multiply-adds; or blocks of them) to the 64*Q lanes of Q wavefronts: first-fit-decreasing
    // into lanes of capacity C, for the smallest C >= max(ceil(total/lanes),
    // d+1) that fits.  Each coefficient stays whole on one lane, so its
    // operation order is the specified one whatever lane computes it.
    LaneSchedule s;
    s.jobs_per_group = J;
    s.waves_per_job = Q;
    const int lanes = kLanes * Q;
    std::vector<std::pair<int, int>> items;  // (length, code)
    long total = 0;
    for (int j = 0; j < J; ++j)
        for (size_t k = 0; k < lengths.size(); ++k) {
            items.push_back({lengths[k], (j << 16) | (int)k});
            total += lengths[k];
        }
    std::stable_sort(items.begin(), items.end(), [](auto &a, auto &b) { return a.first > b.first; });
    std::vector<long> load;
    std::vector<std::vector<int32_t>> lists;
    for (long cap = std::max((total + lanes - 1) / lanes, (long)lengths.back());; ++cap) {
        load.assign(lanes, 0);
        lists.assign(lanes, {});
        bool ok = true;
        for (auto &it : items) {
            int l = 0;
            while (l < lanes && load[l] + it.first > cap) ++l;
            if (l == lanes) {
                ok = false;
                break;
            }
            load[l] += it.first;
            lists[l].push_back(it.second);
        }
        if (ok) break;
    }
    size_t stride = 1;
    for (auto &l : lists) stride = std::max(stride, l.size() + 1);
    s.stride = (int)stride;
    s.steps = (int)*std::max_element(load.begin(), load.end());
    s.chains.assign((size_t)lanes * stride, -1);
    for (int l = 0; l < lanes; ++l)
        for (size_t q = 0; q < lists[l].size(); ++q) s.chains[(size_t)l * stride + q] = lists[l][q];
    return s;
}

LaneSchedule make_lane_schedule(int d, int J, int Q) {
    std::vector<int> lengths(d + 1);
    std::iota(lengths.begin(), lengths.end(), 1);
    return pack_items(lengths, J, Q);
}

LaneSchedule make_block_schedule(int d, int R, int U, int J, int Q) {
    std::vector<int> lengths;
    for (int k = 0; k <= d; k += R) lengths.push_back(k / U + 1);
    return pack_items(lengths, J, Q);
}

LaneSchedule make_paired_schedule(int d, int Q) {
    // One job over the 64*Q lanes of Q wavefronts for large d: coefficients k
    // and d-k (k+1 and d-k+1 terms, d+2 together) share a lane, one pair per
    // lane; the middle coefficient of an even d is alone.  Q*64 must be at
    // least the number of pairs, ceil((d+1)/2).
    LaneSchedule s;
    s.jobs_per_group = 1;
    s.waves_per_job = Q;
    const int lanes = kLanes * Q;
    s.stride = 3;
    s.chains.assign((size_t)lanes * 3, -1);
    int steps = 0;
    for (int k = 0, l = 0; k <= d - k; ++k, ++l) {
        s.chains[(size_t)l * 3] = d - k;                    // the longer coefficient first
        if (k != d - k) s.chains[(size_t)l * 3 + 1] = k;
        steps = std::max(steps, (d - k + 1) + (k != d - k ? k + 1 : 0));
    }
    s.steps = steps;
    return s;
}

int stream_waves_per_job(int d, bool *paired) {
    const int pairs = (d + 2) / 2;
    *paired = d + 1 > 4096;
    if (*paired) return (pairs + kLanes - 1) / kLanes;
    return std::max(1, pairs / kLanes);
}

int dealt_steps(int d, int J, int Q) {
    // steps of dealing J*(d+1) coefficients to the 64*Q lanes of Q wavefronts
    // in turn (item t to lane t mod 64Q): each round of 64 items of a
    // wavefront costs its longest coefficient; the slowest wavefront counts
    const long items = (long)J * (d + 1);
    long worst = 0;
    for (int q = 0; q < Q; ++q) {
        long steps = 0;
        for (long r = (long)q * kLanes; r < items; r += (long)kLanes * Q) {
            int longest = 0;
            for (long t = r; t < std::min(items, r + kLanes); ++t) longest = std::max(longest, (int)(t % (d + 1)) + 1);
            steps += longest;
        }
        worst = std::max(worst, steps);
    }
    return (int)std::min(worst, (long)INT32_MAX);
}

bool prefer_simple_dealing(int d, int J, int w, int schedule_steps) {
    // a dealt step costs about 0.15 (w = 1) or 0.4-0.5 (w = 2) schedule steps
    // (measured on p2 at d = 152; 0.5 keeps the marginal cases of the batched
    // configuration on the schedule)
    if (w > 2) return false;
    return dealt_steps(d, J) * (w == 1 ? 0.15 : 0.5) < schedule_steps;
}

// Pairwise tree over `items`; pushes the jobs of round r into rounds[r].
static int tree_rounds(std::vector<int32_t> live, std::vector<std::vector<std::array<int32_t, 2>>> &rounds) {
    int r = 0;
    while (live.size() > 1) {
        if ((int)rounds.size() <= r) rounds.emplace_back();
        std::vector<int32_t> next;
        size_t pairs = live.size() / 2;
        for (size_t p = 0; p < pairs; ++p) {
            rounds[r].push_back({live[2 * p], live[2 * p + 1]});
            next.push_back(live[2 * p + 1]);
        }
        if (live.size() % 2) next.push_back(live.back());
        live.swap(next);
        ++r;
    }
    return live.empty() ? -1 : live[0];
}

AddPasses make_add_passes(const Plan &P, int cover) {
    AddPasses a;
    a.off.push_back(0);
    struct List {
        int out;
        std::vector<int32_t> slots;
    };
    std::vector<List> lists;
    for (size_t o = 0; o + 1 < P.list_off.size(); ++o)
        lists.push_back({(int)o, std::vector<int32_t>(P.list_slots.begin() + P.list_off[o],
                                                      P.list_slots.begin() + P.list_off[o + 1])});
    while (!lists.empty()) {
        std::vector<List> left;
        for (auto &L : lists) {
            const int n = (int)L.slots.size(), base = (int)a.leaves.size();
            a.leaves.insert(a.leaves.end(), L.slots.begin(), L.slots.end());
            if (n <= cover) {
                a.chunks.push_back({base, n, L.out, 0});
                continue;
            }
            List up{L.out, {}};
            for (int f = 0; f < n; f += cover) {
                const int c = std::min(cover, n - f);
                a.chunks.push_back({base + f, c, -1, 0});
                up.slots.push_back(L.slots[f + c - 1]);
            }
            left.push_back(std::move(up));
        }
        a.off.push_back((int64_t)a.chunks.size());
        lists.swap(left);
    }
    return a;
}

std::string check_hazards(const Plan &P) {
    // Each slot's last writer stage: inputs at stage 0, conv layer L at stage
    // L, addition level r at stage n_layers + r.  A job may read a slot only
    // when it was written at an earlier stage, and two jobs of one stage may
    // not touch a slot that one of them writes.
    std::vector<int> written(P.n_series, -1);
    for (int s = 0; s < 1 + P.N + P.n; ++s) written[s] = 0;
    for (auto &c : P.stage) written[c[0]] = 0;
    auto stage_check = [&](int stage, const std::vector<std::array<int32_t, 3>> &jobs) -> std::string {
        std::unordered_map<int32_t, int> writer;
        for (size_t q = 0; q < jobs.size(); ++q) {
            int32_t w = jobs[q][2];
            // the second operand of a convolution is streamed while outputs are
            // written, so it may never be the job's own output
            const bool conv_stage = stage <= P.n_layers() || stage > P.n_layers() + 1 + P.n_levels();
            if (conv_stage && jobs[q][1] == w) return "second operand is the output";
            // nor the first one when it is streamed, or when a job spans several
            // wavefronts (each stages it on its own, not necessarily before
            // another wavefront of the job stores)
            if (conv_stage && (P.streamed || P.lanes.waves_per_job > 1) && jobs[q][0] == w)
                return "first operand is the output (streamed, or a job over several wavefronts)";
            if (w < 0 || w >= P.n_series) return "slot out of range";
            if (!writer.emplace(w, (int)q).second) return "two jobs write one slot";
        }
        for (size_t q = 0; q < jobs.size(); ++q)
            for (int r = 0; r < 2; ++r) {
                int32_t s = jobs[q][r];
                if (s < 0 || s >= P.n_series) return "slot out of range";
                auto it = writer.find(s);
                if (it != writer.end() && it->second != (int)q) return "read of a slot written in the same stage";
                if (written[s] < 0 || written[s] >= stage) return "read before write";
            }
        for (auto &j : jobs) written[j[2]] = stage;
        return "";
    };
    for (int L = 1; L <= P.n_layers(); ++L) {
        std::vector<std::array<int32_t, 3>> jobs(P.conv.begin() + P.conv_off[L - 1], P.conv.begin() + P.conv_off[L]);
        auto e = stage_check(L, jobs);
        if (!e.empty()) return "conv layer " + std::to_string(L) + ": " + e;
    }
    {
        // the scale stage: job {src, dst, e} reads src and writes dst
        std::vector<std::array<int32_t, 3>> jobs;
        for (auto &c : P.scale) {
            if (c[2] < 2 || c[2] > kMaxExponent) return "scale job with a bad exponent";
            jobs.push_back({c[0], c[0], c[1]});
        }
        auto e = stage_check(P.n_layers() + 1, jobs);
        if (!e.empty()) return "scale stage: " + e;
    }
    for (int r = 1; r <= P.n_levels(); ++r) {
        std::vector<std::array<int32_t, 3>> jobs;
        for (int64_t q = P.add_off[r - 1]; q < P.add_off[r]; ++q) jobs.push_back({P.add[q][0], P.add[q][1], P.add[q][1]});
        auto e = stage_check(P.n_layers() + 1 + r, jobs);
        if (!e.empty()) return "add level " + std::to_string(r) + ": " + e;
    }
    for (auto s : P.out_slots)
        if (s >= 0 && written[s] < 0) return "output slot never written";
    if (!P.corr.empty() || P.ybar_slot >= 0) {
        const int stage = P.n_layers() + P.n_levels() + 2;
        written[P.ybar_slot] = stage - 1;  // staged before the reverse layer
        auto e = stage_check(stage, P.corr);
        if (!e.empty()) return "reverse layer: " + e;
    }
    return "";
}

static std::string build_plan_mode(int n, int N, int d, int m, const int32_t *nvars, const int32_t *vars,
                                   const int32_t *exps, uint32_t flags, bool stream, bool no_inplace, Plan &P,
                                   bool *unsupported);

// Relative cost of a layer plan: each layer takes about ceil(wavefronts /
// SIMDs) wavefront lifetimes (a SIMD's throughput hardly depends on how many
// wavefronts share it), a streamed step costing ~1.2 staged steps (p1 10d: 15.2
// vs 12.9 ms at equal steps).
constexpr long kSimds = 1024;  // MI355X: 256 CUs x 4 SIMDs

static double layer_cost(const Plan &P, int waves_per_job, int jobs_per_group, int steps, double step_cost,
                         int from_layer = 1) {
    double c = 0;
    for (int L = from_layer; L <= P.n_layers(); ++L) {
        const long jobs = P.conv_off[L] - P.conv_off[L - 1];
        const long waves = (jobs + jobs_per_group - 1) / jobs_per_group * waves_per_job;
        c += std::ceil(waves / (double)kSimds) * steps * step_cost;
    }
    return c;
}

// Staged operands: jobs per wavefront J and wavefronts per job Q for the
// layers from_layer.. (the others are launched otherwise).
static void choose_staged_lanes(Plan &P, int from_layer) {
    const int d = P.d, w = P.w;
    // Candidates, by the layer cost model: J jobs per wavefront by the lane
    // schedule (J0 halved down to 1), one job over Q = 2..4 wavefronts,
    // and for coefficients of at most two doubles the same J dealt to the
    // lanes in turn (steps weighted by their lower cost).  Fewer jobs per
    // wavefront or several wavefronts per job pay when layers have fewer
    // wavefronts than the chip has SIMDs (deep chains such as p2).
    // (A candidate replaces the default only when estimated 10% faster: the
    // model ignores staging and per-wavefront costs, e.g. p2 4d d = 64's two jobs
    // per wavefront measure 4% faster than one although it predicts the
    // opposite.)  Dealt steps weigh 0.15 (m = 1) or 0.4 (m = 2): measured
    // on p2 at d = 152.
    const int J0 = choose_jobs_per_group(d, w);
    double best = -1;
    auto consider = [&](LaneSchedule &&ls, bool simple, double c) {
        if (best < 0 || c < 0.9 * best) {
            best = c;
            P.lanes = std::move(ls);
            P.simple = simple;
        }
    };
    for (int J = J0;; J /= 2) {
        LaneSchedule ls = make_lane_schedule(d, J);
        const double c = layer_cost(P, 1, J, ls.steps, 1.0, from_layer);
        if (w <= 2) {
            const double sc = layer_cost(P, 1, J, dealt_steps(d, J), w == 1 ? 0.15 : 0.4, from_layer);
            if (sc < c) {
                consider(std::move(ls), true, sc);
                if (J == 1) break;
                continue;
            }
        }
        consider(std::move(ls), false, c);
        if (J == 1) break;
    }
    for (int Q = 2; Q <= 4 && d + 1 >= kLanes; ++Q) {
        LaneSchedule ls = make_lane_schedule(d, 1, Q);
        const double c = layer_cost(P, Q, 1, ls.steps, 1.0, from_layer);
        consider(std::move(ls), false, c);
    }
    // one job's coefficients dealt over Q wavefronts (deep chains of small
    // layers, such as p2, at one or two doubles per coefficient)
    for (int Q = 2; Q <= 4 && w <= 2 && d + 1 > (Q - 1) * kLanes; ++Q)
        consider(make_lane_schedule(d, 1, Q), true, layer_cost(P, Q, 1, dealt_steps(d, 1, Q), w == 1 ? 0.15 : 0.4, from_layer));
}

// FP64 instructions of one multiply-add of the plan's number field.
static long md_instr(bool mul, int m);
static long mac_instr(const Plan &P) {
    const long mul = md_instr(true, P.m), add = md_instr(false, P.m);
    return P.complex_series() ? 4 * mul + 4 * add : mul + add;
}

// Cycles of one iteration of the blocked convolution (R coefficients, U terms)
// with k wavefronts on a SIMD: the FP64 instructions, the selects of first and
// dropped terms and ~40 instructions of addresses and item switch, 4.4 cycles
// each, for every wavefront (measured: two or more wavefronts issue one
// instruction every 4.4 to 5 cycles between them, a lone one every 7, 6 and 5.5
// cycles at R = 1, 2 and 4), and a lone one also waits for its operands.
static double block_iteration(const Plan &P, int R, int U, double k, double lone1 = 1.5) {
    const int w = P.w;
    const double instr = (double)R * U * mac_instr(P) + 2.0 * w * R + (R == 1 ? 2.0 * w * (U - 1) : 1.0 * w * R * (R - 1)) +
                         1.0 * U * w + 40;
    const double lone = R == 1 ? lone1 : R == 2 ? 1.4 : 1.25, share = R > 1 ? 1.0 : k < 3 ? 1.08 : 1.04;
    return std::max(4.4 * instr * share * k, 4.4 * instr * lone + 350);
}

static double block_cost(const Plan &P, int R, int U, const LaneSchedule &ls, int from_layer) {
    double c = 0;
    for (int L = from_layer; L <= P.n_layers(); ++L) {
        const long jobs = P.conv_off[L] - P.conv_off[L - 1];
        const long waves = (jobs + ls.jobs_per_group - 1) / ls.jobs_per_group * ls.waves_per_job;
        c += ls.steps * block_iteration(P, R, U, (double)((waves + kSimds - 1) / kSimds));
    }
    return c;
}

// The blocked kernels address the workspace by 32-bit byte offsets.
bool small_offsets(int64_t n_series, int64_t series_doubles) { return n_series * series_doubles * 8 <= 0xffff0000LL; }
bool small_workspace(const Plan &P) {
    return !(P.flags & kWideOffsets) && small_offsets(P.n_series, (int64_t)(P.d + 1) * P.w);
}

// Whether reading `before` and `past` coefficients before and past the second
// operand of every job stays inside the workspace.
bool reads_inside(const Plan &P, const std::vector<std::array<int32_t, 3>> &jobs, int before, int past) {
    for (const auto &t : jobs)
        if ((int64_t)t[1] * (P.d + 1) < before || (P.n_series - 1 - t[1]) * (int64_t)(P.d + 1) < past) return false;
    return true;
}

// Whether the staged launches of width w and degree d run blocks.  Against the
// coefficient-by-coefficient kernel (p1, d = 8 / 31 / 63 / 95 / 152, wall time):
// two doubles per coefficient 1.27 / 0.99 / 1.33 / 1.18 / 1.31 times as fast,
// three 1.51 / 1.10 / 1.18 / 1.13 / 1.10, four 1.39 / 1.04 / 1.09 / 1.06 / 1.05,
// five 1.30 / 1.02 / 1.04 / 1.02 / 0.98, eight 1.09 / 1.00 / 0.99 / 0.98 / 0.99:
// what blocks save is the ~60 instructions a step spends around its
// arithmetic, 1124 instructions at eight doubles, where the other kernel's
// overlap of a product with the sum before it is worth more.  Up to d = 16 blocks
// win from six doubles on too (six to ten, layers of 4 to 6000 jobs: 0.98 to 2.2
// times as fast), but at eight doubles and even degrees from 12 on, whose last
// iteration is padded, not in layers of a few lone wavefronts (4 products of two
// variables: d = 12, 14, 16 0.96, 0.96, 0.98; 60 of three 1.00, 1.03, 0.99; 2000
// 1.13, 0.98, 1.14).  One double: d = 32 / 64 / 100 / 128 / 152 / 191 by the largest
// layer's jobs, 4200 0.96 / 1.14 / 0.88 / 1.16 / 1.07 / 0.86, 5000 0.99 / 1.13 /
// 0.94 / 1.25 / 1.15 / 0.95, 6000 1.29 / 1.17 / 1.14 / 1.31 / 1.23 / 1.01, 6400 1.19
// / 1.10 / 1.02 / 1.23 / 1.16 / 1.01: from six rounds of the SIMDs.
static bool blocks_pay(const Plan &P) {
    if (P.streamed || !small_workspace(P)) return false;
    long most = 0;
    for (int L = 1; L <= P.n_layers(); ++L) most = std::max(most, (long)(P.conv_off[L] - P.conv_off[L - 1]));
    if (P.m == 8 && P.w == 8 && P.d >= 12 && P.d % 2 == 0 && most <= 16) return false;
    if (P.w > 1) return P.w <= 4 || (P.w == 5 && P.d <= 127) || P.d <= 16;
    return most > 6144;
}

// Terms an iteration of the blocked per-layer and fused launches takes: four
// keep more independent products in flight, but an item's last iteration is
// padded to them.  Four against two (p1 / p3, wall time): three doubles per
// coefficient 0.97 times as fast at d = 8, 0.98 at 12, 1.00 at 16, 1.04 at 24,
// 1.10 at 31, 1.05 at 63 and 152; four 0.95 at d = 8, 0.97 at 20, 1.01 at 24,
// 1.05 at 31, 1.03 at 63, 1.22 on p3's d = 120; five 0.95, 0.99, 1.02, 1.00,
// 1.02, with exponents 1.11.  Up to two doubles always four (six and eight: 0.92
// to 1.06).
int block_terms_of(int w, int d) { return w <= 2 || (w <= 5 && d >= 24) ? 4 : 2; }

long most_waves(const Plan &P) {
    if (P.single || P.streamed || P.fused_components > 0) return 0;
    const LaneSchedule &ls = P.block_r > 0 ? P.blocks : P.lanes;
    long most = 0;
    for (int L = P.pipe_layers + 1; L <= P.n_layers(); ++L)
        most = std::max<long>(most, (P.conv_off[L] - P.conv_off[L - 1] + ls.jobs_per_group - 1) / ls.jobs_per_group *
                                        (long)ls.waves_per_job);
    if (P.pipe_layers > 0) return most_after_chains(most, P.pipe_waves);
    return lone_at(P.w) ? std::numeric_limits<long>::max() : most;
}

bool lone_at(int w) { return w >= 8; }

long most_after_chains(long largest, int chain_waves) {
    return chain_waves >= 2 ? std::numeric_limits<long>::max() : largest;
}

// A plan's launches all do or none does: a launch without it goes on from wherever
// the last workgroups of the one before fell.
// - A launch of more than a round leaves them unevenly, in this evaluation for the
//   next or for the first of the next one (1820 products of four of sixteen
//   variables, ten doubles, d = 31: the first layer, 910 wavefronts, 160 us with it
//   and 278 without; five doubles, d = 63: the last one 58 and 92).  Two streams
//   gain too (eight doubles, d = 95: 5044 and 5450 us for two evaluations).
// - So does a chain launch of two wavefronts or more per chain for the layers behind
//   it (100 chains of 16, five doubles, d = 20, two wavefronts: 84 us with it and 95
//   without, two streams 108 and 121; 183 of 12, three doubles, d = 27, 56 and 60, 71
//   and 77; 29 of 24, five doubles, d = 57, four wavefronts, two streams 295 and
//   339).  One wavefront per chain leaves them even (13 plans, 1.00), and two
//   streams lose (317 of 17, ten doubles, d = 8: 408 us without it, 536 with).
// - From eight doubles on the placement within a round is not always even either
//   (817 monomials of one to four variables, eight doubles, d = 87: 1127 us with it
//   and 1350 without; ten, d = 141, 411 of two or three: 1970 and 2537; 10 plans
//   1.00), and two streams gain (13 plans, 0.83 to 1.05 of the time, 0.92 together).
// - Below eight doubles it is even up to a round (45 workloads, 0.99 to 1.01 of the
//   time), and it would keep two streams' launches from sharing SIMDs: two
//   evaluations with it and without, 330 products of four of eleven variables at
//   five doubles, d = 63, 342 and 302 us, at four, d = 95, 307 and 267; 631 of two
//   to six variables at two, d = 76, 129 and 100.
// - Up to half a round two streams' launches fit beside each other, and it puts
//   them there: eight and ten doubles, launches of 210 to 495, 0.77 to 0.96 of the
//   time of two streams without it.
// Not below a quarter of the SIMDs, which leave idle ones whatever the placement.
bool lone_launch(long most, long waves, int simds) {
    return waves > simds / 4 && waves <= simds && (most > simds || most <= simds / 2);
}

// Blocks of R coefficients per lane, U terms an iteration, for the staged
// per-layer launches (conv_block.hpp) of the layers from_layer..., J jobs per
// wavefront and Q wavefronts per job, by the estimated cycles of the layers.
// One coefficient and block_terms_of terms; four coefficients and terms too at
// one double, where loads count (p1 d = 152: 1.13 against 0.94 times the other
// kernel's speed).  Tiles of 2 x 2 measured 0.74 to 0.98 on p1 at three and four
// doubles, 1.07 at best (p3): they halve the wavefronts.
static void choose_block_lanes(Plan &P, int from_layer) {
    P.block_r = P.block_u = 0;
    P.blocks = LaneSchedule();
    if (!blocks_pay(P)) return;
    const int w = P.w;
    const int maxq = P.lanes.waves_per_job > 1 ? 4 : 1;
    // candidates with the least a schedule of theirs can cost: its items fill the
    // lanes, and the longest runs whole on one
    struct Cand {
        double bound;
        int R, U, J, Q;
    };
    std::vector<Cand> cands;
    for (int R : {1, 4}) {
        const int U = block_terms_of(w, P.d);
        if (R == 4 && w > 1) continue;
        // second operands in global memory are read up to U - 1 coefficients
        // before (one coefficient's terms, going down) or past their slot
        // (blocks of R; the reverse pass's shared operand)
        if (!stages_second_operand(w) && !(reads_inside(P, P.conv, R == 1 ? U - 1 : 0, R == 1 ? 0 : U - 1) &&
                                           reads_inside(P, P.corr, 0, U - 1)))
            continue;
        const long longest = P.d / U + 1, items = P.d / R + 1;
        long all = 0;  // a job's iterations
        for (int k = 0; k <= P.d; k += R) all += k / U + 1;
        for (int J : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64}) {
            if (block_group_bytes(P.d + 1, w, U, J) > kLdsBudget && J > 1) break;
            if (block_group_bytes(P.d + 1, w, U, J) > kMaxLdsBytes) break;
            if ((long)(J - 1) * items * (longest + 1) / 2 > (long)kLanes * (longest + 1)) break;
            for (int Q = 1; Q <= (J == 1 ? maxq : 1); ++Q) {
                LaneSchedule least;
                least.jobs_per_group = J;
                least.waves_per_job = Q;
                least.steps = (int)std::max((J * all + kLanes * Q - 1) / (kLanes * Q), longest);
                cands.push_back({block_cost(P, R, U, least, from_layer), R, U, J, Q});
            }
        }
    }
    std::stable_sort(cands.begin(), cands.end(), [](const Cand &a, const Cand &b) { return a.bound < b.bound; });
    double best = -1;
    for (const Cand &c : cands) {
        if (best >= 0 && c.bound >= best) break;
        LaneSchedule ls = make_block_schedule(P.d, c.R, c.U, c.J, c.Q);
        const double cost = block_cost(P, c.R, c.U, ls, from_layer);
        if (best < 0 || cost < best) {
            best = cost;
            P.blocks = std::move(ls);
            P.block_r = c.R;
            P.block_u = c.U;
        }
    }
}

// The fused launch by blocks: J of a component's at most `widest` jobs per
// wavefront and as many wavefronts as that takes.
static void choose_fused_blocks(Plan &P, int widest) {
    P.fused_block_waves = 0;
    // p1, against one job per wavefront by coefficients: two doubles 1.07 times as
    // fast at d = 8, 1.21 at d = 31, 0.95 at d = 63; one double 0.57 to 0.9; 210
    // products of four of ten variables at three to five doubles 1.10 to 1.18
    if (P.w == 1 || P.w > 5 || (P.w == 2 && P.d > 40) || !blocks_pay(P) || widest < 1) return;
    const int U = block_terms_of(P.w, P.d);
    if (!stages_second_operand(P.w) && !reads_inside(P, P.conv, U - 1, 0)) return;
    double best = -1;
    for (int waves = 1; waves <= 4; ++waves) {
        const int J = std::min((widest + waves - 1) / waves, 16);
        if (waves * ((block_group_bytes(P.d + 1, P.w, U, J) + 15) / 16 * 16) > kMaxLdsBytes) continue;
        LaneSchedule ls = make_block_schedule(P.d, 1, U, J, 1);
        const int rounds = (widest + waves * J - 1) / (waves * J);
        const double k = std::min(8.0, std::max(1.0, (double)P.fused_components * waves / kSimds));
        const double c = rounds * ls.steps * block_iteration(P, 1, U, k) * std::max(1.0, (double)P.fused_components * waves / kSimds / 8.0);
        if (best < 0 || c < best) {
            best = c;
            P.fused_blocks = std::move(ls);
            P.fused_block_waves = waves;
        }
    }
}

// Layer balancing.  The layering above puts every convolution at its
// earliest layer; many jobs have slack (b_1 of a four-variable monomial is
// needed only by b_2, c_1 by nothing but the additions), and any layering
// that keeps each job after the jobs it depends on gives the same bits.  A
// layer costs about ceil(wavefronts / SIMDs) rounds, so the pass moves jobs
// with slack to later layers until each layer but the last fills whole rounds
// of `per_round` jobs where it can (p1: 3640/5460/5460/1820 jobs, 18 rounds
// of 1024, become 3072/4096/6144/3068, 16 rounds).  The depth stays the same.
//
// Dependencies come from slot accesses in the old layer order: a job depends
// on the last writer of each slot it reads (read after write), on the last
// writer of the slot it writes (write after write) and on every job that read
// that slot since (write after read; a job's in-place read of its own output
// is no dependency).  latest[j] is the last layer j can take with its
// dependants still fitting below the depth.  Layer by layer, the ready jobs
// (all dependencies placed earlier) are taken least slack first, then by
// their old order: all whose latest layer this is, and beyond them as many
// whole rounds as the ready jobs fill (or the rest of the round the
// mandatory ones start).  Within a layer jobs keep their old relative order.
// Returns false (P unchanged) if nothing moved.
static bool balance_layers(Plan &P, long per_round) {
    const int D = P.n_layers();
    const long nj = (long)P.conv.size();
    if (D < 2 || nj == 0 || per_round < 1) return false;
    std::vector<int> old_layer(nj);
    for (int L = 1; L <= D; ++L)
        for (int64_t j = P.conv_off[L - 1]; j < P.conv_off[L]; ++j) old_layer[j] = L;
    // edges (from, to) with from in an earlier old layer than to
    std::vector<std::pair<int, int>> edges;
    std::vector<int> last_writer(P.n_series, -1);
    std::vector<int> reader_head(P.n_series, -1);  // readers since the last write, as linked lists
    std::vector<int> reader_job, reader_next;
    for (int L = 1; L <= D; ++L) {
        const long lo = P.conv_off[L - 1], hi = P.conv_off[L];
        for (long j = lo; j < hi; ++j) {
            const auto &t = P.conv[j];
            for (int r = 0; r < 2; ++r)
                if (last_writer[t[r]] >= 0) edges.push_back({last_writer[t[r]], (int)j});
            if (last_writer[t[2]] >= 0) edges.push_back({last_writer[t[2]], (int)j});
            for (int q = reader_head[t[2]]; q >= 0; q = reader_next[q])
                if (reader_job[q] != (int)j) edges.push_back({reader_job[q], (int)j});
        }
        for (long j = lo; j < hi; ++j)
            for (int r = 0; r < 2; ++r) {
                const int32_t s = P.conv[j][r];
                if (r == 1 && s == P.conv[j][0]) continue;
                reader_job.push_back((int)j);
                reader_next.push_back(reader_head[s]);
                reader_head[s] = (int)reader_job.size() - 1;
            }
        for (long j = lo; j < hi; ++j) {
            last_writer[P.conv[j][2]] = (int)j;
            reader_head[P.conv[j][2]] = -1;
        }
    }
    // successor lists (CSR)
    std::vector<int> sbeg(nj + 1, 0), succ(edges.size()), npred(nj, 0);
    for (auto &e : edges) {
        if (old_layer[e.first] >= old_layer[e.second]) return false;  // not a valid layering: leave it
        sbeg[e.first + 1]++;
        npred[e.second]++;
    }
    for (long j = 0; j < nj; ++j) sbeg[j + 1] += sbeg[j];
    {
        std::vector<int> fill(sbeg.begin(), sbeg.end() - 1);
        for (auto &e : edges) succ[fill[e.first]++] = e.second;
    }
    std::vector<int> latest(nj, D);
    for (long j = nj - 1; j >= 0; --j)
        for (int q = sbeg[j]; q < sbeg[j + 1]; ++q) latest[j] = std::min(latest[j], latest[succ[q]] - 1);
    std::vector<int> layer(nj, 0), ready, next;
    std::vector<int64_t> keys;
    for (long j = 0; j < nj; ++j)
        if (npred[j] == 0) ready.push_back((int)j);
    long placed = 0;
    for (int L = 1; L <= D; ++L) {
        // (latest, job) packed in one key: cheaper to sort than by look-ups
        keys.resize(ready.size());
        for (size_t q = 0; q < ready.size(); ++q) keys[q] = (int64_t)latest[ready[q]] << 32 | (int64_t)ready[q];
        std::sort(keys.begin(), keys.end());
        for (size_t q = 0; q < ready.size(); ++q) ready[q] = (int)(keys[q] & 0x7fffffff);
        const long nr = (long)ready.size();
        long mand = 0;
        while (mand < nr && latest[ready[mand]] <= L) ++mand;
        long take = nr;
        if (L < D) {
            const long whole = nr / per_round * per_round;
            take = whole >= mand ? whole : std::min(nr, (mand + per_round - 1) / per_round * per_round);
            if (take == 0) take = nr;
        }
        next.clear();
        for (long q = 0; q < nr; ++q) {
            const int j = ready[q];
            if (q >= take) {
                next.push_back(j);
                continue;
            }
            layer[j] = L;
            ++placed;
            for (int s = sbeg[j]; s < sbeg[j + 1]; ++s)
                if (--npred[succ[s]] == 0) next.push_back(succ[s]);
        }
        ready.swap(next);
    }
    if (placed != nj || !ready.empty()) return false;
    bool moved = false;
    for (long j = 0; j < nj; ++j) moved |= layer[j] != old_layer[j];
    if (!moved) return false;
    std::vector<std::array<int32_t, 3>> conv;
    conv.reserve(nj);
    std::vector<int64_t> off{0};
    for (int L = 1; L <= D; ++L) {
        for (long j = 0; j < nj; ++j)
            if (layer[j] == L) conv.push_back(P.conv[j]);
        off.push_back((int64_t)conv.size());
    }
    P.conv.swap(conv);
    P.conv_off.swap(off);
    return true;
}

// Independent components of the convolutions.  Two jobs depend on each other
// only through a slot that some convolution writes (the staged inputs a_k and
// z_i are read-only), so a union of every job's output slot with each operand
// slot that is also written puts every read after write, write after write and
// write after read pair in one component.  Numbered by their first job.
int32_t job_components(const Plan &P, std::vector<int32_t> &comp) {
    const size_t nj = P.conv.size();
    std::vector<int64_t> parent(P.n_series);
    for (int64_t s = 0; s < P.n_series; ++s) parent[s] = s;
    auto find = [&](int64_t s) {
        while (parent[s] != s) s = parent[s] = parent[parent[s]];
        return s;
    };
    std::vector<char> written(P.n_series, 0);
    for (const auto &t : P.conv) written[t[2]] = 1;
    for (const auto &t : P.conv)
        for (int o = 0; o < 2; ++o)
            if (written[t[o]]) {
                const int64_t a = find(t[o]), b = find(t[2]);
                if (a != b) parent[a] = b;
            }
    std::vector<int32_t> comp_of_root(P.n_series, -1);
    comp.resize(nj);
    int32_t C = 0;
    for (size_t j = 0; j < nj; ++j) {
        const int64_t r = find(P.conv[j][2]);
        if (comp_of_root[r] < 0) comp_of_root[r] = C++;
        comp[j] = comp_of_root[r];
    }
    return C;
}

// Fused layers: the jobs by independent component; the layers inside a
// component keep the plan's order.
// Returns the most jobs of one component in one layer (0 if nothing was fused).
static int fuse_layers(Plan &P) {
    const int nl = P.n_layers();
    const size_t nj = P.conv.size();
    if (nl < 1 || nj == 0) return 0;
    std::vector<int32_t> comp;
    const int32_t C = job_components(P, comp);
    std::vector<int> layer(nj);
    for (int L = 1; L <= nl; ++L)
        for (int64_t j = P.conv_off[L - 1]; j < P.conv_off[L]; ++j) layer[j] = L;
    // counting sort by (component, layer), stable inside each bucket
    std::vector<int32_t> cnt((size_t)C * (nl + 1) + 1, 0);
    for (size_t j = 0; j < nj; ++j) cnt[(size_t)comp[j] * (nl + 1) + layer[j]]++;
    int widest = 0;
    for (int32_t x : cnt) widest = std::max(widest, (int)x);
    P.fused_off.assign((size_t)C * (nl + 1), 0);
    int32_t acc = 0;
    for (int32_t c = 0; c < C; ++c) {
        P.fused_off[(size_t)c * (nl + 1)] = acc;
        for (int L = 1; L <= nl; ++L) {
            acc += cnt[(size_t)c * (nl + 1) + L];
            P.fused_off[(size_t)c * (nl + 1) + L] = acc;
        }
    }
    std::vector<int32_t> pos(P.fused_off);
    P.fused_conv.assign(nj, {0, 0, 0});
    for (size_t j = 0; j < nj; ++j) {
        const size_t key = (size_t)comp[j] * (nl + 1) + layer[j] - 1;
        P.fused_conv[pos[key]++] = P.conv[j];
    }
    P.fused_components = C;
    P.fused_lanes = make_lane_schedule(P.d, 1);
    P.fused_simple = prefer_simple_dealing(P.d, 1, P.w, P.fused_lanes.steps);
    // up to four wavefronts (one per SIMD of a CU); the launcher lowers this
    // where their LDS would not fit
    P.fused_waves = std::min(4, std::max(1, widest));
    choose_fused_blocks(P, widest);
    return widest;
}

static void unfuse(Plan &P) {
    P.fused_conv.clear();
    P.fused_off.clear();
    P.fused_components = P.fused_waves = 0;
    P.fused_lanes = LaneSchedule();
    P.fused_simple = false;
    P.fused_block_waves = 0;
    P.fused_blocks = LaneSchedule();
}

// Fuse the layers by default where each layer is a short step that the per-layer
// kernel boundary (~4.5 us on MI355X) would dominate: deep plans, one
// wavefront per job, and either small layers (under half a round of the
// SIMDs) at small coefficients or low degree, or coefficients of one double
// (two up to d = 63).  Measured, fused against per-layer: p2 (64 layers of
// 378 jobs) 3.9x at one double and d = 8, 1.7x at d = 63, 1.5x at two doubles
// and d = 63, 1.0x at four doubles and d = 63-95, 1.2x at ten doubles and
// d = 8, slower beyond (ten doubles at d = 31: 0.95x); p1 (4 layers of
// 3072-6144 jobs) 1.14-1.2x at one double, 1.12-1.13x at two up to d = 63,
// 0.99x at d = 152, 0.87x at four doubles and d = 8.  Slower too wherever the
// plan spreads a job over several wavefronts or packs many short jobs into one
// (p3 at d = 8: 0.2x).  On p2 beyond four doubles (wall time): five doubles
// 1.17x at d = 15, 1.0x at d = 31; ten doubles 1.14x at d = 15, 1.05x at
// d = 31; eight doubles 1.2x at d = 8 but 0.99x at d = 15 and 0.89x at d = 31
// (the other widths take eight doubles' limit).  The caller also requires
// every component's layer to fit one round of four wavefronts.  By blocks and with
// addition passes on both sides 147 of 167 random plans of 4 to 8 layers still take
// the faster one within 6%; the line is off where layers run blocks and the fused
// launch does not (eight and ten doubles up to d = 16: 1.08 to 1.15 times as slow
// fused) and at layers of more than 512 short products (three to five doubles, d = 2
// to 8: up to 1.44 by layers).
static bool fuse_by_default(const Plan &P) {
    if (P.streamed || P.lanes.waves_per_job != 1 || P.n_layers() < 4) return false;
    if (P.w == 1 || (P.w == 2 && P.d <= 63)) return true;
    for (int L = 1; L <= P.n_layers(); ++L)
        if (P.conv_off[L] - P.conv_off[L - 1] > 512) return false;
    return P.d <= (P.w <= 4 ? 127 : (P.w == 5 || P.w == 10) ? 31 : 8);
}

// ------------------------------------------------------------ chain launch
// Timing of the chain kernel (conv_chain_kernel): every lane of a chain's
// workgroup runs the same steps.  The first operand of step t is read from
// LDS in iteration t-1 (in the prologue, iteration -1, for t = 0); a
// coefficient is stored -- to A and, for the chain's next product, to the LDS
// slot of that product's first operand -- in the iteration of its last step;
// a workgroup barrier follows iteration s when (s+1) % S == 0.  A store and a
// read of one LDS coefficient are therefore ordered exactly when their
// windows floor(iteration / S) differ.

static inline int chain_window(int it, int S) { return it >= 0 ? it / S : -1; }

// The lanes of a chain's workgroup by the iteration from which they are free:
// an ascending list per iteration and a bit per iteration that has one.
class FreeLanes {
  public:
    explicit FreeLanes(int lanes) : next_(lanes) {
        for (int q = lanes - 1; q >= 0; --q) put(0, q);
    }
    // the first lane of the latest iteration up to `at`, else of the earliest one
    std::pair<int, int> take(int at) {
        int t = last_up_to(at);
        if (t < 0) t = first_from(at + 1);
        const int q = head_[t];
        if ((head_[t] = next_[q]) < 0) bits_[t >> 6] &= ~(1ull << (t & 63));
        return {t, q};
    }
    void put(int t, int q) {
        if (t >= (int)head_.size()) {
            head_.resize(t / 64 * 64 + 64, -1);
            bits_.resize(head_.size() / 64, 0);
        }
        int *at = &head_[t];
        while (*at >= 0 && *at < q) at = &next_[*at];
        next_[q] = *at;
        *at = q;
        bits_[t >> 6] |= 1ull << (t & 63);
        latest_ = std::max(latest_, t);
    }
    int latest() const { return latest_; }

  private:
    int last_up_to(int t) const {
        t = std::min(t, (int)head_.size() - 1);
        for (int w = t >> 6; w >= 0; --w) {
            const uint64_t x = w == t >> 6 ? bits_[w] & (~0ull >> (63 - (t & 63))) : bits_[w];
            if (x) return 64 * w + 63 - __builtin_clzll(x);
        }
        return -1;
    }
    int first_from(int t) const {
        for (int w = t >> 6;; ++w) {  // (every lane is in some list)
            const uint64_t x = w == t >> 6 ? bits_[w] & (~0ull << (t & 63)) : bits_[w];
            if (x) return 64 * w + __builtin_ctzll(x);
        }
    }
    std::vector<int> head_, next_;
    std::vector<uint64_t> bits_;
    int latest_ = 0;
};

// The iterations of make_chain_schedule's schedule, and its lists when `lists`
// is not null.
static int place_chain(int L, int d, int W, int S, int B, int U, std::vector<std::vector<int32_t>> *lists) {
    // Jobs in chain order, each job's coefficients longest first; each at the
    // earliest step its first operand allows (every x_i read after the window
    // of its store by the previous job; its own store into the LDS slot of
    // job l+1 after the last read of the product that slot held, B jobs
    // earlier), on the lane free by then with the least idle time before it,
    // else on the lane that frees first.
    const int lanes = kLanes * W, d1 = d + 1;
    FreeLanes lane_free(lanes);
    if (lists) lists->assign(lanes, {});
    std::vector<int> store(d1, 0), ready(d1);  // (store: the previous job's)
    std::vector<int> last_read(L, -1);
    for (int l = 0; l < L; ++l) {
        // ready[k]: the earliest start of coefficient k by its first operand
        for (int k = 0; k <= d; ++k) {
            ready[k] = k > 0 ? ready[k - 1] : 0;
            if (l > 0) ready[k] = std::max(ready[k], S * (chain_window(store[k], S) + 1) - k / U + 1);
        }
        const bool reuses = l + 1 < L && l + 1 - B >= 0;
        const int from_slot = reuses ? S * (chain_window(last_read[l + 1 - B], S) + 1) : 0;
        for (int k = d; k >= 0; --k) {
            const int s0 = reuses ? std::max(ready[k], from_slot - k / U) : ready[k];
            const auto [from, lane] = lane_free.take(s0);
            const int start = std::max(s0, from);
            if (lists) {
                auto &list = (*lists)[lane];
                for (int g = start - from; g > 0;) {
                    const int q = std::min(g, 0x10000);
                    list.push_back((kIdleJob << 16) | (q - 1));
                    g -= q;
                }
                list.push_back((l << 16) | k);
            }
            lane_free.put(start + k / U + 1, lane);
            store[k] = start + k / U;
            last_read[l] = std::max(last_read[l], start + k / U - 1);
        }
    }
    // a multiple of the window, and even (the kernel may run two steps per iteration)
    const int q = S % 2 ? 2 * S : S;
    return (lane_free.latest() + q - 1) / q * q;
}

int make_chain_schedule(int L, int d, int W, int S, int B, std::vector<int32_t> &codes, int *stride, int U) {
    std::vector<std::vector<int32_t>> lists;
    const int lanes = kLanes * W, steps = place_chain(L, d, W, S, B, U, &lists);
    size_t st = 1;
    for (auto &x : lists) st = std::max(st, x.size() + 1);
    *stride = (int)st;
    codes.assign((size_t)lanes * st, -1);
    for (int q = 0; q < lanes; ++q) std::copy(lists[q].begin(), lists[q].end(), codes.begin() + (size_t)q * st);
    return steps;
}

std::string check_chain_schedule(int L, int d, int W, int S, int B, int steps, const int32_t *codes, int stride,
                                 int U) {
    if (L < 1 || L > kMaxChainLength || d < 0 || W < 1 || W > 16 || S < 1 || B < 2 || steps < 0 || steps % S ||
        stride < 1 || !codes)
        return "bad chain schedule parameters";
    const int lanes = kLanes * W, d1 = d + 1;
    std::vector<int> start((size_t)L * d1, -1);
    for (int q = 0; q < lanes; ++q) {
        const int32_t *row = codes + (size_t)q * stride;
        long t = 0;
        int e = 0;
        for (; e < stride && row[e] >= 0; ++e) {
            const int j = row[e] >> 16, k = row[e] & 0xffff;
            if (j == kIdleJob) {
                t += k + 1;
                continue;
            }
            if (j >= L || k > d) return "code out of range";
            const size_t key = (size_t)j * d1 + k;
            if (start[key] >= 0) return "coefficient scheduled twice";
            start[key] = (int)t;
            t += k / U + 1;
        }
        if (e == stride) return "row without its terminator";
        if (t > steps) return "row longer than the steps";
    }
    for (int v : start)
        if (v < 0) return "coefficient never scheduled";
    // x_i of job l is read by its coefficients k >= i: the earliest of them starts
    // after the barrier that follows its store, the latest before the one after
    // which it is overwritten
    bool ordered = true;
    for (int l = 0; l < L && ordered; ++l) {
        const int wj = l - 1 + B;  // stores the first operand of job l + B into the same slot
        int first = start[(size_t)l * d1 + d], last = first;
        for (int i = d; i >= 0; --i) {
            first = std::min(first, start[(size_t)l * d1 + i]);
            last = std::max(last, start[(size_t)l * d1 + i]);
            auto stored = [&](int job) { return chain_window(start[(size_t)job * d1 + i] + i / U, S); };
            ordered &= !(l > 0 && chain_window(first + i / U - 1, S) <= stored(l - 1)) &&
                       !(wj + 1 < L && stored(wj) <= chain_window(last + i / U - 1, S));
        }
    }
    if (ordered) return "";
    // (which one is not)
    for (int l = 0; l < L; ++l)
        for (int k = 0; k <= d; ++k) {
            const int s = start[(size_t)l * d1 + k];
            for (int i = 0; i <= k; ++i) {
                const int rd = s + i / U - 1;  // iteration that reads x_i
                // job 0's first operand is staged before the first barrier
                if (l > 0 && chain_window(rd, S) <= chain_window(start[(size_t)(l - 1) * d1 + i] + i / U, S))
                    return "job " + std::to_string(l) + " coefficient " + std::to_string(k) +
                           ": first operand read before the barrier after its store";
                // job l-1+B stores the first operand of job l+B into the same slot
                const int wj = l - 1 + B;
                if (wj + 1 < L && chain_window(start[(size_t)wj * d1 + i] + i / U, S) <= chain_window(rd, S))
                    return "job " + std::to_string(l) + " coefficient " + std::to_string(k) +
                           ": first operand overwritten before the barrier after its read";
            }
        }
    return "";
}

// Chains of the plan's convolutions: a job whose second operand is a staged
// input (written by no convolution) starts a chain when its first operand is
// one too, and continues the chain of its first operand's writer when it is
// the first such job to read that output.  Jobs in launch (topological)
// order; chains[c] lists job indices in chain order.  Requires one writer per
// slot (no in-place jobs).
static bool find_chains(const Plan &P, std::vector<std::vector<int64_t>> &chains) {
    const size_t nj = P.conv.size();
    std::vector<int64_t> writer(P.n_series, -1);
    for (size_t j = 0; j < nj; ++j) {
        if (writer[P.conv[j][2]] >= 0) return false;
        writer[P.conv[j][2]] = (int64_t)j;
    }
    std::vector<int64_t> chain_of(nj, -1);
    chains.clear();
    for (size_t j = 0; j < nj; ++j) {
        const auto &t = P.conv[j];
        if (writer[t[1]] >= 0 || t[0] == t[2]) continue;
        const int64_t p = writer[t[0]];
        if (p < 0) {
            chain_of[j] = (int64_t)chains.size();
            chains.push_back({(int64_t)j});
        } else if (chain_of[p] >= 0 && chains[chain_of[p]].back() == p &&
                   (int)chains[chain_of[p]].size() < kMaxChainLength) {
            chain_of[j] = chain_of[p];
            chains[chain_of[p]].push_back((int64_t)j);
        }
    }
    return !chains.empty();
}

bool earliest_layers(const Plan &P, std::vector<std::array<int32_t, 3>> &conv, std::vector<int64_t> &off) {
    std::vector<int> written(P.n_series, 0);  // layer of a slot's last writer
    std::vector<int> layer(P.conv.size());
    int nl = 0;
    for (size_t j = 0; j < P.conv.size(); ++j) {
        const auto &t = P.conv[j];
        layer[j] = std::max(written[t[0]], written[t[1]]) + 1;
        written[t[2]] = std::max(written[t[2]], layer[j]);
        nl = std::max(nl, layer[j]);
    }
    off.assign(nl + 1, 0);
    for (int L : layer) off[L]++;
    for (int L = 1; L <= nl; ++L) off[L] += off[L - 1];
    std::vector<int64_t> at(off.begin(), off.end() - 1);
    conv.resize(P.conv.size());
    for (size_t j = 0; j < P.conv.size(); ++j) conv[at[layer[j] - 1]++] = P.conv[j];
    Plan Q = P;
    Q.conv = conv;
    Q.conv_off = off;
    return check_hazards(Q).empty();
}

// Estimated cycles of the per-layer launches of the layers from_layer...: their
// arithmetic and ~4.5 us (10000 cycles) of launch boundary each.
static double layers_cost(const Plan &P, int from_layer) {
    const double launches = 10000.0 * (P.n_layers() - from_layer + 1);
    if (P.block_r > 0) return launches + block_cost(P, P.block_r, P.block_u, P.blocks, from_layer);
    const int Q = P.lanes.waves_per_job, J = P.lanes.jobs_per_group;
    if (P.simple)
        return launches + layer_cost(P, Q, J, dealt_steps(P.d, J, Q), 4.4 * (mac_instr(P) + 10), from_layer);
    return launches + layer_cost(P, Q, J, P.lanes.steps, 4.4 * (mac_instr(P) + 90), from_layer);
}

// Rebuilds P's convolution layers for the chain launch with W wavefronts per
// chain, a barrier every S steps and B LDS slots of first operands, by
// coefficients (R = 0) or blocks of R, U terms an iteration: layer L <= pipe_layers holds the jobs at
// position L of their chain, the other jobs follow at their earliest layers.
static bool make_chain_plan(Plan &P, const std::vector<std::vector<int64_t>> &chains, int R, int U, int W, int S,
                            int B) {
    const size_t nj = P.conv.size();
    int Lmax = 0;
    std::vector<char> in_chain(nj, 0);
    for (auto &c : chains) {
        Lmax = std::max(Lmax, (int)c.size());
        for (int64_t j : c) in_chain[j] = 1;
    }
    // the other jobs at their earliest layers after the chain launch
    std::vector<int> wlayer(P.n_series, 0);
    std::vector<int> rest_layer(nj, 0);
    int rest_layers = 0;
    for (size_t j = 0; j < nj; ++j) {
        if (in_chain[j]) continue;
        const auto &t = P.conv[j];
        const int L = std::max(wlayer[t[0]], wlayer[t[1]]) + 1;
        rest_layer[j] = L;
        wlayer[t[2]] = std::max(wlayer[t[2]], L);
        rest_layers = std::max(rest_layers, L);
    }
    std::vector<std::array<int32_t, 3>> conv;
    std::vector<int64_t> off{0};
    for (int L = 0; L < Lmax; ++L) {
        for (auto &c : chains)
            if ((int)c.size() > L) conv.push_back(P.conv[c[L]]);
        off.push_back((int64_t)conv.size());
    }
    for (int L = 1; L <= rest_layers; ++L) {
        for (size_t j = 0; j < nj; ++j)
            if (!in_chain[j] && rest_layer[j] == L) conv.push_back(P.conv[j]);
        off.push_back((int64_t)conv.size());
    }
    if (conv.size() != nj) return false;
    // one schedule per chain length
    const int dd = R > 0 ? P.d / R : P.d;
    std::vector<ChainComp> comps;
    std::vector<std::array<int32_t, 3>> pjobs;
    std::vector<int32_t> codes;
    std::vector<std::array<int, 3>> sched(Lmax + 1, {-1, 0, 0});  // length -> {code_off, stride, steps}
    // longest chains first: they start first
    std::vector<size_t> order(chains.size());
    std::iota(order.begin(), order.end(), (size_t)0);
    if (R > 0)
        std::stable_sort(order.begin(), order.end(),
                         [&](size_t a, size_t b) { return chains[a].size() > chains[b].size(); });
    for (size_t o : order) {
        const auto &c = chains[o];
        const int len = (int)c.size();
        if (sched[len][0] < 0) {
            std::vector<int32_t> cs;
            int stride = 0;
            const int u = R == 1 ? U : 1;  // tiles: an iteration is a step over blocks
            const int steps = make_chain_schedule(len, dd, W, S, B, cs, &stride, u);
            if (!check_chain_schedule(len, dd, W, S, B, steps, cs.data(), stride, u).empty()) return false;
            if (codes.size() + cs.size() > (size_t)INT32_MAX / 2) return false;
            sched[len] = {(int)codes.size(), stride, steps};
            codes.insert(codes.end(), cs.begin(), cs.end());
        }
        comps.push_back(ChainComp{(int32_t)pjobs.size(), len, sched[len][0], sched[len][1], sched[len][2], 0, 0, 0});
        for (int64_t j : c) pjobs.push_back(P.conv[j]);
    }
    P.conv.swap(conv);
    P.conv_off.swap(off);
    P.pipe_layers = Lmax;
    P.pipe_waves = W;
    P.pipe_window = S;
    P.pipe_ring = B;
    P.pipe_r = R;
    P.pipe_u = U;
    P.pipe_jobs.swap(pjobs);
    P.pipe_comps.swap(comps);
    P.pipe_codes.swap(codes);
    P.balanced = false;
    choose_staged_lanes(P, Lmax + 1);
    choose_block_lanes(P, Lmax + 1);
    return true;
}

// What chains of one or two wavefronts cost beyond chain_cost's terms.  Once a CU
// holds more of those wavefronts than SIMDs they spread unevenly: the fullest SIMD
// counts, and with two a little more (522 chains of 28, five doubles, d = 130: 2575
// us on two wavefronts each, 1781 on four, where the terms say 1964 and 2116; 620
// chains of 39, four doubles, d = 80: 1144 and 740; of 160 plans 155 then take a
// width within 5% of the best, 140 without this).  Not at one double, whose waits
// leave the SIMDs room (708 chains of 25, d = 100: 96 us on two, 108 on four).
// Long products lose a little more on two (226 chains of 23 at eight doubles, d =
// 15: 227 and 207 us on four, a tie by the terms).
static double narrow_chains(const Plan &P, size_t chains, int W) {
    const long cus = kSimds / 4;
    const double k = std::min(16L / W, ((long)chains + cus - 1) / cus) * W / 4.0;
    const bool even = W >= 4 || k <= 1 || P.w == 1;
    return (even ? 1.0 : std::max(1.0, 0.95 * (std::ceil(k) + (W == 2 ? 0.5 : 0.0)) / k)) *
           (W == 2 && P.w >= 8 ? 1.1 : 1.0);
}

// Estimated cycles of the chain launch: its iterations, and a barrier's wait for
// the slowest of W wavefronts (measured on p2: quad double, d = 64, 320
// iterations on 8 wavefronts 348 us; penta double, d = 37, 222 on 4 245 us).
static double chain_cost(const Plan &P, size_t chains, int R, int U, int W, int S, int steps, long lds) {
    // workgroups of a CU, by LDS and by 16 wavefronts (128 VGPRs each)
    const long cus = kSimds / 4;
    const long fit = std::max(1L, std::min((long)kMaxLdsBytes / lds, 16L / W));
    const long per_cu = std::min(fit, ((long)chains + cus - 1) / cus);
    const double rounds = std::ceil(chains / (double)(cus * per_cu));
    const double k = std::max(1.0, per_cu * W / 4.0);  // wavefronts per SIMD
    // With a chain per CU at most and from five doubles on, whose products hold
    // independent sums, a lone wavefront issues every 5 cycles or so: four
    // wavefronts, not eight, for chains of 23 to 64 (d = 49: 10 doubles 907
    // against 1072 us, 8 538 against 606, 5 209 against 227); eight for longer series
    // up to eight doubles (28 chains of 25, 8 doubles, d = 176: 4605 on four, 4354;
    // 180 of 27, complex quad double, d = 146: 2880 and 2653).  With more chains
    // the estimate of the rounds, made for equal chains, is the larger error and
    // keeps the factor of the narrow ones (211 monomials of 1 to 12 variables,
    // 8 doubles, d = 70: 693 us; with this factor 1146).
    const double lone = chains > (size_t)cus || P.w < 5 ? 1.5 : P.w <= 8 ? 1.2 : 1.12;
    return narrow_chains(P, chains, W) * rounds * steps * (block_iteration(P, R, U, k, lone) + (W > 1 ? (60.0 + 30.0 * W) / S : 0));
}

// The chain launch for a plan without in-place jobs: the cheapest estimate
// over R coefficients per block, W wavefronts per chain, a barrier every S
// iterations and the LDS of a chain, applied when forced or estimated under 0.9
// of `other` (the cycles of the plan without it).  Returns whether P now holds
// a chain launch.  Chains from nine products on, below 16 products from 64 chains
// on (211 monomials of 1 to 12 variables, five doubles, d = 37: 404 -> 130 us): other
// plans keep their layers, their workspace and their build time, not because the
// launch would lose (5, 7, 9 and 12 products against the default, 4 to 128 chains: one
// double, d = 16, 0.83 to 0.97, 1.01 to 1.08, 1.08 to 1.15, 1.14 to 1.25 times as fast;
// two, d = 16, 1.1, 1.3, 1.5, 1.7; four, d = 16, 1.5, 1.9, 2.2, 2.6; eight, d = 64, 2.3,
// 2.7, 3.0, 3.6).
static bool choose_chain_launch(Plan &P, bool forced, double other) {
    if (P.streamed) return false;
    std::vector<std::vector<int64_t>> chains;
    if (!find_chains(P, chains)) return false;
    int Lmax = 0;
    long members = 0;
    for (auto &c : chains) {
        Lmax = std::max(Lmax, (int)c.size());
        members += (long)c.size();
    }
    if (!forced && (Lmax < 9 || (Lmax < 16 && chains.size() < 64) || 4 * members < (long)P.conv.size())) return false;
    // (one double per coefficient beyond d = 190 keeps its layers unless asked; the
    // chain launch wins on both sides of that line, p2 at d = 161, 176, 185 and 191
    // 200, 213, 224 and 232 us against 545 to 568)
    if (!forced && P.w == 1 && P.d > 190) return false;
    // candidates with the least their schedule can cost: its iterations fill the
    // lanes, and a product's first coefficient starts a barrier after the one
    // before it is stored
    struct Cand {
        double bound;
        int R, U, W, S, B;
        long lds;
    };
    std::vector<Cand> cands;
    // by coefficients (R = 0, the 64-bit addresses) where the workspace is 4 GiB or more
    const bool small = small_workspace(P);
    // (four terms of one coefficient: 0.63 to 1.0 on p2, 1.05 at best)
    static const int kRU[5][2] = {{0, 0}, {1, 1}, {1, 2}, {2, 2}, {4, 4}};
    for (auto &ru : kRU) {
        const int R = ru[0], U = ru[1], r1 = std::max(R, 1), u1 = std::max(U, 1);
        if (small ? R == 0 : R > 0) continue;
        if ((R == 4 && P.w > 2) || (R == 2 && P.w > 5) || (R == 1 && U == 2 && P.w > 10)) continue;
        if (U > 1 && !reads_inside(P, P.conv, R == 1 ? U - 1 : 0, R == 1 ? 0 : U - 1)) continue;
        const int items = P.d / r1, tail = R == 1 ? P.d / u1 + 1 : items + 1;
        const long all = R == 1 ? (long)tail * (P.d + 1 - (tail - 1) * (long)u1 / 2) : (long)tail * (tail + 1) / 2;
        int last_B = 0;
        for (long budget : {98304L, 49152L, 24576L}) {
            const int B = (int)std::min<long>(std::max(Lmax, 2), (budget - (long)sizeof(JobOffsets) * Lmax) /
                                                                     ((long)(P.d + 1) * P.w * 8));
            const long lds = chain_lds_bytes(P.d + 1, P.w, u1, B, 2 * Lmax);
            if (B == last_B) continue;
            last_B = B;
            if (B < 2 || lds > kMaxLdsBytes || (budget < 98304 && chains.size() <= (size_t)kSimds / 4)) break;
            for (int W : {1, 2, 4, 8, 12, 16}) {
                // up to 16 wavefronts (1024 threads, 128 VGPRs each) where that
                // needs no spills; one or two only for many chains
                if ((W > 8 && P.w * u1 > 10) || (W == 16 && P.w > 8)) continue;
                if (W < 4 && (R == 0 || chains.size() < 64)) continue;
                for (int S : {1, 2, 4}) {
                    if (W == 1 && S > 1) continue;
                    int start = 0;
                    for (int l = 1; l < Lmax; ++l) start = S * (start / S + 1) + 1;
                    const int fewest = (int)std::max(Lmax * all / (kLanes * W), (long)start + tail);
                    cands.push_back({chain_cost(P, chains.size(), r1, u1, W, S, fewest, lds), R, U, W, S, B, lds});
                }
            }
        }
    }
    // the cheapest, schedules made in the order of the bounds until none can be cheaper
    std::stable_sort(cands.begin(), cands.end(), [](const Cand &a, const Cand &b) { return a.bound < b.bound; });
    double best = -1;
    int br = 0, bu = 0, bw = 0, bs = 0, bb = 0;
    for (const Cand &c : cands) {
        if (best >= 0 && c.bound >= best) break;
        const int steps = place_chain(Lmax, P.d / std::max(c.R, 1), c.W, c.S, c.B, c.R == 1 ? c.U : 1, nullptr);
        const double cost = chain_cost(P, chains.size(), std::max(c.R, 1), std::max(c.U, 1), c.W, c.S, steps, c.lds);
        if (best < 0 || cost < best) {
            best = cost;
            br = c.R;
            bu = c.U;
            bw = c.W;
            bs = c.S;
            bb = c.B;
        }
    }
    if (best < 0 || !make_chain_plan(P, chains, br, bu, bw, bs, bb)) return false;
    const double rest = layers_cost(P, P.pipe_layers + 1);
    return forced || best / narrow_chains(P, chains.size(), bw) + rest < 0.9 * other;
}

// Whether the chain launch of C pays so much against the plan P without it that C
// takes more workspace than the allocation-free entry has, where P fits (callers of
// that entry pass MDPE_NO_CHAIN_LAUNCH): chains of 16 products or more, a quarter
// of the convolutions or more, under 0.9 of P by an estimate that favours P -- steps
// of the coefficient schedules, one chain per CU, four to sixteen wavefronts sharing
// its SIMDs at eff of their lone speed, one double's chain steps at 0.55 of the
// layers' (261 monomials of 15 variables, exponents to 2, five doubles, d = 130,
// 62.8 -> 67.9 MiB: 3080 -> 1790 us).
static bool outgrowing_pays(const Plan &P, const Plan &C) {
    const int Lmax = C.pipe_layers, chains = (int)C.pipe_comps.size();
    if (P.n_layers() < 16 || Lmax < 16 || 4 * C.pipe_jobs.size() < C.conv.size()) return false;
    const int B = (int)std::min<long>(std::max(Lmax, 2), (98304 - (long)sizeof(JobOffsets) * Lmax) /
                                                             ((long)(P.d + 1) * P.w * 8));
    if (B < 2) return false;
    auto layers = [](const Plan &Q, int from) {
        const int q = Q.lanes.waves_per_job, J = Q.lanes.jobs_per_group;
        return Q.simple ? layer_cost(Q, q, J, dealt_steps(Q.d, J, q), Q.w == 1 ? 0.15 : 0.4, from)
                        : layer_cost(Q, q, J, Q.lanes.steps, 1.0, from);
    };
    double other = layers(P, 1);
    if (fuse_by_default(P)) {
        const LaneSchedule one = make_lane_schedule(P.d, 1);
        other = std::min(other, P.n_layers() * (prefer_simple_dealing(P.d, 1, P.w, one.steps)
                                                    ? dealt_steps(P.d, 1) * (P.w == 1 ? 0.15 : 0.5)
                                                    : (double)one.steps));
    }
    static const double eff[2][5] = {{1.0, 1.0, 0.80, 0.73, 0.70}, {1.0, 1.0, 0.89, 0.81, 0.74}};
    const double rounds = std::ceil(chains / (kSimds / 4.0));
    double best = -1;
    for (int W : {4, 8, 12, 16})
        for (int S : {1, 2, 4}) {
            if (W == 16 && P.w > 8) continue;
            const int k = W / 4, steps = place_chain(Lmax, P.d, W, S, B, 1, nullptr);
            const double c = rounds * steps * k * eff[P.w >= 8][k] * (1.0 + 0.08 / S) * (P.w == 1 ? 0.55 : 1.0);
            if (best < 0 || c < best) best = c;
        }
    return best + layers(C, Lmax + 1) < 0.9 * other;
}

// ----------------------------------------------------------- single launch
// FP64 instructions of one md_add / md_mul of the specification (two_sum = 6
// additions, two_prod = 1 mul + 1 fma; the closed forms of the accounting).
static long md_instr(bool mul, int m) {
    const long rs = m >= 2 ? 2 * m - 3 : 0;
    if (!mul) return 6 * ((long)m * (m - 1) / 2 + rs) + m;
    long ntp = m >= 2 ? (m - 1) + (long)(m - 2) * (m - 1) / 2 : 0;
    long tse = m >= 2 ? (long)(m - 2) * (m - 1) / 2 : 0;
    long tsp = 0, plain = m - 1;
    for (int k = 1; k < m - 1; ++k) {
        tsp += (long)k * (2 * m - 3 - 2 * k);
        plain += 2 * k;
    }
    return 6 * (tse + tsp + rs) + plain + (ntp + 1) + (ntp + 2 * (m - 1));
}

// Estimated microseconds of a plan's evaluation layer by layer and in one
// workgroup of `waves` wavefronts that runs every stage.  The coefficients fit 257
// and 266 small plans measured so (2 to 150 monomials of 1 to 8 variables, one to
// ten doubles, d = 1 to 48; errors of 12 and 20%):
// - by layers, 3.3 us and 2.2 a launch (staging, each layer, each addition pass), 1.6
//   more for a layer of one double, 0.73 of the layers' estimated cycles at 2.35
//   GHz, and 0.53 ns an instruction of an addition for each level of the deepest tree;
// - in one workgroup, its rounds of convolutions at 1.48 of their estimate (a
//   multiply-add step costs its md instructions and ~50 of bookkeeping, 4 cycles
//   each at 2.2 GHz, a wavefront sharing its SIMD with k - 1 others k times as
//   long; dealt coefficients of w <= 2 take the measured weight of their steps),
//   1 us and 12 ns an instruction for each of its rounds of additions, 0.47 us a
//   phase, 2.4 us a round of scalings.
struct SingleCost {
    double multi_us, single_us;
    int waves;
    LaneSchedule lanes;
    bool simple;
};

static SingleCost single_launch_cost(const Plan &P) {
    const bool cx = P.complex_series();
    const long mul = cx ? 4 * md_instr(true, P.m) + 2 * md_instr(false, P.m) : md_instr(true, P.m);
    const long add = (cx ? 2 : 1) * md_instr(false, P.m);
    const double step_us = (double)(mul + add + 50) * 4 / 2200.0;
    const double add_us = (double)(add + 20) * 4 / 2200.0;
    const long d1 = P.d + 1;
    SingleCost c{0, 0, 0, LaneSchedule(), false};
    // by layers
    const int nl = P.n_layers(), cover = add_pass_leaves(P.w);
    int64_t longest = 0;
    for (size_t o = 0; o + 1 < P.list_off.size(); ++o) longest = std::max(longest, P.list_off[o + 1] - P.list_off[o]);
    int passes = 1;
    for (int64_t l = longest; l > cover; l = (l + cover - 1) / cover) ++passes;
    const int launches = 1 + nl + passes + (P.scale.empty() ? 0 : 1);
    c.multi_us = 3.3 + 2.2 * launches + (P.w == 1 ? 1.6 * nl : 0.0) +
                 0.73 * (layers_cost(P, 1) - 10000.0 * nl) / 2350.0 +
                 0.00053 * std::ceil(std::log2(std::max<double>((double)longest, 2.0))) * add;
    // one workgroup: 4, 8 or 16 wavefronts (the cheapest by the sum below), one-wavefront
    // groups of J0 (or fewer) jobs within the LDS of the workgroup
    double least = -1;
    c.single_us = -1;
    const long stage_items = (long)P.stage.size() * d1, gather_items = (long)(1 + P.n) * d1;
    for (int W : {4, 8, 16}) {
        const int lds_per_coef = lds_doubles_per_coef(P.w);
        for (int Js = choose_jobs_per_group(P.d, P.w);; Js = std::max(1, Js / 2)) {
            const long bytes = (group_lds_bytes(d1, lds_per_coef, Js) + 15) / 16 * 16;
            if (bytes * W <= kMaxLdsBytes) {
                const LaneSchedule ls = make_lane_schedule(P.d, Js);
                const bool simple = prefer_simple_dealing(P.d, Js, P.w, ls.steps);
                const double st = simple ? dealt_steps(P.d, Js) * (P.w == 1 ? 0.15 : 0.5) : (double)ls.steps;
                const double share = W / 4.0;  // wavefronts per SIMD
                const double threads = 64.0 * W;
                double conv = 0, adds = 0;
                for (int L = 1; L <= nl; ++L)
                    conv += std::ceil((P.conv_off[L] - P.conv_off[L - 1]) / (double)(W * Js)) * st * step_us * share;
                for (int r = 1; r <= P.n_levels(); ++r)
                    adds += std::ceil((P.add_off[r] - P.add_off[r - 1]) * d1 / threads);
                const double scales = std::ceil((double)P.scale.size() * d1 / threads);
                const double u = conv + adds * add_us * share + scales * step_us * share +
                                 std::ceil((stage_items + gather_items) / threads) * 0.2;
                if (least < 0 || u < least) {
                    least = u;
                    c.single_us = 1.48 * conv + adds * (1.0 + 0.012 * add) + 0.47 * (nl + P.n_levels()) + 2.4 * scales;
                    c.waves = W;
                    c.lanes = ls;
                    c.simple = simple;
                }
                break;
            }
            if (Js == 1) break;
        }
    }
    return c;
}

static bool choose_single_launch(Plan &P, bool forced, bool keep) {
    if (P.streamed || P.pipe_layers > 0 || P.fused_components > 0) return false;
    const SingleCost c = single_launch_cost(P);
    // (of 230 plans measured both ways the choice takes 1.02 times the better one's time
    // together; below 17 us, where launches alone tie the estimates, one workgroup
    // keeps the plans up to 1.4: 78 monomials of one or two variables, two doubles, d =
    // 3, 13.1 us and 16.0 by layers).  A plan that keeps the monomial values serves
    // autograd, whose host work for both passes (57 to 115 us) hides some 40 us of one
    // workgroup's evaluation and the reverse pass behind it, and is shorter by three
    // launches or more (55 plans, 0.84 to 0.93 of the time by layers up to 40 us; 120
    // products of two of sixteen variables, one double, d = 15, 107 and 122 us, the
    // evaluation alone 19 and 14)
    double most = c.multi_us < 17.0 ? 1.4 * c.multi_us : c.multi_us;
    if (keep) most = std::max(most, 40.0);
    if (c.single_us < 0 || (!forced && c.single_us >= most)) return false;
    P.single = true;
    P.single_waves = c.waves;
    P.single_lanes = c.lanes;
    P.single_simple = c.simple;
    return true;
}

static std::string build_plan_launches(int n, int N, int d, int m, const int32_t *nvars, const int32_t *vars,
                                       const int32_t *exps, uint32_t flags, Plan &P, bool *unsupported) {
    // Staged operands unless asked otherwise, or unless they do not fit in
    // LDS, or unless streaming with several wavefronts per job is estimated
    // to be faster (large d with few jobs per layer).
    std::string err = build_plan_mode(n, N, d, m, nvars, vars, exps, flags, false, false, P, unsupported);
    if (!err.empty()) return err;
    // The chain launch (deep chains of products, p2's above all), when asked
    // for or estimated well under the layered or fused plan.  Its plans give
    // the in-place products fresh output slots: a chain's products overlap,
    // so b_{n-2} must stay readable while b_{n-2} * a_k is stored.
    const bool chain_forced = (flags & kChainLaunch) != 0;
    // (no second plan is built for less than a monomial of seven variables or a power
    // table of nine: a multilinear chain of nine products takes that much.  Monomials
    // of five or six variables reach it through common factors, with exponents on
    // nearly all of them, and keep their layers)
    int longest = 0;
    int64_t at = 0;
    for (int k = 0; k < N; ++k) {
        longest = std::max(longest, nvars[k] + 2);
        for (int q = 0; q < nvars[k]; ++q, ++at)
            if (exps) longest = std::max(longest, exps[at]);
    }
    if (!P.streamed && !(flags & (kFusedLayers | kLayerLaunches | kNoChainLaunch)) &&
        (chain_forced || (P.n_layers() >= 9 && longest >= 9))) {
        double other = layers_cost(P, 1);
        // ... or, at one double, of the fused launch with a launch less than the chain
        // launch and its layers: 0.65 us a layer and 0.05 a degree (33 plans of 9 to
        // 33 layers at d = 3 to 8, 18 to 39 us with it: 199 monomials of 2 to 9
        // variables, d = 3, 17.8 us, 25.7 by the chain launch; from two doubles on the
        // chain launch is faster in 326 plans of 326)
        if (P.w == 1 && fuse_by_default(P)) {
            Plan F = P;
            if (fuse_layers(F) <= 4) other = std::min(other, P.n_layers() * (1530.0 + 118.0 * d) / 0.9);
        }
        Plan C;
        bool uns = false;
        // (at its earliest layers: make_chain_plan orders the jobs anew)
        std::string e2 = build_plan_mode(n, N, d, m, nvars, vars, exps, flags | kAsapLayers, false, true, C, &uns);
        if (e2.empty() && choose_chain_launch(C, chain_forced, other)) {
            // (a plan that the allocation-free entry takes without the chain launch's
            // fresh slots is not made too large for it, unless long chains pay)
            auto bytes = [](const Plan &Q) { return Q.n_series * (int64_t)(Q.d + 1) * Q.w * (int64_t)sizeof(double); };
            const bool outgrows = bytes(P) <= kScratchBytes && bytes(C) > kScratchBytes;
            if (chain_forced || !outgrows || outgrowing_pays(P, C)) {
                auto h = check_hazards(C);
                if (!h.empty()) return "internal planner error (chain launch): " + h;
                P = std::move(C);
                return "";
            }
        }
    }
    if (chain_forced) {
        *unsupported = true;
        return "MDPE_CHAIN_LAUNCH: no chain of products to pipeline, or its first operands do not fit in LDS";
    }
    auto fuse = [&]() {
        if (P.streamed) return err;
        if (flags & kFusedLayers)
            fuse_layers(P);
        else if (!(flags & (kLayerLaunches | kSingleLaunch)) && fuse_by_default(P) && fuse_layers(P) > 4)
            unfuse(P);  // a component would need several rounds per layer
        return err;
    };
    if (P.streamed || (flags & kStageOperands)) return fuse();
    bool paired = false;
    const int Q = stream_waves_per_job(d, &paired);
    if (Q >= 2 && !(flags & kFusedLayers)) {
        const LaneSchedule ss = paired ? make_paired_schedule(d, Q) : make_lane_schedule(d, 1, Q);
        if (layer_cost(P, Q, 1, ss.steps, 1.2) < layer_cost(P, 1, P.lanes.jobs_per_group, P.lanes.steps, 1.0))
            return build_plan_mode(n, N, d, m, nvars, vars, exps, flags, true, false, P, unsupported);
    }
    return fuse();
}

// The plan's launch structure (per layer, fused, chain launch or streamed),
// then, for plans so small that kernel boundaries dominate, the single launch.
std::string build_plan(int n, int N, int d, int m, const int32_t *nvars, const int32_t *vars, const int32_t *exps,
                       uint32_t flags, Plan &P, bool *unsupported) {
    const bool forced = (flags & kSingleLaunch) != 0;
    std::string err = build_plan_launches(n, N, d, m, nvars, vars, exps, forced ? flags | kNoChainLaunch : flags, P,
                                          unsupported);
    if (!err.empty()) return err;
    P.flags = flags;
    if (forced || !(flags & (kLayerLaunches | kFusedLayers | kChainLaunch | kStreamOperands))) {
        if (!choose_single_launch(P, forced, (flags & kKeepMonomialValues) != 0) && forced) {
            *unsupported = true;
            return "MDPE_SINGLE_LAUNCH: a job group does not fit in the workgroup's LDS";
        }
    }
    return "";
}

static std::string build_plan_mode(int n, int N, int d, int m, const int32_t *nvars, const int32_t *vars,
                                   const int32_t *exps, uint32_t flags, bool stream, bool no_inplace, Plan &P,
                                   bool *unsupported) {
    *unsupported = false;
    if (flags & ~(kKeepMonomialValues | kComplex | kStreamOperands | kStageOperands | kAsapLayers | kFusedLayers |
                  kLayerLaunches | kChainLaunch | kNoChainLaunch | kSingleLaunch | kWideOffsets))
        return "unknown flags";
    if ((flags & kChainLaunch) && (flags & (kFusedLayers | kLayerLaunches | kStreamOperands | kNoChainLaunch)))
        return "MDPE_CHAIN_LAUNCH excludes MDPE_FUSED_LAYERS, MDPE_LAYER_LAUNCHES, MDPE_STREAM_OPERANDS and "
               "MDPE_NO_CHAIN_LAUNCH";
    if ((flags & kSingleLaunch) && (flags & (kFusedLayers | kLayerLaunches | kStreamOperands | kChainLaunch)))
        return "MDPE_SINGLE_LAUNCH excludes MDPE_FUSED_LAYERS, MDPE_LAYER_LAUNCHES, MDPE_STREAM_OPERANDS and "
               "MDPE_CHAIN_LAUNCH";
    if ((flags & kFusedLayers) && (flags & kLayerLaunches)) return "MDPE_FUSED_LAYERS and MDPE_LAYER_LAUNCHES exclude each other";
    if ((flags & kStreamOperands) && (flags & kStageOperands)) return "MDPE_STREAM_OPERANDS and MDPE_STAGE_OPERANDS exclude each other";
    const bool keep = (flags & kKeepMonomialValues) != 0;
    const bool cx = (flags & kComplex) != 0;
    if (keep && cx) {
        *unsupported = true;
        return "the reverse pass (MDPE_KEEP_MONOMIAL_VALUES) is for real series only";
    }
    if (n < 1 || N < 0 || d < 0) return "need n >= 1, N >= 0, d >= 0";
    if (!supported_m(m)) {
        *unsupported = true;
        return "m must be one of 1, 2, 3, 4, 5, 8, 10";
    }
    if (N > 0 && (!nvars || !vars)) return "nvars/vars missing";
    int64_t tot = 0, nb = 0, nc = 0;
    int nmax = 0;
    for (int k = 0; k < N; ++k) {
        int nk = nvars[k];
        if (nk < 1 || nk > n) return "monomial " + std::to_string(k) + ": n_k out of range";
        for (int j = 0; j < nk; ++j) {
            int v = vars[tot + j];
            if (v < 0 || v >= n) return "monomial " + std::to_string(k) + ": variable out of range";
            if (j > 0 && v <= vars[tot + j - 1]) return "monomial " + std::to_string(k) + ": variables not strictly increasing";
        }
        tot += nk;
        nb += std::max(1, nk - 2);
        nc += std::max(0, nk - 2);
        nmax = std::max(nmax, nk);
    }
    // General exponents (Section 3): a table of powers z_i^p, p = 2..maxp[i],
    // and one common-factor slot per monomial with an exponent above one.
    std::vector<int> maxp(n, 0);
    int64_t nfac = 0;
    if (exps) {
        int64_t q = 0;
        for (int k = 0; k < N; ++k) {
            bool any = false;
            for (int j = 0; j < nvars[k]; ++j, ++q) {
                const int e = exps[q];
                if (e < 1 || e > kMaxExponent) return "monomial " + std::to_string(k) + ": exponent out of range 1..64";
                maxp[vars[q]] = std::max(maxp[vars[q]], e - 1);
                any |= e >= 2;
            }
            nfac += any;
        }
    }
    int64_t npow = 0;
    std::vector<int64_t> powoff(n, 0);  // slot of z_i^p is pbase + powoff[i] + p - 2
    for (int i = 0; i < n; ++i) {
        powoff[i] = npow;
        npow += std::max(0, maxp[i] - 1);
    }
    if (keep && nfac > 0) {
        *unsupported = true;
        return "the reverse pass (MDPE_KEEP_MONOMIAL_VALUES) is for multilinear monomials only";
    }
    const int64_t base = 1 + (int64_t)N + n;
    int64_t nmono2 = 0;  // monomials with n_k >= 2: they get an M_k slot when kept
    for (int k = 0; k < N; ++k) nmono2 += nvars[k] >= 2;
    const int64_t pbase = base + tot + nb + nc;  // powers, then common factors
    const int64_t fbase = pbase + npow;
    const int64_t mbase = fbase + nfac;
    const int w = cx ? 2 * m : m;
    // Streamed operands when a job's LDS operands would not fit in one
    // workgroup's LDS, or when asked for.  Then no convolution may write its
    // own first operand: b_{n-2} * a and every common-factor step after the
    // first get fresh output slots, after all others.  The same holds for
    // staged operands when one job is spread over several wavefronts
    // (no_inplace): each wavefront stages the first operand on its own, and
    // the wavefronts of a job need not share a workgroup, so one of them could
    // store output coefficients before another has read them.
    const bool fits = (long)(d + 1) * lds_doubles_per_coef(w) * 8 <= kMaxLdsBytes - 32768;
    if ((flags & kStageOperands) && !fits) {
        *unsupported = true;
        return "MDPE_STAGE_OPERANDS: a job's operands do not fit in one workgroup's LDS "
               "((d+1)*w*8 <= 131072 bytes, w = m doubles per coefficient, 2m complex; twice that when w <= 2)";
    }
    const bool streamed = stream || (flags & kStreamOperands) || !fits;
    const bool fresh_out = streamed || no_inplace;
    int64_t n3 = 0, nfac_extra = 0;
    for (int k = 0, q = 0; k < N; q += nvars[k], ++k) {
        n3 += nvars[k] >= 3;
        int cnt = 0;
        for (int j = 0; exps && j < nvars[k]; ++j) cnt += exps[q + j] >= 2;
        nfac_extra += std::max(0, cnt - 1);
    }
    const int64_t xbase = mbase + (keep ? nmono2 + 1 + N + n : 0);
    const int64_t nser = xbase + (fresh_out ? n3 + nfac_extra : 0);
    if (nser > INT32_MAX / 2) {
        *unsupported = true;
        return "too many series for 32-bit slot indices";
    }
    if (d + 1 > 65535) {
        *unsupported = true;
        return "d too large";
    }
    P = Plan();
    P.n = n;
    P.N = N;
    P.d = d;
    P.m = m;
    P.w = w;
    P.flags = flags;
    P.n_series = nser;
    P.streamed = streamed;
    int64_t xpos = 0;
    auto fresh = [&]() { return (int32_t)(xbase + xpos++); };

    std::vector<std::vector<std::array<int32_t, 3>>> layers(std::max(nmax, 1));
    auto add_job = [&](int layer, int32_t t1, int32_t t2, int32_t t3) {
        if ((int)layers.size() < layer) layers.resize(layer);
        layers[layer - 1].push_back({t1, t2, t3});
    };
    std::vector<int32_t> value_list{0};
    std::vector<std::vector<int32_t>> grad_lists(n);
    std::vector<int32_t> mono_slot(N, -1);  // slot holding M_k = prod of the monomial's variables
    for (int s = 0; s < 1 + N + n; ++s) P.stage.push_back({s, s});

    // table of powers: z_i^p := z_i^{p-1} * z_i at layer p-1, ready after it
    auto pow_slot = [&](int i, int p) {
        return p == 1 ? (int32_t)(1 + N + i) : (int32_t)(pbase + powoff[i] + p - 2);
    };
    for (int i = 0; i < n; ++i)
        for (int p = 2; p <= maxp[i]; ++p) add_job(p - 1, pow_slot(i, p - 1), (int32_t)(1 + N + i), pow_slot(i, p));

    int64_t alpha = 0, beta = 0, gamma = 0, pos = 0, mpos = 0, fpos = 0;
    for (int k = 0; k < N; ++k) {
        const int nk = nvars[k];
        const int32_t *v = vars + pos;
        const int32_t *e = exps ? exps + pos : nullptr;
        // common factor a_k * prod_j z_{i_j}^{e_j - 1}, in increasing j; the
        // monomial's own jobs follow it, `shift` layers later
        int32_t a_slot = (int32_t)(k + 1);
        int shift = 0;
        for (int j = 0; e && j < nk; ++j) {
            if (e[j] < 2) continue;
            const int32_t fac = fresh_out && a_slot != (int32_t)(k + 1) ? fresh() : (int32_t)(fbase + fpos);
            const int ready = e[j] - 1 >= 2 ? e[j] - 2 : 0;
            shift = std::max(shift, ready) + 1;
            add_job(shift, a_slot, pow_slot(v[j], e[j] - 1), fac);
            a_slot = fac;
        }
        if (a_slot != (int32_t)(k + 1)) ++fpos;
        auto A = [&](void) { return a_slot; };
        auto Z = [&](int i) { return (int32_t)(1 + N + v[i - 1]); };  // z_{i_i}, 1-based position
        auto F = [&](int j) { return (int32_t)(base + alpha + j - 1); };
        auto B = [&](int j) { return (int32_t)(base + tot + beta + j - 1); };
        auto C = [&](int j) { return (int32_t)(base + tot + nb + gamma + j - 1); };
        auto job = [&](int layer, int32_t t1, int32_t t2, int32_t t3) { add_job(layer + shift, t1, t2, t3); };
        // a z^e factor's partial derivative is e times the multilinear one
        auto scale = [&](int j0, int32_t src, int32_t dst) {
            if (e && e[j0] >= 2) P.scale.push_back({src, dst, e[j0]});
        };
        if (nk == 1) {
            job(1, A(), Z(1), F(1));
            if (e && e[0] >= 2)
                scale(0, A(), B(1));
            else
                P.stage.push_back({B(1), (int32_t)(k + 1)});
            value_list.push_back(F(1));
            grad_lists[v[0]].push_back(B(1));
            mono_slot[k] = Z(1);
        } else {
            job(1, A(), Z(1), F(1));
            for (int j = 2; j <= nk; ++j) job(j, F(j - 1), Z(j), F(j));
            if (nk == 2) {
                job(1, Z(2), A(), B(1));
                grad_lists[v[0]].push_back(B(1));
                grad_lists[v[1]].push_back(F(1));
                scale(0, B(1), B(1));
                scale(1, F(1), F(1));
                if (keep) {
                    mono_slot[k] = (int32_t)(mbase + mpos++);
                    job(1, Z(2), Z(1), mono_slot[k]);  // M_k = z_{i_2} * z_{i_1}
                }
            } else {
                job(1, Z(nk), Z(nk - 1), B(1));
                for (int j = 2; j <= nk - 2; ++j) job(j, B(j - 1), Z(nk - j), B(j));
                // b_{n-2} := b_{n-2} * a_k, in place unless operands are streamed
                // or a job spans several wavefronts
                const int32_t bfin = fresh_out ? fresh() : B(nk - 2);
                if (keep) {
                    // M_k = b_{n-2} * z_{i_1} reads the backward product before its
                    // multiplication by a_k, which therefore moves one layer later
                    mono_slot[k] = (int32_t)(mbase + mpos++);
                    job(nk - 1, B(nk - 2), Z(1), mono_slot[k]);
                    job(nk, B(nk - 2), A(), bfin);
                } else {
                    job(nk - 1, B(nk - 2), A(), bfin);
                }
                for (int j = 1; j <= nk - 3; ++j) job(std::max(j, nk - 2 - j) + 1, F(j), B(nk - 2 - j), C(j));
                job(nk - 1, F(nk - 2), Z(nk), C(nk - 2));
                grad_lists[v[0]].push_back(bfin);
                for (int j = 1; j <= nk - 2; ++j) grad_lists[v[j]].push_back(C(j));
                grad_lists[v[nk - 1]].push_back(F(nk - 1));
                scale(0, bfin, bfin);
                for (int j = 1; j <= nk - 2; ++j) scale(j, C(j), C(j));
                scale(nk - 1, F(nk - 1), F(nk - 1));
            }
            value_list.push_back(F(nk));
        }
        alpha += nk;
        beta += std::max(1, nk - 2);
        gamma += std::max(0, nk - 2);
        pos += nk;
    }

    P.conv_off.push_back(0);
    if (N > 0)
        for (auto &L : layers) {
            P.conv.insert(P.conv.end(), L.begin(), L.end());
            P.conv_off.push_back((int64_t)P.conv.size());
        }

    P.list_off.push_back(0);
    auto keep_list = [&](const std::vector<int32_t> &l) {
        P.list_slots.insert(P.list_slots.end(), l.begin(), l.end());
        P.list_off.push_back((int64_t)P.list_slots.size());
    };
    keep_list(value_list);
    for (int i = 0; i < n; ++i) keep_list(grad_lists[i]);
    std::vector<std::vector<std::array<int32_t, 2>>> rounds;
    P.out_slots.push_back(tree_rounds(value_list, rounds));
    for (int i = 0; i < n; ++i) P.out_slots.push_back(tree_rounds(grad_lists[i], rounds));
    P.add_off.push_back(0);
    for (auto &r : rounds) {
        P.add.insert(P.add.end(), r.begin(), r.end());
        P.add_off.push_back((int64_t)P.add.size());
    }

    if (keep) {
        // reverse pass: abar_k = corr(ybar, M_k), zbar_i = corr(ybar, dp/dz_i)
        int64_t q = mbase + nmono2;
        P.ybar_slot = (int32_t)q++;
        P.coeff_bar_slots.push_back(P.ybar_slot);
        for (int k = 0; k < N; ++k) {
            int32_t out = (int32_t)q++;
            P.corr.push_back({P.ybar_slot, mono_slot[k], out});
            P.coeff_bar_slots.push_back(out);
        }
        for (int i = 0; i < n; ++i) {
            int32_t out = (int32_t)q++;
            int32_t g = P.out_slots[1 + i];
            if (g >= 0) P.corr.push_back({P.ybar_slot, g, out});
            P.z_bar_slots.push_back(g >= 0 ? out : -1);
        }
    }

    if (xpos != nser - xbase) return "internal planner error: fresh slot count";
    if (streamed) {
        bool paired = false;
        const int Q = stream_waves_per_job(d, &paired);
        if (paired)
            P.lanes = make_paired_schedule(d, Q);
        else
            P.lanes = make_lane_schedule(d, Q > 1 ? 1 : std::max(1, std::min(kLanes, (2 * kLanes + d + 1) / (d + 2))), Q);
    } else {
        choose_staged_lanes(P, 1);
        // A job over several wavefronts may not write its own first operand
        // (see no_inplace above): rebuild with fresh output slots for the
        // in-place jobs.  The jobs and layers are the same, so is the choice.
        if (P.lanes.waves_per_job > 1 && !no_inplace) {
            bool inplace = false;
            for (const auto &t : P.conv) inplace |= t[0] == t[2];
            if (inplace) return build_plan_mode(n, N, d, m, nvars, vars, exps, flags, false, true, P, unsupported);
        }
        choose_block_lanes(P, 1);
    }
    // after the lane choice: the check depends on the wavefronts per job
    auto err = check_hazards(P);
    if (!err.empty()) return "internal planner error: " + err;
    if (!(flags & kAsapLayers)) {
        // whole rounds of the coefficient schedule's wavefronts, and, where the
        // launches run blocks, of the blocks' wavefronts too
        auto cost = [&](const LaneSchedule &ls) {
            return layer_cost(P, ls.waves_per_job, ls.jobs_per_group, ls.steps, 1.0);
        };
        auto balance = [&](const LaneSchedule &round, const LaneSchedule &by) {
            const double before = cost(by);
            auto conv = P.conv;
            auto off = P.conv_off;
            if (!balance_layers(P, std::max(1L, kSimds * round.jobs_per_group / round.waves_per_job))) return;
            if (cost(by) < before) {
                P.balanced = true;
            } else {
                P.conv.swap(conv);
                P.conv_off.swap(off);
            }
        };
        balance(P.lanes, P.lanes);
        if (P.block_r > 0) balance(P.blocks, P.blocks);
        if (P.balanced) {
            auto e = check_hazards(P);
            if (!e.empty()) return "internal planner error after layer balancing: " + e;
        }
    }
    return "";
}

}  // namespace mdpe
