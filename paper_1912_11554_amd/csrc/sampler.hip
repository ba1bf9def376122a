// Host-side dispatch of the sampler kernels (sampler_impl.h): path support,
// grid size, launches.
#include <algorithm>

#include "sampler_impl.h"

namespace nuts {

namespace {

// A chain of at most this many rounds of tiles over one group's workers runs on
// a lone group: with more groups the rounds shrink but every leapfrog step
// waits for an exchange (fp64 32 tiles, 5 rounds: 3.97 us an evaluation on one
// group, 4.39 on five; fp32 79 tiles, 12 rounds: 3.95 against 3.82).
constexpr int64_t kTeamLoneRounds64 = 5, kTeamLoneRounds32 = 11;

// Every exchange slot empty, and the error flag clear if given, before a launch.
__global__ void fill_empty_slots(double* a, int64_t na, double* b, int64_t nb, GridSync* sync)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (first == 0 && sync) sync->error = 0u;
    for (int64_t i = first; i < na + nb; i += stride) {
        unsigned long long* p = reinterpret_cast<unsigned long long*>(i < na ? a + i : b + (i - na));
        *p = sampler::kEmptySlot;
    }
}

const void* pick_grid_kernel(const DataView& dv, bool adapt)
{
    if (adapt) return dv.dtype == NUTS_F64 ? grid_kernel_ext_f64(dv) : grid_kernel_ext_f32(dv);
    return dv.dtype == NUTS_F64 ? grid_kernel_f64(dv) : grid_kernel_f32(dv);
}

const void* pick_team_kernel(const DataView& dv, bool ext)
{
    if (ext) return dv.dtype == NUTS_F64 ? team_kernel_ext_f64(dv.D) : team_kernel_ext_f32(dv.D);
    return dv.dtype == NUTS_F64 ? team_kernel_f64(dv.D) : team_kernel_f32(dv.D);
}

}  // namespace

bool wave_path_supports(const DataView& dv) { return dv.D <= 64; }

int wave_path_resident(const SamplerArgs& a)
{
    return a.data.dtype == NUTS_F64 ? wave_resident_f64(a) : wave_resident_f32(a);
}

hipError_t launch_sampler_wave(const SamplerArgs& a, hipStream_t stream)
{
    if (sampler_extended(a))
        return a.data.dtype == NUTS_F64 ? launch_sampler_wave_ext_f64(a, stream)
                                        : launch_sampler_wave_ext_f32(a, stream);
    return a.data.dtype == NUTS_F64 ? launch_sampler_wave_f64(a, stream) : launch_sampler_wave_f32(a, stream);
}

namespace {

// What an evaluation takes, in microseconds, fitted to runs of the paths over N
// = 1 to 200,000 rows, D = 1 to 300 and 1 to 600 chains (within 15 %, the
// streaming kernel at 17 to 32 columns within 30 %).
//  - The wave path: the tree step and the reductions, and per 64 rows (of its
//    row blocks) what the lanes of a row repeat of its row terms, the rows in
//    LDS or streamed.
//  - A team on a lone group: the first round of tiles over its workers, and
//    as many more tiles; with an exchange between groups a step and a round.
//  - The streaming grid kernel: a step, and 64 rows of a group.  Rows beyond the
//    caches are read from memory at 6.3 TB/s, shared ones once for all the
//    chains of a launch, which go through them at the same pace.
struct PathCost {
    double wave_step, wave_lds, wave_stream, lone_first, lone_round, team_step, team_round, stream_step, stream_tile;
};
PathCost path_cost(const DataView& dv)
{
    static const PathCost f64[] = {{1.36, 0.22, 0.32, 1.6, 0.62, 3.4, 0.52, 4.7, 0.07},
                                   {1.62, 0.27, 0.39, 1.58, 0.9, 4.0, 0.42, 9.6, 0.13},
                                   {1.34, 1.3, 3.4, 1.8, 1.1, 4.7, 0.25, 4.5, 0.72},
                                   {1.3, 2.7, 3.5, 2.15, 1.1, 5.0, 0.4, 5.1, 0.83},
                                   {0, 0, 0, 0, 0, 0, 0, 7.5, 1.4},
                                   {0, 0, 0, 0, 0, 0, 0, 8.0, 2.9},
                                   {0, 0, 0, 0, 0, 0, 0, 11.0, 3.2}};
    static const PathCost f32[] = {{1.3, 0.135, 0.19, 1.46, 0.28, 3.5, 0.24, 4.5, 0.034},
                                   {1.62, 0.17, 0.74, 1.5, 0.42, 3.7, 0.33, 7.6, 0.083},
                                   {1.48, 0.57, 2.0, 1.65, 0.95, 4.1, 0.42, 4.6, 0.37},
                                   {1.4, 1.16, 2.45, 2.1, 0.9, 5.0, 0.4, 4.6, 0.4},
                                   {0, 0, 0, 0, 0, 0, 0, 7.0, 0.7},
                                   {0, 0, 0, 0, 0, 0, 0, 8.0, 1.4},
                                   {0, 0, 0, 0, 0, 0, 0, 10.7, 1.7}};
    const int D = dv.D;  // up to 8, 16, 32, 64, 128, 256 columns, and beyond
    const int c = D <= 8 ? 0 : D <= 16 ? 1 : D <= 32 ? 2 : D <= 64 ? 3 : D <= 128 ? 4 : D <= 256 ? 5 : 6;
    return dv.dtype == NUTS_F64 ? f64[c] : f32[c];
}
constexpr int64_t kMaxLaunchChains = 1 << 20;  // lone groups a launch
constexpr double kCachedBytes = 200e6;     // of the 256 MB cache beside the memory
constexpr double kStreamBytesPerUs = 6.3e6;
double launches(int64_t chains, int64_t per_launch) { return (double)((chains + per_launch - 1) / per_launch); }
GridPlan team_plan(const DataView& dv, int64_t num_chains, int64_t groups, int64_t chains, int64_t tiles)
{
    const PathCost pc = path_cost(dv);
    constexpr int64_t kWorkers = kTeamWaves - 1;
    const double step = groups == 1
                            ? pc.lone_first + pc.lone_round * (double)std::max<int64_t>(tiles - kWorkers, 0) / kWorkers
                            : pc.team_step + pc.team_round * (double)((tiles + kWorkers - 1) / kWorkers);
    return GridPlan{(int)groups, (int)chains, (int)tiles, launches(num_chains, chains) * step};
}

// The team for these chains: as many at a time as the groups that hold a
// chain's rows in LDS leave room for; team = 0 if the device does not hold one.
GridPlan plan_team(const DataView& dv, int max_depth, int sub_merge, int64_t num_chains, int num_cu)
{
    constexpr int kWorkers = kTeamWaves - 1;
    const size_t used = grid_resident_offset(dv.D, max_depth, sub_merge) +
                        sizeof(sampler::GridShared<1, kTeamWaves>) + 64;
    if (used >= sampler::kMaxGroupLds) return GridPlan{};
    const int64_t nt = (dv.N + 63) / 64;
    const int64_t cap = (int64_t)((sampler::kMaxGroupLds - used) / team_tile_bytes(dv.dtype, dv.D));  // tiles a group
    if (cap < 1) return GridPlan{};
    const int64_t lone = kWorkers * (dv.dtype == NUTS_F64 ? kTeamLoneRounds64 : kTeamLoneRounds32);
    if (nt <= lone && nt <= cap) {
        // lone groups wait for no other: one launch of all chains, a CU taking
        // the next chain when it is done with one
        GridPlan p = team_plan(dv, num_chains, 1, num_cu, nt);
        p.chains = (int)std::min<int64_t>(num_chains, kMaxLaunchChains);
        return p;
    }
    const int64_t fit = (nt + cap - 1) / cap;  // the fewest groups that hold the rows
    if (fit > num_cu) return GridPlan{};
    // launches of equal size
    const int64_t most = std::min<int64_t>(num_chains, num_cu / fit);
    const int64_t n = (num_chains + most - 1) / most;
    const int64_t chains = (num_chains + n - 1) / n;
    const int64_t per_group = std::min<int64_t>(cap, kWorkers);
    const int64_t groups = std::min<int64_t>(num_cu / chains, std::max(fit, (nt + per_group - 1) / per_group));
    return team_plan(dv, num_chains, groups, chains, (nt + groups - 1) / groups);
}

// The streaming launches of these chains.  Chains on one group each leave CUs
// idle unless they are as many, and a last launch of few chains takes as long as
// a full one: fewer chains at a time on more groups each can be ahead (130
// chains on 1,000,000 x 100 fp64, ms a step: 23.3 all at once, 15.8 in two
// launches, 13.3 in ten, 15.3 in 26, 18.3 one after another; on 20,000 x 300
// 0.95, 0.66, 0.70, 1.15 and 2.54).  Fewer only where the gain is 4 %: the more
// chains a launch has, the more they share of what they read.
GridPlan plan_stream(const DataView& dv, int64_t num_chains, int num_cu)
{
    const PathCost pc = path_cost(dv);
    const double tiles = (double)((dv.N + 63) / 64);
    const double set_bytes = (double)dv.N * dv.D * (dv.dtype == NUTS_F64 ? 8.0 : 4.0);
    // no more groups than the rows' blocks give work; and a group gathers the
    // partials of its used columns in one pass of its worker lanes: ceil((D +
    // 1) / groups) * groups <= D + groups slots
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>((dv.nb + kGridWaves - 2) / (kGridWaves - 1),
                                                               (int64_t)(kGridWaves - 1) * kWave - dv.D));
    GridPlan best{};
    for (int64_t chains = std::min<int64_t>(num_chains, num_cu); chains >= 1; --chains) {
        const int64_t groups = std::min<int64_t>(num_cu / chains, most);
        const double bytes = set_bytes * (dv.nds > 1 ? (double)chains : 1.0);  // a launch's rows
        const double memory = bytes > kCachedBytes ? bytes / kStreamBytesPerUs : 0.0;
        const double step = std::max(pc.stream_step + pc.stream_tile * tiles / (double)groups, memory);
        const double us = launches(num_chains, chains) * step;
        if (best.groups == 0 || us < 0.96 * best.us) best = GridPlan{(int)groups, (int)chains, 0, us};
    }
    return best;
}

}  // namespace

GridPlan plan_grid_sampler(const DataView& dv, int max_depth, int sub_merge, int64_t num_chains, int num_cu)
{
    const GridPlan stream = plan_stream(dv, num_chains, num_cu);
    if (dv.D <= kWave) {
        const GridPlan team = plan_team(dv, max_depth, sub_merge, num_chains, num_cu);
        if (team.groups > 0 && team.us < stream.us) return team;
    }
    const void* k = pick_grid_kernel(dv, sub_merge != 0);
    int per_cu = 0;
    const size_t lds = (size_t)chain_lds_doubles(dv.D, max_depth, sub_merge, grid_edge_nodes(dv.D)) * sizeof(double);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kGridWaves * kWave, lds) != hipSuccess)
        per_cu = 1;
    else if (per_cu < 1)
        return GridPlan{};  // the group's LDS does not fit a CU
    return stream;
}

bool grid_beats_wave(const SamplerArgs& a, const GridPlan& plan, int num_cu)
{
    if (plan.groups == 0) return false;
    const int cpg = wave_path_resident(a);
    const int64_t slots = (int64_t)num_cu * (cpg > 0 ? cpg : 12);
    const PathCost pc = path_cost(a.data);
    const double tile = cpg > 0 ? pc.wave_lds : pc.wave_stream;
    // (by its blocks: a few rows do not cost it 64)
    const double tiles = (double)(a.data.nb * rows_per_block(a.data)) / 64.0;
    // (level: the wave path, which fills no LDS of its own before the first step
    // and exchanges nothing)
    return plan.us < 0.95 * launches(a.num_chains, slots) * (pc.wave_step + tile * tiles);
}

hipError_t launch_sampler_grid(const SamplerArgs& a, const GridPlan& plan, double* partials, double* result,
                               GridSync* sync, bool clear_error, hipStream_t stream, hipEvent_t at_launch)
{
    hipError_t e = hipSuccess;
    int groups = plan.groups;
    const bool lone = plan.team > 0 && groups == 1;
    if (!lone) {
        hipLaunchKernelGGL(fill_empty_slots, dim3(64), dim3(256), 0, stream, partials,
                           a.num_chains * grid_partial_elems(a.data.D, groups), result,
                           a.num_chains * grid_result_elems(groups), clear_error ? sync : nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool ext = sampler_extended(a);
    const size_t chain = grid_resident_offset(a.data.D, a.max_depth, a.sub_merge);
    const void* k;
    int res = 0;
    size_t lds;
    if (plan.team > 0) {
        k = pick_team_kernel(a.data, ext);
        lds = chain + (size_t)plan.team * team_tile_bytes(a.data.dtype, a.data.D);
    } else {
        // the chain's state, then as many resident blocks a worker as the
        // rest of the group's LDS holds (at most one fewer than the smallest
        // share)
        k = pick_grid_kernel(a.data, ext);
        hipFuncAttributes attr;
        e = hipFuncGetAttributes(&attr, k);
        if (e != hipSuccess) return e;
        const size_t block = (size_t)lds_block_bytes(a.data.dtype, a.data.split, a.data.cols);
        const size_t used = attr.sharedSizeBytes + chain;
        int64_t resident = used < sampler::kMaxGroupLds ? (int64_t)((sampler::kMaxGroupLds - used) / ((kGridWaves - 1) * block)) : 0;
        const int64_t smallest_share = a.data.nb / ((int64_t)groups * (kGridWaves - 1));
        if (resident > smallest_share - 1) resident = smallest_share > 1 ? smallest_share - 1 : 0;
        res = (int)resident;
        lds = chain + (size_t)res * (kGridWaves - 1) * block;
    }
    e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (at_launch) {
        e = hipEventRecord(at_launch, stream);
        if (e != hipSuccess) return e;
    }
    SamplerArgs A = a;
    void* stream_args[] = {&A, &groups, &res, &partials, &result, &sync};
    void* team_args[] = {&A, &groups, &partials, &result, &sync};
    void** args = plan.team > 0 ? team_args : stream_args;
    const dim3 grid((unsigned)(a.num_chains * groups)), threads((plan.team > 0 ? kTeamWaves : kGridWaves) * kWave);
    // lone groups wait for no other group: an ordinary launch
    if (lone) return hipLaunchKernel(k, grid, threads, args, lds, stream);
    return hipLaunchCooperativeKernel(k, grid, threads, args, (unsigned)lds, stream);
}

}  // namespace nuts
