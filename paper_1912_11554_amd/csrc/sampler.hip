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

// What an evaluation takes, in microseconds, from runs of both paths over N =
// 60 to 100,000 rows, D = 3 to 60 and 1 to 2,500 chains.
//  - The wave path: 1.5 for the tree step and the reductions, and per 64 rows
//    what the lanes of a row repeat of its row terms (0.3 fp64, 0.2 fp32 with
//    one lane a row; 1.5, 1.1 with four; 3.7, 1.5 with eight).
//  - A team: 1.7 (3.7 with an exchange between groups) and 0.35 a round of
//    tiles over a group's workers.
//  - The streaming grid kernel: 5, and per 64 rows of a group about a quarter
//    of the wave path's (its fp64 rows of 16 slots spill: 0.35).
struct PathCost {
    double wave_tile, stream_tile;
};
PathCost path_cost(const DataView& dv)
{
    const bool f64 = dv.dtype == NUTS_F64;
    if (dv.split == 1) return {f64 ? 0.3 : 0.2, dv.cols == 16 ? 0.35 : 0.1};
    if (dv.split == 4) return {f64 ? 1.5 : 1.1, f64 ? 0.5 : 0.25};
    return {f64 ? 3.7 : 1.5, f64 ? 0.9 : 0.4};
}
double launches(int64_t chains, int64_t per_launch) { return (double)((chains + per_launch - 1) / per_launch); }
double team_cost(const GridPlan& p, int64_t chains)
{
    const int rounds = (p.team + kTeamWaves - 2) / (kTeamWaves - 1);
    return launches(chains, p.chains) * ((p.groups == 1 ? 1.7 : 3.7) + 0.35 * rounds);
}

// The team for these chains: as many at a time as the groups that hold a
// chain's rows in LDS leave room for; team = 0 if the device does not hold one.
GridPlan plan_team(const DataView& dv, int max_depth, int sub_merge, int64_t num_chains, int num_cu)
{
    constexpr int kWorkers = kTeamWaves - 1;
    const size_t used = grid_resident_offset(dv.D, max_depth, sub_merge) +
                        sizeof(sampler::GridShared<1, kTeamWaves>) + 64;
    if (used >= sampler::kMaxGroupLds) return GridPlan{0, 0, 0};
    const int64_t nt = (dv.N + 63) / 64;
    const int64_t cap = (int64_t)((sampler::kMaxGroupLds - used) / team_tile_bytes(dv.dtype, dv.D));  // tiles a group
    if (cap < 1) return GridPlan{0, 0, 0};
    const int64_t lone = kWorkers * (dv.dtype == NUTS_F64 ? kTeamLoneRounds64 : kTeamLoneRounds32);
    if (nt <= lone && nt <= cap) return GridPlan{1, (int)std::min<int64_t>(num_chains, num_cu), (int)nt};
    const int64_t fit = (nt + cap - 1) / cap;  // the fewest groups that hold the rows
    if (fit > num_cu) return GridPlan{0, 0, 0};
    // launches of equal size
    const int64_t most = std::min<int64_t>(num_chains, num_cu / fit);
    const int64_t n = (num_chains + most - 1) / most;
    const int64_t chains = (num_chains + n - 1) / n;
    const int64_t per_group = std::min<int64_t>(cap, kWorkers);
    const int64_t groups = std::min<int64_t>(num_cu / chains, std::max(fit, (nt + per_group - 1) / per_group));
    return GridPlan{(int)groups, (int)chains, (int)((nt + groups - 1) / groups)};
}

}  // namespace

GridPlan plan_grid_sampler(const DataView& dv, int max_depth, int sub_merge, int64_t num_chains, int num_cu)
{
    const int chains = (int)std::min<int64_t>(num_chains, num_cu);
    int64_t groups = num_cu / chains;  // streaming: the device shared out to the chains
    groups = std::max<int64_t>(1, std::min<int64_t>(groups, (dv.nb + kGridWaves - 2) / (kGridWaves - 1)));
    if (dv.D <= kWave) {
        const GridPlan team = plan_team(dv, max_depth, sub_merge, num_chains, num_cu);
        const double stream = launches(num_chains, chains) *
                              (5.0 + path_cost(dv).stream_tile * (double)((dv.N + 63) / 64) / (double)groups);
        if (team.team > 0 && team_cost(team, num_chains) < stream) return team;
    }
    const void* k = pick_grid_kernel(dv, sub_merge != 0);
    int per_cu = 0;
    const size_t lds = (size_t)chain_lds_doubles(dv.D, max_depth, sub_merge, grid_edge_nodes(dv.D)) * sizeof(double);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kGridWaves * kWave, lds) != hipSuccess)
        per_cu = 1;
    else if (per_cu < 1)
        return GridPlan{0, 0, 0};  // the group's LDS does not fit a CU
    // a group gathers the partials of its used columns in one pass of its
    // worker lanes: ceil((D + 1) / groups) * groups <= D + groups slots
    groups = std::min<int64_t>(groups, (int64_t)(kGridWaves - 1) * kWave - dv.D);
    return GridPlan{(int)groups, chains, 0};
}

// A streaming launch and the wave path read the rows at the same rate per CU,
// so the grid path is ahead while the chains leave the wave path's slots empty
// (4 chains on 100,000 x 50 fp64: 24 us an evaluation against 7,400).
bool grid_beats_wave(const SamplerArgs& a, const GridPlan& plan, int num_cu)
{
    if (plan.groups == 0) return false;
    if (plan.team == 0) return a.num_chains <= num_cu;
    const int cpg = wave_path_resident(a);
    const int64_t slots = (int64_t)num_cu * (cpg > 0 ? cpg : 12);
    const double wave =
        launches(a.num_chains, slots) * (1.5 + (double)((a.data.N + 63) / 64) * path_cost(a.data).wave_tile);
    return team_cost(plan, a.num_chains) < wave;
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
