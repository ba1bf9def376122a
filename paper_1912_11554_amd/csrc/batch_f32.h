// The batched contraction on the fp32 matrix-core instruction, for the sampler
// kernels with the optional features.  (With the bf16 parts of batch.h those
// kernels faulted the GPU in a run of 24 chains with merge-structured subtree
// proposals on 500 x 129: at 117 to 132 columns the loop the compiler then made
// of a position load from a per-lane base overwrote that base, see buffer_of in
// batch.hip.  The loads have one base a wave now; these kernels have not been
// moved since.)
//
// Layout of a stage in memory: 64 rows of `stride32` floats; the first 16 kp of
// a row (kp = kt rounded up to a multiple of 4) hold the matrix columns,
// permuted: slot g * kp + t holds column 16 t + g (zero for t >= kt), so that
// the 16-column chunks t of one column residue g are contiguous.  The last 4
// floats hold the tail columns.  Labels one byte a row.
//
// Operand layout of v_mfma_f32_16x16x4f32 (one 16x16 block): lane l gives
// A[l % 16][l / 16] and B[l / 16][l % 16]; result register r of lane l is
// C[4 (l / 16) + r][l % 16].  The contraction index of instruction (chunk t,
// sub-step i) is column 16 t + 4 (l / 16) + i, so that each lane reads four
// consecutive columns of its row with one 16-byte LDS load.  For G the
// contraction index of sub-step r is row 4 (l / 16) + r: exactly the rows whose
// residuals the lane already holds in register r of the E result.
#pragma once

#include "batch.h"

namespace nuts {
namespace batch32 {

using batch::kTail;
using batch::kTileRows;
using batch::kTiles;
using batch::kWaves;
using batch::row_terms;
using batch::v4f;
using batch::WaveAcc;

constexpr int kMaxStride = 16 * kBatchMaxKT + kTail;        // 132 floats per row in HBM

// LDS geometry of a stage for KT chunks.  The HBM row (16 KP permuted
// matrix-core slots, then the tail) is spread out so that column residue g
// starts at g * GS: GS = 12 for KP = 8 (two 16-byte pieces per residue) and
// 4 for KP = 4, and the row stride RS = 16 GS + 4 is 4 mod 64 floats.  With
// these, a 16-lane phase of every 16-byte LDS read below (16 rows at one
// residue, or 16 residues of one row) touches 64 distinct banks.
template <int KT>
struct Geo {
    static constexpr int KP = (KT + 3) / 4 * 4;
    static constexpr int GS = KP == 8 ? 12 : 4;
    static constexpr int RS = 16 * GS + 4;
    static constexpr int HS = 16 * KP + 4;          // HBM row: floats
    static constexpr int HV = HS / 4;               // HBM row: 16-byte pieces
};
constexpr int kStageFloats = kBatchStageRows * Geo<kBatchMaxKT>::RS;  // largest LDS stage
constexpr int kStageBuf = kStageFloats + 4;                          // plus one junk 16-byte slot
constexpr int kStageVecs = (kBatchStageRows * kMaxStride / 4 + kWaves * kWave - 1) / (kWaves * kWave);

// Column of the matrix-core operand that lane group jj reads as component i
// of its 16-byte piece in chunk t of the column contraction (E = X Q):
// piece f = 4 t + jj of the row is residue g, half h of the permuted slots.
template <int KT>
__host__ __device__ constexpr int e_column(int t, int jj, int i)
{
    constexpr int KP = Geo<KT>::KP;
    const int f = 4 * t + jj;
    const int g = KP == 8 ? f >> 1 : f;
    const int h = KP == 8 ? f & 1 : 0;
    return 16 * (4 * h + i) + g;   // chunk 4 h + i (valid if < KT), residue g
}

__device__ __forceinline__ v4f mfma(float a, float b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// A wave's share of the positions: Q in the B-operand order of the column
// contraction (q[4 t + i] = Q[e_column(t, l / 16, i)][l % 16], zero where
// that chunk is >= KT) and the tail.
struct WaveQ {
    float q[4 * kBatchMaxKT];
    float qt[kTail];
};

// Registers of one stage on its way from HBM to LDS; thread `tid` of the
// kWaves * 64 loaders moves 16-byte pieces tid, tid + 512, ...
struct StageRegs {
    v4f v[kStageVecs];  // clang vector type: HIP's float4 class would pin the registers to scratch
    uint32_t y;
};

// The piece offsets are recomputed at every stage (the sampler kernel's nine
// waves leave 168 registers a lane): hoisted out of the stage loop they were
// kept in scratch memory there, and each reload waited for every load issued
// before it, so the stage's loads went out one by one.
__device__ __forceinline__ void load_stage(const BatchView& bv, int64_t st, int tid, StageRegs& r)
{
    int opaque_zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(opaque_zero));
    tid += opaque_zero;
    const int last = kBatchStageRows * bv.stride32 / 4 - 1;
    const v4f* src = reinterpret_cast<const v4f*>(bv.X32 + st * kBatchStageRows * bv.stride32);
    const uint32_t* ysrc = reinterpret_cast<const uint32_t*>(bv.y32 + st * kBatchStageRows);
    // the labels first: whatever their address waits for (a
    // register reloaded from scratch waits for every load before it) is then
    // not the stage's pieces
    if (tid < kBatchStageRows / 4) r.y = ysrc[tid];
    // unconditional loads (pieces past the stage re-read its last piece and
    // are not stored), so the loop unrolls into straight-line code
#pragma unroll
    for (int i = 0; i < kStageVecs; ++i) r.v[i] = src[min(tid + i * kWaves * kWave, last)];
}

// Scatter a stage into the LDS geometry: HBM piece q of a row goes to
// residue q / (KP / 4), half q % (KP / 4); the last piece is the tail.
// The destinations are recomputed at every stage (a few integer instructions)
// instead of reloaded from scratch.
template <int KT>
__device__ __forceinline__ void store_stage(const StageRegs& r, int tid, float* xs, float* ys)
{
    using G = Geo<KT>;
    constexpr int last = kBatchStageRows * G::HV - 1;
    int opaque_zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(opaque_zero));
    tid += opaque_zero;
#pragma unroll
    for (int i = 0; i < kStageVecs; ++i) {
        const int idx = tid + i * kWaves * kWave;
        const int row = idx / G::HV;
        const int q = idx - row * G::HV;
        int dst;
        if constexpr (G::KP == 8) dst = q < 32 ? (q >> 1) * 3 + (q & 1) : 4 * G::GS;
        else dst = q < 4 * G::KP ? q : 4 * G::GS;  // KP = 4: one piece per residue
        dst += row * (G::RS / 4);
        // pieces past the stage go to a junk slot after the buffer (never read)
        reinterpret_cast<v4f*>(xs)[idx <= last ? dst : kStageFloats / 4] = r.v[i];
    }
    if (tid < kBatchStageRows / 4) {
        // labels as signs 1 - 2y
        v4f sg;
#pragma unroll
        for (int k = 0; k < 4; ++k) sg[k] = ((r.y >> (8 * k)) & 1u) ? -1.0f : 1.0f;
        reinterpret_cast<v4f*>(ys)[tid] = sg;
    }
}

// All four 16-row tiles of one LDS stage for this wave's 16 positions, two
// tiles at a time so that two independent accumulation chains alternate on
// the matrix core.  KT is the chunk count; the four tail slots are always
// processed (slots past the tail hold zero columns and zero positions, so
// they add nothing).
//
// `flip` reverses the pair order: the two waves that share a SIMD (loader
// index w and w + 4) take the pairs in opposite orders.  Each wave raises its
// issue priority while it feeds the matrix core and lowers it for the row
// terms: left to the default (the older wave first), the younger wave of a
// SIMD fell a third behind within each stage and the older one waited for it
// at the stage barrier.
template <int KT>
__device__ __forceinline__ void compute_stage(const float* __restrict__ xs, const float* __restrict__ ys,
                                              const WaveQ& Q, WaveAcc& acc, bool flip, int pair_lo, int pair_hi)
{
    using G = Geo<KT>;
    const int l = lane();
    const int m = l & 15;
    const int jj = l >> 4;
    // this lane's piece of chunk 0 in its E row, and its G residue
    const int e_off = m * G::RS + (G::KP == 8 ? 12 * (jj >> 1) + 4 * (jj & 1) : 4 * jj);
    constexpr int e_step = G::KP == 8 ? 24 : 16;
    const int g_off = 4 * jj * G::RS + m * G::GS;
#pragma unroll 1
    for (int step = 0; step < kTiles; step += 2) {
        const int tp = flip ? kTiles - 2 - step : step;
        if (tp / 2 < pair_lo || tp / 2 >= pair_hi) continue;  // uniform: another group's rows
        const float* x0 = xs + tp * kTileRows * G::RS;
        const float* x1 = x0 + kTileRows * G::RS;
        v4f e0 = {0.0f, 0.0f, 0.0f, 0.0f};
        v4f e1 = {0.0f, 0.0f, 0.0f, 0.0f};
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int t = 0; t < G::KP; ++t) {
            const v4f a0 = *reinterpret_cast<const v4f*>(x0 + e_off + e_step * t);
            const v4f a1 = *reinterpret_cast<const v4f*>(x1 + e_off + e_step * t);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                e0 = mfma(a0[i], Q.q[4 * t + i], e0);
                e1 = mfma(a1[i], Q.q[4 * t + i], e1);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        // tail slots of this lane's four rows 4 jj + r of both tiles
        v4f xr0[4], xr1[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            xr0[r] = *reinterpret_cast<const v4f*>(x0 + (4 * jj + r) * G::RS + 16 * G::GS);
            xr1[r] = *reinterpret_cast<const v4f*>(x1 + (4 * jj + r) * G::RS + 16 * G::GS);
            e0[r] += ((xr0[r][0] * Q.qt[0] + xr0[r][1] * Q.qt[1]) + xr0[r][2] * Q.qt[2]) + xr0[r][3] * Q.qt[3];
            e1[r] += ((xr1[r][0] * Q.qt[0] + xr1[r][1] * Q.qt[1]) + xr1[r][2] * Q.qt[2]) + xr1[r][3] * Q.qt[3];
        }
        const v4f s0 = *reinterpret_cast<const v4f*>(ys + tp * kTileRows + 4 * jj);
        const v4f s1 = *reinterpret_cast<const v4f*>(ys + (tp + 1) * kTileRows + 4 * jj);
        float r0[4], r1[4];
        float lsum = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float l0, l1;
            row_terms(e0[r], s0[r], l0, r0[r]);
            row_terms(e1[r], s1[r], l1, r1[r]);
            lsum += l0 + l1;
        }
        acc.loss += (double)lsum;
        __builtin_amdgcn_s_setprio(2);
        // G: residue m of row 4 jj + r holds chunks 4 h .. 4 h + 3 in piece h
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int h = 0; h < G::KP / 4; ++h) {
                const v4f b0 = *reinterpret_cast<const v4f*>(x0 + g_off + r * G::RS + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * h + i < KT) acc.g[4 * h + i] = mfma(b0[i], r0[r], acc.g[4 * h + i]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int h = 0; h < G::KP / 4; ++h) {
                const v4f b1 = *reinterpret_cast<const v4f*>(x1 + g_off + r * G::RS + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * h + i < KT) acc.g[4 * h + i] = mfma(b1[i], r1[r], acc.g[4 * h + i]);
            }
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int k = 0; k < kTail; ++k) {
            acc.gt[k] += ((xr0[0][k] * r0[0] + xr0[1][k] * r0[1]) + xr0[2][k] * r0[2]) + xr0[3][k] * r0[3];
            acc.gt[k] += ((xr1[0][k] * r1[0] + xr1[1][k] * r1[1]) + xr1[2][k] * r1[2]) + xr1[3][k] * r1[3];
        }
    }
}

// The stage loop over the halves [h0, h1) (stages h0 / 2 .. (h1 - 1) / 2)
// with double-buffered LDS stages.  Workers (tid = loader index, 0 .. 511)
// load and compute; a non-worker wave of the same group passes the same
// workgroup barriers (one more than the stages) and does nothing else.
template <int KT, bool WORKER>
__device__ __forceinline__ void stage_loop(const BatchView& bv, int64_t h0, int64_t h1, int tid, float* xs,
                                           float* ys, const WaveQ& Q, WaveAcc& acc)
{
    const int64_t st0 = h0 / 2;
    const int64_t st1 = h1 > h0 ? (h1 + 1) / 2 : st0;
    if constexpr (!WORKER) {
        for (int64_t st = st0; st <= st1; ++st) __syncthreads();
    } else {
        if (st0 < st1) {
            StageRegs r;
            load_stage(bv, st0, tid, r);
            store_stage<KT>(r, tid, xs, ys);
        }
        __syncthreads();
        for (int64_t st = st0; st < st1; ++st) {
            const int b = (int)((st - st0) & 1);
            const bool more = st + 1 < st1;
            StageRegs r;
            if (more) load_stage(bv, st + 1, tid, r);
            // the halves of this stage that are the group's
            const int lo = (int)(h0 > 2 * st ? h0 - 2 * st : 0);
            const int hi = (int)(h1 < 2 * st + 2 ? h1 - 2 * st : 2);
            compute_stage<KT>(xs + b * kStageBuf, ys + b * kBatchStageRows, Q, acc, tid >= 4 * kWave, lo, hi);
            if (more) store_stage<KT>(r, tid, xs + (b ^ 1) * kStageBuf, ys + (b ^ 1) * kBatchStageRows);
            __syncthreads();
        }
    }
}

}  // namespace batch32
}  // namespace nuts
