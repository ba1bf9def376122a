// Device side of the batched-chain contraction on the gfx950 matrix cores.
//
// One workgroup owns a range of 64-row stages and a tile of 128 positions
// (chains).  Eight waves each take 16 positions; the stage rows are staged in
// LDS once and read by all eight.  Per pair of 16-row tiles a wave computes
//   E[16 rows x 16 positions] = X_tile . Q          (contraction over columns)
//   loss and residual of every (row, position) on E
//   G[D x 16] += X_tile^T . R                       (contraction over rows)
// with G held in registers across the whole row range.
//
// The products are fp32 products on the bf16 matrix cores (16 times the rate
// of the fp32 ones).  Every fp32 factor is split into three bf16 parts, x = x1
// + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2): 8
// bits each, so the three hold all 24 bits of x and the split is exact for |x|
// >= 2^-110 (x1 of values that would round to infinity is held to the largest
// bf16 value); below that the bits of x under 2^-133 are not bf16 values, and
// the sum of the parts is off by at most 2^-134.  x q is then the sum of nine
// products of bf16 parts, each exact in fp32; the six of x1 q1, x1 q2, x2 q1,
// x1 q3, x2 q2 and x3 q1 are taken, and the three left out are below 2^-25
// |x q| together, under half the rounding of one fp32 multiply-add.  The sums are the matrix
// cores' fp32 accumulations over 32 products at a time (the fp32 instruction
// rounded after every four).  Against 64-bit arithmetic the gradient of 256
// positions on 200,000 x 129 is off by 7.4e-7 (8.5e-7 with the fp32
// instruction), the log-likelihood of 500 draws over 581,012 x 55 by 2.1e-9
// (2.2e-9).  256 positions on 200,000 x 129 take 181 to 185 us a call, from 264.
// Of the pass's cycles the matrix cores are busy in 45 %, the vector ALUs with
// other instructions in 42 %, LDS in 31 % (six reads of every element a wave, no
// bank conflict), with two waves a SIMD to overlap them: reading the next step's
// operands ahead of the current products changed nothing, and holding the
// corrections to the finite range costs 5 to 7 %.
//
// v_mfma_f32_16x16x32_bf16: lane l gives A[l % 16][8 (l / 16) + i] and
// B[8 (l / 16) + i][l % 16], i < 8; result register r of lane l is
// C[4 (l / 16) + r][l % 16].  For E the contraction index 8 (l / 16) + i of
// K-step t is column 32 t + 8 (l / 16) + i: one 16-byte LDS read a part.  For G
// the contraction index 8 (l / 16) + i is row 4 (l / 16) + i of the pair's
// first tile (i < 4) or row 4 (l / 16) + i - 4 of its second: exactly the rows
// whose residuals the lane already holds from the E results, so R feeds the
// second product without any data movement; its X operand, a column's four
// rows, comes from the row-major stage by transposing LDS reads
// (ds_read_b64_tr_b16: lane i of 16 receives element i of each of the four
// rows the 16 lanes read).
//
// The row terms use the fp32 hardware exp/log/rcp; the loss is accumulated in
// fp64 per lane and all partial rows are added in fp64 in a fixed order.
#pragma once

#include "device.h"
#include "launch.h"

namespace nuts {
namespace batch {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;                                   // matrix-core waves per group
constexpr int kTileRows = 16;
constexpr int kTiles = kBatchStageRows / kTileRows;         // MFMA tiles per stage
constexpr int kTail = 4;
constexpr int kParts = 3;                                   // bf16 parts of a factor

// Geometry of a stage image (the same in memory and in LDS): three planes (the
// bf16 parts) of 64 rows of kCols columns, then the tail columns (fp32, four a
// row), then the labels as signs 1 - 2 y (fp32).  A row is kSlots 16-byte
// slots; slot s of row r sits at position s ^ swizzle(r).  With it every phase
// of the LDS reads touches all 64 banks once: a phase of the column
// contraction's 16-byte reads takes lanes 0..3, 12..15 and 20..27 (or the other
// 16 of a half wave), that is all 16 rows, rows 4..11 at the neighbour of the
// others' slot; a phase of the row contraction's 8-byte reads takes 32 lanes,
// 8 rows with two neighbouring slots each.
template <int KT>
struct Geo {
    static constexpr int kCols = batch_cols(KT);
    static constexpr int kSteps = (KT + 1) / 2;              // K-steps of 32 columns
    static constexpr int kSlots = kCols / 8;
    static constexpr int kRow = kCols * 2;                   // bytes
    static constexpr int kPlane = kBatchStageRows * kRow;
    static constexpr int kTailAt = kParts * kPlane;
    static constexpr int kSignAt = kTailAt + kBatchStageRows * kTail * 4;
    static constexpr int kBytes = kSignAt + kBatchStageRows * 4;
    static_assert(kBytes == batch_stage_bytes(KT), "the host sizes stages as the kernels read them");
};

// bf16 parts of two fp32 values of at most the largest bf16 value, infinities or
// NaN.
__device__ __forceinline__ void split3(v2f x, v2bf& a, v2bf& b, v2bf& c)
{
    a = __builtin_convertvector(x, v2bf);
    x -= __builtin_convertvector(a, v2f);  // exact
    b = __builtin_convertvector(x, v2bf);
    x -= __builtin_convertvector(b, v2f);  // exact
    c = __builtin_convertvector(x, v2bf);  // exact above 2^-110
}
// The largest bf16 value.  A finite value that would round to infinity keeps it
// as its first part (the rest has 16 bits, which the other two parts hold).
constexpr float kBf16Max = 0x1.fep127f;
__device__ __forceinline__ float first_part_range(float x)
{
    return fabsf(x) <= 0x1.fffffep127f ? __builtin_amdgcn_fmed3f(x, -kBf16Max, kBf16Max) : x;
}
// The same for any values.
__device__ __forceinline__ void split3_any(v2f x, v2bf& a, v2bf& b, v2bf& c)
{
    a = __builtin_convertvector((v2f{first_part_range(x[0]), first_part_range(x[1])}), v2bf);
    x -= __builtin_convertvector(a, v2f);  // exact
    b = __builtin_convertvector(x, v2bf);
    x -= __builtin_convertvector(b, v2f);  // exact
    c = __builtin_convertvector(x, v2bf);  // exact above 2^-110
}
// ANY: split3_any, else split3.
template <bool ANY>
__device__ __forceinline__ void split3(const float (&x)[8], v8bf (&out)[kParts])
{
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        v2bf a, b, c;
        if constexpr (ANY) split3_any(v2f{x[i], x[i + 1]}, a, b, c);
        else split3(v2f{x[i], x[i + 1]}, a, b, c);
        out[0][i] = a[0];
        out[0][i + 1] = a[1];
        out[1][i] = b[0];
        out[1][i + 1] = b[1];
        out[2][i] = c[0];
        out[2][i + 1] = c[1];
    }
}

__device__ __forceinline__ v4f mfma(v8bf a, v8bf b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A sum of corrections, held to the finite range.  Where a factor is infinite
// or a product leaves the fp32 range, the leading products x1 q1 (256 times
// the corrections) hold the infinity or NaN the fp32 product has, and the
// corrections hold inf - inf and inf * 0 on top of it: a NaN becomes
// -FLT_MAX here, which no infinity and no NaN notices.  One instruction a sum
// (the bound and its negation are one scalar register).
__device__ __forceinline__ v4f finite(v4f c)
{
    float big;
    asm("s_mov_b32 %0, 0x7f7fffff" : "=s"(big));
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = __builtin_amdgcn_fmed3f(c[r], -big, big);
    return c;
}

// Negative log-likelihood and residual of one (row, position) from eta in
// fp32, with sgn = 1 - 2y: t = sgn eta, loss = softplus(t) = max(t, 0) +
// ln 2 log2(1 + e), residual = sgn sigmoid(t), e = exp(-|t|); three
// transcendentals (exp2, log2, reciprocal) on the fp32 hardware units.  The
// rounding of 1 + e costs at most 2^-24 absolute per term (log1p accuracy is
// not needed for a sum of softplus values that are O(1) each; one logarithm
// for the product of four rows' 1 + e was 5 times as far off over 581,012
// rows).  Padding rows (zero X, y = 0) have eta = 0 exactly and add exactly
// ln 2 (in fp32) to the loss and nothing to the gradient; the caller subtracts
// them.
constexpr float kLn2f = 0.69314718055994531f;

__device__ __forceinline__ void row_terms(float eta, float sgn, float& loss, float& resid)
{
    const float t = sgn * eta;
    const float e = __builtin_amdgcn_exp2f(-fabsf(t) * 1.4426950408889634f);
    const float u = 1.0f + e;
    const float inv = __builtin_amdgcn_rcpf(u);
    loss = __builtin_fmaf(kLn2f, __builtin_amdgcn_logf(u), fmaxf(t, 0.0f));
    resid = sgn * ((t >= 0.0f ? 1.0f : e) * inv);
}

// A wave's share of the positions: the bf16 parts of Q in the B-operand order
// of the column contraction (q[p][t][i] = part p of Q[32 t + 8 (l / 16) +
// i][l % 16], zero past the matrix columns) and the tail in fp32.
struct WaveQ {
    v8bf q[kParts][kBatchMaxKT / 2];
    float qt[kTail];
};

// Q's parts from the columns v[t][i] of every K-step.  A wave with a value above
// the largest bf16 value takes a form of its own (one uniform branch: 256
// chains on 200,000 x 129 8,297 us; 8,672 with every value held to the range).
template <int STEPS>
__device__ __forceinline__ void split_positions(const float (&v)[STEPS > 0 ? STEPS : 1][8], WaveQ& Q)
{
    float top = 0.0f;
#pragma unroll
    for (int t = 0; t < STEPS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) top = __builtin_fmaxf(top, fabsf(v[t][i]));
    const bool any = __any(top > kBf16Max);
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        v8bf parts[kParts];
        if (any) split3<true>(v[t], parts);
        else split3<false>(v[t], parts);
#pragma unroll
        for (int p = 0; p < kParts; ++p) Q.q[p][t] = parts[p];
    }
}

struct WaveAcc {
    v4f g[kBatchMaxKT];  // G[16 mt + 4 (l / 16) + r][l % 16] in g[mt][r]
    float gt[kTail];     // tail columns, this lane's rows only
    double loss;         // this lane's (row, position) terms
};

__device__ __forceinline__ void zero(WaveAcc& a)
{
#pragma unroll
    for (int mt = 0; mt < kBatchMaxKT; ++mt) a.g[mt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < kTail; ++k) a.gt[k] = 0.0f;
    a.loss = 0.0;
}

// Copy stage st into LDS at `buf` straight from memory (no registers in
// between); thread tid of the kWaves * 64 loaders moves the 16-byte pieces
// tid, tid + 512, ...  The copies are outstanding memory operations of the
// wave until wait_stage.  (An instruction of the compiler's own would make it
// wait for them before every LDS read of the other buffer, which it cannot
// tell apart.  m0 is set and used inside one asm block; nothing else in these
// kernels keeps a value in it.  The five wait states before the load are those
// between a vector instruction that writes a scalar register, which may have
// just reloaded the address, and a memory instruction that reads it: the
// compiler does not see the load inside the block and adds none.)
template <int KT>
__device__ __forceinline__ void load_stage(const BatchView& bv, int64_t st, int tid, char* buf)
{
    constexpr int kPieces = Geo<KT>::kBytes / 16;
    constexpr int kThreads = kWaves * kWave;
    const char* src = reinterpret_cast<const char*>(bv.X) + st * Geo<KT>::kBytes;
    const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)buf;
    const uint32_t wave = __builtin_amdgcn_readfirstlane((uint32_t)(tid / kWave)) * (kWave * 16);
#pragma unroll
    for (int i = 0; i * kThreads < kPieces; ++i) {
        // a lane writes its piece 16 bytes past its neighbour's, from the
        // wave's LDS address in m0
        if ((i + 1) * kThreads <= kPieces || i * kThreads + tid < kPieces) {
            const uint32_t at = __builtin_amdgcn_readfirstlane(lds + i * kThreads * 16 + wave);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                         :
                         : "s"(at), "v"((uint32_t)tid * 16), "s"(src + i * kThreads * 16)
                         : "memory");
        }
    }
}

// Every outstanding memory operation of the wave, its copies among them.
__device__ __forceinline__ void wait_stage() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Position swizzle of the 16-byte slots of row r of a 16-row tile.
template <int KT>
__device__ __forceinline__ int swizzle(int r)
{
    constexpr int n = Geo<KT>::kSlots;
    if constexpr (n < 2) return 0;
    const int rr = r / (16 / n);  // rows that share the 64 banks
    const int middle = ((r >> 2) ^ (r >> 3)) & 1;  // rows 4 .. 11
    return (((rr & (n / 2 - 1)) << 1) | (rr / (n / 2))) ^ middle;
}

__device__ __forceinline__ v8bf read_rows(const char* p) { return *reinterpret_cast<const v8bf*>(p); }

__device__ __forceinline__ v4bf read_transposed(const char* p)
{
    const v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) v4s*)(__attribute__((address_space(3))) char*)const_cast<char*>(p));
    return __builtin_bit_cast(v4bf, v);
}

// E of the stage's tiles tp and tp + 1 for this wave's positions: the leading
// products and the corrections in accumulators of their own (four independent
// chains on the matrix core), then the tail columns where the data has any.
template <int KT>
__device__ __forceinline__ void columns(const char* xs, const WaveQ& Q, int tp, bool tail, v4f& e0, v4f& e1)
{
    using G = Geo<KT>;
    const int l = lane();
    const int m = l & 15;
    const int jj = l >> 4;
    e0 = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    e1 = e0;
    if constexpr (KT > 0) {
        v4f c0 = e0, c1 = e0;
        const char* row = xs + (tp * kTileRows + m) * G::kRow;
        const int at = (jj ^ swizzle<KT>(m)) * 16;
#pragma unroll
        for (int t = 0; t < G::kSteps; ++t) {
            const char* p0 = row + (at ^ (4 * t * 16));
            const char* p1 = p0 + kTileRows * G::kRow;
            const v8bf x0 = read_rows(p0), x1 = read_rows(p1);
            const v8bf y0 = read_rows(p0 + G::kPlane), y1 = read_rows(p1 + G::kPlane);
            const v8bf z0 = read_rows(p0 + 2 * G::kPlane), z1 = read_rows(p1 + 2 * G::kPlane);
            e0 = mfma(x0, Q.q[0][t], e0);
            e1 = mfma(x1, Q.q[0][t], e1);
            c0 = mfma(x0, Q.q[1][t], c0);
            c1 = mfma(x1, Q.q[1][t], c1);
            c0 = mfma(y0, Q.q[0][t], c0);
            c1 = mfma(y1, Q.q[0][t], c1);
            c0 = mfma(x0, Q.q[2][t], c0);
            c1 = mfma(x1, Q.q[2][t], c1);
            c0 = mfma(y0, Q.q[1][t], c0);
            c1 = mfma(y1, Q.q[1][t], c1);
            c0 = mfma(z0, Q.q[0][t], c0);
            c1 = mfma(z1, Q.q[0][t], c1);
        }
        e0 += finite(c0);
        e1 += finite(c1);
    }
    if (tail) {  // uniform
        const char* x = xs + G::kTailAt + (tp * kTileRows + 4 * jj) * (kTail * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const v4f a = *reinterpret_cast<const v4f*>(x + r * kTail * 4);
            const v4f b = *reinterpret_cast<const v4f*>(x + (kTileRows + r) * kTail * 4);
            e0[r] += ((a[0] * Q.qt[0] + a[1] * Q.qt[1]) + a[2] * Q.qt[2]) + a[3] * Q.qt[3];
            e1[r] += ((b[0] * Q.qt[0] + b[1] * Q.qt[1]) + b[2] * Q.qt[2]) + b[3] * Q.qt[3];
        }
    }
}

// All four 16-row tiles of one LDS stage for this wave's 16 positions, in
// pairs (32 rows: one K-step of the row contraction).
//
// `flip` reverses the pair order: the two waves that share a SIMD (loader
// index w and w + 4) take the pairs in opposite orders.  Each wave raises its
// issue priority while it feeds the matrix core and lowers it for the row
// terms, so that one wave of a SIMD feeds the matrix core while the other
// does its row terms.
template <int KT>
__device__ __forceinline__ void compute_stage(const char* xs, const WaveQ& Q, WaveAcc& acc, bool flip, int pair_lo,
                                              int pair_hi, bool tail)
{
    using G = Geo<KT>;
    const int l = lane();
    const int jj = l >> 4;
#pragma unroll 1
    for (int step = 0; step < kTiles; step += 2) {
        const int tp = flip ? kTiles - 2 - step : step;
        if (tp / 2 < pair_lo || tp / 2 >= pair_hi) continue;  // uniform: another group's rows
        v4f e0, e1;
        __builtin_amdgcn_s_setprio(2);
        columns<KT>(xs, Q, tp, tail, e0, e1);
        __builtin_amdgcn_s_setprio(0);
        const char* sg = xs + G::kSignAt + (tp * kTileRows + 4 * jj) * 4;
        const v4f s0 = *reinterpret_cast<const v4f*>(sg);
        const v4f s1 = *reinterpret_cast<const v4f*>(sg + kTileRows * 4);
        float res[8];
        float lsum = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float l0, l1;
            row_terms(e0[r], s0[r], l0, res[r]);
            row_terms(e1[r], s1[r], l1, res[4 + r]);
            lsum += l0 + l1;
        }
        acc.loss += (double)lsum;
        if constexpr (KT > 0) {
            v8bf R[kParts];
            split3<false>(res, R);
            // lane i of a 16-lane group reads columns 4 (i % 4) .. + 3 of row
            // 4 jj + i / 4 of a 16-column chunk
            const int i = l & 15;
            const int row = 4 * jj + (i >> 2);
            const char* base = xs + (tp * kTileRows + row) * G::kRow + (i & 1) * 8;
            const int at = (((i & 3) >> 1) ^ swizzle<KT>(row)) * 16;
            __builtin_amdgcn_s_setprio(2);
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const char* p = base + (at ^ (2 * mt * 16));
                v8bf x[kParts];
#pragma unroll
                for (int q = 0; q < kParts; ++q) {
                    const v4bf a = read_transposed(p + q * G::kPlane);
                    const v4bf b = read_transposed(p + q * G::kPlane + kTileRows * G::kRow);
                    x[q] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
                }
                // the corrections in a sum of their own: two roundings of the
                // running sum per 32 rows instead of six
                v4f c = {0.0f, 0.0f, 0.0f, 0.0f};
                c = mfma(x[0], R[1], c);
                acc.g[mt] = mfma(x[0], R[0], acc.g[mt]);
                c = mfma(x[1], R[0], c);
                c = mfma(x[0], R[2], c);
                c = mfma(x[1], R[1], c);
                c = mfma(x[2], R[0], c);
                acc.g[mt] += finite(c);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        if (tail) {
            const char* x = xs + G::kTailAt + (tp * kTileRows + 4 * jj) * (kTail * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const v4f a = *reinterpret_cast<const v4f*>(x + r * kTail * 4);
                const v4f b = *reinterpret_cast<const v4f*>(x + (kTileRows + r) * kTail * 4);
#pragma unroll
                for (int k = 0; k < kTail; ++k) acc.gt[k] += a[k] * res[r] + b[k] * res[4 + r];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Log-likelihood over draws: the column contraction E = X Q alone, then per
// (row, position) the loss and, with PRED, sigma(eta) summed over the
// positions of each row.

// loss = softplus(t) as in row_terms; p1 = sigmoid(eta) (the probability of
// y = 1): sigma(t) when y = 0 (t = eta), sigma(-t) when y = 1 (t = -eta).
__device__ __forceinline__ void ll_terms(float eta, float sgn, float& loss, float& p1)
{
    const float t = sgn * eta;
    const float e = __builtin_amdgcn_exp2f(-fabsf(t) * 1.4426950408889634f);
    const float u = 1.0f + e;
    const float inv = __builtin_amdgcn_rcpf(u);
    loss = __builtin_fmaf(kLn2f, __builtin_amdgcn_logf(u), fmaxf(t, 0.0f));
    const float sig_t = t >= 0.0f ? inv : e * inv;
    const float sig_mt = t >= 0.0f ? e * inv : inv;
    p1 = sgn > 0.0f ? sig_t : sig_mt;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    // every pattern used here reads a lane of the same row with all rows and
    // banks enabled
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// Sum over the 16 positions of a wave (lanes 16 g .. 16 g + 15, one DPP row,
// share the row group g): pair butterflies inside the row on DPP moves, so no
// LDS instruction (as cross-lane shuffles these were over half of the kernel's
// LDS instructions); every lane of the 16 gets the same bits.
__device__ __forceinline__ float sum16(float v)
{
    v += dpp_f32<kDppXor1>(v);
    v += dpp_f32<kDppXor2>(v);
    v += dpp_f32<kDppHalfMirror>(v);
    v += dpp_f32<kDppMirror>(v);
    return v;
}

// Posterior predictive samples of one position (draw s): y[i] = 1 iff
// u_si < sigmoid(eta_i), the uniforms the words of the Philox block keyed
// (seed, s) at counter (0, kTagPredict << 32, i / 4, 0), word i % 4.
struct PredictOut {
    uint8_t* y;     // the position's row of the [S][N] output, or null (dead position)
    uint64_t seed;
    uint64_t s;
    int64_t N;
    int64_t row0;   // first row of the stage
    bool words;     // every position's row starts at a multiple of four bytes
};

// Draw and store the samples of four consecutive rows r0 .. r0 + 3 (r0 a
// multiple of 4) from their probabilities p.  The block's number fits 32 bits
// (2^34 rows of stages are more than the device's memory) and its first
// word is zero, so the first two rounds need 6 of their 16 partial products
// (two more depend on the draw alone).  A sample is decided by the uniform's
// first 32 bits against floor(2^32 p) (2^32 p is exact in fp32) unless they
// are equal, one time in 2^32, where the 53 bits are compared in fp64 as the
// definition says.  The pass is bound by these rounds: 500 draws over
// 581,012 rows 1,036 us with all products and fp64 comparisons on the fp32
// matrix instruction, 791 on the bf16 one, 760 decided in 32 bits, 659 with
// two groups a CU.
__device__ __forceinline__ void predict_rows(const PredictOut& po, int64_t r0, const float (&p)[4])
{
    const Block4 b = philox4x64_10(0, kTagPredict << 32, (uint32_t)(r0 >> 2), 0, po.seed, po.s);
    const uint64_t w[4] = {b.w0, b.w1, b.w2, b.w3};
    uint32_t y[4];
    bool equal = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t hi = (uint32_t)(w[r] >> 32);
        // (p = 1 becomes 2^32 - 1; a NaN becomes 0 and is decided below)
        const float scaled = fmaxf(p[r], 0.0f) * 4294967296.0f;
        const uint32_t below = scaled >= 4294967296.0f ? 0xFFFFFFFFu : (uint32_t)scaled;
        y[r] = hi < below ? 1u : 0u;
        equal = equal || hi == below || !(p[r] >= 0.0f);
    }
    if (equal) {
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = unit53(w[r]) < (double)p[r] ? 1u : 0u;
    }
    if (po.words && r0 + 4 <= po.N) {
        *reinterpret_cast<uint32_t*>(po.y + r0) = y[0] | y[1] << 8 | y[2] << 16 | y[3] << 24;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r0 + r < po.N) po.y[r0 + r] = (uint8_t)y[r];
    }
}

// One LDS stage for this wave's 16 positions: the loss of every live
// (row, position) into `loss`; with PRED, the wave's sums of sigma(eta) over
// its live positions for each of the 64 rows into rs[0..63]; with SAMPLE,
// the position's predictive samples of the stage's rows.
template <int KT, bool PRED, bool SAMPLE>
__device__ __forceinline__ void compute_stage_ll(const char* xs, const WaveQ& Q, float live, double& loss, float* rs,
                                                 const PredictOut& po, bool tail)
{
    using G = Geo<KT>;
    const int l = lane();
    const int m = l & 15;
    const int jj = l >> 4;
#pragma unroll 1
    for (int tp = 0; tp < kTiles; tp += 2) {
        v4f e0, e1;
        columns<KT>(xs, Q, tp, tail, e0, e1);
        const char* sg = xs + G::kSignAt + (tp * kTileRows + 4 * jj) * 4;
        const v4f s0 = *reinterpret_cast<const v4f*>(sg);
        const v4f s1 = *reinterpret_cast<const v4f*>(sg + kTileRows * 4);
        float lsum = 0.0f;
        float p0[4], p1[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float l0, l1;
            ll_terms(e0[r], s0[r], l0, p0[r]);
            ll_terms(e1[r], s1[r], l1, p1[r]);
            lsum += l0 + l1;
        }
        if constexpr (!SAMPLE) loss += (double)lsum;
        if constexpr (SAMPLE) {
            if (po.y) {
                predict_rows(po, po.row0 + tp * kTileRows + 4 * jj, p0);
                predict_rows(po, po.row0 + (tp + 1) * kTileRows + 4 * jj, p1);
            }
        }
        if constexpr (PRED) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float a = sum16(live * p0[r]);
                const float b = sum16(live * p1[r]);
                if (m == 0) {
                    rs[tp * kTileRows + 4 * jj + r] = a;
                    rs[(tp + 1) * kTileRows + 4 * jj + r] = b;
                }
            }
        }
    }
}

// Stage loop of the log-likelihood: as stage_loop, and with PRED the eight
// waves' row sums of each stage (rs[buffer][wave][64]) are added in wave
// order and stored to prow[stage * 64 + row] one stage later, after the
// barrier that ends it.
template <int KT, bool PRED, bool SAMPLE>
__device__ __forceinline__ void stage_loop_ll(const BatchView& bv, int64_t st0, int64_t st1, int tid, char* xs,
                                              float* rs, const WaveQ& Q, float live, double& loss, float* prow,
                                              PredictOut po)
{
    const int widx = tid / kWave;
    auto flush = [&](int64_t st, int b) {
        if (PRED && tid < kBatchStageRows) {
            float s_ = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) s_ += rs[(b * kWaves + w) * kBatchStageRows + tid];
            prow[st * kBatchStageRows + tid] = s_;
        }
    };
    if (st0 < st1) load_stage<KT>(bv, st0, tid, xs);
    wait_stage();
    __syncthreads();
    for (int64_t st = st0; st < st1; ++st) {
        const int b = (int)((st - st0) & 1);
        if (st + 1 < st1) load_stage<KT>(bv, st + 1, tid, xs + (b ^ 1) * Geo<KT>::kBytes);
        if (st > st0) flush(st - 1, b ^ 1);
        po.row0 = st * kBatchStageRows;
        compute_stage_ll<KT, PRED, SAMPLE>(xs + b * Geo<KT>::kBytes, Q, live, loss,
                                           rs + (b * kWaves + widx) * kBatchStageRows, po, bv.tc > 0);
        wait_stage();
        __syncthreads();
    }
    if (st1 > st0) flush(st1 - 1, (int)((st1 - 1 - st0) & 1));
}

// A group's rows in halves of stages (pairs of 16-row tiles, 32 rows):
// the 2 ns halves split evenly over the groups, so that no group has more
// than one half more than another (whole stages left 53 of 128 groups a
// whole stage more).  A stage whose halves two groups share is loaded by
// both, each computing its own.
__host__ __device__ inline void group_halves(int64_t ns, int64_t i, int64_t groups, int64_t* h0, int64_t* h1)
{
    *h0 = i * 2 * ns / groups;
    *h1 = (i + 1) * 2 * ns / groups;
}

// The stage loop over the halves [h0, h1) (stages h0 / 2 .. (h1 - 1) / 2)
// with double-buffered LDS stages.  Workers (tid = loader index, 0 .. 511)
// load and compute; a non-worker wave of the same group passes the same
// workgroup barriers (one more than the stages) and does nothing else.
template <int KT, bool WORKER>
__device__ __forceinline__ void stage_loop(const BatchView& bv, int64_t h0, int64_t h1, int tid, char* xs,
                                           const WaveQ& Q, WaveAcc& acc)
{
    const int64_t st0 = h0 / 2;
    const int64_t st1 = h1 > h0 ? (h1 + 1) / 2 : st0;
    if constexpr (!WORKER) {
        for (int64_t st = st0; st <= st1; ++st) __syncthreads();
    } else {
        if (st0 < st1) load_stage<KT>(bv, st0, tid, xs);
        wait_stage();
        __syncthreads();
        for (int64_t st = st0; st < st1; ++st) {
            const int b = (int)((st - st0) & 1);
            if (st + 1 < st1) load_stage<KT>(bv, st + 1, tid, xs + (b ^ 1) * Geo<KT>::kBytes);
            // the halves of this stage that are the group's
            const int lo = (int)(h0 > 2 * st ? h0 - 2 * st : 0);
            const int hi = (int)(h1 < 2 * st + 2 ? h1 - 2 * st : 2);
            compute_stage<KT>(xs + b * Geo<KT>::kBytes, Q, acc, tid >= 4 * kWave, lo, hi, bv.tc > 0);
            wait_stage();
            __syncthreads();
        }
    }
}

// Sum the tail and loss accumulators over the four lanes of a position
// (lanes m, m + 16, m + 32, m + 48); every one of them gets the same bits.
__device__ __forceinline__ void reduce_position(WaveAcc& acc)
{
#pragma unroll
    for (int k = 0; k < kTail; ++k) {
        acc.gt[k] += __shfl_xor(acc.gt[k], 16);
        acc.gt[k] += __shfl_xor(acc.gt[k], 32);
    }
    acc.loss += __shfl_xor(acc.loss, 16);
    acc.loss += __shfl_xor(acc.loss, 32);
}

}  // namespace batch
}  // namespace nuts
