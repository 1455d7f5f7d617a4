// Streaming scoring kernel for bf16, fp16 or 8-bit (E4M3) keys of head dim <= 128 (64 excepted, see
// tile_score_supported), window 64, episodic block size <= 256 (paper Sections 2.1-2.3), with every dot product of the
// pass formed by the matrix cores.  (Written out below for bf16 and head dim 128; fp16 differs in the product
// instruction, in unpacking, and in how an fp32 anchor is cut into three terms; 8-bit keys become bf16, exactly, on
// their way from the load; other head dims are padded with zeros to 32 KS, which no dot product and no norm sees.)
//
// The pass is a stream over the keys and nothing else is read from memory, but written for the vector unit it
// needs ~2300 instructions per 64 tokens and is bound by their issue.  Here everything that is a contraction over the head
// dimension goes through v_mfma_f32_16x16x32_bf16, whose products of bf16 values are exact and whose sums are fp32, and what
// is done per token is done for 64 tokens at a time, one per lane:
//
//   * a block is cut into groups of 16 tokens.  T_q = sum of k_hat over group q.  The window sum in
//     front of group q's first token is exact in terms of groups: Seed_q = T_{q-4} + ... + T_{q-1}.
//   * for token i of group G, with P the group 64 tokens earlier (token i' = i - 64 leaves as i enters),
//         W_i = Seed_G + sum_{j in G, j <= i} k_hat_j - sum_{j' in P, j' <= i'} k_hat_j',
//     so <k_i, W_i> = <k_i, Seed_G> + sum_{j <= i} w_j A[i][j] - sum_{j' <= i'} w_j' X[i][j'] with the Gram tiles
//     A = K_G K_G^T and X = K_G K_P^T of the raw keys and w = 1 / ||k||, ||k||^2 being A's diagonal.
//   * ||W_i||^2 follows the window inside the group: it is ||Seed_G||^2 plus the running sum of
//         ||W_i||^2 - ||W_{i-1}||^2 = 2 <W_i, d_i> - ||d_i||^2,   d_i = k_hat_i - k_hat_i',
//     which needs <k_i', W_i> (same tiles, the other triangle) and X[i][i'].  At most 16 terms are added up.
//   * <k, anchor> for the anchors that are vectors (Seed_G, the block total, the unit sum): the fp32 anchor is
//     split into three bf16 terms (8 + 8 + 8 mantissa bits, exact) that form rows of the left operand.  One left operand
//     holds the seeds of a wave's four groups and the block total.
//   * T_q: a product with a selector matrix takes 16 dims out of a group as fp32 (exact), four tokens a lane, which the vector
//     unit weights and adds up.
//
// Layouts.  A wave owns the groups q = w, w + 4, w + 8, w + 12 of the block (so the group 64 tokens earlier is
// its own previous group) and the group of the halo in front of them.  A group is loaded row by row (64 pieces of 16 bytes
// an instruction, whatever the row's length) and passes through rows of LDS private to the wave to become a matrix operand
// (lane (q, n): token n, dims 32 kk + 8q .. + 7 in operand register kk).  Operands stay in registers until the unit's
// sum has arrived.  A 16 x 16 result leaves lane (q, n) with column n, rows 4q .. 4q+3: sums over rows are four
// multiply-adds per lane, and the four groups' partial sums then change places across the lanes so that lane (q, n) ends up
// with group q's token n: one square root, one store an anomaly and so on for 64 tokens.  In calls whose blocks have at most
// 128 tokens no wave has more than two groups: an instance of its own (MG = 2; 94 registers at head dim 128, five workgroups a
// CU, or 98 and four where FINE).
//
// What bounds it.  36 layers x 8 heads x 32768 tokens of head dim 128: 531 us (552 with the tokens' arithmetic group by
// group, dot-product instructions for the norms and unpacking on the vector unit: 1484 vector instructions per 64 tokens,
// 942 now, 148 of them matrix products), keys at 4.6 TB/s, where reading them alone takes 350 us.  No unit is saturated: of a
// workgroup's 27 500 cycles 5 500 pass until its first group is staged, 14 600 in dependent phases that share the vector unit with
// three other workgroups (norms and group sums 5 600, block total and halo group 4 300, anchors and windows 4 800), 1 300 in the
// stable products, and 6 100 in waiting for the slowest of the unit's 128 workgroups.  What was measured instead and is slower:
// workgroups that stay and bring the next block's keys to LDS meanwhile, with a_s one block later, two of four waves (612 us) or of eight
// (790 us) a CU: half the waves, or half the tokens a wave, hide less of the chains than the loads and waits cost.
//
// Protocol.  A block's workgroup adds its total to the unit's self-counting accumulators (nkv_scan_common.h) as
// soon as it has it; the add returns the word's previous contents, and whoever finds that it was the last of the
// unit's blocks to add to a word stores the word's final value, as fp32, into the unit's sum -- memory that
// starts out "unwritten" and in which every word is stored exactly once.  After its window phase a workgroup looks
// at the unit's sum: if it is complete it forms a_s from the operands still in its registers; if not after a
// bounded number of looks, it puts its block on a list and leaves, and deferred_stable_tile_kernel computes a_s
// of the listed blocks after the pass, when every sum is complete.  No workgroup ever waits for anything but
// stores that workgroups already running (or finished) issue unconditionally, and every wait is bounded.
// (Looking at the accumulators themselves instead of a copy stored once was tried: loads of words that other
// workgroups are adding to cost the pass a quarter of its time under sustained load.)
#include "nkv_scan_common.h"

#include <type_traits>

namespace nkv {
namespace {

using bf16x2 = __bf16 __attribute__((ext_vector_type(2)));
using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));
using f16x8 = _Float16 __attribute__((ext_vector_type(8)));
using f32x4 = float __attribute__((ext_vector_type(4)));

// An offset past any buffer of the pass (which are shorter than kNoByte - 512 rows): loads read zeros there, stores are dropped.
// It stays past them with the offset of a token, or of up to 64 tokens in front of the prompt, added, and with itself added (a
// row's missing piece in a group that the block does not have); offsets are unsigned, so that these sums are defined.
constexpr uint32_t kNoByte = 0x40000000u;
static_assert(kNoByte + kNoByte > kNoByte, "the sum of two stays past every buffer (and is a constant: no signed overflow)");
constexpr int kGroup = 16;                       // tokens per group
constexpr int kTileWaves = 4;


// KF: the keys' 16-bit format (kKeyBF16 or kKeyF16), which is also the format the anchors' terms are staged in
template <int KF> __device__ __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, f32x4 c)
{
    if constexpr (KF == kKeyF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// D[m][n] = sum over the head dimension of a's row m and b's row n
template <int KF, int KS> __device__ __forceinline__ f32x4 tile(const u32x4 (&a)[KS], const u32x4 (&b)[KS])
{
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) c = mma<KF>(a[kk], b[kk], c);
    return c;
}

// The same, as two halves where FINE: shorter chains of additions.
template <int KF, int KS, bool FINE> __device__ __forceinline__ f32x4 fine_tile(const u32x4 (&a)[KS], const u32x4 (&b)[KS])
{
    if constexpr (!FINE) {
        return tile<KF, KS>(a, b);
    } else {
        constexpr int HALF = (KS + 1) / 2;
        f32x4 c = {0.f, 0.f, 0.f, 0.f}, e = c;
#pragma unroll
        for (int kk = 0; kk < HALF; ++kk) c = mma<KF>(a[kk], b[kk], c);
#pragma unroll
        for (int kk = HALF; kk < KS; ++kk) e = mma<KF>(a[kk], b[kk], e);
        return c + e;
    }
}

// x summed over the four lanes n, n + 16, n + 32, n + 48; every lane receives the total.
// permlane32_swap(x, x) = (x of the lower half in both halves, x of the upper half in both halves); the 16-lane
// swap does the same with even and odd rows of 16 lanes.
__device__ __forceinline__ float sum_over_rows16(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const uint32_t v = __float_as_uint(s);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Inclusive running sum over the 16 lanes of a row (lanes n = 0 .. 15 of every group of 16), in 64 and in 32 bits.
template <int CTRL> __device__ __forceinline__ double row_shr(double x)       // 0 in front of the row
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double row_prefix_sum(double x)
{
    x += row_shr<0x111>(x);
    x += row_shr<0x112>(x);
    x += row_shr<0x114>(x);
    x += row_shr<0x118>(x);
    return x;
}

__device__ __forceinline__ float row_prefix_sum(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, true));   // row_shr:1
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, true));   // row_shr:2
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, true));   // row_shr:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, true));   // row_shr:8
    return x;
}

// A pair of fp32 values -> three 16-bit terms each, whose sum is the value.  bf16: each term takes the next 8 mantissa bits,
// exact.  fp16: each term is the rounded remainder (11 bits each; the remainders are exact, the last term is off by at most
// 2^-33 of the value or by fp16's smallest step, 6e-8, whichever is larger); the value must be below fp16's largest, 65504.
template <int KF> __device__ __forceinline__ void split3_pair(float x, float y, uint32_t (&t)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if constexpr (KF == kKeyF16) {
            const _Float16 a = (_Float16)x, b = (_Float16)y;
            t[i] = (uint32_t)__builtin_bit_cast(unsigned short, a) | (uint32_t)__builtin_bit_cast(unsigned short, b) << 16;
            x -= (float)a;
            y -= (float)b;
        } else {
            const uint32_t a = __float_as_uint(x), b = __float_as_uint(y);
            t[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);          // the upper halves
            x -= __uint_as_float(a & 0xffff0000u);
            y -= __uint_as_float(b & 0xffff0000u);
        }
    }
}

// The factor that keeps a sum of N unit vectors inside fp16's range; the cosine does not see it.
__device__ __forceinline__ float fp16_sum_scale(int N) { return N <= 131072 ? 0.25f : 0.03125f; }

// Rows of 32 KS 16-bit values in LDS (staged keys, anchors): 16 lanes that read the same piece of 16 rows touch every bank once.
template <int KS> constexpr int kPitch = 64 * KS + 16;

// A vector of which this lane holds dims 2 lane and 2 lane + 1 as its three terms, the largest first, into rows r0, r1, r2.
template <int KF, int KS> __device__ __forceinline__ void stage_anchor(uint8_t *rows, int r0, int r1, int r2, int lane, float v0, float v1)
{
    uint32_t t[3];
    split3_pair<KF>(v0, v1, t);
    if (KS < 4 && lane >= 16 * KS) return;
    *reinterpret_cast<uint32_t *>(rows + r0 * kPitch<KS> + 4 * lane) = t[0];
    *reinterpret_cast<uint32_t *>(rows + r1 * kPitch<KS> + 4 * lane) = t[1];
    *reinterpret_cast<uint32_t *>(rows + r2 * kPitch<KS> + 4 * lane) = t[2];
}

// Staged rows as a matrix operand: lane (q, n) takes dims 32 kk + 8 q .. + 7 of row r.
template <int KS> __device__ __forceinline__ void read_operand(const uint8_t *rows, int r, int q, u32x4 (&x)[KS])
{
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) x[kk] = *reinterpret_cast<const u32x4 *>(rows + r * kPitch<KS> + 16 * q + 64 * kk);
}

// The format the operands are in: 8-bit keys travel as bf16.
template <int KF> constexpr int kStaged = KF == kKeyF16 ? kKeyF16 : kKeyBF16;

// Eight values of a row in the operand format.  E4M3 -> bf16 is exact (3 mantissa bits into 7, exponents -9 .. 8).
template <int KF> __device__ __forceinline__ u32x4 operand_piece(const Piece<KF> &r)
{
    if constexpr (KF == kKeyF8) {
        return u32x4{__builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r.x, 1.0f, false)),
                     __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r.x, 1.0f, true)),
                     __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r.y, 1.0f, false)),
                     __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r.y, 1.0f, true))};
    } else {
        return r;
    }
}

// The diagonal of a 16 x 16 result: lane (n / 4, n) receives element [n][n], the others 0.
__device__ __forceinline__ float diagonal(const f32x4 &x, int qq, int n)
{
    const float a = (n & 1) ? x[1] : x[0], b = (n & 1) ? x[3] : x[2];
    return (n >> 2) == qq ? ((n & 2) ? b : a) : 0.f;
}
// v[m], m < 4: partial sums of group m's token n held by lane (q, n).  Lane (q, n) receives the total of group q's.
__device__ __forceinline__ float sum_to_groups(const float (&v)[4])
{
    float u[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[e]), __float_as_uint(v[e + 2]), false, false);
        u[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u[0]), __float_as_uint(u[1]), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double sum_to_groups(const double (&v)[4])
{
    auto merge = [](double x, double y, bool rows32) {
        const unsigned long long a = __builtin_bit_cast(unsigned long long, x), b = __builtin_bit_cast(unsigned long long, y);
        const auto lo = rows32 ? __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false) : __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
        const auto hi = rows32 ? __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false)
                               : __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
        return __builtin_bit_cast(double, (unsigned long long)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (unsigned long long)hi[1] << 32 | lo[1]);
    };
    return merge(merge(v[0], v[2], true), merge(v[1], v[3], true), false);
}
// the total over a row's 16 lanes
__device__ __forceinline__ double row_total(double v)
{
    v += dpp_partner<0xB1>(v);
    v += dpp_partner<0x4E>(v);
    v += dpp_partner<0x141>(v);
    return v + dpp_partner<0x140>(v);
}
__device__ __forceinline__ float row_total(float v) { return row_sum<16>(v); }
// v[q] without an index that is not known at compile time
__device__ __forceinline__ float of_group(const float (&v)[4], int q)
{
    const float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
    const float a = (q & 1) ? v1 : v0, b = (q & 1) ? v3 : v2;
    return (q & 2) ? b : a;
}

// ||k_hat|| of a token, 1 unless its norm is below the clamp (rare: one uniform test instead of a square root per token)
__device__ __forceinline__ float unit_norm(float ss)
{
    float k = 1.f;
    if (__any(ss < 1e-24f)) k = ss < 1e-24f ? sqrtf(ss) * 1e12f : 1.f;
    return k;
}

// 1 / sqrt(x), once more corrected: half a step of fp32 where the hardware's is good to one.
__device__ __forceinline__ float fine_rsqrt(float x)
{
    const float y = __builtin_amdgcn_rsqf(x), e = fmaf(-(x * y), y, 1.0f);
    return fmaf(0.5f * e, y, y);
}

// -cos of a token's key to an anchor from <k, anchor>, the token's 1 / ||k|| and ||k||^2, and ||anchor||^2.
// FINE: with the corrected reciprocal square roots.
template <bool FINE> __device__ __forceinline__ float token_cos(float dot, float w, float ss, float anchor_sq)
{
    if constexpr (FINE) {
        float k = 1.f;
        if (__any(ss < 1e-24f)) k = ss < 1e-24f ? 1.0f / fmaxf(sqrtf(ss) * 1e12f, kEps) : 1.f;
        const float fw = w > 0.f && ss >= 1e-24f ? fine_rsqrt(ss) : w;
        return -(fw * dot) * k * fine_rsqrt(fmaxf(anchor_sq, kEps * kEps));
    } else {
        return neg_cos(w * dot, unit_norm(ss), anchor_sq);
    }
}

// Dims 2 lane and 2 lane + 1 of a vector of 32 KS floats (0 past its end).
template <int KS> __device__ __forceinline__ float2 dim_pair(const float *v, int lane)
{
    if (KS == 4) return *reinterpret_cast<const float2 *>(v + 2 * lane);
    const float2 t = *reinterpret_cast<const float2 *>(v + 2 * min(lane, 16 * KS - 1));
    return lane < 16 * KS ? t : make_float2(0.f, 0.f);
}

// The same of a unit's sum, which lies in the order of its accumulators: first the even dims, then the odd ones, so that
// the 64 lanes of an atomic instruction add to consecutive words.
template <int KS> __device__ __forceinline__ float2 sum_pair(const float *v, int lane)
{
    const int at = KS == 4 ? lane : min(lane, 16 * KS - 1);
    const float2 t = make_float2(v[at], v[16 * KS + at]);
    return KS == 4 || lane < 16 * KS ? t : make_float2(0.f, 0.f);
}

__device__ __forceinline__ float sum3(const f32x4 &d) { return d[0] + (d[1] + d[2]); }

// sum over this lane's four rows of wm[rho] * d[rho]
__device__ __forceinline__ float weighted(const f32x4 &d, const float (&wm)[4])
{
    return fmaf(wm[3], d[3], fmaf(wm[2], d[2], fmaf(wm[1], d[1], wm[0] * d[0])));
}

// The blocks of a long unit add their totals up in two steps: 32 consecutive blocks into accumulators of their own, and
// whoever completes a word of a group adds it to the unit's word.  Adds to one word take turns at the memory side, and
// hundreds of blocks queueing for the same words hold up everything behind them.  Up to 192 blocks (49 152 tokens) the
// unit is one group, whose words are the unit's: the second step costs more than the queue (8 heads, score call, one
// step against two: 16 layers of 160 blocks 401 / 411 us, 16 layers of 256 blocks 688 / 640 us, 8 layers of 512 blocks
// 812 / 700 us).
constexpr int kOneGroup = 192, kGroupBlocks = 32;
__host__ __device__ __forceinline__ int blocks_per_group(int unit_blocks) { return unit_blocks > kOneGroup ? kGroupBlocks : kOneGroup; }
__host__ __device__ __forceinline__ int unit_groups(int unit_blocks) { const int per = blocks_per_group(unit_blocks); return (unit_blocks + per - 1) / per; }
// first group slot of a prompt with `blocks` blocks and `prompts` prompts in front of it: every prompt rounds up by itself
__host__ __device__ __forceinline__ int group_slots(int blocks, int prompts) { return blocks / kGroupBlocks + prompts; }

// One item of the pass: a block of one (layer, head, prompt) unit with everything a workgroup needs to know about
// it, worked out once by plan_kernel so that the pass itself starts an item with one scalar load instead of a
// chain of dependent ones (kernel arguments, per-prompt tables, divisions).
struct TileItem {
    int64_t key_off;                     // element offset of the unit's first row
    int64_t row0;                        // the unit's first row in the planes of a_raw
    int32_t N;                           // tokens of the unit; < 0: this slot of the die's queue is empty
    int32_t blk_lo, blk_hi;              // the block's tokens, unit-local
    int32_t unit;                        // index of the unit's accumulators and sum
    int32_t id;                          // (layer, head) * blocks per head + block: what the deferred list holds
    int32_t group;                       // index of the accumulators of the block's group
    int32_t group_blocks, unit_groups;   // blocks of that group, groups of the unit
};
static_assert(sizeof(TileItem) == 48, "items are read as three 16-byte pieces");

// Items in launch order: item i belongs to die i % 8 and is entry i / 8 of that die's queue (the queues of
// scan_kernel in nkv_score_fast.hip without the items that add a unit up: for every (layer, head) in turn the
// die's runs of consecutive blocks).  Also clears the counters and the accumulators and marks the units' sums unwritten.
__global__ __launch_bounds__(256) void plan_kernel(TileItem *__restrict__ items, uint32_t n_items, RowMap km, PromptTab tab,
                                                   ScanPlan plan, int LH, uint4 *sync, size_t n_sync, uint4 *accum, size_t n_accum,
                                                   uint4 *sums, size_t n_sums)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u), none = make_uint4(kUnwritten, kUnwritten, kUnwritten, kUnwritten);
    for (size_t k = i; k < n_sync + n_accum + n_sums; k += (size_t)gridDim.x * blockDim.x) {
        if (k < n_sync) sync[k] = zero;
        else if (k < n_sync + n_accum) accum[k - n_sync] = zero;
        else sums[k - n_sync - n_accum] = none;
    }
    for (size_t k = i; k < n_items; k += (size_t)gridDim.x * blockDim.x) {
        const int x = (int)(k & (kDies - 1));
        const uint32_t t = (uint32_t)(k >> 3);
        const int len = plan.len[x];
        TileItem it;
        const int lh = len > 0 ? (int)(t / (uint32_t)len) : LH;
        if (lh >= LH) {
            it.key_off = it.row0 = 0;
            it.N = -1;
            it.blk_lo = it.blk_hi = it.unit = it.id = it.group = it.group_blocks = it.unit_groups = 0;
        } else {
            const int r = (int)(t - (uint32_t)lh * (uint32_t)len);
            const int blk = die_block(plan.run, x, r);
            const int p = prompt_of_block(tab, blk);
            const int b = tab.b[p];
            it.N = tab.tok_off[p + 1] - tab.tok_off[p];
            it.blk_lo = (blk - tab.blk_off[p]) * b;
            it.blk_hi = min(it.blk_lo + b, it.N);
            it.key_off = km.unit(lh, p, tab);
            it.row0 = (int64_t)lh * tab.T + tab.tok_off[p];
            it.unit = lh * tab.n + p;
            it.id = lh * plan.nblk + blk;
            const int unblk = tab.blk_off[p + 1] - tab.blk_off[p], local = blk - tab.blk_off[p];
            const int per = blocks_per_group(unblk), gi = local / per;
            it.group = lh * group_slots(plan.nblk, tab.n) + group_slots(tab.blk_off[p], p) + gi;
            it.group_blocks = min(per, unblk - gi * per);
            it.unit_groups = unit_groups(unblk);
        }
        items[k] = it;
    }
}

// MG: groups a wave has at most (2: no block of the call has more than 128 tokens).
// grid: one workgroup of 256 threads per item, in the items' order.  (Resident workgroups that loop over the items
// instead were tried: without the hardware handing out blocks as slots fall free, all workgroups of the chip move
// through their loading and computing phases in step, and the pass takes 0.90 ms instead of 0.77.)
// KS: head dims the pass works with, in steps of 32 (the rest of the last step reads as zeros); FULL: d = 32 KS.
template <int KF, int KS, bool FULL, bool FINE, int MG> __global__ __launch_bounds__(64 * kTileWaves, 4)
void scan_tile_kernel(const uint8_t *__restrict__ keys, int d, const TileItem *__restrict__ items, float *__restrict__ a_raw,
                      unsigned long long *__restrict__ acc, unsigned long long *__restrict__ acc_group, float *__restrict__ ssum, uint32_t *__restrict__ sync, int64_t rows,
                      int poll_limit)
{
    constexpr int D = 32 * KS, NW = kTileWaves, ES = key_bytes<KF>(), SF = kStaged<KF>;
    constexpr int kPieces = D * ES / 16, kLoads = (kGroup * kPieces + 63) / 64;   // 16-byte pieces of a row; load instructions of a group
    const int row_bytes = FULL ? D * ES : d * ES;
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[NW][kGroup * kPitch<KS>];   // a wave's group on its way to operand layout, later its anchors
    __shared__ __attribute__((aligned(16))) float lds_T[4 + 4 * MG][D];               // group sums: 4 halo groups, then the block's
    __shared__ __attribute__((aligned(16))) float lds_w[NW][5][kGroup];           // 1/||k|| per token of a wave's groups (0: no such token)
    __shared__ __attribute__((aligned(16))) float lds_ss[NW][5][kGroup];          // ||k||^2
    __shared__ __attribute__((aligned(16))) float lds_S[D];                       // the unit's sum, once complete
    __shared__ __attribute__((aligned(16))) float lds_B[D];                       // the block's sum
    __shared__ int s_have;

    const TileItem it = items[blockIdx.x];
    if (it.N < 0) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int qq = lane >> 4, n = lane & 15;                          // operand / result layout: token n, quarter qq
    uint8_t *stage = lds_stage[w];

    const int N = it.N, blk_lo = it.blk_lo, blk_hi = it.blk_hi;
    const int ng = (blk_hi - blk_lo + kGroup - 1) / kGroup;           // groups of the block, <= 16
    const int64_t row0 = it.row0;                                     // row of the prompt's token 0

    // ---- first touch: this wave's groups, then its group of the halo.  Rows outside the prompt read as zeros, and so do
    // groups that the block does not have. ----
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(keys) + it.key_off * ES, 0, N * row_bytes, 0x00020000);
    uint32_t load_off[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int piece = 64 * i + lane, at = piece % kPieces * 16;
        load_off[i] = (FULL || at < row_bytes) && piece < kGroup * kPieces ? piece / kPieces * row_bytes + at : kNoByte;
    }
    u32x4 raw[MG + 1][kLoads];
#pragma unroll
    for (int mm = 0; mm <= MG; ++mm) {
        const int m = (mm + 1) % (MG + 1);                                   // the halo is needed last
        const int q = w + 4 * (m - 1);                                // block-local group index, < 0: halo
        const uint32_t base = q < ng ? (uint32_t)((blk_lo + kGroup * q) * row_bytes) : kNoByte;
#pragma unroll
        // a full block's last 64 tokens (m = 4) are read again, as the next block's halo, and the halo has just been read by
        // the block in front: those stay in the L2; the other rows are marked non-temporal (aux 2)
        for (int i = 0; i < kLoads; ++i)
            raw[m][i] = (m >= 1 && m < MG) ? __builtin_amdgcn_raw_buffer_load_b128(rsrc, base + load_off[i], 0, 2)
                                           : __builtin_amdgcn_raw_buffer_load_b128(rsrc, base + load_off[i], 0, 0);
    }

    // A group through the staging rows into operand layout; the diagonal of its Gram tile are the norms (partial sums: lane
    // (n / 4, n) holds token n's).
    u32x4 X[MG + 1][KS];
    auto stage_group = [&](const u32x4 (&r)[kLoads], u32x4 (&x)[KS]) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int piece = 64 * i + lane, row = piece / kPieces, at = piece % kPieces;
            if (kGroup * kPieces % 64 == 0 || piece < kGroup * kPieces) {
                if constexpr (KF == kKeyF8) {
                    u32x4 *to = reinterpret_cast<u32x4 *>(stage + row * kPitch<KS> + 32 * at);
                    to[0] = operand_piece<KF>(u32x2{r[i][0], r[i][1]});
                    to[1] = operand_piece<KF>(u32x2{r[i][2], r[i][3]});
                } else {
                    *reinterpret_cast<u32x4 *>(stage + row * kPitch<KS> + 16 * at) = r[i];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        read_operand<KS>(stage, n, qq, x);
        __builtin_amdgcn_wave_barrier();                              // the next group reuses the staging rows
        float p = diagonal(fine_tile<SF, KS, true>(x, x), qq, n);
        asm volatile("" : "+v"(p));                                   // (here: one register instead of four)
        __builtin_amdgcn_sched_barrier(0);                            // one group at a time
        return p;
    };
    // A group's sum: a product with a selector takes dims 32 kk + 16 u .. + 15 out of the group as fp32, lane (qq, n): dim n of
    // those, rows 4 qq .. + 3.
    auto selector = [&](int u) {
        u32x4 pick;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            pick[i] = qq == 2 * u + (n >> 3) && (n & 7) >> 1 == i ? (SF == kKeyF16 ? 0x3c00u : 0x3f80u) << (16 * (n & 1)) : 0u;
        return pick;
    };
    auto group_sum = [&](const u32x4 (&x)[KS], const u32x4 &pick, int u, const float *weights, float *to) {
        const float4 f4 = *reinterpret_cast<const float4 *>(weights + 4 * qq);
        const float w4[4] = {f4.x, f4.y, f4.z, f4.w};
        float T[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            T[kk] = weighted(mma<SF>(x[kk], pick, z), w4);
        }
        const float t = sum_to_groups(T);                             // dim 32 qq + 16 u + n
        if (KS == 4 || qq < KS) to[32 * qq + 16 * u + n] = t;
        __builtin_amdgcn_sched_barrier(0);                            // one group at a time
    };

    // ---- the block's own groups: norms and sums, nothing else in front of the block total ----
    auto token = [&] {                                                // lane (q, n): group q's token n (not kept: registers)
        int at = 64 * qq + n;
        asm volatile("" : "+v"(at));
        return blk_lo + kGroup * w + at;
    };
    {
        float own[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < MG; ++m) own[m] = stage_group(raw[m + 1], X[m + 1]);
        const float ss = sum_to_groups(own);
        lds_w[w][1 + qq][n] = token() < blk_hi ? inv_norm(ss) : 0.f;
        lds_ss[w][1 + qq][n] = ss;
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const u32x4 pick = selector(u);
#pragma unroll
        for (int m = 1; m <= MG; ++m) group_sum(X[m], pick, u, lds_w[w][m], lds_T[w + 4 * m]);
    }
    __syncthreads();

    auto sum_of_four = [&](int r) {                                   // groups r .. r + 3 of lds_T
        const float2 t0 = dim_pair<KS>(lds_T[r], lane), t1 = dim_pair<KS>(lds_T[r + 1], lane), t2 = dim_pair<KS>(lds_T[r + 2], lane), t3 = dim_pair<KS>(lds_T[r + 3], lane);
        return make_float2(((t0.x + t1.x) + t2.x) + t3.x, ((t0.y + t1.y) + t2.y) + t3.y);
    };
    // ---- block total = episodic anchor (up to length); lane: dims 2 lane, 2 lane + 1.  One wave adds the groups up in order, posts
    // the total to the unit's sum and leaves it to the others in LDS.  The order is the same whichever wave that is and for both
    // MG (groups that the block does not have are zeros), so a unit's scores depend neither on where it lies in the call nor on
    // its neighbours' blocks.  (Every wave for itself, starting with its own seeds, gave each wave its own rounding and took
    // longer: 36 layers x 8 heads x 32768 tokens 627 us and 622 this way, 32 heads x ragged x head dim 96 113 and 110.)
    // In 64 bits, because groups may cancel: rms error of a_e for keys whose common direction, 60 times the spread, changes
    // sign every 64 tokens, 3.4e-7 added up in 32 bits and 2.5e-7 so (head dim 128; other keys 2.4e-8 both), for 0.5 % of the scan. ----
    unsigned long long *acc_mine = acc_group + (int64_t)it.group * D;
    const bool poster = w == (it.id & (NW - 1));
    unsigned long long after0 = 0ull, after1 = 0ull;                  // the accumulators right after this block's add
    if (poster) {
        double tx = 0., ty = 0.;
#pragma unroll
        for (int q = 0; q < 4 * MG; ++q) {
            const float2 c = dim_pair<KS>(lds_T[4 + q], lane);
            tx += (double)c.x;
            ty += (double)c.y;
        }
        const float2 total = make_float2((float)tx, (float)ty);
        if (KS == 4 || lane < D / 2) {
            const unsigned long long t0 = accum_term(total.x), t1 = accum_term(total.y);
            after0 = __hip_atomic_fetch_add(acc_mine + lane, t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t0;
            after1 = __hip_atomic_fetch_add(acc_mine + D / 2 + lane, t1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t1;
            *reinterpret_cast<float2 *>(&lds_B[2 * lane]) = total;
        }
    }
    // ---- the halo group (the window sums in front of the block's first groups need its sum) ----
    {
        const float ss_h = sum_over_rows16(stage_group(raw[0], X[0]));
        if (qq == 0) {
            lds_w[w][0][n] = blk_lo + kGroup * (w - 4) + n >= 0 ? inv_norm(ss_h) : 0.f;
            lds_ss[w][0][n] = ss_h;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 2; ++u) group_sum(X[0], selector(u), u, lds_w[w][0], lds_T[w]);
    }
    __syncthreads();
    // ---- one left operand: rows 4 m .. + 2 the terms of group m's seed, the window sum in front of it = the four groups before,
    // rows 7, 3, 11 those of the block total ----
    using Norm = std::conditional_t<FINE, double, float>;
    Norm sq[4] = {};
#pragma unroll
    for (int m = 0; m < MG; ++m) {
        const float2 seed = sum_of_four(w + 4 * m);
        const Norm x = seed.x, y = seed.y;
        sq[m] = x * x + y * y;
        stage_anchor<SF, KS>(stage, 4 * m, 4 * m + 1, 4 * m + 2, lane, seed.x, seed.y);
    }
    {
        const float2 total = dim_pair<KS>(lds_B, lane);
        stage_anchor<SF, KS>(stage, 7, 3, 11, lane, total.x, total.y);  // (the small terms' products are added up first)
    }
    Norm P0 = row_total(sum_to_groups(sq));                           // ||W||^2 in front of this lane's group
    asm volatile("" : "+v"(P0));
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // <k, anchor>: lanes of group q hold the seed's of their group's tokens, and of the tokens 64 in front
    float c_seed, e_seed, bd;
    {
        u32x4 An[KS];
        read_operand<KS>(stage, n, qq, An);                           // (row 15 holds a key's row: not used)
        __builtin_amdgcn_wave_barrier();
        float dot[5] = {}, b_part[4] = {};
        dot[0] = sum3(fine_tile<SF, KS, FINE>(An, X[0]));
#pragma unroll
        for (int m = 0; m < MG; ++m) {
            const f32x4 AG = fine_tile<SF, KS, FINE>(An, X[m + 1]);   // [anchor row][i in G]
            dot[m + 1] = sum3(AG);
            b_part[m] = qq < 3 ? AG[3] : 0.f;
            __builtin_amdgcn_sched_barrier(0);
        }
        const float e4[4] = {dot[0], dot[1], dot[2], dot[3]}, c4[4] = {dot[1], dot[2], dot[3], dot[4]};
        c_seed = of_group(c4, qq);
        e_seed = of_group(e4, qq);
        bd = sum_to_groups(b_part);
        asm volatile("" : "+v"(c_seed), "+v"(e_seed), "+v"(bd));
    }
    __builtin_amdgcn_sched_barrier(0);

    float *S_unit = ssum + (int64_t)it.unit * D;
    // (The adds have had the anchors' products to come back.)  The last block to add to a word of the unit stores the word's final
    // value, the last block of a group adds its word's to the unit's word: a word's adds take turns, so exactly one does.
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(S_unit, 0, D * 4, 0x00020000);
    auto store_complete = [&](int adds) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(accum_value(after0)), prs,
                                              accum_complete(after0, adds) ? 4 * lane : kNoByte, 0, 16);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(accum_value(after1)), prs,
                                              accum_complete(after1, adds) ? 4 * lane + D * 2 : kNoByte, 0, 16);
    };
    const bool grouped = it.unit_groups > 1;
    if (poster) {
        if (!grouped) {
            store_complete(it.group_blocks);
        } else {
            unsigned long long *acc_unit = acc + (int64_t)it.unit * D;
            const bool last0 = accum_complete(after0, it.group_blocks), last1 = accum_complete(after1, it.group_blocks);
            const unsigned long long t0 = accum_single(after0), t1 = accum_single(after1);
            after0 = after1 = 0ull;
            if (last0) after0 = __hip_atomic_fetch_add(acc_unit + lane, t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t0;
            if (last1) after1 = __hip_atomic_fetch_add(acc_unit + D / 2 + lane, t1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t1;
        }
    }

    // ---- inside the groups: lane (qq, n) of a result holds rows 4 qq + rho, column n; of those, rows up to n count ----
    float c_in, e_in, xx;                                             // (the totals, lane (q, n): group q's token n)
    {
        float c_part[4] = {}, e_part[4] = {}, x_part[4] = {}, wm_prev[4], alpha_prev = 0.f;
#pragma unroll
        for (int m = 0; m <= MG; ++m) {
            const float4 f4 = *reinterpret_cast<const float4 *>(&lds_w[w][m][4 * qq]);
            const float w4[4] = {f4.x, f4.y, f4.z, f4.w};
            float wm[4];
#pragma unroll
            for (int rho = 0; rho < 4; ++rho) wm[rho] = 4 * qq + rho <= n ? w4[rho] : 0.f;
            float alpha = weighted(fine_tile<SF, KS, FINE && KS < 4>(X[m], X[m]), wm);          // <k_i, rows of its own group up to i>
            asm volatile("" : "+v"(alpha));
            if (m > 0) {
                __builtin_amdgcn_sched_barrier(0);
                const u32x4 (&G)[KS] = X[m], (&B)[KS] = X[m ? m - 1 : 0];
                const f32x4 XT = fine_tile<SF, KS, FINE && KS < 4>(B, G);       // [j' in P][i in G]
                c_part[m - 1] = alpha - weighted(XT, wm_prev);                  // <k_i, entered rows of G less left rows of P>
                asm volatile("" : "+v"(c_part[m - 1]));
                __builtin_amdgcn_sched_barrier(0);
                const f32x4 XX = fine_tile<SF, KS, FINE && KS < 4>(G, B);       // [j in G][i' in P]
                e_part[m - 1] = weighted(XX, wm) - alpha_prev;                  // the same of k_i'
                x_part[m - 1] = diagonal(XX, qq, n);                            // <k_i, k_i'>
                asm volatile("" : "+v"(e_part[m - 1]), "+v"(x_part[m - 1]));
            }
#pragma unroll
            for (int rho = 0; rho < 4; ++rho) wm_prev[rho] = wm[rho];
            alpha_prev = alpha;
            __builtin_amdgcn_sched_barrier(0);                        // one group at a time
        }
        c_in = sum_to_groups(c_part);
        e_in = sum_to_groups(e_part);
        xx = sum_to_groups(x_part);
    }
    if (poster && grouped) store_complete(it.unit_groups);            // (the second adds have had the chain to come back)
    {
        // 1/||k|| and ||k||^2 of this lane's token and of the one 64 in front, which is the group before's
        const float wt = lds_w[w][1 + qq][n], wp = lds_w[w][qq][n], ss = lds_ss[w][1 + qq][n], ssp = lds_ss[w][qq][n];
        const float c = c_seed + c_in, e = e_seed + e_in;             // <k_i, W_i>, <k_i', W_i>
        const Norm dd = 2.f * (wt * c - wp * e) + (2.f * wt * wp * xx - (wt * wt * ss + wp * wp * ssp));
        const float Pn = (float)(P0 + row_prefix_sum(dd));
        const float2 total = dim_pair<KS>(lds_B, lane);               // (again: its square would be one register too many until here)
        const float bsq = sum_over_rows16(row_sum<16>(fmaf(total.x, total.x, total.y * total.y)));
        const float ac = token_cos<FINE>(c, wt, ss, Pn), ae = token_cos<FINE>(bd, wt, ss, bsq);
        const __amdgpu_buffer_rsrc_t out_c = __builtin_amdgcn_make_buffer_rsrc(a_raw + 2 * rows + row0, 0, blk_hi * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t out_e = __builtin_amdgcn_make_buffer_rsrc(a_raw + rows + row0, 0, blk_hi * 4, 0x00020000);
        const int at = 4 * token();
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ac), out_c, at, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ae), out_e, at, 0, 0);
    }
    // ---- stable dots against the unit's sum ----
    if (w == 0) {                                                     // D / 4 lanes look, the other waves sit at the barrier
        const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc(S_unit, 0, D * 4, 0x00020000);
        bool got = false;
        for (int polls = 0; poll_limit >= 0; ++polls) {               // poll_limit < 0: defer without looking
            u32x4 sv = {0u, 0u, 0u, 0u};
            if (lane < D / 4) sv = agent_load16(srs, lane * 16);
            got = __all(all_written(sv));                             // (lanes past the vector hold zeros)
            if (got) {
                if (lane < D / 4) *reinterpret_cast<u32x4 *>(&lds_S[4 * lane]) = sv;
                break;
            }
            if (polls >= poll_limit) break;
            __builtin_amdgcn_s_sleep(8);
        }
        if (lane == 0) {
            s_have = got ? 1 : 0;
            if (!got) sync[kSyncWords + atomicAdd(sync + kDeferCountWord, 1u)] = (uint32_t)it.id;
        }
    }
    __syncthreads();
    if (s_have != 0) {
        float2 s2 = sum_pair<KS>(lds_S, lane);
        if constexpr (KF == kKeyF16) { s2.x *= fp16_sum_scale(N); s2.y *= fp16_sum_scale(N); }
        const float ssq = sum_over_rows16(row_sum<16>(fmaf(s2.x, s2.x, s2.y * s2.y)));
        stage_anchor<SF, KS>(stage, 0, 1, 2, lane, s2.x, s2.y);
        __builtin_amdgcn_wave_barrier();
        u32x4 An[KS];
        read_operand<KS>(stage, min(n & 3, 2), qq, An);               // the three terms in every lane group's rows
        float dot[4] = {};
#pragma unroll
        for (int m = 0; m < MG; ++m) dot[m] = sum3(fine_tile<SF, KS, FINE>(An, X[m + 1]));
        const float as = token_cos<FINE>(of_group(dot, qq), lds_w[w][1 + qq][n], lds_ss[w][1 + qq][n], ssq);
        const __amdgpu_buffer_rsrc_t out_s = __builtin_amdgcn_make_buffer_rsrc(a_raw + row0, 0, blk_hi * 4, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(as), out_s, 4 * token(), 0, 0);
    }
}

// a_s of the blocks whose workgroups did not wait for their unit's sum: the same operands (loaded in operand
// layout directly), norms, split and product as in scan_tile_kernel, so the values are the ones it would have
// stored.
template <int KF, int KS, bool FULL, bool FINE>
__global__ __launch_bounds__(64 * kTileWaves) void deferred_stable_tile_kernel(const uint8_t *__restrict__ keys, int d, RowMap km,
                                                                               PromptTab tab,
                                                                               const float *__restrict__ ssum,
                                                                               const uint32_t *__restrict__ sync,
                                                                               float *__restrict__ a_raw)
{
    constexpr int D = 32 * KS, NW = kTileWaves, ES = key_bytes<KF>(), SF = kStaged<KF>;
    const int dims = FULL ? D : d, row_bytes = dims * ES;
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[NW][3 * kPitch<KS>];
    const int nblk = tab.blk_off[tab.n];
    const uint32_t count = sync[kDeferCountWord];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int qq = lane >> 4, n = lane & 15;
    uint8_t *stage = lds_stage[w];
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
        const int id = (int)sync[kSyncWords + i], lh = id / nblk, blk = id - lh * nblk;
        const int p = prompt_of_block(tab, blk);
        const int b = tab.b[p], N = tab.tok_off[p + 1] - tab.tok_off[p];
        const int blk_lo = (blk - tab.blk_off[p]) * b, blk_hi = min(blk_lo + b, N);
        const int ng = (blk_hi - blk_lo + kGroup - 1) / kGroup;
        const int64_t row0 = (int64_t)lh * tab.T + tab.tok_off[p];
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t *>(keys) + km.unit(lh, p, tab) * ES, 0, N * row_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t out_s = __builtin_amdgcn_make_buffer_rsrc(a_raw + row0, 0, blk_hi * 4, 0x00020000);
        // every word of the unit's sum has been stored by now (the pass has ended)
        float2 s2 = sum_pair<KS>(ssum + ((int64_t)lh * tab.n + p) * D, lane);
        if constexpr (KF == kKeyF16) { s2.x *= fp16_sum_scale(N); s2.y *= fp16_sum_scale(N); }   // as in scan_tile_kernel
        const float ssq = sum_over_rows16(row_sum<16>(fmaf(s2.x, s2.x, s2.y * s2.y)));
        __builtin_amdgcn_wave_barrier();                              // the previous block's reads of the staged rows
        stage_anchor<SF, KS>(stage, 0, 1, 2, lane, s2.x, s2.y);
        __builtin_amdgcn_wave_barrier();
        u32x4 An[KS];
        read_operand<KS>(stage, min(n & 3, 2), qq, An);
        for (int q = w; q < ng; q += 4) {
            const int tok = blk_lo + kGroup * q + n, off = tok * row_bytes + 8 * ES * qq;
            u32x4 X[KS];
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                X[kk] = operand_piece<KF>(row_load<KF>(rsrc, 32 * kk + 8 * qq < dims ? off + 32 * ES * kk : kNoByte));
            const float ss = sum_over_rows16(diagonal(fine_tile<SF, KS, true>(X, X), qq, n)), wn = tok < blk_hi ? inv_norm(ss) : 0.f;
            const float as = token_cos<FINE>(sum3(fine_tile<SF, KS, FINE>(An, X)), wn, ss, ssq);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(as), out_s, qq == 0 ? 4 * tok : kNoByte, 0, 0);
        }
    }
}

int resident_tile_workgroups()
{
    static int cached = -1;                                          // benign if raced
    if (cached < 0) {
        int per_cu = 0, dev = 0;
        hipDeviceProp_t prop;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, scan_tile_kernel<kKeyBF16, 4, true, false, 4>, 64 * kTileWaves, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return 0;
        cached = per_cu * prop.multiProcessorCount;
    }
    return cached;
}

// the launches of one call, in the instance that fits its keys
struct TileLaunch {
    const uint8_t *keys;
    int d;
    const RowMap &km;
    const PromptTab &tab;
    const TileItem *items;
    unsigned n_items, n_deferred;
    float *a_raw, *ssum;
    unsigned long long *accum, *accum_group;
    uint32_t *sync;
    int64_t rows;
    int poll_limit;
    bool fine, blocks_128;
    const Prof &prof;
    hipStream_t st;

    template <int KF, int KS, bool FULL, bool FINE> void run() const
    {
        prof.begin(NKV_KERNEL_SCAN, st);
        if (blocks_128) scan_tile_kernel<KF, KS, FULL, FINE, 2><<<n_items, 64 * kTileWaves, 0, st>>>(keys, d, items, a_raw, accum, accum_group, ssum, sync, rows, poll_limit);
        else scan_tile_kernel<KF, KS, FULL, FINE, 4><<<n_items, 64 * kTileWaves, 0, st>>>(keys, d, items, a_raw, accum, accum_group, ssum, sync, rows, poll_limit);
        prof.end(NKV_KERNEL_SCAN, st);
        deferred_stable_tile_kernel<KF, KS, FULL, FINE><<<n_deferred, 64 * kTileWaves, 0, st>>>(keys, d, km, tab, ssum, sync, a_raw);
    }
    // FINE (double-width window norms, corrected reciprocal square roots, anchors' products added up in two halves) where the
    // kernels before this scan were closer to 64 bits than it is without: 16-bit keys of more than 64 dims, except for head dim
    // 128 and units of up to 256 blocks.  Root mean square errors of a_s, a_e, a_c in 1e-8, keys of the benchmark's kind: head dim 96, 8192
    // tokens 2.4, 3.3, 2.8 before, 2.6, 2.9, 3.1 without and 2.4, 2.7, 2.9 with FINE; head dim 128, 100 000 tokens 2.3, 2.2,
    // 2.6, then 2.5, 2.7, 2.9 and 2.2, 2.5, 2.7 (6 % of the scan's time); 8-bit keys 2.1, 2.2, 2.5 and 2.0, 2.2, 2.5 without.
    // (Those figures are from norms by dot products and terms added up largest first.  With norms in two halves, the small
    // terms first and the block's groups in 64 bits: head dim 96, 2.4, 2.6, 2.6; 128, 100 000 tokens 1.7, 2.3, 2.5 (1.8, 2.5, 2.7 on the
    // same keys before that); 8-bit 2.0, 2.1, 2.3; bf16, 128, 65 536 tokens 2.0, 2.6, 2.7.)
    // Keys that cancel inside the window cost more: a common direction 60 times the spread that changes sign every 64 tokens leaves
    // an rms error of a_c of 5.4e-7 at head dim 128, 2.7e-7 with FINE (96: 3.1e-7), where the vector scan has 0.9e-7.
    template <int KF> void run_format() const
    {
        constexpr bool F = KF != kKeyF8;
        if (d == 128 && fine && F) run<KF, 4, true, F>();
        else if (d == 128) run<KF, 4, true, false>();
        else if (d > 96) run<KF, 4, false, F>();
        else if (d > 64) run<KF, 3, false, F>();
        else run<KF, 2, false, false>();                              // (matches padded_dims)
    }
};

}  // namespace

static int longest_unit(const PromptTab &tab)                        // in blocks
{
    int most = 0;
    for (int p = 0; p < tab.n; ++p) most = max(most, tab.blk_off[p + 1] - tab.blk_off[p]);
    return most;
}

static int longest_block(const PromptTab &tab)                      // in tokens
{
    int most = 0;
    for (int p = 0; p < tab.n; ++p) most = max(most, (int)tab.b[p]);
    return most;
}

bool tile_score_supported(int dtype, int d, int window, const PromptTab &tab, int LH)
{
    // (head dim 64 stays with the vector formulation, whose window norms lose less where keys cancel inside the window: rms
    // error of a_c 1.7e-7 against 7.4e-7 here for a common direction that changes sign every 64 tokens.  16 layers x 8 heads x
    // 4096 tokens take 49.6 us there and 46.2 here.)
    if (dtype == NKV_DTYPE_F32 || d > 128 || d == 64 || window != 64) return false;
    for (int p = 0; p < tab.n; ++p) {
        const int N = tab.tok_off[p + 1] - tab.tok_off[p];
        if (tab.b[p] > 256 || N > kMaxUnitTokens) return false;
        // the count of a word of the unit holds its groups (blocks of fewer than 32 tokens only)
        if (unit_groups(tab.blk_off[p + 1] - tab.blk_off[p]) > kMaxUnitBlocks) return false;
        if ((int64_t)(N + 512) * d * 2 >= kNoByte) return false;
    }
    return (int64_t)LH * (tab.blk_off[tab.n] + tab.n) < (1ll << 28);
}

// A workgroup of this scan takes a block and loads 64 tokens in front of it whatever the block's length.  Where there are more blocks
// of a unit than fit the chip together (so that every one is deferred as well), short ones are done sooner by other kernels.  A call's
// prompts take one scan, so the mean block of all of them decides: this scan's time goes with the blocks, the shape-generic kernels'
// with the tokens.
// 16-bit keys, up to 24 tokens.  Score call of 8 heads x 16384 tokens in blocks of 4, this scan / shape-generic: bf16, head
// dim 128, one layer 455 / 311 us, four layers 1697 / 740; head dim 40 444 / 194 and 1659 / 552.  In blocks of 8: 249 / 193 and
// 872 / 469.  Units of 1100 blocks of 24, one layer, four and sixteen 164 / 164, 519 / 427 and 1962 / 1550, of 28 165 / 172,
// 526 / 473 and 2011 / 1644; head dim 40, of 24 155 / 115 and 491 / 314.
// 8-bit keys, head dim 128 (at others the shape-generic kernels leave more error in a_s, which they add up in 32 bits: head dim 32,
// blocks of 3, 6.1e-8 against 5.3e-8).  Units of 2048 blocks, this scan / shape-generic / vector scan: 8 heads, of 2 tokens 445 / 427 / 1128, of 4
// 239 / 251 / 486; 16 heads, of 4 440 / 398 / 827, of 6 449 / 464 / 833; 64 heads 1675 / 1292 / 2880 and 1683 / 1542 / 2905.  The vector scan holds
// 2048 blocks at a time and is quick where a unit has more, so that none waits, and there are many of them: units of 2100, 32
// heads, of 4 877 / 720 / 815, of 6 880 / 849 / 824; 64 heads 1715 / 1336 / 1088 and 1723 / 1587 / 1115; 256 heads, of 2 6762 / 4775 / 2991.  (Not
// for single tokens: 32 heads x 16384 6586 / 4866 / 8167.)
TinyBlocks tile_tiny_blocks(int dtype, int d, const PromptTab &tab, int LH)
{
    const int longest = longest_unit(tab), resident = resident_tile_workgroups();
    if (longest <= resident) return kTinyNone;
    const int64_t blocks = tab.blk_off[tab.n];
    if (dtype != NKV_DTYPE_F8_E4M3) return tab.T <= 24 * blocks ? kTinyGeneric : kTinyNone;
    if (d != 128) return kTinyNone;
    const bool vector = longest > 2 * resident && tab.T > blocks;
    if (tab.T <= (LH >= 16 ? 5 : 3) * blocks && !(vector && LH >= 64)) return kTinyGeneric;
    return vector && tab.T <= 7 * blocks && LH >= 32 ? kTinyVector : kTinyNone;
}

size_t tile_score_plan_bytes(int LH, const PromptTab &tab)
{
    ScanPlan plan;
    return (size_t)fill_scan_plan(LH, tab, 1, &plan, false) * sizeof(TileItem);
}

size_t tile_score_accum_bytes(int LH, int d, const PromptTab &tab)
{
    return (size_t)LH * (tab.n + group_slots(tab.blk_off[tab.n], tab.n)) * padded_dims(d) * 8;
}

hipError_t launch_score_tile(const void *keys, const RowMap &km, int dtype, int LH, int d, const PromptTab &tab, float *a_raw,
                             void *accum, float *ssum, void *sync_area, void *plan_area, int mode, const Prof &prof,
                             hipStream_t st)
{
    // (no unit is added up by a workgroup of its own here)  Where the blocks of a unit do not fit the chip together, nobody looks
    // for a unit's sum and all blocks take the deferred route.
    const bool defer_all = mode == kScanDeferAll || mode == kScanRepairAll || longest_unit(tab) > resident_tile_workgroups();
    const size_t nu = (size_t)LH * tab.n * padded_dims(d) * 8 / 16;           // the units' accumulators, in 16-byte pieces
    const size_t na = tile_score_accum_bytes(LH, d, tab) / 16;                // theirs, and the groups' behind them
    ScanPlan plan;
    const unsigned n_items = fill_scan_plan(LH, tab, km.H, &plan, false);
    plan_kernel<<<(unsigned)min(((size_t)n_items + 255) / 256, (size_t)2048), 256, 0, st>>>(
        (TileItem *)plan_area, n_items, km, tab, plan, LH, (uint4 *)sync_area, kSyncWords / 4, (uint4 *)accum, na, (uint4 *)ssum,
        nu / 2);
    const TileLaunch go{(const uint8_t *)keys, d, km, tab, (const TileItem *)plan_area, n_items, defer_all ? 4096u : 256u, a_raw,
                        ssum, (unsigned long long *)accum, (unsigned long long *)accum + nu * 2, (uint32_t *)sync_area, (int64_t)LH * tab.T,
                        defer_all ? -1 : kPollLimit, longest_unit(tab) > 256, longest_block(tab) <= 128, prof, st};
    if (dtype == NKV_DTYPE_F16) go.run_format<kKeyF16>();
    else if (dtype == NKV_DTYPE_F8_E4M3) go.run_format<kKeyF8>();
    else go.run_format<kKeyBF16>();
    return hipGetLastError();
}

}  // namespace nkv
