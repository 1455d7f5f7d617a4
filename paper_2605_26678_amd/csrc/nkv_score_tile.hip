// Streaming scoring kernel for bf16, fp16 or 8-bit (E4M3) keys of head dim <= 128 (64 excepted, see
// tile_score_supported), window 64, episodic block size <= 256 (paper Sections 2.1-2.3), with every dot product of the
// pass formed by the matrix cores.  (Written out below for bf16 and head dim 128; fp16 differs in the product
// instruction, in unpacking, and in how an fp32 anchor is cut into three terms; 8-bit keys become bf16, exactly, on
// their way from the load; other head dims are padded with zeros to 32 KS, which no dot product and no norm sees.)
//
// The pass is a stream over the keys and nothing else is read from memory, but written for the vector unit it
// needs ~2300 instructions per 64 tokens and is bound by their issue.  Here the vector unit keeps only the work
// that is a sum over tokens (the partial sums of normalised keys that the anchors are made of); everything that
// is a contraction over the head dimension goes through v_mfma_f32_16x16x32_bf16, whose products of bf16 values
// are exact and whose sums are fp32:
//
//   * a block is cut into groups of 16 tokens.  T_q = sum of k_hat over group q (vector unit).  The window sum in
//     front of group q's first token is exact in terms of groups: Seed_q = T_{q-4} + ... + T_{q-1}.
//   * for token i of group G, with P the group 64 tokens earlier (token i' = i - 64 leaves as i enters),
//         W_i = Seed_G + sum_{j in G, j <= i} k_hat_j - sum_{j' in P, j' <= i'} k_hat_j',
//     so <k_i, W_i> = <k_i, Seed_G> + sum_{j <= i} w_j A[i][j] - sum_{j' <= i'} w_j' X[i][j'] with the Gram tiles
//     A = K_G K_G^T and X = K_G K_P^T of the raw keys and w = 1 / ||k||.
//   * ||W_i||^2 follows the window inside the group: it is ||Seed_G||^2 plus the running sum of
//         ||W_i||^2 - ||W_{i-1}||^2 = 2 <W_i, d_i> - ||d_i||^2,   d_i = k_hat_i - k_hat_i',
//     which needs <k_i', W_i> (same tiles, the other triangle) and X[i][i'].  At most 16 terms are added up.
//   * <k, anchor> for the anchors that are vectors (Seed_G, the block total, the unit sum): the fp32 anchor is
//     split into three bf16 terms (8 + 8 + 8 mantissa bits, exact) that form rows of the left operand.
//
// Layouts.  A wave owns the groups q = w, w + 4, w + 8, w + 12 of the block (so the group 64 tokens earlier is
// its own previous group) and the group of the halo in front of them.  A group is loaded row-wise (lane (g, c):
// rows 4g .. 4g+3, dims 8c .. 8c+7; four contiguous 256-byte pieces per load instruction), which is the layout
// the partial sums want, and passes through 4 KB of LDS private to the wave to become a matrix operand (lane
// (q, n): token n, dims 32 kk + 8q .. + 7 in operand register kk).  Operands stay in registers until the unit's
// sum has arrived.  A 16 x 16 result leaves lane (q, n) with column n, rows 4q .. 4q+3: sums over rows are four
// multiply-adds per lane followed by a sum over the four lanes n, n+16, n+32, n+48.
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

using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));
using f16x8 = _Float16 __attribute__((ext_vector_type(8)));
using f32x4 = float __attribute__((ext_vector_type(4)));

constexpr int kNoByte = 0x40000000;              // an offset past any buffer of the pass, also with a token's offset added:
                                                 // loads read zeros there, stores are dropped
constexpr int kGroup = 16;                       // tokens per group
constexpr int kPitch = 272;                      // bytes between the rows of a staged group: 16 lanes that read the
                                                 // same piece of 16 rows touch every LDS bank once
constexpr int kStageBytes = kGroup * kPitch;
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

// The same, as two halves where FINE: sums of half the length.  (Four quarters are closer still, but do not fit the
// registers; for the products of keys with keys, neither do two where KS = 4.)
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

// T[e], e < 8: partial sums of dims 8c + e held by lane (g, c).  Summed over g; lane (g, c) receives the totals
// of dims 8c + 2g and 8c + 2g + 1.  Each step halves the number of live values.
__device__ __forceinline__ float2 sum_over_rows16_transposing(const float (&T)[8])
{
    float U[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {                // lower half: dim e, upper half: dim e + 4
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(T[e]), __float_as_uint(T[e + 4]), false, false);
        U[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    float V[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {                // rows 0..3 of 16 lanes: dims e, e + 2, e + 4, e + 6
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(U[e]), __float_as_uint(U[e + 2]), false, false);
        V[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return make_float2(V[0], V[1]);
}

// The same in 64 bits, and over the whole wavefront.
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

// inclusive running sum over the 16 lanes of a row (lanes n = 0 .. 15 of every group of 16)
__device__ __forceinline__ float row_prefix_sum(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, true));   // row_shr:1
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, true));   // row_shr:2
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, true));   // row_shr:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, true));   // row_shr:8
    return x;
}

// fp32 -> three 16-bit terms whose sum is the value.  bf16: each term takes the next 8 mantissa bits, exact.  fp16:
// each term is the rounded remainder (11 bits each; the remainders are exact, the last term is off by at most 2^-33
// of the value or by fp16's smallest step, 6e-8, whichever is larger); the value must be below fp16's largest, 65504.
template <int KF> __device__ __forceinline__ void split3(float x, uint32_t &hi, uint32_t &mid, uint32_t &lo)
{
    if constexpr (KF == kKeyF16) {
        const _Float16 h = (_Float16)x;
        const float r1 = x - (float)h;
        const _Float16 m = (_Float16)r1;
        const float r2 = r1 - (float)m;
        const _Float16 l = (_Float16)r2;
        hi = __builtin_bit_cast(unsigned short, h);
        mid = __builtin_bit_cast(unsigned short, m);
        lo = __builtin_bit_cast(unsigned short, l);
        return;
    }
    const uint32_t b0 = __float_as_uint(x) & 0xffff0000u;
    const float r1 = x - __uint_as_float(b0);
    const uint32_t b1 = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(b1);
    hi = b0 >> 16;
    mid = b1 >> 16;
    lo = __float_as_uint(r2) >> 16;
}

// The factor that keeps a sum of N unit vectors inside fp16's range; the cosine does not see it.
__device__ __forceinline__ float fp16_sum_scale(int N) { return N <= 131072 ? 0.25f : 0.03125f; }

// A vector of which this lane holds dims 2 lane and 2 lane + 1, as the three terms of rows row0 .. row0 + 2
// of a staged left operand.
template <int KF> __device__ __forceinline__ void stage_anchor(uint8_t *stage, int row0, int lane, float v0, float v1)
{
    uint32_t h0, m0, l0, h1, m1, l1;
    split3<KF>(v0, h0, m0, l0);
    split3<KF>(v1, h1, m1, l1);
    *reinterpret_cast<uint32_t *>(stage + (row0 + 0) * kPitch + 4 * lane) = h0 | (h1 << 16);
    *reinterpret_cast<uint32_t *>(stage + (row0 + 1) * kPitch + 4 * lane) = m0 | (m1 << 16);
    *reinterpret_cast<uint32_t *>(stage + (row0 + 2) * kPitch + 4 * lane) = l0 | (l1 << 16);
}

// The staged 16 rows as a matrix operand: lane (q, n) takes dims 32 kk + 8 q .. + 7 of row n.
template <int KS> __device__ __forceinline__ void read_operand(const uint8_t *stage, int lane, u32x4 (&x)[KS])
{
    const uint8_t *mine = stage + (lane & 15) * kPitch + 16 * (lane >> 4);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) x[kk] = *reinterpret_cast<const u32x4 *>(mine + 64 * kk);
}

// The format the staged rows are in: 8-bit keys travel as bf16.
template <int KF> constexpr int kStaged = KF == kKeyF16 ? kKeyF16 : kKeyBF16;

// A loaded row piece in the staged format.  E4M3 -> bf16 is exact (3 mantissa bits into 7, exponents -9 .. 8): the
// upper halves of the fp32 values are the bf16 values.
template <int KF> __device__ __forceinline__ u32x4 staged_piece(const Piece<KF> &r)
{
    if constexpr (KF == kKeyF8) {
        float k[8];
        unpack8_f8(r, k);
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_perm(__float_as_uint(k[2 * i + 1]), __float_as_uint(k[2 * i]), 0x07060302u);
        return o;
    } else {
        return r;
    }
}

// Sums of the squares of a lane's eight values of each of its four rows, ready to be read by any vector instruction (the
// compiler does not see the writes inside the assembly): four independent chains of exact products.
template <int KF> __device__ __forceinline__ void rows_sumsq(const u32x4 (&r)[4], float (&ss)[4])
{
#define NKV_DOTS(OP)                                                                                                      \
    asm(OP " %0, %4, %4\n\t" OP " %1, %8, %8\n\t" OP " %2, %12, %12\n\t" OP " %3, %16, %16\n\t"                            \
        OP " %0, %5, %5\n\t" OP " %1, %9, %9\n\t" OP " %2, %13, %13\n\t" OP " %3, %17, %17\n\t"                            \
        OP " %0, %6, %6\n\t" OP " %1, %10, %10\n\t" OP " %2, %14, %14\n\t" OP " %3, %18, %18\n\t"                          \
        OP " %0, %7, %7\n\t" OP " %1, %11, %11\n\t" OP " %2, %15, %15\n\t" OP " %3, %19, %19\n\t"                          \
        "s_nop 3"                                                                                                         \
        : "+v"(ss[0]), "+v"(ss[1]), "+v"(ss[2]), "+v"(ss[3])                                                              \
        : "v"(r[0].x), "v"(r[0].y), "v"(r[0].z), "v"(r[0].w), "v"(r[1].x), "v"(r[1].y), "v"(r[1].z), "v"(r[1].w),          \
          "v"(r[2].x), "v"(r[2].y), "v"(r[2].z), "v"(r[2].w), "v"(r[3].x), "v"(r[3].y), "v"(r[3].z), "v"(r[3].w))
#pragma unroll
    for (int j = 0; j < 4; ++j) ss[j] = 0.f;
    if constexpr (KF == kKeyF16) NKV_DOTS("v_dot2c_f32_f16");
    else NKV_DOTS("v_dot2c_f32_bf16");
#undef NKV_DOTS
}

// One group of 16 tokens in row-wise layout (lane (g, c): rows 4g .. 4g+3, dims 8c .. 8c+7; tok0 = the group's
// first token, which may lie in front of the prompt): ||k||^2 and the weight 1/||k|| of every row (0 for tokens
// outside [0, tok_end)) go to ss_out / w_out.  The four rows of a lane are reduced together by a transposing butterfly,
// after which lane (g, c) holds row 4g + c % 4: one square root per group instead of one per row.
template <int KF> __device__ __forceinline__ void group_norms(const u32x4 (&raw)[4], int tok0, int tok_end, int g, int c, float *w_out,
                                            float *ss_out)
{
    float ss[4];
    rows_sumsq<KF>(raw, ss);
    float s = merge_low4(ss);
    s += dpp_mov<0x124>(s);                                           // row_ror:4
    s += dpp_mov<0x128>(s);                                           // row_ror:8
    const int tok = tok0 + 4 * g + (c & 3);
    const float ww = tok >= 0 && tok < tok_end ? inv_norm(s) : 0.f;
    if (c < 4) {                                                      // (the quads' sums may differ in the last bit: one of them counts)
        w_out[4 * g + c] = ww;
        ss_out[4 * g + c] = s;
    }
}

// The weighted sum of the group's rows to sum_out (32 KS floats), with the weights that group_norms left (same wave: in
// order).
template <int KF, int KS> __device__ __forceinline__ void group_sum(const u32x4 (&raw)[4], int g, int c, const float *w_in, float *sum_out)
{
    const float4 w4 = *reinterpret_cast<const float4 *>(w_in + 4 * g);
    const float ww[4] = {w4.x, w4.y, w4.z, w4.w};
    float T[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) T[e] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float k[8];
        unpack8<KF>(raw[j], k);
#pragma unroll
        for (int e = 0; e < 8; ++e) T[e] = fmaf(ww[j], k[e], T[e]);
    }
    const float2 t2 = sum_over_rows16_transposing(T);
    if (KS == 4 || 8 * c < 32 * KS) *reinterpret_cast<float2 *>(sum_out + 8 * c + 2 * g) = t2;
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

__device__ __forceinline__ float sum3(const f32x4 &d) { return (d[0] + d[1]) + d[2]; }

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

// grid: one workgroup of 256 threads per item, in the items' order.  (Resident workgroups that loop over the items
// instead were tried: without the hardware handing out blocks as slots fall free, all workgroups of the chip move
// through their loading and computing phases in step, and the pass takes 0.90 ms instead of 0.77.)
// KS: head dims the pass works with, in steps of 32 (the rest of the last step reads as zeros); FULL: d = 32 KS.
template <int KF, int KS, bool FULL, bool FINE> __global__ __launch_bounds__(64 * kTileWaves, 4)
void scan_tile_kernel(const uint8_t *__restrict__ keys, int d, const TileItem *__restrict__ items, float *__restrict__ a_raw,
                      unsigned long long *__restrict__ acc, unsigned long long *__restrict__ acc_group, float *__restrict__ ssum, uint32_t *__restrict__ sync, int64_t rows,
                      int poll_limit)
{
    constexpr int D = 32 * KS, NW = kTileWaves, ES = key_bytes<KF>(), SF = kStaged<KF>;
    const int row_bytes = FULL ? D * ES : d * ES;
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[NW][kStageBytes];   // a wave's group on its way to operand layout, later its anchors
    __shared__ __attribute__((aligned(16))) float lds_T[4 + 16][D];               // group sums: 4 halo groups, then the block's
    __shared__ __attribute__((aligned(16))) float lds_w[NW][5][kGroup];           // 1/||k|| per token of a wave's groups (0: no such token)
    __shared__ __attribute__((aligned(16))) float lds_ss[NW][5][kGroup];          // ||k||^2
    __shared__ __attribute__((aligned(16))) float lds_S[D];                       // the unit's sum, once complete
    __shared__ int s_have;

    const TileItem it = items[blockIdx.x];
    if (it.N < 0) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, c = lane & 15;                           // row-wise layout: rows 4g .., dims 8c ..
    const int qq = g, n = c;                                          // operand / result layout: token n, quarter qq
    uint8_t *stage = lds_stage[w];

    const int N = it.N, blk_lo = it.blk_lo, blk_hi = it.blk_hi;
    const int ng = (blk_hi - blk_lo + kGroup - 1) / kGroup;           // groups of the block, <= 16
    const int64_t row0 = it.row0;                                     // row of the prompt's token 0

    // ---- first touch: this wave's groups, then its group of the halo.  Rows outside the prompt read as zeros. ----
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(keys) + it.key_off * ES, 0, N * row_bytes, 0x00020000);
    const int piece_off = FULL && KS == 4 ? 8 * ES * c : (8 * c < (FULL ? D : d) ? 8 * ES * c : kNoByte);
    Piece<KF> raw[5][4];
    bool ex[5];                                                       // group m - 1 of the chain exists (m = 0: halo)
#pragma unroll
    for (int mm = 0; mm < 5; ++mm) {
        const int m = (mm + 1) % 5;                                   // the halo is needed last
        const int q = w + 4 * (m - 1);                                // block-local group index, < 0: halo
        ex[m] = q < ng;
        if (ex[m]) {
            const int off = (blk_lo + kGroup * q + 4 * g) * row_bytes + piece_off;
#pragma unroll
            // a full block's last 64 tokens (m = 4) are read again, as the next block's halo, and the halo has just
            // been read by the block in front: those stay in the L2; the other rows are marked non-temporal (aux 2)
            for (int j = 0; j < 4; ++j)
                raw[m][j] = (m >= 1 && m <= 3) ? row_load<KF, 2>(rsrc, off + j * row_bytes) : row_load<KF>(rsrc, off + j * row_bytes);
        }
    }

    // ---- the block's own groups: norms and partial sums, nothing else in front of the block total ----
    u32x4 row[5][4];                                                  // the rows in the staged format
#pragma unroll
    for (int m = 1; m < 6; ++m) {                                     // a group's sum behind the next one's norms
        if (m < 5 && ex[m]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) row[m][j] = staged_piece<KF>(raw[m][j]);
            group_norms<SF>(row[m], blk_lo + kGroup * (w + 4 * (m - 1)), blk_hi, g, c, lds_w[w][m], lds_ss[w][m]);
        }
        if (m > 1 && ex[m - 1]) group_sum<SF, KS>(row[m - 1], g, c, lds_w[w][m - 1], lds_T[4 + w + 4 * (m - 2)]);
    }
    __syncthreads();

    // ---- block total = episodic anchor (up to length); lane: dims 2 lane, 2 lane + 1 ----
    unsigned long long *acc_mine = acc_group + (int64_t)it.group * D;
    float bsq, b0 = 0.f, b1 = 0.f;
    for (int q = 0; q < ng; ++q) {
        const float2 t2 = dim_pair<KS>(lds_T[4 + q], lane);
        b0 += t2.x;
        b1 += t2.y;
    }
    const bool poster = w == (it.id & (NW - 1));                      // one wave adds the block total to the unit's sum
    unsigned long long after0 = 0ull, after1 = 0ull;                  // the accumulators right after this block's add
    if (poster && (KS == 4 || lane < D / 2)) {
        const unsigned long long t0 = accum_term(b0), t1 = accum_term(b1);
        after0 = __hip_atomic_fetch_add(acc_mine + lane, t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t0;
        after1 = __hip_atomic_fetch_add(acc_mine + D / 2 + lane, t1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + t1;
    }
    bsq = sum_over_rows16(row_sum<16>(fmaf(b0, b0, b1 * b1)));

    // ---- the halo group's sum (the window sums in front of the block's first groups need it) ----
#pragma unroll
    for (int j = 0; j < 4; ++j) row[0][j] = staged_piece<KF>(raw[0][j]);
    group_norms<SF>(row[0], blk_lo + kGroup * (w - 4), blk_hi, g, c, lds_w[w][0], lds_ss[w][0]);
    group_sum<SF, KS>(row[0], g, c, lds_w[w][0], lds_T[w]);

    float *S_unit = ssum + (int64_t)it.unit * D;
    // (The adds have had the halo group to come back.)  The last block to add to a word of the unit stores the word's final
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

    // ---- every group through the staging rows into operand layout ----
    u32x4 X[5][KS];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        if (ex[m]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(stage + (4 * g + j) * kPitch + 16 * c) = row[m][j];
            __builtin_amdgcn_wave_barrier();
            read_operand<KS>(stage, lane, X[m]);
            __builtin_amdgcn_wave_barrier();                          // the next group reuses the staging rows
        }
    }
    if (poster && grouped) store_complete(it.unit_groups);            // (the second adds have had the staging to come back)
    stage_anchor<SF>(stage, 4, lane, b0, b1);                             // rows 4 .. 6: the block total's three terms
    __syncthreads();                                                  // the halo groups' sums
    // ---- the chain of this wave's groups ----
    // lane (qq, n) of a result holds rows 4 qq + rho, column n.  Masked weights of the rows: rows j <= n count.
    const __amdgpu_buffer_rsrc_t out_c = __builtin_amdgcn_make_buffer_rsrc(a_raw + 2 * rows + row0, 0, blk_hi * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t out_e = __builtin_amdgcn_make_buffer_rsrc(a_raw + rows + row0, 0, blk_hi * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t out_s = __builtin_amdgcn_make_buffer_rsrc(a_raw + row0, 0, blk_hi * 4, 0x00020000);
    const int off_q0 = qq == 0 ? 4 * n : kNoByte, off_q1 = qq == 1 ? 4 * n : kNoByte;
    float wm_prev[4], alpha_prev;
    {
        const float4 w4 = *reinterpret_cast<const float4 *>(&lds_w[w][0][4 * qq]);
        const float ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int rho = 0; rho < 4; ++rho) wm_prev[rho] = 4 * qq + rho <= n ? ww[rho] : 0.f;
        alpha_prev = weighted(tile<SF, KS>(X[0], X[0]), wm_prev);          // halo group: its own triangle only
    }
#pragma unroll
    for (int m = 1; m < 5; ++m) {
        if (ex[m]) {
            const int q = w + 4 * (m - 1);
            // window sum in front of the group = the four groups before it
            float s0, s1;
            {
                const float2 t0 = dim_pair<KS>(lds_T[q], lane);
                const float2 t1 = dim_pair<KS>(lds_T[q + 1], lane);
                const float2 t2 = dim_pair<KS>(lds_T[q + 2], lane);
                const float2 t3 = dim_pair<KS>(lds_T[q + 3], lane);
                s0 = ((t0.x + t1.x) + t2.x) + t3.x;
                s1 = ((t0.y + t1.y) + t2.y) + t3.y;
            }
            std::conditional_t<FINE, double, float> P0;               // ||W||^2 in front of the group
            if constexpr (FINE) P0 = wave_sum(fma((double)s0, (double)s0, (double)s1 * (double)s1));
            else P0 = sum_over_rows16(row_sum<16>(fmaf(s0, s0, s1 * s1)));
            stage_anchor<SF>(stage, 0, lane, s0, s1);                     // rows 0 .. 2: the seed's three terms
            __builtin_amdgcn_wave_barrier();
            u32x4 An[KS];
            read_operand<KS>(stage, lane, An);
            __builtin_amdgcn_wave_barrier();                          // the next group rewrites rows 0 .. 2
            const f32x4 AT = fine_tile<SF, KS, FINE && KS < 4>(X[m], X[m]);                     // [j in G][i in G]
            const f32x4 XT = fine_tile<SF, KS, FINE && KS < 4>(X[m - 1], X[m]);                 // [j' in P][i in G]
            const f32x4 XX = fine_tile<SF, KS, FINE && KS < 4>(X[m], X[m - 1]);                 // [j in G][i' in P]
            const f32x4 AG = fine_tile<SF, KS, FINE>(An, X[m]);                       // [anchor row][i in G]
            const f32x4 AP = fine_tile<SF, KS, FINE && KS < 4>(An, X[m - 1]);                   // [anchor row][i' in P]
            float wm[4];
            {
                const float4 w4 = *reinterpret_cast<const float4 *>(&lds_w[w][m][4 * qq]);
                const float ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int rho = 0; rho < 4; ++rho) wm[rho] = 4 * qq + rho <= n ? ww[rho] : 0.f;
            }
            const float alpha = weighted(AT, wm);                     // <k_i, entered rows of G>, partial
            const float beta = weighted(XT, wm_prev);                 // <k_i, left rows of P>, partial
            const float gamma = weighted(XX, wm);                     // <k_i', entered rows of G>, partial
            // X[i][i']: row i of this lane's column i' = n sits in lane group n / 4, register n % 4
            float xd = (n & 2) ? ((n & 1) ? XX[3] : XX[2]) : ((n & 1) ? XX[1] : XX[0]);
            xd = (n >> 2) == qq ? xd : 0.f;
            // 1/||k|| (0: no such token) and ||k||^2 of token n of this group and of the one 64 tokens earlier
            const float wn = lds_w[w][m][n], wp = lds_w[w][m - 1][n], ssn = lds_ss[w][m][n], ssp = lds_ss[w][m - 1][n];
            const float c_part = (qq == 0 ? sum3(AG) : 0.f) + (alpha - beta);
            const float e_part = (qq == 0 ? sum3(AP) : 0.f) + (gamma - alpha_prev);
            const float gsum = qq == 0 ? wn * wn * ssn + wp * wp * ssp : 0.f;
            const float d_part = 2.f * (wn * c_part - wp * e_part) + (2.f * wn * wp * xd - gsum);
            const float cdot = sum_over_rows16(c_part);               // <k_i, W_i>
            const decltype(P0) d_all = sum_over_rows16(d_part);
            const float Pn = (float)(P0 + row_prefix_sum(d_all));
            const float ac = token_cos<FINE>(cdot, wn, ssn, Pn);
            const float ae = token_cos<FINE>(sum3(AG), wn, ssn, bsq); // meaningful in lane group 1 (rows 4 .. 6)
            const int soff = (blk_lo + kGroup * q) * 4;                // (an offset that was past the buffer stays past it)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ac), out_c, off_q0 + soff, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ae), out_e, off_q1 + soff, 0, 0);
#pragma unroll
            for (int rho = 0; rho < 4; ++rho) wm_prev[rho] = wm[rho];
            alpha_prev = alpha;
            __builtin_amdgcn_sched_barrier(0);                        // one group at a time
        }
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
        stage_anchor<SF>(stage, 0, lane, s2.x, s2.y);
        __builtin_amdgcn_wave_barrier();
        u32x4 An[KS];
        read_operand<KS>(stage, lane, An);
#pragma unroll
        for (int m = 1; m < 5; ++m) {
            if (ex[m]) {
                const int q = w + 4 * (m - 1);
                const f32x4 AS = fine_tile<SF, KS, FINE>(An, X[m]);
                const float wn = lds_w[w][m][n], ssn = lds_ss[w][m][n];
                const float as = token_cos<FINE>(sum3(AS), wn, ssn, ssq);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(as), out_s, off_q0 + (blk_lo + kGroup * q) * 4, 0, 0);
            }
        }
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
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[NW][kStageBytes];
    __shared__ __attribute__((aligned(16))) float lds_w[NW][kGroup], lds_ss[NW][kGroup];
    const int nblk = tab.blk_off[tab.n];
    const uint32_t count = sync[kDeferCountWord];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int qq = lane >> 4, n = lane & 15, g = qq, c = n;
    uint8_t *stage = lds_stage[w];
    const int off_q0 = qq == 0 ? 4 * n : kNoByte;
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
        stage_anchor<SF>(stage, 0, lane, s2.x, s2.y);
        __builtin_amdgcn_wave_barrier();
        u32x4 An[KS];
        read_operand<KS>(stage, lane, An);
        for (int q = w; q < ng; q += 4) {
            const int tok0 = blk_lo + kGroup * q;
            u32x4 raw[4], X[KS];                                      // the group row-wise (norms) and as an operand
            const int roff = (tok0 + 4 * g) * row_bytes + (8 * c < dims ? 8 * ES * c : kNoByte);
            const int off = (tok0 + n) * row_bytes + 8 * ES * qq;
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[j] = staged_piece<KF>(row_load<KF>(rsrc, roff + j * row_bytes));
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                X[kk] = staged_piece<KF>(row_load<KF>(rsrc, 32 * kk + 8 * qq < dims ? off + 32 * ES * kk : kNoByte));
            group_norms<SF>(raw, tok0, blk_hi, g, c, lds_w[w], lds_ss[w]);
            __builtin_amdgcn_wave_barrier();
            const float wn = lds_w[w][n], ss = lds_ss[w][n];
            __builtin_amdgcn_wave_barrier();                          // the next group rewrites them
            const f32x4 AS = fine_tile<SF, KS, FINE>(An, X);
            const float as = token_cos<FINE>(sum3(AS), wn, ss, ssq);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(as), out_s, off_q0 + tok0 * 4, 0, 0);
        }
    }
}

int resident_tile_workgroups()
{
    static int cached = -1;                                          // benign if raced
    if (cached < 0) {
        int per_cu = 0, dev = 0;
        hipDeviceProp_t prop;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, scan_tile_kernel<kKeyBF16, 4, true, false>, 64 * kTileWaves, 0) != hipSuccess ||
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
    bool fine;
    const Prof &prof;
    hipStream_t st;

    template <int KF, int KS, bool FULL, bool FINE> void run() const
    {
        prof.begin(NKV_KERNEL_SCAN, st);
        scan_tile_kernel<KF, KS, FULL, FINE><<<n_items, 64 * kTileWaves, 0, st>>>(keys, d, items, a_raw, accum, accum_group, ssum, sync, rows, poll_limit);
        prof.end(NKV_KERNEL_SCAN, st);
        deferred_stable_tile_kernel<KF, KS, FULL, FINE><<<n_deferred, 64 * kTileWaves, 0, st>>>(keys, d, km, tab, ssum, sync, a_raw);
    }
    // FINE (double-width window norms, corrected reciprocal square roots, anchors' products added up in two halves) where the
    // kernels before this scan were closer to 64 bits than it is without: 16-bit keys of more than 64 dims, except for head dim
    // 128 and units of up to 256 blocks.  Root mean square errors of a_s, a_e, a_c in 1e-8, keys of the benchmark's kind: head dim 96, 8192
    // tokens 2.4, 3.3, 2.8 before, 2.6, 2.9, 3.1 without and 2.4, 2.7, 2.9 with FINE; head dim 128, 100 000 tokens 2.3, 2.2,
    // 2.6, then 2.5, 2.7, 2.9 and 2.2, 2.5, 2.7 (6 % of the scan's time); 8-bit keys 2.1, 2.2, 2.5 and 2.0, 2.2, 2.5 without.
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

bool tile_score_supported(int dtype, int d, int window, const PromptTab &tab, int LH)
{
    // (head dim 64 stays with the vector formulation: half of the lanes of a row would hold nothing here)
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

// A workgroup of this scan takes a block and loads 64 tokens in front of it whatever the block's length.  Blocks of fewer
// than 8 tokens, more of a unit than fit the chip together (so that every one is deferred as well), are done sooner by
// other kernels.  Score call of 8 heads x 16384 tokens in blocks of 4, this scan / vector scan / shape-generic: bf16, head
// dim 128, one layer 466 / 1204 / 423 us, four layers 1722 / 1800 / 1128; head dim 40 457 / - / 291 and 1683 / - / 883; 8-bit,
// head dim 128 470 / 1135 / 643 and 1727 / 1558 / 1988 (in blocks of one 6746 / 8167 / 6226).  In blocks of 8: bf16 258 / 639 / 288 and 891 / 946 / 785.
TinyBlocks tile_tiny_blocks(int dtype, int d, const PromptTab &tab, int LH)
{
    int shortest = 8;
    for (int p = 0; p < tab.n; ++p)
        if (tab.blk_off[p + 1] - tab.blk_off[p] > resident_tile_workgroups()) shortest = min(shortest, (int)tab.b[p]);
    if (shortest == 8) return kTinyNone;
    if (dtype != NKV_DTYPE_F8_E4M3) return kTinyGeneric;
    return shortest > 1 && d == 128 && (int64_t)LH * tab.blk_off[tab.n] > 65536 ? kTinyVector : kTinyNone;
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
                        defer_all ? -1 : kPollLimit, longest_unit(tab) > 256, prof, st};
    if (dtype == NKV_DTYPE_F16) go.run_format<kKeyF16>();
    else if (dtype == NKV_DTYPE_F8_E4M3) go.run_format<kKeyF8>();
    else go.run_format<kKeyBF16>();
    return hipGetLastError();
}

}  // namespace nkv
