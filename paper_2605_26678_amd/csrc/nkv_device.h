// Device-side helpers shared by the libnkv kernels (gfx950, 64-wide wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nkv_internal.h"

namespace nkv {

constexpr int kWave = 64;

// Order-preserving map float -> uint32 (larger float <=> larger key); -0 and +0 share a key.
__device__ __forceinline__ uint32_t ord_key(float x)
{
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_value(uint32_t k)
{
    uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Element types that share a storage width are told apart by these wrappers.
struct f16_t { uint16_t bits; };
struct f8e4m3_t { uint8_t bits; };

// OCP 8-bit float, 4 exponent bits (bias 7), 3 mantissa bits, no infinities, S.1111.111 = NaN.
__device__ __forceinline__ float f8e4m3_to_f32(uint8_t v)
{
    const uint32_t e = (v >> 3) & 15u, m = v & 7u;
    uint32_t mag;
    if (e == 0u) mag = __float_as_uint((float)m * 0.001953125f);            // subnormal: m * 2^-9
    else if (e == 15u && m == 7u) mag = 0x7fc00000u;
    else mag = ((e + 120u) << 23) | (m << 20);
    return __uint_as_float(mag | ((uint32_t)(v & 0x80u) << 24));
}

template <typename T> __device__ __forceinline__ float load_elem(const T *p);
template <> __device__ __forceinline__ float load_elem<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float load_elem<uint16_t>(const uint16_t *p) { return bf16_to_f32(*p); }
template <> __device__ __forceinline__ float load_elem<f16_t>(const f16_t *p)
{
    return (float)*reinterpret_cast<const _Float16 *>(p);
}
template <> __device__ __forceinline__ float load_elem<f8e4m3_t>(const f8e4m3_t *p) { return f8e4m3_to_f32(p->bits); }

// Prompt that owns global token row t (0 <= t < tab.T).
__device__ __forceinline__ int prompt_of_token(const PromptTab &tab, int t)
{
    int p = 0;
    while (p + 1 < tab.n && t >= tab.tok_off[p + 1]) ++p;
    return p;
}

// Prompt that owns per-head block index blk (0 <= blk < tab.blk_off[tab.n]).
__device__ __forceinline__ int prompt_of_block(const PromptTab &tab, int blk)
{
    int p = 0;
    while (p + 1 < tab.n && blk >= tab.blk_off[p + 1]) ++p;
    return p;
}

// ---- reductions and scans over a whole wavefront: cross-lane data paths of the vector unit only (DPP inside rows of 16
// lanes, permlane swaps between them), which answer in a few cycles where a shuffle through the LDS crossbar takes a
// hundred.  All 64 lanes must be active. ----
template <int CTRL> __device__ __forceinline__ uint32_t dpp_word(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
// the value of the lane that CTRL pairs this lane with, for 4- and 8-byte types
template <int CTRL, typename T> __device__ __forceinline__ T dpp_partner(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "4- or 8-byte types");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp_word<CTRL>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        return __builtin_bit_cast(T, (unsigned long long)dpp_word<CTRL>((uint32_t)(u >> 32)) << 32 | dpp_word<CTRL>((uint32_t)u));
    }
}
// op over the lanes that differ in bit 4 (ROWS = 16) or bit 5 (ROWS = 32) of the lane index
template <int ROWS, typename T, typename Op> __device__ __forceinline__ T swap_reduce(T v, Op op)
{
    auto swap = [](uint32_t u, uint32_t &x, uint32_t &y) {
        if constexpr (ROWS == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
            x = r[0];
            y = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
            x = r[0];
            y = r[1];
        }
    };
    uint32_t x, y;
    if constexpr (sizeof(T) == 4) {
        swap(__builtin_bit_cast(uint32_t, v), x, y);
        return op(__builtin_bit_cast(T, x), __builtin_bit_cast(T, y));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        uint32_t xh, yh;
        swap((uint32_t)u, x, y);
        swap((uint32_t)(u >> 32), xh, yh);
        return op(__builtin_bit_cast(T, (unsigned long long)xh << 32 | x), __builtin_bit_cast(T, (unsigned long long)yh << 32 | y));
    }
}
// Two values whose lanes differ in that bit: lanes with the bit clear receive op over a's pair, the others op over b's.
template <int ROWS, typename T, typename Op> __device__ __forceinline__ T swap_merge(T a, T b, Op op)
{
    auto swap = [](uint32_t u, uint32_t v, uint32_t &x, uint32_t &y) {
        if constexpr (ROWS == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(u, v, false, false);
            x = r[0];
            y = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
            x = r[0];
            y = r[1];
        }
    };
    uint32_t x, y;
    if constexpr (sizeof(T) == 4) {
        swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), x, y);
        return op(__builtin_bit_cast(T, x), __builtin_bit_cast(T, y));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, a), v = __builtin_bit_cast(unsigned long long, b);
        uint32_t xh, yh;
        swap((uint32_t)u, (uint32_t)v, x, y);
        swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), xh, yh);
        return op(__builtin_bit_cast(T, (unsigned long long)xh << 32 | x), __builtin_bit_cast(T, (unsigned long long)yh << 32 | y));
    }
}
template <typename T, typename Op> __device__ __forceinline__ T row16_reduce(T v, Op op)     // over a row of 16 lanes
{
    v = op(v, dpp_partner<0xB1>(v));             // quad_perm [1,0,3,2]
    v = op(v, dpp_partner<0x4E>(v));             // quad_perm [2,3,0,1]
    v = op(v, dpp_partner<0x141>(v));            // row_half_mirror: the other quad of the 8-lane half
    return op(v, dpp_partner<0x140>(v));         // row_mirror: the other half of the 16-lane row
}
template <typename T, typename Op> __device__ __forceinline__ T wave_reduce(T v, Op op)
{
    v = row16_reduce(v, op);
    v = swap_reduce<16>(v, op);
    return swap_reduce<32>(v, op);
}
template <typename T> __device__ __forceinline__ T wave_sum(T v)
{
    return wave_reduce(v, [](T a, T b) { return a + b; });
}
// Eight values reduced at once: lanes 8 i .. 8 i + 7 receive value i's result.  The halves of the wavefront share the values out, then
// the rows of 16 lanes, then the halves of a row, so that there are 10 steps where eight reductions by themselves take 48.
template <typename T, typename Op> __device__ __forceinline__ T wave_reduce8(const T (&v)[8], Op op)
{
    T x[4], y[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = swap_merge<32>(v[e], v[e + 4], op);
#pragma unroll
    for (int e = 0; e < 2; ++e) y[e] = swap_merge<16>(x[e], x[e + 2], op);
    const bool hi = (threadIdx.x & 8) != 0;
    T r = op(hi ? y[1] : y[0], dpp_partner<0x128>(hi ? y[0] : y[1]));       // row_ror:8
    r = op(r, dpp_partner<0xB1>(r));
    r = op(r, dpp_partner<0x4E>(r));
    return op(r, dpp_partner<0x141>(r));
}
__device__ __forceinline__ float wave_min(float v)
{
    return wave_reduce(v, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ float wave_max(float v)
{
    return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}

// inclusive sum over the lanes up to / from this one
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);    // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);    // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);    // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);    // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_suffix_sum(uint32_t x)
{
    const uint32_t incl = wave_prefix_sum(x);
    return (uint32_t)__builtin_amdgcn_readlane((int)incl, 63) - incl + x;
}

// Adds the active lanes to their bins, those of the first lane's bin with one add: equal values would queue for one word,
// a few cycles each.
__device__ __forceinline__ void count_bin(uint32_t *hist, int bin)
{
    const unsigned long long same = __ballot(bin == __builtin_amdgcn_readfirstlane(bin));
    const bool mine = (same >> (threadIdx.x & 63)) & 1ull;
    const bool first = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) == 0u;
    if (!mine || first) atomicAdd(&hist[bin], mine ? (uint32_t)__popcll(same) : 1u);
}

// The largest u in [0, n) with off(u) <= x, for ascending off(0 .. n - 1) with off(0) <= x: a whole wavefront narrows the
// range to a 64th with every step, so 4096 entries take two load latencies where a binary search takes twelve.
template <typename T, typename F> __device__ __forceinline__ int wave_search_fn(int n, T x, F off)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0;
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave, at = lane * step;
        const unsigned long long le = __ballot(at < n && off(lo + min(at, n - 1)) <= x);   // a prefix of the lanes, never empty
        const int k = 63 - __builtin_clzll(le);
        lo += k * step;
        n = min(step, n - k * step);
    }
    return lo;
}
template <typename T> __device__ __forceinline__ int wave_search(const T *__restrict__ off, int n, T x)
{
    return wave_search_fn(n, x, [off](int i) { return off[i]; });
}

// Block-wide reductions for blockDim.x a multiple of 64 and <= 1024.  `scratch` holds >= 16 elements.
// Every thread receives the result; contains two barriers.
template <typename T> __device__ __forceinline__ T block_sum(T v, T *scratch)
{
    v = wave_sum(v);
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) scratch[w] = v;
    __syncthreads();
    T r = scratch[0];
    for (int i = 1; i < nw; ++i) r += scratch[i];
    return r;
}
__device__ __forceinline__ float block_min(float v, float *scratch)
{
    v = wave_min(v);
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) scratch[w] = v;
    __syncthreads();
    float r = scratch[0];
    for (int i = 1; i < nw; ++i) r = fminf(r, scratch[i]);
    return r;
}
__device__ __forceinline__ float block_max(float v, float *scratch)
{
    v = wave_max(v);
    const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) scratch[w] = v;
    __syncthreads();
    float r = scratch[0];
    for (int i = 1; i < nw; ++i) r = fmaxf(r, scratch[i]);
    return r;
}

// One digit step of a most-significant-digit-first radix select over 256-bin histograms.
// hist: counts of the current digit among candidates.  top != 0: walk from bin 255 down, else from 0 up,
// until the running count reaches `want` (1-based rank among the candidates).  Returns the digit and
// reduces `want` by the candidates passed over.  Serial; called by one thread per select.
__device__ __forceinline__ uint32_t radix_pick(const uint32_t *hist, uint32_t &want, int top)
{
    uint32_t cum = 0;
    if (top) {
        for (int b = 255; b > 0; --b) {
            uint32_t c = hist[b];
            if (cum + c >= want) { want -= cum; return (uint32_t)b; }
            cum += c;
        }
        want -= cum;
        return 0u;
    }
    for (int b = 0; b < 255; ++b) {
        uint32_t c = hist[b];
        if (cum + c >= want) { want -= cum; return (uint32_t)b; }
        cum += c;
    }
    want -= cum;
    return 255u;
}

}  // namespace nkv
