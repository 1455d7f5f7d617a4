// Exact selection among a few hundred keys by a single wavefront (gfx950, 64 lanes).
#pragma once

#include "nkv_device.h"

namespace nkv {

// The digit that holds rank `want` (1-based) from the top of a 256-digit histogram, and how many entries lie above it.
__device__ __forceinline__ void wave_pick_digit(const uint32_t *hist, uint32_t want, uint32_t &dig, uint32_t &below)
{
    // lane owns digits 4 lane .. 4 lane + 3; running count from the top
    const int lane = threadIdx.x & 63;
    const uint32_t c0 = hist[lane * 4], c1 = hist[lane * 4 + 1], c2 = hist[lane * 4 + 2], c3 = hist[lane * 4 + 3];
    const uint32_t group = c0 + c1 + c2 + c3;
    const uint32_t incl = wave_suffix_sum(group);
    const uint32_t cum = incl - group;
    dig = below = 0u;
    const bool mine = cum < want && want <= incl;
    if (mine) {
        if (want <= cum + c3) { dig = lane * 4 + 3; below = cum; }
        else if (want <= cum + c3 + c2) { dig = lane * 4 + 2; below = cum + c3; }
        else if (want <= cum + c3 + c2 + c1) { dig = lane * 4 + 1; below = cum + c3 + c2; }
        else { dig = lane * 4; below = cum + c3 + c2 + c1; }
    }
    const unsigned long long who = __ballot(mine);
    const int src = __ffsll((long long)who) - 1;
    dig = (uint32_t)__builtin_amdgcn_readlane((int)dig, src);
    below = (uint32_t)__builtin_amdgcn_readlane((int)below, src);
}

// `want`-th largest (1-based) of the n keys key_at(0..n-1): radix select by one wavefront, eight bits a pass, over the bits in
// which the keys differ (those of one bin of values share half of theirs or more); hist: 256 words of LDS owned by the wave.
// Returns the key; gt = how many keys are larger, eq = how many are equal.  (With always four passes and one to count, all else
// the same, the finishing kernel of the budgets of 8 heads x 32768 tokens takes 11.0 us instead of 9.4, that of the statistics 10.2
// instead of 9.2, mean of 36 layers x 8 heads x 32768 and 8 layers x 8 heads x 131 072.)
template <typename F>
__device__ __forceinline__ uint32_t wave_select_fn(int n, uint32_t want, uint32_t *hist, uint32_t &gt, uint32_t &eq,
                                                   F key_at)
{
    const int lane = threadIdx.x & 63;
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (int i = lane; i < n; i += 64) {
        const uint32_t k = key_at(i);
        lo = min(lo, k);
        hi = max(hi, k);
    }
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_reduce(lo, [](uint32_t a, uint32_t b) { return min(a, b); }));
    hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_reduce(hi, [](uint32_t a, uint32_t b) { return max(a, b); }));
    gt = 0u;
    eq = (uint32_t)n;
    int bits = 32 - __clz((int)(lo ^ hi));                           // low bits still open; the keys looked at share the others
    uint32_t prefix = bits == 32 ? 0u : hi >> bits << bits;
    while (bits > 0) {
        const int shift = max(bits - 8, 0);
        for (int j = lane; j < 256; j += 64) hist[j] = 0u;
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < n; i += 64) {
            const uint32_t k = key_at(i);
            if (bits == 32 || k >> bits == prefix >> bits) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t dig, below;
        wave_pick_digit(hist, want, dig, below);
        want -= below;
        gt += below;
        prefix |= dig << shift;
        eq = hist[dig];
        bits = shift;
        __builtin_amdgcn_wave_barrier();
    }
    return prefix;
}

// The same for n <= 64 keys, one per lane (lanes from n on are ignored): every lane ranks its key against all others.
__device__ __forceinline__ uint32_t wave_select_64(uint32_t mine, int n, uint32_t want, uint32_t &gt, uint32_t &eq)
{
    uint32_t beyond = 0u, equal = 0u;
    for (int i = 0; i < n; ++i) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
        beyond += other > mine ? 1u : 0u;
        equal += other == mine ? 1u : 0u;
    }
    const bool it = (int)(threadIdx.x & 63) < n && beyond < want && want <= beyond + equal;   // lanes of equal keys
    const int src = __ffsll((long long)__ballot(it)) - 1;
    gt = (uint32_t)__builtin_amdgcn_readlane((int)beyond, src);
    eq = (uint32_t)__builtin_amdgcn_readlane((int)equal, src);
    return (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
}

// The same over an array (LDS or memory).
__device__ __forceinline__ uint32_t wave_select(const uint32_t *key, int n, uint32_t want, uint32_t *hist,
                                                uint32_t &gt, uint32_t &eq)
{
    if (n <= 64) return wave_select_64((int)(threadIdx.x & 63) < n ? key[threadIdx.x & 63] : 0u, n, want, gt, eq);
    return wave_select_fn(n, want, hist, gt, eq, [key](int i) { return key[i]; });
}

}  // namespace nkv
