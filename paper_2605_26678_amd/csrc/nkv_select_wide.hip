// Top-B_h selection with ordered compaction (paper Section 2.5) spread over the whole chip: same kept_idx as
// select_fast_kernel / select_kernel of nkv_select.hip, but a head's scores are cut into slices of 8192 tokens
// and every step that touches them runs on one small workgroup per slice (see nkv_slices.h).
//   slice_hist_kernel   (per slice)  2048-bin value histogram of the slice
//   sel_collect_kernel  (per slice)  the bin that holds the unit's B_h-th best score (found by every slice's workgroup
//                                    from the unit's histograms); how many of the slice's scores lie in bins above
//                                    it; the keys of that bin -> the slice's segment.  The first workgroup also places
//                                    all units in the output
//   sel_compact_kernel  (per slice)  the exact threshold T inside the bin, how many of the scores tied at T are kept and
//                                    how many kept / tied scores precede the slice, found by one wavefront of every
//                                    slice's workgroup from the unit's segments (a few dozen keys: cheaper than a
//                                    kernel of its own in between); then ballots over 64 consecutive tokens + a scan
//                                    over the slice's groups give every kept token its output row; optional count of
//                                    near-threshold scores
// If a segment overflows (thousands of equal scores in one bin), the slice's workgroup walks the head's scores itself.
#include "nkv_slices.h"

namespace nkv {
namespace {

constexpr int kList = 2048;              // keys of a unit's boundary bin that fit the list

struct SelPick {
    int32_t bT;                          // boundary bin; -1: everything is kept; kBins: nothing is kept
    uint32_t needT;                      // how many entries of the boundary bin are kept
};

struct SelSlice {
    uint32_t above;                      // scores of the slice in bins above the boundary bin
    uint32_t n;                          // keys in the slice's segment
};

// The boundary bin of unit u: the bin that holds its B-th best score, and how many of that bin's entries are kept
// (B = 0: {kBins, 0}, nothing is kept; B = N: {-1, 0}, everything is).  Called by all threads of a workgroup,
// the first 256 of which own 8 bins each; c_own[i] receives the count of bin 8 tid + i in slice `own` of the unit (own < 0: not asked for).
// wtot: 4 words, s_pick: 2 words of LDS; the result is valid for every thread after the call.
__device__ __forceinline__ SelPick pick_boundary_bin(const uint16_t *__restrict__ part, int64_t slice0, int S, int B, int N, int own,
                                                     uint32_t (&c_own)[8], uint32_t *wtot, int32_t *s_pick)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint4 *rows = reinterpret_cast<const uint4 *>(part + slice0 * kBins);
    uint32_t c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { c[i] = 0u; c_own[i] = 0u; }
    for (int s0 = 0; s0 < S && tid < kBins / 8; s0 += 4) {
        uint4 r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = rows[(int64_t)min(s0 + i, S - 1) * (kBins / 8) + tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s0 + i < S) {
                const uint32_t t[8] = {r[i].x & 0xffffu, r[i].x >> 16, r[i].y & 0xffffu, r[i].y >> 16,
                                       r[i].z & 0xffffu, r[i].z >> 16, r[i].w & 0xffffu, r[i].w >> 16};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    c[e] += t[e];
                    if (s0 + i == own) c_own[e] = t[e];
                }
            }
        }
    }
    if (B == 0 || B == N) return SelPick{B == 0 ? kBins : -1, 0u};  // no threshold to find (uniform in the workgroup)
    uint32_t group = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) group += c[i];
    uint32_t incl = wave_suffix_sum(group);                                           // inclusive sum from the top bin downwards
    if (lane == 0 && w < 4) wtot[w] = incl;
    __syncthreads();
    for (int ww = w + 1; ww < 4; ++ww) incl += wtot[ww];
    const uint32_t want = (uint32_t)B;
    uint32_t cum = incl - group;                                     // scores in bins above this thread's eight
    if (cum < want && want <= incl && tid < kBins / 8) {
#pragma unroll
        for (int i = 7; i >= 0; --i) {
            if (cum < want && want <= cum + c[i]) { s_pick[0] = tid * 8 + i; s_pick[1] = (int32_t)(want - cum); }
            cum += c[i];
        }
    }
    __syncthreads();
    return SelPick{s_pick[0], (uint32_t)s_pick[1]};
}

// head_off of all units, from their budgets, by one workgroup of TH threads.
template <int TH>
__device__ __forceinline__ void place_units(const int32_t *__restrict__ k_per_head, int LH, const PromptTab &tab, int64_t *__restrict__ head_off)
{
    constexpr int NW = TH / 64;
    __shared__ unsigned long long wave_rows[NW];
    const int n = tab.n * LH, per = (n + TH - 1) / TH, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int u0 = min(tid * per, n), u1 = min(u0 + per, n);
    auto rows = [&](int u) {
        const int p = u / LH;
        return (unsigned long long)min(max(k_per_head[u], 0), tab.tok_off[p + 1] - tab.tok_off[p]);
    };
    unsigned long long mine = 0ull;
    for (int u = u0; u < u1; ++u) mine += rows(u);
    unsigned long long incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wave_rows[w] = incl;
    __syncthreads();
    unsigned long long run = incl - mine;
    for (int i = 0; i < w; ++i) run += wave_rows[i];
    for (int u = u0; u < u1; ++u) {
        head_off[u] = (int64_t)run;
        run += rows(u);
    }
    if (tid == TH - 1) head_off[n] = (int64_t)run;
}

// grid: slices.  Every slice's workgroup finds the boundary bin of its unit itself from the unit's slice histograms
// (a few 4 KB rows that the histogram kernel has just written: cheaper than a kernel of its own in between), counts
// its own slice's scores above that bin, and copies its scores of that bin into its segment.  The first slice's
// workgroup records the unit's pick.  place: head_off is not filled yet, the first workgroup of all does it.  (Where every
// workgroup of the compaction added up the budgets in front of its unit, that kernel took 51.3 us instead of 49.7 for 1792
// units in 3584 slices.)
template <int TH>
__global__ __launch_bounds__(TH) void sel_collect_kernel(const float *__restrict__ scores,
                                                                   const int32_t *__restrict__ k_per_head, int L, int H,
                                                                   PromptTab tab, SliceTab st,
                                                                   const uint16_t *__restrict__ part,
                                                                   SelPick *__restrict__ picks,
                                                                   uint32_t *__restrict__ seg,
                                                                   SelSlice *__restrict__ ss,
                                                                   int64_t *__restrict__ near_count, bool place,
                                                                   int64_t *__restrict__ head_off)
{
    constexpr int PT = per_thread<TH>();
    __shared__ uint32_t n_hit;
    __shared__ uint32_t wtot[4];
    __shared__ int32_t s_pick[2];
    int p, lh, s, S;
    locate(st, tab, blockIdx.x, p, lh, s, S);
    const int u = p * L * H + lh;
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const float *sc = scores + (int64_t)lh * tab.T + tab.tok_off[p];
    const int tid = threadIdx.x;
    float v[PT];
    const __amdgpu_buffer_rsrc_t vals = slice_values(sc, s, N);
#pragma unroll
    for (int j = 0; j < PT; ++j) v[j] = slice_value<TH>(vals, tid, j);
    if (place && blockIdx.x == 0) place_units<TH>(k_per_head, L * H, tab, head_off);
    uint32_t c_own[8];
    const SelPick pk = pick_boundary_bin(part, blockIdx.x - s, S, min(max(k_per_head[u], 0), N), N, s, c_own, wtot, s_pick);
    const int bT = pk.bT;
    {                                                                // this slice's scores in bins above bT
        uint32_t a = 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) a += tid * 8 + i > bT ? c_own[i] : 0u;
        a = wave_sum(a);
        __syncthreads();                                             // (wtot is free again)
        if ((tid & 63) == 0 && tid < 256) wtot[tid >> 6] = a;
    }
    if (tid == 0) {
        n_hit = 0u;
        if (blockIdx.x == 0 && near_count) *near_count = 0;          // the compaction kernel, next on the stream, adds to it
    }
    __syncthreads();
    if (tid == 0) {
        ss[blockIdx.x].above = (wtot[0] + wtot[1]) + (wtot[2] + wtot[3]);
        if (s == 0) picks[u] = pk;
    }
    uint32_t *out = seg + (int64_t)blockIdx.x * kSeg;
    auto take = [&](float x) {
        const uint32_t at = atomicAdd(&n_hit, 1u);
        if (at < (uint32_t)kSeg) out[at] = ord_key(x);
    };
    if (bT > 0 && bT < kBins - 2) {                                  // score_bin's inner bins: a range of the scaled value
        const float from = (float)bT, to = (float)(bT + 1);          // (not met by the zeros past the head's end; 3584 slices: 28.0 -> 25.2 us)
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const float x = v[j] * 2046.0f;
            if (x >= from && x < to) take(v[j]);
        }
    } else if (bT >= 0 && bT < kBins) {
#pragma unroll
        for (int j = 0; j < PT; ++j)
            if (s * kSlice + j * TH + tid < N && score_bin(v[j]) == bT) take(v[j]);
    }
    __syncthreads();
    if (tid == 0) ss[blockIdx.x].n = n_hit;                          // more than kSeg: the compaction sees it and walks the scores
}

// set bits of m in the lanes below this one
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// More scores in one bin than the lists hold (thousands of equal scores): the slice's whole workgroup walks the head's N scores
// itself, four times for the threshold's digits and once to count -- slow, exact, and rare.  B: scores kept, 0 < B < N; begin:
// the slice's first token.  found: as in sel_compact_kernel.  (By a single wavefront of every slice, as a unit's one
// wavefront did before: 8 heads x 131 072 scores of 17 values 2006 us and 1800; this 190.)
template <int TH>
__device__ __forceinline__ void walk_head(const float *__restrict__ sc, int N, uint32_t B, int begin, uint32_t *hist, uint32_t *found)
{
    constexpr int U = 8;
    const int tid = threadIdx.x;
    auto for_keys = [&](int n, auto f) {                              // f(key, counts): the keys of [0, n), U loads in flight
        for (int i0 = 0; i0 < n; i0 += U * TH) {
            float x[U];
#pragma unroll
            for (int j = 0; j < U; ++j) x[j] = sc[min(i0 + j * TH + tid, n - 1)];
#pragma unroll
            for (int j = 0; j < U; ++j) f(ord_key(x[j]), i0 + j * TH + tid);
        }
    };
    uint32_t want = B, T = 0u;
    for (int shift = 24; shift >= 0; shift -= 8) {
        __syncthreads();                                             // (found and hist have been read)
        for (int j = tid; j < 256; j += TH) hist[j] = 0u;
        __syncthreads();
        for_keys(N, [&](uint32_t key, int i) {
            if (i < N && (shift == 24 || (key >> (shift + 8)) == (T >> (shift + 8)))) count_bin(hist, (int)((key >> shift) & 255u));
        });
        __syncthreads();
        if (tid < 64) {
            uint32_t dig, below;
            wave_pick_digit(hist, want, dig, below);
            if (tid == 0) { found[0] = dig; found[1] = below; }
        }
        __syncthreads();
        T |= found[0] << shift;
        want -= found[1];
    }
    __syncthreads();
    if (tid == 0) { found[0] = T; found[1] = want; found[2] = found[3] = 0u; }     // (what is left of B is kept of the tied ones)
    __syncthreads();
    uint32_t g = 0u, e = 0u;
    for_keys(begin, [&](uint32_t key, int i) {
        g += i < begin && key > T ? 1u : 0u;
        e += i < begin && key == T ? 1u : 0u;
    });
    g = wave_sum(g);
    e = wave_sum(e);
    if ((tid & 63) == 0) {
        atomicAdd(&found[2], g);
        atomicAdd(&found[3], e);
    }
    __syncthreads();
}

// grid: slices
template <int TH>
__global__ __launch_bounds__(TH) void sel_compact_kernel(const float *__restrict__ scores, const int32_t *__restrict__ k_per_head,
                                                         int L, int H, PromptTab tab, SliceTab st, const SelPick *__restrict__ picks,
                                                         const uint32_t *__restrict__ seg, const SelSlice *__restrict__ ss,
                                                         const int64_t *__restrict__ head_off, int64_t row_capacity, float near_tol,
                                                         int32_t *__restrict__ kept_idx, int64_t *__restrict__ near_count)
{
    constexpr int PT = per_thread<TH>(), NW = TH / 64;
    constexpr int kGroups = kSlice / 64;                             // 64-token groups of a slice, in token order
    __shared__ uint32_t cnt_gt[kGroups], cnt_eq[kGroups];
    __shared__ unsigned long long near_acc[NW];
    __shared__ uint32_t keys[kList];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t found[6];                                    // T, rem, kept-for-sure / tied scores of the unit before this slice; walk; plain
    int p, lh, s, S;
    locate(st, tab, blockIdx.x, p, lh, s, S);
    const int u = p * L * H + lh;
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const float *sc = scores + (int64_t)lh * tab.T + tab.tok_off[p];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float v[PT];
    const __amdgpu_buffer_rsrc_t vals = slice_values(sc, s, N);
#pragma unroll
    for (int j = 0; j < PT; ++j) v[j] = slice_value<TH>(vals, tid, j);
    const SelPick pk = picks[u];
    const bool all = pk.bT < 0, none = pk.bT >= kBins;
    const int64_t out0 = head_off[u];
    if (none) return;                                                // nothing kept
    if (w == 0) {
        const SelSlice *unit_ss = ss + (blockIdx.x - s);
        const uint32_t *unit_seg = seg + (int64_t)(blockIdx.x - s) * kSeg;
        uint32_t T = 0u, rem = 0u, gt_before = 0u, eq_before = 0u;
        bool walk = false, plain = false;
        for (int q = lane; q < s; q += 64) gt_before += unit_ss[q].above;
        gt_before = wave_sum(gt_before);
        if (!all) {
            int mine;                                                // where this slice's keys start in the list
            const int n = gather_segments(unit_seg, S, [&](int q) { return unit_ss[q].n; }, keys, kList, s, mine);
            __builtin_amdgcn_wave_barrier();
            uint32_t gt, eq;
            if (n >= 0) {
                T = wave_select(keys, n, pk.needT, hist, gt, eq);
                rem = pk.needT - gt;
                plain = rem == eq && T > 0x80000000u;                // no tie is cut, and T is above both zeros
                uint32_t g = 0u, e = 0u;
                for (int i = lane; i < mine; i += 64) {
                    g += keys[i] > T ? 1u : 0u;
                    e += keys[i] == T ? 1u : 0u;
                }
                gt_before += wave_sum(g);
                eq_before = wave_sum(e);
            } else {
                walk = true;
            }
        }
        if (lane == 0) { found[0] = T; found[1] = rem; found[2] = gt_before; found[3] = eq_before; found[4] = walk; found[5] = plain; }
    }
    __syncthreads();
    // Every tied score is kept and T is positive, as nearly always: a score is kept iff its bits, as an integer, are not below
    // T's, and the zeros past the head's end are not kept.  The wave's 64-token groups become 64-bit masks, group j's in lane j,
    // whose bits are counted for all groups at once; the stores go through a descriptor that ends at row_capacity.
    // Against the two kinds of kept scores below, 3584 slices: 50.0 us, now 40.3; 1152: 27.2 and 20.3; 32: 10.0 and 8.3.  (It
    // then waits: registers for seven or eight workgroups a compute unit instead of six, a few of them spilled: 43.5 and 44.6.)
    if (__builtin_amdgcn_readfirstlane(found[5]) != 0u) {
        const int ti = __builtin_amdgcn_readfirstlane(found[0]) ^ (int)0x80000000u;
        const float tv = __int_as_float(ti);
        if (near_count && s * kSlice + kSlice > N) {                 // nor are they near it
#pragma unroll
            for (int j = 0; j < PT; ++j) v[j] = s * kSlice + j * TH + tid < N ? v[j] : __uint_as_float(0xffc00000u);
        }
        int lo = 0, hi = 0, near = 0;
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const unsigned long long m = __ballot(__float_as_int(v[j]) >= ti);
            lo = lane == j ? (int)(uint32_t)m : lo;
            hi = lane == j ? (int)(uint32_t)(m >> 32) : hi;
            if (near_count) near += __popcll(__ballot(fabsf(v[j] - tv) <= near_tol));
        }
        if (lane < PT) cnt_gt[lane * NW + w] = (uint32_t)(__popc((uint32_t)lo) + __popc((uint32_t)hi));
        if (lane == 0) near_acc[w] = (unsigned long long)near;
        __syncthreads();
        static_assert(kGroups == 128, "two groups a lane");
        if (w == 0) {                                                // exclusive scan over the groups, in token order
            const uint32_t g0 = cnt_gt[2 * lane], g1 = cnt_gt[2 * lane + 1], before = wave_prefix_sum(g0 + g1) - g0 - g1;
            cnt_gt[2 * lane] = before;
            cnt_gt[2 * lane + 1] = before + g0;
            if (near_count && lane == 0) {
                unsigned long long t = 0;
                for (int i = 0; i < NW; ++i) t += near_acc[i];
                if (t) atomicAdd((unsigned long long *)near_count, t);
            }
        }
        __syncthreads();
        const int base = lane < PT ? (int)cnt_gt[lane * NW + w] : 0;
        const int64_t first = out0 + __builtin_amdgcn_readfirstlane(found[2]) + __builtin_amdgcn_readfirstlane(found[3]);
        const int64_t room = row_capacity - first;
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(kept_idx + first, 0, room > 0 ? (int)(room < kSlice ? room : kSlice) * 4 : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const uint32_t mlo = (uint32_t)__builtin_amdgcn_readlane(lo, j), mhi = (uint32_t)__builtin_amdgcn_readlane(hi, j);
            const int row = __builtin_amdgcn_readlane(base, j) + (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
            if (__builtin_amdgcn_inverse_ballot_w64((unsigned long long)mhi << 32 | mlo))
                __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(s * kSlice + j * TH + tid), rows, 4 * row, 0, 0);
        }
        return;
    }
    if (found[4]) walk_head<TH>(sc, N, (uint32_t)min(max(k_per_head[u], 0), N), s * kSlice, hist, found);
    const uint32_t T = found[0], rem = found[1], unit_gt = found[2], unit_eq = found[3];
    // population of every 64-token group (chunk j, wave w) = tokens s*kSlice + j*TH + w*64 ...
    uint32_t near = 0u;
    const float tv = key_value(T);
    uint32_t gmask = 0u, emask = 0u;                                 // bit j: slot j is kept for sure / is tied at T
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const bool in = s * kSlice + j * TH + tid < N;
        const uint32_t key = ord_key(v[j]);
        const bool gt = in && (all || key > T);
        const bool eq = in && !all && key == T;
        gmask |= (gt ? 1u : 0u) << j;
        emask |= (eq ? 1u : 0u) << j;
        const unsigned long long mg = __ballot(gt), me = __ballot(eq);
        if (lane == 0) {
            cnt_gt[j * NW + w] = (uint32_t)__popcll(mg);
            cnt_eq[j * NW + w] = (uint32_t)__popcll(me);
        }
        if (near_count && in && !all && fabsf(v[j] - tv) <= near_tol) ++near;
        // one group at a time, its flags folded into the words right away: a condition kept for later is two scalar
        // registers, and 128 of them do not fit
        asm volatile("" : "+v"(gmask), "+v"(emask), "+v"(near));
    }
    __syncthreads();
    if (w == 0) {                                                    // exclusive scan over the groups: 2 per lane
        constexpr int PER = kGroups / 64;
        uint32_t g[PER], e[PER], tg = 0u, te = 0u;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            g[q] = cnt_gt[lane * PER + q];
            e[q] = cnt_eq[lane * PER + q];
            tg += g[q];
            te += e[q];
        }
        uint32_t rg = wave_prefix_sum(tg) - tg, re = wave_prefix_sum(te) - te;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            cnt_gt[lane * PER + q] = rg;
            cnt_eq[lane * PER + q] = re;
            rg += g[q];
            re += e[q];
        }
    }
    __syncthreads();
    // The two flag words are all the second pass needs of the values (and the compiler is kept from carrying the
    // first pass's 64 ballots over instead, which costs it more registers than it has).
    asm volatile("" : "+v"(gmask), "+v"(emask));
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int i = s * kSlice + j * TH + tid;
        const bool gt = (gmask >> j) & 1u, eq = (emask >> j) & 1u;
        const unsigned long long mg = __ballot(gt), me = __ballot(eq);
        const int grp = j * NW + w;
        const uint32_t gt_before = unit_gt + cnt_gt[grp] + lanes_below(mg);
        const uint32_t eq_before = unit_eq + cnt_eq[grp] + lanes_below(me);
        if (gt || (eq && eq_before < rem)) {
            const int64_t row = out0 + gt_before + min(eq_before, rem);
            if (row < row_capacity) kept_idx[row] = i;
        }
    }
    if (near_count) {
        const unsigned long long near_w = wave_sum((unsigned long long)near);
        if (lane == 0) near_acc[w] = near_w;
        __syncthreads();
        if (tid == 0) {
            unsigned long long t = 0;
            for (int i = 0; i < NW; ++i) t += near_acc[i];
            if (t) atomicAdd((unsigned long long *)near_count, t);
        }
    }
}

struct WideWs {
    size_t part, picks, ss, seg, total;
};

WideWs wide_ws(int L, int H, const PromptTab &tab)
{
    SliceTab st;
    const size_t slices = (size_t)fill_slices(L, H, tab, &st), units = (size_t)tab.n * L * H;
    WideWs w;
    size_t off = 0;
    w.part = off;    off += align256(slices * kBins * sizeof(uint16_t));
    w.picks = off;   off += align256(units * sizeof(SelPick));
    w.ss = off;      off += align256(slices * sizeof(SelSlice));
    w.seg = off;     off += align256(slices * kSeg * sizeof(uint32_t));
    w.total = off;
    return w;
}

}  // namespace

size_t select_wide_ws_bytes(int L, int H, const PromptTab &tab) { return wide_ws(L, H, tab).total; }

// Enqueues the three kernels.  with_head_off: head_off is not on the stream yet and the second kernel fills it
// (select_wide_places_units() says when it can: one workgroup reads all units' budgets).
bool select_wide_places_units(int n_units) { return n_units <= 4096; }

hipError_t launch_select_wide(const float *scores, const int32_t *k_per_head, int L, int H, const PromptTab &tab,
                              float near_tol, int64_t *head_off, int64_t row_capacity, int32_t *kept_idx,
                              int64_t *near_count, bool with_head_off, void *ws, hipStream_t st)
{
    SliceTab stab;
    const int slices = fill_slices(L, H, tab, &stab);
    const WideWs lay = wide_ws(L, H, tab);
    char *base = (char *)ws;
    uint16_t *part = (uint16_t *)(base + lay.part);
    SelPick *picks = (SelPick *)(base + lay.picks);
    SelSlice *ss = (SelSlice *)(base + lay.ss);
    uint32_t *seg = (uint32_t *)(base + lay.seg);
    const bool few = few_slices(slices);
    const unsigned threads = few ? 1024 : 256;
    (few ? slice_hist_kernel<1024> : slice_hist_kernel<256>)<<<(unsigned)slices, threads, 0, st>>>(scores, tab, stab, part);
    (few ? sel_collect_kernel<1024> : sel_collect_kernel<256>)<<<(unsigned)slices, threads, 0, st>>>(scores, k_per_head, L, H, tab,
                                                                                                   stab, part, picks, seg, ss, near_count,
                                                                                                   with_head_off, head_off);
    (few ? sel_compact_kernel<1024> : sel_compact_kernel<256>)<<<(unsigned)slices, threads, 0, st>>>(
        scores, k_per_head, L, H, tab, stab, picks, seg, ss, head_off, row_capacity, near_tol, kept_idx, near_count);
    return hipGetLastError();
}

}  // namespace nkv
