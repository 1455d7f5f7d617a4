// Per-head statistics of the three anomaly scales (paper Sections 2.3-2.4: min-max range, reliability gap =
// mean of the m_p largest minus mean of the m_p smallest normalised anomalies) spread over the whole chip.
//
// Same numbers as finalize_unit_kernel in nkv_finalize.hip (up to the order of floating-point additions), but a
// head's anomalies are not held by one workgroup: they are cut into slices of 8192 tokens and every step
// that touches them runs on one small workgroup per (slice, scale).
//
// Anomalies are -cos, so they lie in [-1, 1]; they are binned by value, bin(a) = floor(1023.5 (a + 1)), a
// monotone map.  "The m largest" is then: all bins above a boundary bin plus the largest few of the boundary
// bin's entries, and only those entries are looked at exactly; likewise from below.
//   stats_hist_kernel    (slice, scale)  2048-bin histogram as 16-bit counts; min and max of the slice
//   stats_pick_kernel    (unit, scale)   the bins that hold the m-th largest and the m-th smallest value
//   stats_collect_kernel (quarter of a slice) all three scales: sums of the values above the upper / below the lower
//                                        boundary bin; the boundary bins' entries (as order-preserving keys)
//                                        into two short lists per slice and scale; and, the ranges being known,
//                                        min / max / sum of the slice's surprise statistic
//   stats_finish_kernel  (unit, scale)   two wavefronts, one per boundary bin: exact thresholds inside the bins, the
//                                        two means, min, 1/range, gap
//   route_slice_kernel   (quarter)       weights, surprise statistics of the head, routed scores, pinning
// A list that overflows (hundreds of values of one slice in one bin) marks the (unit, scale), and the first wavefront of its
// finishing workgroup walks the head's values itself.
#include "nkv_learner.h"
#include "nkv_slices.h"

namespace nkv {
namespace {

constexpr int kList = 1024;              // keys the finishing wavefront takes per list

struct StatPick {
    int32_t bTop, bBot;                  // boundary bins
    uint32_t needTop, needBot;           // how many of their entries belong to the m largest / smallest
    float lo, inv;                       // min of the (unit, scale) and 1 / range (0 if flat)
};

struct SliceSurprise {                   // the surprise statistic (Section 2.4) over one slice
    float lo, hi;
    double sum;
};

struct SlicePart {                       // what one slice contributes besides its histogram and lists
    float lo, hi;                        // min, max of the slice
    uint32_t nTop, nBot;                 // entries in the two lists
    double sTop, sBot;                   // sums above the upper / below the lower boundary bin
};

__device__ __forceinline__ double rounded_sum(float x)               // to a multiple of 2^-40
{
    constexpr double kRound = 6144.;                                 // 1.5 * 2^12: the last place of a sum with it is 2^-40
    return ((double)x + kRound) - kRound;
}

constexpr int kQuarter = kSlice / 4;

// grid (slices, 3)
template <int TH>
__global__ __launch_bounds__(TH) void stats_hist_kernel(const float *__restrict__ a_raw, int64_t rows,
                                                                  PromptTab tab, SliceTab st, int n_slices,
                                                                  uint16_t *__restrict__ part,
                                                                  SlicePart *__restrict__ sp,
                                                                  SliceSurprise *__restrict__ sur)
{
    constexpr int PT = per_thread<TH>();
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins];
    __shared__ float red[2][TH / 64];
    int p, lh, s, S;
    locate(st, tab, blockIdx.x, p, lh, s, S);
    const int k = blockIdx.y;
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const float *a = a_raw + (int64_t)k * rows + (int64_t)lh * tab.T + tab.tok_off[p];
    const int tid = threadIdx.x;
    for (int j = tid; j < kBins; j += TH) hist[j] = 0u;
    float v[PT / 4][4];
    const __amdgpu_buffer_rsrc_t vals = slice_values(a, s, N);
#pragma unroll
    for (int j = 0; j < PT / 4; ++j) slice_values4<TH>(vals, tid, j, v[j]);
    __syncthreads();
    float lo = INFINITY, hi = -INFINITY;
    auto count = [&](float x) {                                      // (medians of three: minimum and maximum in one instruction each)
        lo = __builtin_amdgcn_fmed3f(x, lo, -INFINITY);
        hi = __builtin_amdgcn_fmed3f(x, hi, INFINITY);
        atomicAdd(&hist[anomaly_bin(x)], 1u);
    };
    if ((s + 1) * kSlice <= N) {
#pragma unroll
        for (int j = 0; j < PT / 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) count(v[j][e]);
    } else {
#pragma unroll
        for (int j = 0; j < PT / 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (s * kSlice + 4 * (j * TH + tid) + e < N) count(v[j][e]);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) { red[0][tid >> 6] = lo; red[1][tid >> 6] = hi; }
    __syncthreads();
    const int64_t job_slice = (int64_t)k * n_slices + blockIdx.x;
    if (tid == 0) {
        for (int i = 1; i < TH / 64; ++i) { lo = fminf(lo, red[0][i]); hi = fmaxf(hi, red[1][i]); }
        sp[job_slice] = SlicePart{lo, hi, 0u, 0u, 0.0, 0.0};          // (the quarters of a slice add to the rest)
        if (k == 0) sur[blockIdx.x] = SliceSurprise{INFINITY, 0.f, 0.0};
    }
    store_hist16(hist, part + job_slice * kBins);
}

// grid (units, 3); 256 threads, 8 bins each
__global__ __launch_bounds__(256) void stats_pick_kernel(int L, int H, PromptTab tab, SliceTab st,
                                                                  int n_slices, const uint16_t *__restrict__ part,
                                                                  const SlicePart *__restrict__ sp,
                                                                  StatPick *__restrict__ picks,
                                                                  uint32_t *__restrict__ failed)
{
    __shared__ uint32_t wtot[256 / 64];
    const int u = blockIdx.x, k = blockIdx.y;
    const int lh = u % (L * H), p = u / (L * H);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const int S = (N + kSlice - 1) / kSlice;
    const uint32_t m = (uint32_t)min(tab.m_p[p], N);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint4 *rows = reinterpret_cast<const uint4 *>(part + ((int64_t)k * n_slices + st.off[p] + (int64_t)lh * S) * kBins);
    uint32_t c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = 0u;
    for (int s0 = 0; s0 < S; s0 += 4) {
        uint4 r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = rows[(int64_t)min(s0 + i, S - 1) * (kBins / 8) + tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s0 + i < S) {
                c[0] += r[i].x & 0xffffu; c[1] += r[i].x >> 16; c[2] += r[i].y & 0xffffu; c[3] += r[i].y >> 16;
                c[4] += r[i].z & 0xffffu; c[5] += r[i].z >> 16; c[6] += r[i].w & 0xffffu; c[7] += r[i].w >> 16;
            }
        }
    }
    uint32_t group = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) group += c[i];
    uint32_t incl = wave_prefix_sum(group);                                           // inclusive prefix from bin 0 upwards
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    for (int ww = 0; ww < w; ++ww) incl += wtot[ww];
    const uint32_t below = incl - group;                             // entries in bins below this thread's eight
    const uint32_t above = (uint32_t)N - incl;                       // entries in bins above them
    StatPick *out = picks + (int64_t)u * 3 + k;
    if (below < m && m <= incl) {                                    // the m-th smallest lies in one of my bins
        uint32_t cum = below;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (cum < m && m <= cum + c[i]) { out->bBot = tid * 8 + i; out->needBot = m - cum; }
            cum += c[i];
        }
    }
    if (above < m && m <= above + group) {                           // the m-th largest lies in one of my bins
        uint32_t cum = above;
#pragma unroll
        for (int i = 7; i >= 0; --i) {
            if (cum < m && m <= cum + c[i]) { out->bTop = tid * 8 + i; out->needTop = m - cum; }
            cum += c[i];
        }
    }
    if (w == 0) {                                                    // min, max over the unit's slices
        float lo = INFINITY, hi = -INFINITY;
        for (int s = lane; s < S; s += 64) {
            const SlicePart q = sp[(int64_t)k * n_slices + st.off[p] + (int64_t)lh * S + s];
            lo = fminf(lo, q.lo);
            hi = fmaxf(hi, q.hi);
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0) {
            const float range = hi - lo;
            out->lo = lo;
            out->inv = range < kFlat ? 0.f : 1.0f / range;
            failed[(int64_t)u * 3 + k] = 0u;
        }
    }
}

// grid: quarters of slices.  All three scales of 2048 tokens in one pass: what stats_finish_kernel needs of each scale, and -- the ranges
// being known -- min, max and sum of the surprise statistic.  Bound by instruction issue: values are compared with the boundary
// bins' edges instead of binned.  What a quarter finds is added to its slice's; the keys go to lists in LDS first and take their places in the
// slice's by one atomic a list.
// Sums: a thread's eight tokens, 256 apart, in 32 bits; their sums, rounded to 2^-40, add up exactly in 64 bits (fewer than 2^13 in
// all), across lanes and by atomics, so that they do not depend on the order.
// (By one workgroup a slice, of 1024 threads up to 512 slices and of 256, four such sums a thread, from there on, score calls of 8 heads x
// 32768 tokens: 1 layer 52.4 us, 50.4 this way; 4 layers 96.9 and 95.0; 17 312 and 304; 36 613 and 611; 8 layers of 131 072 8-bit keys 518 and 512.)
template <bool ALL>
__global__ __launch_bounds__(256) void stats_collect_kernel(const float *__restrict__ a_raw, int64_t rows, int L, int H,
                                                                    PromptTab tab, SliceTab st, int n_slices, int scale_mask,
                                                                    const StatPick *__restrict__ picks, uint32_t *__restrict__ segTop,
                                                                    uint32_t *__restrict__ segBot, SlicePart *__restrict__ sp,
                                                                    SliceSurprise *__restrict__ sur, uint32_t *__restrict__ failed)
{
    constexpr int EACH = kQuarter / 256, NW = 4;
    __shared__ uint32_t cnt[6], base[6], keys[6][kSeg];              // list 2 k: the upper boundary bin of scale k, 2 k + 1 the lower one
    __shared__ double red[8][NW];
    __shared__ float fred[2][NW];
    const int slice = blockIdx.x / 4, quarter = blockIdx.x & 3;
    int p, lh, s, S;
    locate(st, tab, slice, p, lh, s, S);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p], first = quarter * kQuarter;
    if (s * kSlice + first >= N) return;
    const float *a = a_raw + (int64_t)lh * tab.T + tab.tok_off[p];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t job0 = ((int64_t)p * L * H + lh) * 3;
    float v[3][EACH];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const __amdgpu_buffer_rsrc_t vals = slice_values(a + k * rows, s, N);
#pragma unroll
        for (int j = 0; j < EACH; ++j) v[k][j] = slice_value<256>(vals, first + tid, j);
    }
    BinEdges top[3], bot[3];
    HeadStats hs;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const StatPick pk = picks[job0 + k];
        top[k] = bin_edges(pk.bTop);
        bot[k] = bin_edges(pk.bBot);
        hs.lo[k] = pk.lo;
        hs.inv_range[k] = pk.inv;
    }
    if (tid < 6) cnt[tid] = 0u;
    __syncthreads();
    float part[7] = {}, smin = INFINITY, smax = 0.f;
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
        if (s * kSlice + first + j * 256 + tid >= N) continue;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float x = v[k][j], y = anomaly_scaled(x);
            const bool over = y >= top[k].above, under = y < bot[k].below;
            part[k] += over ? x : 0.f;
            part[3 + k] += under ? x : 0.f;
            const bool in[2] = {!over && y >= top[k].from, !under && y < bot[k].to};
            if (!in[0] && !in[1]) continue;
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (in[e]) {
                    const uint32_t at = atomicAdd(&cnt[2 * k + e], 1u);
                    if (at < (uint32_t)kSeg) keys[2 * k + e][at] = e == 0 ? ord_key(x) : ~ord_key(x);
                }
        }
        const float raw[3] = {v[0][j], v[1][j], v[2][j]};
        float at[3];
        normalised(raw, hs, at);
        const float sv = surprise_std<ALL>(at, scale_mask);
        smin = fminf(smin, sv);
        smax = fmaxf(smax, sv);
        part[6] += sv;
    }
    const double sums[8] = {rounded_sum(part[0]), rounded_sum(part[3]), rounded_sum(part[1]), rounded_sum(part[4]),
                            rounded_sum(part[2]), rounded_sum(part[5]), rounded_sum(part[6]), 0.0};
    const double total = wave_reduce8(sums, [](double x, double y) { return x + y; });
    if ((lane & 7) == 0) red[lane >> 3][w] = total;
    smin = wave_min(smin);
    smax = wave_max(smax);
    if (lane == 0) { fred[0][w] = smin; fred[1][w] = smax; }
    __syncthreads();
    if (tid < 6) {
        SlicePart *q = sp + (int64_t)(tid >> 1) * n_slices + slice;
        const uint32_t n = cnt[tid];
        base[tid] = atomicAdd(tid & 1 ? &q->nBot : &q->nTop, n);
        unsafeAtomicAdd(tid & 1 ? &q->sBot : &q->sTop, (red[tid][0] + red[tid][1]) + (red[tid][2] + red[tid][3]));
        if (base[tid] + n > (uint32_t)kSeg) failed[job0 + (tid >> 1)] = 1u;
    } else if (tid == 64) {
        unsafeAtomicAdd(&sur[slice].sum, (red[6][0] + red[6][1]) + (red[6][2] + red[6][3]));
        // (no deviation is negative, so the floats compare as integers)
        atomicMin((int *)&sur[slice].lo, __float_as_int(fminf(fminf(fred[0][0], fred[0][1]), fminf(fred[0][2], fred[0][3]))));
        atomicMax((int *)&sur[slice].hi, __float_as_int(fmaxf(fmaxf(fred[1][0], fred[1][1]), fmaxf(fred[1][2], fred[1][3]))));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        uint32_t *seg = (i & 1 ? segBot : segTop) + ((int64_t)(i >> 1) * n_slices + slice) * kSeg;
        if ((uint32_t)tid < min(cnt[i], (uint32_t)kSeg) && base[i] + tid < (uint32_t)kSeg) seg[base[i] + tid] = keys[i][tid];
    }
    static_assert(kSeg <= 256, "a key a thread");
}

// grid: quarters of slices.  Blend, gate, route and pinning of the slice's tokens (Section 2.4); every workgroup forms its
// head's weights and surprise statistics itself from the few numbers they depend on.
template <bool ALL>
__global__ __launch_bounds__(256) void route_slice_kernel(const float *__restrict__ a_raw, int64_t rows,
                                                                   int L, int H, PromptTab tab, SliceTab st,
                                                                   LearnerConsts lc, const float *__restrict__ stats,
                                                                   const SliceSurprise *__restrict__ sur,
                                                                   float *__restrict__ scores)
{
    __shared__ HeadStats hs;
    int p, lh, s, S;
    const int slice = blockIdx.x / 4, first = (int)(blockIdx.x & 3) * kQuarter;
    locate(st, tab, slice, p, lh, s, S);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    if (s * kSlice + first >= N) return;
    const int64_t base = (int64_t)lh * tab.T + tab.tok_off[p];
    const float *a = a_raw + base;
    const int tid = threadIdx.x;
    constexpr int EACH = kQuarter / 256;
    float v[3][EACH];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const __amdgpu_buffer_rsrc_t vals = slice_values(a + k * rows, s, N);
#pragma unroll
        for (int j = 0; j < EACH; ++j) v[k][j] = slice_value<256>(vals, first + tid, j);
    }
    if (tid < 64) {
        const float *sk = stats + ((int64_t)p * L * H + lh) * 12 + 4 * min(tid, 2);
        head_weights(sk[0], sk[1], sk[2], lc, hs);
    }
    if (tid == 64) {
        float smin = INFINITY, smax = -INFINITY;
        double ssum = 0.0;
        const SliceSurprise *q = sur + (slice - s);
        for (int i = 0; i < S; ++i) {                                // the head's slices in order
            smin = fminf(smin, q[i].lo);
            smax = fmaxf(smax, q[i].hi);
            ssum += q[i].sum;
        }
        const float srange = smax - smin;
        hs.s_lo = smin;
        hs.s_inv_range = srange < kFlat ? 0.f : 1.0f / srange;
        hs.s_mean = (float)((ssum / (double)N - (double)smin) * (double)hs.s_inv_range);
    }
    __syncthreads();
    const HeadStats h = hs;
    float *out = scores + base;
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
        const int i = s * kSlice + first + j * 256 + tid;
        if (i < N) {
            const float raw[3] = {v[0][j], v[1][j], v[2][j]};
            float at[3];
            normalised(raw, h, at);
            out[i] = i < lc.n_sink ? NKV_PIN : routed_score<ALL>(at, h, lc);
        }
    }
}

// grid (units, 3); two wavefronts: 0 takes the upper boundary bin, 1 the lower one (on inverted keys).
// stats[(u * 3 + k) * 4 + {0, 1, 2}] = min, 1 / range (0 if flat), gap
__global__ __launch_bounds__(128) void stats_finish_kernel(const float *__restrict__ a_raw, int64_t rows, int L, int H,
                                                           PromptTab tab, SliceTab st, int n_slices,
                                                           const StatPick *__restrict__ picks,
                                                           const uint32_t *__restrict__ segTop,
                                                           const uint32_t *__restrict__ segBot,
                                                           const SlicePart *__restrict__ sp,
                                                           const uint32_t *__restrict__ failed, float *__restrict__ stats)
{
    __shared__ uint32_t keys[2][kList];
    __shared__ uint32_t hist[2][256];
    __shared__ double total[2];
    __shared__ uint32_t s_bad;
    const int u = blockIdx.x, k = blockIdx.y;
    const int64_t job = (int64_t)u * 3 + k;
    const int lh = u % (L * H), p = u / (L * H);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const int S = (N + kSlice - 1) / kSlice;
    const uint32_t m = (uint32_t)min(tab.m_p[p], N);
    const int lane = threadIdx.x & 63, side = threadIdx.x >> 6;
    const int64_t slice0 = (int64_t)k * n_slices + st.off[p] + (int64_t)lh * S;
    const StatPick pk = picks[job];
    const bool marked = failed[job] != 0u;
    if (threadIdx.x == 0) s_bad = 0u;
    // this side's list; sums over the slices (slice s0 + lane of a batch), min, max
    int none;
    const uint32_t *seg = (side == 0 ? segTop : segBot) + slice0 * kSeg;
    const int n = marked ? -1 : gather_segments(seg, S, [&](int s) { return side == 0 ? sp[slice0 + s].nTop : sp[slice0 + s].nBot; },
                                                keys[side], kList, -1, none);
    double sum = 0.0;
    float lo = INFINITY, hi = -INFINITY;
    for (int s = lane; s < S; s += 64) {
        const SlicePart q = sp[slice0 + s];
        sum += side == 0 ? q.sTop : q.sBot;
        lo = fminf(lo, q.lo);
        hi = fmaxf(hi, q.hi);
    }
    sum = wave_sum(sum);
    lo = wave_min(lo);
    hi = wave_max(hi);
    __syncthreads();
    if (n < 0 && lane == 0) s_bad = 1u;
    __syncthreads();
    // The lists' order depends on the timing of the collecting workgroups, so their entries are added up in
    // fixed point (2^-40 units, exact for fp32 values of magnitude <= 1 down to that resolution): the sum does
    // not depend on the order, and the statistics are reproducible bit for bit.
    constexpr double kFix = 1099511627776.0;                         // 2^40
    if (s_bad) {
        if (side != 0) return;
        // More values in one bin than the lists hold (thousands of equal anomalies): the first wavefront walks the
        // head's values itself -- slow, exact, and rare.
        const float *a = a_raw + (int64_t)k * rows + (int64_t)lh * tab.T + tab.tok_off[p];
        lo = INFINITY;
        hi = -INFINITY;
        for (int i = lane; i < N; i += 64) {
            lo = fminf(lo, a[i]);
            hi = fmaxf(hi, a[i]);
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        uint32_t gt, eq;
        const uint32_t Tt = wave_select_fn(N, m, hist[0], gt, eq, [a](int i) { return ord_key(a[i]); });
        long long part = 0;
        for (int i = lane; i < N; i += 64)
            part += ord_key(a[i]) > Tt ? __double2ll_rn((double)a[i] * kFix) : 0ll;
        const double top = (double)wave_sum(part) / kFix + (double)(m - gt) * (double)key_value(Tt);
        const uint32_t Tb = wave_select_fn(N, m, hist[0], gt, eq, [a](int i) { return ~ord_key(a[i]); });
        part = 0;
        for (int i = lane; i < N; i += 64)
            part += ~ord_key(a[i]) > Tb ? __double2ll_rn((double)a[i] * kFix) : 0ll;
        const double bot = (double)wave_sum(part) / kFix + (double)(m - gt) * (double)key_value(~Tb);
        if (lane == 0) {
            const float range = hi - lo;
            const float inv = range < kFlat ? 0.f : 1.0f / range;
            float *o = stats + job * 4;
            o[0] = lo;
            o[1] = inv;
            o[2] = (float)((top - bot) / (double)m * (double)inv);
        }
        return;
    }
    {
        // the `need` best of the bin's entries belong to the m largest / smallest
        const uint32_t need = side == 0 ? pk.needTop : pk.needBot;
        uint32_t gt, eq;
        const uint32_t T = wave_select(keys[side], n, need, hist[side], gt, eq);
        long long part = 0;
        for (int i = lane; i < n; i += 64) {
            const uint32_t key = keys[side][i];
            part += key > T ? __double2ll_rn((double)key_value(side == 0 ? key : ~key) * kFix) : 0ll;
        }
        const double t = sum + (double)wave_sum(part) / kFix + (double)(need - gt) * (double)key_value(side == 0 ? T : ~T);
        if (lane == 0) total[side] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float range = hi - lo;
        const float inv = range < kFlat ? 0.f : 1.0f / range;
        float *o = stats + job * 4;
        o[0] = lo;
        o[1] = inv;
        o[2] = (float)((total[0] - total[1]) / (double)m * (double)inv);
    }
}

struct WideWs {
    size_t part, sp, sur, picks, segTop, segBot, failed, total;
};

WideWs wide_ws(int L, int H, const PromptTab &tab)
{
    SliceTab st;
    const size_t slices = 3 * (size_t)fill_slices(L, H, tab, &st), jobs = 3 * (size_t)tab.n * L * H;
    WideWs w;
    size_t off = 0;
    w.part = off;    off += align256(slices * kBins * sizeof(uint16_t));
    w.sp = off;      off += align256(slices * sizeof(SlicePart));
    w.sur = off;     off += align256(slices / 3 * sizeof(SliceSurprise));
    w.picks = off;   off += align256(jobs * sizeof(StatPick));
    w.segTop = off;  off += align256(slices * kSeg * sizeof(uint32_t));
    w.segBot = off;  off += align256(slices * kSeg * sizeof(uint32_t));
    w.failed = off;  off += align256(jobs * sizeof(uint32_t));
    w.total = off;
    return w;
}

}  // namespace

size_t stats_wide_ws_bytes(int L, int H, const PromptTab &tab) { return wide_ws(L, H, tab).total; }

// Enqueues the four kernels that fill `stats`.
hipError_t launch_stats_wide(const float *a_raw, int L, int H, const PromptTab &tab, int scale_mask, float *stats, void *ws,
                             hipStream_t st)
{
    SliceTab stab;
    const int slices = fill_slices(L, H, tab, &stab);
    const WideWs lay = wide_ws(L, H, tab);
    char *base = (char *)ws;
    uint16_t *part = (uint16_t *)(base + lay.part);
    SlicePart *sp = (SlicePart *)(base + lay.sp);
    StatPick *picks = (StatPick *)(base + lay.picks);
    uint32_t *segTop = (uint32_t *)(base + lay.segTop), *segBot = (uint32_t *)(base + lay.segBot);
    uint32_t *failed = (uint32_t *)(base + lay.failed);
    SliceSurprise *sur = (SliceSurprise *)(base + lay.sur);
    const int64_t rows = (int64_t)L * H * tab.T;
    const unsigned units = (unsigned)(tab.n * L * H);
    const bool few = few_slices(slices);
    (few ? stats_hist_kernel<1024> : stats_hist_kernel<256>)<<<dim3((unsigned)slices, 3), few ? 1024 : 256, 0, st>>>(
        a_raw, rows, tab, stab, slices, part, sp, sur);
    stats_pick_kernel<<<dim3(units, 3), 256, 0, st>>>(L, H, tab, stab, slices, part, sp, picks, failed);
    const bool all = scale_mask == 7;
    (all ? stats_collect_kernel<true> : stats_collect_kernel<false>)<<<4u * (unsigned)slices, 256, 0, st>>>(
        a_raw, rows, L, H, tab, stab, slices, scale_mask, picks, segTop, segBot, sp, sur, failed);
    stats_finish_kernel<<<dim3(units, 3), 128, 0, st>>>(a_raw, rows, L, H, tab, stab, slices, picks, segTop, segBot,
                                                       sp, failed, stats);
    return hipGetLastError();
}

// Final scores from the statistics and the slices' surprise sums that launch_stats_wide left in the same scratch.
hipError_t launch_route_wide(const float *a_raw, int L, int H, const PromptTab &tab, const LearnerConsts &lc,
                             const float *stats, void *ws, float *scores, hipStream_t st)
{
    SliceTab stab;
    const int slices = fill_slices(L, H, tab, &stab);
    const WideWs lay = wide_ws(L, H, tab);
    const SliceSurprise *sur = (const SliceSurprise *)((char *)ws + lay.sur);
    (lc.scale_mask == 7 ? route_slice_kernel<true> : route_slice_kernel<false>)<<<4u * (unsigned)slices, 256, 0, st>>>(
        a_raw, (int64_t)L * H * tab.T, L, H, tab, stab, lc, stats, sur, scores);
    return hipGetLastError();
}

}  // namespace nkv
