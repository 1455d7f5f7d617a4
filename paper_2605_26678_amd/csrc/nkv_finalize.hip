// Outer learner: from the three raw anomalies of a head to its final scores
// (paper Section 2.3 min-max, Section 2.4 reliability gaps / blend / surprise / gate, sink pinning).
//
//   finalize_unit_kernel  calls whose prompts are all of up to 16384 tokens: one workgroup of 1024 threads per unit
//                         (prompt, layer, head), values in registers; up to 32768 tokens where the caller asks for
//                         per-head kernels
//   nkv_finalize_wide.hip calls with a longer prompt: slice by slice over the whole chip
//   finalize_kernel       calls with a still longer prompt where the caller asks for per-head kernels: one workgroup of
//                         1024 threads per unit walks the head's values in memory seven times:
//     pass 1      min / max of each scale
//     pass 2..5   byte-wise radix select (most significant digit first) of the m_p-th largest and the
//                 m_p-th smallest value of each scale, six selects at once in LDS histograms
//     pass 6      sums above / below those thresholds (fp64), and min / max / sum of the surprise
//     pass 7      blend, gate, route, pin, write
// The sum of the m largest values is  sum(a > T) + (m - count(a > T)) * T  with T the m-th largest,
// which does not depend on how ties at T are broken.  Min-max is affine and increasing, so the
// selects run on the raw anomalies and the gap is rescaled afterwards.
#include "nkv_blocksel.h"
#include "nkv_learner.h"
#include "nkv_slices.h"

namespace nkv {
namespace {

constexpr int kThreads = 1024;

__global__ __launch_bounds__(kThreads) void finalize_kernel(const float *__restrict__ a_raw, int L, int H,
                                                            PromptTab tab, LearnerConsts lc,
                                                            float *__restrict__ scores)
{
    __shared__ uint32_t hist[6][256];
    __shared__ uint32_t sel_prefix[6], sel_want[6];
    __shared__ float fscratch[16];
    __shared__ double dscratch[16];
    __shared__ HeadStats hs;

    const int u = blockIdx.x;                    // (p * L + l) * H + h
    const int h = u % H, l = (u / H) % L, p = u / (H * L);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const int64_t rows = (int64_t)L * H * tab.T;
    const int64_t base = ((int64_t)l * H + h) * tab.T + tab.tok_off[p];
    const float *a[3] = {a_raw + base, a_raw + rows + base, a_raw + 2 * rows + base};
    const int tid = threadIdx.x;

    // ---- pass 1: min / max per scale ----
    float lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float mn = INFINITY, mx = -INFINITY;
        for (int i = tid; i < N; i += kThreads) {
            const float v = a[k][i];
            mn = fminf(mn, v);
            mx = fmaxf(mx, v);
        }
        lo[k] = block_min(mn, fscratch);
        hi[k] = block_max(mx, fscratch);
    }
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float range = hi[k] - lo[k];
            hs.lo[k] = lo[k];
            hs.inv_range[k] = range < kFlat ? 0.f : 1.0f / range;
        }
    }
    if (tid < 6) { sel_prefix[tid] = 0u; sel_want[tid] = (uint32_t)min(tab.m_p[p], N); }
    __syncthreads();

    // ---- passes 2..5: six radix selects; select s = 2*k + e, e = 0 top (m-th largest), 1 bottom ----
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        for (int j = tid; j < 6 * 256; j += kThreads) (&hist[0][0])[j] = 0u;
        __syncthreads();
        uint32_t pre[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) pre[s] = sel_prefix[s];
        for (int i = tid; i < N; i += kThreads) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint32_t key = ord_key(a[k][i]);
                const uint32_t hi_bits = pass == 0 ? 0u : key >> (shift + 8);
                const uint32_t dig = (key >> shift) & 255u;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t want_hi = pass == 0 ? 0u : pre[2 * k + e] >> (shift + 8);
                    if (hi_bits == want_hi) atomicAdd(&hist[2 * k + e][dig], 1u);
                }
            }
        }
        __syncthreads();
        if (tid < 6) {
            uint32_t want = sel_want[tid];
            const uint32_t dig = radix_pick(hist[tid], want, (tid & 1) == 0);
            sel_want[tid] = want;
            sel_prefix[tid] |= dig << shift;
        }
        __syncthreads();
    }

    // ---- pass 6: sums beyond the thresholds; surprise statistics ----
    const int m = min(tab.m_p[p], N);
    HeadStats st = hs;
    double sums[6];
    {
        uint32_t thr[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) { thr[s] = sel_prefix[s]; sums[s] = 0.0; }
        float smin = INFINITY, smax = -INFINITY;
        double ssum = 0.0;
        for (int i = tid; i < N; i += kThreads) {
            float av[3], at[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                av[k] = a[k][i];
                const uint32_t key = ord_key(av[k]);
                if (key > thr[2 * k]) sums[2 * k] += (double)av[k];
                if (key < thr[2 * k + 1]) sums[2 * k + 1] += (double)av[k];
            }
            normalised(av, st, at);
            const float s = surprise_std(at, lc.scale_mask);
            smin = fminf(smin, s);
            smax = fmaxf(smax, s);
            ssum += (double)s;
        }
#pragma unroll
        for (int s = 0; s < 6; ++s) sums[s] = block_sum(sums[s], dscratch);
        smin = block_min(smin, fscratch);
        smax = block_max(smax, fscratch);
        ssum = block_sum(ssum, dscratch);
        if (tid == 0) {
            double z[3], zmax = -INFINITY, zsum = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                // ties at the threshold: sel_want of them belong to the set
                const double top = sums[2 * k] + (double)sel_want[2 * k] * (double)key_value(thr[2 * k]);
                const double bot = sums[2 * k + 1] + (double)sel_want[2 * k + 1] * (double)key_value(thr[2 * k + 1]);
                const double delta = (top - bot) / (double)m * (double)st.inv_range[k];
                z[k] = lc.log_prior[k] + lc.beta * delta;
                zmax = fmax(zmax, z[k]);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) { z[k] = exp(z[k] - zmax); zsum += z[k]; }
#pragma unroll
            for (int k = 0; k < 3; ++k) hs.w[k] = (float)(z[k] / zsum);
            const float srange = smax - smin;
            hs.s_lo = smin;
            hs.s_inv_range = srange < kFlat ? 0.f : 1.0f / srange;
            hs.s_mean = (float)((ssum / (double)N - (double)smin) * (double)hs.s_inv_range);
        }
        __syncthreads();
    }

    // ---- pass 7: blend, gate, route, pin ----
    st = hs;
    float *out = scores + base;
    for (int i = tid; i < N; i += kThreads) {
        float av[3], at[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) av[k] = a[k][i];
        normalised(av, st, at);
        const float star = routed_score(at, st, lc);
        out[i] = i < lc.n_sink ? NKV_PIN : star;
    }
}


// ------------------------------------------------------------------------------------------------------
// Units of up to 1024 * EPT tokens: everything in one launch, the three anomalies of a token in registers from the only
// read of them to the routed score.  One workgroup of 1024 threads per unit.
//
// A short unit's arithmetic is small and what takes time is the chain of dependent steps, so there are few of them (as
// two kernels of radix selects, one workgroup per scale, 16 x 8 units of 4096 tokens took 33 us, this takes 12), and inside them the
// instructions that sixteen wavefronts issue on four SIMDs.  Of 31 000 cycles of a unit of 4096 tokens with a bin formed for every value and
// every wavefront's result reduced by itself, step 3 took 10 000, ranges and histograms 5 000 each.  Against that, values compared with
// the boundary bins' edges, eight reductions at once, weights in three lanes, ranges and edges worked out a scale or list a lane: the score call
// of those units 49.4 -> 45.8 us, the batch below 104.5 -> 90.5.
//   1. min and max of each scale, then its histogram over that range (2048 bins);
//   2. one scan per scale gives the bins that hold the m-th largest and the m-th smallest value; a bin that holds more
//      than kUnitList values is narrowed down first (see below);
//   3. sums beyond those bins, their entries into six lists; surprise statistics (the ranges are known);
//   4. six wavefronts find the exact thresholds in the lists, another one adds the surprise up;
//   5. weights; blend, gate, route, pin.
// Same numbers as the slice-wise kernels (the sums over a boundary bin's entries in fixed point: independent of the
// order the entries arrive in).
//
// Narrowing: anomalies may all lie close together but for a few outliers (keys with a strong common direction), or be
// equal by the thousand (repeated keys).  A crowded bin is cut, between the smallest and the largest key in it, into 1024
// bins of integer keys, all six boundary bins at once, until it holds few keys or a single one: one round for
// values that are merely close, two where they also repeat.  With a histogram over the whole range of a cosine, a wavefront
// that walked the unit's values where a list overflowed, and an add per value, the scores of 8 heads x 8192 tokens took
// 34 us for spread-out keys, 224 us for keys close together; now 35 and 35, 50 where half of the keys are equal.
// ------------------------------------------------------------------------------------------------------
constexpr int kUnitList = 256;              // keys a list holds

// Where the m largest (list 2k of scale k) or the m smallest (2k + 1, on inverted keys) end.
struct UnitCut {
    int bin;                                  // boundary bin
    uint32_t need, pop;                       // of the pop values between lo and hi in it, the need best belong to the m
    uint32_t lo, hi;                          // keys; better ones of the bin belong to the m, worse ones do not
};

// monotone in x
__device__ __forceinline__ float unit_scaled(float x, float lo, float scale) { return (x - lo) * scale; }
__device__ __forceinline__ int unit_bin(float x, float lo, float scale) { return min(max((int)unit_scaled(x, lo, scale), 0), kBins - 1); }

constexpr int kUnitWaves = kSelThreads / 64;
struct UnitScratch {
    uint32_t buf[3 * kBins];                  // the histograms, then the lists
    uint32_t whist[6][256];
    uint32_t ext[12];                         // per scale, of the wavefronts' minima and maxima as keys: max of ~min, max, min, ~max
    uint32_t wtot[6][kUnitWaves];
    UnitCut cut[6];
    float lo[3], to_bin[3];
    uint32_t range[6][2];                     // of a crowded bin: max of ~key and of key
    uint32_t cnt[6];
    uint32_t crowded;                         // a boundary bin holds more values than a list
    double sums[7][kUnitWaves];               // beyond the boundary bins, per wavefront; the surprise
    float sext[2][kUnitWaves];
    double side[6];
    HeadStats hs;
};

// EPT: values a thread holds per scale.  32 values (asked for by flag only) do not fit the registers and are read from the caches every
// time.
template <int EPT, bool ALL>
__device__ __forceinline__ void finalize_unit(UnitScratch &sh, const float *__restrict__ a_raw, int L, int H, const PromptTab &tab,
                                              const LearnerConsts &lc, float *__restrict__ scores)
{
    constexpr int NW = kUnitWaves, kSub = kSelThreads;
    auto &buf = sh.buf;
    auto &ext = sh.ext;
    auto &cnt = sh.cnt;
    auto &whist = sh.whist;
    auto &wtot = sh.wtot;
    auto &s_cut = sh.cut;
    auto &s_lo = sh.lo, &s_to_bin = sh.to_bin;
    auto &range = sh.range;
    auto &sums = sh.sums;
    auto &sext = sh.sext;
    auto &side = sh.side;
    auto &hs = sh.hs;
    static_assert(6 * kUnitList <= 3 * kBins && 6 * kSub <= 3 * kBins, "lists and narrowed bins lie where the histograms were");

    const int u = blockIdx.x;
    const int h = u % H, l = (u / H) % L, p = u / (H * L);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const int64_t rows = (int64_t)L * H * tab.T;
    const int64_t base = ((int64_t)l * H + h) * tab.T + tab.tok_off[p];
    const float *a = a_raw + base;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t m = (uint32_t)min(tab.m_p[p], N);

    constexpr bool kHeld = EPT <= 16;
    constexpr int kUnroll = kHeld ? EPT : 4;
    float v[3][kHeld ? EPT : 1];
    auto load = [&](int k, int j) { return a[k * rows + min(tid + j * kSelThreads, N - 1)]; };
    auto value = [&](int k, int j) { return kHeld ? v[k][kHeld ? j : 0] : load(k, j); };
    if constexpr (kHeld) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < EPT; ++j) v[k][j] = load(k, j);
    }
    auto clear_buf = [&]() {
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int j = 0; j < 3 * kBins / 4 / kSelThreads + 1; ++j)
            if (tid + j * kSelThreads < 3 * kBins / 4) reinterpret_cast<uint4 *>(buf)[tid + j * kSelThreads] = zero;
    };
    clear_buf();
    if (tid < 12) ext[tid] = 0u;
    if (tid == 12) sh.crowded = 0u;
    if (tid < 6) {
        cnt[tid] = range[tid][0] = range[tid][1] = 0u;
        s_cut[tid] = UnitCut{-1, 0u, 0u, 0u, 0xffffffffu};            // (what a flat scale keeps: its gap does not count)
    }
    __syncthreads();

    // ---- 1: ranges, histograms ----
    // The histogram's range leaves the outliers aside that a few wavefronts hold (they go to its end bins): it lies between
    // the largest minimum and the smallest maximum of a wavefront, where there is anything between them and a wavefront
    // holds 128 values and more (the tenth of them that is looked for lies inside, then).
    auto smaller = [](float x, float y) { return fminf(x, y); };
    {
        float least[8];                                               // the scales' minima, their negated maxima
#pragma unroll
        for (int i = 0; i < 8; ++i) least[i] = INFINITY;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll kUnroll
            for (int j = 0; j < EPT; ++j) {                           // (what a thread holds past the unit repeats its last value)
                const float x = value(k, j);
                least[k] = fminf(least[k], x);
                least[3 + k] = fminf(least[3 + k], -x);
            }
        const float r = wave_reduce8(least, smaller);
        const int i = lane >> 3, k = i < 3 ? i : i - 3;
        if ((lane & 7) == 0 && i < 6) {
            const uint32_t key = ord_key(i < 3 ? r : -r);
            atomicMax(&ext[4 * k + (i < 3 ? 0 : 3)], ~key);
            atomicMax(&ext[4 * k + (i < 3 ? 2 : 1)], key);
        }
    }
    __syncthreads();
    auto of_lane = [](float x, int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k)); };
    HeadStats st;
    float bins_lo[3], to_bin[3];                                      // to_bin: bins per unit of the scale; 0: the scale is flat
    {
        const int k = min(lane, 2);                                   // (lane k: scale k)
        const float lo = key_value(~ext[4 * k]), hi = key_value(ext[4 * k + 1]), inner_lo = key_value(ext[4 * k + 2]), inner_hi = key_value(~ext[4 * k + 3]);
        const float range = hi - lo, inv = range < kFlat ? 0.f : 1.0f / range;
        const bool inner = inner_hi > inner_lo && N >= 2 * kSelThreads;
        const float from = inner ? inner_lo : lo, scale = range < kFlat ? 0.f : (float)kBins * __builtin_amdgcn_rcpf(inner ? inner_hi - inner_lo : range);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            st.lo[q] = of_lane(lo, q);
            st.inv_range[q] = of_lane(inv, q);
            bins_lo[q] = of_lane(from, q);
            to_bin[q] = of_lane(scale, q);
        }
    }
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) { s_lo[k] = bins_lo[k]; s_to_bin[k] = to_bin[k]; }
    }
    auto bin_of = [&](int k, float x) { return unit_bin(x, bins_lo[k], to_bin[k]); };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (to_bin[k] == 0.f) continue;
        bool queue = false;                                           // many equal values, going by three of the slots
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int j = i * (EPT - 1) / 2, b = bin_of(k, value(k, j));
            queue |= __popcll(__ballot(b == __builtin_amdgcn_readfirstlane(b) && tid + j * kSelThreads < N)) > 16;
        }
        if (queue) {
#pragma unroll kUnroll
            for (int j = 0; j < EPT; ++j) {
                const float x = value(k, j);
                if (tid + j * kSelThreads < N) count_bin(buf + k * kBins, bin_of(k, x));
            }
        } else {
#pragma unroll kUnroll
            for (int j = 0; j < EPT; ++j) {
                const float x = value(k, j);
                if (tid + j * kSelThreads < N) atomicAdd(&buf[k * kBins + bin_of(k, x)], 1u);
            }
        }
    }
    __syncthreads();

    // ---- 2: boundary bins; thread: bins 2 tid, 2 tid + 1 of every scale ----
    uint2 c[3];
    uint32_t incl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        c[k] = reinterpret_cast<const uint2 *>(buf + k * kBins)[tid];
        incl[k] = wave_prefix_sum(c[k].x + c[k].y);
        if (lane == 63) wtot[k][w] = incl[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (to_bin[k] == 0.f) continue;
        const uint32_t group = c[k].x + c[k].y;
        const uint32_t up = incl[k] + wave_sum(lane < w ? wtot[k][lane & (NW - 1)] : 0u);   // entries up to and with my bins
        const uint32_t below = up - group, above = (uint32_t)N - up;
        if (below < m && m <= up) {                                   // the m-th smallest lies in one of my bins
            const bool second = below + c[k].x < m;
            s_cut[2 * k + 1].bin = 2 * tid + (second ? 1 : 0);
            s_cut[2 * k + 1].need = m - below - (second ? c[k].x : 0u);
            s_cut[2 * k + 1].pop = second ? c[k].y : c[k].x;
            if ((second ? c[k].y : c[k].x) > (uint32_t)kUnitList) sh.crowded = 1u;
        }
        if (above < m && m <= above + group) {                        // the m-th largest
            const bool first = above + c[k].y < m;
            s_cut[2 * k].bin = 2 * tid + (first ? 0 : 1);
            s_cut[2 * k].need = m - above - (first ? c[k].y : 0u);
            s_cut[2 * k].pop = first ? c[k].x : c[k].y;
            if ((first ? c[k].x : c[k].y) > (uint32_t)kUnitList) sh.crowded = 1u;
        }
    }
    __syncthreads();
    auto key_of = [](int i, float x) { return i & 1 ? ~ord_key(x) : ord_key(x); };   // inverted: the smallest value has the largest key
    auto crowded = [](const UnitCut &q) { return q.pop > (uint32_t)kUnitList && q.lo != q.hi; };
    auto any_crowded = [&]() {                                        // the same for every thread
        bool any = false;
        for (int i = 0; i < 6; ++i) any |= crowded(s_cut[i]);
        return any;
    };
    if (__builtin_amdgcn_readfirstlane((int)sh.crowded) != 0) {
        // f(list, its cut, up to 8 of a thread's keys, which of them are in the list's boundary bin).  From 16 values a thread
        // on they are read again: the rare path then costs the common one no registers.
        constexpr int kKeys = EPT < 16 ? EPT : 8, kLists = EPT < 16 ? 6 : 1;
        auto for_crowded = [&](auto f) {
#pragma unroll kLists
            for (int i = 0; i < 6; ++i) {
                const UnitCut q = s_cut[i];
                if (!crowded(q)) continue;
                const int k = i >> 1;
                const float lo = s_lo[k], scale = s_to_bin[k];
#pragma unroll 1
                for (int j0 = 0; j0 < EPT; j0 += kKeys) {
                    uint32_t key[kKeys];
                    bool in[kKeys];
                    float x[kKeys];
#pragma unroll
                    for (int j = 0; j < kKeys; ++j) {
                        x[j] = EPT < 16 ? v[k][EPT < 16 ? j : 0] : load(k, j0 + j);
                        asm volatile("" : "+v"(x[j]));
                    }
#pragma unroll
                    for (int j = 0; j < kKeys; ++j) {
                        key[j] = key_of(i, x[j]);
                        in[j] = tid + (j0 + j) * kSelThreads < N && unit_bin(x[j], lo, scale) == q.bin;
                    }
                    f(i, q, key, in);
                }
            }
        };
        for_crowded([&](int i, const UnitCut &, const uint32_t (&key)[kKeys], const bool (&in)[kKeys]) {
            uint32_t nlo = 0u, hi = 0u;
#pragma unroll
            for (int j = 0; j < kKeys; ++j) {
                nlo = max(nlo, in[j] ? ~key[j] : 0u);
                hi = max(hi, in[j] ? key[j] : 0u);
            }
            auto larger = [](uint32_t x, uint32_t y) { return max(x, y); };
            nlo = wave_reduce(nlo, larger);
            hi = wave_reduce(hi, larger);
            if (lane == 0) {
                atomicMax(&range[i][0], nlo);
                atomicMax(&range[i][1], hi);
            }
        });
        __syncthreads();
        if (tid < 6 && crowded(s_cut[tid])) {
            s_cut[tid].lo = ~range[tid][0];
            s_cut[tid].hi = range[tid][1];
        }
        __syncthreads();
        auto shift_of = [](const UnitCut &q) { return q.hi - q.lo < (uint32_t)kSub ? 0 : 22 - __builtin_clz(q.hi - q.lo); };
        for (int round = 0; round < 4 && any_crowded(); ++round) {    // every round cuts an interval to a 1024th
            clear_buf();
            __syncthreads();
            for_crowded([&](int i, const UnitCut &q, const uint32_t (&key)[kKeys], const bool (&in)[kKeys]) {
                const int shift = shift_of(q);
#pragma unroll
                for (int j = 0; j < kKeys; ++j)
                    if (in[j] && key[j] - q.lo <= q.hi - q.lo) count_bin(buf + i * kSub, (int)((key[j] - q.lo) >> shift));
            });
            __syncthreads();
#pragma unroll 1
            for (int i = 0; i < 6; ++i) {                             // thread: bin tid of the interval, counted from the top
                const UnitCut q = s_cut[i];
                if (!crowded(q)) continue;
                const uint32_t mine = buf[i * kSub + tid], up = wave_suffix_sum(mine);
                if (lane == 0) wtot[0][w] = up;
                __syncthreads();
                const uint32_t counted = up + wave_sum(lane > w && lane < NW ? wtot[0][lane & (NW - 1)] : 0u), above = counted - mine;
                if (above < q.need && q.need <= counted) {
                    const uint32_t lo = q.lo + ((uint32_t)tid << shift_of(q));
                    s_cut[i] = UnitCut{q.bin, q.need - above, mine, lo, min(q.hi, lo + ((1u << shift_of(q)) - 1u))};
                }
                __syncthreads();
            }
        }
    }
    // (bins are cheaper worked out again than kept: the compiler would carry those of all values over from step 1)
    if constexpr (kHeld) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < EPT; ++j) asm volatile("" : "+v"(v[k][j]));
    }
    uint32_t cut_lo[6], cut_hi[6];                                    // uniform; lane i worked list i's out
    BinEdges edge[6];
    {
        const UnitCut q = s_cut[min(lane, 5)];
        const float low = bin_low_edge(q.bin), high = bin_high_edge(q.bin);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const float l = of_lane(low, i), h = of_lane(high, i);
            edge[i] = BinEdges{h, l, l, h};
            cut_lo[i] = (uint32_t)__builtin_amdgcn_readlane((int)q.lo, i);
            cut_hi[i] = (uint32_t)__builtin_amdgcn_readlane((int)q.hi, i);
        }
    }

    // ---- 3: sums beyond the boundary bins, their entries, the surprise ----
    float pt[3] = {0.f, 0.f, 0.f}, pb[3] = {0.f, 0.f, 0.f};           // at most EPT terms of magnitude <= 1
    float smin = INFINITY, smax = -INFINITY;
    double ssum = 0.0;
#pragma unroll kUnroll
    for (int j = 0; j < EPT; ++j) {
        float raw[3] = {value(0, j), value(1, j), value(2, j)};
        if (tid + j * kSelThreads < N) {
            float at[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float x = raw[k], y = unit_scaled(x, bins_lo[k], to_bin[k]);
                const bool over = y >= edge[2 * k].above, under = y < edge[2 * k + 1].below;
                pt[k] += over ? x : 0.f;
                pb[k] += under ? x : 0.f;
                const bool in[2] = {!over && y >= edge[2 * k].from, !under && y < edge[2 * k + 1].to};
                if (!in[0] && !in[1]) continue;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * k + e;
                    if (in[e]) {
                        const uint32_t key = key_of(i, x);
                        if (key > cut_hi[i]) {
                            (e == 0 ? pt : pb)[k] += x;
                        } else if (key >= cut_lo[i] && cut_lo[i] != cut_hi[i]) {   // (a single key needs no list)
                            const uint32_t at = atomicAdd(&cnt[i], 1u);
                            if (at < (uint32_t)kUnitList) buf[i * kUnitList + at] = key;
                        }
                    }
                }
            }
            normalised(raw, st, at);
            const float s = surprise_std<ALL>(at, lc.scale_mask);
            smin = fminf(smin, s);
            smax = fmaxf(smax, s);
            ssum += (double)s;
        }
    }
    {
        const double part[8] = {(double)pt[0], (double)pb[0], (double)pt[1], (double)pb[1], (double)pt[2], (double)pb[2], ssum, 0.0};
        const double t = wave_reduce8(part, [](double x, double y) { return x + y; });
        if ((lane & 7) == 0 && lane < 56) sums[lane >> 3][w] = t;
        float r = swap_merge<32>(smin, -smax, smaller);
        r = swap_reduce<16>(row16_reduce(r, smaller), smaller);
        if (lane == 0) sext[0][w] = r;
        if (lane == 32) sext[1][w] = -r;
    }
    __syncthreads();

    // ---- 4: exact thresholds in the lists (wavefront = list), the surprise's range and mean ----
    if (w < 6) {
        constexpr double kFix = 1099511627776.0;                      // 2^40: exact for fp32 values of magnitude <= 1 down to that step
        const bool low = (w & 1) != 0;
        const UnitCut q = s_cut[w];
        const int n = min((int)cnt[w], kUnitList);
        uint32_t T = q.lo, gt = 0u, eq;
        long long part = 0;
        if (n > 0) {
            const uint32_t *list = buf + w * kUnitList;
            T = wave_select(list, n, q.need, whist[w], gt, eq);
            for (int i = lane; i < n; i += 64)
                part += list[i] > T ? __double2ll_rn((double)key_value(low ? ~list[i] : list[i]) * kFix) : 0ll;
        }
        double total = wave_sum(lane < NW ? sums[w][lane & (NW - 1)] : 0.0) + (double)wave_sum(part) / kFix;
        if (q.need > 0u) total += (double)(q.need - gt) * (double)key_value(low ? ~T : T);   // (0: a flat scale)
        if (lane == 0) side[w] = total;
    } else if (w == 6) {
        const int i = lane & (NW - 1);
        const float lo = wave_min(sext[0][i]), hi = wave_max(sext[1][i]);
        const double t = wave_sum(lane < NW ? sums[6][i] : 0.0);
        if (lane == 0) {
            const float range = hi - lo;
            hs.s_lo = lo;
            hs.s_inv_range = range < kFlat ? 0.f : 1.0f / range;
            hs.s_mean = (float)((t / (double)N - (double)lo) * (double)hs.s_inv_range);
        }
    }
    __syncthreads();
    if (w == 0) {
        const int k = min(lane, 2);
        const float lo = k == 0 ? st.lo[0] : k == 1 ? st.lo[1] : st.lo[2], inv = k == 0 ? st.inv_range[0] : k == 1 ? st.inv_range[1] : st.inv_range[2];
        head_weights(lo, inv, (float)((side[2 * k] - side[2 * k + 1]) / (double)m * (double)inv), lc, hs);
    }
    __syncthreads();

    // ---- 5: blend, gate, route, pin ----
    st = hs;
    float *out = scores + base;
#pragma unroll kUnroll
    for (int j = 0; j < EPT; ++j) {
        const int i = tid + j * kSelThreads;
        const float raw[3] = {value(0, j), value(1, j), value(2, j)};
        if (i < N) {
            float at[3];
            normalised(raw, st, at);
            out[i] = i < lc.n_sink ? NKV_PIN : routed_score<ALL>(at, st, lc);
        }
    }
}

// grid: units.  Units of up to 1024 LO tokens, and of up to 1024 HI, are done in the same launch; those of other length classes are
// passed over, so that a ragged batch takes one launch for prompts of up to 8192 tokens and one for longer ones (4 layers x 32 heads x
// prompts of 1531, 4099, 777 and 2050 tokens, score call: 116.8 us with a launch for each of its two classes, 104.5 this way).  Up to 8192
// tokens two workgroups share a compute unit, at 64 registers a thread: the instances with units of more than 4096 tokens spill one or
// two of them.
template <int LO, int HI, bool ALL>
__global__ __launch_bounds__(kSelThreads, HI <= 8 ? 8 : 4) void finalize_unit_kernel(const float *__restrict__ a_raw, int L, int H,
                                                                                     PromptTab tab, LearnerConsts lc,
                                                                                     float *__restrict__ scores)
{
    __shared__ __attribute__((aligned(16))) UnitScratch sh;
    const int p = blockIdx.x / (L * H), cls = length_class(tab.tok_off[p + 1] - tab.tok_off[p]);
    if (cls == LO) finalize_unit<LO, ALL>(sh, a_raw, L, H, tab, lc, scores);
    else if (LO != HI && cls == HI) finalize_unit<HI, ALL>(sh, a_raw, L, H, tab, lc, scores);
}

}  // namespace

hipError_t launch_finalize(const float *a_raw, int L, int H, const PromptTab &tab, const LearnerConsts &lc,
                           float *scores, float *stats, void *wide_ws, bool per_head_route, const Prof &prof,
                           hipStream_t st)
{
    int nmax = 0;
    for (int p = 0; p < tab.n; ++p) nmax = max(nmax, tab.tok_off[p + 1] - tab.tok_off[p]);
    const unsigned units = (unsigned)(tab.n * L * H);
    const bool per_head = wide_ws == nullptr || per_head_route;
    prof.begin(NKV_KERNEL_FINALIZE, st);
    // By default one launch with a workgroup per unit for prompts of up to kUnitTokens and slices for longer ones; asked for
    // whole heads, a workgroup per unit as far as it goes (a score call of 8 heads x 32768 tokens: 89 us, 406 with
    // finalize_kernel).
    if (nmax > (per_head ? 2 * kUnitTokens : kUnitTokens)) {
        if (per_head) {
            finalize_kernel<<<units, kThreads, 0, st>>>(a_raw, L, H, tab, lc, scores);
        } else {
            hipError_t e = launch_stats_wide(a_raw, L, H, tab, lc.scale_mask, stats, wide_ws, st);
            if (e != hipSuccess) return e;
            e = launch_route_wide(a_raw, L, H, tab, lc, stats, wide_ws, scores, st);
            if (e != hipSuccess) return e;
        }
    } else {
        bool present[33] = {};
        for (int p = 0; p < tab.n; ++p) present[length_class(tab.tok_off[p + 1] - tab.tok_off[p])] = true;
#define NKV_UNIT(LO, HI)                                                                                            \
    (lc.scale_mask == 7 ? finalize_unit_kernel<LO, HI, true> : finalize_unit_kernel<LO, HI, false>)<<<units, kSelThreads, 0, st>>>( \
        a_raw, L, H, tab, lc, scores)
        if (present[4] && present[8]) NKV_UNIT(4, 8);
        else if (present[4]) NKV_UNIT(4, 4);
        else if (present[8]) NKV_UNIT(8, 8);
        if (present[16]) NKV_UNIT(16, 16);
        if (present[32]) NKV_UNIT(32, 32);
#undef NKV_UNIT
    }
    prof.end(NKV_KERNEL_FINALIZE, st);
    return hipGetLastError();
}

}  // namespace nkv
