// Outer learner: from the three raw anomalies of a head to its final scores
// (paper Section 2.3 min-max, Section 2.4 reliability gaps / blend / surprise / gate, sink pinning).
//
//   finalize_unit_kernel  calls whose prompts are all of up to 16384 tokens: one workgroup of 1024 threads per unit
//                         (prompt, layer, head), values in registers
//   nkv_finalize_wide.hip calls with a longer prompt: slice by slice over the whole chip
//   finalize_kernel       the same where the caller asks for per-head kernels: one workgroup of 1024 threads per
//                         unit walks the head's values in memory seven times:
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
// two kernels of radix selects, one workgroup per scale, 16 x 8 units of 4096 tokens took 33 us, this takes 11):
//   1. histograms of the three scales over the fixed range of a cosine (2048 bins), min and max of each;
//   2. one scan per scale gives the bins that hold the m-th largest and the m-th smallest value;
//   3. sums beyond those bins, their entries into six lists; surprise statistics (the ranges are known);
//   4. six wavefronts find the exact thresholds in the lists, another one adds the surprise up;
//   5. weights; blend, gate, route, pin.
// Same numbers as the slice-wise kernels (the sums over a boundary bin's entries in fixed point: independent of the
// order the entries arrive in).  A list that overflows (more than 1024 equal or nearly equal values) sends its wavefront
// over the unit's values in memory.
// ------------------------------------------------------------------------------------------------------
constexpr int kUnitList = 1024;              // keys a list holds

// grid: units.  EPT: values a thread holds per scale; units of prompts of another length class are passed over, so that a
// ragged batch takes one launch per class it holds, not one per run of prompts (4 layers x 32 heads x prompts of 1531,
// 4099, 777 and 2050 tokens: 39 -> 28 us).
template <int EPT, bool ALL>
__global__ __launch_bounds__(kSelThreads, EPT <= 4 ? 8 : 4) void finalize_unit_kernel(const float *__restrict__ a_raw, int L, int H,
                                                                                      PromptTab tab, LearnerConsts lc,
                                                                                      float *__restrict__ scores)
{
    constexpr int NW = kSelThreads / 64;
    __shared__ __attribute__((aligned(16))) uint32_t buf[3 * kBins];  // the histograms, then the lists
    __shared__ uint32_t whist[6][256];
    __shared__ uint32_t ext[6];                  // per scale: max of ~key and of key = ~min, max as ordered integers
    __shared__ uint32_t wtot[3][NW];
    __shared__ int bin[6];                       // list 2k: upper boundary bin of scale k, 2k + 1: lower
    __shared__ uint32_t need[6], cnt[6];
    __shared__ double sums[7][NW];               // beyond the boundary bins, per wavefront; the surprise
    __shared__ float sext[2][NW];
    __shared__ double side[6];
    __shared__ HeadStats hs;
    static_assert(6 * kUnitList <= 3 * kBins, "the lists lie where the histograms were");

    const int u = blockIdx.x;
    const int h = u % H, l = (u / H) % L, p = u / (H * L);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    if (length_class(N) != EPT) return;
    const int64_t rows = (int64_t)L * H * tab.T;
    const int64_t base = ((int64_t)l * H + h) * tab.T + tab.tok_off[p];
    const float *a = a_raw + base;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t m = (uint32_t)min(tab.m_p[p], N);

    float v[3][EPT];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < EPT; ++j) v[k][j] = a[k * rows + min(tid + j * kSelThreads, N - 1)];
#pragma unroll
    for (int j = 0; j < 3 * kBins / 4 / kSelThreads + 1; ++j)
        if (tid + j * kSelThreads < 3 * kBins / 4) reinterpret_cast<uint4 *>(buf)[tid + j * kSelThreads] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < 6) { ext[tid] = 0u; cnt[tid] = 0u; }
    __syncthreads();

    // ---- 1: histograms, ranges ----
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            if (tid + j * kSelThreads < N) {
                lo = fminf(lo, v[k][j]);
                hi = fmaxf(hi, v[k][j]);
                atomicAdd(&buf[k * kBins + anomaly_bin(v[k][j])], 1u);
            }
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0) {
            atomicMax(&ext[2 * k], ~ord_key(lo));
            atomicMax(&ext[2 * k + 1], ord_key(hi));
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
        const uint32_t group = c[k].x + c[k].y;
        const uint32_t up = incl[k] + wave_sum(lane < w ? wtot[k][lane & (NW - 1)] : 0u);   // entries up to and with my bins
        const uint32_t below = up - group, above = (uint32_t)N - up;
        if (below < m && m <= up) {                                   // the m-th smallest lies in one of my bins
            const bool second = below + c[k].x < m;
            bin[2 * k + 1] = 2 * tid + (second ? 1 : 0);
            need[2 * k + 1] = m - below - (second ? c[k].x : 0u);
        }
        if (above < m && m <= above + group) {                        // the m-th largest
            const bool first = above + c[k].y < m;
            bin[2 * k] = 2 * tid + (first ? 0 : 1);
            need[2 * k] = m - above - (first ? c[k].y : 0u);
        }
    }
    __syncthreads();

    // ---- 3: sums beyond the boundary bins, their entries, the surprise ----
    HeadStats st;
    float pt[3], pb[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        st.lo[k] = key_value(~ext[2 * k]);
        const float range = key_value(ext[2 * k + 1]) - st.lo[k];
        st.inv_range[k] = range < kFlat ? 0.f : 1.0f / range;
        pt[k] = pb[k] = 0.f;                                          // at most EPT terms of magnitude <= 1
    }
    float smin = INFINITY, smax = -INFINITY, ssum = 0.f;
    {
        int bT[3], bB[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) { bT[k] = bin[2 * k]; bB[k] = bin[2 * k + 1]; }
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            if (tid + j * kSelThreads < N) {
                float raw[3], at[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float x = raw[k] = v[k][j];
                    const int b = anomaly_bin(x);
                    pt[k] += b > bT[k] ? x : 0.f;
                    pb[k] += b < bB[k] ? x : 0.f;
                    if (b == bT[k]) {
                        const uint32_t i = atomicAdd(&cnt[2 * k], 1u);
                        if (i < (uint32_t)kUnitList) buf[2 * k * kUnitList + i] = ord_key(x);
                    }
                    if (b == bB[k]) {                                 // inverted: the smallest value has the largest key
                        const uint32_t i = atomicAdd(&cnt[2 * k + 1], 1u);
                        if (i < (uint32_t)kUnitList) buf[(2 * k + 1) * kUnitList + i] = ~ord_key(x);
                    }
                }
                normalised(raw, st, at);
                const float s = surprise_std<ALL>(at, lc.scale_mask);
                smin = fminf(smin, s);
                smax = fmaxf(smax, s);
                ssum += s;                                            // at most EPT terms of magnitude <= 0.5
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double t = wave_sum((double)pt[k]), b = wave_sum((double)pb[k]);
        if (lane == 0) { sums[2 * k][w] = t; sums[2 * k + 1][w] = b; }
    }
    {
        const double t = wave_sum((double)ssum);
        smin = wave_min(smin);
        smax = wave_max(smax);
        if (lane == 0) { sums[6][w] = t; sext[0][w] = smin; sext[1][w] = smax; }
    }
    __syncthreads();

    // ---- 4: exact thresholds in the lists (wavefront = list), the surprise's range and mean ----
    if (w < 6) {
        constexpr double kFix = 1099511627776.0;                      // 2^40: exact for fp32 values of magnitude <= 1 down to that step
        const int k = w >> 1;
        const bool low = (w & 1) != 0;
        const uint32_t n = cnt[w];
        uint32_t T, gt, eq;
        long long part = 0;
        double total;
        if (n <= (uint32_t)kUnitList) {
            const uint32_t *list = buf + w * kUnitList;
            T = wave_select(list, (int)n, need[w], whist[w], gt, eq);
            for (uint32_t i = lane; i < n; i += 64)
                part += list[i] > T ? __double2ll_rn((double)key_value(low ? ~list[i] : list[i]) * kFix) : 0ll;
            total = wave_sum(lane < NW ? sums[w][lane & (NW - 1)] : 0.0) + (double)(need[w] - gt) * (double)key_value(low ? ~T : T);
        } else {
            const float *x = a + k * rows;
            auto key_at = [x, low](int i) { return low ? ~ord_key(x[i]) : ord_key(x[i]); };
            T = wave_select_fn(N, m, whist[w], gt, eq, key_at);
            for (int i = lane; i < N; i += 64) part += key_at(i) > T ? __double2ll_rn((double)x[i] * kFix) : 0ll;
            total = (double)(m - gt) * (double)key_value(low ? ~T : T);
        }
        total += (double)wave_sum(part) / kFix;
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
    if (tid == 0) {
        float stats[12];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            stats[4 * k] = st.lo[k];
            stats[4 * k + 1] = st.inv_range[k];
            stats[4 * k + 2] = (float)((side[2 * k] - side[2 * k + 1]) / (double)m * (double)st.inv_range[k]);
        }
        head_weights(stats, lc, hs);
    }
    __syncthreads();

    // ---- 5: blend, gate, route, pin ----
    st = hs;
    float *out = scores + base;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const int i = tid + j * kSelThreads;
        if (i < N) {
            const float raw[3] = {v[0][j], v[1][j], v[2][j]};
            float at[3];
            normalised(raw, st, at);
            out[i] = i < lc.n_sink ? NKV_PIN : routed_score<ALL>(at, st, lc);
        }
    }
}

}  // namespace

hipError_t launch_finalize(const float *a_raw, int L, int H, const PromptTab &tab, const LearnerConsts &lc,
                           float *scores, float *stats, void *wide_ws, bool per_head_route, const Prof &prof,
                           hipStream_t st)
{
    int nmax = 0;
    for (int p = 0; p < tab.n; ++p) nmax = max(nmax, tab.tok_off[p + 1] - tab.tok_off[p]);
    const unsigned units = (unsigned)(tab.n * L * H);
    const int per_unit = kUnitTokens;                                 // prompts of up to this length: one launch, a workgroup per unit
    prof.begin(NKV_KERNEL_FINALIZE, st);
    if (nmax > per_unit) {
        if (wide_ws == nullptr || per_head_route) {
            finalize_kernel<<<units, kThreads, 0, st>>>(a_raw, L, H, tab, lc, scores);
        } else {
            hipError_t e = launch_stats_wide(a_raw, L, H, tab, lc.scale_mask, stats, wide_ws, st);
            if (e != hipSuccess) return e;
            e = launch_route_wide(a_raw, L, H, tab, lc, stats, wide_ws, scores, st);
            if (e != hipSuccess) return e;
        }
    } else {
        bool present[17] = {};
        for (int p = 0; p < tab.n; ++p) present[length_class(tab.tok_off[p + 1] - tab.tok_off[p])] = true;
#define NKV_UNIT(EPT)                                                                                                         \
    if (present[EPT])                                                                                                         \
    (lc.scale_mask == 7 ? finalize_unit_kernel<EPT, true> : finalize_unit_kernel<EPT, false>)<<<units, kSelThreads, 0, st>>>( \
        a_raw, L, H, tab, lc, scores)
        NKV_UNIT(4);
        NKV_UNIT(8);
        NKV_UNIT(16);
#undef NKV_UNIT
    }
    prof.end(NKV_KERNEL_FINALIZE, st);
    return hipGetLastError();
}

}  // namespace nkv
