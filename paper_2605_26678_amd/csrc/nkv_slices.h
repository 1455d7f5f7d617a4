// Slices: the unit of work of the kernels that spread a head's per-token values over the whole chip.
//
// A head's N values are cut into slices of 8192 tokens; a kernel that touches the values runs one workgroup of TH
// threads per slice (8192 / TH values per thread, element i of the slice in slot i / TH of thread i % TH, so
// every load instruction of a wavefront is one contiguous 256-byte piece).  TH is 256, four workgroups to a compute unit,
// or 1024 where there are too few slices to fill the chip: a slice is then done in a quarter of the time (see
// slice_threads).  Slices are numbered prompt by prompt; inside a prompt (layer * H + head)-major, so the slices of a head -- and of a layer -- are contiguous.
//
// Values are binned by a monotone map of the value into 2048 bins; a per-slice histogram is stored as 2048
// 16-bit counts.  Exact work happens only on the entries of one boundary bin, which every slice copies into
// its own segment of kSeg keys.
#pragma once

#include "nkv_wavesel.h"

namespace nkv {
namespace {

constexpr int kSlice = 8192;             // tokens per slice (the counts of a slice fit 16 bits)
constexpr int kBins = 2048;
// Threads of the kernels that take a slice a workgroup: the histograms, the budgets' and the selection's.  Up to two slices per compute unit
// workgroups of 1024 are all resident, and quicker; many slices keep the chip full either way, and the smaller workgroup has fewer
// wavefronts at its barriers.  Heads of 32768 tokens of bf16 keys, 256 threads / 1024, us: 32 slices budgets 26.9 / 24.8, selection with its
// gather 33.1 / 30.7; 256 slices 28.7 / 26.4 and 115.1 / 112.4; 512 29.5 / 28.7 and 207.7 / 205.7; 544 30.2 / 30.7 and 223.9 / 226.8; 1152 38.5 / 39.3
// and 453 / 461.  The score call, whose histograms alone are left, does not tell the two apart.
constexpr int kFewSlices = 512;
inline bool few_slices(int slices) { return slices <= kFewSlices; }
template <int TH> constexpr int per_thread() { return kSlice / TH; }
constexpr int kSeg = 256;                // keys one slice may contribute to a list

struct SliceTab {                        // first slice of every prompt; a prompt has L*H*S_p slices
    int32_t off[NKV_MAX_PROMPTS + 1];
};

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

inline int fill_slices(int L, int H, const PromptTab &tab, SliceTab *st)
{
    int n = 0;
    for (int p = 0; p < tab.n; ++p) {
        st->off[p] = n;
        const int N = tab.tok_off[p + 1] - tab.tok_off[p];
        n += L * H * ((N + kSlice - 1) / kSlice);
    }
    st->off[tab.n] = n;
    return n;
}

// slice id -> prompt, (layer*H + head), slice within the unit, slices per unit
__device__ __forceinline__ void locate(const SliceTab &st, const PromptTab &tab, int id, int &p, int &lh, int &s,
                                       int &S)
{
    p = 0;
    while (p + 1 < tab.n && id >= st.off[p + 1]) ++p;
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    S = (N + kSlice - 1) / kSlice;
    const int local = id - st.off[p];
    lh = local / S;
    s = local - lh * S;
}

// The values of slice s of a head of N tokens, as the hardware's bounds-checked buffer: slot j of thread tid is
// element j * TH + tid of the slice (one instruction of a wavefront reads one contiguous 256-byte piece, the
// address is a 32-bit register and a constant), and elements past the head's last token read as 0.  The whole
// offset goes into the per-lane offset, which the range check is sure to cover.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slice_values(const float *head, int s, int N)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(head + (int64_t)s * kSlice), 0,
                                             min(N - s * kSlice, kSlice) * 4, 0x00020000);
}

template <int TH> __device__ __forceinline__ float slice_value(__amdgpu_buffer_rsrc_t r, int tid, int j)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, tid * 4 + j * (TH * 4), 0, 0));
}

// Four consecutive values per thread and load, for kernels that do not care which thread holds which value
// (histograms, minima): slot j of thread tid holds elements 4 (j * TH + tid) .. + 3 of the slice.  The range check
// is per 32-bit word, so a head's last values are delivered and the words behind them read as 0.
template <int TH> __device__ __forceinline__ void slice_values4(__amdgpu_buffer_rsrc_t r, int tid, int j, float (&v)[4])
{
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(r, (j * TH + tid) * 16, 0, 0);
    v[0] = __uint_as_float(q[0]); v[1] = __uint_as_float(q[1]); v[2] = __uint_as_float(q[2]); v[3] = __uint_as_float(q[3]);
}

// Scores: floor(2046 v) for 0 <= v <= 1, 0 below, 2047 above 1 (the pinned positions).  Monotone in v.  (The histogram kernels are
// bound by the instructions they issue per value: a median of three clamps in one.)
__device__ __forceinline__ int score_bin(float v)
{
    return (int)__builtin_amdgcn_fmed3f(v * 2046.0f, 0.f, 2046.0f) + (v > 1.0f ? 1 : 0);
}

// Anomalies (-cos, so in [-1, 1]): floor(1023.5 (a + 1)), clamped.  Monotone in a.
__device__ __forceinline__ float anomaly_scaled(float a) { return (a + 1.0f) * 1023.5f; }
__device__ __forceinline__ int anomaly_bin(float a)
{
    return (int)__builtin_amdgcn_fmed3f(anomaly_scaled(a), 0.f, 2047.0f);
}

// Where y = a value on the scale of its bins lies to a boundary bin: bin > q <=> y >= above, bin < q <=> y < below, and what is neither is in
// bin q.  (Of kBins bins, the end ones take what lies beyond; q = -1: every value is above.)  A comparison each instead of
// forming the bin.
struct BinEdges {
    float above, below, from, to;        // from, to: the same edges from the other side (in bin q <=> y >= from and not y >= above)
};
__device__ __forceinline__ float bin_low_edge(int q) { return q <= 0 ? -INFINITY : (float)q; }
__device__ __forceinline__ float bin_high_edge(int q) { return q < 0 ? -INFINITY : q >= kBins - 1 ? INFINITY : (float)(q + 1); }
__device__ __forceinline__ BinEdges bin_edges(int q)                  // q: the same in every lane
{
    auto uniform = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
    const float low = uniform(bin_low_edge(q)), high = uniform(bin_high_edge(q));
    return BinEdges{high, low, low, high};
}

// The same for scores, whose upper two bins are those of 1 and of everything above (y is infinite for the pinned ones): in bin q <=>
// y >= from and not y >= above.  q = kBins: no value is.
__device__ __forceinline__ float score_scaled(float v) { return v * 2046.0f; }
__device__ __forceinline__ BinEdges score_edges(int q)               // q: the same in every lane
{
    auto uniform = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
    auto from = [](int b) { return b <= 0 ? -INFINITY : b <= 2046 ? (float)b : b == 2047 ? 2046.0001220703125f : NAN; };   // the float after 2046
    const float low = uniform(from(q)), high = uniform(from(q + 1));
    return BinEdges{high, low, low, high};
}

// The 2048 counts of a workgroup's LDS histogram as 16-bit values: 8 bins per thread and 16-byte store, by 256 threads.
__device__ __forceinline__ void store_hist16(const uint32_t *hist, uint16_t *row)
{
    if (threadIdx.x >= kBins / 8) return;
    const uint4 a = reinterpret_cast<const uint4 *>(hist)[2 * threadIdx.x], b = reinterpret_cast<const uint4 *>(hist)[2 * threadIdx.x + 1];
    reinterpret_cast<uint4 *>(row)[threadIdx.x] = make_uint4(a.x | (a.y << 16), a.z | (a.w << 16), b.x | (b.y << 16), b.z | (b.w << 16));
}

// Histogram of the scores of one slice.  grid: slices; part: [slices][kBins] 16-bit counts.
template <int TH>
__global__ __launch_bounds__(TH) void slice_hist_kernel(const float *__restrict__ scores, PromptTab tab, SliceTab st,
                                                        uint16_t *__restrict__ part)
{
    constexpr int PT = per_thread<TH>();
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins];
    int p, lh, s, S;
    locate(st, tab, blockIdx.x, p, lh, s, S);
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const float *sc = scores + (int64_t)lh * tab.T + tab.tok_off[p];
    const int tid = threadIdx.x;
    for (int j = tid; j < kBins; j += TH) hist[j] = 0u;
    float v[PT / 4][4];
    const __amdgpu_buffer_rsrc_t vals = slice_values(sc, s, N);
#pragma unroll
    for (int j = 0; j < PT / 4; ++j) slice_values4<TH>(vals, tid, j, v[j]);
    __syncthreads();
    if ((s + 1) * kSlice <= N) {
#pragma unroll
        for (int j = 0; j < PT / 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(&hist[score_bin(v[j][e])], 1u);
    } else {
#pragma unroll
        for (int j = 0; j < PT / 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (s * kSlice + 4 * (j * TH + tid) + e < N) atomicAdd(&hist[score_bin(v[j][e])], 1u);
    }
    __syncthreads();
    store_hist16(hist, part + (int64_t)blockIdx.x * kBins);
}

// Copies the lists of a unit's S slices (segment s: `count(s)` keys from seg + s * kSeg on) one behind the other to
// keys[0 .. cap), by one wavefront with the loads of the next four segments in flight, the first four's while the counts are
// on their way; returns the number of keys, or -1 if a segment or the list overflows.  before: keys of the slices in front of
// slice `own`.
template <typename F>
__device__ __forceinline__ int gather_segments(const uint32_t *__restrict__ seg, int S, F count, uint32_t *keys, int cap, int own,
                                               int &before)
{
    const int lane = threadIdx.x & 63;
    int n = 0;
    before = 0;
    uint32_t next[4];
    auto load = [&](int s0, int last) {
#pragma unroll
        for (int i = 0; i < 4; ++i) next[i] = seg[(int64_t)min(s0 + i, last) * kSeg + lane];
    };
    for (int s0 = 0; s0 < S; s0 += 64) {
        load(s0, S - 1);
        const uint32_t c = s0 + lane < S ? count(s0 + lane) : 0u;
        if (__any(c > (uint32_t)kSeg)) return -1;
        const uint32_t incl = wave_prefix_sum(c);
        const int total = __builtin_amdgcn_readlane((int)incl, 63);
        if (n + total > cap) return -1;
        const int off = n + (int)(incl - c);
        if (own >= s0 && own < s0 + 64) before = __builtin_amdgcn_readlane(off, own - s0);
        const int m = min(64, S - s0);
        for (int i0 = 0; i0 < m; i0 += 4) {
            const uint32_t first[4] = {next[0], next[1], next[2], next[3]};
            if (i0 + 4 < m) load(s0 + i0 + 4, S - 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i0 + i >= m) break;
                const int ci = __builtin_amdgcn_readlane((int)c, i0 + i), oi = __builtin_amdgcn_readlane(off, i0 + i);
                if (lane < ci) keys[oi + lane] = first[i];
                for (int j = lane + 64; j < ci; j += 64) keys[oi + j] = seg[(int64_t)(s0 + i0 + i) * kSeg + j];
            }
        }
        n += total;
    }
    return n;
}

}  // namespace
}  // namespace nkv
