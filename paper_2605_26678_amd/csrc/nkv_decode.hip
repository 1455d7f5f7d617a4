// Decode-side consumer of the compressed cache: one new token's attention over the rows the compression
// operator kept (paper Section 2.5 for the layout of the cache, Appendix A "Complexity": retained keys and
// values are unchanged, so ordinary attention applies; Section 3.5 reports the per-token decode latency).
//
// For unit u = (prompt, layer, KV head) and the G query heads that read it (grouped-query attention, query
// head j reads KV head j / G):   out_j = sum_i softmax_i(scale <q_j, k_i>) v_i   over the unit's rows.
//
// The work is one read of every retained K and V row, so it is bound by HBM.  A workgroup handles rows of one unit for all G
// query heads at once (K and V are read once, not G times).  Units have different lengths (head-wise budgets) that the host
// does not know, and what a workgroup spends on finding its rows, merging its lanes' results and waiting for its stores costs as much
// as 100 to 200 rows do, so large calls give every workgroup as many rows as there are for it:
//   decode_run_kernel     : stretches of the cache of the same length, one for every workgroup the device holds, across the units' ends
//   decode_piece_kernel   : pieces of 256 rows of a unit where units are short, of 64 rows where there are few
//   decode_combine_kernel : per (unit, query head) merges the partial results: per query head running maximum, sum, weighted values
//                           (m, l, o[0..D)) of a running-maximum softmax in base 2
// All three work out from head_off which unit a piece belongs to: no kernel plans in front.  As chunks of 256 rows that a kernel of
// its own numbered, 288 units of 8192 rows, head dim 128, G = 4, took 217 us (chunk kernel 5.9 TB/s, planning 4 us), now 205; 288 units of
// 615 rows 27.6 and 25.4; 64 units of 768 rows, G = 8 18.9 and 16.9.  Reading the same rows without arithmetic or merging takes 179.
// Lane layout in attend as in the scoring kernel: a row is spread over D/8 lanes (16 bytes each),
// one wave load fetches 64/(D/8) rows; <q, k> uses the packed 16-bit dot instruction on the stored bits (exact
// products, fp32 accumulation) and a DPP sum over the lanes of a row; every group of D/8 lanes keeps its own
// running (m, l, o) for the rows it sees, rescaled once per batch of four rows, and the groups and waves are
// merged through LDS at the end.
// Anything outside bf16 / fp16 with d = dv in {64, 128} and G <= 8 goes to decode_generic_kernel (one workgroup per
// unit and query head, no scratch).
#include "nkv_device.h"

#include <algorithm>
#include <type_traits>

namespace nkv {
namespace {

// Rows per workgroup: 256, or 64 where a call has too few rows to fill the chip with workgroups of 256 (a wavefront then
// has one batch of rows instead of four in turn).
constexpr int kChunk = 256, kSmallChunk = 64, kSmallUnits = 256;
constexpr int kUnitCost = 128;           // a unit's own work in a stretch, in rows
constexpr int kLeastRun = 192;           // rows of a stretch at least
// Chunks per unit from which 512 threads combine them instead of one per dimension (64 units of G = 3, head dim 64: 7 chunks a
// unit 8.0 -> 7.1 us; 256 units of G = 8, 300 rows in two chunks 21.4 us with 512, 19.4 with 64).
// Stretches have 256 at least: one unit may hold nearly all rows (511 units of one row beside one of 600 000, head dim 64, G = 3 100 us with 64
// threads, 52 with 256; 288 units of 750, G = 8 29.5 and 31.2).
constexpr int kManyChunks = 4;
constexpr int kDecThreads = 256;
constexpr float kNone = -1.0e30f;        // running maximum before any row was seen
constexpr float kLn2 = 0.6931471805599453f;

using u32x4 = unsigned int __attribute__((ext_vector_type(4)));

template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int LPR> __device__ __forceinline__ float group_sum(float v)
{
    v = dpp_add<0xB1>(v);                        // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);                        // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);                       // row_half_mirror
    if (LPR == 16) v = dpp_add<0x140>(v);        // row_mirror
    return v;
}

// <a, b> over the eight bf16 pairs of two packed 16-byte pieces.  The compiler does not see the register
// write inside the assembly, so the wait states a DPP read of the result needs are spent here.
// F16: the sixteen-bit values are fp16 instead of bf16 (the only two places that know).
template <bool F16> __device__ __forceinline__ float dot8_for_dpp(const u32x4 &a, const u32x4 &b)
{
    float acc = 0.f;
    if constexpr (F16)
        asm("v_dot2c_f32_f16 %0, %1, %5\n\t"
            "v_dot2c_f32_f16 %0, %2, %6\n\t"
            "v_dot2c_f32_f16 %0, %3, %7\n\t"
            "v_dot2c_f32_f16 %0, %4, %8\n\t"
            "s_nop 1"
            : "+v"(acc)
            : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w));
    else
        asm("v_dot2c_f32_bf16 %0, %1, %5\n\t"
            "v_dot2c_f32_bf16 %0, %2, %6\n\t"
            "v_dot2c_f32_bf16 %0, %3, %7\n\t"
            "v_dot2c_f32_bf16 %0, %4, %8\n\t"
            "s_nop 1"
            : "+v"(acc)
            : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w));
    return acc;
}

template <bool F16> __device__ __forceinline__ void unpack2(uint32_t r, float (&v)[2])
{
    if constexpr (F16) {
        using f16x2 = _Float16 __attribute__((ext_vector_type(2)));
        const f16x2 x = __builtin_bit_cast(f16x2, r);
        v[0] = (float)x.x;
        v[1] = (float)x.y;
    } else {
        v[0] = __uint_as_float(r << 16);
        v[1] = __uint_as_float(r & 0xffff0000u);
    }
}

__host__ __device__ inline int64_t divide(int64_t a, int64_t b)      // for a >= 0, b > 0; in 32 bits where they do
{
    return (a | b) >> 32 == 0 ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

// How many stretches `rows` rows (with kUnitCost rows for every unit) are cut into, and how long they are.  Up to four for every workgroup
// that the device holds, of 1024 rows and more: what runs at a time lies closer together then, and the first pass over a cache spends less on
// address translation (288
// units of 8192 rows, G = 4, first pass / later ones, one stretch: 262 / 196 us, two 243 / 199, four 233 / 203, eight 230 / 209; pieces of 256
// rows 245 / 217).  Of 512 rows and more instead: 384 units of 3518 rows, head dim 128, G = 4 122.8 us and 115.6, G = 8 181.7 and 168.9.
__host__ __device__ inline int64_t stretch_count(int64_t rows, int resident)
{
    const int64_t each = divide(rows, (int64_t)1024 * resident);
    return (each < 1 ? 1 : each > 4 ? 4 : each) * resident;
}
constexpr int64_t kMostRun = 1 << 20;
__host__ __device__ inline int64_t stretch_rows(int64_t rows, int resident)
{
    const int64_t n = stretch_count(rows, resident), per = (divide(rows + n - 1, n) + 15) / 16 * 16;
    return per < kLeastRun ? kLeastRun : per > kMostRun ? kMostRun : per;
}

__device__ __forceinline__ int64_t clamp_row(int64_t r, int64_t rows) { return r < 0 ? 0 : (r > rows ? rows : r); }

// One workgroup's pass over the n >= 1 rows of a unit from row r0 on, for the G heads whose queries start at q: D + 2 floats a head to
// part: running maximum (base-2 logits), sum of weights, weighted values.  A wavefront takes U loads of rows at a time, the four
// wavefronts in turn.  MOST: n is no larger (0: any n).
// Measured instead, in pieces of 256 rows: the next batch's rows asked for as soon as a batch's are used up, and the lane groups merged in
// registers (permlane swaps) in front of the waves.  The registers that this holds cost waves: whole calls of 2 359 296 rows, us without and
// that way, head dim 128 G = 3 213 / 210, 4 220 / 219, 6 253 / 277, 8 326 / 326; head dim 64 G = 3 105 / 103, 4 112 / 119,
// 6 144 / 162, 8 192 / 212; small calls 11.0 / 11.2.
template <int D, int G, bool F16, int MOST>
__device__ __forceinline__ void attend(const uint16_t *__restrict__ q, const uint16_t *__restrict__ pk, const uint16_t *__restrict__ pv,
                                       int64_t r0, int n, float scale_log2, float *__restrict__ part)
{
    constexpr int LPR = D / 8, RPW = 64 / LPR, NW = kDecThreads / 64;
    constexpr int U = MOST > 0 && MOST < 4 * NW * RPW ? MOST / (NW * RPW) : 4;
    constexpr int STRETCH = U * RPW, STEP = NW * STRETCH;            // rows of a wavefront at a time, of the workgroup
    constexpr int kRowBytes = D * 2;
    __shared__ float lds_m[NW * RPW][G], lds_l[NW * RPW][G];
    __shared__ float lds_o[NW * RPW][G][D];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, gi = lane / LPR, c = lane % LPR;
    u32x4 qv[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
        qv[g] = *reinterpret_cast<const u32x4 *>(q + (int64_t)g * D + c * 8);

    float m[G], l[G], o[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = kNone;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = 0.f;
    }
    // rows past the end of the run read as zeros and get weight 0
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(pk) + r0 * D, 0,
                                                                         n * kRowBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(pv) + r0 * D, 0,
                                                                         n * kRowBytes, 0x00020000);
    {
#pragma unroll 1
        for (int at = w * STRETCH; at < n; at += STEP) {             // uniform in the wave
            const int row0 = at + gi;                                // this lane group's row in the first load
            u32x4 kr[U], vr[U];
#pragma unroll
            for (int i = 0; i < U; ++i)
                kr[i] = __builtin_amdgcn_raw_buffer_load_b128(krs, (row0 + i * RPW) * kRowBytes + c * 16, 0, 2);   // aux 2: non-temporal
#pragma unroll
            for (int i = 0; i < U; ++i)
                vr[i] = __builtin_amdgcn_raw_buffer_load_b128(vrs, (row0 + i * RPW) * kRowBytes + c * 16, 0, 2);
            float s[U][G];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const bool valid = row0 + i * RPW < n;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float d = group_sum<LPR>(dot8_for_dpp<F16>(kr[i], qv[g]));
                    s[i][g] = valid ? d * scale_log2 : kNone;
                }
            }
            // Long sums (MOST = 0): a batch's terms are added up by themselves, then to what there was before: as many instructions as
            // one by one and a quarter of the roundings (error of the output, 288 units of 8192 rows, G = 4, in 1e-7: 2.6, one by one 3.3,
            // one by one in pieces of 256 rows 2.8).  Of pieces, calls of G = 5 to 8 would take 4 % longer that way.
            constexpr bool BATCH = MOST == 0;
            float p[U][G], corr[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float mb = m[g];
#pragma unroll
                for (int i = 0; i < U; ++i) mb = fmaxf(mb, s[i][g]);
                corr[g] = __builtin_amdgcn_exp2f(m[g] - mb);         // 1 if nothing changed, 0 from kNone
                m[g] = mb;
                float lb = 0.f;
                if (!BATCH) {
                    l[g] *= corr[g];
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[g][e] *= corr[g];
                }
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    p[i][g] = row0 + i * RPW < n ? __builtin_amdgcn_exp2f(s[i][g] - mb) : 0.f;
                    if (BATCH) lb = i == 0 ? p[i][g] : lb + p[i][g];
                    else l[g] += p[i][g];
                }
                if (BATCH) l[g] = fmaf(l[g], corr[g], lb);
            }
            if constexpr (!BATCH) {
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; e += 2) unpack2<F16>(vr[i][e / 2], *reinterpret_cast<float (*)[2]>(&v[e]));
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[g][e] = fmaf(p[i][g], v[e], o[g][e]);
                }
                if (MOST == STEP) break;                             // (and no loop)
                continue;
            }
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                float v[U][2];
#pragma unroll
                for (int i = 0; i < U; ++i) unpack2<F16>(vr[i][e / 2], v[i]);
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        float t = p[0][g] * v[0][h];
#pragma unroll
                        for (int i = 1; i < U; ++i) t = fmaf(p[i][g], v[i][h], t);
                        o[g][e + h] = fmaf(o[g][e + h], corr[g], t);
                    }
            }
        }
    }
    // ---- merge the lane groups and waves of the workgroup ----
    const int slot = w * RPW + gi;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (c == 0) {
            lds_m[slot][g] = m[g];
            lds_l[slot][g] = l[g];
        }
        *reinterpret_cast<float4 *>(&lds_o[slot][g][c * 8]) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
        *reinterpret_cast<float4 *>(&lds_o[slot][g][c * 8 + 4]) = make_float4(o[g][4], o[g][5], o[g][6], o[g][7]);
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < G * D; idx += kDecThreads) {
        const int g = idx / D, e = idx - g * D;
        float mm = kNone;
#pragma unroll
        for (int sl = 0; sl < NW * RPW; ++sl) mm = fmaxf(mm, lds_m[sl][g]);
        float ll = 0.f, oo = 0.f;
#pragma unroll
        for (int wv = 0; wv < NW; ++wv) {
            // a wavefront's lane groups first, shorter chains of additions: relative error of the output 2.49e-7 -> 2.34e-7 (head dim 64,
            // G = 8), 1.81e-7 -> 1.69e-7 (128, 3), 2.69e-7 -> 2.58e-7 (128, 6), in the same time
            float lw = 0.f, ow = 0.f;
#pragma unroll
            for (int sl = wv * RPW; sl < wv * RPW + RPW; ++sl) {
                const float f = __builtin_amdgcn_exp2f(lds_m[sl][g] - mm);
                lw = fmaf(f, lds_l[sl][g], lw);
                ow = fmaf(f, lds_o[sl][g][e], ow);
            }
            ll += lw;
            oo += ow;
        }
        float *dst = part + g * (D + 2);
        if (e == 0) {
            dst[0] = mm;
            dst[1] = ll;
        }
        dst[2 + e] = oo;
    }
}

// x, which is the same in every lane, in scalar registers (64-bit comparisons are made in vector registers).
__device__ __forceinline__ int64_t uniform(int64_t x)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t of_lane(int64_t x, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}

struct Piece {
    int unit, k;                         // the unit's k-th piece; unit < 0: there are fewer pieces
    int64_t first, end;                  // the unit's rows
};

// Piece i of all units' pieces of CH rows.  Up to 64 units every wavefront counts them by itself, up to PER * kDecThreads the workgroup.
template <int CH>
__device__ __forceinline__ Piece counted_by_wave(const int64_t *__restrict__ head_off, int n_units, int64_t rows, uint32_t i)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t from = clamp_row(head_off[min(lane, n_units)], rows), to = clamp_row(head_off[min(lane + 1, n_units)], rows);
    const uint32_t c = (uint32_t)((max(to - from, (int64_t)0) + CH - 1) / CH), at = i - (wave_prefix_sum(c) - c);
    const unsigned long long here = __ballot(at < c);
    if (here == 0ull) return Piece{-1, 0, 0, 0};
    const int u = __builtin_ctzll(here);
    return Piece{u, __builtin_amdgcn_readlane((int)at, u), of_lane(from, u), of_lane(to, u)};
}
template <int CH, int PER>
__device__ __forceinline__ Piece counted_by_workgroup(const int64_t *__restrict__ head_off, int n_units, int64_t rows, uint32_t piece)
{
    constexpr int NW = kDecThreads / 64;
    __shared__ uint32_t wsum[NW];
    __shared__ Piece found;
    const int tid = threadIdx.x, w = tid >> 6, u0 = tid * PER;
    uint32_t c[PER], mine = 0u;
    int64_t off[PER + 1];
#pragma unroll
    for (int i = 0; i <= PER; ++i) off[i] = clamp_row(head_off[min(u0 + i, n_units)], rows);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = (uint32_t)((max(off[i + 1] - off[i], (int64_t)0) + CH - 1) / CH);
        mine += c[i];
    }
    const uint32_t incl = wave_prefix_sum(mine);
    if ((tid & 63) == 63) wsum[w] = incl;
    if (tid == 0) found.unit = -1;
    __syncthreads();
    uint32_t at = piece - (incl - mine);                              // from this thread's first piece on
#pragma unroll
    for (int i = 0; i < NW - 1; ++i) at -= i < w ? wsum[i] : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (at < c[i]) found = Piece{u0 + i, (int)at, off[i], off[i + 1]};
        at -= c[i];
    }
    __syncthreads();
    return Piece{__builtin_amdgcn_readfirstlane(found.unit), __builtin_amdgcn_readfirstlane(found.k), uniform(found.first), uniform(found.end)};
}

// Pieces of CH rows of a unit, the first from its first row on.  Their partial results are numbered from off[u] / CH + u on, which leaves
// room for all of them and needs no plan.  Workgroups take the pieces that there are, one after the other; more units than a workgroup
// can count in less time than its rows take (2048 of them, G = 4 61 us, 68 with 16 units a thread) leave it with the numbers' pieces, some
// of which are empty.  Empty ones in between would take the place of others, which then share a compute unit: 8 units of 8192 rows, head dim
// 128, G = 8 24.0 us by numbers, 18.4 counted.  And workgroups go to the eight XCDs in turn, so what recurs every two, four or eight pieces,
// empty ones or a unit's short last one, would be the same XCDs' share: every eight are dealt out one place further on than the eight
// before, and every 64 another one.  By numbers in their order / this way: 1024 units of 256 rows, every other number empty, 79 / 48 us; 512 of
// 768, every fourth, 78 / 62; 4096 of 256 288 / 175; 1024 of 300 68 / 69, counted but not dealt out 79.
// grid: as many numbers as there are.
template <int D, int G, bool F16, int CH>
__global__ __launch_bounds__(kDecThreads) void decode_piece_kernel(const uint16_t *__restrict__ q, const uint16_t *__restrict__ pk,
                                                                   const uint16_t *__restrict__ pv, const int64_t *__restrict__ head_off,
                                                                   int n_units, int64_t rows, float scale_log2, float *__restrict__ part)
{
    const uint32_t eight = blockIdx.x / 8u;
    const uint32_t i = (blockIdx.x | 7u) < gridDim.x ? eight * 8u + ((blockIdx.x + eight + eight / 8u) & 7u) : blockIdx.x;
    Piece p;
    if (n_units <= kWave) p = counted_by_wave<CH>(head_off, n_units, rows, i);
    else if (CH == kSmallChunk || n_units <= kDecThreads) p = counted_by_workgroup<CH, 1>(head_off, n_units, rows, i);   // (kSmallUnits)
    else if (n_units <= 4 * kDecThreads) p = counted_by_workgroup<CH, 4>(head_off, n_units, rows, i);
    else {
        p.unit = __builtin_amdgcn_readfirstlane(wave_search_fn(n_units, (int64_t)i, [&](int u) { return u == 0 ? (int64_t)0 : clamp_row(head_off[u], rows) / CH + u; }));
        p.first = clamp_row(head_off[p.unit], rows);
        p.end = clamp_row(head_off[p.unit + 1], rows);
        p.k = (int)((int64_t)i - p.unit - p.first / CH);
    }
    if (p.unit < 0) return;
    const int64_t a = p.first + (int64_t)p.k * CH, b = min(p.end, a + CH);
    if (p.first <= a && a < b)
        attend<D, G, F16, CH>(q + (int64_t)p.unit * G * D, pk, pv, a, (int)(b - a), scale_log2, part + (p.first / CH + p.unit + p.k) * G * (D + 2));
}
static_assert(kSmallUnits <= kDecThreads, "a thread counts one unit's pieces of 64 rows");

// The rows of all units, one unit after the other, each with kUnitCost rows in front for its queries, its merge and its stores, in
// stretches of `run`.  (Cut by rows alone, a stretch of short units took many of them in turn: 288 units of 26 rows beside 288 of 6554,
// head dim 64, G = 3 134 us, 84 this way, about the same with 64, 96 or 192 rows a unit; chunks of 256 rows 92; 511 units of one row beside one of
// 600 000, head dim 128, G = 8 2640, 126 and 175.)  Their length follows from the rows that there are, which the
// host does not know: a buffer may hold room for many more.  (288 units in buffers of 2 359 296 rows, stretches as for full ones / as they
// are / chunks of 256 rows as it was: head dim 128, G = 4, 147 456 rows 28.6 / 25.7 / 25.9 us, 18 432 rows 43.5 / 19.1 / 16.5; head dim 64,
// G = 8, 38.3 / 30.6 / 28.0 and 100 / 27 / 18.)
struct Stretches {
    const int64_t *head_off;
    int64_t rows, base, len, run;
    __device__ Stretches(const int64_t *off, int n_units, int64_t rows_, int resident) : head_off(off), rows(rows_)
    {
        base = clamp_row(off[0], rows);
        len = max(clamp_row(off[n_units], rows) - base, (int64_t)0) + (int64_t)kUnitCost * n_units;
        run = stretch_rows(len, resident);
    }
    __device__ int64_t first(int u) const { return clamp_row(head_off[u], rows); }
    __device__ int64_t pos(int u) const { return first(u) - base + (int64_t)kUnitCost * u; }
};

// Long units: the cache is cut into stretches, whichever units they belong to, so that every workgroup of the call has
// the same work.  What stretch i holds of unit u is piece i + u (no two share a number: both grow with the row).  grid: stretches, or more.
// (Two workgroups a compute unit: left to itself the compiler takes registers for one with fp16 and G = 8, 288 units of 1438 rows 93 us instead of 66.)
template <int D, int G, bool F16>
__global__ __launch_bounds__(kDecThreads, 2) void decode_run_kernel(const uint16_t *__restrict__ q, const uint16_t *__restrict__ pk,
                                                                 const uint16_t *__restrict__ pv, const int64_t *__restrict__ head_off,
                                                                 int n_units, int64_t rows, int resident, float scale_log2,
                                                                 float *__restrict__ part)
{
    const Stretches st(head_off, n_units, rows, resident);
    const int64_t lo = uniform(blockIdx.x * st.run), hi = uniform(min(lo + st.run, st.len));
    if (lo >= hi) return;
    const int64_t base = uniform(st.base);
    int u = __builtin_amdgcn_readfirstlane(wave_search_fn(n_units, lo, [&](int i) { return st.pos(i); }));
    int64_t first = uniform(st.first(u));
    for (; u < n_units; ++u) {
        const int64_t next = uniform(st.first(u + 1)), at = first - base + (int64_t)kUnitCost * (u + 1);   // of its first row
        const int64_t a = uniform(first + max(lo - at, (int64_t)0)), n = uniform(min(next, first + hi - at) - a);
        if (n > 0) attend<D, G, F16, 0>(q + (int64_t)u * G * D, pk, pv, a, (int)n, scale_log2, part + ((int64_t)blockIdx.x + u) * G * (D + 2));
        if (next - base + (int64_t)kUnitCost * (u + 1) >= hi) break;
        first = next;
        __syncthreads();                                              // (the merge's memory is used anew)
    }
}

// Where the partial results of unit u lie: [x, y).  resident > 0: of stretches; else of pieces of `piece` rows of a unit.  limit: there are
// no more (offsets that do not ascend are not read beyond it).
__device__ __forceinline__ int2 unit_pieces(const int64_t *head_off, int n_units, int u, int64_t rows, int resident, int piece, int limit)
{
    int64_t x, y;
    if (resident > 0) {
        const Stretches st(head_off, n_units, rows, resident);
        const int64_t at = max(st.pos(u), (int64_t)0) + kUnitCost, n = st.first(u + 1) - st.first(u);
        x = divide(at, st.run) + u;
        y = n > 0 ? divide(at + n - 1, st.run) + u + 1 : x;
    } else {
        const int64_t a = clamp_row(head_off[u], rows), n = clamp_row(head_off[u + 1], rows) - a;
        const int shift = __builtin_ctz(piece);                       // (a power of two)
        x = (a >> shift) + u;
        y = n > 0 ? x + ((n + piece - 1) >> shift) : x;
    }
    return make_int2((int)min(x, (int64_t)limit), (int)min(y, (int64_t)limit));
}

// grid: n_units * G workgroups of TH threads: TH / D slices of the unit's chunks, added up in the slices' order.
template <int D, int TH>
__global__ __launch_bounds__(TH) void decode_combine_kernel(const float *__restrict__ part, const int64_t *__restrict__ head_off,
                                                            int n_units, int64_t rows, int resident, int piece, int limit, int G, float *__restrict__ out,
                                                            float *__restrict__ lse)
{
    constexpr int NS = TH / D, NW = TH / 64, U = 4;
    __shared__ float red[NW];
    __shared__ float lds_l[NS], lds_o[NS][D];
    const int u = blockIdx.x / G, g = blockIdx.x - u * G, tid = threadIdx.x, e = tid % D, sl = tid / D;
    // a unit of four or so pieces of stretches takes one slice: the other threads only meet it at the barriers
    bool few = false;
    if (NS > 1 && resident > 0) {
        const int64_t len = clamp_row(head_off[n_units], rows) - clamp_row(head_off[0], rows) + (int64_t)kUnitCost * n_units;
        few = (clamp_row(head_off[u + 1], rows) - clamp_row(head_off[u], rows)) * resident <= 4 * len;
    }
    const int slices = few ? 1 : NS;
    const bool works = sl < slices;
    float mm = kNone, ll = 0.f, oo = 0.f;
    int c0 = 0, c1 = 0;
    if (works) {
        const int2 pieces = unit_pieces(head_off, n_units, u, rows, resident, piece, limit);
        c0 = pieces.x, c1 = pieces.y;
        // the largest running maximum: chunks spread over the threads, then one reduction
        for (int ch = c0 + tid; ch < c1; ch += slices * D) mm = fmaxf(mm, part[((int64_t)ch * G + g) * (D + 2)]);
        mm = wave_max(mm);
    }
    if ((tid & 63) == 0) red[tid >> 6] = mm;
    __syncthreads();
    if (works) {
#pragma unroll
        for (int i = 0; i < NW; ++i) mm = fmaxf(mm, red[i]);
        // weighted sums, four chunks' loads in flight at a time; the order of the additions is fixed
        for (int ch = c0 + sl; ch < c1; ch += U * slices) {
            float pm[U], pl[U], po[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const float *src = part + ((int64_t)min(ch + i * slices, c1 - 1) * G + g) * (D + 2);
                pm[i] = src[0];
                pl[i] = src[1];
                po[i] = src[2 + e];
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                if (ch + i * slices < c1) {
                    const float f = __builtin_amdgcn_exp2f(pm[i] - mm);
                    ll = fmaf(f, pl[i], ll);
                    oo = fmaf(f, po[i], oo);
                }
            }
        }
        lds_o[sl][e] = oo;
        if (e == 0) lds_l[sl] = ll;
    }
    __syncthreads();
    if (sl > 0) return;
    for (int i = 1; i < slices; ++i) {
        oo += lds_o[i][e];
        ll += lds_l[i];
    }
    out[((int64_t)u * G + g) * D + e] = ll > 0.f ? oo / ll : 0.f;
    if (lse && e == 0) lse[(int64_t)u * G + g] = ll > 0.f ? (mm + log2f(ll)) * kLn2 : -INFINITY;
}

// Any dtype, d, dv and group size.  grid: n_units * G workgroups of 256 threads; wave w takes rows w, w+4, ...;
// lane owns dims lane, lane + 64, ... of the key (dot) and of the value (accumulation).
template <typename T, int NQ>
__global__ __launch_bounds__(kDecThreads) void decode_generic_kernel(const T *__restrict__ q, const T *__restrict__ pk,
                                                                     const T *__restrict__ pv,
                                                                     const int64_t *__restrict__ head_off, int G,
                                                                     int d, int dv, int64_t rows, float scale_log2,
                                                                     float *__restrict__ out, float *__restrict__ lse)
{
    constexpr int NW = kDecThreads / 64;
    __shared__ float lds_m[NW], lds_l[NW];
    __shared__ float lds_o[NW][NQ * 64];
    const int u = blockIdx.x / G, g = blockIdx.x - u * G;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t first = clamp_row(head_off[u], rows), len = max(clamp_row(head_off[u + 1], rows) - first, (int64_t)0);
    const T *qj = q + ((int64_t)u * G + g) * d;
    float m = kNone, l = 0.f, acc[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.f;
    for (int64_t i = w; i < len; i += NW) {
        const T *kr = pk + (first + i) * d;
        float dot = 0.f;
        for (int cc = lane; cc < d; cc += 64) dot = fmaf(load_elem<T>(qj + cc), load_elem<T>(kr + cc), dot);
        const float s = wave_sum(dot) * scale_log2;
        const float mb = fmaxf(m, s), corr = __builtin_amdgcn_exp2f(m - mb), p = __builtin_amdgcn_exp2f(s - mb);
        m = mb;
        l = fmaf(l, corr, p);
        const T *vr = pv + (first + i) * dv;
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int cc = lane + 64 * k;
            acc[k] = fmaf(acc[k], corr, cc < dv ? p * load_elem<T>(vr + cc) : 0.f);
        }
    }
    if (lane == 0) {
        lds_m[w] = m;
        lds_l[w] = l;
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) lds_o[w][lane + 64 * k] = acc[k];
    __syncthreads();
    float mm = kNone;
    for (int i = 0; i < NW; ++i) mm = fmaxf(mm, lds_m[i]);
    float ll = 0.f;
    for (int i = 0; i < NW; ++i) ll = fmaf(__builtin_amdgcn_exp2f(lds_m[i] - mm), lds_l[i], ll);
    for (int e = threadIdx.x; e < dv; e += kDecThreads) {
        float oo = 0.f;
        for (int i = 0; i < NW; ++i) oo = fmaf(__builtin_amdgcn_exp2f(lds_m[i] - mm), lds_o[i][e], oo);
        out[((int64_t)u * G + g) * dv + e] = ll > 0.f ? oo / ll : 0.f;
    }
    if (lse && threadIdx.x == 0) lse[(int64_t)u * G + g] = ll > 0.f ? (mm + log2f(ll)) * kLn2 : -INFINITY;
}

int64_t max_chunks(int64_t n_units, int64_t rows, int chunk) { return rows / chunk + n_units; }

// Chunks of 64 rows where there are few units, at most two chunks of 256 rows per compute unit, and no more of 64 rows than
// the chip holds at once (what a chunk merges, 16 or 32 partial results of G heads, takes 8 KB of LDS a head), if the caller's
// scratch holds their partial results (it need not, see decode_ws_bytes).  128 units of G = 8, head dim 128, 700 rows: 34 us with
// 1528 chunks of 64 rows, 27 with 478 of 256; 64 units: 19.7 with 704 of 64, 20.4 with 256 rows; 64 units of 300 rows 13 against 20.
// (Those figures are from before the planning kernel went: 2 to 4 us less for 256 rows, up to 0.8 for 64.)
int64_t small_chunks_limit(int G) { return 256 * std::min(8, 160 * 1024 / (8448 * G + 1032)); }
bool decode_small(int64_t n_units, int64_t rows, int G)
{
    return n_units <= kSmallUnits && max_chunks(n_units, rows, kChunk) <= 512 && max_chunks(n_units, rows, kSmallChunk) <= small_chunks_limit(G);
}

// (The units' words in front of the partial results are room that is not used: sizes that were asked for once stay what they are.)
size_t part_offset(int64_t n_units) { return ((size_t)(n_units + 1) * 4 + 255) / 256 * 256; }
size_t ws_for(int64_t chunks, int64_t n_units, int G, int d) { return part_offset(n_units) + (size_t)chunks * G * (d + 2) * 4; }

// Workgroups of decode_run_kernel that the device holds at once, by the registers it takes (the compiler's report), a wavefront of each
// workgroup to a SIMD: 64 and 97 for G = 1 and head dim 128 and 64, 101 to 109 for G = 2, 126 to 157 for 3 to 5, 207 to 255 from 6 on.  A
// table, not a question to the runtime: a call asks nothing and keeps nothing, also the first one of a process and one being captured.
constexpr int resident_workgroups(int D, int G) { return 256 * (G == 1 ? (D == 128 ? 8 : 4) : G == 2 ? 4 : G <= 5 ? 3 : 2); }

// Stretches where every workgroup that the device holds gets 256 rows and more, and the units have more than three pieces in the mean (four
// where there are many).  Whole calls, chunks of 256 rows with a planning kernel in front (as it was) / pieces / stretches, us: 288 units
// of 8192 rows, head dim 128, G = 1 201 / 205 / 190, 4 217 / 222 / 202, 8 323 / 325 / 276, head dim 64, G = 8 192 / 190 / 155; 288 units of
// 512 rows, 128, G = 8 36.4 / 34.3 / 37.5, 64, G = 8 24.4 / 22.2 / 26.5, of 700 43.8 / 40.3 / 44.5 and 29.3 / 27.1 / 30.1, of 768 43.9 / 43.0 / 44.6 and
// 29.6 / 27.5 / 28.7, of 800 55.4 / 50.3 / 46.1 and 37.1 / 34.5 / 31.2; 456 units, 128, G = 5, of 700 42.0 / 39.1 / 41.9, of 800 54.2 / 50.2 / 45.6.  (Held
// to the registers of a third workgroup, G = 6 takes 10 to 20 % longer: rows spilled in the loop.)
bool by_stretches(int64_t n_units, int64_t rows, int resident)
{
    return rows >= (int64_t)kChunk * resident && (rows >= 1024 * n_units || (rows > 3 * kChunk * n_units && 5 * n_units <= 3 * (int64_t)resident));
}
// The stretches of a call that fills its buffer; one with fewer rows has no more.  (No more than pieces of 256 rows, for whose partial
// results every caller's scratch has room: where there are stretches, resident <= rows / 256 and kUnitCost * n_units <= rows / 3.)
unsigned most_stretches(int64_t n_units, int64_t rows, int resident)
{
    const int64_t len = rows + kUnitCost * n_units;
    return (unsigned)std::max(stretch_count(len, resident), len / kMostRun + 1);
}

template <int D, bool F16>
hipError_t run_fast(const uint16_t *q, const uint16_t *pk, const uint16_t *pv, const int64_t *head_off, int n_units,
                    int G, int64_t rows, float scale_log2, float *out, float *lse, void *ws, size_t ws_bytes, const Prof &prof,
                    hipStream_t st)
{
    float *part = (float *)((char *)ws + part_offset(n_units));
    const bool small = decode_small(n_units, rows, G) && ws_bytes >= ws_for(max_chunks(n_units, rows, kSmallChunk), n_units, G, D);
    const int piece = small ? kSmallChunk : kChunk;
    int64_t pieces = max_chunks(n_units, rows, piece);
    int in_stretches = 0;
    prof.begin(NKV_KERNEL_DECODE, st);
    auto go = [&](auto heads) {
        constexpr int GG = decltype(heads)::value, resident = resident_workgroups(D, GG);
        if (!small && by_stretches(n_units, rows, resident)) {
            const unsigned stretches = most_stretches(n_units, rows, resident);
            in_stretches = resident;
            pieces = (int64_t)stretches + n_units;
            decode_run_kernel<D, GG, F16><<<stretches, kDecThreads, 0, st>>>(q, pk, pv, head_off, n_units, rows, resident, scale_log2, part);
        } else {
            (small ? decode_piece_kernel<D, GG, F16, kSmallChunk> : decode_piece_kernel<D, GG, F16, kChunk>)<<<(unsigned)pieces, kDecThreads, 0, st>>>(
                q, pk, pv, head_off, n_units, rows, scale_log2, part);
        }
    };
    switch (G) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    case 8: go(std::integral_constant<int, 8>{}); break;
    default: return hipErrorInvalidValue;
    }
    prof.end(NKV_KERNEL_DECODE, st);
    const bool many = pieces > (int64_t)kManyChunks * n_units;
    (many ? decode_combine_kernel<D, 512> : in_stretches > 0 ? decode_combine_kernel<D, 256> : decode_combine_kernel<D, D>)
        <<<(unsigned)(n_units * G), many ? 512 : in_stretches > 0 ? 256 : D, 0, st>>>(part, head_off, n_units, rows, in_stretches, piece, (int)pieces, G, out, lse);
    return hipGetLastError();
}

template <typename T>
hipError_t run_generic(const T *q, const T *pk, const T *pv, const int64_t *head_off, int n_units, int G, int d,
                       int dv, int64_t rows, float scale_log2, float *out, float *lse, const Prof &prof,
                       hipStream_t st)
{
    const unsigned groups = (unsigned)(n_units * G);
    const int nq = (dv + 63) / 64;
    prof.begin(NKV_KERNEL_DECODE, st);
#define NKV_DECG(NQ) \
    decode_generic_kernel<T, NQ><<<groups, kDecThreads, 0, st>>>(q, pk, pv, head_off, G, d, dv, rows, scale_log2, out, lse)
    if (nq <= 1) NKV_DECG(1);
    else if (nq <= 2) NKV_DECG(2);
    else if (nq <= 4) NKV_DECG(4);
    else if (nq <= 8) NKV_DECG(8);
    else NKV_DECG(16);
#undef NKV_DECG
    prof.end(NKV_KERNEL_DECODE, st);
    return hipGetLastError();
}

}  // namespace

bool decode_fast_supported(int dtype, int d, int dv, int G)
{
    return (dtype == NKV_DTYPE_BF16 || dtype == NKV_DTYPE_F16) && d == dv && (d == 64 || d == 128) && G >= 1 && G <= 8;
}

size_t decode_ws_bytes(int dtype, int d, int dv, int G, int64_t n_units, int64_t rows, bool least)
{
    if (!decode_fast_supported(dtype, d, dv, G)) return 0;
    const size_t need = ws_for(max_chunks(n_units, rows, kChunk), n_units, G, d);
    if (least || n_units > kSmallUnits) return need;
    // room for chunks of 64 rows up to the row count where they end, so that more rows never ask for less
    const int64_t most = std::max<int64_t>(0, std::min((512 - n_units) * kChunk + kChunk - 1, (small_chunks_limit(G) - n_units) * kSmallChunk + kSmallChunk - 1));
    const size_t small = ws_for(max_chunks(n_units, rows < most ? rows : most, kSmallChunk), n_units, G, d);
    return need > small ? need : small;
}

hipError_t launch_decode(const void *q, const void *pk, const void *pv, const int64_t *head_off, int dtype,
                         int n_units, int G, int d, int dv, int64_t rows, double scale, float *out, float *lse,
                         void *ws, size_t ws_bytes, const Prof &prof, hipStream_t st)
{
    const float scale_log2 = (float)(scale * 1.4426950408889634);
    if (decode_fast_supported(dtype, d, dv, G)) {
        const uint16_t *q16 = (const uint16_t *)q, *k16 = (const uint16_t *)pk, *v16 = (const uint16_t *)pv;
        if (dtype == NKV_DTYPE_F16) {
            if (d == 128) return run_fast<128, true>(q16, k16, v16, head_off, n_units, G, rows, scale_log2, out, lse, ws, ws_bytes, prof, st);
            return run_fast<64, true>(q16, k16, v16, head_off, n_units, G, rows, scale_log2, out, lse, ws, ws_bytes, prof, st);
        }
        if (d == 128) return run_fast<128, false>(q16, k16, v16, head_off, n_units, G, rows, scale_log2, out, lse, ws, ws_bytes, prof, st);
        return run_fast<64, false>(q16, k16, v16, head_off, n_units, G, rows, scale_log2, out, lse, ws, ws_bytes, prof, st);
    }
    if (dtype == NKV_DTYPE_F32)
        return run_generic<float>((const float *)q, (const float *)pk, (const float *)pv, head_off, n_units, G, d, dv,
                                  rows, scale_log2, out, lse, prof, st);
    if (dtype == NKV_DTYPE_F16)
        return run_generic<f16_t>((const f16_t *)q, (const f16_t *)pk, (const f16_t *)pv, head_off, n_units, G, d, dv,
                                  rows, scale_log2, out, lse, prof, st);
    return run_generic<uint16_t>((const uint16_t *)q, (const uint16_t *)pk, (const uint16_t *)pv, head_off, n_units, G,
                                 d, dv, rows, scale_log2, out, lse, prof, st);
}

}  // namespace nkv
