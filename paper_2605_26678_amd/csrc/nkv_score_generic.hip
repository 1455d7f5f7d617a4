// Shape-generic scoring kernels: per-scale cosine anomalies a_s, a_e, a_c (paper Sections 2.1-2.3)
// for any head dim (multiple of 8, <= 1024), any window and block size, fp32, bf16, fp16 or 8-bit (E4M3) keys.
//
// Three kernels that cover what the streaming kernels do not (fp32 keys, head dims above 128, other windows or blocks):
//   1. block   : 1 / max(||k_i||, eps) per token (Section 2.1) and the sum of k_hat over every episodic block
//                (Section 2.2, episodic memory); one workgroup per block
//   2. ssum    : sum of k_hat over the prompt = sum of its block sums  (Section 2.2, stable memory)
//   3. anomaly : a_s, a_e from the two sums; a_c from a window sum that slides over 16 consecutive tokens and is formed
//                afresh in front of them (Section 2.2 current memory; Section 2.3); one wavefront per 16 tokens.  The window
//                sum is held in 64 bits (the products of 32-bit factors are exact then), so that what has entered
//                leaves again without a trace: in 32 bits, keys that cancel inside the window left twice the error of a
//                window added up afresh for every token.  One kernel for windows of 64 tokens of keys of up to 128 dims, one
//                for any
// Everywhere a lane owns dims lane, lane + 64, ... of a row.  The time of a small call is a chain of load latencies, so
// loads go out eight or sixteen rows at a time.  (With the window added up for every token, a wave per token and a serial loop over
// a block's tokens, 2 heads x 4096 fp32 tokens took 86 us.)
// Cosines do not depend on the length of the anchor, so sums stand in for the means.
#include "nkv_device.h"

namespace nkv {
namespace {

constexpr int kBlockThreads = 1024, kSsumThreads = 1024;
constexpr int kChunk = 16;               // tokens a wavefront slides the window over

template <int NQ> constexpr int rows_in_flight() { return NQ <= 2 ? 8 : NQ <= 4 ? 4 : 2; }

// U rows from row0 on that are `step` rows apart, as floats; rows below 0 or from `end` >= 1 on and dims from d on are
// zeros.  The loads are unconditional (of a clamped address), so that all of them go out together.
template <typename T, int NQ, int U>
__device__ __forceinline__ void load_rows(const T *__restrict__ unit, int d, int lane, int row0, int step, int end, float (&x)[U][NQ])
{
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int row = row0 + j * step, c = lane + q * kWave;
            const float v = load_elem<T>(unit + (int64_t)min(max(row, 0), end - 1) * d + min(c, d - 1));
            x[j][q] = row >= 0 && row < end && c < d ? v : 0.f;
        }
}

// grid (blocks per head, L*H); wave w takes the block's tokens w, w + 16, ...
template <typename T, int NQ>
__global__ __launch_bounds__(kBlockThreads) void block_kernel(const T *__restrict__ keys, RowMap km, int d, PromptTab tab,
                                                              float *__restrict__ rnorm, float *__restrict__ bsum)
{
    constexpr int NW = kBlockThreads / kWave, U = rows_in_flight<NQ>();
    __shared__ float part[NW][kWave];
    const int blk = blockIdx.x, lh = blockIdx.y;
    const int p = prompt_of_block(tab, blk);
    const int b = tab.b[p];
    const int n = tab.tok_off[p + 1] - tab.tok_off[p];
    const int lo = (blk - tab.blk_off[p]) * b;
    const int hi = min(lo + b, n);
    const int64_t row0 = (int64_t)lh * tab.T + tab.tok_off[p];
    const T *unit = keys + km.unit(lh, p, tab);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    float acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.f;
    for (int t = lo + w; t < hi; t += U * NW) {
        float x[U][NQ], rn[U];
        load_rows<T, NQ, U>(unit, d, lane, t, NW, hi, x);
        float ss[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            ss[j] = 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) ss[j] = fmaf(x[j][q], x[j][q], ss[j]);
        }
        if constexpr (U == 8) {                                       // lanes 8 j .. 8 j + 7: token j's
            const float r = 1.0f / fmaxf(sqrtf(wave_reduce8(ss, [](float a, float b) { return a + b; })), kEps);
            if ((lane & 7) == 0 && t + (lane >> 3) * NW < hi) rnorm[row0 + t + (lane >> 3) * NW] = r;
#pragma unroll
            for (int j = 0; j < U; ++j) rn[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), 8 * j));
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                rn[j] = 1.0f / fmaxf(sqrtf(wave_sum(ss[j])), kEps);
                if (lane == 0 && t + j * NW < hi) rnorm[row0 + t + j * NW] = rn[j];
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] = fmaf(rn[j], x[j][q], acc[q]);   // (rows past the block are zeros)
        }
    }
    float *out = bsum + ((int64_t)lh * tab.blk_off[tab.n] + blk) * d;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q > 0) __syncthreads();
        part[w][lane] = acc[q];
        __syncthreads();
        if (w == 0 && lane + q * kWave < d) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < NW; ++i) s += (double)part[i][lane];
            out[lane + q * kWave] = (float)s;
        }
    }
}

// grid (prompts, L*H); thread = (slice, dim): slice s adds blocks s, s + slices, ... up
__global__ __launch_bounds__(kSsumThreads) void ssum_kernel(const float *__restrict__ bsum, int d, PromptTab tab, float *__restrict__ ssum)
{
    __shared__ double part[kSsumThreads];
    const int p = blockIdx.x, lh = blockIdx.y;
    const int nblk = tab.blk_off[tab.n], n = tab.blk_off[p + 1] - tab.blk_off[p];
    const int slices = kSsumThreads / d, c = threadIdx.x % d, slice = threadIdx.x / d;       // d <= 1024; some threads may be idle
    const float *mine = bsum + ((int64_t)lh * nblk + tab.blk_off[p]) * d + c;
    double s = 0.0;
    if (slice < slices) {
        for (int b = slice; b < n; b += 4 * slices) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = b + i * slices < n ? mine[(int64_t)(b + i * slices) * d] : 0.f;
            s += ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
        }
    }
    part[threadIdx.x] = s;
    __syncthreads();
    if ((int)threadIdx.x < d) {
        double t = 0.0;
        for (int i = 0; i < slices; ++i) t += part[i * d + threadIdx.x];
        ssum[((int64_t)lh * tab.n + p) * d + threadIdx.x] = (float)t;
    }
}

// grid (chunks of 16 tokens / 4, L*H): every wavefront takes one chunk of one prompt.
template <typename T, int NQ>
__global__ __launch_bounds__(256) void anomaly_kernel(const T *__restrict__ keys, RowMap km, const float *__restrict__ rnorm,
                                                      const float *__restrict__ bsum, const float *__restrict__ ssum, int LH, int d,
                                                      int window, PromptTab tab, float *__restrict__ a_raw)
{
    constexpr int U = NQ <= 2 ? 16 : rows_in_flight<NQ>(), US = NQ <= 2 ? 8 : NQ <= 4 ? 4 : NQ <= 8 ? 2 : 1;
    const int lane = threadIdx.x & (kWave - 1), lh = blockIdx.y;
    const int64_t rows = (int64_t)LH * tab.T;
    int chunk = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave, p = 0;
    for (;; ++p) {
        if (p == tab.n) return;                                       // (uniform in the wavefront)
        const int nc = (tab.tok_off[p + 1] - tab.tok_off[p] + kChunk - 1) / kChunk;
        if (chunk < nc) break;
        chunk -= nc;
    }
    const int N = tab.tok_off[p + 1] - tab.tok_off[p], b = tab.b[p];
    const int i0 = chunk * kChunk, i1 = min(i0 + kChunk, N);
    const int64_t row0 = (int64_t)lh * tab.T + tab.tok_off[p];
    const T *unit = keys + km.unit(lh, p, tab);
    const float *rn_unit = rnorm + row0;
    const float *S = ssum + ((int64_t)lh * tab.n + p) * d;
    const float *B0 = bsum + ((int64_t)lh * tab.blk_off[tab.n] + tab.blk_off[p]) * d;

    // the weighted sum of rows [lo, hi)
    auto add_rows = [&](int lo, int hi, double (&sum)[NQ]) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) sum[q] = 0.0;
        for (int j = lo; j < hi; j += U) {
            float x[U][NQ];
            load_rows<T, NQ, U>(unit, d, lane, j, 1, hi, x);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const double r = (double)rn_unit[min(j + i, hi - 1)];
#pragma unroll
                for (int q = 0; q < NQ; ++q) sum[q] = fma(r, (double)x[i][q], sum[q]);
            }
        }
    };
    float s[NQ], e[NQ], ns = 0.f, ne = 0.f;
    double W[NQ];                                                     // the window in front of the next token
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int c = lane + q * kWave;
        s[q] = c < d ? S[c] : 0.f;
        e[q] = 0.f;
        ns = fmaf(s[q], s[q], ns);
    }
    ns = wave_sum(ns);
    add_rows(max(0, i0 - window), i0, W);
    int blk = -1;
    float as = 0.f, ae = 0.f, ac = 0.f;                               // lane t: the anomalies of token i0 + t
    for (int i = i0; i < i1; i += US) {
        float x[US][NQ], y[US][NQ];                                   // rows that enter and that leave the window
        load_rows<T, NQ, US>(unit, d, lane, i, 1, i1, x);
        load_rows<T, NQ, US>(unit, d, lane, i - window, 1, i1, y);
#pragma unroll
        for (int j = 0; j < US; ++j) {
            const int tok = i + j;
            if (tok >= i1) break;
            if (tok / b != blk) {                                     // the token's episodic block
                blk = tok / b;
                ne = 0.f;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int c = lane + q * kWave;
                    e[q] = c < d ? B0[(int64_t)blk * d + c] : 0.f;
                    ne = fmaf(e[q], e[q], ne);
                }
                ne = wave_sum(ne);
            }
            const float rn = rn_unit[tok];
            float kk = 0.f, ds = 0.f, de = 0.f, dc = 0.f, nc = 0.f;
            const float ry = tok >= window ? rn_unit[tok - window] : 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                W[q] = fma((double)rn, (double)x[j][q], fma(-(double)ry, (double)y[j][q], W[q]));
                const float kh = rn * x[j][q], wq = (float)W[q];
                kk = fmaf(kh, kh, kk);
                ds = fmaf(kh, s[q], ds);
                de = fmaf(kh, e[q], de);
                dc = fmaf(kh, wq, dc);
                nc = fmaf(wq, wq, nc);
            }
            kk = wave_sum(kk); ds = wave_sum(ds); de = wave_sum(de); dc = wave_sum(dc); nc = wave_sum(nc);
            const float nk = fmaxf(sqrtf(kk), kEps);
            const bool me = lane == tok - i0;
            as = me ? -ds / (nk * fmaxf(sqrtf(ns), kEps)) : as;
            ae = me ? -de / (nk * fmaxf(sqrtf(ne), kEps)) : ae;
            ac = me ? -dc / (nk * fmaxf(sqrtf(nc), kEps)) : ac;
        }
    }
    if (lane < i1 - i0) {
        float *out = a_raw + row0 + i0 + lane;
        out[0] = as;
        out[rows] = ae;
        out[2 * rows] = ac;
    }
}

// The same for windows of 64 tokens and head dims up to 128.  A workgroup takes 64 consecutive tokens of a prompt, a wavefront 16 of
// them and the 16 rows that lie 64 tokens in front, which are the ones that leave the window: 32 rows, all on their way at once, and the
// window in front of a wavefront's tokens is the sum of four of the workgroup's eight groups of rows.  (With every wavefront adding up
// the 64 rows in front of its tokens, sixteen loads at a time, and every token's five sums over the lanes reduced by themselves, the
// score call of 2 heads x 4096 fp32 tokens of head dim 128 took 43 us, 26 now; of 64 heads x 16384 640 and 290.)  grid (groups of 64 tokens, L*H).
template <typename T, int NQ>
__global__ __launch_bounds__(256) void anomaly_window64_kernel(const T *__restrict__ keys, RowMap km, const float *__restrict__ rnorm,
                                                               const float *__restrict__ bsum, const float *__restrict__ ssum, int LH,
                                                               int d, PromptTab tab, float *__restrict__ a_raw)
{
    constexpr int C = kChunk, NW = 4;
    __shared__ double lds_sum[2][NW][NQ][kWave];                      // the groups' sums: in front of, and of, the workgroup's tokens
    const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lh = blockIdx.y;
    const int64_t rows = (int64_t)LH * tab.T;
    int part = blockIdx.x, p = 0;
    for (; p + 1 < tab.n; ++p) {                                      // (the grid ends with the last prompt)
        const int np = (tab.tok_off[p + 1] - tab.tok_off[p] + NW * C - 1) / (NW * C);
        if (part < np) break;
        part -= np;
    }
    const int N = tab.tok_off[p + 1] - tab.tok_off[p], b = tab.b[p];
    const int i0 = part * NW * C + C * w, i1 = min(i0 + C, N);        // this wavefront's tokens (none past the prompt's end)
    const int64_t row0 = (int64_t)lh * tab.T + tab.tok_off[p];
    const T *unit = keys + km.unit(lh, p, tab);
    const float *rn_unit = rnorm + row0;
    const float *S = ssum + ((int64_t)lh * tab.n + p) * d;
    const float *B0 = bsum + ((int64_t)lh * tab.blk_off[tab.n] + tab.blk_off[p]) * d;

    float x[C][NQ], y[C][NQ];                                         // rows that enter and that leave the window
    load_rows<T, NQ, C>(unit, d, lane, i0 - NW * C, 1, N, y);
    load_rows<T, NQ, C>(unit, d, lane, i0, 1, N, x);
    // 1 / ||k||, 0 where there is no row: lanes 0 .. 15 of x's rows, 16 .. 31 of y's
    const int mine = i0 + (lane & 15) - (lane < C ? 0 : NW * C);
    float r = rn_unit[min(max(mine, 0), N - 1)];
    r = mine >= 0 && mine < N ? r : 0.f;
    auto of_row = [&](int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), j)); };
    float s[NQ], e[NQ], ns = 0.f, ne = 0.f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int c = lane + q * kWave;
        s[q] = c < d ? S[c] : 0.f;
        e[q] = 0.f;
        ns = fmaf(s[q], s[q], ns);
    }
    ns = wave_sum(ns);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double sx = 0.0, sy = 0.0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            sy = fma((double)of_row(C + j), (double)y[j][q], sy);
            sx = fma((double)of_row(j), (double)x[j][q], sx);
        }
        lds_sum[0][w][q][lane] = sy;
        lds_sum[1][w][q][lane] = sx;
    }
    __syncthreads();
    double W[NQ];                                                     // the window in front of the next token
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        W[q] = 0.0;
#pragma unroll
        for (int g = 0; g < NW; ++g) W[q] += lds_sum[g >= w ? 0 : 1][g][q][lane];
    }
    if (i0 >= N) return;                                              // (no barrier follows)
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) asm volatile("" : "+v"(x[j][q]), "+v"(y[j][q]));   // (or all of them would be kept as doubles)
    asm volatile("" : "+v"(r));
    auto add = [](float u, float v) { return u + v; };
    int blk_end = i0;                                                 // first token past the block whose sum e holds
#pragma unroll
    for (int h = 0; h < C; h += 8) {
        float kk[8], ds[8], de[8], dc[8], nc[8], nb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int tok = min(i0 + h + j, N - 1);                   // (what lies past the end is not stored)
            if (tok >= blk_end) {                                     // the token's episodic block
                const int blk = tok / b;
                blk_end = (blk + 1) * b;
                ne = 0.f;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int c = lane + q * kWave;
                    e[q] = c < d ? B0[(int64_t)blk * d + c] : 0.f;
                    ne = fmaf(e[q], e[q], ne);
                }
            }
            const float rx = of_row(h + j), ry = of_row(C + h + j);
            kk[j] = ds[j] = de[j] = dc[j] = nc[j] = 0.f;
            nb[j] = ne;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                W[q] = fma((double)rx, (double)x[h + j][q], fma(-(double)ry, (double)y[h + j][q], W[q]));
                const float kh = rx * x[h + j][q], wq = (float)W[q];
                kk[j] = fmaf(kh, kh, kk[j]);
                ds[j] = fmaf(kh, s[q], ds[j]);
                de[j] = fmaf(kh, e[q], de[j]);
                dc[j] = fmaf(kh, wq, dc[j]);
                nc[j] = fmaf(wq, wq, nc[j]);
            }
            __builtin_amdgcn_sched_barrier(0);                        // one token at a time: registers
        }
        // lanes 8 j .. 8 j + 7: token j's
        const float nk = fmaxf(sqrtf(wave_reduce8(kk, add)), kEps);
        const float as = -wave_reduce8(ds, add) / (nk * fmaxf(sqrtf(ns), kEps));
        const float ae = -wave_reduce8(de, add) / (nk * fmaxf(sqrtf(wave_reduce8(nb, add)), kEps));
        const float ac = -wave_reduce8(dc, add) / (nk * fmaxf(sqrtf(wave_reduce8(nc, add)), kEps));
        const int tok = i0 + h + (lane >> 3);
        if ((lane & 7) == 0 && tok < i1) {
            float *out = a_raw + row0 + tok;
            out[0] = as;
            out[rows] = ae;
            out[2 * rows] = ac;
        }
    }
}

template <typename T>
hipError_t run(const T *keys, const RowMap &km, int LH, int d, int window, const PromptTab &tab, float *a_raw, float *rnorm,
               float *bsum, float *ssum, const Prof &prof, hipStream_t st)
{
    int chunks = 0;
    for (int p = 0; p < tab.n; ++p) chunks += (tab.tok_off[p + 1] - tab.tok_off[p] + kChunk - 1) / kChunk;
    const dim3 blocks((unsigned)tab.blk_off[tab.n], (unsigned)LH), waves((unsigned)(chunks + 3) / 4, (unsigned)LH);
    int parts = 0;
    for (int p = 0; p < tab.n; ++p) parts += (tab.tok_off[p + 1] - tab.tok_off[p] + 4 * kChunk - 1) / (4 * kChunk);
    const dim3 groups((unsigned)parts, (unsigned)LH);
    const int nq = (d + kWave - 1) / kWave;
#define NKV_BY_DIMS(CALL) \
    do { if (nq <= 1) CALL(1); else if (nq <= 2) CALL(2); else if (nq <= 4) CALL(4); else if (nq <= 8) CALL(8); else CALL(16); } while (0)
#define NKV_BLOCK(NQ) block_kernel<T, NQ><<<blocks, kBlockThreads, 0, st>>>(keys, km, d, tab, rnorm, bsum)
#define NKV_ANOM(NQ) anomaly_kernel<T, NQ><<<waves, 256, 0, st>>>(keys, km, rnorm, bsum, ssum, LH, d, window, tab, a_raw)
    NKV_BY_DIMS(NKV_BLOCK);
    ssum_kernel<<<dim3(tab.n, LH), kSsumThreads, 0, st>>>(bsum, d, tab, ssum);
    prof.begin(NKV_KERNEL_SCAN, st);
    if (window == 4 * kChunk && nq <= 2) {
        if (nq <= 1) anomaly_window64_kernel<T, 1><<<groups, 256, 0, st>>>(keys, km, rnorm, bsum, ssum, LH, d, tab, a_raw);
        else anomaly_window64_kernel<T, 2><<<groups, 256, 0, st>>>(keys, km, rnorm, bsum, ssum, LH, d, tab, a_raw);
    } else {
        NKV_BY_DIMS(NKV_ANOM);
    }
#undef NKV_BLOCK
#undef NKV_ANOM
#undef NKV_BY_DIMS
    prof.end(NKV_KERNEL_SCAN, st);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_score_generic(const void *keys, const RowMap &km, int dtype, int LH, int d, int window, const PromptTab &tab,
                                float *a_raw, float *rnorm, float *bsum, float *ssum, const Prof &prof,
                                hipStream_t st)
{
    if (dtype == NKV_DTYPE_F32)
        return run<float>((const float *)keys, km, LH, d, window, tab, a_raw, rnorm, bsum, ssum, prof, st);
    if (dtype == NKV_DTYPE_F16)
        return run<f16_t>((const f16_t *)keys, km, LH, d, window, tab, a_raw, rnorm, bsum, ssum, prof, st);
    if (dtype == NKV_DTYPE_F8_E4M3)
        return run<f8e4m3_t>((const f8e4m3_t *)keys, km, LH, d, window, tab, a_raw, rnorm, bsum, ssum, prof, st);
    return run<uint16_t>((const uint16_t *)keys, km, LH, d, window, tab, a_raw, rnorm, bsum, ssum, prof, st);
}

}  // namespace nkv
