// The budgets of one layer by nine byte-wise passes over its scores: any prompt length, up to NKV_MAX_HEADS heads, any
// number of ties.  Used by the shape-generic kernel, and by the slice-wise kernels for a layer whose lists overflow.
#pragma once

#include "nkv_device.h"

namespace nkv {

struct BudgetScratch {
    uint32_t hist[NKV_MAX_HEADS][256];             // 32 KB
    uint32_t Th[NKV_MAX_HEADS];                    // key of the m_safe-th best score of the head
    uint32_t want_h[NKV_MAX_HEADS];                // running rank, ends as #protected among ties at Th
    uint32_t ties_h[NKV_MAX_HEADS];                // #scores of the head equal to Th
    uint32_t cnt_gt[NKV_MAX_HEADS], cnt_eq[NKV_MAX_HEADS];
    uint32_t lhist[256];
    uint32_t TL, want_l;
};

// pl = p * L + l; called by all 1024 threads of a workgroup; x: LDS.
__device__ __forceinline__ void budget_of_layer(const float *__restrict__ scores, int L, int H, const PromptTab &tab, int pl,
                                                BudgetScratch &x, int32_t *__restrict__ k_per_head)
{
    const int l = pl % L, p = pl / L;
    const int N = tab.tok_off[p + 1] - tab.tok_off[p];
    const int k0 = tab.k0[p], m_safe = tab.m_safe[p];
    const int64_t R = (int64_t)H * (k0 - m_safe);
    const float *sc = scores + (int64_t)l * H * tab.T + tab.tok_off[p];   // head h at sc + h*T
    const int tid = threadIdx.x;

    // ---- A: per-head safeguard thresholds ----
    if (tid < H) { x.Th[tid] = 0xFFFFFFFFu; x.want_h[tid] = (uint32_t)m_safe; x.ties_h[tid] = 0u; }
    __syncthreads();
    if (m_safe > 0) {
        if (tid < H) x.Th[tid] = 0u;
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            for (int j = tid; j < H * 256; j += 1024) (&x.hist[0][0])[j] = 0u;
            __syncthreads();
            for (int h = 0; h < H; ++h) {
                const uint32_t th = x.Th[h];
                for (int i = tid; i < N; i += 1024) {
                    const uint32_t key = ord_key(sc[(int64_t)h * tab.T + i]);
                    if (pass == 0 || (key >> (shift + 8)) == (th >> (shift + 8)))
                        atomicAdd(&x.hist[h][(key >> shift) & 255u], 1u);
                }
            }
            __syncthreads();
            if (tid < H) {
                uint32_t want = x.want_h[tid];
                const uint32_t dig = radix_pick(x.hist[tid], want, 1);
                x.want_h[tid] = want;
                x.Th[tid] |= dig << shift;
                if (pass == 3) x.ties_h[tid] = x.hist[tid][dig];
            }
            __syncthreads();
        }
    }

    // ---- B: layer threshold over the unprotected pool ----
    if (tid == 0) { x.TL = 0u; x.want_l = (uint32_t)R; }
    __syncthreads();
    if (R > 0) {
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            if (tid < 256) x.lhist[tid] = 0u;
            __syncthreads();
            const uint32_t pre = x.TL;
            for (int h = 0; h < H; ++h) {
                const uint32_t th = x.Th[h];
                for (int i = tid; i < N; i += 1024) {
                    const uint32_t key = ord_key(sc[(int64_t)h * tab.T + i]);
                    if (key < th && (pass == 0 || (key >> (shift + 8)) == (pre >> (shift + 8))))
                        atomicAdd(&x.lhist[(key >> shift) & 255u], 1u);
                }
            }
            if (tid < H) {                               // unprotected ties at the head's own threshold
                const uint32_t ex = x.ties_h[tid] - (m_safe > 0 ? x.want_h[tid] : 0u);
                const uint32_t key = x.Th[tid];
                if (m_safe > 0 && ex > 0u && (pass == 0 || (key >> (shift + 8)) == (pre >> (shift + 8))))
                    atomicAdd(&x.lhist[(key >> shift) & 255u], ex);
            }
            __syncthreads();
            if (tid == 0) {
                uint32_t want = x.want_l;
                const uint32_t dig = radix_pick(x.lhist, want, 1);
                x.want_l = want;
                x.TL |= dig << shift;
            }
            __syncthreads();
        }
    }

    // ---- C: per-head counts ----
    if (tid < H) { x.cnt_gt[tid] = 0u; x.cnt_eq[tid] = 0u; }
    __syncthreads();
    if (R > 0) {
        const uint32_t tl = x.TL;
        for (int h = 0; h < H; ++h) {
            const uint32_t th = x.Th[h];
            for (int i = tid; i < N; i += 1024) {
                const uint32_t key = ord_key(sc[(int64_t)h * tab.T + i]);
                if (key < th) {
                    if (key > tl) atomicAdd(&x.cnt_gt[h], 1u);
                    else if (key == tl) atomicAdd(&x.cnt_eq[h], 1u);
                }
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t remaining = R > 0 ? x.want_l : 0u;
        for (int h = 0; h < H; ++h) {
            uint32_t b = (uint32_t)m_safe;
            if (R > 0) {
                const uint32_t ex = m_safe > 0 ? x.ties_h[h] - x.want_h[h] : 0u;
                uint32_t gt = x.cnt_gt[h], eq = x.cnt_eq[h];
                if (x.Th[h] > x.TL) gt += ex;
                else if (x.Th[h] == x.TL) eq += ex;
                const uint32_t take = min(remaining, eq);
                remaining -= take;
                b += gt + take;
            }
            k_per_head[(int64_t)pl * H + h] = (int32_t)b;
        }
    }
}

}  // namespace nkv
