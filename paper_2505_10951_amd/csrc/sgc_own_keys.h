// Decode, head_dim 128: one wavefront's attention of a query's new token over the query's own keys (question and generated tokens).
#pragma once

#include "sgc_internal.h"

namespace sgc {

typedef __attribute__((ext_vector_type(8))) _Float16 dec_f16x8;
typedef __attribute__((ext_vector_type(8))) __bf16 dec_bf16x8;
typedef __attribute__((ext_vector_type(4))) float dec_f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t dec_u32x4;

__device__ inline float dec_bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ inline uint16_t dec_f32_to_bf16(float x)   // round to nearest even; NaN stays NaN
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

struct OwnKeys {
    char *pages;              // K part of the KV head in the query's first suffix page
    int64_t page_stride;      // bytes from page to page
    int64_t v_part;           // bytes from a page's K part to its V part
    int32_t n_keys;           // the new token's own key, the last, among them
    const uint16_t *q;        // the lane's query row (any valid row in lanes that are no head's)
    float scale;              // softmax scale in log2 units, 0 in such lanes
    const float2 *rope;       // the rotation's entries at the new token's position, or null
    // FRESH: the new token's key and value are not in the pages yet: taken from here, and put there where `append` says so
    const uint16_t *k_new, *v_new;
    bool append;
};

// 8 channels of a bf16 row
__device__ inline void dec_load8(const uint16_t *p, float out[8])
{
    const uint4 a = *reinterpret_cast<const uint4 *>(p);
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = __uint_as_float(w[i] << 16);
        out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}

// Products on the matrix cores, up to 16 query heads of one KV head, no LDS.  v_mfma_f32_16x16x32: a page's 16 tokens are the 16 rows
// of the first product's left operand (32 channels per instruction are 1 KiB of the page, in lane order), the heads are its columns
// (the unused columns carry zeros), so lane (j, q) = (lane % 16, lane / 16) ends up with the scores of head j against tokens
// 4 q .. 4 q + 3 of every page.  Those four values of two neighbouring pages are, as they stand, the lane's eight contraction slots of
// the second product (keys x heads), whose left operand V^T takes, per lane, the 8-byte run of four tokens of channel
// 16 cb + lane % 16 from each of the two pages.  Keys come in chunks of CH pages with an online softmax over the chunks.
// What bounds it is the chain of dependent loads: the first chunk's keys are requested before the query rows, a chunk's values before
// its softmax or, TOGETHER, with its keys.  (Many wavefronts a SIMD: chunks of 2, apart; chunks of 4 pages, and 2 pages with the next
// chunk's keys requested before the softmax, were no faster.  Wavefronts beside attn_few_kernel's others: chunks of 2, together; of 4 spill and
// cost 10 %.)
// Results: O (unnormalised, relative to 2^m; channels 16 cb + 4 q .. + 3 of head j), m and the sum l of the rounded weights.
template <bool FRESH, int CH, bool TOGETHER>
__device__ __forceinline__ void own_keys_attend(const OwnKeys &w, dec_f32x4 (&O)[8], float &m_run, float &l_run)
{
    constexpr int half = 64;
    static_assert(CH % 2 == 0, "two pages are one right operand");
    const int lane = threadIdx.x & 63, j = lane & 15, q = lane >> 4;
    const int n_pages = (w.n_keys + kPageTokens - 1) / kPageTokens;
    const int slot = (w.n_keys - 1) & (kPageTokens - 1);       // FRESH: the new token's place in the last page
    // the scores' left operands of a chunk: pages past the last are read as the last page again and masked
    dec_u32x4 ka[CH][4], k_fresh[4];
    uint16_t v_fresh[8];
    auto load_keys = [&](int pg0) {
#pragma unroll
        for (int p = 0; p < CH; ++p) {
            const char *kp = w.pages + (int64_t)min(pg0 + p, n_pages - 1) * w.page_stride + lane * 16;
#pragma unroll
            for (int cbk = 0; cbk < 4; ++cbk) ka[p][cbk] = *reinterpret_cast<const dec_u32x4 *>(kp + cbk * 1024);
        }
    };
    // channel 16 cb + j of V: 32-channel group cb / 2, token block q & 1, channel (cb % 2) * 16 + j inside it, tokens
    // 4 q .. 4 q + 3 = the half 8 (q >> 1) of the 16-byte run
    auto v_off = [&](int cb) { return ((((cb >> 1) * 2 + (q & 1)) * 32 + (cb & 1) * 16 + j) * 16) + 8 * (q >> 1); };
    uint2 v[CH][8];
    auto load_values = [&](int pg0) {
#pragma unroll
        for (int p = 0; p < CH; ++p) {
            const char *vp = w.pages + (int64_t)min(pg0 + p, n_pages - 1) * w.page_stride + w.v_part;
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) v[p][cb] = *reinterpret_cast<const uint2 *>(vp + v_off(cb));
        }
    };
    load_keys(0);
    // the query rows as right operands: chunk c8 = 4 cbk + q of 8 channels for cbk = 0..3; the rotation pairs chunk c8 with
    // chunk c8 + 8, both of which this lane holds (cbk and cbk + 2); the new key the same way, as left operand
    dec_f16x8 qb[4];
    {
        float x1[2][8], x2[2][8], y1[2][8], y2[2][8];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int c0 = 8 * (4 * cb + q);
            dec_load8(w.q + c0, x1[cb]);
            dec_load8(w.q + half + c0, x2[cb]);
            if (FRESH) {
                dec_load8(w.k_new + c0, y1[cb]);
                dec_load8(w.k_new + half + c0, y2[cb]);
            }
            if (w.rope)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float2 cs = w.rope[c0 + i];
                    rotate_pair(x1[cb][i], x2[cb][i], cs.x, cs.y);
                    if (FRESH) rotate_pair(y1[cb][i], y2[cb][i], cs.x, cs.y);
                }
        }
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                qb[cb][e] = (_Float16)(x1[cb][e] * w.scale);
                qb[cb + 2][e] = (_Float16)(x2[cb][e] * w.scale);
            }
        if (FRESH) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    k_fresh[cb][e] = pack2_f16(y1[cb][2 * e], y1[cb][2 * e + 1]);
                    k_fresh[cb + 2][e] = pack2_f16(y2[cb][2 * e], y2[cb][2 * e + 1]);
                }
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) v_fresh[cb] = w.v_new[16 * cb + j];
        }
    }
    if (TOGETHER) load_values(0);
    if (FRESH && w.append) {
        char *kp = w.pages + (int64_t)(n_pages - 1) * w.page_stride;
        if (j == slot)
#pragma unroll
            for (int cbk = 0; cbk < 4; ++cbk) *reinterpret_cast<dec_u32x4 *>(kp + lane * 16 + cbk * 1024) = k_fresh[cbk];
        if (q == (slot >> 2))
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) *reinterpret_cast<uint16_t *>(kp + w.v_part + v_off(cb) + 2 * (slot & 3)) = v_fresh[cb];
    }

#pragma unroll
    for (int cb = 0; cb < 8; ++cb) O[cb] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
    m_run = -INFINITY;
    l_run = 0.f;
    for (int pg0 = 0; pg0 < n_pages; pg0 += CH) {
        if (FRESH && pg0 + CH >= n_pages) {
#pragma unroll
            for (int p = 0; p < CH; ++p)
                if (pg0 + p >= n_pages - 1 && j == slot)
#pragma unroll
                    for (int cbk = 0; cbk < 4; ++cbk) ka[p][cbk] = k_fresh[cbk];
        }
        // scores of the chunk (log2 units)
        dec_f32x4 S[CH];
#pragma unroll
        for (int p = 0; p < CH; ++p) {
            dec_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cbk = 0; cbk < 4; ++cbk)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(dec_f16x8, ka[p][cbk]), qb[cbk], acc, 0, 0, 0);
            S[p] = acc;
        }
        // the values, on their way while the scores become weights
        if (!TOGETHER) load_values(pg0);
        float cmax = -INFINITY;
#pragma unroll
        for (int p = 0; p < CH; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = (pg0 + p) * kPageTokens + 4 * q + r;
                if (key >= w.n_keys) S[p][r] = -INFINITY;
                cmax = fmaxf(cmax, S[p][r]);
            }
        cmax = fmaxf(cmax, __shfl_xor(cmax, 16));
        cmax = fmaxf(cmax, __shfl_xor(cmax, 32));
        const float m_new = fmaxf(m_run, cmax);          // finite: every chunk holds at least one visible key
        const float alpha = exp2f(m_run - m_new);         // 0 on the first chunk
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int cb = 0; cb < 8; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) O[cb][r] *= alpha;
        if (FRESH && pg0 + CH >= n_pages) {
#pragma unroll
            for (int p = 0; p < CH; ++p)
                if (pg0 + p >= n_pages - 1 && q == (slot >> 2))
#pragma unroll
                    for (int cb = 0; cb < 8; ++cb) {
                        const uint32_t bits = (uint32_t)v_fresh[cb] << (16 * (slot & 1)), keep = 0xFFFF0000u >> (16 * (slot & 1));
                        if (slot & 2)
                            v[p][cb].y = (v[p][cb].y & keep) | bits;
                        else
                            v[p][cb].x = (v[p][cb].x & keep) | bits;
                    }
        }
        // weights, rounded to bf16 (the row sum adds the rounded values), two pages = one right operand
#pragma unroll
        for (int pp = 0; pp < CH; pp += 2) {
            if (pg0 + pp >= n_pages) break;            // (wave-uniform)
            uint16_t wt[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                wt[e] = dec_f32_to_bf16(exp2f(S[pp + (e >> 2)][e & 3] - m_new));
                l_run += dec_bf16_to_f32(wt[e]);
            }
            const dec_u32x4 wb = {(uint32_t)wt[0] | ((uint32_t)wt[1] << 16), (uint32_t)wt[2] | ((uint32_t)wt[3] << 16),
                                  (uint32_t)wt[4] | ((uint32_t)wt[5] << 16), (uint32_t)wt[6] | ((uint32_t)wt[7] << 16)};
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) {
                const dec_u32x4 av = {v[pp][cb].x, v[pp][cb].y, v[pp + 1][cb].x, v[pp + 1][cb].y};
                O[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8, av), __builtin_bit_cast(dec_bf16x8, wb), O[cb], 0, 0, 0);
            }
        }
        if (pg0 + CH < n_pages) {
            load_keys(pg0 + CH);
            if (TOGETHER) load_values(pg0 + CH);
        }
    }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
}

}  // namespace sgc
