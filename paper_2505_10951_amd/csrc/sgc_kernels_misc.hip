// Support kernels of libsgc (gfx950): rotary table, prefix K/V ingest into cache pages,
// canonical export/import of a cluster's cache, and the generic fp32-arithmetic attention kernel
// that serves shapes the MFMA kernel does not cover.
//
// SubGCache (arXiv 2505.10951) Sec. 3.4: the representative prompt's K/V are computed once per
// cluster and kept in GPU memory; each query's question tokens are appended to it.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include <type_traits>

#include "sgc_internal.h"
#include "sgc_own_keys.h"

namespace sgc {

namespace {

constexpr int kWave = 64;

// ---- element load/store helpers ------------------------------------------------------------
__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline uint16_t f32_to_bf16(float x)   // round to nearest even; NaN stays NaN
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// OCP E4M3 codes (bias 7, largest finite 448, no infinities) of x / scale, to nearest, ties to even.  The code is that of
// the correctly rounded fp32 quotient.  One division per element and a software encoder were what the ingest of an fp8
// cache spent its time on; the scale's reciprocal is taken once (correctly rounded) and a quotient is corrected
// twice by its residual, after which it is the correctly rounded one (Markstein: a quotient off by at most one unit,
// corrected with a correctly rounded reciprocal; the first correction brings it there).  Residuals must not underflow,
// so scales far from 1 divide.  A NaN (also of Inf / Inf, the scale of a head with an infinite element) is code 0x7F whatever
// its sign; the hardware conversion gives 0xFF.
struct E4m3Scale {
    float s, r;
    bool plain;          // wave-uniform: divide
};
__device__ inline E4m3Scale e4m3_scale(float s) { return {s, 1.0f / s, !(s > 0x1p-60f && s < 0x1p60f)}; }
__device__ inline float e4m3_quotient(float x, const E4m3Scale &q)
{
    if (q.plain) return x / q.s;
    float y = x * q.r;
    y = fmaf(fmaf(-y, q.s, x), q.r, y);
    return copysignf(fmaf(fmaf(-y, q.s, x), q.r, y), x);        // (the residual of a negative zero is a positive one)
}
// 0xFF -> 0x7F in each byte: the addition carries into a byte's top bit only where its lower seven are all ones
__device__ inline uint32_t e4m3_one_nan(uint32_t w) { return w & ~(((w & 0x7F7F7F7Fu) + 0x01010101u) & 0x80808080u); }
__device__ inline uint2 e4m3_codes8(const float x[8], const E4m3Scale &q)
{
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = e4m3_quotient(x[i], q);
    int a = 0, b = 0;
    a = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], a, false);
    a = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], a, true);
    b = __builtin_amdgcn_cvt_pk_fp8_f32(y[4], y[5], b, false);
    b = __builtin_amdgcn_cvt_pk_fp8_f32(y[6], y[7], b, true);
    return make_uint2(e4m3_one_nan((uint32_t)a), e4m3_one_nan((uint32_t)b));
}

__device__ inline float e4m3_to_f32(uint8_t c)
{
    const uint32_t e = (c >> 3) & 15u, m = c & 7u;
    float mag;
    if (e == 0)
        mag = (float)m * 0.001953125f;   // m * 2^-9
    else if (e == 15 && m == 7)
        mag = __uint_as_float(0x7FC00000u);
    else
        mag = __uint_as_float(((e + 120u) << 23) | (m << 20));
    return (c & 0x80) ? -mag : mag;
}

// 8 consecutive elements starting at element index `idx` (multiple of 8) of a typed array.
__device__ inline void load8(const void *base, int64_t idx, int dtype, float out[8])
{
    if (dtype == SGC_F32) {
        const float4 *p = reinterpret_cast<const float4 *>(static_cast<const float *>(base) + idx);
        const float4 a = p[0], b = p[1];
        out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
        out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
    } else if (dtype == SGC_BF16) {
        const uint4 a = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + idx);
        const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    } else if (dtype == kElemF16) {
        const uint4 a = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + idx);
        const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = f16_bits_to_f32((uint16_t)(w[i] & 0xFFFFu));
            out[2 * i + 1] = f16_bits_to_f32((uint16_t)(w[i] >> 16));
        }
    } else {
        const uint2 a = *reinterpret_cast<const uint2 *>(static_cast<const uint8_t *>(base) + idx);
        const uint32_t w[2] = {a.x, a.y};
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = e4m3_to_f32((uint8_t)(w[i >> 2] >> (8 * (i & 3))));
    }
}

__device__ inline float load1(const void *base, int64_t idx, int dtype)
{
    if (dtype == SGC_F32) return static_cast<const float *>(base)[idx];
    if (dtype == SGC_BF16) return bf16_to_f32(static_cast<const uint16_t *>(base)[idx]);
    if (dtype == kElemF16) return f16_bits_to_f32(static_cast<const uint16_t *>(base)[idx]);
    return e4m3_to_f32(static_cast<const uint8_t *>(base)[idx]);
}

// Stores x as fp32, bf16 or binary16 (fp8 caches have an ingest kernel of their own).
__device__ inline void store1(void *base, int64_t idx, int dtype, float x)
{
    if (dtype == SGC_F32)
        static_cast<float *>(base)[idx] = x;
    else if (dtype == SGC_BF16)
        static_cast<uint16_t *>(base)[idx] = f32_to_bf16(x);
    else
        static_cast<uint16_t *>(base)[idx] = f32_to_f16_bits(x);
}

__device__ inline void store8(void *base, int64_t idx, int dtype, const float x[8])
{
    if (dtype == SGC_F32) {
        float4 *p = reinterpret_cast<float4 *>(static_cast<float *>(base) + idx);
        p[0] = make_float4(x[0], x[1], x[2], x[3]);
        p[1] = make_float4(x[4], x[5], x[6], x[7]);
    } else if (dtype == SGC_BF16) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f32_to_bf16(x[2 * i]) | ((uint32_t)f32_to_bf16(x[2 * i + 1]) << 16);
        *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(base) + idx) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(base) + idx) =
            make_uint4(pack2_f16(x[0], x[1]), pack2_f16(x[2], x[3]), pack2_f16(x[4], x[5]), pack2_f16(x[6], x[7]));
    }
}

// Rotated pair of 8-channel chunks: x1 holds channels c0..c0+7, x2 channels c0+d/2.. of one head
// vector; tab points at the (cos, sin) entries of this position for channels c0..c0+7.
__device__ inline void rope8(float x1[8], float x2[8], const float2 *tab)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float2 cs = tab[i];
        rotate_pair(x1[i], x2[i], cs.x, cs.y);
    }
}

// ---- rotary table ----------------------------------------------------------------------------
__global__ void rope_table_kernel(float2 *table, int n_pos, int half, double base, double inv_d)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_pos * half) return;
    const int pos = (int)(idx / half), t = (int)(idx % half);
    const double theta = pow(base, -2.0 * (double)t * inv_d);
    double s, c;
    sincos((double)pos * theta, &s, &c);
    table[idx] = make_float2((float)c, (float)s);
}

// ---- tables from the host ---------------------------------------------------------------------
// The tables a batch sends to the device are a few hundred KiB at most.  A copy engine transfer of that size spends most of
// its 25-35 us getting started; a kernel that reads the pinned, mapped staging buffer over the host link is done in
// the time the link needs.
// Up to two pieces per launch (a call's own tables and the cache's page tables, when both are due).
// Tables and tile records that one workgroup brings to the device by itself; past that its own turns cost more.  Beside an ingest (two
// reads over the link one behind the other less), one workgroup against several, us of a prompts' call: 104 tiles 18.2 / 19.2, 128
// 16.6-17.4 / 16.7, 160 18.4 / 17.9, 256 19.0-19.7 / 18.8, 416 28.3 / 25.8.  As a launch of its own (one less): 64 tiles 15.2 / 15.8,
// 128 16.9 / 17.2, 192 17.7 / 17.3, 256 19.6 / 18.2, 640 33.1 / 30.2; but the host, which bounds passes this small, has 2 to 3 us less
// to do (a whole pass with 200 tiles 50.5 / 52.2), so there the line lies past the crossover.
constexpr int kOneGroupTiles = 128, kOneLaunchTiles = 256;
constexpr size_t kOneGroupBytes = 32 << 10;
typedef __attribute__((ext_vector_type(4))) uint32_t copy_u32x4;
struct CopyPiece {
    copy_u32x4 *dst;
    const copy_u32x4 *src;
    size_t n16, n4;      // 16-byte chunks, then 4-byte words behind them
};
__device__ inline void copy_piece(const CopyPiece &p, size_t first, size_t stride)
{
    constexpr int AT_ONCE = 8;          // reads a lane has under way over the link
    for (size_t i = first; i < p.n16; i += AT_ONCE * stride) {
        copy_u32x4 v[AT_ONCE];
#pragma unroll
        for (int k = 0; k < AT_ONCE; ++k) v[k] = p.src[i + k * stride < p.n16 ? i + k * stride : i];
#pragma unroll
        for (int k = 0; k < AT_ONCE; ++k)
            if (i + k * stride < p.n16) p.dst[i + k * stride] = v[k];
    }
    uint32_t *d4 = reinterpret_cast<uint32_t *>(p.dst + p.n16);
    const uint32_t *s4 = reinterpret_cast<const uint32_t *>(p.src + p.n16);
    for (size_t i = first; i < p.n4; i += stride) d4[i] = s4[i];
}
// Says that this workgroup has read its part of the staging buffer (what it read it has stored, so the reads are done): its
// word in mapped host memory takes the copy's number.
__device__ inline void signal_read(const CopyDone &done, int word)
{
    __syncthreads();
    if (threadIdx.x == 0 && done.words)
        __hip_atomic_store(done.words + word, done.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void copy_from_host_kernel(CopyPiece a, CopyPiece b, CopyDone done)
{
    const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    copy_piece(a, first, stride);
    copy_piece(b, first, stride);
    signal_read(done, blockIdx.x);
}

// ---- prefix ingest ---------------------------------------------------------------------------
// Linear copy of n bytes (a multiple of 16) from LDS to global memory, 16 bytes per thread and turn.
__device__ inline void copy_out_16(char *dst, const char *lds_src, int n)
{
    for (int off = threadIdx.x * 16; off < n; off += blockDim.x * 16)
        *reinterpret_cast<uint4 *>(dst + off) = *reinterpret_cast<const uint4 *>(lds_src + off);
}

// bf16 pages of 128-channel heads: V is a transpose (a page keeps, per channel, runs of 8 tokens), and element-sized
// scattered LDS writes of it collide in the banks.  The tokens' values go into a staging tile [16 tokens][128
// channels] instead, 16 bytes (8 channels) at a time, the sixteen chunks of token t's row at position
// vt_pos(chunk, t) so that the 16 lanes of a write cover all banks; the page's 16-byte units are then gathered from
// it column-wise (64 lanes read 64 neighbouring channels of one token) and stored straight to global memory.
__device__ inline int vt_pos(int chunk, int tok) { return chunk ^ ((tok & 1) << 3) ^ ((tok >> 1) & 7); }

__device__ inline void v_part_from_tile(char *vg, const uint16_t *vt)
{
    for (int u = threadIdx.x; u < 256; u += blockDim.x) {       // unit u = ((c / 32) * 2 + h) * 32 + c % 32, see v_page_index
        const int hh = (u >> 5) & 1, c = (u >> 6) * 32 + (u & 31);
        uint32_t w[4];
#pragma unroll
        for (int i2 = 0; i2 < 4; ++i2) {
            uint32_t e[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = 2 * i2 + k, t = 4 * hh + (i & 3) + 8 * (i >> 2);
                e[k] = vt[t * 128 + vt_pos(c >> 3, t) * 8 + (c & 7)];
            }
            w[i2] = e[0] | (e[1] << 16);
        }
        *reinterpret_cast<uint4 *>(vg + u * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// fp8 cache, first pass: the largest |rotated K| and |V| of one head over a chunk of a job's pages, into the job's part
// [2][Hkv][chunk] of amax.  The second pass takes the maximum over a job's chunks: one or a few loads of neighbouring values per
// lane.  (With [chunk][2][Hkv] and eight pages to a chunk whatever the prompt, those loads grew with its square: 131072 tokens
// of 8 heads 840 us for both passes, 381 now; 16384 of 32 heads 200 and 160.)  HBM-bound: it reads what the second pass
// reads.  (With one workgroup per page and an atomic maximum per wavefront into the job's 2 Hkv slots the launch waited
// for the atomics: 243 us for 29 000 tokens of 8 heads, 33 us now.)
__global__ void __launch_bounds__(256) ingest_amax_kernel(const PrefixJob *jobs, const int32_t *page_job, const int32_t *chunk_page0, float *amax,
                                                          int Hkv, int d, const float2 *rope)
{
    const int pg0 = chunk_page0[blockIdx.x];           // first launch-wide page of the chunk
    const PrefixJob job = jobs[page_job[pg0]];
    const int hk = blockIdx.y;
    const int chunk = blockIdx.x - job.chunk0;
    const int j0 = (pg0 - job.page0) * kPageTokens;
    const int j1 = chunk + 1 < job.n_chunks ? (chunk_page0[blockIdx.x + 1] - job.page0) * kPageTokens : job.prefix_len;
    const int half = d / 2, pairs = d / 16;
    float mk = 0.f, mv = 0.f;
    for (int it = threadIdx.x; it < (j1 - j0) * pairs; it += blockDim.x) {
        const int j = j0 + it / pairs, cc = it % pairs;
        float x1[8], x2[8], y1[8], y2[8];
        const int64_t row = ((int64_t)j * Hkv + hk) * d;
        load8(job.k, row + cc * 8, SGC_BF16, x1);
        load8(job.k, row + half + cc * 8, SGC_BF16, x2);
        load8(job.v, row + cc * 8, SGC_BF16, y1);
        load8(job.v, row + half + cc * 8, SGC_BF16, y2);
        if (rope) rope8(x1, x2, rope + (int64_t)j * half + cc * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mk = fmaxf(mk, fmaxf(fabsf(x1[i]), fabsf(x2[i])));
            mv = fmaxf(mv, fmaxf(fabsf(y1[i]), fabsf(y2[i])));
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        mk = fmaxf(mk, __shfl_xor(mk, o));
        mv = fmaxf(mv, __shfl_xor(mv, o));
    }
    __shared__ float part[4][2];
    const int wave = threadIdx.x / kWave;
    if (threadIdx.x % kWave == 0) {
        part[wave][0] = mk;
        part[wave][1] = mv;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        float m = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 4; ++w) m = fmaxf(m, part[w][threadIdx.x]);
        amax[(int64_t)job.chunk0 * 2 * Hkv + ((int64_t)threadIdx.x * Hkv + hk) * job.n_chunks + chunk] = m;
    }
}

// The scale of one head of a job (which: 0 = K, 1 = V) from the chunks' maxima; every wavefront of the caller takes part.
__device__ inline float scale_from_chunks(const float *amax, const PrefixJob &job, int which, int Hkv, int hk)
{
    const float *p = amax + (int64_t)job.chunk0 * 2 * Hkv + ((int64_t)which * Hkv + hk) * job.n_chunks;
    float m = 0.f;
    for (int i = threadIdx.x % kWave; i < job.n_chunks; i += kWave) m = fmaxf(m, p[i]);
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    return m > 0.f ? m / 448.0f : 1.0f;
}

// ---- tile records -----------------------------------------------------------------------------
// The record the attention kernel reads for tile i, put together from the tile's seed and from the tables the device
// holds (the cluster's prompt length and pages, the plan's per-query records).
__device__ inline void expand_one_tile(const ExpandArgs &e, int i)
{
    const TileSeed sd = e.seeds[i];
    Tile t;
    t.cluster = sd.cluster;
    t.hk = sd.hk;
    t.row0 = sd.row0;
    t.n_rows = sd.n_rows;
    t.prefix_len = 0;
    t.pt_off = 0;
    t.tok_base = 0;
    t.sq_lo = sd.sq_lo;
    t.sq_hi = sd.sq_hi;
    t.last_qpos = sd.last_qpos;
    t.n_q = sd.sq_hi - sd.sq_lo + 1;
    t.pad = 0;
#pragma unroll
    for (int k = 0; k < 12; ++k) t.first_pages[k] = 0;
#pragma unroll
    for (int k = 0; k < kTileQueries; ++k) t.q[k] = {INT32_MAX, 0, 0};
    t.own_page0 = 0;
    t.n_own_pages = 0;
    t.row_tile = t.unused = 0;
    if (sd.n_rows > 0) {
        if (e.jobs) {
            const PrefixJob &j = e.jobs[sd.cluster];
            t.cluster = j.cluster;
            t.prefix_len = j.prefix_len;
            t.pt_off = j.pt_off;
            t.tok_base = sd.cluster;          // prefix mode: the job index travels here
            t.sq_lo = 0;
            t.sq_hi = -1;
            t.last_qpos = 0;
            t.n_q = 0;
        } else {
            t.prefix_len = e.prefix_len[sd.cluster];
            t.pt_off = e.pt_off[sd.cluster];
            t.tok_base = e.cl_tok_off[sd.cluster];
#pragma unroll
            for (int k = 0; k < kTileQueries; ++k) {
                const int sq = sd.sq_lo + k;
                if (sq <= sd.sq_hi) t.q[k] = {e.sq_tok0[sq], e.sq_src0[sq], e.sq_own0[sq]};
            }
            t.own_page0 = e.sq_own0[sd.sq_lo];
            t.n_own_pages = e.sq_own0[sd.sq_hi] - t.own_page0 + sd.last_qpos / kPageTokens + 1;
        }
        const int n_pages = (t.prefix_len + kPageTokens - 1) / kPageTokens;
        if (n_pages > 0) {
#pragma unroll
            for (int k = 0; k < 12; ++k) t.first_pages[k] = e.page_table[t.pt_off + min(k, n_pages - 1)];
        }
    } else {
        t.cluster = 0;
        t.n_q = 0;
    }
    e.tiles[i] = t;
}

// One thread per tile.
__global__ void expand_tiles_kernel(ExpandArgs e)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < e.n) expand_one_tile(e, i);
}

// The ingest kernels below run on (pages, KV heads) grids of 128 threads.  The tile records of the attention launch that
// follows depend on nothing the ingest writes, so they are written by workgroups appended to the same grid (columns
// blockIdx.x >= n_pages, 128 tiles per workgroup) instead of by a launch of their own between the two.
__device__ inline void expand_in_ingest_grid(const ExpandArgs &e, int n_pages)
{
    const int i = (((int)blockIdx.x - n_pages) * (int)gridDim.y + (int)blockIdx.y) * 128 + (int)threadIdx.x;
    if (i < e.n) expand_one_tile(e, i);
}
// grid columns to append for e.n tiles
inline unsigned expand_columns(int n_tiles, int n_kv_heads)
{
    const int groups = (n_tiles + 127) / 128;
    return (unsigned)((groups + n_kv_heads - 1) / n_kv_heads);
}

// One workgroup per (page, KV head): rotate K, convert, write K and V parts in page order.
// Tokens past the prefix end are written as zeros so that a whole page can always be read.
// pg: page of the job, page: its id in the pool.
__device__ inline void ingest_write_page(const PoolGeom &g, int layer, const PrefixJob &job, int pg, int page, int hk, int io_dtype, const float2 *rope)
{
    const int P = job.prefix_len;
    const void *k = job.k, *v = job.v;
    const int d = g.head_dim, Hkv = g.n_kv_heads, half = d / 2, pairs = d / 16;
    // The page images are put together in LDS (V is a transpose: element-sized scattered writes) and go out
    // as whole 16-byte rows.
    extern __shared__ __attribute__((aligned(16))) char page_img[];
    const int part_bytes = (int)g.head_part_bytes;
    char *kp = page_img, *vp = page_img + part_bytes;
    const bool via_tile = g.kv_dtype == SGC_BF16 && d == 128;     // V through the staging tile (see v_part_from_tile)
    const bool v_as_given = via_tile && io_dtype == SGC_BF16;      // bf16 values into a bf16 cache: moved, not converted
    for (int it = threadIdx.x; it < kPageTokens * pairs; it += blockDim.x) {
        const int tok = it / pairs, cc = it % pairs;
        const int j = pg * kPageTokens + tok;
        float x1[8], x2[8], y1[8], y2[8];
        uint4 r1 = make_uint4(0, 0, 0, 0), r2 = r1;
        if (j < P) {
            const int64_t row = ((int64_t)j * Hkv + hk) * d;
            load8(k, row + cc * 8, io_dtype, x1);
            load8(k, row + half + cc * 8, io_dtype, x2);
            if (rope) rope8(x1, x2, rope + (int64_t)j * half + cc * 8);
            if (v_as_given) {
                r1 = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(v) + row + cc * 8);
                r2 = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(v) + row + half + cc * 8);
            } else {
                load8(v, row + cc * 8, io_dtype, y1);
                load8(v, row + half + cc * 8, io_dtype, y2);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x1[i] = x2[i] = y1[i] = y2[i] = 0.f;
        }
        store8(kp, k_page_index(tok, cc * 8), k_elem_type(g.kv_dtype), x1);
        store8(kp, k_page_index(tok, half + cc * 8), k_elem_type(g.kv_dtype), x2);
        if (v_as_given) {
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(vp) + tok * 128 + vt_pos(cc, tok) * 8) = r1;
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(vp) + tok * 128 + vt_pos(8 + cc, tok) * 8) = r2;
        } else if (via_tile) {
            store8(vp, tok * 128 + vt_pos(cc, tok) * 8, SGC_BF16, y1);
            store8(vp, tok * 128 + vt_pos(8 + cc, tok) * 8, SGC_BF16, y2);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                store1(vp, v_page_index(tok, cc * 8 + i), g.kv_dtype, y1[i]);
                store1(vp, v_page_index(tok, half + cc * 8 + i), g.kv_dtype, y2[i]);
            }
        }
    }
    __syncthreads();
    copy_out_16(g.k_part(layer, page, hk), kp, part_bytes);
    if (via_tile)
        v_part_from_tile(g.v_part(layer, page, hk), reinterpret_cast<const uint16_t *>(vp));
    else
        copy_out_16(g.v_part(layer, page, hk), vp, part_bytes);
}

__global__ void ingest_write_kernel(PoolGeom g, int layer, const int32_t *page_table, const PrefixJob *jobs,
                                    const int32_t *page_job, int n_pages, int io_dtype, const float2 *rope, ExpandArgs ex)
{
    if ((int)blockIdx.x >= n_pages) {
        expand_in_ingest_grid(ex, n_pages);
        return;
    }
    const PrefixJob job = jobs[page_job[blockIdx.x]];
    const int pg = blockIdx.x - job.page0;
    ingest_write_page(g, layer, job, pg, page_table[job.pt_off + pg], blockIdx.y, io_dtype, rope);
}

// A small call's ingest (16- and 32-bit caches): jobs and page ids travel with the launch, so no table has to be on the device
// before it.  More workgroups of the same launch copy what the attention launch behind it reads there and write its tile records.
// That is a launch less in front of the ingest, its 4 us and its boundary: one prompt of 411 tokens with its question 43.5 ->
// 38.6 us, ten prompts of 150 to 1000 tokens with their batch, four layers, 508 -> 491.
// expand_groups > 0: the records are written from the staged tables (three reads over the host link one behind the other, by
// many wavefronts while the pages are written); 0: by the one workgroup that copies, from what it has copied (a prompt of 411
// tokens: 38.7 us against 39.3).
template <typename ARGS>
__global__ void ingest_small_kernel(PoolGeom g, int layer, ARGS small, int n_pages, int io_dtype, const float2 *rope, CopyPiece a, CopyPiece b,
                                    int copy_groups, int expand_groups, CopyDone done, ExpandArgs ex)
{
    if ((int)blockIdx.x >= n_pages) {
        const int extra = ((int)blockIdx.x - n_pages) * (int)gridDim.y + (int)blockIdx.y;
        if (extra < copy_groups) {
            const size_t first = (size_t)extra * blockDim.x + threadIdx.x, stride = (size_t)copy_groups * blockDim.x;
            copy_piece(a, first, stride);
            copy_piece(b, first, stride);
            signal_read(done, extra);
            if (expand_groups == 0)
                for (int i = threadIdx.x; i < ex.n; i += blockDim.x) expand_one_tile(ex, i);
        } else if (extra < copy_groups + expand_groups) {
            const int i = (extra - copy_groups) * (int)blockDim.x + (int)threadIdx.x;
            if (i < ex.n) expand_one_tile(ex, i);
            signal_read(done, extra);
        }
        return;
    }
    int j = 0;
#pragma unroll
    for (int i = 1; i < ARGS::kJobs; ++i)
        if (i < small.n_jobs && (int)blockIdx.x >= small.jobs[i].page0) j = i;
    const PrefixJob &job = small.jobs[j];
    ingest_write_page(g, layer, job, blockIdx.x - job.page0, small.pages[blockIdx.x], blockIdx.y, io_dtype, rope);
}

// 4 x 4 bytes: w[t] holds channels 0..3 of token t, out[c] tokens 0..3 of channel c.
__device__ inline void transpose4(const uint32_t w[4], uint32_t out[4])
{
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// The second pass of an fp8 cache's ingest, one workgroup of two wavefronts per (page, KV head): the same page images in
// e4m3 codes, with the head's scales taken from the chunks' maxima (the job's first page writes them down).  V is
// transposed four channels at a time: a lane reads the 8 tokens of a run for 4 channels and stores 4 channels' 8-byte
// runs, which are neighbours in the page.  77 -> 43 us for 29 000 tokens of 8 heads (119 MB in, 60 MB out).
template <int D>
__global__ void __launch_bounds__(128) ingest_write_fp8_kernel(PoolGeom g, int layer, const int32_t *page_table, const PrefixJob *jobs,
                                                               const int32_t *page_job, int n_pages, const float *amax, const float2 *rope,
                                                               ExpandArgs ex)
{
    if ((int)blockIdx.x >= n_pages) {
        expand_in_ingest_grid(ex, n_pages);
        return;
    }
    constexpr int half = D / 2, pairs = D / 16, VS = D + 8;       // VS: bytes between the token rows of the V tile
    __shared__ __attribute__((aligned(16))) char kp[kPageTokens * D], vt[kPageTokens * VS];
    const PrefixJob job = jobs[page_job[blockIdx.x]];
    const int pg = blockIdx.x - job.page0, hk = blockIdx.y;
    const int Hkv = g.n_kv_heads;
    const int page = page_table[job.pt_off + pg];
    const int tok = threadIdx.x / pairs, cc = threadIdx.x % pairs;
    const int j = pg * kPageTokens + tok;
    float x1[8], x2[8], y1[8], y2[8];
    if (tok < kPageTokens && j < job.prefix_len) {
        const int64_t row = ((int64_t)j * Hkv + hk) * D;
        load8(job.k, row + cc * 8, SGC_BF16, x1);
        load8(job.k, row + half + cc * 8, SGC_BF16, x2);
        load8(job.v, row + cc * 8, SGC_BF16, y1);
        load8(job.v, row + half + cc * 8, SGC_BF16, y2);
        if (rope) rope8(x1, x2, rope + (int64_t)j * half + cc * 8);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) x1[i] = x2[i] = y1[i] = y2[i] = 0.f;
    }
    const float sk = scale_from_chunks(amax, job, 0, Hkv, hk), sv = scale_from_chunks(amax, job, 1, Hkv, hk);
    if (pg == 0 && threadIdx.x == 0) {
        job.scale_kv[hk] = sk;
        job.scale_kv[Hkv + hk] = sv;
    }
    const E4m3Scale qk = e4m3_scale(sk), qv = e4m3_scale(sv);
    if (tok < kPageTokens) {
        *reinterpret_cast<uint2 *>(kp + k_page_index(tok, cc * 8)) = e4m3_codes8(x1, qk);
        *reinterpret_cast<uint2 *>(kp + k_page_index(tok, half + cc * 8)) = e4m3_codes8(x2, qk);
        *reinterpret_cast<uint2 *>(vt + tok * VS + cc * 8) = e4m3_codes8(y1, qv);
        *reinterpret_cast<uint2 *>(vt + tok * VS + half + cc * 8) = e4m3_codes8(y2, qv);
    }
    __syncthreads();
    const int lane = threadIdx.x % kWave;
    if (threadIdx.x < kWave) {
        char *kg = g.k_part(layer, page, hk);
#pragma unroll
        for (int o = 0; o < kPageTokens * D; o += kWave * 16)
            *reinterpret_cast<uint4 *>(kg + o + lane * 16) = *reinterpret_cast<const uint4 *>(kp + o + lane * 16);
    } else if (lane < D / 2) {
        const int hh = lane & 1, c = (lane >> 1) * 4;
        uint32_t lo[4], hi[4], w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const uint32_t *>(vt + (4 * hh + i) * VS + c);
        transpose4(w, lo);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const uint32_t *>(vt + (8 + 4 * hh + i) * VS + c);
        transpose4(w, hi);
        uint4 *vg = reinterpret_cast<uint4 *>(g.v_part(layer, page, hk) + v_page_index(4 * hh, c));
        vg[0] = make_uint4(lo[0], hi[0], lo[1], hi[1]);
        vg[1] = make_uint4(lo[2], hi[2], lo[3], hi[3]);
    }
}

// ---- suffix ingest ---------------------------------------------------------------------------
// Same page layout as the cache, 16-bit only (K binary16, V bf16), for the question tokens of every query of the batch
// (SubGCache Sec. 3.4: the question tokens are appended to the cached prompt, so suffix token j of a
// query whose cluster has P prefix tokens is rotated at position P + j).  One workgroup per
// (own page, KV head); tokens past the query's end are written as zeros.
__global__ void suffix_ingest_kernel(AttnArgs a, int n_spages, ExpandArgs ex)
{
    if ((int)blockIdx.x >= n_spages) {
        expand_in_ingest_grid(ex, n_spages);
        return;
    }
    const int hk = blockIdx.y;
    const int Hkv = a.n_kv_heads, d = a.head_dim, half = d / 2, pairs = d / 16;
    const SuffixPage pg = a.spages[blockIdx.x];
    const int64_t part = (int64_t)kPageTokens * d * 2;
    char *kg = const_cast<char *>(a.spool) + (int64_t)pg.page * 2 * Hkv * part + (int64_t)hk * part;
    char *vg = kg + (int64_t)Hkv * part;
    extern __shared__ __attribute__((aligned(16))) char page_img[];     // both images are built in LDS first
    char *kp = page_img, *vp = page_img + part;
    const bool via_tile = d == 128;          // V through the staging tile (see v_part_from_tile)
    const bool v_as_given = via_tile && a.io_dtype == SGC_BF16;      // bf16 values into bf16 pages: moved, not converted
    for (int it = threadIdx.x; it < kPageTokens * pairs; it += blockDim.x) {
        const int tok = it / pairs, cc = it % pairs;
        float x1[8], x2[8], y1[8], y2[8];
        uint4 r1 = make_uint4(0, 0, 0, 0), r2 = r1;
        if (tok < pg.n) {
            const int64_t row = ((int64_t)(pg.row0 + tok) * Hkv + hk) * d;
            load8(a.k, row + cc * 8, a.io_dtype, x1);
            load8(a.k, row + half + cc * 8, a.io_dtype, x2);
            if (a.rope) rope8(x1, x2, a.rope + (int64_t)(pg.pos0 + tok) * half + cc * 8);
            if (v_as_given) {
                r1 = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(a.v) + row + cc * 8);
                r2 = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(a.v) + row + half + cc * 8);
            } else {
                load8(a.v, row + cc * 8, a.io_dtype, y1);
                load8(a.v, row + half + cc * 8, a.io_dtype, y2);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x1[i] = x2[i] = y1[i] = y2[i] = 0.f;
        }
        store8(kp, k_page_index(tok, cc * 8), kElemF16, x1);
        store8(kp, k_page_index(tok, half + cc * 8), kElemF16, x2);
        if (v_as_given) {
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(vp) + tok * 128 + vt_pos(cc, tok) * 8) = r1;
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(vp) + tok * 128 + vt_pos(8 + cc, tok) * 8) = r2;
        } else if (via_tile) {
            store8(vp, tok * 128 + vt_pos(cc, tok) * 8, SGC_BF16, y1);
            store8(vp, tok * 128 + vt_pos(8 + cc, tok) * 8, SGC_BF16, y2);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                store1(vp, v_page_index(tok, cc * 8 + i), SGC_BF16, y1[i]);
                store1(vp, v_page_index(tok, half + cc * 8 + i), SGC_BF16, y2[i]);
            }
        }
    }
    __syncthreads();
    copy_out_16(kg, kp, (int)part);
    if (via_tile)
        v_part_from_tile(vg, reinterpret_cast<const uint16_t *>(vp));
    else
        copy_out_16(vg, vp, (int)part);
}

// ---- decode ------------------------------------------------------------------------------------
// SubGCache App. A.2 caps generation at 32 tokens per query; every generated token attends over the
// cluster's cached prompt, the query's question tokens and the tokens generated before it (Sec. 3.4:
// all queries of a cluster reuse the same cache).  The cached-prompt part of a step runs in the MFMA
// kernel with the rows of all sibling queries stacked into one tile, so the prompt's K/V are read once
// per cluster instead of once per query (blocks behind that launch's tiles append the step's new tokens to the
// queries' suffix pages); the kernel here does what is per query.

// One wavefront per (sorted query, group of G query heads that share a KV head): scores of the new token
// against the query's own len + step + 1 keys (lane = key, each key read once for the G heads), softmax,
// weighted V sum (lane = channel pair), merged with the cached-prefix part by the log-sum-exp rule.
// Both products run on 16-bit pairs with fp32 accumulation (v_dot2_f32_f16 on the binary16 keys and the rotated
// query rounded to binary16; v_dot2_f32_bf16 on the bf16 values and the softmax weights rounded to bf16), the
// operands a matrix-core kernel would use; the row sum is taken over the rounded weights.  G divides the GQA
// group size.
typedef __attribute__((ext_vector_type(2))) __bf16 dec_bf16x2;

__device__ inline float dot8_f16(const uint4 &x, const uint4 &y, float acc)
{
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(sgc_f16x2, x.x), __builtin_bit_cast(sgc_f16x2, y.x), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(sgc_f16x2, x.y), __builtin_bit_cast(sgc_f16x2, y.y), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(sgc_f16x2, x.z), __builtin_bit_cast(sgc_f16x2, y.z), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(sgc_f16x2, x.w), __builtin_bit_cast(sgc_f16x2, y.w), acc, false);
    return acc;
}

__device__ inline float dot8_bf16(const uint4 &x, const uint4 &y, float acc)
{
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2, x.x), __builtin_bit_cast(dec_bf16x2, y.x), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2, x.y), __builtin_bit_cast(dec_bf16x2, y.y), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2, x.z), __builtin_bit_cast(dec_bf16x2, y.z), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2, x.w), __builtin_bit_cast(dec_bf16x2, y.w), acc, false);
    return acc;
}

template <int G>
__global__ void __launch_bounds__(64) decode_own_keys_kernel(DecodeArgs a)
{
    constexpr int d = 128, half = 64;
    // LDS: the G rotated query rows as binary16 [G][128]; G rows of key_cap scores (fp32); G rows of key_cap weights as
    // bf16 in the order the V pages hold their tokens (key_cap = the batch's largest key count, rounded up to a page;
    // sized at launch so that many wavefronts fit a CU)
    extern __shared__ __attribute__((aligned(16))) char dec_lds[];
    const int key_cap = a.key_cap;
    uint16_t *q_s = reinterpret_cast<uint16_t *>(dec_lds);                          // [G][d]
    float *p_base = reinterpret_cast<float *>(dec_lds + G * d * 2);                  // [G][key_cap]
    uint16_t *w_s = reinterpret_cast<uint16_t *>(dec_lds + G * d * 2 + G * key_cap * 4);   // [G][key_cap]
    const int lane = threadIdx.x;
    const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, g = Hq / Hkv;
    const int units_per_query = Hq / G;
    const int sq = blockIdx.x / units_per_query;
    const int h0 = (blockIdx.x % units_per_query) * G;      // first head of the unit
    const int hk = h0 / g;
    const int n = a.sq_query[sq];
    const int n_keys = a.sq_len[sq] + a.step + 1;
    const int P = a.cl_prefix_len[a.sq_cluster[sq]];
    const int64_t io = ((int64_t)n * Hq + h0) * d;           // first of G consecutive rows
    for (int it = lane; it < G * (half / 8); it += kWave) {    // rotated query rows into LDS
        const int gi = it / (half / 8), cc = it % (half / 8);
        float x1[8], x2[8];
        load8(a.q, io + gi * d + cc * 8, SGC_BF16, x1);
        load8(a.q, io + gi * d + half + cc * 8, SGC_BF16, x2);
        if (a.rope) rope8(x1, x2, a.rope + (int64_t)(P + n_keys - 1) * half + cc * 8);
        uint32_t w1[4], w2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w1[i] = pack2_f16(x1[2 * i], x1[2 * i + 1]);
            w2[i] = pack2_f16(x2[2 * i], x2[2 * i + 1]);
        }
        *reinterpret_cast<uint4 *>(q_s + gi * d + cc * 8) = make_uint4(w1[0], w1[1], w1[2], w1[3]);
        *reinterpret_cast<uint4 *>(q_s + gi * d + half + cc * 8) = make_uint4(w2[0], w2[1], w2[2], w2[3]);
    }
    __syncthreads();
    const int64_t part = (int64_t)kPageTokens * d * 2;
    const char *pages = a.spool + (int64_t)a.sq_page0[sq] * 2 * Hkv * part + (int64_t)hk * part;
    const int64_t page_stride = 2 * Hkv * part;
    // scores (log2 units), lane = key
    float m[G], l[G];
#pragma unroll
    for (int gi = 0; gi < G; ++gi) m[gi] = -INFINITY;
    for (int j = lane; j < n_keys; j += kWave) {
        const char *kp = pages + (int64_t)(j / kPageTokens) * page_stride;
        const int tok = j % kPageTokens;
        uint4 raw[d / 8];                      // the key's 128 channels: all 16 loads in flight before any is used
#pragma unroll
        for (int cc = 0; cc < d / 8; ++cc)
            raw[cc] = *reinterpret_cast<const uint4 *>(kp + (int64_t)k_page_index(tok, cc * 8) * 2);
        float sc[G];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) sc[gi] = 0.f;
#pragma unroll
        for (int cc = 0; cc < d / 8; ++cc) {
#pragma unroll
            for (int gi = 0; gi < G; ++gi)
                sc[gi] = dot8_f16(raw[cc], *reinterpret_cast<const uint4 *>(q_s + gi * d + cc * 8), sc[gi]);
        }
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            sc[gi] *= a.scale_log2e;
            p_base[gi * key_cap + j] = sc[gi];
            m[gi] = fmaxf(m[gi], sc[gi]);
        }
    }
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
        for (int o = 32; o > 0; o >>= 1) m[gi] = fmaxf(m[gi], __shfl_xor(m[gi], o));
        l[gi] = 0.f;
    }
    // weights, rounded to bf16, stored where the V pages keep their tokens: a page holds, per channel, two runs of
    // 8 tokens; token t of a page is element (t & 3) | ((t >> 3) << 2) of run (t >> 2) & 1
    const int n_pages = (n_keys + kPageTokens - 1) / kPageTokens;
    for (int j = lane; j < n_pages * kPageTokens; j += kWave) {
        const int pg = j / kPageTokens, t = j % kPageTokens;
        const int slot = (pg * 2 + ((t >> 2) & 1)) * 8 + ((t & 3) | ((t >> 3) << 2));
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            uint16_t wb = 0;                                    // the unused tail of the last page weighs nothing
            if (j < n_keys) {
                wb = f32_to_bf16(exp2f(p_base[gi * key_cap + j] - m[gi]));
                l[gi] += bf16_to_f32(wb);
            }
            w_s[gi * key_cap + slot] = wb;
        }
    }
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
        for (int o = 32; o > 0; o >>= 1) l[gi] += __shfl_xor(l[gi], o);
    __syncthreads();
    // weighted V sum, lane = channels (lane, lane + 64)
    float acc[G][2];
#pragma unroll
    for (int gi = 0; gi < G; ++gi) acc[gi][0] = acc[gi][1] = 0.f;
    // (pages are taken four at a time: their sixteen 16-byte runs are all requested before the first is used)
    for (int pg0 = 0; pg0 < n_pages; pg0 += 4) {
        uint4 raw[4][4];
#pragma unroll
        for (int pi = 0; pi < 4; ++pi) {
            const int pg = min(pg0 + pi, n_pages - 1);           // a repeated page is skipped below
            const char *vp = pages + (int64_t)pg * page_stride + (int64_t)Hkv * part;
#pragma unroll
            for (int cI = 0; cI < 2; ++cI) {
                const int c = lane + cI * 64;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
                    raw[pi][cI * 2 + hh] =
                        *reinterpret_cast<const uint4 *>(vp + (int64_t)((((c >> 5) * 2 + hh) * 32 + (c & 31)) * 8) * 2);
            }
        }
#pragma unroll
        for (int pi = 0; pi < 4; ++pi) {
            const int pg = pg0 + pi;
            if (pg >= n_pages) break;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    const uint4 wts = *reinterpret_cast<const uint4 *>(w_s + gi * key_cap + (pg * 2 + hh) * 8);
                    acc[gi][0] = dot8_bf16(raw[pi][hh], wts, acc[gi][0]);
                    acc[gi][1] = dot8_bf16(raw[pi][2 + hh], wts, acc[gi][1]);
                }
            }
        }
    }
    // merge with the cached-prefix part, which comes as n_splits partial results over key ranges (natural-log
    // LSE there, -inf for an empty range; log2 units here).  The loops are unrolled over the ranges a plan gives this
    // kernel at most: unrolled over sixteen a step of 64 heads over 2 took 29.1 us where it takes 27.0 (16 queries, one
    // prompt of 200; 89.5 and 83.4 with 64 queries on each of 16 prompts).
    uint16_t *og = static_cast<uint16_t *>(a.o);
    const uint16_t *oc = static_cast<const uint16_t *>(a.o_cached);
    const int S = a.n_splits;
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
        const int h = h0 + gi;
        const float lse_own = m[gi] + log2f(l[gi]);
        float lse_c[kDecodeDotSplits];
        float M = lse_own;
#pragma unroll
        for (int sp = 0; sp < kDecodeDotSplits; ++sp) {
            lse_c[sp] = -INFINITY;
            if (sp < S && a.lse_cached) lse_c[sp] = a.lse_cached[sp * a.split_lse_elems + (int64_t)h * a.n_queries + n] * 1.4426950408889634f;
            M = fmaxf(M, lse_c[sp]);
        }
        const float wo = exp2f(m[gi] - M);                       // weight of the unnormalised own sum
        float denom = exp2f(lse_own - M);
        float sum[2] = {wo * acc[gi][0], wo * acc[gi][1]};
#pragma unroll
        for (int sp = 0; sp < kDecodeDotSplits; ++sp) {
            if (lse_c[sp] == -INFINITY) continue;          // (a range that came out NaN stays in)
            const float wc = exp2f(lse_c[sp] - M);
            denom += wc;
#pragma unroll
            for (int cI = 0; cI < 2; ++cI)
                sum[cI] += wc * bf16_to_f32(oc[sp * a.split_o_elems + io + gi * d + lane + cI * 64]);
        }
#pragma unroll
        for (int cI = 0; cI < 2; ++cI) og[io + gi * d + lane + cI * 64] = f32_to_bf16(sum[cI] / denom);
        if (a.lse && lane == 0) a.lse[(int64_t)h * a.n_queries + n] = (M + log2f(denom)) * 0.6931471805599453f;
    }
}

// The same step on the matrix cores, head_dim 128, groups of up to 16 query heads per KV head: one wavefront per (sorted
// query, KV head), see own_keys_attend.  The cached part's log-sum-exps are requested first, its outputs of four ranges
// together.  Decode step of 320 queries over prompts of 1024 (8 KV heads, 57 own keys on average): 34.7 -> 34.0 us; without head
// groups (32 KV heads, prompts of 500) 88.9 -> 82.3.
__global__ void __launch_bounds__(256, 3) decode_own_keys_mfma_kernel(DecodeArgs a)
{
    constexpr int d = 128, half = 64;
    const int lane = threadIdx.x & 63;
    const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, g = Hq / Hkv;
    const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= a.n_sq * Hkv) return;                 // (no barrier anywhere in this kernel)
    const int sq = unit / Hkv, hk = unit - sq * Hkv;
    const int j = lane & 15, q = lane >> 4;
    const int n = a.sq_query[sq];
    const int n_keys = a.sq_len[sq] + a.step + 1;
    const int P = a.cl_prefix_len[a.sq_cluster[sq]];
    const bool live = j < g;                           // the lane's column is a head of the group
    const int h = hk * g + (live ? j : 0);
    const int64_t io = ((int64_t)n * Hq + h) * d;
    const int64_t part = (int64_t)kPageTokens * d * 2;
    const int64_t page_stride = 2 * Hkv * part;
    const char *pages = a.spool + (int64_t)a.sq_page0[sq] * page_stride + (int64_t)hk * part;

    // the cached part's log-sum-exps of the lane's head, range q + 4 i in lane group q
    const int S_n = a.n_splits;
    constexpr int LR = kDecodeMaxSplits / 4;
    float lse_q[LR];
#pragma unroll
    for (int i = 0; i < LR; ++i) {
        lse_q[i] = -INFINITY;
        if (q + 4 * i < S_n && a.lse_cached) lse_q[i] = a.lse_cached[(q + 4 * i) * a.split_lse_elems + (int64_t)h * a.n_queries + n];
    }

    OwnKeys own{};
    own.pages = const_cast<char *>(pages);
    own.page_stride = page_stride;
    own.v_part = (int64_t)Hkv * part;
    own.n_keys = n_keys;
    own.q = static_cast<const uint16_t *>(a.q) + io;
    own.scale = live ? a.scale_log2e : 0.f;
    own.rope = a.rope ? a.rope + (int64_t)(P + n_keys - 1) * half : nullptr;
    dec_f32x4 O[8];
    float m_run, l_run;
    own_keys_attend<false, 2, false>(own, O, m_run, l_run);
    // merge with the cached-prefix part (natural-log LSE there, -inf for an empty range; log2 units here); the lane holds
    // channels 16 cb + 4 q .. + 3 of its head
    const uint16_t *oc = static_cast<const uint16_t *>(a.o_cached);
    uint16_t *og = static_cast<uint16_t *>(a.o);
    const float lse_own = m_run + log2f(l_run);
    float lse_c[kDecodeMaxSplits];
    float M = lse_own;
#pragma unroll
    for (int sp = 0; sp < kDecodeMaxSplits; ++sp) {
        lse_c[sp] = __shfl(lse_q[sp / 4], j + 16 * (sp % 4)) * 1.4426950408889634f;
        M = fmaxf(M, lse_c[sp]);
    }
    if (!live) return;
    const float wo = exp2f(m_run - M);                        // weight of the unnormalised own sum
    float denom = exp2f(lse_own - M);
    float sum[8][4];
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[cb][r] = wo * O[cb][r];
    // four ranges' outputs are requested together: asked for one range at a time, each costs a round trip of its own
#pragma unroll
    for (int s0 = 0; s0 < kDecodeMaxSplits; s0 += 4) {
        if (s0 >= S_n) break;
        uint2 raw[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s0 + i >= S_n) break;
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) raw[i][cb] = *reinterpret_cast<const uint2 *>(oc + (s0 + i) * a.split_o_elems + io + cb * 16 + 4 * q);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s0 + i >= S_n) break;
            if (lse_c[s0 + i] == -INFINITY) continue;        // an empty range's output means nothing (one that came out NaN stays in)
            const float wc = exp2f(lse_c[s0 + i] - M);
            denom += wc;
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) {
                sum[cb][0] += wc * bf16_to_f32((uint16_t)(raw[i][cb].x & 0xFFFF));
                sum[cb][1] += wc * bf16_to_f32((uint16_t)(raw[i][cb].x >> 16));
                sum[cb][2] += wc * bf16_to_f32((uint16_t)(raw[i][cb].y & 0xFFFF));
                sum[cb][3] += wc * bf16_to_f32((uint16_t)(raw[i][cb].y >> 16));
            }
        }
    }
    const float inv = 1.0f / denom;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
        uint2 out;
        out.x = (uint32_t)f32_to_bf16(sum[cb][0] * inv) | ((uint32_t)f32_to_bf16(sum[cb][1] * inv) << 16);
        out.y = (uint32_t)f32_to_bf16(sum[cb][2] * inv) | ((uint32_t)f32_to_bf16(sum[cb][3] * inv) << 16);
        *reinterpret_cast<uint2 *>(og + io + cb * 16 + 4 * q) = out;
    }
    if (a.lse && q == 0) a.lse[(int64_t)h * a.n_queries + n] = (M + log2f(denom)) * 0.6931471805599453f;
}

__global__ void fill_zero_bytes_kernel(uint4 *p, size_t n16)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

// ---- export / import: raw element moves between page order and [P][Hkv][d] --------------------
template <typename T>
__global__ void cache_export_kernel(PoolGeom g, int layer, const int32_t *pages, int P, T *k, T *v)
{
    const int d = g.head_dim, Hkv = g.n_kv_heads;
    const int64_t n = (int64_t)P * Hkv * d;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(idx % d);
        const int hk = (int)((idx / d) % Hkv);
        const int j = (int)(idx / ((int64_t)d * Hkv));
        const int page = pages[j / kPageTokens], tok = j % kPageTokens;
        k[idx] = reinterpret_cast<const T *>(g.k_part(layer, page, hk))[k_page_index(tok, c)];
        v[idx] = reinterpret_cast<const T *>(g.v_part(layer, page, hk))[v_page_index(tok, c)];
    }
}

template <typename T>
__global__ void cache_import_kernel(PoolGeom g, int layer, const int32_t *pages, int P, const T *k, const T *v)
{
    const int d = g.head_dim, Hkv = g.n_kv_heads;
    const int n_pages = (P + kPageTokens - 1) / kPageTokens;
    const int64_t n = (int64_t)n_pages * kPageTokens * Hkv * d;   // whole pages: the tail is zeroed
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(idx % d);
        const int hk = (int)((idx / d) % Hkv);
        const int j = (int)(idx / ((int64_t)d * Hkv));
        const int page = pages[j / kPageTokens], tok = j % kPageTokens;
        const T kk = j < P ? k[idx] : T(0);
        const T vv = j < P ? v[idx] : T(0);
        reinterpret_cast<T *>(g.k_part(layer, page, hk))[k_page_index(tok, c)] = kk;
        reinterpret_cast<T *>(g.v_part(layer, page, hk))[v_page_index(tok, c)] = vv;
    }
}

// ---- generic attention: fp32 matrix cores, any type and head size ----------------------------------------
// A workgroup takes 16 rows (token, head-in-group) of one (cluster or prompt, KV head); its NW wavefronts deal the blocks of
// 16 keys among themselves and merge their partial softmax states at the end, so that a few hundred rows over a few hundred
// keys fill the chip and a wavefront's chain is a handful of blocks.  v_mfma_f32_16x16x4, everything in fp32:
//   scores: left operand = 16 keys (lane (j, q) = (lane % 16, lane / 16) holds channels q D/4 .. of key j), right operand =
//           the 16 rows (row j, the same channels); lane (j, q) ends up with row j's scores of keys 4 q .. 4 q + 3;
//   values: those four weights are, one register per instruction, the right operand of the second product, whose left
//           operand takes channel 16 cb + j of keys 4 q .. 4 q + 3: one run of four tokens in a V page.
// Sums: a block's 16 weighted values are added up by themselves and then to the running sum, and a score is two chains of
// D/2 products.  One chain through all of a wavefront's keys was off by 5.9e-7 (2-norm) over 6001 keys (d 64) and 6.4e-7 over
// 3000 (d 128), more than the 3.8e-7 and 4.3e-7 of the form with a row's keys dealt to 64 lanes; so it is 2.7e-7 and 3.0e-7,
// for 0 (d 64) and 4 % (d 128) of the time.
// Bound on small shapes by the round trips of its look-ups and first loads: 44 -> 14 us for 380 tokens of 4 heads, d 64,
// over 256 and 192 keys, the two prompts' own attention 2 x 37 -> 11 us in one launch (one wavefront per row, its lanes
// walking the keys one by one, before).  8 wavefronts with heads of 64 channels (14.8 us with 4); 4 with 128, whose partial
// outputs would not fit LDS otherwise.
typedef __attribute__((ext_vector_type(4))) float gen_f32x4;

// 4 consecutive elements from element index idx (a multiple of 4)
__device__ inline void load4(const void *base, int64_t idx, int dtype, float out[4])
{
    if (dtype == SGC_F32) {
        const float4 a = *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + idx);
        out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    } else if (dtype == SGC_BF16) {
        const uint2 a = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(base) + idx);
        out[0] = __uint_as_float(a.x << 16);
        out[1] = __uint_as_float(a.x & 0xFFFF0000u);
        out[2] = __uint_as_float(a.y << 16);
        out[3] = __uint_as_float(a.y & 0xFFFF0000u);
    } else {
        const uint32_t a = *reinterpret_cast<const uint32_t *>(static_cast<const uint8_t *>(base) + idx);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = e4m3_to_f32((uint8_t)(a >> (8 * i)));
    }
}

// Channels [q D/4, (q + 1) D/4) of a head vector at element index row, rotated at pos (rotate-half: a channel's partner is
// D/2 away, in the vector's other half).
template <int D>
__device__ inline void load_rotated_quarter(const void *base, int64_t row, int dtype, const float2 *rope, int64_t pos, int q, float out[D / 4])
{
    constexpr int half = D / 2;
    const int c0 = q * (D / 4), t0 = c0 & (half - 1);
    const float sign = c0 < half ? -1.f : 1.f;
#pragma unroll
    for (int i = 0; i < D / 4; i += 8) {
        float x[8];
        load8(base, row + c0 + i, dtype, x);
        if (rope) {
            float y[8];
            load8(base, row + (c0 ^ half) + i, dtype, y);
            const float2 *tab = rope + pos * half + t0 + i;
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = x[e] * tab[e].x + sign * (y[e] * tab[e].y);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) out[i + e] = x[e];
    }
}

__device__ __forceinline__ const AttnArgs &generic_args(const AttnArgs &a) { return a; }
__device__ __forceinline__ const AttnArgs &generic_args(const CarriedGeneric &c) { return c.a; }

// ARGS: AttnArgs, or CarriedGeneric, whose tables are read where they arrive, among the launch's arguments.
template <int D, int NW, int IO, int KV, typename ARGS>
__global__ void __launch_bounds__(NW * 64) attn_generic_kernel(const ARGS args)
{
    constexpr bool CARRIED = std::is_same_v<ARGS, CarriedGeneric>;
    const AttnArgs &a = generic_args(args);
    constexpr int NQ = D / 4, NB = D / 16, LD = D + 4;
    __shared__ __attribute__((aligned(16))) float o_s[NW][16][LD];
    __shared__ float m_s[NW][16], l_s[NW][16];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int j = lane & 15, q = lane >> 4;
    const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, g = a.group;
    const int hk = blockIdx.y;

    // ---- the lane's row (rows past the end repeat the last one)
    const void *q_base = a.q;
    void *o_base = a.o;
    float *lse_base = a.lse;
    int64_t lse_stride = a.lse_stride;
    int cluster = 0, P, n_rows, row0, tok_base = 0;
    int t_sq_lo = 0, t_sq_hi = 0;            // (carried) the tile's queries
    const int32_t *pt;
    if constexpr (CARRIED) {
        const CarriedGeneric::Tile t = args.tiles[blockIdx.x];
        const CarriedGeneric::Unit &u = args.units[t.unit];
        row0 = t.row0;
        t_sq_lo = t.sq_lo;
        t_sq_hi = t.sq_hi;
        P = u.prefix_len;
        pt = args.pages + u.page0;
        if (a.mode == MODE_SUFFIX) {
            tok_base = u.tok_base;
            n_rows = u.n_tokens * g;
        } else {
            n_rows = P * g;
            q_base = u.q;
            o_base = u.o;
            lse_base = u.lse;
            lse_stride = P;
        }
    } else if (a.mode == MODE_SUFFIX) {
        const GenericTile t = a.gtiles[blockIdx.x];
        cluster = t.unit;
        row0 = t.row0;
        pt = a.page_table + a.cl_pt_off[cluster];
        P = a.cl_prefix_len[cluster];
        tok_base = a.cl_tok_off[cluster];
        n_rows = (a.cl_tok_off[cluster + 1] - tok_base) * g;
    } else {
        const GenericTile t = a.gtiles[blockIdx.x];
        const PrefixJob &job = a.jobs[t.unit];
        row0 = t.row0;
        cluster = job.cluster;
        pt = a.page_table + a.cl_pt_off[cluster];
        P = job.prefix_len;
        n_rows = P * g;
        q_base = job.q;
        o_base = job.o;
        lse_base = job.lse;
        lse_stride = P;
    }
    auto row_of = [&](int i, int &head, int &src, int &qpos, int &sq) {
        const int r = min(row0 + i, n_rows - 1), tk = r / g;
        head = hk * g + (r - tk * g);
        if (CARRIED && a.mode == MODE_SUFFIX) {
            if constexpr (CARRIED) {
                const int tok = tok_base + tk;
                CarriedGeneric::Query mine = args.queries[t_sq_lo];
                sq = t_sq_lo;
                for (int k = t_sq_lo + 1; k <= t_sq_hi; ++k) {
                    const CarriedGeneric::Query other = args.queries[k];
                    if (tok >= other.tok0) {
                        mine = other;
                        sq = k;
                    }
                }
                qpos = tok - mine.tok0;
                src = mine.src0 + qpos;
            }
        } else if (a.mode == MODE_SUFFIX) {
            src = a.tok_src[tok_base + tk];
            qpos = a.tok_qpos[tok_base + tk];
            sq = a.tok_sq[tok_base + tk];
        } else {
            src = qpos = tk;
            sq = 0;
        }
    };
    int head, src, qpos, sq;
    row_of(j, head, src, qpos, sq);
    const int last_qpos = __shfl(qpos, 15), sq_lo = __shfl(sq, 0), sq_hi = __shfl(sq, 15);
    const int n_cache = a.mode == MODE_SUFFIX ? P : qpos + 1;            // cached keys the row sees
    const int n_blocks = ((a.mode == MODE_SUFFIX ? P : last_qpos + 1) + 15) / 16;
    float qf[NQ];
    load_rotated_quarter<D>(q_base, ((int64_t)src * Hq + head) * D, IO, a.rope, (a.mode == MODE_SUFFIX ? P : 0) + qpos, q, qf);

    float k_scale = 1.f, v_scale = 1.f;
    if (KV == SGC_FP8_E4M3) {
        const float *sc = a.kv_scale + ((int64_t)cluster * a.n_layers + a.layer) * 2 * Hkv;
        k_scale = sc[hk];
        v_scale = sc[Hkv + hk];
    }
    gen_f32x4 O[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) O[cb] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -1e30f, l = 0.f;
    // A key that a row does not see has weight 0 in the second product, and 0 x Inf and 0 x NaN are NaN.  Where some row does
    // not see some key, values that are not finite are therefore taken out of the product (vf gets zeros) and added here, to the
    // rows that see their key.
    // (j and q by value: captured by reference q lived in scratch memory)
    auto add_nonfinite = [j, q](const float (&p)[4], float (&vf)[NB][4], int keep, gen_f32x4 (&sum)[NB]) {
        for (int qq = 0; qq < 4; ++qq) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float w = __shfl(p[r], j + 16 * qq);
                const bool sees = r < __shfl(keep, j + 16 * qq);
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v = __shfl(vf[cb][r], 4 * q + e + 16 * qq);
                        if (sees && !(v * 0.f == 0.f)) sum[cb][e] += w * v;
                    }
            }
        }
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) vf[cb][r] = vf[cb][r] * 0.f == 0.f ? vf[cb][r] : 0.f;
    };
    // one block of 16 keys: kf = the lane's key's channels, vf = channel 16 cb + j of keys 4 q .. 4 q + 3, keep = first
    // invisible of the lane's four keys
    auto block = [&](const float (&kf)[NQ], float (&vf)[NB][4], float scale, int keep) {
        gen_f32x4 part[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) part[i] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NQ; ++c) part[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c], qf[c], part[c & 1], 0, 0, 0);
        gen_f32x4 s = part[0] + part[1];
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = r < keep ? s[r] * scale : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx), alpha = exp2f(m - m_new);
        m = m_new;
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = exp2f(s[r] - m_new);
        l = fmaf(l, alpha, (p[0] + p[1]) + (p[2] + p[3]));
        gen_f32x4 seen[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) seen[cb] = gen_f32x4{0.f, 0.f, 0.f, 0.f};
        if (__any(keep < 4)) {
            float z = 0.f;                  // NaN if one of the lane's values is not finite
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) z = fmaf(vf[cb][r], 0.f, z);
            if (__any(!(z == 0.f))) add_nonfinite(p, vf, keep, seen);
        }
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) seen[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[cb][r], p[r], seen[cb], 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) O[cb][r] = fmaf(O[cb][r], alpha, seen[cb][r]);
        }
    };

    // ---- cached keys: a block is a page
    auto fetch = [&](int b, float (&kf)[NQ], float (&vf)[NB][4]) {
        const int page = pt[b];
        const char *kp = a.pool.k_part(a.layer, page, hk), *vp = a.pool.v_part(a.layer, page, hk);
#pragma unroll
        for (int i = 0; i < NQ; i += 8) load8(kp, k_page_index(j, q * NQ + i), k_elem_type(KV), kf + i);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) load4(vp, v_page_index(4 * q, 16 * cb + j), KV, vf[cb]);
    };
    {
        float kf[NQ], vf[NB][4];
        if (wave < n_blocks) fetch(wave, kf, vf);
        for (int b = wave; b < n_blocks; b += NW) {
            float kn[NQ], vn[NB][4];
            fetch(min(b + NW, n_blocks - 1), kn, vn);              // the next block's loads travel meanwhile
            if (KV == SGC_FP8_E4M3) {
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) vf[cb][r] *= v_scale;
            }
            block(kf, vf, a.scale_log2e * k_scale, n_cache - (16 * b + 4 * q));
#pragma unroll
            for (int i = 0; i < NQ; ++i) kf[i] = kn[i];
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) vf[cb][r] = vn[cb][r];
        }
    }
    // ---- the suffix keys of every query the rows belong to, rotated at P + key on the way
    if (a.mode == MODE_SUFFIX) {
        int turn = n_blocks;
        for (int si = sq_lo; si <= sq_hi; ++si) {
            int len, first;
            if constexpr (CARRIED) {
                len = args.queries[si].len;
                first = args.queries[si].src0;
            } else {
                len = a.sq_len[si];
                first = a.sq_src0[si];
            }
            const int n_own = si == sq_hi ? last_qpos + 1 : len;
            const int64_t src0 = first;
            for (int b = 0; b * 16 < n_own; ++b, ++turn) {
                if (turn % NW != wave) continue;
                float kf[NQ], vf[NB][4];
                const int key = min(16 * b + j, n_own - 1);
                load_rotated_quarter<D>(a.k, ((src0 + key) * Hkv + hk) * D, IO, a.rope, P + key, q, kf);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t vrow = ((src0 + min(16 * b + 4 * q + r, n_own - 1)) * Hkv + hk) * D;
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb) vf[cb][r] = load1(a.v, vrow + 16 * cb + j, IO);
                }
                block(kf, vf, a.scale_log2e, sq == si ? qpos + 1 - (16 * b + 4 * q) : 0);
            }
        }
    }
    // ---- merge the wavefronts' states: lane (j, q) holds channels 16 cb + 4 q .. + 3 of row j
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (q == 0) {
        m_s[wave][j] = m;
        l_s[wave][j] = l;
    }
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) *reinterpret_cast<gen_f32x4 *>(&o_s[wave][j][16 * cb + 4 * q]) = O[cb];
    __syncthreads();
    const int i = threadIdx.x >> 4, c0 = (threadIdx.x & 15) * NB;         // row i, channels c0 .. c0 + NB - 1
    if (i >= 16) return;
    if (row0 + i >= n_rows) return;
    row_of(i, head, src, qpos, sq);
    float M = m_s[0][i];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, m_s[w][i]);
    float sum[NB], L = 0.f;
#pragma unroll
    for (int c = 0; c < NB; ++c) sum[c] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = exp2f(m_s[w][i] - M);
        L += f * l_s[w][i];
#pragma unroll
        for (int c = 0; c < NB; ++c) sum[c] += f * o_s[w][i][c0 + c];
    }
    const float inv = 1.0f / L;
    const int64_t orow = ((int64_t)src * Hq + head) * D + c0;
    if (IO == SGC_F32) {
#pragma unroll
        for (int c = 0; c < NB; c += 4)
            *reinterpret_cast<float4 *>(static_cast<float *>(o_base) + orow + c) = make_float4(sum[c] * inv, sum[c + 1] * inv, sum[c + 2] * inv, sum[c + 3] * inv);
    } else {
#pragma unroll
        for (int c = 0; c < NB; c += 4) {
            uint2 y;
            y.x = (uint32_t)f32_to_bf16(sum[c] * inv) | ((uint32_t)f32_to_bf16(sum[c + 1] * inv) << 16);
            y.y = (uint32_t)f32_to_bf16(sum[c + 2] * inv) | ((uint32_t)f32_to_bf16(sum[c + 3] * inv) << 16);
            *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(o_base) + orow + c) = y;
        }
    }
    if (lse_base && (threadIdx.x & 15) == 0)
        lse_base[(int64_t)head * lse_stride + (a.mode == MODE_SUFFIX ? src : qpos)] = (M + log2f(L)) * 0.6931471805599453f;
}

}  // namespace

// ---- launchers -------------------------------------------------------------------------------
hipError_t launch_rope_table(float2 *table, int n_pos, int head_dim, double base, hipStream_t s)
{
    const int half = head_dim / 2;
    const int64_t n = (int64_t)n_pos * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, table, n_pos, half, base,
                       1.0 / (double)head_dim);
    return hipGetLastError();
}

hipError_t launch_prefix_ingest(const PoolGeom &g, int layer, const int32_t *d_page_table, const PrefixJob *d_jobs,
                                int n_jobs, const int32_t *d_page_job, int n_pages, const int32_t *d_chunk_page0, float *d_amax,
                                int n_chunks, int io_dtype, const float2 *rope, const ExpandArgs *expand, hipStream_t s)
{
    if (n_pages == 0 || n_jobs == 0) return expand ? launch_expand_tiles(*expand, s) : hipSuccess;
    ExpandArgs ex{};
    if (expand) ex = *expand;
    const dim3 grid_all(n_pages + expand_columns(ex.n, g.n_kv_heads), g.n_kv_heads);
    if (g.kv_dtype == SGC_FP8_E4M3) {
        hipLaunchKernelGGL(ingest_amax_kernel, dim3(n_chunks, g.n_kv_heads), dim3(256), 0, s, d_jobs, d_page_job, d_chunk_page0, d_amax,
                           g.n_kv_heads, g.head_dim, rope);
        if (g.head_dim == 128)
            hipLaunchKernelGGL(ingest_write_fp8_kernel<128>, grid_all, dim3(128), 0, s, g, layer, d_page_table, d_jobs, d_page_job, n_pages,
                               d_amax, rope, ex);
        else
            hipLaunchKernelGGL(ingest_write_fp8_kernel<64>, grid_all, dim3(128), 0, s, g, layer, d_page_table, d_jobs, d_page_job, n_pages,
                               d_amax, rope, ex);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(ingest_write_kernel, grid_all, dim3(128), 2 * (size_t)g.head_part_bytes, s, g, layer, d_page_table, d_jobs,
                       d_page_job, n_pages, io_dtype, rope, ex);
    return hipGetLastError();
}

static CopyPiece copy_piece_of(void *dst, const void *mapped_src, size_t bytes)
{
    return {static_cast<copy_u32x4 *>(dst), static_cast<const copy_u32x4 *>(mapped_src), bytes / 16, (bytes % 16) / 4};
}

// Limits: what fits the launch's arguments, and a done word for every workgroup that reads staged tables.
static_assert(sizeof(PoolGeom) + 2 * sizeof(CopyPiece) + sizeof(CopyDone) + sizeof(ExpandArgs) + sizeof(float2 *) + 5 * 8 + 256 <= kSmallIngestOtherArgs,
              "arguments of ingest_small_kernel beside jobs and pages");
constexpr int kIngestThreads = 128;
struct SmallGroups {
    int copy, expand;
};
static SmallGroups small_groups(int n_tiles, size_t staged_bytes)
{
    if (n_tiles <= kOneGroupTiles && staged_bytes <= kOneGroupBytes) return {1, 0};
    const size_t per_group = 16 * 8 * kIngestThreads;
    return {(int)std::min<size_t>((staged_bytes + per_group - 1) / per_group, 16), (n_tiles + kIngestThreads - 1) / kIngestThreads};
}
SmallIngestUse small_ingest_use(const PoolGeom &g, int n_jobs, int n_pages, int n_tiles, size_t staged_bytes)
{
    const SmallGroups n = small_groups(n_tiles, staged_bytes);
    if (g.kv_dtype == SGC_FP8_E4M3 || n_jobs > SmallIngest::kJobs || n_pages > SmallIngest::kPages || n.copy + n.expand > kCopyDoneWords)
        return SMALL_INGEST_NO;
    return n.expand > 0 ? SMALL_INGEST_STAGED_TABLES : SMALL_INGEST_COPIED_TABLES;
}

hipError_t launch_small_ingest(const PoolGeom &g, int layer, const SmallIngest &small, int n_pages, int io_dtype, const float2 *rope, void *dst,
                               const void *mapped_src, size_t bytes, void *dst2, const void *mapped_src2, size_t bytes2, const CopyDone &done,
                               int *n_words, const ExpandArgs *expand, hipStream_t s)
{
    const CopyPiece a = copy_piece_of(dst, mapped_src, bytes), b = copy_piece_of(dst2, mapped_src2, bytes2);
    ExpandArgs ex{};
    if (expand) ex = *expand;
    const auto [copy_groups, expand_groups] = bytes + bytes2 > 0 ? small_groups(ex.n, bytes + bytes2) : SmallGroups{0, 0};
    if (n_words) *n_words = copy_groups + expand_groups;
    const int columns = (copy_groups + expand_groups + g.n_kv_heads - 1) / g.n_kv_heads;
    // (arguments are copied with every launch: a short prompt does not send the 3.6 KB that ten may need: 39.3 us with them, 39.0 without)
    if (small.n_jobs <= SmallIngestShort::kJobs && n_pages <= SmallIngestShort::kPages) {
        SmallIngestShort few;
        few.n_jobs = small.n_jobs;
        std::copy(small.jobs, small.jobs + small.n_jobs, few.jobs);
        std::copy(small.pages, small.pages + n_pages, few.pages);
        hipLaunchKernelGGL(ingest_small_kernel<SmallIngestShort>, dim3(n_pages + columns, g.n_kv_heads), dim3(kIngestThreads),
                           2 * (size_t)g.head_part_bytes, s, g, layer, few, n_pages, io_dtype, rope, a, b, copy_groups, expand_groups, done, ex);
    } else {
        hipLaunchKernelGGL(ingest_small_kernel<SmallIngest>, dim3(n_pages + columns, g.n_kv_heads), dim3(kIngestThreads), 2 * (size_t)g.head_part_bytes, s,
                           g, layer, small, n_pages, io_dtype, rope, a, b, copy_groups, expand_groups, done, ex);
    }
    return hipGetLastError();
}

hipError_t launch_expand_tiles(const ExpandArgs &e, hipStream_t s)
{
    if (e.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(expand_tiles_kernel, dim3((e.n + 127) / 128), dim3(128), 0, s, e);
    return hipGetLastError();
}

hipError_t launch_suffix_ingest(const AttnArgs &a, int n_spages, const ExpandArgs *expand, hipStream_t s)
{
    if (n_spages <= 0) return expand ? launch_expand_tiles(*expand, s) : hipSuccess;
    const size_t lds = 2 * (size_t)kPageTokens * a.head_dim * 2;
    ExpandArgs ex{};
    if (expand) ex = *expand;
    const dim3 grid(n_spages + expand_columns(ex.n, a.n_kv_heads), a.n_kv_heads);
    hipLaunchKernelGGL(suffix_ingest_kernel, grid, dim3(128), lds, s, a, n_spages, ex);
    return hipGetLastError();
}

hipError_t launch_decode_own_keys(const DecodeArgs &d, hipStream_t s)
{
    if (d.n_sq <= 0) return hipSuccess;
    const int g = d.n_q_heads / d.n_kv_heads;
    if (d.use_mfma && g <= 16) {                  // head_dim 128, bf16 rows: the matrix-core form
        const int units = d.n_sq * d.n_kv_heads;
        hipLaunchKernelGGL(decode_own_keys_mfma_kernel, dim3((units + 3) / 4), dim3(256), 0, s, d);
        return hipGetLastError();
    }
    if (d.n_splits > kDecodeDotSplits) return hipErrorInvalidValue;          // (no plan does)
    const int G = g % 8 == 0 ? 8 : g % 4 == 0 ? 4 : g % 2 == 0 ? 2 : 1;      // heads per wavefront
    const dim3 grid((unsigned)((int64_t)d.n_sq * (d.n_q_heads / G)));
    const size_t lds = (size_t)G * (128 * 2 + (size_t)d.key_cap * (4 + 2));      // q rows (bf16), scores (fp32), weights (bf16)
    switch (G) {
        case 8: hipLaunchKernelGGL(decode_own_keys_kernel<8>, grid, dim3(64), lds, s, d); break;
        case 4: hipLaunchKernelGGL(decode_own_keys_kernel<4>, grid, dim3(64), lds, s, d); break;
        case 2: hipLaunchKernelGGL(decode_own_keys_kernel<2>, grid, dim3(64), lds, s, d); break;
        default: hipLaunchKernelGGL(decode_own_keys_kernel<1>, grid, dim3(64), lds, s, d); break;
    }
    return hipGetLastError();
}

// The same by one workgroup, which then writes the tile records that are put together from what it has copied: a launch less
// (its boundary and its own look-ups) for the tables of ordinary batches.
__global__ void __launch_bounds__(1024) copy_and_expand_kernel(CopyPiece a, CopyPiece b, CopyDone done, ExpandArgs e)
{
    copy_piece(a, threadIdx.x, blockDim.x);
    copy_piece(b, threadIdx.x, blockDim.x);
    signal_read(done, 0);          // (its barrier is also what the records below wait for)
    for (int i = threadIdx.x; i < e.n; i += blockDim.x) expand_one_tile(e, i);
}

hipError_t launch_copy_from_host(void *dst, const void *mapped_src, size_t bytes, hipStream_t s, void *dst2,
                                 const void *mapped_src2, size_t bytes2, const ExpandArgs *expand, const CopyDone &done, int *n_words)
{
    *n_words = 0;
    if (bytes == 0 && bytes2 == 0) return expand ? launch_expand_tiles(*expand, s) : hipSuccess;
    const CopyPiece a = copy_piece_of(dst, mapped_src, bytes), b = copy_piece_of(dst2, mapped_src2, bytes2);
    if (expand && expand->n > 0 && expand->n <= kOneLaunchTiles && bytes + bytes2 <= kOneGroupBytes) {
        *n_words = 1;
        hipLaunchKernelGGL(copy_and_expand_kernel, dim3(1), dim3(1024), 0, s, a, b, done, *expand);
        return hipGetLastError();
    }
    const size_t most = std::max(a.n16, b.n16);
    const unsigned blocks = (unsigned)std::min<size_t>(std::max<size_t>((most + 255) / 256, 1), kCopyDoneWords);
    *n_words = (int)blocks;
    hipLaunchKernelGGL(copy_from_host_kernel, dim3(blocks), dim3(256), 0, s, a, b, done);
    return expand ? launch_expand_tiles(*expand, s) : hipGetLastError();
}

hipError_t launch_fill_zero_bytes(void *p, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    const size_t n16 = bytes / 16;      // callers pass multiples of 16 bytes
    const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_zero_bytes_kernel, dim3(blocks), dim3(256), 0, s, static_cast<uint4 *>(p), n16);
    return hipGetLastError();
}

hipError_t launch_cache_export(const PoolGeom &g, int layer, const int32_t *d_pages, int prefix_len, void *k, void *v,
                               hipStream_t s)
{
    const int64_t n = (int64_t)prefix_len * g.n_kv_heads * g.head_dim;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
    if (g.kv_bytes == 4)
        hipLaunchKernelGGL(cache_export_kernel<uint32_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (uint32_t *)k, (uint32_t *)v);
    else if (g.kv_bytes == 2)
        hipLaunchKernelGGL(cache_export_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (uint16_t *)k, (uint16_t *)v);
    else
        hipLaunchKernelGGL(cache_export_kernel<uint8_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (uint8_t *)k, (uint8_t *)v);
    return hipGetLastError();
}

hipError_t launch_cache_import(const PoolGeom &g, int layer, const int32_t *d_pages, int prefix_len, const void *k,
                               const void *v, hipStream_t s)
{
    const int n_pages = (prefix_len + kPageTokens - 1) / kPageTokens;
    const int64_t n = (int64_t)n_pages * kPageTokens * g.n_kv_heads * g.head_dim;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
    if (g.kv_bytes == 4)
        hipLaunchKernelGGL(cache_import_kernel<uint32_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (const uint32_t *)k, (const uint32_t *)v);
    else if (g.kv_bytes == 2)
        hipLaunchKernelGGL(cache_import_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (const uint16_t *)k, (const uint16_t *)v);
    else
        hipLaunchKernelGGL(cache_import_kernel<uint8_t>, dim3(blocks), dim3(256), 0, s, g, layer, d_pages, prefix_len,
                           (const uint8_t *)k, (const uint8_t *)v);
    return hipGetLastError();
}

template <int IO, int KV, typename ARGS>
static hipError_t launch_generic(const ARGS &args, const AttnArgs &a, int n_gtiles, hipStream_t s)
{
    const dim3 grid(n_gtiles, a.n_kv_heads);
    if (a.head_dim == 64)
        hipLaunchKernelGGL((attn_generic_kernel<64, 8, IO, KV, ARGS>), grid, dim3(512), 0, s, args);
    else
        hipLaunchKernelGGL((attn_generic_kernel<128, 4, IO, KV, ARGS>), grid, dim3(256), 0, s, args);
    return hipGetLastError();
}
template <typename ARGS>
static hipError_t launch_generic(const ARGS &args, const AttnArgs &a, int n_gtiles, hipStream_t s)
{
    if (n_gtiles <= 0) return hipSuccess;
    if (a.io_dtype == SGC_F32) return launch_generic<SGC_F32, SGC_F32>(args, a, n_gtiles, s);
    if (a.pool.kv_dtype == SGC_BF16) return launch_generic<SGC_BF16, SGC_BF16>(args, a, n_gtiles, s);
    if constexpr (std::is_same_v<ARGS, AttnArgs>)
        return launch_generic<SGC_BF16, SGC_FP8_E4M3>(args, a, n_gtiles, s);
    else
        return hipErrorInvalidValue;          // (no call carries the tables of an fp8 cache)
}
hipError_t launch_attn_generic(const AttnArgs &a, int n_gtiles, hipStream_t s) { return launch_generic(a, a, n_gtiles, s); }
hipError_t launch_attn_generic(const CarriedGeneric &c, int n_gtiles, hipStream_t s) { return launch_generic(c, c.a, n_gtiles, s); }

}  // namespace sgc
