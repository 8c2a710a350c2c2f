// Matrix-core attention kernel of libsgc for gfx950 (MI355X), head_dim 128: first product on binary16 operands
// (rotated keys and queries; on the e4m3 codes of an fp8 cache in the QK8 variant), second product on bf16.
//
// SubGCache (arXiv 2505.10951) Sec. 3.4: every query of a cluster appends its question tokens to
// the cluster's cached prompt.  One workgroup takes a tile of rows that all belong to one
// (cluster, KV head): rows are (query, token, head-in-group) of ANY query of the cluster, so the
// cached prefix K/V tiles staged in LDS are shared by several queries at once.  After the
// prefix keys the same rows run causally over their own query's suffix keys.
//
// Matrix-core mapping (v_mfma_f32_32x32x16_f16 / _bf16, 64-lane wavefronts):
//   S^T = K Q^T : A = 32 keys x 16 channels (from LDS), B = 16 channels x 32 rows (Q, registers).
//                 Lane (n, h) = (lane % 32, lane / 32) then owns row n and, in accumulator
//                 register r, key 8 (r / 4) + 4 h + r % 4: a row's scores sit in ONE lane pair, so
//                 the row max/sum need a single exchange between the two 32-lane halves.
//   O^T = V^T P^T : A = 32 channels x 16 keys (from LDS, V is stored transposed per 16-token page),
//                 B = 16 keys x 32 rows = the probabilities exactly as the score accumulator
//                 holds them (registers 8 kb .. 8 kb + 7), no cross-lane movement.
// A key tile is 64 keys = 4 pages; in LDS it is the linear image of those pages (8 parts of 4 KiB:
// K of the 4 pages, then V), copied global -> LDS without passing through registers.
//
// Softmax is online, fp32, base 2.  The reference maximum of a row is set from the first tile it
// sees and afterwards only raised (with a rescale of the accumulators) when a tile's weights
// against it would sum beyond 2^30, or in tiles that need masking; the result is the same
// softmax, since any reference that avoids overflow gives the same quotient.  The row sum adds
// the weights after their rounding to bf16, the values the second product uses.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sgc_internal.h"
#include "sgc_own_keys.h"

namespace sgc {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int D = 128;                       // head dim
constexpr int BN = 64;                       // keys per LDS tile (4 pages)
constexpr int PART_BYTES = kPageTokens * D * 2;   // one page's K (or V) of one head as bf16: 4 KiB
constexpr int HALF_BYTES = 4 * PART_BYTES;   // the K (or V) of one 64-key tile: 16 KiB
constexpr int NW = 4, MI = 1;                // wavefronts of a workgroup, 32-row blocks of a wavefront
constexpr int K8_PART_BYTES = kPageTokens * D;    // one page's K of one head as e4m3 codes: 2 KiB
constexpr int K8_PART_STRIDE = K8_PART_BYTES + 128;   // in LDS consecutive pages sit 2 KiB + 128 bytes apart: the two pages
                                                      // a 32-key operand read touches then fall into different banks
constexpr int OWN_PAGES = BN / kPageTokens;   // pages of own-suffix keys in one of the K (V) buffers
constexpr float kKeepBelow = 1073741824.0f;  // 2^30: a tile's weights may sum to this against a stale maximum

// Combine a value with the one held by the lane 32 away (the other half of a score row), through
// v_permlane32_swap: with both operands x, the two results hold x's lower half and x's upper half, each
// in all 64 lanes.
__device__ inline float half_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Unpacks 2 fp8 e4m3 codes (low or high half of w) to 16-bit floats: binary16 for keys, bf16 for values (both
// exact: e4m3 is a subset of either).
template <bool TO_F16>
__device__ inline uint32_t fp8x2_to_16x2(uint32_t w, bool high)
{
    if (TO_F16) {
        const auto r = high ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, false);
        return __builtin_bit_cast(uint32_t, r);
    }
    const auto r = high ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    return __builtin_bit_cast(uint32_t, r);
}

// A record that no launch writes while it is read, at a wave-uniform address: through the scalar path, into scalar registers.
// (The compiler must take a plain load for one that a store of the same kernel could change, and fetch it per lane.)
template <typename T>
__device__ inline T uniform_record(const T *p)
{
    const auto *words = (const __attribute__((address_space(4))) uint32_t *)p;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) w[i] = words[i];
    return __builtin_bit_cast(T, w);
}

// V operands of two pages of token rows: eight blocks (page i / 4, 32-channel group i % 4) for the second product, read
// transposed (ds_read_b64_tr_b16): of the 16 lanes of a group, lane 4 t + u asks for channels 4 u .. 4 u + 3 of token t and gets
// channel (lane % 16) of all four tokens; the second read of a block is eight tokens further.  at: LDS address per block.  One asm block with
// its wait: in front of the builtin the compiler waits for every copy to LDS in flight, the next chunk's among them.
__device__ __forceinline__ void read_v_rows(const uint32_t (&at)[8], bf16x8 (&out)[8])
{
    s16x4 v[16];
    asm volatile("ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %8, %20\n\tds_read_b64_tr_b16 %9, %20 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %10, %21\n\tds_read_b64_tr_b16 %11, %21 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %12, %22\n\tds_read_b64_tr_b16 %13, %22 offset:2048\n\t"
                 "ds_read_b64_tr_b16 %14, %23\n\tds_read_b64_tr_b16 %15, %23 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]),
                   "=&v"(v[8]), "=&v"(v[9]), "=&v"(v[10]), "=&v"(v[11]), "=&v"(v[12]), "=&v"(v[13]), "=&v"(v[14]), "=&v"(v[15])
                 : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7])
                 : "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[2 * i], v[2 * i + 1], 0, 1, 2, 3, 4, 5, 6, 7));
}

// 4 KiB global -> LDS as four 1 KiB instructions, 16 bytes per lane: byte 1024 q + 16 lane of the source
// lands at the same offset of lds_part.  The four share one address pair and differ in the immediate.
__device__ inline void copy_4k_to_lds(const char *src_lane, char *lds_part)
{
    const auto *g = (const __attribute__((address_space(1))) void *)src_lane;
    auto *l = (__attribute__((address_space(3))) void *)lds_part;
    __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
    __builtin_amdgcn_global_load_lds(g, l, 16, 1024, 0);
    __builtin_amdgcn_global_load_lds(g, l, 16, 2048, 0);
    __builtin_amdgcn_global_load_lds(g, l, 16, 3072, 0);
}

// Rows 16 HF .. 16 HF + 15 of a wavefront's 32 x 128 block of bf16 query rows, from the lanes that loaded them whole
// (a_jj: 16-byte chunk lane % 16 of row 4 jj + lane / 16 of the half) to the lanes that use them as matrix operands (lane
// (n, h) of row n: chunks 2 kb + h and 8 + 2 kb + h), through 4 KiB of LDS that belongs to this wavefront alone.
// The chunks of row r sit permuted by r % 16, so that both the writes and the reads cover all banks.
template <int HF>
__device__ __forceinline__ void q_turn_half(char *qst, const uint4 &a0, const uint4 &a1, const uint4 &a2, const uint4 &a3, int lane, int n,
                                            int h, uint4 (&qlo)[4], uint4 (&qhi)[4])
{
    {
        const int r0 = lane >> 4, c = lane & 15;      // a_jj: chunk c of row 4 jj + r0 of the half
        *reinterpret_cast<uint4 *>(qst + (r0 + 0) * 256 + ((c ^ (r0 + 0)) * 16)) = a0;
        *reinterpret_cast<uint4 *>(qst + (r0 + 4) * 256 + ((c ^ (r0 + 4)) * 16)) = a1;
        *reinterpret_cast<uint4 *>(qst + (r0 + 8) * 256 + ((c ^ (r0 + 8)) * 16)) = a2;
        *reinterpret_cast<uint4 *>(qst + (r0 + 12) * 256 + ((c ^ (r0 + 12)) * 16)) = a3;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    const int n16 = n & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        const uint4 lo = *reinterpret_cast<const uint4 *>(qst + n16 * 256 + (((2 * kb + h) ^ n16) * 16));
        const uint4 hi = *reinterpret_cast<const uint4 *>(qst + n16 * 256 + (((8 + 2 * kb + h) ^ n16) * 16));
        if ((n >> 4) == HF) {
            qlo[kb] = lo;
            qhi[kb] = hi;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Decode (SubGCache App. A.2: up to 32 generated tokens per query): the blocks behind the tiles of a decode
// step's launch append the step's new token of every query to its suffix pages, K rotated at position
// P + len + step, V as given; 8 lanes per (sorted query, KV head), one 8-channel chunk of each half per lane.
// Nothing in the same launch reads those pages (the tiles of a decode step only read the cluster's cache).
__device__ inline void append_new_tokens(const AttnArgs &a, int blk)
{
    const int unit = blk * ((int)blockDim.x >> 3) + ((int)threadIdx.x >> 3), cc = (int)threadIdx.x & 7;
    const int Hkv = a.n_kv_heads;
    const int sq = unit / Hkv, hk = unit - sq * Hkv;
    if (sq >= a.n_append) return;
    const int j = a.sq_len[sq] + a.pos_shift;
    const int pos = a.cl_prefix_len[a.sq_cluster[sq]] + j;
    const int tok = j % kPageTokens;
    char *kp = const_cast<char *>(a.spool) + (int64_t)(a.sq_page0[sq] + j / kPageTokens) * 2 * Hkv * PART_BYTES + (int64_t)hk * PART_BYTES;
    char *vp = kp + (int64_t)Hkv * PART_BYTES;
    const int64_t row = ((int64_t)a.sq_query[sq] * Hkv + hk) * D;
    const uint16_t *kg = static_cast<const uint16_t *>(a.k) + row, *vg = static_cast<const uint16_t *>(a.v) + row;
    const uint4 k1 = *reinterpret_cast<const uint4 *>(kg + cc * 8), k2 = *reinterpret_cast<const uint4 *>(kg + D / 2 + cc * 8);
    const uint4 v1 = *reinterpret_cast<const uint4 *>(vg + cc * 8), v2 = *reinterpret_cast<const uint4 *>(vg + D / 2 + cc * 8);
    const uint32_t w1[4] = {k1.x, k1.y, k1.z, k1.w}, w2[4] = {k2.x, k2.y, k2.z, k2.w};
    uint32_t o1[4], o2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x1[2] = {__uint_as_float(w1[i] << 16), __uint_as_float(w1[i] & 0xFFFF0000u)};
        float x2[2] = {__uint_as_float(w2[i] << 16), __uint_as_float(w2[i] & 0xFFFF0000u)};
        if (a.rope) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float2 cs = a.rope[(int64_t)pos * (D / 2) + cc * 8 + 2 * i + e];
                rotate_pair(x1[e], x2[e], cs.x, cs.y);
            }
        }
        o1[i] = pack2_f16(x1[0], x1[1]);       // keys are kept as binary16
        o2[i] = pack2_f16(x2[0], x2[1]);
    }
    *reinterpret_cast<uint4 *>(kp + (int64_t)k_page_index(tok, cc * 8) * 2) = make_uint4(o1[0], o1[1], o1[2], o1[3]);
    *reinterpret_cast<uint4 *>(kp + (int64_t)k_page_index(tok, D / 2 + cc * 8) * 2) = make_uint4(o2[0], o2[1], o2[2], o2[3]);
    const uint32_t y1[4] = {v1.x, v1.y, v1.z, v1.w}, y2[4] = {v2.x, v2.y, v2.z, v2.w};
    uint16_t *vq = reinterpret_cast<uint16_t *>(vp);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        vq[v_page_index(tok, cc * 8 + i)] = (uint16_t)(y1[i >> 1] >> (16 * (i & 1)));
        vq[v_page_index(tok, D / 2 + cc * 8 + i)] = (uint16_t)(y2[i >> 1] >> (16 * (i & 1)));
    }
}

__device__ __forceinline__ const AttnArgs &attn_args(const AttnArgs &a) { return a; }
template <typename ARGS>
__device__ __forceinline__ const AttnArgs &attn_args(const ARGS &c) { return c.a; }

// QK8 (fp8 cache only): the first product runs on the cache's e4m3 codes as they are (v_mfma_scale_f32_32x32x64_f8f6f4,
// twice the bf16 rate): the rotated, scaled query row is quantised to e4m3 with a power-of-two scale of its own, which
// the instruction applies to the row's products in hardware, so scores come out in the same units as on the other
// paths.  K codes then go to LDS as they are (2 KiB per page part); V is still widened to bf16 for the second product.
//
// OWN_RAW: the question tokens' keys and values are taken as the caller gives them (a.k, a.v), rotated and turned on their
// way into LDS; otherwise they are read from the suffix page pool.
//
// ARGS: AttnArgs, or CarriedSuffix / CarriedPrefix, whose tables are read where they arrive, among the launch's arguments.
template <bool KV_FP8, int MODE, bool QK8, bool OWN_RAW, typename ARGS>
__global__ void __launch_bounds__(NW * 64, 2) attn_mfma_kernel(const ARGS args)
{
    constexpr bool CARRIED = !std::is_same_v<ARGS, AttnArgs>;
    static_assert(!CARRIED || (!KV_FP8 && std::is_same_v<ARGS, std::conditional_t<MODE == MODE_PREFIX, CarriedPrefix, CarriedSuffix>>), "tables of the mode");
    const AttnArgs &a = attn_args(args);
    static_assert(NW == 4 && MI == 1, "the own-suffix part deals pages to four wavefronts of 32 rows");
    static_assert(!QK8 || KV_FP8, "the fp8 first product needs an fp8 cache");
    if (!CARRIED && MODE == MODE_SUFFIX && (int)blockIdx.x >= a.n_tiles) {
        append_new_tokens(a, (int)blockIdx.x - a.n_tiles);
        return;
    }
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int n = lane & 31, h = lane >> 5;
    const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, g = a.group;

    // ---- which tile ----
    Tile t;
    const int32_t *page_table = a.page_table;
    const SuffixPage *spages = a.spages;
    // where the rows come from and go to: the batch's packed arrays, or (prefix mode) the job's
    const void *q_base = a.q;
    void *o_base = a.o;
    float *lse_base = a.lse;
    int64_t lse_stride = a.lse_stride;
    if constexpr (CARRIED) {
        const auto *c = (const __attribute__((address_space(4))) ARGS *)__builtin_amdgcn_kernarg_segment_ptr();
        page_table = (const int32_t *)c->pages;
        t.tok_base = 0;
        t.pad = 0;
        t.n_q = 0;
        t.cluster = 0;
        if constexpr (MODE == MODE_PREFIX) {
            const uint32_t code = c->tiles[blockIdx.x];
            const CarriedJob job = uniform_record((const CarriedJob *)&c->jobs[code >> 28]);
            t.hk = (code >> 18) & 1023;
            t.row0 = (code & 0x3FFFF) * NW * MI * 32;
            t.n_rows = min(NW * MI * 32, job.prefix_len * a.group - t.row0);
            t.prefix_len = job.prefix_len;
            t.pt_off = job.page0;
            t.own_page0 = t.n_own_pages = 0;
            q_base = job.q;
            o_base = job.o;
            lse_base = job.lse;
            lse_stride = job.prefix_len;
        } else {
            spages = (const SuffixPage *)c->own_pages;
            const TileSeed sd = uniform_record((const TileSeed *)&c->tiles[blockIdx.x]);
            const auto cl = uniform_record((const CarriedSuffix::Cluster *)&c->clusters[sd.cluster]);
            t.hk = sd.hk;
            t.row0 = sd.row0;
            t.n_rows = sd.n_rows;
            t.prefix_len = cl.prefix_len;
            t.pt_off = cl.page0;
            t.tok_base = cl.tok_base;
            t.n_q = sd.sq_hi - sd.sq_lo + 1;          // (kTileQueries at most)
#pragma unroll
            for (int k = 0; k < kTileQueries; ++k) {
                const TileQuery tq = uniform_record((const TileQuery *)&c->queries[min(sd.sq_lo + k, sd.sq_hi)]);
                t.q[k] = tq;
                if (k >= t.n_q) t.q[k].tok0 = INT32_MAX;
                if (k == 0) t.own_page0 = tq.own0;
                t.n_own_pages = tq.own0 - t.own_page0 + sd.last_qpos / kPageTokens + 1;      // (the last of them is query sq_hi)
            }
        }
        const int last_page = max((t.prefix_len + kPageTokens - 1) / kPageTokens - 1, 0);
#pragma unroll
        for (int k = 0; k < 12; ++k) t.first_pages[k] = t.prefix_len > 0 ? uniform_record(page_table + t.pt_off + min(k, last_page)) : 0;
        if (t.n_rows <= 0) return;
    } else {
        t = uniform_record(a.tiles + blockIdx.x);
        // (the whole record is asked for before its first use decides anything: one round trip)
        asm volatile("" ::"s"(t.n_rows), "s"(t.prefix_len), "s"(t.pad), "s"(t.first_pages[0]), "s"(t.first_pages[11]), "s"(t.q[0].tok0), "s"(t.q[3].own0),
                     "s"(t.own_page0));
        if (t.n_rows == 0) return;
        if (MODE == MODE_PREFIX) {
            const PrefixJob job = uniform_record(a.jobs + __builtin_amdgcn_readfirstlane(t.tok_base));
            q_base = job.q;
            o_base = job.o;
            lse_base = job.lse;
            lse_stride = t.prefix_len;
            t.tok_base = 0;
        }
    }
    // decode tiles cover one key range of the cluster's cache: own output set, positions continue behind ALL cached keys
    const int key_range = __builtin_amdgcn_readfirstlane(t.pad) >> 24;
    const int pos_extra = __builtin_amdgcn_readfirstlane(t.pad) & 0xFFFFFF;
    if (MODE == MODE_SUFFIX) {
        o_base = static_cast<char *>(o_base) + key_range * a.split_o_bytes;
        if (lse_base) lse_base += key_range * a.split_lse_elems;
    }
    // everything that steers the tile loop is made explicitly wave-uniform (scalar registers)
    const int cluster = __builtin_amdgcn_readfirstlane(t.cluster), hk = __builtin_amdgcn_readfirstlane(t.hk);
    t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
    t.n_rows = __builtin_amdgcn_readfirstlane(t.n_rows);
    const int P = __builtin_amdgcn_readfirstlane(t.prefix_len);
    const int n_pages = (P + kPageTokens - 1) / kPageTokens;
    const int32_t *pt = page_table + __builtin_amdgcn_readfirstlane(t.pt_off);
    const int tok_base = __builtin_amdgcn_readfirstlane(t.tok_base);
    const int last_row = t.row0 + t.n_rows - 1;

    // ---- copy machinery ----------------------------------------------------------------------------
    // A tile is 8 parts: K of its 4 pages, then V of its 4 pages; a part is 4 KiB of bf16 (2 KiB of fp8
    // codes that widen to 4 KiB).  Wavefront w moves K and V of page w.  A part's source is a scalar base (pool base +
    // page offset) plus a per-lane offset fixed for the launch; page ids are loaded a step or more ahead, on the scalar path:
    // no copy waits for them, and waiting for them is not waiting for copies.
    const int my_page = wave_u & 3;
    const char *cache_base = a.pool.pool + (int64_t)a.layer * a.pool.layer_bytes + (int64_t)hk * a.pool.head_part_bytes;
    const uint32_t cache_v_off = (uint32_t)(Hkv * a.pool.head_part_bytes);
    const char *spool_base = a.spool + (int64_t)hk * PART_BYTES;
    const uint32_t spool_v_off = (uint32_t)Hkv * PART_BYTES;
    const int64_t spool_page = 2 * (int64_t)spool_v_off;
    // fp8 cache only: codes on their way to LDS.  A 2 KiB part is fetched as four runs of 512 codes, 8 per lane; widened,
    // a lane's 8 codes are 16 bytes at 16 * lane of the run's 1 KiB image, so the stores cover all banks.
    uint2 stage[8];      // [K runs 0..3, V runs 0..3]
    bool staged_k = false, staged_v = false;

    // Page indices past the last page are clamped to it: such keys are masked out of the scores, and what
    // they multiply in the second product is finite cache content times a zero weight.
    auto cache_page = [&](int kt) __attribute__((always_inline)) -> int {       // id of this wavefront's page of tile kt
        if (n_pages == 0) return 0;       // no cached keys: nothing is ever copied from the cache
        return uniform_record(pt + min(kt * 4 + my_page, n_pages - 1));
    };
    auto cache_src = [&](int page) __attribute__((always_inline)) -> const char * { return cache_base + (int64_t)page * a.pool.page_bytes; };
    const uint32_t lane16 = lane * 16;
    char *kdst_codes = nullptr;      // QK8: where the next K tile's codes go
    auto issue_load_fp8 = [&](int page_k, bool want_k, int page_v, bool want_v) __attribute__((always_inline)) {
        staged_k = want_k;
        staged_v = want_v;
        if (staged_k) {
            const char *src = cache_src(page_k) + lane16;
            if (QK8) {      // the codes as they are, straight into LDS (kdst_codes: set by the caller)
                const auto *g = (const __attribute__((address_space(1))) void *)src;
                auto *l = (__attribute__((address_space(3))) void *)(kdst_codes + my_page * K8_PART_STRIDE);
                __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
                __builtin_amdgcn_global_load_lds(g, l, 16, 1024, 0);
                staged_k = false;
            } else {
                const char *src8 = cache_src(page_k) + lane * 8;
#pragma unroll
                for (int r = 0; r < 4; ++r) stage[r] = *reinterpret_cast<const uint2 *>(src8 + r * 512);
            }
        }
        if (staged_v) {
            const char *src8 = cache_src(page_v) + cache_v_off + lane * 8;
#pragma unroll
            for (int r = 0; r < 4; ++r) stage[4 + r] = *reinterpret_cast<const uint2 *>(src8 + r * 512);
        }
    };
    // 8 codes -> 8 16-bit floats = 16 bytes
    auto widen_to_lds = [&](const uint2 &codes, char *dst, auto f16_tag) __attribute__((always_inline)) {
        constexpr bool F = decltype(f16_tag)::value;
        uint4 o;
        o.x = fp8x2_to_16x2<F>(codes.x, false); o.y = fp8x2_to_16x2<F>(codes.x, true);
        o.z = fp8x2_to_16x2<F>(codes.y, false); o.w = fp8x2_to_16x2<F>(codes.y, true);
        *reinterpret_cast<uint4 *>(dst) = o;
    };
    // Writes what the last issue_load_fp8 staged; a staged half is written once, and only to a real buffer.
    auto store_fp8 = [&](char *kdst, char *vdst) __attribute__((always_inline)) {
        if (staged_k && kdst) {
#pragma unroll
            for (int r = 0; r < 4; ++r) widen_to_lds(stage[r], kdst + my_page * PART_BYTES + r * 1024 + lane * 16, std::true_type{});
        }
        if (staged_v && vdst) {
#pragma unroll
            for (int r = 0; r < 4; ++r) widen_to_lds(stage[4 + r], vdst + my_page * PART_BYTES + r * 1024 + lane * 16, std::false_type{});
        }
        staged_k = false;
        staged_v = false;
    };
    // K of one cached tile (this wavefront's page_k of it) and / or V of another: kdst / vdst null = none
    auto fetch_cache = [&](int page_k, char *kdst, int page_v, char *vdst) __attribute__((always_inline)) {
        if (KV_FP8) {
            kdst_codes = kdst;
            issue_load_fp8(page_k, kdst != nullptr, page_v, vdst != nullptr);
        } else {
            if (kdst) copy_4k_to_lds(cache_src(page_k) + lane16, kdst + my_page * PART_BYTES);
            if (vdst) copy_4k_to_lds(cache_src(page_v) + cache_v_off + lane16, vdst + my_page * PART_BYTES);
        }
    };
    auto land_cache = [&](char *kdst, char *vdst) __attribute__((always_inline)) {   // make what was fetched visible in LDS (before the barrier)
        if (KV_FP8) store_fp8(kdst, vdst);
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): direct copies have landed
    };
    char *const kbuf0 = smem, *const vbuf0 = smem + 2 * HALF_BYTES;
    auto kbuf_of = [&](int i) __attribute__((always_inline)) -> char * { return kbuf0 + (i & 1) * HALF_BYTES; };
    auto vbuf_of = [&](int i) __attribute__((always_inline)) -> char * { return vbuf0 + (i & 1) * HALF_BYTES; };

    // The first cached tiles are requested before anything else: page ids now, the copies (bf16 cache) as soon
    // as the ids are there, so that they travel while Q is loaded and rotated.
    const int n_cache_keys = (MODE == MODE_SUFFIX) ? P : min(P, last_row / g + 1);
    const int n_kt = (n_cache_keys + BN - 1) / BN;
    // This wavefront's pages of tiles 0, 1, 2 come with the tile record; the steps take pg_v, of tile kt + 1, and pg_k, of tile
    // kt + 2.
    auto of_wave = [&](const int32_t *p4) __attribute__((always_inline)) -> int {
        const int p0 = __builtin_amdgcn_readfirstlane(p4[0]), p1 = __builtin_amdgcn_readfirstlane(p4[1]);
        const int p2 = __builtin_amdgcn_readfirstlane(p4[2]), p3 = __builtin_amdgcn_readfirstlane(p4[3]);
        const int lo = (my_page & 1) ? p1 : p0, hi = (my_page & 1) ? p3 : p2;
        return (my_page & 2) ? hi : lo;
    };
    const int pg0 = of_wave(t.first_pages), pg1 = of_wave(t.first_pages + 4), pg2 = of_wave(t.first_pages + 8);
    int pg_v = pg1, pg_k = pg2;
    float k_scale = 1.f, v_scale = 1.f;
    if (KV_FP8 && P > 0) {      // (nothing has written the scales of a cluster without cached keys)
        const float *sc = a.kv_scale + ((int64_t)cluster * a.n_layers + a.layer) * 2 * Hkv;
        k_scale = sc[hk];
        v_scale = sc[Hkv + hk];
    }
    // Scores are kept in log2 units.  Q carries the factor for cached keys; scores against the (unquantised)
    // suffix keys of the batch are brought to the same units by self_ratio.
    const float c_cache = a.scale_log2e * k_scale;
    const float self_ratio = KV_FP8 ? 1.0f / k_scale : 1.0f;

    // ---- per-lane row bookkeeping ----
    const bool inline_queries = MODE == MODE_SUFFIX && __builtin_amdgcn_readfirstlane(t.n_q) <= kTileQueries;
    int tq_tok0[kTileQueries], tq_src0[kTileQueries], tq_own0[kTileQueries];
#pragma unroll
    for (int k = 0; k < kTileQueries; ++k) {
        tq_tok0[k] = __builtin_amdgcn_readfirstlane(t.q[k].tok0);
        tq_src0[k] = __builtin_amdgcn_readfirstlane(t.q[k].src0);
        tq_own0[k] = __builtin_amdgcn_readfirstlane(t.q[k].own0);
    }
    // Own keys are numbered by slots, 16 to a page, over the own pages of all queries the tile touches: page 0 is the
    // first page of the tile's first query, and the last one holds the tile's last row's own key.
    const bool own = MODE == MODE_SUFFIX && !a.skip_self;
    const int own_page0 = __builtin_amdgcn_readfirstlane(t.own_page0), n_own = own ? __builtin_amdgcn_readfirstlane(t.n_own_pages) : 0;
    bool valid[MI];
    int64_t io_row[MI];     // element offset of the row in q / o
    int qpos[MI], lim[MI], src_tok[MI], head[MI];
    int own_first = 0;      // slot of the first key of the row's query
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int r = t.row0 + (wave * MI + mi) * 32 + n;
        valid[mi] = r <= last_row;
        const int rc = valid[mi] ? r : last_row;
        const int tk = rc / g;
        head[mi] = hk * g + (rc - tk * g);
        if (MODE == MODE_SUFFIX) {
            const int tau = tok_base + tk;
            if (inline_queries) {        // which of the (at most 4) queries of the tile record the token belongs to
                const bool ge1 = tau >= tq_tok0[1], ge2 = tau >= tq_tok0[2], ge3 = tau >= tq_tok0[3];
                const int first = ge3 ? tq_tok0[3] : ge2 ? tq_tok0[2] : ge1 ? tq_tok0[1] : tq_tok0[0];
                const int src0 = ge3 ? tq_src0[3] : ge2 ? tq_src0[2] : ge1 ? tq_src0[1] : tq_src0[0];
                qpos[mi] = tau - first;
                src_tok[mi] = src0 + qpos[mi];
                own_first = ((ge3 ? tq_own0[3] : ge2 ? tq_own0[2] : ge1 ? tq_own0[1] : tq_own0[0]) - own_page0) * kPageTokens;
            } else {
                const TokInfo ti = a.tok_info[tau];
                src_tok[mi] = ti.src;
                qpos[mi] = ti.qpos;
                own_first = (ti.own0 - own_page0) * kPageTokens;
            }
            lim[mi] = P;
        } else {
            src_tok[mi] = tk;
            qpos[mi] = tk;
            lim[mi] = tk + 1;
        }
        io_row[mi] = ((int64_t)src_tok[mi] * Hq + head[mi]) * D;
    }
    // wave-uniform bounds of the visible cached keys.  Rows are in
    // sorted order (and rows past the tile's end repeat its last row), so the first lane holds the minima
    // and lane 31 of the last row block the maxima.
    const int lim_min = __builtin_amdgcn_readlane(lim[0], 0), lim_max = __builtin_amdgcn_readlane(lim[MI - 1], 31);

    if (!KV_FP8 && n_kt > 0) {
        fetch_cache(pg0, kbuf_of(0), pg0, vbuf_of(0));
        if (n_kt > 1) fetch_cache(pg1, kbuf_of(1), 0, nullptr);
    }
    // ---- Q: load, rotate at position P + qpos (suffix) / qpos (prefix), keep as B operands ----
    // All loads of the phase (Q row halves, then the rotation table entries) are issued before any of them is
    // used, so the phase costs one memory round trip and not one per channel group.
    f16x8 qf[MI][8];
    i32x8 q8[2];            // QK8: the row as e4m3 codes, operand t = channels 64 t .. 64 t + 63 in the order kc_block reads keys
    int qscale = 127;       // QK8: the row's scale as a biased power-of-two exponent (what the scaled product takes)
    {
        uint4 qlo[MI][4], qhi[MI][4];
        float4 cs[MI][4][4];            // (cos, sin) of two channels per entry
        const bool rotate = a.rope != nullptr;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) cs[mi][kb][i] = make_float4(1.f, 0.f, 1.f, 0.f);
        if (rotate) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const int pos = (MODE == MODE_SUFFIX ? P + pos_extra + a.pos_shift : 0) + qpos[mi];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    const float4 *tab = reinterpret_cast<const float4 *>(a.rope + (int64_t)pos * 64 + kb * 16 + h * 8);
#pragma unroll
                    for (int i = 0; i < 4; ++i) cs[mi][kb][i] = tab[i];
                }
            }
        }
        if (!KV_FP8) {       // (with an fp8 cache the registers for it are not there, and prompts are long)
            // The operand layout wants 16-byte pieces of 32 different rows per instruction.  Loaded that way the
            // requests are 32 scattered 32-byte runs each; instead instruction j fetches rows 4 j .. 4 j + 3 whole
            // (lane = 16-byte chunk lane % 16 of row 4 j + lane / 16), and the wavefront turns the block by
            // passing it, 16 rows at a time, through its 4 KiB share of the V buffer that nothing uses before the
            // first step (chunks of row r permuted by r % 16: writes and reads cover all banks).
            char *const qst = smem + 3 * HALF_BYTES + wave * 4096;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const int row_index = (int)(io_row[mi] / D);        // src_tok * Hq + head of this lane's row
                auto whole_row_chunk = [&](int j) __attribute__((always_inline)) -> uint4 {
                    const int64_t ro = (int64_t)__shfl(row_index, 4 * j + (lane >> 4)) * D;
                    return *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(q_base) + ro + (lane & 15) * 8);
                };
                const uint4 r0 = whole_row_chunk(0), r1 = whole_row_chunk(1), r2 = whole_row_chunk(2), r3 = whole_row_chunk(3);
                const uint4 r4 = whole_row_chunk(4), r5 = whole_row_chunk(5), r6 = whole_row_chunk(6), r7 = whole_row_chunk(7);
                q_turn_half<0>(qst, r0, r1, r2, r3, lane, n, h, qlo[mi], qhi[mi]);
                q_turn_half<1>(qst, r4, r5, r6, r7, lane, n, h, qlo[mi], qhi[mi]);
            }
        } else {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const uint16_t *qrow = static_cast<const uint16_t *>(q_base) + io_row[mi];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    const int c0 = kb * 16 + h * 8;
                    qlo[mi][kb] = *reinterpret_cast<const uint4 *>(qrow + c0);
                    qhi[mi][kb] = *reinterpret_cast<const uint4 *>(qrow + 64 + c0);
                }
            }
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const uint32_t wl[4] = {qlo[mi][kb].x, qlo[mi][kb].y, qlo[mi][kb].z, qlo[mi][kb].w};
                const uint32_t wh[4] = {qhi[mi][kb].x, qhi[mi][kb].y, qhi[mi][kb].z, qhi[mi][kb].w};
                float x1[8], x2[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a0 = __uint_as_float(wl[i] << 16), a1 = __uint_as_float(wl[i] & 0xFFFF0000u);
                    const float b0 = __uint_as_float(wh[i] << 16), b1 = __uint_as_float(wh[i] & 0xFFFF0000u);
                    const float4 t4 = cs[mi][kb][i];
                    x1[2 * i] = a0;
                    x2[2 * i] = b0;
                    x1[2 * i + 1] = a1;
                    x2[2 * i + 1] = b1;
                    rotate_sums(x1[2 * i], x2[2 * i], t4.x, t4.y);
                    rotate_sums(x1[2 * i + 1], x2[2 * i + 1], t4.z, t4.w);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {      // the score scale (log2 units, cached-K scale included) rides on Q
                    qf[mi][kb][i] = (_Float16)(x1[i] * c_cache);
                    qf[mi][kb + 4][i] = (_Float16)(x2[i] * c_cache);
                }
            }
        }
        if constexpr (QK8) {
            // The row as e4m3 codes with one power-of-two scale: largest magnitude of the row (both lanes of the pair)
            // = m 2^x with m in [0.5, 1); values times 2^(8 - x) lie below 256 (the format reaches 448), rounded to
            // nearest even by the conversion instruction.
            float amax = 0.f;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb)
#pragma unroll
                for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)qf[0][kb][i]));
            amax = half_max(amax);
            int e = __builtin_amdgcn_frexp_expf(amax) - 8;
            e = amax > 0.f ? max(-120, min(e, 120)) : 0;
            qscale = 127 + e;
            const float down = __uint_as_float((uint32_t)(127 - e) << 23);      // 2^-e
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int pc = 0; pc < 4; ++pc) {
                    const f16x8 v = qf[0][4 * t + pc];
                    int w0 = 0, w1 = 0;
                    w0 = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[0] * down, (float)v[1] * down, w0, false);
                    w0 = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[2] * down, (float)v[3] * down, w0, true);
                    w1 = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[4] * down, (float)v[5] * down, w1, false);
                    w1 = __builtin_amdgcn_cvt_pk_fp8_f32((float)v[6] * down, (float)v[7] * down, w1, true);
                    q8[t][2 * pc] = w0;
                    q8[t][2 * pc + 1] = w1;
                }
        }
    }

    // ---- accumulators ----
    // m_ref is the reference maximum of the row's softmax; the score products start from -m_ref (neg_ref, the
    // same value in all 16 accumulator registers of a lane, which all belong to one row), so finished scores
    // are already relative to it.  seen: the row has met at least one visible key.
    // (With 64 rows per wavefront the registers for neg_ref are not there: FOLD is off, the products start
    // from zero and the weights subtract m_ref themselves.)
    constexpr bool FOLD = MI == 1;
    f32x16 oacc[MI][4], neg_ref[MI];
    float m_ref[MI], l_part[MI];
    bool seen[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        m_ref[mi] = 0.f;
        l_part[mi] = 0.f;
        seen[mi] = false;
#pragma unroll
        for (int r = 0; r < 16; ++r) neg_ref[mi][r] = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[mi][db][r] = 0.f;
    }
    bool fresh = true;     // no tile processed yet by this wavefront

    // Per-lane LDS offsets of the operand blocks.  K block (nb, kb): lane (m, hh) reads key m of the 32-key
    // group nb (page 2 nb + m / 16, token m % 16), channels kb * 16 + hh * 8 .. + 7.  Each 16-lane group
    // reads 256 contiguous bytes, which is conflict-free.  V block (pg, db) is 1 KiB contiguous.
    const int lane_koff = ((n >> 4) * PART_BYTES) + (h * kPageTokens + (n & 15)) * 16;
    const int lane_voff = lane * 16;

    // ---- the pieces of one 32-key half step ---------------------------------------------------------
    // A 64-key tile is worked on as two 32-key halves (nb = 0, 1): half nb is K blocks 8 nb .. 8 nb + 7 of
    // the first product (one per 16 channels) and V blocks 8 nb .. 8 nb + 7 of the second (pages 2 nb and
    // 2 nb + 1, four 32-channel groups each).  LDS operand blocks are read through a rolling window of 8
    // register sets: each matrix instruction is followed by the read that refills the slot it used with a
    // block of the NEXT product, so that product never waits on LDS.
    bf16x8 frag[8];
    uint32_t pf[MI][2][4];     // weights of one half as bf16 pairs: [row block][page of the half][register pair]
    float psum[MI];
    auto k_block = [&](const char *kbuf, int nb, int kb) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8 *>(kbuf + lane_koff + nb * 2 * PART_BYTES + kb * 512);
    };
    auto v_block = [&](const char *vbuf, int nb, int i) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8 *>(vbuf + lane_voff + (nb * 8 + i) * 1024);
    };
    // Cached keys.  QK8: the 64-channel operand of the fp8 product is eight 8-byte pieces (lane (m, hh): key m, channels
    // 64 t + 16 p + 8 hh .. + 7 for p = 0..3; the contraction does not care which of its 64 slots a channel takes as
    // long as the query operand uses the same ones); window slot i < 4 holds pieces 2 (i % 2), 2 (i % 2) + 1 of operand
    // t = i / 2, slots 4..7 are not used by this product.
    const int lane_k8off = (n >> 4) * K8_PART_STRIDE + (h * kPageTokens + (n & 15)) * 8;
    auto kc_block = [&](const char *kbuf, int nb, int i) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (QK8) {
            if (i >= 4) return frag[i];
            const char *p = kbuf + lane_k8off + nb * 2 * K8_PART_STRIDE + (4 * (i >> 1) + 2 * (i & 1)) * 256;
            const uint2 a0 = *reinterpret_cast<const uint2 *>(p), a1 = *reinterpret_cast<const uint2 *>(p + 256);
            const u32x4 w = {a0.x, a0.y, a1.x, a1.y};
            return __builtin_bit_cast(bf16x8, w);
        } else {
            return k_block(kbuf, nb, i);
        }
    };
    auto no_refill = [&](int) __attribute__((always_inline)) {};
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // S^T = K Q^T - m_ref for the half whose K blocks the window holds; slot kb is refilled by refill(kb).
    auto qk_half = [&](f32x16 (&s)[MI], auto refill) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                s[mi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, frag[kb]), qf[mi][kb], kb == 0 ? (FOLD ? neg_ref[mi] : zero16) : s[mi], 0, 0, 0);
            refill(kb);
        }
    };
    // The same against cached keys.  QK8: two 64-channel products on the codes; the query row's own scale (a power of two)
    // is applied by the instruction, so the scores leave it in the usual units with -m_ref already taken off.
    auto qk_half_cache = [&](f32x16 (&s)[MI], auto refill) __attribute__((always_inline)) {
        if constexpr (QK8) {
            refill(4);
            refill(5);
            refill(6);
            refill(7);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u32x4 lo = __builtin_bit_cast(u32x4, frag[2 * t]), hi = __builtin_bit_cast(u32x4, frag[2 * t + 1]);
                const i32x8 kop = {(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
                s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kop, q8[t], t == 0 ? neg_ref[0] : s[0], 0, 0, 0, 127, 0, qscale);
                refill(2 * t);
                refill(2 * t + 1);
            }
        } else {
            qk_half(s, refill);
        }
    };
    // O^T += V^T P^T for the half whose V blocks the window holds (slot i = page i / 4, channel group i % 4).
    auto pv_half = [&](auto refill) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) l_part[mi] += psum[mi];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int pg = i >> 2, db = i & 3;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const u32x4 w = {pf[mi][pg][0], pf[mi][pg][1], pf[mi][pg][2], pf[mi][pg][3]};
                oacc[mi][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i], __builtin_bit_cast(bf16x8, w), oacc[mi][db], 0, 0, 0);
            }
            refill(i);
        }
    };
    // Weights of one half from scores relative to the reference maximum: one exp2 per score.
    auto weights = [&](const f32x16 (&s)[MI]) __attribute__((always_inline)) {
        bf16x2 ones;
        ones[0] = (__bf16)1.0f;
        ones[1] = (__bf16)1.0f;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            float acc = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                bf16x2 pk;
                pk[0] = (__bf16)__builtin_amdgcn_exp2f(FOLD ? s[mi][r] : s[mi][r] - m_ref[mi]);
                pk[1] = (__bf16)__builtin_amdgcn_exp2f(FOLD ? s[mi][r + 1] : s[mi][r + 1] - m_ref[mi]);
                acc = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, acc, false);   // sum of the ROUNDED weights
                pf[mi][r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
            }
            psum[mi] = acc;
        }
    };
    auto weights_overflow = [&]() __attribute__((always_inline)) {       // wave-uniform: some row's weights of this half summed beyond the limit
        bool bad = false;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) bad |= !(psum[mi] <= kKeepBelow);    // also catches inf / nan
        return __any(bad);
    };
    // The careful part of a softmax step, run before weights().  Masks the half through keep(mi, j) = "row mi
    // may see key j of the tile" when `masked`; raises the reference maximum to the half's own where that is
    // larger (rows that have seen no key yet take it as it is), rescales the accumulators and re-bases the
    // scores.  Returns nothing; m_ref, neg_ref, seen, l_part, oacc and s are updated.
    auto raise_reference = [&](f32x16 (&s)[MI], const int nb, const bool masked, auto keep) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            if (masked) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = nb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                    if (!keep(mi, j)) s[mi][r] = -INFINITY;
                }
            }
            float tmax = s[mi][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, s[mi][r]);
            tmax = half_max(tmax);
            const bool has = tmax > -INFINITY;
            if (!FOLD) tmax -= m_ref[mi];                      // relative to m_ref (FOLD: the scores already are)
            const float delta = seen[mi] ? fmaxf(tmax, 0.f) : (has ? tmax : 0.f);     // new m_ref - old m_ref
            if (__any(delta != 0.f)) {
                const float alpha = seen[mi] ? __builtin_amdgcn_exp2f(-delta) : 1.0f;
                m_ref[mi] += delta;
                l_part[mi] *= alpha;
#pragma unroll
                for (int db = 0; db < 4; ++db) {       // one accumulator block at a time keeps the temporaries few
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[mi][db][r] *= alpha;
                    if (MI > 1) __builtin_amdgcn_sched_barrier(0);
                }
                if (FOLD) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        s[mi][r] -= delta;
                        neg_ref[mi][r] = -m_ref[mi];
                    }
                }
            }
            seen[mi] = seen[mi] || has;
        }
    };
    auto keep_all = [&](int, int) __attribute__((always_inline)) { return true; };
    // fp8 cache only: scores against suffix keys were formed with the cached-K scale on Q; undo it.  mb is the
    // reference maximum the product was started from.
    auto rescale_self = [&](f32x16 (&s)[MI], const float (&mb)[MI]) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[mi][r] = FOLD ? (s[mi][r] + mb[mi]) * self_ratio - mb[mi] : s[mi][r] * self_ratio;
    };

    // ---- cached prefix tiles, software pipelined ------------------------------------------------------
    // The two products of a half frame its softmax: while the vector unit turns the scores of half j into
    // weights, the matrix unit already forms the scores of half j + 1 (independent instruction streams in
    // one straight-line region); then comes the second product of half j.  So K runs one tile ahead of V:
    // during tile step kt, K of tile kt + 2 and V of tile kt + 1 are copied into LDS while K of tile kt + 1
    // and V of tile kt are read.  At the top of step kt a wavefront holds the scores of (kt, half 0) and, in
    // its window, the K blocks of (kt, half 1).
    const int n_my = min(n_kt, (lim_max + BN - 1) / BN);      // tiles this wavefront has rows for
    f32x16 s0[MI], s1[MI];
    if (n_kt > 0) {
        if (KV_FP8) {      // through registers: one tile's worth at a time
            fetch_cache(pg0, kbuf_of(0), pg0, vbuf_of(0));
            land_cache(kbuf_of(0), vbuf_of(0));
            if (n_kt > 1) {
                fetch_cache(pg1, kbuf_of(1), 0, nullptr);
                land_cache(kbuf_of(1), nullptr);
            }
        } else {
            land_cache(nullptr, nullptr);
        }
    }
    __syncthreads();
    if (n_my > 0) {
        const char *k0 = kbuf_of(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) frag[i] = kc_block(k0, 0, i);
        qk_half_cache(s0, [&](int i) __attribute__((always_inline)) { frag[i] = kc_block(k0, 1, i); });
    }
    __syncthreads();       // every wavefront has read K of tile 0 before step 0 overwrites it
    // ---- own-suffix keys: bringing pages into LDS -----------------------------------------------------------
    // The tile's own pages come in chunks of four, one page per wavefront, double buffered: chunk i in K buffer i & 1 and, counted
    // from the one that the last cached step leaves free, V buffer i & 1.
    auto own_kbuf = [&](int i) __attribute__((always_inline)) -> char * { return kbuf_of(i); };
    auto own_vbuf = [&](int i) __attribute__((always_inline)) -> char * { return vbuf_of(n_kt + i); };
    // (lane_again: per-lane offsets are worked out where they are used; kept from one use to the next they would push others out
    // of the registers)
    auto lane_again = [&]() __attribute__((always_inline)) -> int {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // Starts the copy of this wavefront's page of chunk i.  OWN_RAW: the rows as given, 256 bytes a token, tokens past the query's
    // end repeating its last one; the 16-byte chunks of K's row r sit permuted by r, those of V's by 4 (r % 4), so that what
    // reads them below covers all banks.
    auto own_copy = [&](int i) __attribute__((always_inline)) {
        const int p = i * OWN_PAGES + wave_u;
        if (p >= n_own) return;
        char *kd = own_kbuf(i) + wave_u * PART_BYTES, *vd = own_vbuf(i) + wave_u * PART_BYTES;
        const SuffixPage pg = uniform_record(spages + own_page0 + p);
        if constexpr (OWN_RAW) {
            const int l = lane_again(), r0 = l >> 4, c = l & 15;
#pragma unroll
            for (int j = 0; j < 4; ++j) {           // rows 4 j .. 4 j + 3 of the page
                const int r = 4 * j + r0;
                const int64_t row = ((int64_t)(pg.row0 + min(r, pg.n - 1)) * Hkv + hk) * (D * 2);
                const auto *gk = (const __attribute__((address_space(1))) void *)(static_cast<const char *>(a.k) + row + ((c ^ r) * 16));
                const auto *gv = (const __attribute__((address_space(1))) void *)(static_cast<const char *>(a.v) + row + ((c ^ (4 * r0)) * 16));
                __builtin_amdgcn_global_load_lds(gk, (__attribute__((address_space(3))) void *)(kd + j * 1024), 16, 0, 0);
                __builtin_amdgcn_global_load_lds(gv, (__attribute__((address_space(3))) void *)(vd + j * 1024), 16, 0, 0);
            }
        } else {
            const char *src = spool_base + pg.page * spool_page + lane16;
            copy_4k_to_lds(src, kd);
            copy_4k_to_lds(src + spool_v_off, vd);
        }
    };
    // OWN_RAW: this wavefront's page of chunk i is rotated in place and put into the pages' order: lane (r, c0) = (lane % 16,
    // lane / 16) takes the 16-byte chunks c0, c0 + 4 of token r and their partners 8 further.  own_table requests the rotation's
    // entries ahead of that.
    float4 own_cs[2][4];
    auto own_table = [&](int i) __attribute__((always_inline)) {
        if constexpr (OWN_RAW) {
            const int p = i * OWN_PAGES + wave_u;
            if (p >= n_own) return;
            const SuffixPage pg = uniform_record(spages + own_page0 + p);
            const int l = lane_again(), pos = pg.pos0 + min(l & 15, pg.n - 1);
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    own_cs[k][e] = a.rope ? reinterpret_cast<const float4 *>(a.rope + (int64_t)pos * (D / 2) + ((l >> 4) + 4 * k) * 8)[e]
                                          : make_float4(1.f, 0.f, 1.f, 0.f);
        }
    };
    auto own_rotate = [&](int i) __attribute__((always_inline)) {
        if constexpr (OWN_RAW) {
            if (i * OWN_PAGES + wave_u >= n_own) return;
            const int l = lane_again(), r = l & 15, c0 = l >> 4;
            char *kp = own_kbuf(i) + wave_u * PART_BYTES;
            uint4 lo[2], hi[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int c = c0 + 4 * k;
                lo[k] = *reinterpret_cast<const uint4 *>(kp + r * 256 + ((c ^ r) * 16));
                hi[k] = *reinterpret_cast<const uint4 *>(kp + r * 256 + (((c + 8) ^ r) * 16));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int c = c0 + 4 * k;
                const uint32_t wl[4] = {lo[k].x, lo[k].y, lo[k].z, lo[k].w}, wh[4] = {hi[k].x, hi[k].y, hi[k].z, hi[k].w};
                uint32_t o1[4], o2[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float a0 = __uint_as_float(wl[e] << 16), a1 = __uint_as_float(wl[e] & 0xFFFF0000u);
                    float b0 = __uint_as_float(wh[e] << 16), b1 = __uint_as_float(wh[e] & 0xFFFF0000u);
                    const float4 t4 = own_cs[k][e];
                    rotate_pair(a0, b0, t4.x, t4.y);
                    rotate_pair(a1, b1, t4.z, t4.w);
                    o1[e] = pack2_f16(a0, a1);
                    o2[e] = pack2_f16(b0, b1);
                }
                *reinterpret_cast<uint4 *>(kp + c * 256 + r * 16) = make_uint4(o1[0], o1[1], o1[2], o1[3]);
                *reinterpret_cast<uint4 *>(kp + (c + 8) * 256 + r * 16) = make_uint4(o2[0], o2[1], o2[2], o2[3]);
            }
        }
    };

    // One part's copy: per-lane source address and LDS destination.  Issued as four 1 KiB instructions that
    // the steady-state step spreads between its matrix instructions, so that a wavefront never sits on a
    // full memory-instruction queue while the matrix unit idles.
    struct PartCopy {
        const char *src;
        char *dst;
    };
    auto cache_part = [&](bool is_v, int page, char *dst_half) __attribute__((always_inline)) -> PartCopy {
        return {cache_src(page) + (is_v ? cache_v_off : 0u) + lane16, dst_half + my_page * PART_BYTES};
    };
    auto copy_quarter = [&](const PartCopy &pc, int slot) __attribute__((always_inline)) {     // slot 0, 2, 4, 6 -> quarter 0..3; odd slots: nothing
        const auto *gp = (const __attribute__((address_space(1))) void *)pc.src;
        auto *lp = (__attribute__((address_space(3))) void *)pc.dst;
        switch (slot) {
            case 0: __builtin_amdgcn_global_load_lds(gp, lp, 16, 0, 0); break;
            case 2: __builtin_amdgcn_global_load_lds(gp, lp, 16, 1024, 0); break;
            case 4: __builtin_amdgcn_global_load_lds(gp, lp, 16, 2048, 0); break;
            case 6: __builtin_amdgcn_global_load_lds(gp, lp, 16, 3072, 0); break;
            default: break;
        }
    };
    // Step kt.  SPREAD issues its copies between the matrix instructions (needs a bf16 cache, both copies due and this
    // wavefront computing), TOP at the step's top.  LAST (kt = n_kt - 1) has no next tile: no scores are started for one
    // and the second half's V takes the window's places instead (8 of 32 products less).
    enum { SPREAD, TOP, LAST };
    auto cache_step = [&](const int kt, auto kind_tag) __attribute__((always_inline)) {
        constexpr int kind = decltype(kind_tag)::value;
        constexpr bool spread = kind == SPREAD, last = kind == LAST;
        char *kd = !last && kt + 2 < n_kt ? kbuf_of(kt + 2) : nullptr;
        char *vd = !last && kt + 1 < n_kt ? vbuf_of(kt + 1) : nullptr;
        const int pg_new = last ? 0 : cache_page(kt + 3);
        PartCopy first = {nullptr, nullptr}, second = {nullptr, nullptr};
        if (spread) {
            first = cache_part(true, pg_v, vd);      // V is needed first
            second = cache_part(false, pg_k, kd);
        } else if (last) {
            if (own) own_copy(0);
        } else {
            if (kd || vd) fetch_cache(pg_k, kd, pg_v, vd);
        }
        pg_v = pg_k;
        pg_k = pg_new;
        if (spread || MODE == MODE_SUFFIX || kt < n_my) {  // some row of this wave still sees keys of this tile
            const int key0 = kt * BN;
            const bool masked = key0 + BN > lim_min;
            const bool careful = masked || fresh;
            // Past this wave's last tile (but not the workgroup's) the "next" scores are formed from the other K buffer
            // and never used; this keeps the step free of branches around the matrix instructions.
            const char *kn = kbuf_of(kt + 1), *vc = vbuf_of(kt);
            auto keep = [&](int mi, int j) __attribute__((always_inline)) { return key0 + j < lim[mi]; };
            // A reference raised after the next half's scores were started must be applied to those as well.
            auto redo = [&](f32x16 (&sc)[MI], f32x16 (&sn)[MI], int nb) __attribute__((always_inline)) {
                float before[MI];
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) before[mi] = m_ref[mi];
                raise_reference(sc, nb, false, keep_all);
                weights(sc);
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (FOLD) sn[mi][r] -= m_ref[mi] - before[mi];
            };
            // half 0
            if (careful) raise_reference(s0, 0, masked, keep);
            qk_half_cache(s1, [&](int i) __attribute__((always_inline)) {
                frag[i] = v_block(vc, 0, i);
                if (spread) copy_quarter(first, i);
            });
            weights(s0);
            if (weights_overflow()) redo(s0, s1, 0);
            pv_half([&](int i) __attribute__((always_inline)) {
                frag[i] = last ? v_block(vc, 1, i) : kc_block(kn, 0, i);
                if (spread) copy_quarter(second, i);
            });
            // half 1
            if (careful) raise_reference(s1, 1, masked, keep);
            if (!last) qk_half_cache(s0, [&](int i) __attribute__((always_inline)) { frag[i] = v_block(vc, 1, i); });
            weights(s1);
            if (weights_overflow()) redo(s1, s0, 1);
            if (last) {
                if (own) own_table(0);
                pv_half(no_refill);
            } else
                pv_half([&](int i) __attribute__((always_inline)) { frag[i] = kc_block(kn, 1, i); });
            fresh = false;
        }
        land_cache(kd, vd);
        if (!last || !own) __syncthreads();      // (the own-suffix part has barriers of its own)
    };
    {
        int kt = 0;
        if (!KV_FP8) {
            const int n_spread = min(n_kt - 2, MODE == MODE_SUFFIX ? n_kt : n_my);
            for (; kt < n_spread; ++kt) cache_step(kt, std::integral_constant<int, SPREAD>{});
        }
        for (; kt < n_kt - 1; ++kt) cache_step(kt, std::integral_constant<int, TOP>{});
        if (n_kt > 0) cache_step(n_kt - 1, std::integral_constant<int, LAST>{});
    }

    // ---- the own-suffix keys of the queries this row tile touches --------------------------------------------
    // What this part costs is round trips and barriers, hardly any products: a tile touches two or three queries of some tens of
    // tokens.  So the queries' pages are packed, four to a chunk whatever query they belong to, and the keys and values
    // are taken as given where nothing else needs them as pages: an ingest launch in front of this one read and wrote as
    // many bytes as the queries' rows themselves, and a 64-key step with a barrier per touched query cost more than the rotation
    // of a page per wavefront and chunk does.  100 questions over ten prompts, four layers 588 -> 546 us with their prompts' prefill,
    // 320 questions 432 -> 415 us, 1024 questions of 32 heads without groups 3370 -> 3005 us.
    // Every wavefront walks the pages its own rows see, two at a time and with no barrier between them: a page belongs to one
    // query, and a row sees the slots own_first .. own_first + qpos.
    bool v_scaled = !KV_FP8;
    if (MODE == MODE_SUFFIX) {
        if (!v_scaled) {        // fp8 cache: the accumulated cached part takes the V scale once
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[mi][db][r] *= v_scale;
            v_scaled = true;
        }
        if (own && n_kt == 0) {
            own_copy(0);
            own_table(0);
        }
        const int wpg_lo = __builtin_amdgcn_readlane(own_first, 0) / kPageTokens;
        const int wpg_hi = __builtin_amdgcn_readlane(own_first + qpos[0], 31) / kPageTokens;
        const int tr = (lane & 15) >> 2;
        const int lane_trow = (4 * h + tr) * 256 + (n >> 4) * 32 + (lane & 3) * 8;
        for (int ci = 0, c0 = 0; c0 < n_own; ++ci, c0 += OWN_PAGES) {
            const int c1 = min(c0 + OWN_PAGES, n_own);
            __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the chunk's pages have landed
            own_rotate(ci);
            __syncthreads();                             // (also: the chunk before this one has been read)
            own_copy(ci + 1);
            if (c1 < n_own) own_table(ci + 1);
            const char *kc = own_kbuf(ci), *vc = own_vbuf(ci);
            const int row_end = min(own_first + qpos[0], c1 * kPageTokens - 1);
            const int p_last = min(wpg_hi, c1 - 1);
            for (int p = max(wpg_lo, c0); p <= p_last; p += 2) {
                const int i0 = p - c0, i1 = min(p + 1, p_last) - c0;       // (past the last page the rows see: the first again, masked)
                const char *kp = kc + ((n >> 4) ? i1 : i0) * PART_BYTES + (h * kPageTokens + (n & 15)) * 16;
                const char *v0 = vc + i0 * PART_BYTES, *v1 = vc + i1 * PART_BYTES;
#pragma unroll
                for (int i = 0; i < 8; ++i) frag[i] = *reinterpret_cast<const bf16x8 *>(kp + i * 512);
                if constexpr (OWN_RAW) {
                    qk_half(s0, no_refill);
                    uint32_t at[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        at[i] = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)((i < 4 ? v0 : v1) + lane_trow + (((i & 3) ^ tr) * 64));
                    read_v_rows(at, frag);
                } else {
                    qk_half(s0, [&](int i) __attribute__((always_inline)) {
                        frag[i] = *reinterpret_cast<const bf16x8 *>((i < 4 ? v0 : v1) + lane_voff + (i & 3) * 1024);
                    });
                }
                if (KV_FP8) rescale_self(s0, m_ref);
                // slot 16 p + j is visible iff own_first <= slot <= row_end: one comparison of unsigned numbers (a row that sees no
                // slot of the chunk has a range of one, far off; as a second condition it became a branch per score, 300
                // instructions for 32 keys, and a question of 8192 tokens took 1365 us instead of 1012).  The 4 h of the lane's
                // key index is taken off once.
                const bool any = row_end >= own_first;
                const int first = any ? own_first - p * kPageTokens - 4 * h : -(1 << 30);
                const uint32_t span = any ? (uint32_t)(row_end - own_first) : 0u;
                raise_reference(s0, 0, true, [&](int, int j) __attribute__((always_inline)) { return (uint32_t)(j - 4 * h - first) <= span; });
                weights(s0);
                pv_half(no_refill);
            }
        }
    }

    // ---- normalise and store ----
    // A lane holds 4-channel pieces of its row; written out as they are they would make 8-byte stores scattered
    // over 32 rows per instruction.  The wavefront instead stages its 32 x 128 outputs in
    // 8 KiB of the K and V buffers that the chunk after the last own one would take (every wavefront is past the barrier behind
    // their last read), the 16-byte chunks of row n permuted by n % 16 so that the writes and the reads below spread over all banks, and stores
    // four whole rows of 256 bytes per instruction.
    uint16_t *og = static_cast<uint16_t *>(o_base);
    const int own_chunks = (n_own + OWN_PAGES - 1) / OWN_PAGES;
    char *const ostage[2] = {own_kbuf(own_chunks) + wave_u * PART_BYTES, own_vbuf(own_chunks) + wave_u * PART_BYTES};    // rows 0 .. 15, 16 .. 31
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const float l = half_sum(l_part[mi]);
        const float inv_l = (v_scaled ? 1.0f : v_scale) / l;
        char *st = ((n >> 4) ? ostage[1] : ostage[0]) + (n & 15) * 256 + h * 8;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                bf16x4 y;
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = (__bf16)(oacc[mi][db][q4 * 4 + i] * inv_l);
                *reinterpret_cast<bf16x4 *>(st + (((db * 4 + q4) ^ (n & 15)) * 16)) = y;
            }
        if (valid[mi] && lse_base && h == 0) {
            const int64_t col = (MODE == MODE_SUFFIX) ? (int64_t)src_tok[mi] : (int64_t)qpos[mi];
            lse_base[(int64_t)head[mi] * lse_stride + col] = (m_ref[mi] + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = 4 * k + (lane >> 4), c = lane & 15;     // row r of the block sits in lanes r and r + 32
            const uint4 y = *reinterpret_cast<const uint4 *>(ostage[k >> 2] + (r & 15) * 256 + ((c ^ (r & 15)) * 16));
            const int64_t row = __shfl(io_row[mi], r);
            const int ok = __shfl((int)valid[mi], r);
            if (ok) *reinterpret_cast<uint4 *>(og + row + c * 8) = y;
        }
    }
}

template <bool FP8, int MODE, bool QK8, bool OWN_RAW, typename ARGS>
hipError_t launch_one(const ARGS &a, int blocks, hipStream_t s)
{
    static bool configured = false;     // raise the dynamic LDS limit once per instantiation
    auto kern = attn_mfma_kernel<FP8, MODE, QK8, OWN_RAW, ARGS>;
    const size_t lds = 4 * HALF_BYTES;      // two K buffers, two V buffers
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(NW * 64), lds, s, a);
    return hipGetLastError();
}

// ---- decode steps of few rows ----------------------------------------------------------------------------------
// A decode step of few rows per cluster is latency: its tiles are key ranges of row tiles with one row group of 32, for which three of
// four wavefronts of the kernel above compute nothing, and the one takes about a microsecond a 64-key step.  Here a workgroup has
// the row tile's up to 32 rows, and its wavefronts deal the range's 32-key halves (units) among themselves, each with 16 KiB of LDS of its own
// for its half's K and V: no barrier but the merge's.  The next unit is requested as soon as this one's operands are in registers.
// Some of the wavefronts attend over the queries' own keys meanwhile, put the step's new token into its page on the way, and the last of a row
// tile's ranges to finish adds the ranges up: the whole step is one launch.  As two (cached part; own keys and sums) it took, us
// with their launches (32 query heads, 8 KV heads): 5 queries over 3001 keys 19.3, now 14.7; one over 9000 24.0 -> 14.0; 16 over a prompt of 1000
// each 26.0 -> 16.9; 5 without head groups over 500 17.8 -> 11.0.
// (Suffix prefills over few rows gain as much, but their rows' sums would then follow from the other clusters of the call, and a
// cluster served by itself would no longer equal the same cluster in a batch bit for bit.  A step's ranges follow from the call
// as it is.)
constexpr int NWF = 8;        // wavefronts of a workgroup

// Memory that workgroups of one launch hand to each other: stored through to and loaded from the level that all XCDs share (agent-scope
// accesses).  A release and an acquire fence instead write back and invalidate a whole XCD's L2, under the other workgroups' reads
// of the cache: 16 prompts of 1000 tokens in two ranges 27 us a step.
template <typename T>
__device__ __forceinline__ void store_shared(T *p, const T &v)
{
    static_assert(sizeof(T) % 8 == 0, "eight bytes at a time");
    uint64_t w[sizeof(T) / 8];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) __hip_atomic_store(reinterpret_cast<uint64_t *>(p) + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_shared(const T *p)
{
    uint64_t w[sizeof(T) / 8];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

__global__ void __launch_bounds__(NWF * 64, 2) attn_few_kernel(const AttnArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    constexpr int SLOT = 4 * PART_BYTES;        // a wavefront's K (two pages), then V; later its 32 x 128 partial outputs
    // behind the wavefronts' slots one for the rows' own keys, then [slot][row]: reference maximum, row sum
    char *const own_slot = smem + NWF * SLOT;
    float2 *const stats = reinterpret_cast<float2 *>(smem + (NWF + 1) * SLOT);

    const int wave_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 31, h = lane >> 5;
    const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, g = a.group;
    char *const slot = smem + wave_u * SLOT;

    const Tile t = uniform_record(a.tiles + blockIdx.x);
    asm volatile("" ::"s"(t.n_rows), "s"(t.prefix_len), "s"(t.pad));
    if (t.n_rows == 0) return;
    const int P = t.prefix_len, n_pages = (P + kPageTokens - 1) / kPageTokens;
    const int range = t.pad >> 24, all_cached = P + (t.pad & 0xFFFFFF);
    const int last_row = t.n_rows - 1;         // (a unit's rows are one tile of 32 at most: row0 is 0)

    // ---- the lane's row (rows past the end repeat the last one) ----
    const bool valid = n <= last_row;
    const int rc = min(n, last_row), tk = rc / g, head = t.hk * g + (rc - tk * g);
    const TokInfo ti = a.tok_info[t.tok_base + tk];
    const int qpos = ti.qpos, src_tok = ti.src;
    const int64_t io_row = ((int64_t)src_tok * Hq + head) * D;
    const int n_units = (P + 31) / 32;

    // ---- K and V of a unit, half a 64-key tile, on their way to the wavefront's slot ----
    const char *cache_base = a.pool.pool + (int64_t)a.layer * a.pool.layer_bytes + (int64_t)t.hk * a.pool.head_part_bytes + lane * 16;
    const int32_t *pt = a.page_table + t.pt_off;
    // Own keys, below: 16 heads of a query are a task; task k belongs to range k % ranges.  A range's tasks have wavefronts of their own:
    // a task is a longer chain of round trips than a unit, as many of them as own_cost2 says in halves.
    const int S = a.n_ranges, halves = (g + 15) / 16, n_tasks = t.n_rows / g * halves;
    const int tasks_here = n_tasks > range ? (n_tasks - range + S - 1) / S : 0, own_load = a.own_cost2 * tasks_here, own_share = (NWF * own_load + own_load / 2) / max(own_load + 2 * n_units, 1);
    const int own_waves = tasks_here > 0 ? min(tasks_here, max(1, min(own_share, n_units > 0 ? NWF - 1 : NWF))) : 0, unit_waves = NWF - own_waves;
    const int my_first = wave_u < unit_waves ? wave_u : n_units;
    // (the first units' pages come with the tile record)
    int pg_first0 = 0, pg_first1 = 0;
#pragma unroll
    for (int w = 0; w < 6; ++w)
        if (wave_u == w) {
            pg_first0 = t.first_pages[2 * w];
            pg_first1 = t.first_pages[2 * w + 1];
        }
    auto copy_unit = [&](int u, bool first) __attribute__((always_inline)) {
        if (u >= n_units) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // (a page past the last is the last one again: its keys are masked)
            const int page = first ? (i ? pg_first1 : pg_first0) : uniform_record(pt + min(2 * u + i, n_pages - 1));
            const char *src = cache_base + (int64_t)page * a.pool.page_bytes;
            copy_4k_to_lds(src, slot + i * PART_BYTES);
            copy_4k_to_lds(src + Hkv * a.pool.head_part_bytes, slot + (2 + i) * PART_BYTES);
        }
    };
    copy_unit(my_first, wave_u < 6);

    if (wave_u >= unit_waves) {
        // ---- own keys; their rows go into a slot that all tasks of the workgroup share ----
        for (int k = range + (NWF - 1 - wave_u) * S; k < n_tasks; k += own_waves * S) {
            const int qi = k / halves, h0 = (k - qi * halves) * 16, j = lane & 15, quad = lane >> 4;
            const int sq = t.tok_base + qi;
            const TokInfo own_ti = uniform_record(a.tok_info + sq);
            const bool live = h0 + j < g;
            const int64_t part = PART_BYTES, kv_row = ((int64_t)own_ti.src * Hkv + t.hk) * D;
            OwnKeys w{};
            w.page_stride = 2 * Hkv * part;
            w.pages = const_cast<char *>(a.spool) + own_ti.own0 * w.page_stride + t.hk * part;
            w.v_part = Hkv * part;
            w.n_keys = own_ti.qpos + a.pos_shift + 1;
            w.q = static_cast<const uint16_t *>(a.q) + ((int64_t)own_ti.src * Hq + t.hk * g + (live ? h0 + j : 0)) * D;
            w.scale = live ? a.scale_log2e : 0.f;
            w.rope = a.rope ? a.rope + (int64_t)(all_cached + w.n_keys - 1) * (D / 2) : nullptr;
            w.k_new = static_cast<const uint16_t *>(a.k) + kv_row;
            w.v_new = static_cast<const uint16_t *>(a.v) + kv_row;
            w.append = h0 == 0;
            dec_f32x4 O[8];
            float m, l;
            own_keys_attend<true, 2, true>(w, O, m, l);
            const int row = qi * g + h0 + j;
            if (live) {
#pragma unroll
                for (int cb = 0; cb < 8; ++cb)
                    *reinterpret_cast<float4 *>(own_slot + row * 512 + (((4 * cb + quad) ^ row) * 16)) = make_float4(O[cb][0], O[cb][1], O[cb][2], O[cb][3]);
                if (quad == 0) stats[NWF * 32 + row] = make_float2(m, l);
            }
        }
    } else {
        // ---- Q: rotated and scaled, as operands ----
        f16x8 qf[8];
        {
            float4 cs[4][4];
            uint4 qlo[4], qhi[4];
            const int pos = all_cached + a.pos_shift + qpos;
            const uint16_t *qrow = static_cast<const uint16_t *>(a.q) + io_row + h * 8;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                qlo[kb] = *reinterpret_cast<const uint4 *>(qrow + kb * 16);
                qhi[kb] = *reinterpret_cast<const uint4 *>(qrow + 64 + kb * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    cs[kb][i] = a.rope ? reinterpret_cast<const float4 *>(a.rope + (int64_t)pos * (D / 2) + kb * 16 + h * 8)[i] : make_float4(1.f, 0.f, 1.f, 0.f);
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const uint32_t wl[4] = {qlo[kb].x, qlo[kb].y, qlo[kb].z, qlo[kb].w}, wh[4] = {qhi[kb].x, qhi[kb].y, qhi[kb].z, qhi[kb].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float a0 = __uint_as_float(wl[i] << 16), a1 = __uint_as_float(wl[i] & 0xFFFF0000u);
                    float b0 = __uint_as_float(wh[i] << 16), b1 = __uint_as_float(wh[i] & 0xFFFF0000u);
                    const float4 t4 = cs[kb][i];
                    rotate_sums(a0, b0, t4.x, t4.y);
                    rotate_sums(a1, b1, t4.z, t4.w);
                    qf[kb][2 * i] = (_Float16)(a0 * a.scale_log2e);
                    qf[kb][2 * i + 1] = (_Float16)(a1 * a.scale_log2e);
                    qf[kb + 4][2 * i] = (_Float16)(b0 * a.scale_log2e);
                    qf[kb + 4][2 * i + 1] = (_Float16)(b1 * a.scale_log2e);
                }
            }
        }

        // ---- the wavefront's units: online softmax as in the kernel above ----
        f32x16 oacc[4], neg_ref;
        float m_ref = 0.f, l_part = 0.f;
        bool seen = false, fresh = true;          // fresh: some row of the wavefront has met no key yet
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            neg_ref[r] = 0.f;
#pragma unroll
            for (int db = 0; db < 4; ++db) oacc[db][r] = 0.f;
        }
        const int lane_koff = (n >> 4) * PART_BYTES + (h * kPageTokens + (n & 15)) * 16;
        for (int u = my_first; u < n_units; u += unit_waves) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the unit has landed (and what waits here is this wavefront's own)
            bf16x8 kf[8], vf[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) kf[i] = *reinterpret_cast<const bf16x8 *>(slot + lane_koff + i * 512);
#pragma unroll
            for (int i = 0; i < 8; ++i) vf[i] = *reinterpret_cast<const bf16x8 *>(slot + 2 * PART_BYTES + lane * 16 + i * 1024);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // operands are in registers: the slot takes the next unit
            copy_unit(u + unit_waves, false);

            f32x16 s = neg_ref;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) s = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, kf[kb]), qf[kb], s, 0, 0, 0);
            const bool masked = 32 * u + 32 > P, first = u == my_first;
            if (masked) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * u + 8 * (r >> 2) + 4 * h + (r & 3) >= P) s[r] = -INFINITY;
            }
            uint32_t pf[2][4];
            float psum;
            auto raise_reference = [&]() __attribute__((always_inline)) {
                float tmax = s[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, s[r]);
                tmax = half_max(tmax);
                const bool has = tmax > -INFINITY;          // (a unit whose scores are all -inf leaves the row as it was)
                const float delta = seen ? fmaxf(tmax, 0.f) : (has ? tmax : 0.f);
                if (__any(delta != 0.f)) {
                    m_ref += delta;
                    if (!first) {                           // (nothing is accumulated before a wavefront's first unit)
                        const float alpha = seen ? __builtin_amdgcn_exp2f(-delta) : 1.0f;
                        l_part *= alpha;
#pragma unroll
                        for (int r = 0; r < 16; ++r)
#pragma unroll
                            for (int db = 0; db < 4; ++db) oacc[db][r] *= alpha;
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        s[r] -= delta;
                        neg_ref[r] = -m_ref;
                    }
                }
                seen = seen || has;
                fresh = __any(!seen);
            };
            auto weights = [&]() __attribute__((always_inline)) {
                bf16x2 ones;
                ones[0] = (__bf16)1.0f;
                ones[1] = (__bf16)1.0f;
                psum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    bf16x2 pk;
                    pk[0] = (__bf16)__builtin_amdgcn_exp2f(s[r]);
                    pk[1] = (__bf16)__builtin_amdgcn_exp2f(s[r + 1]);
                    psum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, psum, false);
                    pf[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, pk);
                }
            };
            const bool careful = masked || fresh;
            if (careful) raise_reference();
            weights();
            if (!careful && __any(!(psum <= kKeepBelow))) {
                raise_reference();
                weights();
            }
            l_part += psum;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const u32x4 w = {pf[i >> 2][0], pf[i >> 2][1], pf[i >> 2][2], pf[i >> 2][3]};
                oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], __builtin_bit_cast(bf16x8, w), oacc[i & 3], 0, 0, 0);
            }
        }

        // ---- partial outputs into the slots: 16-byte chunk c of row n at place c ^ n ----
        {
            const float l = half_sum(l_part);
            if (h == 0) stats[wave_u * 32 + n] = make_float2(seen ? m_ref : -INFINITY, l);
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *reinterpret_cast<float4 *>(slot + n * 512 + (((db * 8 + 2 * q4 + h) ^ n) * 16)) =
                        make_float4(oacc[db][q4 * 4], oacc[db][q4 * 4 + 1], oacc[db][q4 * 4 + 2], oacc[db][q4 * 4 + 3]);
        }
    }

    // ---- merge: every thread a few chunks ----
    // A part that saw no key of a row has reference -inf and sum 0 and is left out; with a sum that is NaN it counts, and so does the NaN.
    auto part_weight = [](const float2 &st, float M) __attribute__((always_inline)) { return st.x > -INFINITY ? __builtin_amdgcn_exp2f(st.x - M) : st.y; };
    auto finish = [&](int row, int c, float M, float L, const float4 &sum) __attribute__((always_inline)) {
        const float inv = 1.0f / L;
        const int64_t at = __shfl(io_row, row);
        const int r_head = __shfl(head, row), r_tok = __shfl(src_tok, row);
        if (row <= last_row) {
            bf16x4 y;
            y[0] = (__bf16)(sum.x * inv);
            y[1] = (__bf16)(sum.y * inv);
            y[2] = (__bf16)(sum.z * inv);
            y[3] = (__bf16)(sum.w * inv);
            *reinterpret_cast<bf16x4 *>(static_cast<uint16_t *>(a.o) + at + c * 4) = y;
            if (a.lse && c == 0) a.lse[(int64_t)r_head * a.lse_stride + r_tok] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
        }
    };
    float4 *const parts = reinterpret_cast<float4 *>(a.parts + (int64_t)t.row_tile * S * kFewPartBytes);      // [range][row][chunk], then ...
    float2 *const part_stats = reinterpret_cast<float2 *>(parts + (int64_t)S * 32 * 32);                     // ... [range][row]
    // (The row tile's counter starts at the launch's number: what earlier calls that ran into each other may have left in it is below.  A
    // captured launch keeps its number, so later calls' leftovers are not: a capture clears the counters in front of its first step.)
    if (S > 1 && threadIdx.x == 0) (void)__hip_atomic_fetch_max(a.arrived + t.row_tile, a.launch << 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16 / NWF; ++k) {
        const int row = ((int)threadIdx.x >> 5) + k * 2 * NWF, c = lane & 31;
        const int qi = row / g, task = qi * halves + (row - qi * g) / 16;
        const bool own_here = row <= last_row && task % S == range;      // the shared slot holds the row's own keys
        float2 st[NWF + 1];
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w <= NWF; ++w) {
            st[w] = (w < NWF ? w < unit_waves : own_here) ? stats[w * 32 + row] : make_float2(-INFINITY, 0.f);
            M = fmaxf(M, st[w].x);
        }
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w <= NWF; ++w) {
            if (!(w < NWF ? w < unit_waves : own_here)) continue;
            const float f = part_weight(st[w], M);
            const float4 o = *reinterpret_cast<const float4 *>(smem + w * SLOT + row * 512 + ((c ^ row) * 16));
            L += f * st[w].y;
            sum.x += f * o.x;
            sum.y += f * o.y;
            sum.z += f * o.z;
            sum.w += f * o.w;
        }
        if (S == 1) {
            finish(row, c, M, L, sum);
        } else if (row <= last_row) {
            store_shared(parts + (range * 32 + row) * 32 + c, sum);
            if (c == 0) store_shared(part_stats + range * 32 + row, make_float2(M, L));
        }
    }
    if (S == 1) return;

    // ---- the last of a row tile's ranges to get here adds all of them up, in their order ----
    // (Every workgroup stores, counts, and goes; nobody waits for another.  The counter is zero between launches.)
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): this wavefront's results are where the others will read them
    __syncthreads();
    uint32_t *const flag = reinterpret_cast<uint32_t *>(smem);
    if (threadIdx.x == 0) {
        const uint32_t before = __hip_atomic_fetch_add(a.arrived + t.row_tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xff;
        if (before == (uint32_t)(S - 1)) __hip_atomic_store(a.arrived + t.row_tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = before;
    }
    __syncthreads();
    if (*flag != (uint32_t)(S - 1)) return;
#pragma unroll
    for (int k = 0; k < 16 / NWF; ++k) {
        const int row = ((int)threadIdx.x >> 5) + k * 2 * NWF, c = lane & 31;
        if (__builtin_amdgcn_readfirstlane(row) > last_row) continue;       // (of the two rows of a wavefront the first)
        const int rr = min(row, last_row);
        float M = -INFINITY, L = 0.f;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r0 = 0; r0 < S; r0 += 4) {          // four ranges to a round trip; what is added so far is rescaled to the new maximum
            float2 st[4];
            float4 o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = min(r0 + i, S - 1);
                st[i] = load_shared(part_stats + r * 32 + rr);
                o[i] = load_shared(parts + (r * 32 + rr) * 32 + c);
                if (r0 + i >= S) st[i] = make_float2(-INFINITY, 0.f);
            }
            float m_new = M;
#pragma unroll
            for (int i = 0; i < 4; ++i) m_new = fmaxf(m_new, st[i].x);
            const float keep = M > -INFINITY ? __builtin_amdgcn_exp2f(M - m_new) : 1.f;
            M = m_new;
            L *= keep;
            sum.x *= keep;
            sum.y *= keep;
            sum.z *= keep;
            sum.w *= keep;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (r0 + i >= S) continue;
                const float f = part_weight(st[i], M);
                L += f * st[i].y;
                sum.x += f * o[i].x;
                sum.y += f * o[i].y;
                sum.z += f * o[i].z;
                sum.w += f * o[i].w;
            }
        }
        finish(row, c, M, L, sum);
    }
}

hipError_t launch_few(const AttnArgs &a, hipStream_t s)
{
    static bool configured = false;     // raise the dynamic LDS limit once
    auto kern = attn_few_kernel;
    const size_t lds = (NWF + 1) * (4 * PART_BYTES + 32 * sizeof(float2));
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, dim3(a.n_tiles), dim3(NWF * 64), lds, s, a);
    return hipGetLastError();
}

}  // namespace

// One shape of the 128-row kernel is built: 4 wavefronts x 32 rows, two workgroups per CU.  (8 wavefronts x 32 rows run in lock-step
// through the step barrier and lose the overlap two independent workgroups have; 64 rows per wavefront need more than
// 256 vector registers.  Both were measured slower and are not compiled.)
int mfma_tile_rows() { return NW * MI * 32; }

hipError_t launch_attn_mfma(const AttnArgs &a, hipStream_t s)
{
    const bool fp8 = a.pool.kv_dtype == SGC_FP8_E4M3;
    if (a.n_tiles <= 0 && a.n_append <= 0) return hipSuccess;
    if (a.few) return launch_few(a, s);
    if (a.mode == MODE_SUFFIX) {
        // a decode step's launch carries, behind its tiles, the blocks that append the step's new tokens
        const int per_block = NW * 64 / 8;
        const int blocks = a.n_tiles + (a.n_append * a.n_kv_heads + per_block - 1) / per_block;
        if (fp8 && a.fp8_first_product)
            return a.own_raw ? launch_one<true, MODE_SUFFIX, true, true>(a, blocks, s) : launch_one<true, MODE_SUFFIX, true, false>(a, blocks, s);
        if (fp8) return a.own_raw ? launch_one<true, MODE_SUFFIX, false, true>(a, blocks, s) : launch_one<true, MODE_SUFFIX, false, false>(a, blocks, s);
        return a.own_raw ? launch_one<false, MODE_SUFFIX, false, true>(a, blocks, s) : launch_one<false, MODE_SUFFIX, false, false>(a, blocks, s);
    }
    // the prompt's own causal attention always takes the 16-bit first product
    return fp8 ? launch_one<true, MODE_PREFIX, false, false>(a, a.n_tiles, s) : launch_one<false, MODE_PREFIX, false, false>(a, a.n_tiles, s);
}

hipError_t launch_attn_carried(const CarriedPrefix &c, hipStream_t s)
{
    return c.a.n_tiles > 0 ? launch_one<false, MODE_PREFIX, false, false>(c, c.a.n_tiles, s) : hipSuccess;
}

hipError_t launch_attn_carried(const CarriedSuffix &c, hipStream_t s)
{
    return c.a.n_tiles > 0 ? launch_one<false, MODE_SUFFIX, false, true>(c, c.a.n_tiles, s) : hipSuccess;
}

}  // namespace sgc
