// Projection kernels of libsgc for gfx950 (MI355X): the linear maps around the cached attention.
//
// SubGCache (arXiv 2505.10951) Sec. 3.4 feeds the representative prompt and then every query's question
// tokens through the LLM's layers.  In each layer the hidden states x [rows][K] are projected by the fused
// weight w_qkv [(Hq + 2 Hkv) d][K] ("out features x in features") to queries, keys and values, and the
// attention output is projected back by w_o.  Both are C = A B^T with A and B contiguous along the
// contraction, which is exactly what the 32x32x16 bf16 matrix-core instruction wants for both operands.
//
// bf16 kernel: a workgroup of 4 wavefronts computes a 256 x 256 tile of C; wavefront (wm, wn) owns the
// 128 x 128 quadrant and keeps it in 16 accumulators of 32 x 32 (256 registers, one wavefront per SIMD).
// The contraction runs in steps of 64: the 256 x 64 slabs of A and B (32 KiB each) are copied
// global -> LDS without passing through registers, into a ring of five, one barrier per step.  In LDS a slab is
// row-major with 128-byte rows whose eight 16-byte chunks are permuted by (row & 7) ^ ((row >> 3) & 1); the
// permutation is applied on the global side of the copy (the LDS side of such a copy is linear in the lane
// index), and it spreads the 16-byte operand reads of 32 consecutive rows over all banks.
//
// Epilogue of the QKV projection (a wavefront's 128 columns are exactly one head, d = 128):
//   Q heads: stored as they are (the attention kernel rotates Q itself);
//   K heads: rotated at the token's position (rotate-half pairs channel t with t + 64, which sit in the
//            same lane and register of accumulators pi and pi + 2) and written straight into the 16-token
//            pages in the cache's K order: 8 consecutive channels of a token are one 16-byte unit;
//   V heads: the matrix-core operands are swapped for these wavefronts so that a lane owns ONE channel and
//            16 tokens; when the 16 rows are one page this is the cache's V order (8 tokens of a channel
//            contiguous) and goes out as 16-byte stores; a batch's, whose questions begin at any row, pass through LDS
//            and leave in whole pages as well, but for those that reach over the tile's rows (store_own_values).
// With an fp8 cache (the scale needs the maximum over the whole prompt first) K and V go to a staging
// matrix and the ingest kernels take it from there.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "sgc_internal.h"

namespace sgc {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int TM = 256, TN = 256, TK = 64;
constexpr int SLAB_BYTES = TM * TK * 2;          // 32 KiB: 256 rows of 128 bytes
constexpr int RING = 5;                          // slabs in LDS
constexpr int GEMM_LDS = RING * SLAB_BYTES;      // 160 KiB
constexpr int HD = 128;                          // head dim of the fused epilogue

__device__ inline uint32_t pack2(float a, float b)
{
    const bf16x2 p = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, p);
}

// 1 KiB (64 lanes x 16 bytes) to the LDS block at lds (wave-uniform), from `lane_off` + `off` of the operand.  A buffer load: the address
// costs no vector instruction, and the compiler does not take it for a flat one, behind which it waits for every LDS read in flight.
typedef __amdgpu_buffer_rsrc_t Operand;
__device__ __forceinline__ Operand operand(const void *base, uint32_t bytes)
{
    const uint64_t at = reinterpret_cast<uint64_t>(base);          // (wave-uniform, which the compiler does not see of a row tile's record)
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));      // (the builtin's int would be sign-extended)
    const uint64_t u = (uint64_t)hi << 32 | lo;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(u), 0, bytes, 0x00027000);
}
__device__ __forceinline__ void copy_1k_to_lds(Operand from, uint32_t lane_off, uint32_t off, char *lds)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)lds, 16, lane_off, off, 0, 0);
}

// Barrier of a step: at most N of this wavefront's copies are still on their way and all its LDS reads have returned.
// (__syncthreads() waits for every outstanding copy, which would leave one step in flight whatever the depth.)
template <int N>
__device__ __forceinline__ void step_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));      // vmcnt(N), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Row tile rt of the launch; ARGS: GemmArgs, or GemmCarried, whose tiles are read where they arrive, among the launch's arguments.
__device__ __forceinline__ const GemmArgs &gemm_args(const GemmArgs &a) { return a; }
__device__ __forceinline__ const GemmArgs &gemm_args(const GemmCarried &c) { return c.a; }
template <class ARGS>
__device__ __forceinline__ GemmRowTile row_tile(const GemmArgs &g, int rt, int height)
{
    GemmRowTile t;
    if constexpr (std::is_same_v<ARGS, GemmCarried>) {
        const auto *c = (const __attribute__((address_space(4))) GemmCarried *)__builtin_amdgcn_kernarg_segment_ptr();
        t.a = c->tiles[rt].a;
        t.c = c->tiles[rt].c;
        t.ck = c->tiles[rt].ck;
        t.cv = c->tiles[rt].cv;
        t.rows = c->tiles[rt].rows;
        t.pos0 = c->tiles[rt].pos0;
        t.pt_off = c->tiles[rt].pt_off;
        t.dest0 = c->tiles[rt].dest0;
    } else if (g.tiles) {
        t = g.tiles[rt];
    } else {
        t.a = static_cast<const char *>(g.a) + (int64_t)rt * height * g.K * 2;
        t.c = g.c ? static_cast<char *>(g.c) + (int64_t)rt * height * g.ldc * 2 : nullptr;
        t.ck = t.cv = nullptr;
        t.rows = (int32_t)min<int64_t>(height, g.M - (int64_t)rt * height);
        t.pos0 = 0;
        t.pt_off = 0;
        t.dest0 = rt * height;
    }
    return t;
}

// The slots behind a question's last row in its last page, which the attention kernel multiplies by zero weights and which
// therefore have to be finite: the wavefront whose rows (d: its lanes', mine: which of them) hold that last row clears them, for the
// CH channels that its tile has of the head (channel j of them is half32 + j of the first half of the head, or of the second).
// A launch of its own before the
// projection, over all last pages, took 4.0 to 4.8 us: with the row tiles' copy (see sgc_project_qkv_prefix_batched) the layer over a
// prompt of 300 tokens and 6 questions went 117.4 -> 110.5 us.
template <int CH>
__device__ __forceinline__ void clear_behind_last(const GemmArgs &g, const int4 d, bool mine, int kind, int hk, int half32, int lane)
{
    const int n_rows = abs(d.z);
    uint64_t last = __ballot(mine && n_rows < kPageTokens && (d.x & 15) == n_rows - 1);
    while (last) {
        const int r = __builtin_ctzll(last);
        last &= last - 1;
        const int x = __builtin_amdgcn_readlane(d.x, r), slot = x & 15;
        char *page = g.kv_base + (int64_t)(x >> 4) * g.page_bytes + (int64_t)(kind == 1 ? hk : g.n_kv_heads + hk) * g.part_bytes;
        auto channel = [&](int j) __attribute__((always_inline)) { return CH == HD ? j : (j >> 5) * 64 + half32 + (j & 31); };
        if (kind == 1) {
#pragma unroll
            for (int u0 = 0; u0 < 2 * CH; u0 += 64) {
                const int u = u0 + lane, s = u & 15;
                if (s > slot) *reinterpret_cast<uint4 *>(page + k_page_index(s, channel(8 * (u >> 4))) * 2) = make_uint4(0, 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int u0 = 0; u0 < 4 * CH; u0 += 64) {
                const int u = u0 + lane, j = u % CH, s0 = 4 * (u / CH);
                uint16_t *p = reinterpret_cast<uint16_t *>(page) + v_page_index(s0, channel(j));      // four slots of a channel
                if (s0 > slot)
                    *reinterpret_cast<uint2 *>(p) = make_uint2(0, 0);
                else
#pragma unroll
                    for (int e = 1; e < 4; ++e)
                        if (s0 + e > slot) p[e] = 0;
            }
        }
    }
}

// A batch's values: a wavefront's n (at most 128) rows of a head's 128 channels into the questions' pages.  They lie in acc as lane =
// channel 32 qj + l31, register r of accumulator pi = row 32 pi + 8 (r / 4) + 4 h + r % 4, and questions begin at any row: the wavefront
// lays them out in LDS as [channel][row] and reads a page's 16 tokens of a channel from where they begin, for two 16-byte stores.  Pages
// that reach over the rows' ends are written row by row.  (All rows one by one from the registers, two bytes
// a lane: with the slots behind the last row cleared here Llama-3-8B's layer over ten prompts of 1024 tokens and 320 questions of 16 to
// 64 went 1 944 -> 1 961 us; this way 1 860 -> 1 849, on another card.)
constexpr int V_TILE_LD = 128 * 2 + 8, V_TILE = 128 * V_TILE_LD;
static_assert(4 * V_TILE + 64 <= GEMM_LDS, "the slabs' place, and what a page's reads take too much");
__device__ __forceinline__ void store_own_values(const GemmArgs &g, const f32x16 (&acc)[4][4], int dest0, int n, int hk, char *tile, int lane)
{
    const int h = lane >> 5, l31 = lane & 31;
#pragma unroll
    for (int pi = 0; pi < 4; ++pi)
#pragma unroll
        for (int qj = 0; qj < 4; ++qj) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<uint2 *>(tile + (32 * qj + l31) * V_TILE_LD + (32 * pi + 8 * q4 + 4 * h) * 2) =
                    make_uint2(pack2(acc[pi][qj][4 * q4], acc[pi][qj][4 * q4 + 1]), pack2(acc[pi][qj][4 * q4 + 2], acc[pi][qj][4 * q4 + 3]));
            __builtin_amdgcn_sched_barrier(0);
        }
    char *const pages = g.kv_base + (int64_t)(g.n_kv_heads + hk) * g.part_bytes;
    for (int r0 = 0; r0 < n; r0 += 64) {
        const bool valid = r0 + lane < n;
        const int4 d = g.row_dest[dest0 + (valid ? r0 + lane : r0)];
        const int slot = d.x & 15, first = r0 + lane - slot;
        const bool whole = d.z > 0 && first >= 0 && first + d.z <= n;
        for (uint64_t m = __ballot(valid && whole && slot == 0); m; m &= m - 1) {
            const int bit = __builtin_ctzll(m), r = r0 + bit;
            const int x = __builtin_amdgcn_readlane(d.x, bit), held = __builtin_amdgcn_readlane(d.z, bit);
            char *page = pages + (int64_t)(x >> 4) * g.page_bytes;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint2 *src = reinterpret_cast<const uint2 *>(tile + (64 * c + lane) * V_TILE_LD + (r & ~3) * 2);
                uint32_t w[10], out[8];
#pragma unroll
                for (int e = 0; e < 5; ++e) {
                    const uint2 p = src[e];
                    w[2 * e] = p.x;
                    w[2 * e + 1] = p.y;
                }
#pragma unroll
                for (int e = 0; e < 9; ++e) w[e] = (r & 2) ? w[e + 1] : w[e];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    out[e] = __builtin_amdgcn_alignbit(w[e + 1], w[e], (r & 1) * 16) & (held > 2 * e + 1 ? 0xffffffffu : held > 2 * e ? 0xffffu : 0u);
                uint4 *dst = reinterpret_cast<uint4 *>(page + v_page_index(0, 64 * c + lane) * 2);
                dst[0] = make_uint4(out[0], out[1], out[4], out[5]);
                dst[32] = make_uint4(out[2], out[3], out[6], out[7]);
            }
        }
        for (uint64_t m = __ballot(valid && !whole); m; m &= m - 1) {
            const int bit = __builtin_ctzll(m), r = r0 + bit;
            const int x = __builtin_amdgcn_readlane(d.x, bit);
            uint16_t *page = reinterpret_cast<uint16_t *>(pages + (int64_t)(x >> 4) * g.page_bytes);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                uint16_t v;
                __builtin_memcpy(&v, tile + (64 * c + lane) * V_TILE_LD + r * 2, 2);
                page[v_page_index(x & 15, 64 * c + lane)] = v;
            }
        }
        clear_behind_last<HD>(g, d, valid && !whole, 2, hk, 0, lane);
    }
}

template <bool QKV, class ARGS>
__global__ void __launch_bounds__(256, 1) proj_gemm_kernel(const ARGS args)
{
    const GemmArgs &g = gemm_args(args);
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int h = lane >> 5, l31 = lane & 31;

    // ---- which tile: workgroup b runs on XCD b % 8; every XCD takes a contiguous run of tile ids, and ids
    // walk the tile grid in groups of 4 row tiles, column by column, so that the 32 workgroups an XCD runs
    // together cover about 4 x 8 tiles and share their A and B slabs in that XCD's L2.
    const int n_ct = g.n_col_tiles, n_rt = g.n_row_tiles;
    const int total = n_ct * n_rt;
    const int per = (total + 7) >> 3;
    const int local = (int)blockIdx.x >> 3;
    const int tid = ((int)blockIdx.x & 7) * per + local;
    if (local >= per || tid >= total) return;
    constexpr int GM = 4;
    const int grp = tid / (GM * n_ct);
    const int gsz = min(GM, n_rt - grp * GM);
    const int in = tid - grp * GM * n_ct;
    const int rt = __builtin_amdgcn_readfirstlane(grp * GM + in % gsz);
    const int ct = __builtin_amdgcn_readfirstlane(in / gsz);

    const GemmRowTile t = row_tile<ARGS>(g, rt, TM);
    const int rows = __builtin_amdgcn_readfirstlane(t.rows);
    const int K = g.K, N = g.N;
    const int n_steps = K / TK;

    // ---- copies: wavefront w moves rows [64 w, 64 w + 64) of both slabs, 8 rows (1 KiB) per instruction.
    // Lane (lr, slot) = (lane / 8, lane % 8) lands at LDS chunk `slot` of row 8 i + lr and therefore fetches the
    // global chunk slot ^ perm(row); rows past the operand's end are clamped (their results are never stored).
    const int lr = lane >> 3, slot = lane & 7;
    const int b_rows = min(TN, N - ct * TN);
    const Operand a_op = operand(t.a, (uint32_t)rows * (uint32_t)(K * 2));
    const Operand b_op = operand(static_cast<const char *>(g.w) + (int64_t)ct * TN * K * 2, (uint32_t)b_rows * (uint32_t)(K * 2));
    uint32_t a_off[8], b_off[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 64 * wave + 8 * i + lr;
        const uint32_t chunk = (uint32_t)(slot ^ lr ^ (i & 1));
        a_off[i] = (uint32_t)min(row, rows - 1) * (uint32_t)(K * 2) + chunk * 16;
        b_off[i] = (uint32_t)min(row, b_rows - 1) * (uint32_t)(K * 2) + chunk * 16;
    }
    // copies [lo, hi) of this wavefront's eight of a slab: contraction step kt, ring slot `to`
    auto copy_a = [&](int kt, int to, auto lo, auto hi) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)kt * (TK * 2);
        char *as = smem + to * SLAB_BYTES + wave * 8192;
#pragma unroll
        for (int i = lo; i < hi; ++i) copy_1k_to_lds(a_op, a_off[i], off, as + i * 1024);
    };
    auto copy_b = [&](int kt, int to, auto lo, auto hi) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)kt * (TK * 2);
        char *bs = smem + to * SLAB_BYTES + wave * 8192;
#pragma unroll
        for (int i = lo; i < hi; ++i) copy_1k_to_lds(b_op, b_off[i], off, bs + i * 1024);
    };

    // ---- which output this wavefront makes
    const int col0 = ct * TN + wn * HD;              // first column of the wavefront's 128
    bool v_orient = false;
    int kind = 0, hk = 0;                            // 0 plain, 1 K head, 2 V head
    if (QKV && col0 >= g.n_plain) {
        const int kvh = (col0 - g.n_plain) / HD;
        kind = kvh < g.n_kv_heads ? 1 : 2;
        hk = kind == 1 ? kvh : kvh - g.n_kv_heads;
        v_orient = kind == 2 && g.kv_dest != 2;
    }

    // ---- operand reads: lane (l31, h) of block b reads row 32 b + l31, chunk 2 kk + h
    const uint32_t perm = (uint32_t)(h ^ (lane & 7) ^ ((lane >> 3) & 1));
    uint32_t r_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) r_off[kk] = (uint32_t)l31 * 128 + (((uint32_t)kk * 32) ^ (perm * 16));
    // first operand (from slab A if v_orient, else B): its rows land in the accumulator registers; second: in the lanes
    const uint32_t p_half = (uint32_t)(v_orient ? wm : wn) * 16384, q_half = (uint32_t)(v_orient ? wn : wm) * 16384;

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Sub-step kk of a step multiplies the 16-wide slice kk of the slabs: 8 operand reads, 16 products.  The
    // reads run one sub-step ahead of the products, and the step's barrier sits in front of its LAST sub-step:
    // by then every wavefront holds that sub-step's operands in registers, so the step's two slots take B of step
    // kt + 2 and A of step kt + 3, and the first operands of step kt + 1 are requested while the last 16 products run.
    //
    // The slabs lie in a ring of five (A of step kt in slot 2 kt mod 5, B in the next), so that a step's 16 copies can be
    // dealt over all its products, one to four: half of B's in the last sub-step, half in the next step's first, A's in
    // the second and third.  A CU takes in 64 bytes a clock, which for the 64 KiB of a step is half of its products'
    // time, and copies issued faster than that hold up the products behind them.  With two pairs of slabs all of them had
    // to go out in the last sub-step; the layer over ten prompts of 1024 and 320 questions (d_model 4096) took 2142 us
    // that way, 2050 with B's eight in the last sub-step and A's over the next three, 2014 dealt evenly.
    auto load_ops = [&](int sa, int kk, bf16x8 (&p)[4], bf16x8 (&q)[4]) __attribute__((always_inline)) {
        const int sb = sa == RING - 1 ? 0 : sa + 1;
        const char *ps = smem + (v_orient ? sa : sb) * SLAB_BYTES + p_half, *qs = smem + (v_orient ? sb : sa) * SLAB_BYTES + q_half;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            p[b] = *reinterpret_cast<const bf16x8 *>(ps + r_off[kk] + b * 4096);
            q[b] = *reinterpret_cast<const bf16x8 *>(qs + r_off[kk] + b * 4096);
        }
    };
    auto products = [&](const bf16x8 (&p)[4], const bf16x8 (&q)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int pi = 0; pi < 4; ++pi)
#pragma unroll
            for (int qj = 0; qj < 4; ++qj)
                acc[pi][qj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[pi], q[qj], acc[pi][qj], 0, 0, 0);
    };
    // Issue order of a sub-step: the 8 reads of the next sub-step go out in the shadow of the first 4 products,
    // so that they have landed long before the next sub-step's first product asks for them; the copies at even distances.
    auto order = [&](auto reads, auto copies) __attribute__((always_inline)) {
        constexpr int C = decltype(copies)::value;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one matrix-core instruction
            if (decltype(reads)::value && i < 4) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);     // two LDS reads
            if ((i + 1) * C / 16 != i * C / 16) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);      // one copy
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 4> c4{};
    const std::integral_constant<int, 8> c8{};
    bf16x8 p0[4], q0[4], p1[4], q1[4];
    int sa = 0;                                  // ring slot of A of step kt
    auto ring = [&](int s) __attribute__((always_inline)) { return s >= RING ? s - RING : s; };
    copy_a(0, 0, c0, c8);
    copy_b(0, 1, c0, c8);
    __builtin_amdgcn_sched_barrier(0);           // the waits count copies: they leave in this order
    if (n_steps > 1) {
        copy_a(1, 2, c0, c8);
        copy_b(1, 3, c0, c4);
        step_barrier<12>();                      // the first two slabs have landed
    } else {
        step_barrier<0>();
    }
    load_ops(0, 0, p0, q0);
    __builtin_amdgcn_sched_barrier(0);
    // one step; NEXT: a step follows (barrier, first operands of it), NEXT2: two follow (copies of that one are due)
    auto step = [&](int kt, auto next, auto next2) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next)::value, NEXT2 = decltype(next2)::value;
        const std::true_type reads{};
        const int s4 = ring(sa + 4);
        load_ops(sa, 1, p1, q1);
        if (NEXT) copy_b(kt + 1, ring(sa + 3), c4, c8);
        products(p0, q0);
        order(reads, std::integral_constant<int, NEXT ? 4 : 0>{});
        load_ops(sa, 2, p0, q0);
        if (NEXT2) copy_a(kt + 2, s4, c0, c4);
        products(p1, q1);
        order(reads, std::integral_constant<int, NEXT2 ? 4 : 0>{});
        load_ops(sa, 3, p1, q1);
        if (NEXT2) copy_a(kt + 2, s4, c4, c8);
        products(p0, q0);
        order(reads, std::integral_constant<int, NEXT2 ? 4 : 0>{});
        if (NEXT) {
            // the slabs of step kt + 1 are there when only A of step kt + 2 is on its way; this step's are read out
            step_barrier<NEXT2 ? 8 : 0>();
            __builtin_amdgcn_sched_barrier(0);
            load_ops(ring(sa + 2), 0, p0, q0);
            if (NEXT2) copy_b(kt + 2, sa, c0, c4);
            sa = ring(sa + 2);
        }
        products(p1, q1);
        order(std::integral_constant<bool, NEXT>{}, std::integral_constant<int, NEXT2 ? 4 : 0>{});
    };
    int kt = 0;
    for (; kt + 2 < n_steps; ++kt) step(kt, std::true_type{}, std::true_type{});
    if (kt + 1 < n_steps) step(kt++, std::true_type{}, std::false_type{});
    step(kt, std::false_type{}, std::false_type{});

    if (QKV && g.kv_dest == 1) step_barrier<0>();      // values pass through the slabs' place in LDS: every operand is read
    if (col0 >= N) return;          // the second half of a ragged last column tile
    const int rows16 = (rows + 15) & ~15;

    if (!v_orient) {
        // lane = token 128 wm + 32 qj + l31; register r of accumulator pi = feature 32 pi + 8 (r / 4) + 4 h + r % 4
        const bool to_pages = QKV && kind == 1 && g.kv_dest != 2;
#pragma unroll
        for (int qj = 0; qj < 4; ++qj) {
            const int i = 128 * wm + 32 * qj + l31;
            const bool valid = i < rows;
            bool store = valid;
            char *dst = nullptr;
            int64_t chunk_stride = 16;
            const float2 *tab = nullptr;                         // (to_pages) the rotation's entries at the token's position
            if (to_pages) {
                int page, slot16, pos;
                if (g.kv_dest == 0) {
                    const int p = t.pos0 + i;
                    store = i < rows16;                          // the last page's unused slots are zeroed
                    page = store ? g.page_table[t.pt_off + (p >> 4)] : 0;
                    slot16 = p & 15;
                    pos = p;
                } else {
                    const int4 d = g.row_dest[t.dest0 + (valid ? i : 0)];
                    page = d.x >> 4;
                    slot16 = d.x & 15;
                    pos = d.y;
                }
                dst = g.kv_base + (int64_t)page * g.page_bytes + (int64_t)hk * g.part_bytes + slot16 * 16;
                chunk_stride = 256;
                if (g.rope) tab = g.rope + (int64_t)(valid ? pos : 0) * (HD / 2);
            } else if (kind == 0) {
                store = valid && t.c != nullptr;
                dst = static_cast<char *>(t.c) + ((int64_t)i * g.ldc + col0) * 2;
            } else {
                char *base = static_cast<char *>(kind == 1 ? t.ck : t.cv);
                dst = base + ((int64_t)i * (g.n_kv_heads * HD) + hk * HD) * 2;
            }
            // registers 8 u .. 8 u + 3 are features 16 u + 4 h + 0..3, registers 8 u + 4 .. + 7 features 16 u + 8 + 4 h + 0..3; after the
            // swap between the two 32-lane halves lane h holds the eight consecutive features 16 u + 8 h .. + 7.  Accumulators pi and
            // pi + 2 hold the rotation's partners.  Piece by piece, behind a scheduling barrier each: taken together, the accumulators'
            // copies in ordinary registers did not fit and 80 were spilled.  Llama-3-8B's layer over ten prompts of
            // 1024 tokens and 320 questions of 16 to 64: 1 957 -> 1 942 us.  (32 were left then; with the values' way through LDS and the
            // clearing of last pages beside it 48 are, 240 bytes of scratch memory a lane.)
            auto put = [&](const float (&v)[8], int pi, int u) __attribute__((always_inline)) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = valid ? v[e] : 0.f;
                // keys that go straight into pages are binary16 there; everything else is bf16
                const uint32_t a0 = to_pages ? pack2_f16(x[0], x[1]) : pack2(x[0], x[1]);
                const uint32_t a1 = to_pages ? pack2_f16(x[2], x[3]) : pack2(x[2], x[3]);
                const uint32_t b0 = to_pages ? pack2_f16(x[4], x[5]) : pack2(x[4], x[5]);
                const uint32_t b1 = to_pages ? pack2_f16(x[6], x[7]) : pack2(x[6], x[7]);
                const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
                const uint4 out = make_uint4(s0[0], s1[0], s0[1], s1[1]);
                const int chunk = 4 * pi + 2 * u + h;
                if (store) *reinterpret_cast<uint4 *>(dst + chunk * chunk_stride) = out;
            };
#pragma unroll
            for (int pi = 0; pi < 2; ++pi)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    float x1[8], x2[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        x1[e] = acc[pi][qj][8 * u + e];
                        x2[e] = acc[pi + 2][qj][8 * u + e];
                    }
                    if (tab)
#pragma unroll
                        for (int q4 = 0; q4 < 2; ++q4) {
                            const float4 *cs = reinterpret_cast<const float4 *>(tab + 32 * pi + 8 * (2 * u + q4) + 4 * h);
                            const float4 c01 = cs[0], c23 = cs[1];
                            const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) rotate_pair(x1[4 * q4 + e], x2[4 * q4 + e], co[e], si[e]);
                        }
                    put(x1, pi, u);
                    put(x2, pi + 2, u);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    } else if (g.kv_dest == 1) {
        store_own_values(g, acc, t.dest0 + 128 * wm, min(rows - 128 * wm, 128), hk, smem + wave * V_TILE, lane);
    } else {
        // lane = channel 32 qj + l31 of the head; register r of accumulator pi = token 32 pi + 8 (r / 4) + 4 h + r % 4
#pragma unroll
        for (int pi = 0; pi < 4; ++pi)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r16 = 128 * wm + 32 * pi + 16 * e;      // first of the 16 rows registers 8 e .. 8 e + 7 belong to
                if (r16 >= rows16) continue;
                {
                    // the 16 rows are one page; register 8 e + i is the page's token 4 h + (i & 3) + 8 (i >> 2)
                    const int page = g.page_table[t.pt_off + ((t.pos0 + r16) >> 4)];
                    char *vp = g.kv_base + (int64_t)page * g.page_bytes + (int64_t)(g.n_kv_heads + hk) * g.part_bytes;
#pragma unroll
                    for (int qj = 0; qj < 4; ++qj) {
                        float x[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int tok = r16 + 4 * h + (i & 3) + 8 * (i >> 2);
                            x[i] = tok < rows ? acc[pi][qj][8 * e + i] : 0.f;
                        }
                        const uint4 out = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7]));
                        *reinterpret_cast<uint4 *>(vp + (((qj * 2 + h) * 32) + l31) * 16) = out;
                    }
                }
            }
    }
    if (QKV && kind == 1 && g.kv_dest == 1)
        for (int r = 128 * wm; r < min(rows, 128 * wm + 128); r += 64) {
            const bool mine = r + lane < rows;
            clear_behind_last<HD>(g, g.row_dest[t.dest0 + (mine ? r + lane : r)], mine, kind, hk, 0, lane);
        }
}

// ---- the same products in smaller tiles -----------------------------------------------------------------
// Few rows (a prompt, a handful of questions) make few 256 x 256 tiles: 300 rows x 6144 columns are 48 workgroups on 256
// CUs, each walking the whole contraction alone, 85 us whatever the rows.  Here a workgroup of 4 wavefronts computes a
// TM x TN tile with NST steps of 64 in LDS.  One barrier per step: behind it the step after is visible, and the step's own
// buffer, whose operands every wavefront holds in registers by then, is free for the copies of step kt + NST.  The copies
// are dealt between the products: issued in a row they hold up a wavefront's products for as long as the CU takes to
// accept all of them (14.9 -> 13.8 us at 160 x 4096 x 4096, 41.9 -> 30.5 at 300 rows in 128 x 128 tiles).
// What bounds such a launch is the CUs' intake (64 bytes a clock at best) and a step's chain of barrier, operand reads and
// products.  Tiles of 64 rows therefore split the CONTRACTION between the wavefronts (KS: wavefront w multiplies the
// 16-wide slice w of every step for the whole tile), which reads every operand from LDS once and not twice (22.3 ->
// 14.9 us at 160 x 4096 x 4096); the four partial tiles are added through LDS at the end.
// Tiles of 128 x 128 are split 2 x 2 (their partial tiles would take all registers).
// The result lies in LDS as fp32 [TM][TN + 4], so that the stores to pages and rows can be arranged freely.
// A tile of 64 columns takes channels 32 s .. 32 s + 31 of a head and their rotation partners 64 channels on.
template <int TM_, int TN_, int NST_, int WGS_, bool KS_>
struct SmallTile {
    static constexpr int TM = TM_, TN = TN_;
    static constexpr bool KS = KS_;
    static constexpr int A_BYTES = TM * TK * 2, B_BYTES = TN * TK * 2;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int NST = NST_;
    static constexpr int WGS = WGS_;                             // workgroups per CU (LDS decides), one wavefront per SIMD each
    static constexpr int LD = TN + 4;
    static constexpr int PART = KS ? TM * TN * 4 : 0;            // one wavefront's partial tile
    static constexpr int SUM_BYTES = PART + TM * LD * 4;
    static constexpr int END_BYTES = SUM_BYTES + TM * 16;        // and where the rows go, in a batch's pages
    static constexpr int LDS = NST * STAGE > END_BYTES ? NST * STAGE : END_BYTES;
    static constexpr int COPIES = STAGE / 4096;                  // 1 KiB copies per wavefront and step
};
using Tile64 = SmallTile<64, 64, 5, 2, true>;
using Tile64x128 = SmallTile<64, 128, 6, 1, true>;
using Tile128Deep = SmallTile<128, 128, 4, 1, false>;
using Tile128Pair = SmallTile<128, 128, 2, 2, false>;

template <class T, bool QKV, class ARGS>
__global__ void __launch_bounds__(256, T::WGS) proj_gemm_small_kernel(const ARGS args)
{
    const GemmArgs &g = gemm_args(args);
    constexpr int TM_ = T::TM, TN_ = T::TN, NST = T::NST, LD = T::LD;
    constexpr int KK = T::KS ? 1 : 4;                            // 16-wide slices of a step this wavefront multiplies
    constexpr int MB = TM_ / (T::KS ? 32 : 64), NB = TN_ / (T::KS ? 32 : 64);    // its 32 x 32 blocks
    static_assert(NST >= 2 && T::COPIES * (NST - 1) < 64, "copies in flight are counted in 6 bits");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = T::KS ? 0 : wave >> 1, wn = T::KS ? 0 : wave & 1;
    const int h = lane >> 5, l31 = lane & 31;

    // tile ids walk groups of up to 8 row tiles, column by column; every XCD takes a contiguous run of them, so a weight
    // slab is fetched into one L2 and used there by all row tiles of the group
    const int n_ct = g.n_col_tiles, n_rt = g.n_row_tiles;
    const int total = n_ct * n_rt;
    const int per = (total + 7) >> 3;
    const int local = (int)blockIdx.x >> 3;
    const int tid = ((int)blockIdx.x & 7) * per + local;
    if (local >= per || tid >= total) return;
    constexpr int GM = 8;
    const int grp = tid / (GM * n_ct);
    const int gsz = min(GM, n_rt - grp * GM);
    const int in = tid - grp * GM * n_ct;
    const int rt = __builtin_amdgcn_readfirstlane(grp * GM + in % gsz);
    const int ct = __builtin_amdgcn_readfirstlane(in / gsz);

    const GemmRowTile t = row_tile<ARGS>(g, rt, TM_);
    const int rows = __builtin_amdgcn_readfirstlane(t.rows);
    const int K = g.K;
    const int n_steps = K / TK;

    // column j of the tile is column head0 + col_of(j) of the product
    const int head0 = TN_ == 128 ? ct * 128 : (ct >> 1) * 128;
    const int half32 = TN_ == 128 ? 0 : (ct & 1) * 32;
    auto col_of = [&](int j) __attribute__((always_inline)) { return TN_ == 128 ? j : (j >> 5) * 64 + half32 + (j & 31); };

    // ---- copies: instruction i of a wavefront moves 8 rows; lane (lr, slot) fetches chunk slot ^ perm(row), as above
    const int lr = lane >> 3, slot = lane & 7;
    uint32_t off[T::COPIES];
    constexpr int A_COPIES = T::A_BYTES / 4096;
    const Operand a_op = operand(t.a, (uint32_t)rows * (uint32_t)(K * 2));
    const Operand b_op = operand(static_cast<const char *>(g.w) + (int64_t)head0 * K * 2, 128u * (uint32_t)(K * 2));
#pragma unroll
    for (int i = 0; i < T::COPIES; ++i) {
        const bool is_a = i < A_COPIES;
        const int row = is_a ? (TM_ / 4) * wave + 8 * i + lr : (TN_ / 4) * wave + 8 * (i - A_COPIES) + lr;
        const uint32_t chunk = (uint32_t)(slot ^ lr ^ ((row >> 3) & 1));
        off[i] = (uint32_t)(is_a ? min(row, rows - 1) : col_of(row)) * (uint32_t)(K * 2) + chunk * 16;
    }
    auto issue = [&](int kt, int stage) __attribute__((always_inline)) {
        char *st = smem + stage * T::STAGE;
        const uint32_t k_off = (uint32_t)kt * (TK * 2);
#pragma unroll
        for (int i = 0; i < T::COPIES; ++i) {
            if (i < A_COPIES)
                copy_1k_to_lds(a_op, off[i], k_off, st + wave * (T::A_BYTES / 4) + i * 1024);
            else
                copy_1k_to_lds(b_op, off[i], k_off, st + T::A_BYTES + wave * (T::B_BYTES / 4) + (i - A_COPIES) * 1024);
        }
    };

    f32x16 acc[NB][MB];          // rows of the weight in the registers, rows of the left operand in the lanes
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // operand reads: lane (l31, h) of block b reads row 32 b + l31, chunk 2 kk + h of the step's eight (KS: kk = wave)
    uint32_t r_off[KK];
#pragma unroll
    for (int k = 0; k < KK; ++k)
        r_off[k] = (uint32_t)l31 * 128 + (((uint32_t)(T::KS ? wave : k) * 32) ^ ((uint32_t)(h ^ (lane & 7) ^ ((lane >> 3) & 1)) * 16));
    const uint32_t x_region = (uint32_t)wm * (T::A_BYTES / 2), w_region = T::A_BYTES + (uint32_t)wn * (T::B_BYTES / 2);
    auto load_ops = [&](int stage, bf16x8 (&x)[KK][MB], bf16x8 (&w)[KK][NB]) __attribute__((always_inline)) {
        const char *st = smem + stage * T::STAGE;
#pragma unroll
        for (int k = 0; k < KK; ++k) {
#pragma unroll
            for (int b = 0; b < MB; ++b) x[k][b] = *reinterpret_cast<const bf16x8 *>(st + x_region + b * 4096 + r_off[k]);
#pragma unroll
            for (int b = 0; b < NB; ++b) w[k][b] = *reinterpret_cast<const bf16x8 *>(st + w_region + b * 4096 + r_off[k]);
        }
    };
    int stage = 0;               // buffer of step kt
    auto after = [&](int s) __attribute__((always_inline)) { return s == NST - 1 ? 0 : s + 1; };
    // One step: its operands are in x, w; those of the step behind it go to xn, wn.  STEADY: copies of step kt + NST are due,
    // dealt between the products (all of a workgroup's copies in a row would hold up its products for as long as they take).
    auto step = [&](int kt, const bf16x8 (&x)[KK][MB], const bf16x8 (&w)[KK][NB], bf16x8 (&xn)[KK][MB], bf16x8 (&wn_)[KK][NB], auto steady) __attribute__((always_inline)) {
        constexpr bool STEADY = decltype(steady)::value;
        if (STEADY || kt + NST <= n_steps)     // step kt + 1 has landed when only the copies of the NST - 2 behind it are outstanding
            step_barrier<(NST - 2) * T::COPIES>();
        else
            step_barrier<0>();
        const int mine = stage;
        stage = after(stage);
        if (!STEADY && kt + NST < n_steps) issue(kt + NST, mine);
        load_ops(stage, xn, wn_);         // (behind the last step: some old step's operands, never used)
        if (STEADY) issue(kt + NST, mine);
#pragma unroll
        for (int k = 0; k < KK; ++k)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < MB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[k][i], x[k][j], acc[i][j], 0, 0, 0);
        if (STEADY) {                    // order: one-slice reads first; then products, reads and a copy in turn
            if (T::KS) __builtin_amdgcn_sched_group_barrier(0x100, MB + NB, 0);
#pragma unroll
            for (int i = 0; i < T::COPIES; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, KK * MB * NB / T::COPIES, 0);
                if (!T::KS) __builtin_amdgcn_sched_group_barrier(0x100, KK * (MB + NB) / T::COPIES, 0);
                __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < NST; ++i)
        if (i < n_steps) issue(i, i);
    bf16x8 x0[KK][MB], w0[KK][NB], x1[KK][MB], w1[KK][NB];
    if (n_steps >= NST)
        step_barrier<(NST - 1) * T::COPIES>();
    else
        step_barrier<0>();
    load_ops(0, x0, w0);
    int kt = 0;
    for (; kt + 1 + NST < n_steps; kt += 2) {
        step(kt, x0, w0, x1, w1, std::true_type{});
        step(kt + 1, x1, w1, x0, w0, std::true_type{});
    }
    for (; kt + 2 <= n_steps; kt += 2) {
        step(kt, x0, w0, x1, w1, std::false_type{});
        step(kt + 1, x1, w1, x0, w0, std::false_type{});
    }
    if (kt < n_steps) step(kt, x0, w0, x1, w1, std::false_type{});
    step_barrier<0>();           // every operand is read; the sums take the slabs' place

    int kind = 0, hk = 0;        // 0 plain, 1 K head, 2 V head
    if (QKV && head0 >= g.n_plain) {
        const int kvh = (head0 - g.n_plain) / HD;
        kind = kvh < g.n_kv_heads ? 1 : 2;
        hk = kind == 1 ? kvh : kvh - g.n_kv_heads;
    }
    const bool slots = QKV && kind != 0 && g.kv_dest == 1;
    int4 *const dest = reinterpret_cast<int4 *>(smem + T::SUM_BYTES);
    int4 my_dest = make_int4(0, 0, 0, 0);
    if (slots && (int)threadIdx.x < rows) my_dest = g.row_dest[t.dest0 + threadIdx.x];

    // ---- (KS) the four slices' sums: wavefronts 2 and 3 hand theirs to 0 and 1, which then hand each other half of theirs; the
    // result is written as [TM][LD] behind the hand-over area.
    auto slot_of = [&](char *area, int i, int j, int q4) __attribute__((always_inline)) { return reinterpret_cast<float4 *>(area + (((i * MB + j) * 4 + q4) * 64 + lane) * 16); };
    auto give = [&](char *area, auto i0, auto i1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = i0; i < i1; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *slot_of(area, i, j, q4) = make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
    };
    auto take = [&](char *area, auto i0, auto i1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = i0; i < i1; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const float4 s = *slot_of(area, i, j, q4);
                    acc[i][j][4 * q4] += s.x;
                    acc[i][j][4 * q4 + 1] += s.y;
                    acc[i][j][4 * q4 + 2] += s.z;
                    acc[i][j][4 * q4 + 3] += s.w;
                }
    };
    float *const cs = reinterpret_cast<float *>(smem + T::PART);
    auto put = [&](auto i0, auto i1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = i0; i < i1; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *reinterpret_cast<float4 *>(cs + ((wm * MB + j) * 32 + l31) * LD + (wn * NB + i) * 32 + 8 * q4 + 4 * h) =
                        make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
    };
    const std::integral_constant<int, 0> first{};
    const std::integral_constant<int, NB / 2> middle{};
    const std::integral_constant<int, NB> last{};
    if constexpr (T::KS) {
        if (wave >= 2) give(smem + (wave - 2) * T::PART, first, last);
        __syncthreads();
        if (wave < 2) take(smem + wave * T::PART, first, last);
        __syncthreads();
        if (wave == 0)
            give(smem, middle, last);
        else if (wave == 1)
            give(smem, first, middle);
        __syncthreads();
        if (wave == 0) {
            take(smem, first, middle);
            put(first, middle);
        } else if (wave == 1) {
            take(smem, middle, last);
            put(middle, last);
        }
    } else {
        put(first, last);
    }
    if (slots && (int)threadIdx.x < rows) dest[threadIdx.x] = my_dest;
    __syncthreads();

    const int rows16 = (rows + 15) & ~15;
    if (kind == 0 || g.kv_dest == 2) {
        char *c = static_cast<char *>(kind == 0 ? t.c : kind == 1 ? t.ck : t.cv);
        const int64_t ld = kind == 0 ? g.ldc : g.n_kv_heads * HD;
        const int c0 = kind == 0 ? head0 : hk * HD;
        if (!c) return;
        for (int u = threadIdx.x; u < rows * (TN_ / 8); u += 256) {
            const int i = u / (TN_ / 8), j = (u % (TN_ / 8)) * 8;
            const float4 a = *reinterpret_cast<const float4 *>(cs + i * LD + j), b = *reinterpret_cast<const float4 *>(cs + i * LD + j + 4);
            *reinterpret_cast<uint4 *>(c + (i * ld + c0 + col_of(j)) * 2) = make_uint4(pack2(a.x, a.y), pack2(a.z, a.w), pack2(b.x, b.y), pack2(b.z, b.w));
        }
    } else if (kind == 1) {
        // 8 channels of a token and their partners; slots past a prompt's end in its last page are zeroed
        const int n_rows = g.kv_dest == 0 ? min(rows16, TM_) : rows;
        for (int u = threadIdx.x; u < n_rows * (TN_ / 16); u += 256) {
            const int i = u / (TN_ / 16), p = (u % (TN_ / 16)) * 8;
            const bool valid = i < rows;
            int page, slot16, pos;
            if (g.kv_dest == 0) {
                pos = t.pos0 + i;
                page = g.page_table[t.pt_off + (pos >> 4)];
                slot16 = pos & 15;
            } else {
                const int4 d = dest[i];
                page = d.x >> 4;
                slot16 = d.x & 15;
                pos = d.y;
            }
            float x1[8], x2[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x1[e] = valid ? cs[i * LD + p + e] : 0.f;
                x2[e] = valid ? cs[i * LD + TN_ / 2 + p + e] : 0.f;
            }
            const int c1 = half32 + p;
            if (g.rope && valid) {
                const float4 *tab = reinterpret_cast<const float4 *>(g.rope + (int64_t)pos * (HD / 2) + c1);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 t4 = tab[e];
                    rotate_pair(x1[2 * e], x2[2 * e], t4.x, t4.y);
                    rotate_pair(x1[2 * e + 1], x2[2 * e + 1], t4.z, t4.w);
                }
            }
            char *dst = g.kv_base + (int64_t)page * g.page_bytes + (int64_t)hk * g.part_bytes;
            *reinterpret_cast<uint4 *>(dst + k_page_index(slot16, c1) * 2) = make_uint4(pack2_f16(x1[0], x1[1]), pack2_f16(x1[2], x1[3]), pack2_f16(x1[4], x1[5]), pack2_f16(x1[6], x1[7]));
            *reinterpret_cast<uint4 *>(dst + k_page_index(slot16, c1 + HD / 2) * 2) = make_uint4(pack2_f16(x2[0], x2[1]), pack2_f16(x2[2], x2[3]), pack2_f16(x2[4], x2[5]), pack2_f16(x2[6], x2[7]));
        }
    } else if (g.kv_dest == 0) {
        // a page's 16 tokens of one channel: two runs of 8 tokens, 16 bytes each
        for (int u = threadIdx.x; u < (rows16 / 16) * 2 * TN_; u += 256) {
            const int j = u % TN_, hh = (u / TN_) & 1, r16 = (u / (2 * TN_)) * 16;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int tok = r16 + 4 * hh + (e & 3) + 8 * (e >> 2);
                x[e] = tok < rows ? cs[tok * LD + j] : 0.f;
            }
            const int page = g.page_table[t.pt_off + ((t.pos0 + r16) >> 4)];
            char *vp = g.kv_base + (int64_t)page * g.page_bytes + (int64_t)(g.n_kv_heads + hk) * g.part_bytes;
            *reinterpret_cast<uint4 *>(vp + v_page_index(4 * hh, col_of(j)) * 2) = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7]));
        }
    } else {
        // a page whose rows all lie in this tile: its first row's turn writes it, as above; other rows one by one.  (All rows one by
        // one, two bytes a lane: the projection of the 168 rows of 6 questions 28.5 us, 26.8 so.)
        for (int u = threadIdx.x; u < rows * TN_; u += 256) {
            const int i = __builtin_amdgcn_readfirstlane(u / TN_), j = u % TN_;      // (a wavefront has one row's channels)
            const int4 d = dest[i];
            const int x0 = __builtin_amdgcn_readfirstlane(d.x), n = __builtin_amdgcn_readfirstlane(d.z), slot = x0 & 15;
            const bool whole = n > 0 && i >= slot && i - slot + n <= rows;
            if (whole && slot > 0) continue;
            char *vp = g.kv_base + (int64_t)(x0 >> 4) * g.page_bytes + (int64_t)(g.n_kv_heads + hk) * g.part_bytes;
            if (whole) {
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int tok = 4 * hh + (e & 3) + 8 * (e >> 2);
                        x[e] = tok < n ? cs[(i + tok) * LD + j] : 0.f;
                    }
                    *reinterpret_cast<uint4 *>(vp + v_page_index(4 * hh, col_of(j)) * 2) = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7]));
                }
            } else {
                *reinterpret_cast<__bf16 *>(vp + v_page_index(slot, col_of(j)) * 2) = (__bf16)cs[i * LD + j];
            }
        }
    }
    if (slots) {
        const int r0 = wave * (TM_ / 4), i = r0 + lane;
        const bool in_tile = lane < TM_ / 4 && i < rows;
        const int4 d = dest[in_tile ? i : 0];
        const int slot = d.x & 15;
        const bool whole = kind == 2 && d.z > 0 && i >= slot && i - slot + d.z <= rows;
        clear_behind_last<TN_>(g, d, in_tile && !whole, kind, hk, half32, lane);
    }
}

// Any shape and both io types, one output element per thread, fp32 accumulation; columns are dealt to up to
// three row-major outputs (Q, K, V or just one).
__device__ inline float load_io(const void *p, int64_t i, int io_dtype)
{
    return io_dtype == SGC_F32 ? static_cast<const float *>(p)[i] : (float)static_cast<const __bf16 *>(p)[i];
}
__device__ inline void store_io(void *p, int64_t i, int io_dtype, float x)
{
    if (io_dtype == SGC_F32)
        static_cast<float *>(p)[i] = x;
    else
        static_cast<__bf16 *>(p)[i] = (__bf16)x;
}

__global__ void __launch_bounds__(256) proj_generic_kernel(const void *a, const void *w, int64_t M, int N, int K, int io_dtype,
                                                           void *c0, int n0, void *c1, int n1, void *c2)
{
    __shared__ float as[16][17], ws[16][17];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int64_t m = (int64_t)blockIdx.y * 16 + ty;
    const int n = blockIdx.x * 16 + tx;
    float sum = 0.f;
    for (int k0 = 0; k0 < K; k0 += 16) {
        const int64_t am = (int64_t)blockIdx.y * 16 + ty;
        const int wn_ = blockIdx.x * 16 + ty;
        as[ty][tx] = (am < M && k0 + tx < K) ? load_io(a, am * K + k0 + tx, io_dtype) : 0.f;
        ws[ty][tx] = (wn_ < N && k0 + tx < K) ? load_io(w, (int64_t)wn_ * K + k0 + tx, io_dtype) : 0.f;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += as[ty][k] * ws[tx][k];
        __syncthreads();
    }
    if (m >= M || n >= N) return;
    if (n < n0) {
        if (c0) store_io(c0, m * n0 + n, io_dtype, sum);
    } else if (n < n0 + n1) {
        store_io(c1, m * n1 + (n - n0), io_dtype, sum);
    } else {
        store_io(c2, m * (N - n0 - n1) + (n - n0 - n1), io_dtype, sum);
    }
}

}  // namespace


namespace {

const GemmArgs &gemm_host_args(const GemmArgs &a) { return a; }
const GemmArgs &gemm_host_args(const GemmCarried &c) { return c.a; }

template <bool QKV, class ARGS>
hipError_t launch_tiles(const ARGS &args, hipStream_t s)
{
    const GemmArgs &g = gemm_host_args(args);
    const int blocks = (g.n_row_tiles * g.n_col_tiles + 7) / 8 * 8;
    auto launch = [&](auto kern, int lds, bool &configured) {
        if (!configured) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            configured = true;
        }
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, s, args);
        return hipGetLastError();
    };
    static bool configured[GEMM_64 + 1] = {};
    switch (g.kind) {
        case GEMM_128_DEEP: return launch(proj_gemm_small_kernel<Tile128Deep, QKV, ARGS>, Tile128Deep::LDS, configured[g.kind]);
        case GEMM_128_PAIR: return launch(proj_gemm_small_kernel<Tile128Pair, QKV, ARGS>, Tile128Pair::LDS, configured[g.kind]);
        case GEMM_64X128: return launch(proj_gemm_small_kernel<Tile64x128, QKV, ARGS>, Tile64x128::LDS, configured[g.kind]);
        case GEMM_64: return launch(proj_gemm_small_kernel<Tile64, QKV, ARGS>, Tile64::LDS, configured[g.kind]);
        default: return launch(proj_gemm_kernel<QKV, ARGS>, GEMM_LDS, configured[GEMM_256]);
    }
}

// What a launch of n tiles takes, in microseconds, on a chip of 256 CUs: a start, per round of tiles a fixed part (first
// copies, sums, stores) and one per 64-wide step, less for a last round that leaves CUs idle or with one workgroup instead of
// two; tiles that write keys and values into pages cost more, most where the slots are a batch's.
// Fitted to 1053 shapes (16 to 16384 rows, 128 to 12288 columns, contractions of 64 to 8192; plain, prompt and batch
// products), every tile kind measured on each, when the kernels copied slabs by global loads, stored a batch's values two
// bytes a lane and cleared its last pages by a launch of its own: within 5 % in the median and 22 % for nine in ten then.  The present ones,
// on 1 410 other shapes of these ranges: within 7 % and 24 %, most off for a batch's tiles, which have become cheaper.  Some, us,
// 256 x 256 / 128 x 128 deep / pairs / 64 x 128 / 64 x 64, then and now:
//   1000 x 4096 x 4096 (plain)                   73 / 40 / 46 / 45 / 49            73 / 39 / 47 / 46 / 50
//   16384 x 4096 x 4096 (plain)                  421 / 620 / 509 / 699 / 760       395 / 607 / 487 / 700 / 744
//   6400 x 6144 x 1024, batch                    123 / 152 / 118 / 205 / 154       108 / 143 / 105 / 196 / 145
//   10 x 1024 x 10240 x 1024, prompts            242 / 296 / 236 / 474 / 387       214 / 310 / 229 / 480 / 373
struct TileCost {
    double start, round, step;              // per full round
    double last, last_step;                 // of a last round with (nearly) idle CUs
    double kv_pages, kv_slots;              // per round made of key and value tiles alone ...
    double kv_pages_last, kv_slots_last;    // ... and what the last of their stores adds
};
constexpr TileCost kTileCost[5] = {
    {0.3, 9.0, 1.52, 6.5, 1.045, 2.2, 14.7, 11.5, 13.5},        // GEMM_256
    {2.2, 2.3, 0.546, 2.3, 0.42, 2.4, 10.3, 2.0, 7.5},          // GEMM_128_DEEP
    {3.0, 2.8, 0.925, 0.4, 0.525, 2.0, 11.4, 2.8, 9.5},         // GEMM_128_PAIR: a round is 512 tiles
    {1.4, 4.5, 0.281, 4.7, 0.199, 1.4, 5.2, 1.6, 2.7},          // GEMM_64X128
    {2.5, 2.0, 0.34, 2.9, 0.122, 0.65, 2.7, 0.5, 0.0},          // GEMM_64: a round is 512 tiles
};
// kv: share of the columns that are keys and values, kv_dest where they go (GemmArgs)
double proj_gemm_estimate(int kind, int64_t n, int K, double kv, int kv_dest)
{
    const TileCost &c = kTileCost[kind];
    const bool pairs = kind == GEMM_128_PAIR || kind == GEMM_64;
    const int64_t slots = pairs ? 512 : 256, full = n / slots;
    const double steps = K / 64, x = (double)(n % slots) / (double)slots;      // x: how full the last round is
    const double whole = c.round + c.step * steps, least = c.last + c.last_step * steps;
    double last = 0.0, rounds = (double)full;
    if (x > 0.0) {
        if (kind == GEMM_128_PAIR)
            last = least + std::max(0.0, (x - 0.25) / 0.75) * (whole - least);
        else if (kind == GEMM_64)
            last = x <= 0.5 ? least : whole;
        else
            last = least + x * x * x * (c.step - c.last_step) * steps;
        rounds += kind == GEMM_128_PAIR ? x : kind == GEMM_64 && x <= 0.5 ? 0.5 : 1.0;
    }
    double us = c.start + (double)full * whole + last;
    if (kv > 0.0 && kv_dest < 2) us += rounds * kv * (kv_dest == 0 ? c.kv_pages : c.kv_slots) + (kv_dest == 0 ? c.kv_pages_last : c.kv_slots_last);
    return us;
}

}  // namespace

int proj_gemm_tile_rows(int kind) { return kind == GEMM_256 ? 256 : kind == GEMM_128_DEEP || kind == GEMM_128_PAIR ? 128 : 64; }
int proj_gemm_tile_cols(int kind) { return kind == GEMM_256 ? 256 : kind == GEMM_64 ? 64 : 128; }

// The cheapest way by the estimate: all rows in tiles of one kind, or as many 256-row slabs as fill whole rounds of the chip
// with 256 x 256 tiles and the rest in smaller ones (12977 x 4096 columns are 3.2 rounds: the fifth of a round that would
// take a whole one goes out in 192 tiles of 128 x 128).  A second launch costs its start and the first one's drain: 4 us, 6
// where slots of a batch are written, nothing beyond the stores counted above where whole pages are.  256 x 256 tiles alone
// are kept unless something is 3 % cheaper: over the fit's shapes the choice took 1.0 % longer than the best one in the
// mean, and more than 3 % longer than 256 x 256 tiles alone on three (800 x 12288 x 128 to 512 of a batch, 1 to 4 us).  With the present kernels
// it takes 2.0 % longer in the mean of those 1 410, and more than 3 % longer than 256 x 256 tiles alone on 42, nearly all of a batch and short
// contractions (784 x 12288 x 640 46.6 us for 35.3, 3853 x 3072 x 128 38.0 for 26.2; 10 x 1024 x 10240 x 1024 of prompts 229 for 214).  (One
// time per step whatever the columns hold, and nothing per round, sent 6400 rows x 6144 x 1024 of a batch out in two
// launches, 140 us for 123.)
GemmPlan proj_gemm_plan(const int32_t *slab_rows, int n_slabs, int N, int K, int n_plain, int kv_dest)
{
    const double kv = (double)(N - n_plain) / (double)N;
    // row tiles of the slabs behind the first `skip`, by tile height
    auto cheapest = [&](int skip, bool big_too, int *kind) {
        double best = 1e30;
        for (int k = GEMM_256; k <= GEMM_64; ++k) {
            if (k == GEMM_256 && !big_too) continue;
            const int tm = proj_gemm_tile_rows(k), tn = proj_gemm_tile_cols(k);
            int64_t rt = 0;
            for (int i = skip; i < n_slabs; ++i) rt += (slab_rows[i] + tm - 1) / tm;
            const double e = proj_gemm_estimate(k, rt * ((N + tn - 1) / tn), K, kv, kv_dest) * (k == GEMM_256 ? 0.97 : 1.0);
            if (e < best) {
                best = e;
                *kind = k;
            }
        }
        return best;
    };
    GemmPlan p{0, GEMM_256};
    const double best = cheapest(0, true, &p.rest);
    if (p.rest == GEMM_256) p.big_slabs = n_slabs;
    const int ct = (N + 255) / 256;
    const int64_t rounds = (int64_t)n_slabs * ct / 256;
    const int big = (int)(rounds * 256 / ct);
    if (big > 0 && big < n_slabs) {
        int rest = GEMM_64;
        const double both = proj_gemm_estimate(GEMM_256, (int64_t)big * ct, K, kv, kv_dest) + cheapest(big, false, &rest) + (kv > 0.0 && kv_dest == 0 ? 0.0 : kv > 0.0 && kv_dest == 1 ? 6.0 : 4.0);
        if (both < best) p = GemmPlan{big, rest};
    }
    return p;
}

extern "C" void sgc_debug_projection_plan(const int32_t *slab_rows, int32_t n_slabs, int32_t N, int32_t K, int32_t n_plain, int32_t kv_dest, int32_t *out)
{
    const GemmPlan p = proj_gemm_plan(slab_rows, n_slabs, N, K, n_plain, kv_dest);
    out[0] = p.big_slabs;
    out[1] = p.rest;
}

hipError_t launch_proj_gemm(const GemmArgs &g, bool qkv, hipStream_t s, const GemmRowTile *carried)
{
    if (g.n_row_tiles * g.n_col_tiles <= 0) return hipSuccess;
    if (!carried) return qkv ? launch_tiles<true>(g, s) : launch_tiles<false>(g, s);
    if (!qkv || g.n_row_tiles > GemmCarried::kTiles) return hipErrorInvalidValue;
    GemmCarried c;
    c.a = g;
    memcpy(c.tiles, carried, (size_t)g.n_row_tiles * sizeof(GemmRowTile));
    memset(c.tiles + g.n_row_tiles, 0, (size_t)(GemmCarried::kTiles - g.n_row_tiles) * sizeof(GemmRowTile));
    return launch_tiles<true>(c, s);
}

hipError_t launch_proj_generic(const void *a, const void *w, int64_t M, int N, int K, int io_dtype, void *c0, int n0, void *c1,
                               int n1, void *c2, hipStream_t s)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    hipLaunchKernelGGL(proj_generic_kernel, dim3((N + 15) / 16, (unsigned)((M + 15) / 16)), dim3(256), 0, s, a, w, M, N, K, io_dtype,
                       c0, n0, c1, n1, c2);
    return hipGetLastError();
}

}  // namespace sgc
