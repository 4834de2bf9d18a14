// Streaming-mask prefill attention (Sec. 3.2, "Streaming Attention Mask Matrix", Eq. 2).
//
// The dense additive mask of Eq. 2 never exists here.  Work is cut into query tiles
// of one stream of one sequence (st::WorkItem), and each item walks two runs of key
// tiles in stream-compact coordinates:
//   block A -- causal over the row's own stream (source x source, or reasoning x
//              reasoning),
//   block B -- for reasoning rows, the prefix of the source stream they may see.
// Inside a run, tiles [0, full) need no mask, tiles [full, total) compare the column
// index with a per-row limit, tiles past `total` are never read.
//
// Kernels:
//   prefill_attn_kernel<D, NH, ROPE, PACK>
//                         bf16, 4 waves of 32 query rows x NH query heads (1 or 2) of one KV head -- 128 rows of the
//                         same head(s), or fewer rows of more heads (head_waves); K and V
//                         tiles copied asynchronously into swizzled LDS buffers, with one head per wave straight from the
//                         rows of the tensors (no packed copy: 4 x 4K tokens 272 -> 257 us, 96 short sequences
//                         486 -> 461, results the same bit for bit); QK^T and PV on
//                         v_mfma_f32_32x32x16_bf16, fp32 softmax state.  Both products are computed
//                         TRANSPOSED (S^T = K Q^T, O^T = V^T P^T): a lane then owns one query row, so a
//                         row sum is an in-register reduction plus one exchange with lane^32, and the S^T
//                         accumulators are already laid out as the B operand of the second product.  The
//                         loop is software-pipelined by hand (see the kernel).
//   tile_pack_kernel      packed tiles (PACK: the two-head form always; the one-head form on long sequences, where a result
//                         lies over K or V, and for tensors within 4 KB of 4 GiB): K rows and TRANSPOSED V rows of every
//                         64-row key tile (stream-compact order) gathered into contiguous 16 KB blocks.
//   rope_table_kernel, key_pack_rope_kernel
//                         the fused rotation of st_attn_prefill_rope: (cos, sin) of every token once, keys rotated
//                         on their way into the key tiles; the attention kernel's ROPE form rotates its query rows.
// (fp32 tensors take the kernel of st_attn_f32.hip, over the same work items.)
#include <type_traits>

#include "st_tiles.h"

namespace st {

// Fused rotation (Sec. 3.2), step 1: the (cos, sin) pairs of every packed row, evaluated ONCE per token (not once per head):
// the key pack below and the attention kernel's query load both rotate with them.  Laid out for the latter, whose lane (n, hg)
// holds the dims 16 j + 8 hg .. + 7 of row n: per 32 rows of a packed tile [j][w][hg][n] pairs 16 j + 8 hg + 2 w and + 1, so
// that a load instruction takes 1 KB in one piece (row by row it took 16 bytes of each of 32 rows, and the rotation was a
// quarter of the kernel on short sequences).  The angle position * theta^(-2i/D) is reduced in fp64, cos / sin are fp32
// (rope_cos_sin).  One workgroup per packed tile.
template <int D>
__device__ __forceinline__ size_t rope_table_at(size_t packed_row, int j, int w, int hg) {       // in f32x4 units
    return (packed_row >> 5) * (32 * D / 4) + ((j * 4 + w) * 2 + hg) * 32 + (packed_row & 31);
}
template <int D>
__global__ __launch_bounds__(256) void rope_table_kernel(float2* __restrict__ tab, const int32_t* __restrict__ positions, PlanView pv,
                                                         RopeFreq freq) {
    constexpr int HALF = D / 2;
    __shared__ double s_freq[HALF];
    __shared__ int s_pos[kTileN];
    const int tile = blockIdx.x;
    const TileInfo info = pv.tiles[tile];
    if (info.valid == 0) return;                    // spare tile of a sequence: never read
    if (threadIdx.x < kTileN) s_pos[threadIdx.x] = positions[pv.perm[info.base + min(int(threadIdx.x), info.valid - 1)]];
    else if (threadIdx.x < kTileN + HALF) s_freq[threadIdx.x - kTileN] = freq.f[threadIdx.x - kTileN];
    __syncthreads();
    f32x4* out = reinterpret_cast<f32x4*>(tab) + rope_table_at<D>(size_t(tile) * kTileN, 0, 0, 0);
    for (int x = threadIdx.x; x < kTileN * D / 4; x += 256) {        // in the order of the layout, two pairs each
        const int n = x & 31, hg = (x >> 5) & 1, jw = (x >> 6) % (D / 8), blk = x / (32 * D / 4);
        const int i = 16 * (jw >> 2) + 8 * hg + 2 * (jw & 3);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            float cs, sn;
            rope_cos_sin(s_pos[32 * blk + n], s_freq[i + e], &cs, &sn);
            v[2 * e] = cs;
            v[2 * e + 1] = sn;
        }
        out[x] = v;
    }
}

// Step 2: UNROTATED keys into packed row tiles -- every key row is rotated with its table row on its way.  A thread owns two rows (one with
// heads of 64 dims) x one pair of 8-dim pieces (dims 8 cp .. + 7 and D/2 + the same) of `heads` heads: the table rows, twice the
// bytes of a key row, are read once for all of them.
template <int D>
__global__ __launch_bounds__(256) void key_pack_rope_kernel(uint16_t* __restrict__ kc, const float2* __restrict__ tab, const uint16_t* __restrict__ k,
                                                           PlanView pv, int n_kv_heads, int heads) {
    constexpr int KCH = D / 8, CP = KCH / 2;
    constexpr int PER_THREAD = kTileN * CP / 256;
    const int sets = (n_kv_heads + heads - 1) / heads;
    const int tile = blockIdx.x / sets, h0 = int(blockIdx.x % sets) * heads, h1 = min(h0 + heads, n_kv_heads);
    const TileInfo info = pv.tiles[tile];
    if (info.valid == 0) return;                    // spare tile of a sequence: never read
    const uint32_t row_stride = uint32_t(n_kv_heads) * D;
    const f32x4* tab4 = reinterpret_cast<const f32x4*>(tab);
    f32x4 cs[PER_THREAD][4];                        // (cos, sin) of pairs 8 cp + 2 w and + 1
    uint32_t at[PER_THREAD];                        // the piece of head 0
    bool live[PER_THREAD];
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        const int c = int(threadIdx.x) + 256 * u, row = c / CP, cp = c % CP;
        live[u] = row < info.valid;
        const int r = min(row, info.valid - 1);
        at[u] = uint32_t(pv.perm[info.base + r]) * row_stride + uint32_t(cp) * 8;
#pragma unroll
        for (int w = 0; w < 4; ++w) cs[u][w] = tab4[rope_table_at<D>(size_t(tile) * kTileN + r, cp >> 1, w, cp & 1)];
    }
    for (int h = h0; h < h1; ++h) {
        uint16_t* kdst = kc + (size_t(h) * pv.pack_tiles + tile) * (kTileN * D);
        u32x4 lo_in[PER_THREAD], hi_in[PER_THREAD];
#pragma unroll
        for (int u = 0; u < PER_THREAD; ++u) {
            const uint16_t* kr = k + at[u] + uint32_t(h) * D;
            lo_in[u] = *reinterpret_cast<const u32x4*>(kr);
            hi_in[u] = *reinterpret_cast<const u32x4*>(kr + D / 2);
        }
#pragma unroll
        for (int u = 0; u < PER_THREAD; ++u) {
            const int c = int(threadIdx.x) + 256 * u, row = c / CP, cp = c % CP;
            u32x4 lo, hi;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t out_lo = 0, out_hi = 0;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const float c1 = cs[u][w][2 * half], s1 = cs[u][w][2 * half + 1];
                    const float x = bf16_bits_to_f32(uint16_t(lo_in[u][w] >> (16 * half))), y = bf16_bits_to_f32(uint16_t(hi_in[u][w] >> (16 * half)));
                    out_lo |= uint32_t(f32_to_bf16_bits(x * c1 - y * s1)) << (16 * half);
                    out_hi |= uint32_t(f32_to_bf16_bits(y * c1 + x * s1)) << (16 * half);
                }
                lo[w] = live[u] ? out_lo : 0u;
                hi[w] = live[u] ? out_hi : 0u;
            }
            const int lr = swap23(row);                                    // row position in the tile
            *reinterpret_cast<u32x4*>(kdst + lr * D + (cp ^ swizzle_key<2 * D>(lr)) * 8) = lo;
            *reinterpret_cast<u32x4*>(kdst + lr * D + ((cp + CP) ^ swizzle_key<2 * D>(lr)) * 8) = hi;
        }
    }
}

// V^T tiles (blockIdx.y = 0: [D][64 rows], swizzled) and row tiles of K as it is (1; not where the key pack above has written rotated ones).
// On long sequences a tile is copied into LDS a hundred times and more, and 16 KB in one piece and operands of one LDS read cost the
// attention less than rows looked up and read transposed (two-head form, 8 x 16K tokens, 32 / 8 heads: 11.89 ms with this pass over
// memory, 12.04 with gathered rows, 12.0 with packed row tiles of V; the one-head form's lines stand at the dispatch).
template <int D>
__global__ __launch_bounds__(256) void tile_pack_kernel(uint16_t* __restrict__ vc, const uint16_t* __restrict__ v, uint16_t* __restrict__ kc,
                                                        const uint16_t* __restrict__ k, PlanView pv, int n_kv_heads) {
    const int tile = blockIdx.x / n_kv_heads, h = blockIdx.x % n_kv_heads;
    const TileInfo info = pv.tiles[tile];
    if (info.valid == 0) return;                    // spare tile of a sequence: never read
    const int base = info.base, valid = info.valid;
    const uint32_t row_stride = uint32_t(n_kv_heads) * D;
    const size_t at = (size_t(h) * pv.pack_tiles + tile) * (kTileN * D);
    if (blockIdx.y == 1) {
        pack_rows<D>(kc + at, k, pv.perm + base, valid, row_stride, uint32_t(h), [](int, uint32_t, const u32x4&) {});
        return;
    }
    // 8 keys x 8 d per thread (16-byte loads), transposed in registers to 8 d x 8 keys (16-byte stores)
    const int kvb = threadIdx.x & 7, dq = threadIdx.x >> 3;
    if (dq >= D / 8) return;
    u32x4 vreg[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int row = kvb * 8 + r;
        vreg[r] = u32x4{0u, 0u, 0u, 0u};
        if (row < valid) vreg[r] = *reinterpret_cast<const u32x4*>(v + (uint32_t(pv.perm[base + row]) * row_stride + uint32_t(h) * D + dq * 8));
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {                   // word w of every row holds d = 2 w and 2 w + 1
        u32x4 even, odd;
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const uint32_t a = vreg[2 * pr][w], bb = vreg[2 * pr + 1][w];
            even[pr] = __builtin_amdgcn_perm(bb, a, 0x05040100u);   // low halves
            odd[pr] = __builtin_amdgcn_perm(bb, a, 0x07060302u);    // high halves
        }
        const int d0 = dq * 8 + 2 * w;
        *reinterpret_cast<u32x4*>(vc + at + d0 * kTileN + (kvb ^ swizzle_key<2 * kTileN>(d0)) * 8) = even;
        *reinterpret_cast<u32x4*>(vc + at + (d0 + 1) * kTileN + (kvb ^ swizzle_key<2 * kTileN>(d0 + 1)) * 8) = odd;
    }
}

template <int D, int STAGES>
struct PipeSmem {
    uint16_t k[STAGES][kTileN * D], v[STAGES][kTileN * D];       // K row tiles; V row tiles, packed V^T tiles
    unsigned char tokens[STAGES == 2 ? RowGather<D>::kBytes : 16];       // (gathered rows)
};
// --------------------------------------------------------------------------
// The attention kernel (bf16): NH = 1 or 2 query heads of one KV head per workgroup.
// Every wave owns 32 query rows of a work item for NH query heads that share a KV head.
//   NH = 2  A K (or V^T) operand fragment read from LDS feeds two matrix instructions and one tile copied into
//           LDS serves twice the arithmetic: LDS read traffic and L2 -> LDS copy traffic per flop are both halved.
//           The price is registers (two output accumulators, two score blocks, two Q operands: about 430 per lane,
//           the accumulators in accumulation registers), so one wave per SIMD; three K and three V^T buffers
//           (96 KB), K copied two tiles ahead.
//   NH = 1  fits the ordinary vector registers twice per SIMD: two workgroups per CU, two buffers each (64 KB,
//           and 4 KB of tokens of gathered rows), copies one tile ahead.
// Either way a wave cannot count on other waves to fill the matrix pipe while it does its softmax, so the loop
// is software-pipelined by hand, in the exact instruction order wanted:
//   phase X of tile t:  scores of tile t+1   beside  exp2 / bf16 P / row sum of tile t
//   phase Y of tile t:  O^T += V^T P^T        beside  the exponents of tile t+1 leaving the accumulation registers
// with ONE barrier per key tile, and the vector work per matrix instruction cut to what one wave can issue beside
// its own matrix instructions: it issues at most one instruction every few cycles; beside a
// v_mfma_f32_32x32x16_bf16 (32 cycles of the matrix pipe) about 3.5 plain vector instructions are free, every
// further one costs about 5 cycles, a ds_read_b128 about 4 and a v_dot2_f32_bf16 about 18 -- it shares the matrix
// pipe (measured on this chip, one wave per SIMD).
//   * The queries are multiplied by scale * log2(e) once, when they are loaded (and rounded to bf16 again), and
//     the first matrix instruction of a score block starts from -m_ref instead of 0: a score leaves the matrix
//     pipe as the base-2 exponent of its probability relative to the row's reference exponent m_ref -- no
//     multiply-add per element.  (NH = 1 keeps -m_ref in registers of its own,
//     NH = 2 parks it in the last score block between two tiles.)
//   * No running maximum.  m_ref is the row maximum of the FIRST tile (every row sees column 0 of its own stream,
//     so it is finite); bf16 and fp32 have the same exponent range, so probabilities may grow far beyond 1 without
//     any loss.  Only when a tile's row sum exceeds 2^kRiseLog2 (or is not finite) -- seen right after the
//     probabilities of that tile were formed, before they are used -- the reference is moved, out of line: the
//     tile's probabilities are formed again, the sum and the output accumulator are rescaled.
//   * The first operand fragments of a phase are read from LDS in the slots of the phase before that need no
//     fragment of their own any more (with three buffers the K tile is known to have landed one tile early), and
//     the copies of the next tiles are issued behind the first matrix instructions instead of in front of them.
//   * The last tile of an item has no scores behind it: it is peeled out of the loop, whose body has no branch
//     around its matrix instructions.
// What was tried on top and did not pay: the first product's matrix instructions placed by hand with their results
// in ordinary vector registers (no move out of the accumulation registers, a third of the vector instructions
// gone): as fast, not faster -- the vector instructions co-execute less often with matrix instructions that use the
// same register file (SQ_VALU_MFMA_COEXEC_CYCLES fell by a quarter); longer LDS rings (tiles requested three or four
// tiles ahead): no change, the copies are not waited for.  Removing the tile copies altogether (wrong results, same
// instruction stream otherwise) makes the kernel 15 % faster through the CLOCK, not through cycles: the chip is
// power-limited under this kernel and the L2 -> LDS traffic is part of the bill; what can be saved of it is saved
// by the order of the work items (see st_plan.hip).
// --------------------------------------------------------------------------
constexpr float kRiseLog2 = 24.f;

// PACK: K and V^T come as packed tiles (always with NH = 2); else V's rows, and K's without ROPE, are gathered from the tensors.
template <int D, int NH, bool ROPE, bool PACK>
__global__ __launch_bounds__(256, NH == 2 ? 1 : 2) void prefill_attn_kernel(uint16_t* __restrict__ out, float* __restrict__ lse,
                                                                   const uint16_t* __restrict__ q,
                                                                   const uint16_t* __restrict__ k,
                                                                   const uint16_t* __restrict__ v, PlanView pv,
                                                                   int n_q_heads, int n_kv_heads, float scale_log2,
                                                                   const float2* __restrict__ rope_tab, int head_waves) {
    constexpr int KS = D / 16, DB = D / 32, SB = kTileN / 32;
    constexpr int TILE = kTileN * D;
    constexpr int STAGES = NH == 2 ? 3 : 2;
    static_assert(NH == 1 || PACK, "three buffers, no tokens");
    constexpr bool PACKED_V = PACK, PACKED_K = PACK || ROPE;
    constexpr bool EARLY_K = STAGES == 3;          // K(t + 2) has landed when tile t starts: its first fragments may be read a phase early
    constexpr int PER = 16 / KS;                   // score elements of vector work per matrix instruction (both phases)
    constexpr int kPF = 3;                         // operand fragments read ahead
    extern __shared__ __align__(16) unsigned char smem_raw[];
    PipeSmem<D, STAGES>& sm = *reinterpret_cast<PipeSmem<D, STAGES>*>(smem_raw);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hg = lane >> 5;

    // workgroup -> (work item, part of its rows, set of NH x head_waves query heads of one KV head)
    const int heads_here = NH * head_waves;
    const int n_sets = n_q_heads / heads_here;
    const int row_parts = item_parts(pv, head_waves);
    const int per_item = n_sets * row_parts;
    const int rank = blockIdx.x / per_item;
    const int rem = blockIdx.x % per_item;
    const int hh0 = rem % n_sets, sub = row_parts - 1 - rem / n_sets;              // (later rows have the longer loops: first)
    const int group = n_q_heads / n_kv_heads;
    const int hk = hh0 % n_kv_heads;                // consecutive workgroups -> consecutive KV heads
    const int hq0 = hk * group + heads_here * (hh0 / n_kv_heads) + NH * (wave % head_waves);
    WorkItem it = pv.sorted[rank];
    if (head_waves > 1) it = item_part(it, pv, sub, kTileM / head_waves);
    if (it.n_rows <= 0) return;
    const int n_tiles = it.a_total + it.b_total;

    constexpr int NL = TILE * 2 / 1024 / 4;         // 1 KB copies per wave per tile
    // K and V tiles: packed ones (PACK: K rows, V^T; ROPE: the rotated K rows), each a linear copy, or rows gathered from the tensor.
    // A copy instruction takes its base from scalar registers and one 32-bit byte offset per lane.
    const uint16_t* k_head = PACKED_K ? k + size_t(hk) * pv.pack_tiles * TILE : k + hk * D;
    const uint16_t* v_head = PACKED_V ? v + size_t(hk) * pv.pack_tiles * TILE : v + hk * D;
    const uint32_t lane_off = uint32_t(wave) * (NL * 1024) + uint32_t(lane) * 16;
    const RowGather<D> rows(sm.tokens, wave, lane, uint32_t(n_kv_heads) * (2 * D));
    auto tile_of = [&](int ti) {
        ti = min(ti, n_tiles - 1);                   // past the end: fetch the last tile again (never used)
        return ti < it.a_total ? it.tile_a0 + ti : it.tile_b0 + (ti - it.a_total);
    };
    auto copy_tokens = [&](int ti) {
        const int t = min(ti, n_tiles - 1);
        const bool in_a = t < it.a_total;
        rows.copy_tokens(pv.perm + (in_a ? it.a_base : it.b_base), (in_a ? t : t - it.a_total) * kTileN, (in_a ? it.n_stream : it.n_src) - 1, ti);
    };
    const uint32_t lds_k0 = uint32_t(uintptr_t(&sm.k[0][0])) + uint32_t(wave) * (NL * 1024);
    const uint32_t lds_v0 = uint32_t(uintptr_t(&sm.v[0][0])) + uint32_t(wave) * (NL * 1024);
    // byte offsets of the lane's pieces of a tile (gathered rows): K's, and V's of the same tile an iteration later
    uint32_t off_k[NL], off_v[NL];
    auto issue_k = [&](int ti, int stage) {
        if constexpr (PACKED_K) async_copy_rows<NL>(k_head + size_t(tile_of(ti)) * TILE, lane_off, lds_k0 + stage * (TILE * 2));
        else RowGather<D>::copy(RowGather<D>::base(k_head), off_k, lds_k0 + stage * (TILE * 2));
    };
    auto issue_v = [&](int ti, int stage) {
        if constexpr (PACKED_V) async_copy_rows<NL>(v_head + size_t(tile_of(ti)) * TILE, lane_off, lds_v0 + stage * (TILE * 2));
        else RowGather<D>::copy(RowGather<D>::base(v_head), off_v, lds_v0 + stage * (TILE * 2));
    };
    // offsets of tile ti as K's (or V's, where K is packed); V's are K's of an iteration ago
    auto next_offsets = [&](int ti) {
        if constexpr (PACKED_K) rows.offsets(off_v, ti);
        else rows.offsets(off_k, ti);
    };
    auto keep_offsets = [&]() {
        if constexpr (!PACKED_K) {
#pragma unroll
            for (int i = 0; i < NL; ++i) off_v[i] = off_k[i];
        }
    };
    // The tokens of the rows and of the first tiles, then the queries and the first key tile, then the other copies: a wait for an ordinary load also waits
    // for the copies in flight (they are counted alike), so only what the first scores need is asked for before the queries
    // are there.
    const int row_in_tile = (wave / head_waves) * 32 + n;
    const bool active = row_in_tile < it.n_rows;
    const int my_row = it.row0 + min(row_in_tile, it.n_rows - 1);
    const int tok_q = pv.perm[it.a_base + my_row];
    const int my_vis = pv.vis[it.a_base + my_row];
    constexpr int kAhead = PACKED_K ? 1 : 2;         // an iteration needs the offsets of the tile this far on
    if constexpr (!PACKED_V) {
#pragma unroll
        for (int ti = 0; ti <= kAhead; ++ti) copy_tokens(ti);
        {
            int t = tok_q;
            asm volatile("" : "+v"(t));
        }
        wait_vmcnt<0>();                             // (the rows' own tokens are waited for in any case, and nothing else is under way)
        next_offsets(0);
    }

    bf16x8 qf[NH][KS];
    {
        const uint16_t* qp = q + (int64_t(tok_q) * n_q_heads + hq0) * D + 8 * hg;
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int j = 0; j < KS; ++j) qf[h][j] = *reinterpret_cast<const bf16x8*>(qp + h * D + 16 * j);
    }
    // copy order (tile x lives in buffer x % STAGES):
    //   three buffers: K0 | V0 K1 K2 V1 | K3 V2 | K4 V3 | ...   K two tiles ahead, V one
    //   two buffers:   K0 | V0 K1       | V1 K2 | V2 K3 | ...   one tile ahead
    issue_k(0, 0);
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            u32x4 t = __builtin_bit_cast(u32x4, qf[h][j]);
            asm volatile("" : "+v"(t));
            qf[h][j] = __builtin_bit_cast(bf16x8, t);
        }
    keep_offsets();
    issue_v(0, 0);
    if constexpr (!PACKED_K) next_offsets(1);
    issue_k(1, 1);
    keep_offsets();
    if (STAGES == 3) {
        issue_k(2, 2);
        issue_v(1, 1);
    }

    // The queries times scale * log2(e), rounded to bf16 once: scores in base-2 exponent units straight out of the matrix pipe.
    // Rotated ones (ROPE) take the factor with (cos, sin); two elements at a time, as they lie in a register (one by one the
    // rotation was a sixth of all vector instructions on sequences of a few hundred tokens: 96 of 60 to 900 tokens 493 -> 487 us, with
    // what the loop says of neg_ref below).
    auto element = [](uint32_t word, int e) { return __builtin_bit_cast(float, e == 0 ? word << 16 : word & 0xffff0000u); };
    auto rounded = [](float lo, float hi) {
        bf16x2 r;
        r[0] = (__bf16)lo;
        r[1] = (__bf16)hi;
        return __builtin_bit_cast(uint32_t, r);
    };
    if (ROPE) {
        const f32x4* tab4 = reinterpret_cast<const f32x4*>(rope_tab);
#pragma unroll
        for (int j = 0; j < KS / 2; ++j) {
            f32x4 cs4[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) cs4[w] = tab4[rope_table_at<D>(size_t(it.tile_a0) * kTileN + my_row, j, w, hg)] * scale_log2;
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                u32x4 lo = __builtin_bit_cast(u32x4, qf[h][j]), hi = __builtin_bit_cast(u32x4, qf[h][j + KS / 2]);
#pragma unroll
                for (int w = 0; w < 4; ++w) {                         // pairs 2 w and 2 w + 1
                    const float x0 = element(lo[w], 0), x1 = element(lo[w], 1), y0 = element(hi[w], 0), y1 = element(hi[w], 1);
                    const f32x4 r = cs4[w];
                    lo[w] = rounded(x0 * r[0] - y0 * r[1], x1 * r[2] - y1 * r[3]);
                    hi[w] = rounded(y0 * r[0] + x0 * r[1], y1 * r[2] + x1 * r[3]);
                }
                qf[h][j] = __builtin_bit_cast(bf16x8, lo);
                qf[h][j + KS / 2] = __builtin_bit_cast(bf16x8, hi);
            }
        }
    } else {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                u32x4 x = __builtin_bit_cast(u32x4, qf[h][j]);
#pragma unroll
                for (int w = 0; w < 4; ++w) x[w] = rounded(element(x[w], 0) * scale_log2, element(x[w], 1) * scale_log2);
                qf[h][j] = __builtin_bit_cast(bf16x8, x);
            }
    }

    f32x16 o_acc[NH][DB];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) o_acc[h][db][i] = 0.f;
    // Softmax state of a row, per head, in base-2 exponent units: m_ref is the reference exponent, l_run the sum of
    // the probabilities 2^(s - m_ref) so far (this lane's half of the row).
    float l_run[NH], m_ref[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        l_run[h] = 0.f;
        m_ref[h] = 0.f;
    }

    int koff[KS];
    {
        const int xk = swizzle_key<2 * D>(n) ^ hg;
#pragma unroll
        for (int j = 0; j < KS; ++j) koff[j] = n * D + ((2 * j) ^ xk) * 8;
    }
    // V^T operands: columns of a row tile, or (packed) rows of a V^T tile
    const TrOffsets<D> v_cols(lane);
    int voff[4];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) voff[qd] = n * kTileN + ((2 * qd) ^ swizzle_key<2 * kTileN>(n) ^ hg) * 8;
    {
        int t0 = my_vis, t1 = tok_q;
        asm volatile("" : "+v"(t0), "+v"(t1));
    }
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            u32x4 t = __builtin_bit_cast(u32x4, qf[h][j]);
            asm volatile("" : "+v"(t));
            qf[h][j] = __builtin_bit_cast(bf16x8, t);
        }

    // K fragment f of a tile: key block f % SB, k-step f / SB; V^T fragment f: d block f % DB, 16-key step f / DB
    auto ld_k = [&](const uint16_t* kb, int f) { return *reinterpret_cast<const bf16x8*>(kb + 32 * (f % SB) * D + koff[f / SB]); };
    auto ld_v = [&](const uint16_t* vb, int f) {
        if constexpr (PACKED_V) return *reinterpret_cast<const bf16x8*>(vb + 32 * (f % DB) * kTileN + voff[f / DB]);
        else return v_cols.fragment(vb, f / DB, f % DB);
    };

    struct TileInfo { bool partial; int room; };          // room: columns the row sees from this lane's first one of the tile on
    auto tile_info = [&](int ti) {
        const bool in_a = ti < it.a_total;
        const int kt = in_a ? ti : ti - it.a_total;
        const bool partial = kt >= (in_a ? it.a_full : it.b_full) || (kt + 1) * kTileN > (in_a ? it.n_stream : it.n_src);
        return TileInfo{partial, (in_a ? my_row + 1 : my_vis) - (kt * kTileN + 8 * hg)};
    };
    auto max_with_partner = [&](float x) {
        float a = x, b = x;
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
        return fmaxf(a, b);
    };
    auto rescale_acc = [&](int h, float alpha) {
        if constexpr (NH == 2) {
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float x = o_acc[h][db][i], tmp;
                    asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                                 : "+a"(x), "=&v"(tmp) : "v"(alpha));
                    o_acc[h][db][i] = x;
                }
            asm volatile("s_nop 7" ::: "memory");
        } else {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o_acc[h][db][i] *= alpha;
        }
    };
    // the columns of a partial tile that a row may not see: exponent -inf, probability 0
    // lane (n, hg), block sb, register i  <->  key column kt*64 + 32 sb + 16 (i/8) + 8 hg + i%8
    auto mask_tile = [&](f32x16 (&sv)[NH][SB], const TileInfo& ti) {
        uint32_t seen[SB];                               // bit i: register i of the block
        const uint32_t none = 0xff800000u;               // -inf
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
            seen[sb] = ((1u << min(max(ti.room - 32 * sb, 0), 8)) - 1u) | ((1u << min(max(ti.room - 32 * sb - 16, 0), 8)) - 1u) << 8;
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    // (by bits: a compare and the select that reads it have to be kept apart by a wait state)
                    const uint32_t keep = uint32_t(__builtin_amdgcn_sbfe(int(seen[sb]), i, 1));
                    const float x = sv[h][sb][i];
                    sv[h][sb][i] = __builtin_bit_cast(float, (keep & __builtin_bit_cast(uint32_t, x)) | (~keep & none));
                }
    };
    // row maximum (both lanes of the row) of a tile's exponents
    auto row_max = [&](const f32x16 (&blk)[SB]) {
        float mx = -INFINITY;
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, blk[sb][i]);
        return max_with_partner(mx);
    };

    // ---- prologue: tile 0 gives every row its reference exponent ----
    // sv: the exponents of the tile whose probabilities are formed next; s_next: the score blocks the matrix pipe is
    // filling.  The first matrix instruction of every score block starts from -m_ref, so a score leaves the pipe as
    // s - m_ref.
    //   NH = 1  neg_ref holds -m_ref for good; the scores are copied, two per instruction, beside the matrix instructions of
    //           phase Y, which has no other vector work (4 x 4K tokens 273 -> 271.7 us: the chip's power is the limit there).
    //   NH = 2  s_next lives in accumulation registers; between two tiles its LAST block holds -m_ref in all its 16 registers and
    //           starts in place.
    f32x16 sv[NH][SB], s_next[NH][SB], neg_ref;
    wait_vmcnt<(STAGES == 3 ? 4 : 2) * NL>();            // K0 has landed
    __syncthreads();
    {
        const uint16_t* kb = &sm.k[0][0];
        const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < SB * KS; ++f) {
            const bf16x8 a = ld_k(kb, f);
#pragma unroll
            for (int h = 0; h < NH; ++h)
                sv[h][f % SB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[h][f / SB], f / SB == 0 ? zero16 : sv[h][f % SB], 0, 0, 0);
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float x = sv[h][sb][i];
                    asm volatile("" : "+v"(x));                   // in vector registers from here on
                    sv[h][sb][i] = x;
                }
        const TileInfo t0 = tile_info(0);
        if (t0.partial) mask_tile(sv, t0);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            m_ref[h] = row_max(sv[h]);                            // finite: column 0 is visible to every row
#pragma unroll
            for (int sb = 0; sb < SB; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) sv[h][sb][i] -= m_ref[h];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if constexpr (NH == 2) s_next[h][SB - 1][i] = -m_ref[h];
                else neg_ref[i] = -m_ref[h];
            }
        }
    }

    u32x4 pw[NH][SB][2];                                 // probabilities of the current tile (bf16 pairs), as the second product's operand
    float psum[NH];
    // slot m of NH SB KS: PER elements of the probabilities of the tile in sv, in the order (head, block, register)
    // (the two-head form sums the probabilities as the second product will see them, rounded to bf16, two per
    // instruction: one vector instruction less per pair, +0.8 % there; the one-head form measured 1 % slower with it
    // and keeps its fp32 adds)
    bf16x2 ones2;
    ones2[0] = (__bf16)1.f;
    ones2[1] = (__bf16)1.f;
    static_assert(PER % 2 == 0, "probabilities are formed in pairs");
    auto exp_slot = [&](int m) {
#pragma unroll
        for (int u = 0; u < PER; u += 2) {
            const int e = m * PER + u;
            const int hh = e / (SB * 16), sb2 = (e / 16) % SB, i = e % 16;
            const float pr0 = __builtin_amdgcn_exp2f(sv[hh][sb2][i]), pr1 = __builtin_amdgcn_exp2f(sv[hh][sb2][i + 1]);
            bf16x2 p2;
            p2[0] = (__bf16)pr0;
            p2[1] = (__bf16)pr1;
            if constexpr (NH == 2) psum[hh] = __builtin_amdgcn_fdot2_f32_bf16(p2, ones2, psum[hh], false);
            else psum[hh] += pr0 + pr1;
            uint32_t word = __builtin_bit_cast(uint32_t, p2);
            if constexpr (NH == 1) asm volatile("" : "+v"(word));   // HERE, not behind the check of the row sums (NH = 2: 3 % slower)
            pw[hh][sb2][i >> 3][(i & 7) / 2] = word;
        }
    };
    // A row sum beyond 2^kRiseLog2 (or not finite) means the tile's exponents outgrew the reference: move it to the
    // tile's row maximum, form the tile's probabilities again, rescale what has been accumulated.  Scores already in
    // flight relative to the old reference still have `late` to lose when they arrive.
    float late[NH];
    auto check_rise = [&]() {
        bool trig = false;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            asm volatile("" : "+v"(psum[h]));
            late[h] = 0.f;
            trig = trig || !(psum[h] <= __builtin_exp2f(kRiseLog2));
        }
        const bool any = __any(trig);
        if (any) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const float rise = row_max(sv[h]);
                const float shift = rise > 0.f ? rise : 0.f;           // (-inf: the row sees nothing in this tile)
                const float alpha = __builtin_amdgcn_exp2f(-shift);
                late[h] = shift;
                psum[h] = 0.f;
#pragma unroll
                for (int sb = 0; sb < SB; ++sb)
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        const float pr0 = __builtin_amdgcn_exp2f(sv[h][sb][i] - shift), pr1 = __builtin_amdgcn_exp2f(sv[h][sb][i + 1] - shift);
                        psum[h] += pr0;
                        psum[h] += pr1;
                        pw[h][sb][i >> 3][(i & 7) / 2] = rounded(pr0, pr1);
                    }
                l_run[h] *= alpha;
                rescale_acc(h, alpha);
                m_ref[h] += shift;
            }
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) l_run[h] += psum[h];
        return any;
    };

    int stage = 0;                                       // buffer of tile ti
    bf16x8 kpre[kPF], vpre[kPF];                         // first fragments of a phase, read during the phase before
    // every tile but the last: the loop body has no branch around its matrix instructions
    for (int ti = 0; ti + 1 < n_tiles; ++ti) {
        // three buffers: K(ti+2) and V^T(ti) have landed (V^T(ti+1) is in flight behind them); two: K(ti+1), V^T(ti);
        // everybody is done with K(ti) and V^T(ti-1), whose buffers the next copies go to
        wait_vmcnt<(STAGES == 3 ? 1 : 0) * NL>();
        __syncthreads();
        const int stage1 = stage == STAGES - 1 ? 0 : stage + 1;
        const int stage2 = stage1 == STAGES - 1 ? 0 : stage1 + 1;
        if constexpr (!PACKED_V) next_offsets(ti + kAhead);
        // The copies of this round, behind the first matrix instructions.  NH = 2: K, then V^T, one copy each -- the four waves are here
        // together, and with four in one place they wait for one another's (8 x 16K tokens, attention alone 11.01 -> 10.91 ms; the whole step
        // moves by 1 %, no more than its runs differ).  NH = 1: the tokens, then V
        // and K, all of a tile at once (one by one: the same on 4 x 4K tokens, 2 % slower with heads of 64).
        auto copies = [&](int i) {
            if constexpr (NH == 2) {
                if (i < NL) async_copy_1k(k_head + size_t(tile_of(ti + 3)) * TILE, lane_off, lds_k0 + stage * (TILE * 2), i);
                else async_copy_1k(v_head + size_t(tile_of(ti + 2)) * TILE, lane_off, lds_v0 + (stage == 0 ? 2 : stage - 1) * (TILE * 2), i - NL);
            } else if (i == 0) {
                if constexpr (!PACKED_V) copy_tokens(ti + kAhead + 1);
                issue_v(ti + 1, stage1);
            } else {
                issue_k(ti + 2, stage);
            }
        };
        const uint16_t* kb = &sm.k[0][0] + stage1 * TILE;
        const uint16_t* vb = &sm.v[0][0] + stage * TILE;
        const uint16_t* kb2 = &sm.k[0][0] + stage2 * TILE;        // K(ti+2): the tile of the next round's phase X
        if (!EARLY_K || ti == 0) {
#pragma unroll
            for (int f = 0; f < kPF; ++f) kpre[f] = ld_k(kb, f);
        }

        // ---- phase X: scores of tile ti+1  |  probabilities of tile ti ----
#pragma unroll
        for (int h = 0; h < NH; ++h) psum[h] = 0.f;
        {
            constexpr int NF = SB * KS;
            bf16x8 a[NF];
#pragma unroll
            for (int f = 0; f < kPF; ++f) a[f] = kpre[f];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (f + kPF < NF) a[f + kPF] = ld_k(kb, f + kPF);
                else vpre[f + kPF - NF] = ld_v(vb, f + kPF - NF);     // the first V^T fragments of phase Y
                const int sb = f % SB, j = f / SB;
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    // k-step 0 starts from -m_ref
                    s_next[h][sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[f], qf[h][j], j > 0 ? s_next[h][sb] : NH == 2 ? s_next[h][SB - 1] : neg_ref, 0, 0, 0);
                    // the copies of this round go out behind the first matrix instructions
                    if (f * NH + h < (NH == 2 ? 2 * NL : 2)) copies(f * NH + h);
                    exp_slot(f * NH + h);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        const bool moved = check_rise();

        // ---- phase Y: O^T += V^T P^T of tile ti  |  the exponents of tile ti+1 leave the registers of the scores ----
        // slot m of NH DB SB 2: PER fresh exponents, in the order (block, head, register); the last block is left
        // holding -m_ref for the next round
        float neg[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) neg[h] = -m_ref[h];
        auto move_slot = [&](int m) {
#pragma unroll
            for (int u = 0; u < PER; u += 2) {
                const int e = m * PER + u;
                const int sb2 = e / (NH * 16), hh = (e / 16) % NH, i = e % 16;
                // ONE move per register, HERE (a plain copy would be sunk to its use, into the crowded phase X); the producing
                // matrix instruction retired at least two (NH = 1) or three of them ago
                if constexpr (NH == 2) {
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        float x;
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(s_next[hh][sb2][i + w]));
                        sv[hh][sb2][i + w] = x;
                        if (sb2 == SB - 1) {
                            float t;
                            asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(t) : "v"(neg[hh]));
                            s_next[hh][sb2][i + w] = t;
                        }
                    }
                } else {
                    f32x2 x;
                    asm volatile("v_mov_b64 %0, %1" : "=v"(x) : "v"(f32x2{s_next[hh][sb2][i], s_next[hh][sb2][i + 1]}));
                    sv[hh][sb2][i] = x[0];
                    sv[hh][sb2][i + 1] = x[1];
                }
            }
        };
        {
            constexpr int NF = DB * SB * 2;
            bf16x8 a[NF];
#pragma unroll
            for (int f = 0; f < kPF; ++f) a[f] = vpre[f];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (f + kPF < NF) a[f + kPF] = ld_v(vb, f + kPF);
                else if (EARLY_K) kpre[f + kPF - NF] = ld_k(kb2, f + kPF - NF);   // the first K fragments of the next round
                const int db = f % DB, st = f / DB;              // keys 16 st .. 16 st + 15
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    o_acc[h][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[f], __builtin_bit_cast(bf16x8, pw[h][st >> 1][st & 1]), o_acc[h][db], 0, 0, 0);
                    if (NH == 1 && f == 0) __builtin_amdgcn_sched_barrier(0);        // (two matrix instructions behind the last one of block 0)
                    move_slot(f * NH + h);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (moved) {
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int sb = 0; sb < SB; ++sb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) sv[h][sb][i] -= late[h];
            if constexpr (NH == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) neg_ref[i] = -m_ref[0];
            }
        }
        if constexpr (!PACKED_V) keep_offsets();
        const TileInfo fresh = tile_info(ti + 1);
        if (fresh.partial) mask_tile(sv, fresh);
        stage = stage1;
    }
    // ---- the last tile: its probabilities and the second product, no scores behind it ----
    {
        wait_vmcnt<0>();                                 // (also: no copy into LDS may outlive the workgroup)
        __syncthreads();
        const uint16_t* vb = &sm.v[0][0] + stage * TILE;
        constexpr int NF = DB * SB * 2;
        bf16x8 a[NF];
#pragma unroll
        for (int f = 0; f < kPF; ++f) a[f] = ld_v(vb, f);
#pragma unroll
        for (int h = 0; h < NH; ++h) psum[h] = 0.f;
#pragma unroll
        for (int m = 0; m < NH * SB * KS; ++m) exp_slot(m);
        check_rise();
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f + kPF < NF) a[f + kPF] = ld_v(vb, f + kPF);
            const int db = f % DB, st = f / DB;
#pragma unroll
            for (int h = 0; h < NH; ++h)
                o_acc[h][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[f], __builtin_bit_cast(bf16x8, pw[h][st >> 1][st & 1]), o_acc[h][db], 0, 0, 0);
        }
    }

#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const float l_tot = l_run[h] + __shfl_xor(l_run[h], 32);   // wave-wide exchange: inactive rows take part
        const float inv = 1.f / l_tot;
        uint16_t* op = out + (int64_t(tok_q) * n_q_heads + hq0 + h) * D;
        // lane (n, hg), block db, register i  <->  d = 32 db + 8 (i/4) + 4 hg + i%4: the two lanes of a row hold four dims each of
        // every eight.  One exchange of 32-lane rows per word pair (the upper half of an even group's words against the lower
        // half of the odd group's) leaves lane hg with all eight of group 2 g + hg: half as many stores, 16 bytes each
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                u32x2 lo, hi;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    bf16x2 a, b;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        a[e] = (__bf16)(o_acc[h][db][8 * g + 2 * c + e] * inv);
                        b[e] = (__bf16)(o_acc[h][db][8 * g + 4 + 2 * c + e] * inv);
                    }
                    lo[c] = __builtin_bit_cast(uint32_t, a);
                    hi[c] = __builtin_bit_cast(uint32_t, b);
                    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(lo[c]), "+v"(hi[c]));
                }
                if (active) *reinterpret_cast<u32x4*>(op + 32 * db + 16 * g + 8 * hg) = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        if (lse && active && hg == 0) lse[int64_t(tok_q) * n_q_heads + hq0 + h] = (m_ref[h] + __builtin_amdgcn_logf(l_tot)) * kLn2;
    }
}


}  // namespace st

using namespace st;

// packed K and V^T tiles (not every form uses them), then the (cos, sin) table of the fused rotation (one float2 per packed row and pair)
static size_t prefill_tile_bytes(const st_plan* plan, int n_kv_heads, int head_dim) {
    return 2 * size_t(n_kv_heads) * size_t(plan->pack_tiles) * kTileN * size_t(head_dim) * sizeof(uint16_t);
}
static size_t prefill_ws_bytes(const st_plan* plan, int n_kv_heads, int head_dim, st_dtype dt) {
    if (dt != ST_BF16) return 0;                     // the fp32 path reads q / k / v in place
    return prefill_tile_bytes(plan, n_kv_heads, head_dim) + size_t(plan->pack_tiles) * kTileN * size_t(head_dim / 2) * sizeof(float2);
}

extern "C" size_t st_prefill_workspace_bytes(const st_plan* plan, int32_t n_kv_heads, int32_t head_dim, st_dtype dt) {
    if (!plan || n_kv_heads <= 0 || head_dim <= 0) return 0;
    return prefill_ws_bytes(plan, n_kv_heads, head_dim, dt);
}

// positions == nullptr: rotated q / k (st_attn_prefill); otherwise unrotated, rotated here (st_attn_prefill_rope)
static st_status prefill_impl(void* out, float* lse, const void* q, const void* k, const void* v, const int32_t* positions,
                              double theta_base, const st_plan* plan, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                              float scale, st_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!out || !q || !k || !v || !plan) return fail(ST_ERR_INVALID_ARG, "st_attn_prefill: null pointer");
    if (!aligned16(out) || !aligned16(q) || !aligned16(k) || !aligned16(v))
        return fail(ST_ERR_INVALID_ARG, "st_attn_prefill: tensors must be 16-byte aligned");
    if (n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0)
        return fail(ST_ERR_SHAPE, "st_attn_prefill: n_q_heads %d must be a positive multiple of n_kv_heads %d", n_q_heads, n_kv_heads);
    if (head_dim != 64 && head_dim != 128) return fail(ST_ERR_UNSUPPORTED, "st_attn_prefill: head_dim %d (64 or 128)", head_dim);
    if (dt != ST_F32 && dt != ST_BF16) return fail(ST_ERR_UNSUPPORTED, "st_attn_prefill: dtype %d", int(dt));
    if (plan->n_tokens == 0) return ST_OK;
    if (plan->n_tokens * int64_t(n_q_heads) * head_dim >= (int64_t(1) << 31))
        return fail(ST_ERR_SHAPE, "st_attn_prefill: n_tokens * n_q_heads * head_dim must stay below 2^31 elements");
    const size_t need = prefill_ws_bytes(plan, n_kv_heads, head_dim, dt);
    if (need > 0) {
        if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
            return fail(ST_ERR_INVALID_ARG, "st_attn_prefill: workspace must be non-null and 256-byte aligned");
        if (workspace_bytes < need)
            return fail(ST_ERR_CAPACITY, "st_attn_prefill: workspace has %zu bytes, needs %zu", workspace_bytes, need);
    }
    if (scale <= 0.f) scale = 1.f / sqrtf(float(head_dim));
    const int64_t blocks = int64_t(plan->m_max) * n_q_heads;
    const int64_t pack_blocks = int64_t(plan->pack_tiles) * n_kv_heads;
    if (blocks > 0x7fffffff || pack_blocks > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_prefill: grid too large");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    ST_HIP(plan->wait_built(s));
    const PlanView pv = plan->view();
    if (dt == ST_F32)
        return launch_prefill_f32(static_cast<float*>(out), lse, static_cast<const float*>(q), static_cast<const float*>(k),
                                  static_cast<const float*>(v), pv, n_q_heads, n_kv_heads, head_dim, scale, s);
    const size_t tile_bytes = prefill_tile_bytes(plan, n_kv_heads, head_dim);
    uint16_t* kc = static_cast<uint16_t*>(workspace);
    uint16_t* vc = kc + tile_bytes / (2 * sizeof(uint16_t));
    float2* tab = reinterpret_cast<float2*>(static_cast<char*>(workspace) + tile_bytes);
    const bool rope = positions != nullptr;
    const RopeFreq freq = rope ? make_rope_freq(theta_base, head_dim) : RopeFreq{};
    const float scale_log2 = scale * kLog2e;
    // Two query heads per workgroup when heads come in pairs over a KV head and the sequences are long (an item then
    // walks a hundred key tiles and more, and the halved LDS / L2 traffic per flop pays); short sequences finish
    // sooner with twice as many, lighter workgroups, two per compute unit.
    const int heads_wanted = plan->heads_per_workgroup;
    const bool can_pair = (n_q_heads / n_kv_heads) % 2 == 0;
    const bool pair = can_pair && (heads_wanted == 2 || (heads_wanted == 0 && plan->n_tokens / plan->batch >= 8192));
    // Packed tiles also for one head where the sequences are long enough that a tile's many copies and reads outweigh the pass over memory: the
    // gathered rows of V cost their transposing reads.  Gathered against packed, batches of 2K / 4K / 8K tokens a sequence, four head
    // geometries: rotated keys (packed in any case) 0.94 to 0.98 / 0.99 to 1.01 / 1.00 to 1.03 of the time (heads of 64 dims 1.00); plain 0.74 to
    // 0.92 / 0.90 to 0.99 / 0.97 to 0.99, and 1.02 with eight query heads over a KV head of 128 dims.
    // Packed always where a result lies over K or V: workgroups still gather rows that others have written over.
    const int64_t mean_tokens = plan->n_tokens / plan->batch;
    const size_t rows = size_t(plan->n_tokens), q_bytes = rows * n_q_heads * head_dim * 2, kv_bytes = rows * n_kv_heads * head_dim * 2;
    auto written_over = [&](const void* kv) {
        return overlap(out, q_bytes, kv, kv_bytes) || (lse && overlap(lse, rows * n_q_heads * sizeof(float), kv, kv_bytes));
    };
    const bool packed = pair || written_over(k) || written_over(v) || !gather_fits(plan->n_tokens, n_kv_heads, head_dim) ||
                        (head_dim == 128 && mean_tokens >= (rope ? 3500 : n_q_heads / n_kv_heads >= 8 ? 5000 : INT64_MAX));
    // The four waves of a workgroup share the key tiles of one KV head; they take 4, 2 or 1 (sets of) query heads of it and
    // 32, 64 or 128 rows of the item -- as many heads as the group has: fewer rows end closer to their item's last visible
    // column, so less of the issued arithmetic is masked or belongs to no row (useful share 0.89 / 0.93 / 0.95 with 1 / 2 / 4
    // heads on 4 x 4K tokens, 0.52 / 0.68 / 0.74 on 96 sequences of 60 to 900), at the same copy traffic per product.
    // Whole steps, us: 8 x 6K to 8K tokens, 32 / 8 heads 2820 -> 2770; 4 x 4K, 16 / 8 307 -> 300; 96 short 660 -> 638.
    const int sets = n_q_heads / n_kv_heads / (pair ? 2 : 1);
    const int head_waves = sets % 4 == 0 ? 4 : sets % 2 == 0 ? 2 : 1;
    auto launch = [&](auto dtag) -> st_status {
        constexpr int HD = decltype(dtag)::value;
        const bool packs = rope || packed;             // (else the attention kernel takes its rows from the tensors)
        prof_begin(kProfTilePack, s);                  // (a reading per call, of nothing where nothing is packed)
        for (int rep = 0; packs && rep < prof_repeat(); ++rep) {
        if (rope) {
            hipLaunchKernelGGL((rope_table_kernel<HD>), dim3((unsigned)plan->pack_tiles), dim3(256), 0, s, tab, positions, pv, freq);
            // Four heads per workgroup where that still leaves four workgroups for every compute unit, else one: a small batch would only wait
            // for one head behind the other (96 sequences of 60 to 900 tokens, 8 KV heads of 128 dims: 57.7 us one by one, 46 by twos, 42.6 by
            // fours, 42.3 by eights).
            const int heads = pack_blocks >= 4 * 1024 ? 4 : 1;
            hipLaunchKernelGGL((key_pack_rope_kernel<HD>), dim3((unsigned)(plan->pack_tiles * ((n_kv_heads + heads - 1) / heads))), dim3(256), 0, s, kc,
                               (const float2*)tab, (const uint16_t*)k, pv, n_kv_heads, heads);
        }
        if (packed)
            hipLaunchKernelGGL((tile_pack_kernel<HD>), dim3((unsigned)pack_blocks, rope ? 1 : 2), dim3(256), 0, s, vc, (const uint16_t*)v, kc,
                               (const uint16_t*)k, pv, n_kv_heads);
        }
        prof_end(kProfTilePack, s);
        auto run = [&](auto nh_tag, auto rope_tag, auto pack_tag) -> st_status {
            constexpr int NH = decltype(nh_tag)::value;
            constexpr bool ROPE = decltype(rope_tag)::value, PACK = decltype(pack_tag)::value;
            const size_t smem = sizeof(PipeSmem<HD, NH == 2 ? 3 : 2>);
            auto* kern = &prefill_attn_kernel<HD, NH, ROPE, PACK>;
            ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem)));
            prof_begin(kProfPrefillAttn, s);
            for (int rep = 0; rep < prof_repeat(); ++rep)
                hipLaunchKernelGGL(kern, dim3((unsigned)(blocks / (NH * head_waves) * item_parts(pv, head_waves))), dim3(256), smem, s, (uint16_t*)out,
                                   lse, (const uint16_t*)q, rope || packed ? kc : (const uint16_t*)k, packed ? vc : (const uint16_t*)v, pv, n_q_heads, n_kv_heads, scale_log2, (const float2*)tab, head_waves);
            prof_end(kProfPrefillAttn, s);
            return ST_OK;
        };
        auto heads_of = [&](auto rope_tag) -> st_status {
            if (pair) return run(std::integral_constant<int, 2>{}, rope_tag, std::true_type{});
            return packed ? run(std::integral_constant<int, 1>{}, rope_tag, std::true_type{}) : run(std::integral_constant<int, 1>{}, rope_tag, std::false_type{});
        };
        return rope ? heads_of(std::true_type{}) : heads_of(std::false_type{});
    };
    const st_status lr = head_dim == 64 ? launch(std::integral_constant<int, 64>{}) : launch(std::integral_constant<int, 128>{});
    if (lr != ST_OK) return lr;
    ST_LAUNCH_CHECK("key_pack_rope_kernel / prefill_attn_kernel");
    return ST_OK;
}

extern "C" st_status st_attn_prefill(void* out, float* lse, const void* q, const void* k, const void* v,
                                     const st_plan* plan, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                     float scale, st_dtype dt, void* workspace, size_t workspace_bytes,
                                     void* hip_stream) {
    return prefill_impl(out, lse, q, k, v, nullptr, 0.0, plan, n_q_heads, n_kv_heads, head_dim, scale, dt, workspace, workspace_bytes,
                        hip_stream);
}

extern "C" st_status st_attn_prefill_rope(void* out, float* lse, const void* q, const void* k, const void* v,
                                          const int32_t* positions, double theta_base, const st_plan* plan, int32_t n_q_heads,
                                          int32_t n_kv_heads, int32_t head_dim, float scale, st_dtype dt, void* workspace,
                                          size_t workspace_bytes, void* hip_stream) {
    if (!positions) return fail(ST_ERR_INVALID_ARG, "st_attn_prefill_rope: positions is null");
    if (!(theta_base > 0.0)) return fail(ST_ERR_INVALID_ARG, "st_attn_prefill_rope: theta_base must be positive");
    if (dt != ST_BF16) return fail(ST_ERR_UNSUPPORTED, "st_attn_prefill_rope: bf16 only (dtype %d); rotate fp32 inputs with st_rope_apply", int(dt));
    return prefill_impl(out, lse, q, k, v, positions, theta_base, plan, n_q_heads, n_kv_heads, head_dim, scale, dt, workspace,
                        workspace_bytes, hip_stream);
}

extern "C" st_status st_attn_prefill_ids(void* out, float* lse, const void* q, const void* k, const void* v,
                                         const int32_t* segment_ids, const int32_t* stream_ids,
                                         const int32_t* positions, const int32_t* cu_seqlens_host, int32_t batch,
                                         int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, float scale,
                                         st_dtype dt, void* hip_stream) {
    st_plan* plan = nullptr;
    st_status r = st_plan_create(&plan, segment_ids, stream_ids, positions, cu_seqlens_host, batch, nullptr, 0, 1, hip_stream);
    if (r != ST_OK) return r;
    void* ws = nullptr;
    const size_t ws_bytes = (n_kv_heads > 0 && head_dim > 0) ? prefill_ws_bytes(plan, n_kv_heads, head_dim, dt) : 0;
    if (ws_bytes > 0) {
        hipError_t e = hipMalloc(&ws, ws_bytes);
        if (e != hipSuccess) {
            st_plan_destroy(plan);
            return fail(ST_ERR_RUNTIME, "st_attn_prefill_ids: hipMalloc(%zu) failed: %s", ws_bytes, hipGetErrorString(e));
        }
    }
    r = st_attn_prefill(out, lse, q, k, v, plan, n_q_heads, n_kv_heads, head_dim, scale, dt, ws, ws_bytes, hip_stream);
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(hip_stream));
    if (ws) (void)hipFree(ws);
    st_plan_destroy(plan);
    if (r == ST_OK && e != hipSuccess) return fail(ST_ERR_RUNTIME, "st_attn_prefill_ids: %s", hipGetErrorString(e));
    return r;
}
