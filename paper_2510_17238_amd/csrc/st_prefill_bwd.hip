// Backward of the streaming-mask prefill attention (streaming-constrained training, Sec. 3.2: the mask
// of Eq. 2 is part of the forward pass of supervised fine-tuning, so only visible pairs carry gradient).
//
// With P = softmax over the visible keys (recomputed from the forward's log-sum-exp), delta_i = dO_i . O_i:
//     dV_j = sum_i P_ij dO_i      dP_ij = dO_i . V_j      dS_ij = P_ij (dP_ij - delta_i)
//     dQ_i = scale sum_j dS_ij K_j                       dK_j = scale sum_i dS_ij Q_i
// The forward's segment tables drive it: query rows walk the forward's work items (tiles past `total` are
// never read); key rows find the queries that see them from the same tables read the other way round --
// a source key c is seen by source rows >= c and by the reasoning rows whose visible-source count exceeds
// c (a suffix of the reasoning stream, found by bisection), a reasoning key by reasoning rows >= c.
// bf16 here; fp32 tensors take the kernels of st_attn_f32.hip.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "st_tiles.h"

namespace st {

// --------------------------------------------------------------------------
// MFMA path (bf16).
// --------------------------------------------------------------------------
// dQ: the forward's loop over the key tiles of a query tile (same work items, same transposed products, a lane
// owns one query row), with three products per key tile:
//   S^T  = K  Q^T     (K row tile from LDS, Q^T in registers)        -> P^T = exp2(S^T scale - lse)
//   dP^T = V  dO^T    (V row tile from LDS, dO^T in registers)       -> dS^T = P^T (dP^T - delta)
//   dQ^T += K^T dS^T  (K^T read out of the same K row tile with transposing LDS reads; dS^T from the accumulators,
//                      rounded to bf16)
// The kernel fits 256 registers, so TWO workgroups share a CU (two waves per SIMD fill each other's gaps between
// matrix and vector work); the K and V row tiles are double-buffered and copied one tile ahead (64 KB of LDS per
// workgroup, and 4 KB of tokens), one barrier per key tile.
// The rows of all tiles, here and on the key side, are gathered from the tensors on their way into LDS (RowGather): a pass that packed
// row tiles and row statistics before took 87 to 100 us of a training step over 4 x 4K tokens, 16 / 8 heads of 128 dims (whole step
// 1,167 -> 1,075 us with the statistics formed here), 32 of 347 over 10 x 1.7K, 16 / 2 of 64.
template <int D>
struct BwdDqSmem {
    uint16_t k[2][kTileN * D];        // K rows
    uint16_t v[2][kTileN * D];        // V rows
    unsigned char tokens[RowGather<D>::kBytes];
};

// delta of a row, half of it per lane (hg): dims 8 hg + 16 j .. + 7; the two halves are then added.  (One order of the sum for all that form it.)
template <int KS>
__device__ __forceinline__ float half_delta(const bf16x8 (&d_out)[KS], const uint16_t* out) {
    float x = 0.f;
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        const bf16x8 o = *reinterpret_cast<const bf16x8_a2*>(out + 16 * j);
#pragma unroll
        for (int e = 0; e < 8; ++e) x = fmaf(float(d_out[j][e]), float(o[e]), x);
    }
    return x;
}

// GATHER: k and v are the tensors, delta is formed from `out`; else k and v are packed row tiles, and delta has been formed with them.
template <int D, bool GATHER>
__global__ __launch_bounds__(256, 2) void bwd_dq_mfma_kernel(uint16_t* __restrict__ dq, const uint16_t* __restrict__ d_out,
                                                             const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                             const uint16_t* __restrict__ v, const uint16_t* __restrict__ out,
                                                             const float* __restrict__ delta, const float* __restrict__ lse,
                                                             float* __restrict__ stats, PlanView pv, int n_q_heads, int n_kv_heads,
                                                             float scale, int head_waves) {
    constexpr int KS = D / 16, DB = D / 32, SB = kTileN / 32;
    constexpr int TILE = kTileN * D;
    constexpr int NL = TILE * 2 / 1024 / 4;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    BwdDqSmem<D>& sm = *reinterpret_cast<BwdDqSmem<D>*>(smem_raw);

    // workgroup -> (work item, part of its rows, set of head_waves query heads of one KV head), as in the forward
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_sets = n_q_heads / head_waves;
    const int row_parts = item_parts(pv, head_waves);
    const int rank = blockIdx.x / (n_sets * row_parts);
    const int rem = blockIdx.x % (n_sets * row_parts);
    const int hh0 = rem % n_sets, sub = row_parts - 1 - rem / n_sets;              // (later rows have the longer loops: first)
    const int group = n_q_heads / n_kv_heads;
    const int hk = hh0 % n_kv_heads;
    const int hq = hk * group + head_waves * (hh0 / n_kv_heads) + wave % head_waves;
    WorkItem it = pv.sorted[rank];
    if (head_waves > 1) it = item_part(it, pv, sub, kTileM / head_waves);
    if (it.n_rows <= 0) return;
    const int n = lane & 31, hg = lane >> 5;
    const int n_tiles = it.a_total + it.b_total;

    const uint16_t* k_head = GATHER ? k + hk * D : k + size_t(hk) * pv.pack_tiles * TILE;
    const uint16_t* v_head = GATHER ? v + hk * D : v + size_t(hk) * pv.pack_tiles * TILE;
    const uint32_t wave_off = uint32_t(wave) * (NL * 1024), lane_off = wave_off + uint32_t(lane) * 16u;
    const RowGather<D> rows(sm.tokens, wave, lane, uint32_t(n_kv_heads) * (2 * D));
    auto tile_of = [&](int ti) {
        ti = min(ti, n_tiles - 1);
        return ti < it.a_total ? it.tile_a0 + ti : it.tile_b0 + (ti - it.a_total);
    };
    auto copy_tokens = [&](int ti) {
        const int t = min(ti, n_tiles - 1);
        const bool in_a = t < it.a_total;
        rows.copy_tokens(pv.perm + (in_a ? it.a_base : it.b_base), (in_a ? t : t - it.a_total) * kTileN, (in_a ? it.n_stream : it.n_src) - 1, ti);
    };
    const uint32_t lds_k = uint32_t(uintptr_t(&sm.k[0][0])) + wave_off, lds_v = uint32_t(uintptr_t(&sm.v[0][0])) + wave_off;
    uint32_t row_off[NL];                                       // (gathered rows) of the tile that is copied
    // copy c of tile ti, NL of K and NL of V
    auto issue = [&](int ti, int buf, int c) {
        const uint16_t* head = c < NL ? k_head : v_head;
        const uint32_t lds = (c < NL ? lds_k : lds_v) + buf * (TILE * 2);
        if constexpr (GATHER) RowGather<D>::copy_one(RowGather<D>::base(head), row_off, lds, c % NL);
        else async_copy_1k(head + size_t(tile_of(ti)) * TILE, lane_off, lds, c % NL);
    };

    const int row_in_tile = (wave / head_waves) * 32 + n;
    const bool active = row_in_tile < it.n_rows;
    const int my_row = it.row0 + min(row_in_tile, it.n_rows - 1);
    const int tok_q = pv.perm[it.a_base + my_row];
    const int my_vis = pv.vis[it.a_base + my_row];
    if constexpr (GATHER) {
        copy_tokens(0);
        int t = tok_q;
        asm volatile("" : "+v"(t));
        wait_vmcnt<0>();             // (the rows' own tokens are waited for in any case, and nothing else is under way)
        rows.offsets(row_off, 0);
        copy_tokens(1);
    }
#pragma unroll
    for (int c = 0; c < 2 * NL; ++c) issue(0, 0, c);
    const int64_t rowhead = int64_t(tok_q) * n_q_heads + hq;
    const float lse2 = lse[rowhead] * kLog2e;
    const float scale_log2 = scale * kLog2e;

    bf16x8 qf[KS], dof[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        qf[j] = *reinterpret_cast<const bf16x8_a2*>(q + rowhead * D + 8 * hg + 16 * j);
        dof[j] = *reinterpret_cast<const bf16x8_a2*>(d_out + rowhead * D + 8 * hg + 16 * j);
    }
    // delta of the row; what the key side needs of it -- for every 64-row tile of a stream and every query head one 1 KB block of 256 floats:
    // [0, 64) MINUS lse in base-2 units (-inf for rows past the end of the stream: their probabilities become 0), [64, 128) MINUS
    // delta, [128, 192) the visible-source count of the row (as int bits) -- comes from here, where dO is at hand.
    float my_delta;
    if constexpr (GATHER) {
        my_delta = half_delta<KS>(dof, out + rowhead * D + 8 * hg);
        my_delta += __shfl_xor(my_delta, 32);
    } else {
        my_delta = delta[rowhead];
    }
    {
        auto put_stats = [&](int row, float neg_lse, float neg_delta, int vis) {
            float* blk = stats + (size_t(hq) * pv.pack_tiles + it.tile_a0 + row / kTileN) * 256 + row % kTileN;
            blk[0] = neg_lse;
            blk[64] = neg_delta;
            blk[128] = __int_as_float(vis);
        };
        if (active && hg == 0) put_stats(my_row, -lse2, -my_delta, my_vis);
        // the wave that holds the stream's last row fills the rest of its tile
        const int last = it.n_stream - 1 - it.row0, row = it.n_stream + lane;
        if (last >= (wave / head_waves) * 32 && last < (wave / head_waves) * 32 + 32 && row < (it.n_stream + kTileN - 1) / kTileN * kTileN) put_stats(row, -INFINITY, 0.f, 0);
    }
    // queries times scale * log2(e), rounded to bf16 again (as in the forward kernel): K q' is a score in exponent units
#pragma unroll
    for (int j = 0; j < KS; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[j][e] = (__bf16)(float(qf[j][e]) * scale_log2);
    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;

    // byte of the lane's piece of k-step 0 in a row tile; step j's lies at that XOR 32 j, formed on the tile's LDS address (the tiles begin at
    // multiples of 256 bytes)
    const uint32_t piece0 = uint32_t(n * D + (swizzle_key<2 * D>(n) ^ hg) * 8) * 2u;
    const TrOffsets<D> tr(lane);
    // Score and dP blocks of a tile.  A lane owns one query row, so what has to be taken off every score (the row's
    // log-sum-exp) and off every dP (the row's delta) is one number per lane: between tiles the LAST block of each
    // kind holds it, negated, in all sixteen registers, and the first matrix instruction of every block takes that as
    // its accumulator input (the last block in place, after the others have read it).
    f32x16 s_acc[SB], dp_acc[SB];
    const float neg_lse2 = -lse2, neg_delta = -my_delta;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        asm volatile("v_mov_b32 %0, %1" : "=v"(s_acc[SB - 1][i]) : "v"(neg_lse2));
        asm volatile("v_mov_b32 %0, %1" : "=v"(dp_acc[SB - 1][i]) : "v"(neg_delta));
    }

    for (int ti = 0; ti < n_tiles; ++ti) {
        const int buf = ti & 1;
        wait_vmcnt<0>();                 // the row tiles of ti have landed; everybody is done with tile ti - 1
        __syncthreads();
        if constexpr (GATHER) rows.tokens(row_off, ti + 1);       // (past the end: the last tile again, never used)
        const bool in_a = ti < it.a_total;
        const int kt = in_a ? ti : ti - it.a_total;
        const bool partial = kt >= (in_a ? it.a_full : it.b_full) || (kt + 1) * kTileN > (in_a ? it.n_stream : it.n_src);
        const int limit = in_a ? my_row + 1 : my_vis;

        // The tile's two 32-key halves are staggered, so that the vector work of one runs beside matrix work of the other:
        //     matrix pipe:  S, dP of half 0 | S, dP of half 1 | dQ of half 0    | dQ of half 1
        //     vector ALU :                  | dS of half 0    | dS of half 1    | start values
        // Matrix instructions in pairs: 2 KS of (S, dP), then DB * SB of dQ.  A pair's operands leave LDS two pairs ahead, one copy of the next
        // tile stands behind every pair from the second on.
        // (Groups of eight instructions, all dS between the two products, eight copies in one place: 325 us against 312 on 4 x 4K tokens, 16 / 8
        // heads of 128 dims, 92 against 87 on 10 x 1.7K, 16 / 2 of 64; the other wave of the SIMD already filled most of those gaps.)
        typedef bf16x8 lds_bf16x8 __attribute__((address_space(3)));
        const uint32_t k0 = uint32_t(uintptr_t(&sm.k[0][0])) + buf * (TILE * 2) + piece0, dv = uint32_t(uintptr_t(&sm.v[0][0])) - uint32_t(uintptr_t(&sm.k[0][0]));
        const uint16_t* kb = &sm.k[buf][0];
        constexpr int NS = SB * KS, NG = DB * SB, RING = 3;
        bf16x8 f0[RING], f1[RING];
        auto request = [&](int p) {
            if (p < NS) {
                const uint32_t at = (k0 ^ uint32_t(32 * (p % KS))) + 64u * (p / KS) * D;
                f0[p % RING] = *(const lds_bf16x8*)(at);
                f1[p % RING] = *(const lds_bf16x8*)(at + dv);
            } else if (p < NS + NG) {
                const int e = 2 * (p - NS);                       // K^T fragments e and e + 1: d block e % DB, 16-key step e / DB
                f0[p % RING] = tr.fragment(kb, e / DB, e % DB);
                f1[p % RING] = tr.fragment(kb, (e + 1) / DB, (e + 1) % DB);
            }
        };
        u32x4 dsb[SB][2];
        // lane (n, hg), block sb, register i  <->  key column kt*64 + 32 sb + 16 (i/8) + 8 hg + i%8
        auto mask = [&](int sb) {
            const int c0 = kt * kTileN + 8 * hg + 32 * sb;
#pragma unroll
            for (int i = 0; i < 16; ++i) s_acc[sb][i] = c0 + 16 * (i >> 3) + (i & 7) < limit ? s_acc[sb][i] : -INFINITY;
        };
        auto soft = [&](int sb, int piece, int pieces) {         // dS of 16 / pieces registers
#pragma unroll
            for (int i = piece * 16 / pieces; i < (piece + 1) * 16 / pieces; i += 2) {
                bf16x2 ds;
                ds[0] = (__bf16)(__builtin_amdgcn_exp2f(s_acc[sb][i]) * dp_acc[sb][i]);
                ds[1] = (__bf16)(__builtin_amdgcn_exp2f(s_acc[sb][i + 1]) * dp_acc[sb][i + 1]);
                uint32_t w = __builtin_bit_cast(uint32_t, ds);
                asm volatile("" : "+v"(w));                      // HERE, not in front of its use
                dsb[sb][i >> 3][(i & 7) / 2] = w;
            }
        };
        request(0);
        request(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            const int sb = p / KS, j = p % KS;
            s_acc[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f0[p % RING], qf[j], j == 0 ? s_acc[SB - 1] : s_acc[sb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            request(p + 2);
            __builtin_amdgcn_sched_barrier(0);
            dp_acc[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[p % RING], dof[j], j == 0 ? dp_acc[SB - 1] : dp_acc[sb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (GATHER && p == 0) rows.form(row_off);
            if (p > 0 && p <= 2 * NL) issue(ti + 1, buf ^ 1, p - 1);
            if (sb == 1) soft(0, j, KS);
            __builtin_amdgcn_sched_barrier(0);
            // (uniform) only the tiles on the edge of what the rows may see
            if (j == KS - 1 && partial) mask(sb);
        }
        static_assert(2 * NL < NS, "a pair for every copy");
#pragma unroll
        for (int p = 0; p < NG; ++p) {
            const int e = 2 * p, slot = (NS + p) % RING, half = p / (NG / 2);
            acc[e % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f0[slot], __builtin_bit_cast(bf16x8, dsb[half][(e / DB) & 1]), acc[e % DB], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            request(NS + p + 2);
            __builtin_amdgcn_sched_barrier(0);
            acc[(e + 1) % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[slot], __builtin_bit_cast(bf16x8, dsb[half][((e + 1) / DB) & 1]), acc[(e + 1) % DB], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (half == 0) {
                soft(1, p, NG / 2);
            } else {
                // the start values again (written as instructions: left to the compiler, the two constant blocks become thirty-two more live registers)
#pragma unroll
                for (int i = (p - NG / 2) * 32 / NG; i < (p - NG / 2 + 1) * 32 / NG; ++i) {
                    asm volatile("v_mov_b32 %0, %1" : "=v"(s_acc[SB - 1][i]) : "v"(neg_lse2));
                    asm volatile("v_mov_b32 %0, %1" : "=v"(dp_acc[SB - 1][i]) : "v"(neg_delta));
                }
            }
            if (GATHER && p == 0) copy_tokens(ti + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    wait_vmcnt<0>();
    if (!active) return;
    uint16_t* op = dq + rowhead * D;
    // lane (n, hg), block db, register i  <->  d = 32 db + 8 (i/4) + 4 hg + i%4
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            bf16x4 o4;
#pragma unroll
            for (int c = 0; c < 4; ++c) o4[c] = (__bf16)(acc[db][4 * q4 + c] * scale);
            *reinterpret_cast<bf16x4_a2*>(op + 32 * db + 8 * q4 + 4 * hg) = o4;
        }
}


// Row tiles of dO, Q, K and V, and delta, for tensors that are not aligned to 16 bytes (a gradient may be a slice of a flat buffer): the
// asynchronous copies of the gradient kernels take aligned pieces; and for gradients that are written over an input, which would be
// gathered after that.  All is read in one pass before anything is written.  A workgroup takes one tile of one head of one
// tensor, the heads of all four side by side: 0 .. n_q_heads - 1 dO and delta, then Q, then K, then V.
struct BwdPackArgs {
    const uint16_t *d_out, *q, *k, *v, *out;
    uint16_t *dorows, *qrows, *krows, *vrows;
    float* delta;
    int n_q_heads, n_kv_heads;
};
template <int D>
__global__ __launch_bounds__(256) void bwd_pack_kernel(BwdPackArgs a, PlanView pv) {
    const int n_slots = 2 * (a.n_q_heads + a.n_kv_heads);
    const int tile = int(blockIdx.x) / n_slots;
    int h = int(blockIdx.x) % n_slots;
    const TileInfo info = pv.tiles[tile];
    if (info.valid == 0) return;                    // spare tile of a sequence: never read
    const bool query_side = h < 2 * a.n_q_heads;
    if (!query_side) h -= 2 * a.n_q_heads;
    const int heads = query_side ? a.n_q_heads : a.n_kv_heads;
    const bool second = h >= heads;                 // Q or V
    if (second) h -= heads;
    uint16_t* dst = query_side ? (second ? a.qrows : a.dorows) : second ? a.vrows : a.krows;
    const uint16_t* src = query_side ? (second ? a.q : a.d_out) : second ? a.v : a.k;
    pack_rows<D>(dst + (size_t(h) * pv.pack_tiles + tile) * (kTileN * D), src, pv.perm + info.base, info.valid, uint32_t(heads) * D, uint32_t(h),
                 [](int, uint32_t, const u32x4&) {});
    if (!query_side || second) return;
    // delta: two lanes per row
    const int row = int(threadIdx.x) >> 1, hg = int(threadIdx.x) & 1;
    if (row >= info.valid) return;
    const int64_t rowhead = int64_t(pv.perm[info.base + row]) * a.n_q_heads + h;
    bf16x8 x[D / 16];
#pragma unroll
    for (int j = 0; j < D / 16; ++j) x[j] = *reinterpret_cast<const bf16x8_a2*>(a.d_out + rowhead * D + 8 * hg + 16 * j);
    float dl = half_delta<D / 16>(x, a.out + rowhead * D + 8 * hg);
    dl += __shfl_xor(dl, 1);
    if (hg == 0) a.delta[rowhead] = dl;
}

// dK, dV: one workgroup per (128 keys of one stream of one sequence, KV head) -- the forward's work items read
// as KEYS -- 4 waves x 32 keys, a lane owns one key.  It loops over the 64-row query tiles that can see its keys
// (own stream: tiles from the one holding its first key on; for source keys also the reasoning tiles from the
// first row whose visible-source count exceeds its first key on), for every query head of its group:
//   S   = Q  K^T    (Q row tile from LDS, K^T in registers)      -> P  = exp2(S scale - lse_row)
//   dP  = dO V^T    (dO row tile from LDS, V^T in registers)     -> dS = P (dP - delta_row)
//   dV^T += dO^T P  (dO^T out of the dO row tile with transposing LDS reads, P from the accumulators, rounded to bf16)
//   dK^T += Q^T dS  (Q^T out of the Q row tile likewise, dS from the accumulators)
// Rows run along the accumulator registers here, so lse / delta / visible count of the rows come from the
// tile's 1 KB statistics block (written by the query side) in LDS.  Three buffers per tile kind (103 KB), one barrier per query tile.
// acc += A B with the accumulator in ACCUMULATION registers, whatever form the compiler gives the file's other matrix
// instructions: the key-side kernel's two output accumulators (128 registers) live there for the whole kernel, the
// score and dP blocks in vector registers where the exponentials read them -- no copies between the two files.
__device__ __forceinline__ void mfma_into_agprs(f32x16& acc, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

template <int D>
struct BwdDkvSmem {
    uint16_t qr[3][kTileN * D];       // Q rows
    uint16_t dor[3][kTileN * D];      // dO rows
    float stats[3][256];
    unsigned char tokens[RowGather<D>::kBytes];
};

// parts > 1: the query heads of a KV head are dealt out to `parts` workgroups (a divisor of the group), which leave fp32
// sums in `partial` ([2: dK, dV][parts][N][n_kv_heads][D]) for bwd_dkv_sum_kernel instead of writing dk / dv -- see dkv_parts.
// GATHER: qrows and dorows are the tensors, else their packed row tiles.
template <int D, bool GATHER>
__global__ __launch_bounds__(256, 1) void bwd_dkv_mfma_kernel(uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                              const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                              const uint16_t* __restrict__ qrows, const uint16_t* __restrict__ dorows,
                                                              const float* __restrict__ stats, PlanView pv, int n_q_heads,
                                                              int n_kv_heads, float scale, int parts, float* __restrict__ partial,
                                                              int64_t partial_stride) {
    constexpr int KS = D / 16, DB = D / 32, SB = kTileN / 32;
    constexpr int TILE = kTileN * D;
    constexpr int NL = TILE * 2 / 1024 / 4;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    BwdDkvSmem<D>& sm = *reinterpret_cast<BwdDkvSmem<D>*>(smem_raw);

    // The table is sorted by the FORWARD's cost (late rows first); a key's cost runs the other way (early keys
    // are seen by the most rows), so walk the table backwards: longest first again, unused slots at once.
    const int per_item = n_kv_heads * parts;
    const int rank = pv.m_max - 1 - int(blockIdx.x / per_item);
    const int hk = blockIdx.x % n_kv_heads;
    const int part = int(blockIdx.x % per_item) / n_kv_heads;
    const int group = n_q_heads / n_kv_heads / parts;           // query heads of this workgroup: hq0 .. hq0 + group - 1
    const int hq0 = (hk * parts + part) * group;
    const WorkItem it = pv.sorted[rank];
    if (it.n_rows == 0) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, hg = lane >> 5;
    const bool key_is_src = it.kind == ST_SOURCE;
    const int S = it.n_src;
    const int n_rsn = key_is_src ? (pv.cu[it.seq + 1] - pv.cu[it.seq] - S) : it.n_stream;

    // query tiles that can see keys >= row0: run A over the own stream, run B (source keys) over the reasoning stream
    const int a_first = it.row0 / kTileN, a_end = (it.n_stream + kTileN - 1) / kTileN;
    int b_first = 0, b_end = 0;
    if (key_is_src) {
        // first reasoning row whose visible count exceeds row0 (counts do not decrease along the stream), searched by
        // the whole wave: every lane tests the end of one 64th of the range, so the range shrinks 64-fold per memory
        // round trip (three for a few thousand rows, where a bisection takes a dozen)
        int lo = 0, hi = n_rsn;                                 // the answer lies in [lo, hi]; hi == n_rsn: no such row
        const int32_t* vr = pv.vis + it.b_base + S;
        while (lo < hi) {
            const int span = hi - lo, step = (span + 63) >> 6;
            const int last = min(span - 1, lane * step + step - 1);             // end of this lane's piece
            const unsigned long long seen = __ballot(vr[lo + last] > it.row0);  // (monotone along the lanes)
            if (seen == 0ull) {
                lo = hi;
            } else {
                const int first = __ffsll((long long)seen) - 1;
                hi = lo + min(span - 1, first * step + step - 1);               // this row exceeds row0 ...
                lo = lo + first * step;                                         // ... and none before this piece does
            }
            lo = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
        }
        b_first = lo / kTileN;
        b_end = (n_rsn + kTileN - 1) / kTileN;
        if (lo >= n_rsn) b_first = b_end;
    }
    const int n_a = a_end - a_first, n_b = b_end - b_first;
    const int n_iter = (n_a + n_b) * group;
    const int tile_own0 = it.tile_a0;                           // packed tile of row 0 of the own stream
    const int tile_rsn0 = it.tile_b0 + (S + kTileN - 1) / kTileN;   // ... of the reasoning stream (source keys)

    const int key_in_tile = wave * 32 + n;
    const int wave_last_key = it.row0 + min(__builtin_amdgcn_readfirstlane(wave) * 32 + 31, it.n_rows - 1);
    const bool active = key_in_tile < it.n_rows;
    const int my_key = it.row0 + min(key_in_tile, it.n_rows - 1);
    const int tok_k = pv.perm[it.a_base + my_key];
    const int64_t keyhead = int64_t(tok_k) * n_kv_heads + hk;
    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        kf[j] = *reinterpret_cast<const bf16x8_a2*>(k + keyhead * D + 8 * hg + 16 * j);
        vf[j] = *reinterpret_cast<const bf16x8_a2*>(v + keyhead * D + 8 * hg + 16 * j);
    }
    // keys times scale * log2(e), rounded to bf16 again: Q k' is a score in exponent units (dK takes Q, not K)
#pragma unroll
    for (int j = 0; j < KS; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) kf[j][e] = (__bf16)(float(kf[j][e]) * (scale * kLog2e));
#pragma unroll
    for (int j = 0; j < KS; ++j) {                              // landed before the loop (it counts its own copies)
        u32x4 t = __builtin_bit_cast(u32x4, kf[j]), u = __builtin_bit_cast(u32x4, vf[j]);
        asm volatile("" : "+v"(t), "+v"(u));
        kf[j] = __builtin_bit_cast(bf16x8, t);
        vf[j] = __builtin_bit_cast(bf16x8, u);
    }

    // iteration -> (query tile, head): heads fastest, so that a tile's row statistics change slowest; tiles from the LAST one
    // down (reasoning tiles, then the own stream's) -- every key block of a sequence then starts at the same query tile, and
    // the blocks that start together read the same tiles at about the same time (a quarter less traffic into L2)
    struct Iter { int tile; int hq; int row0; bool rs; int step; };      // (step: query tiles walked before this one)
    auto iter_at = [&](int t, int g) {                          // (tile count t of the walk, head g of the group)
        Iter r;
        r.hq = hq0 + g;
        r.step = n_a + n_b - 1 - t;
        if (t < n_a) {
            r.tile = tile_own0 + a_first + t;
            r.row0 = (a_first + t) * kTileN;
            r.rs = false;
        } else {
            r.tile = tile_rsn0 + b_first + (t - n_a);
            r.row0 = (b_first + (t - n_a)) * kTileN;
            r.rs = true;
        }
        return r;
    };
    const uint32_t wave_off = uint32_t(__builtin_amdgcn_readfirstlane(wave)) * (NL * 1024);
    const uint32_t lds_qr = uint32_t(uintptr_t(&sm.qr[0][0])) + wave_off, lds_dor = uint32_t(uintptr_t(&sm.dor[0][0])) + wave_off,
                   lds_st = uint32_t(uintptr_t(&sm.stats[0][0]));
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    // the copies of one iteration, NL of Q and NL of dO (the statistics with the first): the loop issues them one by one from the shadows of
    // its first matrix instructions
    const uint32_t lane_off = uint32_t(lane) * 16u;
    const RowGather<D> rows(sm.tokens, wave_u, lane, uint32_t(n_q_heads) * (2 * D));
    uint32_t row_off[NL];                                       // (gathered rows) of the next iteration's tile
    auto copy_tokens = [&](const Iter& r) {
        rows.copy_tokens(pv.perm + (r.rs ? it.b_base + S : it.a_base), r.row0, (r.rs ? n_rsn : it.n_stream) - 1, r.step);
    };
    auto issue = [&](const Iter& r, int buf, int c) {
        const uint16_t* tensor = c < NL ? qrows : dorows;
        const uint32_t lds = (c < NL ? lds_qr : lds_dor) + buf * (TILE * 2);
        if (c == 0 && wave_u == 0) async_copy16(stats + (size_t(r.hq) * pv.pack_tiles + r.tile) * 256 + lane * 4, lds_st + buf * 1024);
        if constexpr (GATHER) RowGather<D>::copy_one(RowGather<D>::base(tensor + r.hq * D), row_off, lds, c % NL);
        else async_copy_1k(tensor + (size_t(r.hq) * pv.pack_tiles + r.tile) * TILE + size_t(wave_u * NL) * 512, lane_off, lds, c % NL);
    };
    // the walk, two iterations ahead of the arithmetic (no division in the loop: it is stepped)
    int t_copy = n_a + n_b - 1, g_copy = 0;
    auto step_copy = [&]() {
        if (++g_copy == group) {
            g_copy = 0;
            --t_copy;
        }
    };
    if (GATHER && n_iter > 0) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
            if (t < n_a + n_b) copy_tokens(iter_at(n_a + n_b - 1 - t, 0));
        wait_vmcnt<0>();
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
        if (x < n_iter) {
            const Iter r = iter_at(t_copy, g_copy);
            if (GATHER && g_copy == 0) rows.offsets(row_off, r.step);
#pragma unroll
            for (int c = 0; c < 2 * NL; ++c) issue(r, x, c);
            step_copy();
        }

    f32x16 dk_acc[DB], dv_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            dk_acc[db][i] = 0.f;
            dv_acc[db][i] = 0.f;
        }
    // byte of the lane's piece of k-step 0 in a row tile; step j's lies at that XOR 32 j, formed on the tile's LDS address (the tiles begin at
    // multiples of 256 bytes), so that one register stays instead of one per step
    const uint32_t piece0 = uint32_t(n * D + (swizzle_key<2 * D>(n) ^ hg) * 8) * 2u;
    const TrOffsets<D> tr(lane);

    // Operands come out of LDS a group of matrix instructions ahead of their use (one wave per SIMD: nobody else hides that latency), one
    // fragment of either tensor behind every pair of instructions.  A tile's two 32-row halves are staggered so that the vector work of one
    // half runs beside matrix work of the other:
    //     matrix pipe:  S, dP of half 0 | S, dP of half 1     | dV, dK of half 0    | dV, dK of half 1
    //     vector ALU :                  | P, dS of half 0     | P, dS of half 1     |
    // and the first fragments and start values of a tile are read beside the last block of the tile before it: three buffers, so that it has
    // landed by then.  One piece of each kind of work behind every instruction, no branch between them: 4,580 -> 3,690 cycles per tile of
    // 64 rows and head of 128 dims (2,048 of the matrix pipe), against fragments and copies a group at a time, the first ones behind the
    // barrier where all four waves asked for them at once (550 cycles), and a branch per piece of vector work for the masks.  4 x 4K tokens,
    // 16 / 8 heads: 555 -> 500 us (the chip's clock gives back half of it); 10 x 1.7K, 16 / 2 of 64: 133 -> 126.  The copies still cost 270
    // cycles: without them 480 us.
    static_assert(SB == 2 && (DB == 4 || DB == 2) && KS == 2 * DB, "the stagger below is written for 64-row tiles of 64 or 128 dims");
    constexpr int G = DB;                                    // pairs of matrix instructions per group, two groups per block
    constexpr int PIECES = 4 / G;                            // (two score pairs per piece: eight per half beside 2 G pairs of instructions)
    f32x16 s_acc[SB], dp_acc[SB];
    bf16x8 fq[2][G], fo[2][G];
    u32x4 pb[SB][2], dsb[SB][2];                             // P and dS, bf16 pairs
    typedef bf16x8 lds_bf16x8 __attribute__((address_space(3)));
    typedef f32x4 lds_f32x4 __attribute__((address_space(3)));
    const uint32_t lds_q = uint32_t(uintptr_t(&sm.qr[0][0])), lds_o = uint32_t(uintptr_t(&sm.dor[0][0]));
    // Q and dO rows of half rb, k-step G g + u
    auto load1 = [&](int buf, int rb, int g, int u, int slot) {
        const uint32_t at = ((lds_q + buf * (TILE * 2) + piece0) ^ uint32_t(32 * (G * g + u))) + 64u * rb * D;
        fq[slot][u] = *(const lds_bf16x8*)(at);
        fo[slot][u] = *(const lds_bf16x8*)(at + (lds_o - lds_q));
    };
    // lane (n, hg), block rb, register i  <->  query row cur.row0 + 32 rb + 16 (i/8) + 8 hg + i%8, key my_key.
    // The accumulators start at minus the rows' log-sum-exp (scores) and minus their delta (dP), straight from the
    // tile's statistics block: what comes out is the exponent of P and dP - delta.  Piece c, 0 .. 7: four registers of either.
    auto start_values = [&](int buf, int rb, int c) {
        const int q4 = c >> 1;
        const f32x4 x = *(const lds_f32x4*)(lds_st + buf * 1024 + 4 * (32 * rb + 16 * (q4 >> 1) + 8 * hg + 4 * (q4 & 1)) + 256 * (c & 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) (c & 1 ? dp_acc : s_acc)[rb][4 * q4 + e] = x[e];
    };
    auto start_values_beside = [&](int buf, int rb, int i) {         // over the 2 G pairs of a block
#pragma unroll
        for (int c = 0; c < PIECES; ++c) start_values(buf, rb, i * PIECES + c);
    };
    // P and dS of half rb, the part that goes beside pair i
    auto soft = [&](int rb, int i) {
#pragma unroll
        for (int k = 0; k < PIECES; ++k) {
            const int e = 2 * (i * PIECES + k);
            const float p0 = __builtin_amdgcn_exp2f(s_acc[rb][e]), p1 = __builtin_amdgcn_exp2f(s_acc[rb][e + 1]);
            bf16x2 p, ds;
            p[0] = (__bf16)p0;
            p[1] = (__bf16)p1;
            ds[0] = (__bf16)(p0 * dp_acc[rb][e]);
            ds[1] = (__bf16)(p1 * dp_acc[rb][e + 1]);
            uint32_t wp = __builtin_bit_cast(uint32_t, p), wds = __builtin_bit_cast(uint32_t, ds);
            asm volatile("" : "+v"(wp), "+v"(wds));          // HERE, not in front of their use
            pb[rb][e >> 3][(e & 7) / 2] = wp;
            dsb[rb][e >> 3][(e & 7) / 2] = wds;
        }
    };

    int t_cur = n_a + n_b - 1, g_cur = 0;
    int buf = 0;
    if (n_iter > 0) {
        wait_vmcnt<0>();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < G; ++u) load1(0, 0, 0, u, 0);
#pragma unroll
        for (int c = 0; c < 8; ++c) start_values(0, 0, c);
    }
    for (int x = 0; x < n_iter; ++x) {
        wait_vmcnt<0>();                 // the tiles of iteration x + 1 have landed; everybody is done with x - 1
        __syncthreads();
        const Iter cur = iter_at(t_cur, g_cur);
        if (++g_cur == group) {
            g_cur = 0;
            --t_cur;
        }
        const Iter ahead = iter_at(max(t_copy, 0), g_copy);              // iteration x + 2 (past the end: some tile again, never used)
        const int buf1 = buf == 2 ? 0 : buf + 1, buf2 = buf1 == 2 ? 0 : buf1 + 1;
        if constexpr (GATHER) rows.tokens(row_off, ahead.step);
        const uint16_t* qb = &sm.qr[buf][0];
        const uint16_t* ob = &sm.dor[buf][0];
        const float* st = &sm.stats[buf][0];
        auto load2 = [&](int stp, int u, int slot) {         // dO^T and Q^T of rows 16 stp .. 16 stp + 15, d block u
            fo[slot][u] = tr.fragment(ob, stp, u);
            fq[slot][u] = tr.fragment(qb, stp, u);
        };
        // pairs of half rb that the rows do not see: exponent -inf
        auto mask = [&](int rb) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int r0 = 32 * rb + 16 * half + 8 * hg;           // first of the 8 consecutive rows of these registers
                int limit[8];                                          // keys of the stream that the rows see
                if (cur.rs) {
#pragma unroll
                    for (int q4 = 0; q4 < 2; ++q4) {
                        const f32x4 c2 = *reinterpret_cast<const f32x4*>(st + 128 + r0 + 4 * q4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) limit[4 * q4 + e] = __float_as_int(c2[e]);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) limit[e] = cur.row0 + r0 + e + 1;
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) s_acc[rb][8 * half + e] = limit[e] > my_key ? s_acc[rb][8 * half + e] : -INFINITY;
            }
        };
        // Blocks of 2 G pairs of matrix instructions: ahead(g, u) requests a fragment of the group after next behind a pair's first instruction,
        // beside(i) is the other work that goes with pair i
        auto scores = [&](int rb, auto request, auto beside) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    s_acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[g][u], kf[G * g + u], s_acc[rb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    request(g, u);
                    __builtin_amdgcn_sched_barrier(0);
                    dp_acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo[g][u], vf[G * g + u], dp_acc[rb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    beside(G * g + u);
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        auto grads = [&](int rb, auto request, auto beside) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    mfma_into_agprs(dv_acc[u], fo[g][u], __builtin_bit_cast(bf16x8, pb[rb][g]));
                    __builtin_amdgcn_sched_barrier(0);
                    request(g, u);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_into_agprs(dk_acc[u], fq[g][u], __builtin_bit_cast(bf16x8, dsb[rb][g]));
                    __builtin_amdgcn_sched_barrier(0);
                    beside(G * g + u);
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        // the copies of iteration x + 2, one behind every second pair of the two score blocks
        auto copies = [&](int i) {
            if (i % 2 == 1) issue(ahead, buf2, i / 2);
        };
        static_assert(2 * NL == 2 * G, "as many copies as every second pair of two blocks");
        scores(0, [&](int g, int u) { g == 0 ? load1(buf, 0, 1, u, 1) : load1(buf, 1, 0, u, 0); }, [&](int i) {
            if (GATHER && i == 1) rows.form(row_off);
            copies(i);
            start_values_beside(buf, 1, i);
        });
        // every row of the tile sees every key of this wave?  (rows are ordered, visible counts do not decrease)
        const int first_vis = __builtin_amdgcn_readfirstlane(__float_as_int(st[128]));
        const bool all_seen = cur.rs ? first_vis > wave_last_key : cur.row0 >= wave_last_key;
        // (uniform; only vector work is conditional: a branch around matrix instructions makes the compiler copy their accumulators)
        if (!all_seen) mask(0);
        scores(1, [&](int g, int u) { g == 0 ? load1(buf, 1, 1, u, 1) : load2(0, u, 0); }, [&](int i) {
            copies(2 * G + i);
            soft(0, i);
        });
        if (!all_seen) mask(1);
        grads(0, [&](int g, int u) { load2(g == 0 ? 1 : 2, u, g == 0 ? 1 : 0); }, [&](int i) { soft(1, i); });
        // (the tokens of the query tile after `ahead`'s: an iteration before its copies at the latest)
        if constexpr (GATHER) copy_tokens(iter_at(max(t_copy - 1, 0), 0));
        grads(1, [&](int g, int u) { g == 0 ? load2(3, u, 1) : load1(buf1, 0, 0, u, 0); }, [&](int i) { start_values_beside(buf1, 0, i); });
        step_copy();
        buf = buf1;
    }
    wait_vmcnt<0>();
    // (the matrix instructions above are written as text: the compiler does not know that their results need some
    // cycles before an ordinary instruction may read them)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    if (!active) return;
    const int64_t out_row = int64_t(pv.perm[it.a_base + my_key]) * n_kv_heads + hk;         // (keyhead: not kept in registers over the loop)
    if (parts > 1) {
        float* pk = partial + part * partial_stride + out_row * D + 4 * hg;
        float* pvv = pk + parts * partial_stride;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                *reinterpret_cast<f32x4*>(pk + 32 * db + 8 * q4) = f32x4{dk_acc[db][4 * q4], dk_acc[db][4 * q4 + 1], dk_acc[db][4 * q4 + 2], dk_acc[db][4 * q4 + 3]};
                *reinterpret_cast<f32x4*>(pvv + 32 * db + 8 * q4) = f32x4{dv_acc[db][4 * q4], dv_acc[db][4 * q4 + 1], dv_acc[db][4 * q4 + 2], dv_acc[db][4 * q4 + 3]};
            }
        return;
    }
    uint16_t* pk = dk + out_row * D;
    uint16_t* pvv = dv + out_row * D;
    // lane (n, hg), block db, register i  <->  d = 32 db + 8 (i/4) + 4 hg + i%4
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            bf16x4 a4, b4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                a4[c] = (__bf16)(dk_acc[db][4 * q4 + c] * scale);
                b4[c] = (__bf16)dv_acc[db][4 * q4 + c];
            }
            *reinterpret_cast<bf16x4_a2*>(pk + 32 * db + 8 * q4 + 4 * hg) = a4;
            *reinterpret_cast<bf16x4_a2*>(pvv + 32 * db + 8 * q4 + 4 * hg) = b4;
        }
}

// dK (blockIdx.y = 0) or dV (1) from the partial sums of the key-side kernel, in a fixed order; n8 groups of eight elements
__global__ __launch_bounds__(256) void bwd_dkv_sum_kernel(uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, const float* __restrict__ partial,
                                                          int64_t partial_stride, int parts, int n8, float scale) {
    const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
    if (i >= n8) return;
    const float* p = partial + blockIdx.y * parts * partial_stride + int64_t(i) * 8;
    f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
    for (int x = 1; x < parts; ++x) {
        a += *reinterpret_cast<const f32x4*>(p + x * partial_stride);
        b += *reinterpret_cast<const f32x4*>(p + x * partial_stride + 4);
    }
    const float f = blockIdx.y == 0 ? scale : 1.f;
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        r[e] = (__bf16)(a[e] * f);
        r[4 + e] = (__bf16)(b[e] * f);
    }
    *reinterpret_cast<bf16x8_a2*>((blockIdx.y == 0 ? dk : dv) + int64_t(i) * 8) = r;
}

}  // namespace st

using namespace st;

namespace {
inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }
// Workgroups per (128 keys, KV head) of the key-side kernel.  Its work items are KEYS: with few KV heads and many query heads
// over each, a small or a ragged batch leaves compute units idle and its few long workgroups end far apart.  The query heads of a
// group are then split into parts, each with a fp32 partial dK / dV of its own.  One more step of the split pays while the longest
// workgroup's walk (rows of the longest sequence times query heads) is longer than an even share of all rows (a workgroup walks
// half of its sequence's in the mean) plus what the further partial sums cost, 7 rows of a walk for a partial row: fitted to
// 270 shapes of twelve head geometries, even and ragged, where this is within 0.4 % of the best split in the mean and never loses
// more than 2 % to no split.  At 64 dims the share counts 1.1 times for 0.9: two workgroups sit on a compute unit, and one
// left alone there ends sooner.  Beyond two workgroups per slot of the chip nothing is split further, and nothing at all where the
// sequences have less than 512 tokens in the mean (the second launch: 17 x 150 tokens, whole step: 129 -> 143 us).
// us for the gradients, with 1 / 2 / 4 / 8 parts: 1 x 7.5K tokens, 16 / 8 heads of 128 dims 690 / 679; 3 x 2.4K 295 / 314; 8 x 760
// 148 / 186; 10 x 0.9K, 16 / 8 of 64 128 / 137; 4 x 3.1K, 16 / 2 of 128 953 / 615 / 547 / 571; 10 x 1.7K, 16 / 2 of 64
// 550 / 379 / 307 / 316; ragged: 6,000 and eight of 300 tokens, 8 / 4 of 128 498 / 359, 16 / 2 of 64 1000 / 580 / 384 / 305.
int dkv_parts(const st_plan* plan, int n_q_heads, int n_kv_heads, int head_dim) {
    const int group = n_q_heads / n_kv_heads;
    if (plan->n_tokens < int64_t(512) * plan->batch) return 1;
    const int64_t workgroups = (plan->n_tokens / kTileM + plan->batch) * n_kv_heads;
    const int64_t slots = 256 * (head_dim == 64 ? 2 : 1);
    const double share = plan->squared_tokens / (2 * kTileM) * n_q_heads / slots * (head_dim == 64 ? 1.1 : 0.9);
    const double partial_rows = double(plan->n_tokens) * n_kv_heads / slots;
    int parts = 1;
    for (int p = 2; p <= std::min(group, 8); ++p) {
        if (group % p != 0) continue;
        const double walk = double(plan->longest) * group / parts;
        if (workgroups * parts >= 2 * slots || walk <= share + 256 + 7 * (p - parts) * partial_rows) break;
        parts = p;
    }
    return parts;
}
// The same for the fp32 key side, whose workgroups own 32 keys and keep a compute unit to themselves: parts only while there is
// less than one workgroup per unit of the chip, at whatever length (a wave's chain of (row block, head) pairs is what a small
// problem takes).  Whole training steps: 3 x 100 to 200 tokens, 8 / 4 heads of 128 dims (80 workgroups) 110 -> 90 us; 4 x 60 to
// 120, 32 / 8 of 64 (152) 72 -> 64; but 2 x 900, 16 / 8 of 128 (480) 432 -> 438.
int dkv_parts_f32(const st_plan* plan, int n_q_heads, int n_kv_heads) {
    const int group = n_q_heads / n_kv_heads;
    const int64_t workgroups = (plan->n_tokens / 32 + 2 * int64_t(plan->batch)) * n_kv_heads;
    int parts = 1;
    for (int p = 2; p <= std::min(group, 8) && workgroups * parts < 256; ++p)
        if (group % p == 0) parts = p;
    return parts;
}
// workspace of the fp32 path: delta | partial dK, dV; of the bf16 path: delta (token order) | row statistics | K rows | V rows | Q rows | dO rows | partial dK, dV;
// delta and the four kinds of rows are those of the packed form alone: the size does not know the tensors' addresses
struct BwdLayout {
    size_t delta, stats, krows, vrows, qrows, dorows, partial, total;
    int parts;
    int64_t partial_stride;       // elements of one part
};
BwdLayout bwd_layout(const st_plan* plan, int n_q_heads, int n_kv_heads, int head_dim, st_dtype dt) {
    BwdLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += up256(bytes); return at; };
    L.delta = take(size_t(plan->n_tokens) * size_t(n_q_heads) * sizeof(float));
    if (dt == ST_BF16) {
        const size_t tile = size_t(kTileN) * head_dim * sizeof(uint16_t);
        const size_t kvt = size_t(n_kv_heads) * plan->pack_tiles * tile, qt = size_t(n_q_heads) * plan->pack_tiles * tile;
        L.stats = take(size_t(n_q_heads) * plan->pack_tiles * 256 * sizeof(float));
        L.krows = take(kvt);
        L.vrows = take(kvt);
        L.qrows = take(qt);
        L.dorows = take(qt);
    }
    L.parts = dt == ST_BF16 ? dkv_parts(plan, n_q_heads, n_kv_heads, head_dim) : dkv_parts_f32(plan, n_q_heads, n_kv_heads);
    L.partial_stride = plan->n_tokens * n_kv_heads * head_dim;
    if (L.parts > 1) L.partial = take(2 * size_t(L.parts) * size_t(L.partial_stride) * sizeof(float));
    L.total = off + 256;
    return L;
}
}  // namespace

extern "C" size_t st_prefill_bwd_workspace_bytes(const st_plan* plan, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                                 st_dtype dt) {
    if (!plan || n_q_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0) return 0;
    return bwd_layout(plan, n_q_heads, n_kv_heads, head_dim, dt).total;
}

extern "C" st_status st_attn_prefill_bwd(void* dq, void* dk, void* dv, const void* d_out, const void* q, const void* k,
                                         const void* v, const void* out, const float* lse, const st_plan* plan,
                                         int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, float scale, st_dtype dt,
                                         void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!dq || !dk || !dv || !d_out || !q || !k || !v || !out || !lse || !plan)
        return fail(ST_ERR_INVALID_ARG, "st_attn_prefill_bwd: null pointer");
    if (n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0)
        return fail(ST_ERR_SHAPE, "st_attn_prefill_bwd: n_q_heads %d must be a positive multiple of n_kv_heads %d", n_q_heads, n_kv_heads);
    if (head_dim != 64 && head_dim != 128) return fail(ST_ERR_UNSUPPORTED, "st_attn_prefill_bwd: head_dim %d (64 or 128)", head_dim);
    if (dt != ST_F32 && dt != ST_BF16) return fail(ST_ERR_UNSUPPORTED, "st_attn_prefill_bwd: dtype %d", int(dt));
    if (plan->n_tokens == 0) return ST_OK;
    if (plan->n_tokens * int64_t(n_q_heads) * head_dim >= (int64_t(1) << 31))
        return fail(ST_ERR_SHAPE, "st_attn_prefill_bwd: n_tokens * n_q_heads * head_dim must stay below 2^31 elements");
    const BwdLayout L = bwd_layout(plan, n_q_heads, n_kv_heads, head_dim, dt);
    const size_t need = L.total;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return fail(ST_ERR_INVALID_ARG, "st_attn_prefill_bwd: workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < need) return fail(ST_ERR_CAPACITY, "st_attn_prefill_bwd: workspace has %zu bytes, needs %zu", workspace_bytes, need);
    if (scale <= 0.f) scale = 1.f / sqrtf(float(head_dim));
    const int64_t qblocks = int64_t(plan->m_max) * n_q_heads, kblocks = int64_t(plan->m_max) * n_kv_heads;
    const int64_t pack_blocks = int64_t(plan->pack_tiles) * 2 * (n_q_heads + n_kv_heads);
    if (qblocks > 0x7fffffff || kblocks * 8 > 0x7fffffff || pack_blocks > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_prefill_bwd: grid too large");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    ST_HIP(plan->wait_built(s));
    const PlanView pv = plan->view();
    float* delta = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + L.delta);
    // bf16: two MFMA kernels over the rows of the tensors, or over packed row tiles (a tensor that is not aligned to 16 bytes, or of 4 GiB, or
    // that is written over by a gradient while or before its rows are read)
    auto run_mfma = [&](auto dtag, auto gtag) -> st_status {
        constexpr int HD = decltype(dtag)::value;
        constexpr bool GATHER = decltype(gtag)::value;
        unsigned char* w = static_cast<unsigned char*>(workspace);
        auto at = [&](size_t o) { return reinterpret_cast<uint16_t*>(w + o); };
        float* stats = reinterpret_cast<float*>(w + L.stats);
        float* partial = reinterpret_cast<float*>(w + L.partial);
        if (!GATHER) {
            const BwdPackArgs pack{(const uint16_t*)d_out, (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)out,
                                   at(L.dorows), at(L.qrows), at(L.krows), at(L.vrows), delta, n_q_heads, n_kv_heads};
            hipLaunchKernelGGL((bwd_pack_kernel<HD>), dim3((unsigned)pack_blocks), dim3(256), 0, s, pack, pv);
        }
        const size_t smem_q = sizeof(BwdDqSmem<HD>), smem_k = sizeof(BwdDkvSmem<HD>);
        ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_dq_mfma_kernel<HD, GATHER>), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem_q)));
        ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_dkv_mfma_kernel<HD, GATHER>), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem_k)));
        const int group = n_q_heads / n_kv_heads;
        // the waves take as many heads as the group has, as in the forward and for the same reason: fewer rows end closer to
        // their last visible column (training step, 4 x 4K tokens, 16 / 8 heads of 128 dims, 1195 -> 1181 us; 10 x 1.7K, 16 / 2
        // of 64, 369 -> 364)
        const int head_waves = group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
        prof_begin(kProfBwdDq, s);
        for (int rep = 0; rep < prof_repeat(); ++rep)
        hipLaunchKernelGGL((bwd_dq_mfma_kernel<HD, GATHER>), dim3((unsigned)(qblocks / head_waves * item_parts(pv, head_waves))), dim3(256), smem_q, s, (uint16_t*)dq, (const uint16_t*)d_out,
                           (const uint16_t*)q, GATHER ? (const uint16_t*)k : at(L.krows), GATHER ? (const uint16_t*)v : at(L.vrows), (const uint16_t*)out, delta, lse, stats, pv,
                           n_q_heads, n_kv_heads, scale, head_waves);
        prof_end(kProfBwdDq, s);
        prof_begin(kProfBwdDkv, s);
        for (int rep = 0; rep < prof_repeat(); ++rep)
        hipLaunchKernelGGL((bwd_dkv_mfma_kernel<HD, GATHER>), dim3((unsigned)(kblocks * L.parts)), dim3(256), smem_k, s, (uint16_t*)dk, (uint16_t*)dv,
                           (const uint16_t*)k, (const uint16_t*)v, GATHER ? (const uint16_t*)q : at(L.qrows), GATHER ? (const uint16_t*)d_out : at(L.dorows), stats, pv,
                           n_q_heads, n_kv_heads, scale, L.parts, partial, L.partial_stride);
        prof_end(kProfBwdDkv, s);
        if (L.parts > 1) {
            const int n8 = int(L.partial_stride / 8);
            hipLaunchKernelGGL(bwd_dkv_sum_kernel, dim3((unsigned)((n8 + 255) / 256), 2), dim3(256), 0, s, (uint16_t*)dk, (uint16_t*)dv, partial,
                               L.partial_stride, L.parts, n8, scale);
        }
        return ST_OK;
    };
    st_status r;
    if (dt == ST_F32)
        r = launch_bwd_f32(static_cast<float*>(dq), static_cast<float*>(dk), static_cast<float*>(dv), delta, static_cast<const float*>(d_out),
                           static_cast<const float*>(q), static_cast<const float*>(k), static_cast<const float*>(v), static_cast<const float*>(out), lse,
                           pv, n_q_heads, n_kv_heads, head_dim, scale, plan->n_tokens, L.parts,
                           reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + L.partial), s);
    else {
        auto run = [&](auto dtag) {
            // dq is written while K, V and the rows of `out` are read and before Q and dO are gathered, dk and dv while Q and dO are.  (A
            // workgroup's own keys and values are read before they may be written over.)
            const size_t row_bytes = size_t(plan->n_tokens) * head_dim * 2, q_bytes = row_bytes * n_q_heads, kv_bytes = row_bytes * n_kv_heads;
            const bool written_over = overlap(dq, q_bytes, q, q_bytes) || overlap(dq, q_bytes, d_out, q_bytes) || overlap(dq, q_bytes, k, kv_bytes) ||
                                      overlap(dq, q_bytes, v, kv_bytes) || overlap(dq, q_bytes, out, q_bytes) ||
                                      overlap(dk, kv_bytes, q, q_bytes) || overlap(dk, kv_bytes, d_out, q_bytes) ||
                                      overlap(dv, kv_bytes, q, q_bytes) || overlap(dv, kv_bytes, d_out, q_bytes);
            const bool gather = !written_over && aligned16(q) && aligned16(k) && aligned16(v) && aligned16(d_out) &&
                                gather_fits(plan->n_tokens, n_q_heads, head_dim);
            return gather ? run_mfma(dtag, std::true_type{}) : run_mfma(dtag, std::false_type{});
        };
        r = head_dim == 64 ? run(std::integral_constant<int, 64>{}) : run(std::integral_constant<int, 128>{});
    }
    if (r != ST_OK) return r;
    ST_LAUNCH_CHECK("st_attn_prefill_bwd kernels");
    return ST_OK;
}
