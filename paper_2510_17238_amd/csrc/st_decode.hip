// Dual-cache decode (Sec. 3.3 "Parallel KV caches"; Alg. 1: merge the visible source
// slice with the reasoning cache, then decode).
//
// Nothing is merged in memory.  The two caches are cut into work units of 128 to 4,096 tokens
// (decode_unit_tokens); a workgroup of four waves takes one (sequence, KV head, unit), streams that unit's K and V
// pages from HBM exactly once for all query heads of the group, and emits an un-normalised partial (o, m, l).  A second
// kernel merges all partials of BOTH caches per (sequence, query row, head) by log-sum-exp -- identical to a softmax over
// the concatenated cache.
//
// HBM-bound: 4 * D bytes per cached token and KV head, 2 * G * D useful flops for it.
// The arithmetic rides on the matrix cores only to keep the vector ALUs out of the
// way: S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16, where the 32
// columns are the (up to 32) query rows q_len * G.  The pool layouts make every operand
// a contiguous 16-byte load straight from global memory into MFMA registers:
//   K [page][head][d/8][slot][8] : lane (m, hg) reads slot m of d-chunk 2 j + hg
//   V [page][head][d][slot]      : lane (n, hg) reads slots 8 hg .. 8 hg + 7 of row d
#include <algorithm>
#include <type_traits>

#include "st_cache.h"
#include <mutex>

#include "st_tiles.h"

namespace st {

constexpr int kChunk = 512;                 // tokens per work unit
constexpr int kSmallDecodeTokens = 1024;    // both caches together: up to here one workgroup per (sequence, KV head) finishes the rows itself (small_decode)
constexpr int kChunkMin = 128;              // ... of a decode step of a few sequences
constexpr int kChunkLong = 4096;            // ... of a decode step when there is plenty of work (a wave's quarter is 64 pages: one id per lane)

// 16 bytes of a pool that this launch reads once and never again, taken in whole 128-byte lines per instruction: the
// load carries the non-temporal hint.  Value loads always do (measured on the decode step of 28 layers: 3 to 4 %
// faster).  Key loads do in launches of up to about 2 GB (STREAM_KEYS; 1 to 2.5 % faster on 0.7 GB per launch,
// 2 to 4 % slower on 3.8 GB per launch, A/B on one box each time).
template <typename T>
__device__ __forceinline__ u32x4 stream_load(const T* p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); }
template <bool STREAM, typename T>
__device__ __forceinline__ u32x4 key_load(const T* p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return *reinterpret_cast<const u32x4*>(p);
}

struct DecodeArgs {
    CacheView src, rsn;
    const int32_t* src_len;
    const int32_t* rsn_len;
    const uint16_t* q;
    float* part_o;     // [B][Hkv][nc][rows][D]
    float* part_ml;    // [B][Hkv][nc][rows][2]
    int batch, q_len, n_q_heads, n_kv_heads, group, rows;
    int ncs, ncr;      // chunk slots per (sequence, head) for the two caches
    int chunk;         // tokens per work unit (kChunkMin .. kChunkLong)
    float scale_log2;
    // source-chunk prefill only: ragged query counts and 32-row blocks
    const int32_t* n_new;   // [B] query tokens per sequence, or null for max_new everywhere
    int max_new;            // token stride of q / out
    int row_blocks;         // ceil(max_new * group / 32)
    // fused query rotation: q holds unrotated queries; row t is the token at index len - q_len + t of its own
    // stream (reasoning for a decode step, source for a source chunk), which is its position id
    int rope;
    RopeFreq freq;
    // one decoding step in one call (bf16, q_len = 1, <= 16 rows): the token k_new / v_new [batch][Hkv][D] is the one at
    // index rsn_len[b] - 1 of the reasoning stream and is NOT in the cache yet -- the launch stores it, attends over
    // the cached tokens before it, and takes the token itself from registers as one more partial state
    int append;
    const uint16_t* k_new;
    const uint16_t* v_new;
    // wave timeline (st_profile_wave_trace): (start, end) wall-clock pairs per workgroup, or null
    unsigned long long* trace;
    int trace_cap;
};

// A barrier for data exchanged through LDS alone: __syncthreads() also waits for every global load in flight -- here the first
// keys and values, requested before the queries are rotated.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Stamps the workgroup's start and end into the timeline buffer, whichever way the kernel is left.
struct WaveStamp {
    unsigned long long* slot;
    unsigned long long t0;
    __device__ __forceinline__ WaveStamp(const DecodeArgs& a) : slot(nullptr), t0(0) {
        if (a.trace && int(blockIdx.x) < a.trace_cap) {
            slot = a.trace + 2 * size_t(blockIdx.x);
            t0 = wall_clock64();
        }
    }
    __device__ __forceinline__ ~WaveStamp() {
        if (slot && threadIdx.x == 0) {
            slot[0] = t0;
            slot[1] = wall_clock64();
        }
    }
};

// The split kernels: a workgroup of FOUR WAVES takes one work unit (one cache of one sequence and KV head, a.chunk tokens)
// and deals its steps out to the waves in turn; their states meet in LDS and ONE partial result leaves the
// workgroup.  A partial is rows x D floats, written and read back by the merge kernel: with a wave per unit either the units
// were short and the partials cost more than the bytes alone say (64 sequences of up to 24K tokens, 32 rows: 512-token units
// 910 us, 1,024-token units 852), or they were long and the launch ended with a few of them.
constexpr int kSplitWaves = 4;

// what the waves of a workgroup leave for the merge: [4][rows][D] un-normalised outputs, [4][rows] reference exponents and sums
template <int D>
struct SplitLds {
    float *o, *m, *l;
    __device__ __forceinline__ SplitLds(unsigned char* smem, int rows)
        : o(reinterpret_cast<float*>(smem)), m(o + kSplitWaves * rows * D), l(m + kSplitWaves * rows) {}
};
inline size_t split_lds_bytes(int rows, int d) { return sizeof(float) * size_t(kSplitWaves) * rows * (d + 2); }

// A state (reference exponent m, sum l) without a finite score: nothing that its row sees -- or NaN scores alone, whose sum says
// so and has to reach the row (its weight 2^(-inf) = 0 keeps a NaN one).
__device__ __forceinline__ bool holds_nothing(float m, float l) { return m == -INFINITY && l == 0.f; }

// log-sum-exp merge of the waves' states into the unit's partial result at row slot `slot`
template <int D>
__device__ __forceinline__ void merge_waves(const SplitLds<D>& sm, const DecodeArgs& a, int64_t slot) {
    for (int e = int(threadIdx.x) * 4; e < a.rows * D; e += 64 * kSplitWaves * 4) {
        const int row = e / D, d0 = e % D;
        float m_all = -INFINITY;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) m_all = fmaxf(m_all, sm.m[w * a.rows + row]);
        const float m_use = m_all == -INFINITY ? 0.f : m_all;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) {
            const float mw = sm.m[w * a.rows + row], lw = sm.l[w * a.rows + row];
            if (holds_nothing(mw, lw)) continue;
            const float wt = __builtin_amdgcn_exp2f(mw - m_use);
            den = fmaf(wt, lw, den);
            const f32x4 o = *reinterpret_cast<const f32x4*>(sm.o + (w * a.rows + row) * D + d0);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fmaf(wt, o[i], acc[i]);
        }
        *reinterpret_cast<f32x4*>(a.part_o + (slot + row) * D + d0) = acc;
        if (d0 == 0) {
            a.part_ml[(slot + row) * 2] = m_all;
            a.part_ml[(slot + row) * 2 + 1] = den;
        }
    }
}

// Fused query rotation (Sec. 3.2, stream-local position ids): fragments j and j + KS/2 of a lane hold the two halves of
// eight rotation pairs, head dims STRIDE j + off + e and D/2 + the same; `row` holds (cos, sin) of the pairs at the row's
// position (rope_table_to_lds).
template <int KS, int STRIDE>
__device__ __forceinline__ void rotate_fragments(bf16x8 (&f)[KS], int off, const float2* row) {
#pragma unroll
    for (int j = 0; j < KS / 2; ++j) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float2 r = row[STRIDE * j + off + e];
            const float x = float(f[j][e]), y = float(f[j + KS / 2][e]);
            f[j][e] = (__bf16)(x * r.x - y * r.y);
            f[j + KS / 2][e] = (__bf16)(y * r.x + x * r.y);
        }
        __builtin_amdgcn_sched_barrier(0);               // (all table reads at once would take 128 registers)
    }
}

// Unit of a workgroup among the nc of its (sequence, KV head).  Consecutive workgroups go to the eight XCDs in turn: where nc shares a
// factor g with 8, the same unit of every head would land on the same 8 / g of them -- and with caches of unlike length it is the
// first units that have tokens (128 sequences of 300 + 300 tokens and one of 12,000, eight slots a head: 163 us, with 72 us of
// work; now 97).  So the units of a head are turned by one place whenever the heads have been once around the XCDs.
__device__ __forceinline__ int unit_of(unsigned block, int nc) {
    const unsigned bh = block / unsigned(nc), i = block % unsigned(nc), g = min(unsigned(nc & -nc), 8u);
    return int(g == 1 ? i : (i + bh * g / 8) % unsigned(nc));
}

// The decode step with 17 .. 32 query rows q_len * G per sequence and KV head (several tokens in one call, or wide groups) on
// v_mfma_f32_32x32x16_bf16, whose 32 columns are the query rows.  As in the 16-row kernel below the bytes in flight are what
// counts -- 4 D bytes per token against 128 flop per byte: the page ids of a wave's run are fetched once, the 16 KB of the next
// 32 tokens are requested before the present ones are multiplied (two register sets), whole 128-byte lines per instruction,
// value loads with the non-temporal hint.  That only fits two waves per SIMD with the queries in LDS, in fragment order (one
// copy for the four waves; each fragment is read back right before its matrix instruction).  A lane owns a query row, whose
// reference exponent is the largest score of the present step: the weights are rounded to bf16 for the second product, and the
// largest is then 1, which rounds to itself.  (A reference that moved only when a step exceeded it by 2^8 spared the rescale of the
// accumulator and cost 4 % of precision against a running maximum; this gives 4 % more.  Error of the rows against 64 bits, 64
// sequences of up to 8K + 16K tokens: 2.76e-3 with a running maximum over 512 tokens, 2.88e-3, 2.63e-3.  Time: 0 to 2 %.)
// 64 sequences of up to 8K + 16K tokens, 8 tokens x 4 heads, 8 KV heads of 128 dims (3.78 GB of cache), with the merge
// of the partial results: 1.50 ms with loads requested when they were needed, 0.89 with a wave per unit of 1,024 tokens, 0.75 with four
// waves and longer ones, 0.71 with the units spread over the XCDs (unit_of).
template <int D, bool STREAM_KEYS>
__global__ __launch_bounds__(64 * kSplitWaves, 2) void decode_split32_kernel(DecodeArgs a) {
    constexpr int KS = D / 16, DB = D / 32, KCH = D / 8;
    constexpr float kDrop = 16.f;
    // query fragments [KS][64 lanes], behind them the (cos, sin) of the q_len query positions; after the loop: SplitLds
    extern __shared__ __align__(16) unsigned char smem_raw[];
    bf16x8* s_q = reinterpret_cast<bf16x8*>(smem_raw);
    float2* s_rot = reinterpret_cast<float2*>(s_q + KS * 64);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nc = a.ncs + a.ncr;
    const unsigned bh = blockIdx.x / unsigned(nc);       // (sequence, KV head)
    const int c = unit_of(blockIdx.x, nc);
    const int h = int(bh % unsigned(a.n_kv_heads));
    const int b = int(bh / unsigned(a.n_kv_heads));
    const bool is_src = c < a.ncs;
    const CacheView& cv = is_src ? a.src : a.rsn;
    const int unit0 = (is_src ? c : c - a.ncs) * a.chunk;
    // wave w takes the 32-token steps w, w + 4, ...; the page ids of all of them (one per lane, 32 steps at most) are asked for
    // before the length is known, as in Pages16
    int my_page = cv.page_table[int64_t(b) * cv.max_pages + min(unit0 / kPage + 2 * (kSplitWaves * (lane >> 1) + wave) + (lane & 1), cv.max_pages - 1)];
    my_page = min(max(my_page, 0), cv.n_pages - 1);
    const int len = min(max(is_src ? a.src_len[b] : a.rsn_len[b], 0), cv.max_pages * kPage);
    if (unit0 >= len) return;
    const int n_steps = (min(len - unit0, a.chunk) - 32 * wave + 32 * kSplitWaves - 1) / (32 * kSplitWaves);

    const int n = lane & 31, hg = lane >> 5;
    const bool valid_row = n < a.rows;                  // row of this (sequence, KV head): token n / G, head n % G
    const int nr = min(n, a.rows - 1);                  // rows past the end repeat the last one (never stored)
    const int t_row = nr / a.group;
    const int hq = h * a.group + nr % a.group;
    // visible reasoning tokens of query row t: [0, len - q_len + t]; the source slice is seen whole
    const int limit = is_src ? len : min(max(len - a.q_len + t_row + 1, 0), len);
    const int limit_min = is_src ? len : min(max(len - a.q_len + 1, 0), len);

    const int64_t page_k = int64_t(cv.n_kv_heads) * KCH * (kPage * 8);
    const int64_t page_v = int64_t(cv.n_kv_heads) * D * kPage;
    // K: lane (m = n, hg) reads slot swap23(m % 16) of page m / 16, d-chunk 2 j + hg; V: lane (m = n, hg) reads slots
    // 8 hg .. + 7 of row d = 32 db + m
    const uint16_t* k_lane = cv.k_pool + int64_t(h) * KCH * (kPage * 8) + hg * (kPage * 8) + swap23(n & 15) * 8;
    const uint16_t* v_lane = cv.v_pool + int64_t(h) * D * kPage + n * kPage + 8 * hg;
    auto load = [&](int s, u32x4 (&kk)[KS], u32x4 (&vv)[2][DB]) {
        const int id0 = __builtin_amdgcn_readlane(my_page, 2 * s), id1 = __builtin_amdgcn_readlane(my_page, 2 * s + 1);
        const uint16_t* kp = k_lane + int64_t(n >> 4 ? id1 : id0) * page_k;
#pragma unroll
        for (int j = 0; j < KS; ++j) kk[j] = key_load<STREAM_KEYS>(kp + 2 * j * (kPage * 8));
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db) vv[t][db] = stream_load(v_lane + int64_t(t ? id1 : id0) * page_v + db * 32 * kPage);
    };
    u32x4 ka[KS], va[2][DB], kb[KS], vb[2][DB];
    if (n_steps > 0) load(0, ka, va);
    // the queries: wave w takes fragments w and w + KS / 2 (the two halves of their rotation pairs), rotates them by the
    // row's position -- its index in the reasoning stream -- and leaves them for all four
    if (a.rope) rope_table_to_lds<D>(s_rot, min(max(a.rsn_len[b], 0), a.rsn.max_pages * kPage) - a.q_len, a.q_len, rope_frequency<D>(a.freq), 64 * kSplitWaves);
    lds_barrier();
    if (wave < KS / 2) {
        const uint16_t* qp = a.q + ((int64_t(b) * a.q_len + t_row) * a.n_q_heads + hq) * D + 8 * hg + 16 * wave;
        bf16x8 qf[2] = {*reinterpret_cast<const bf16x8*>(qp), *reinterpret_cast<const bf16x8*>(qp + D / 2)};
        if (a.rope) rotate_fragments<2, 16>(qf, 8 * hg + 16 * wave, s_rot + t_row * (D / 2));
        s_q[wave * 64 + lane] = qf[0];
        s_q[(wave + KS / 2) * 64 + lane] = qf[1];
    }
    lds_barrier();
    f32x16 o_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[db][i] = 0.f;
    float m_ref = 0.f, m_top = -INFINITY, l_run = 0.f;

    auto compute = [&](int s, const u32x4 (&kk)[KS], u32x4 (&vv)[2][DB]) {
        const int tok = unit0 + 32 * (kSplitWaves * s + wave);
        f32x16 t;
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = 0.f;
#pragma unroll
        for (int j = 0; j < KS; ++j) t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kk[j]), s_q[j * 64 + lane], t, 0, 0, 0);
        // register i <-> token tok + 16 (i/8) + 8 hg + i%8
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = fmaf(t[i], a.scale_log2, -m_ref);
        if (tok + 32 > limit_min) {                     // uniform: a step that reaches some row's limit
#pragma unroll
            for (int i = 0; i < 16; ++i) t[i] = tok + 16 * (i >> 3) + 8 * hg + (i & 7) < limit ? t[i] : -INFINITY;
        }
        float mx = t[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, t[i]);
        // the reference moves to the step's largest score, but stays within kDrop of the largest so far (the accumulators of a long
        // run of small scores would overflow); a step in which the row sees nothing leaves it (a row lives in lanes n and n + 32)
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        const float rise = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
        const float m_new = rise > -INFINITY ? fmaxf(m_ref + rise, m_top - kDrop) : m_ref;
        const float shift = m_new - m_ref;              // (what is left of it in 32 bits: scores and sums move alike)
        const float alpha = m_top > -INFINITY ? __builtin_amdgcn_exp2f(-shift) : 1.f;
        m_top = rise > -INFINITY ? fmaxf(m_top, m_new) : m_top;
        m_ref = m_new;
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] -= shift;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) o_acc[db][i] *= alpha;
        bf16x8 pb[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float p = __builtin_amdgcn_exp2f(t[i]);
            l_run += p;
            pb[i >> 3][i & 7] = (__bf16)p;
        }
        if (tok + 32 > len) {                           // uniform: slots past the visible length may hold anything
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int first = tok + 16 * u + 8 * hg;
                u32x4 keep;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    keep[e] = (first + 2 * e < len ? 0x0000ffffu : 0u) | (first + 2 * e + 1 < len ? 0xffff0000u : 0u);
#pragma unroll
                for (int db = 0; db < DB; ++db) vv[u][db] &= keep;
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv[u][db]), pb[u], o_acc[db], 0, 0, 0);
    };
    for (int s = 0; s < n_steps; s += 2) {
        if (s + 1 < n_steps) load(s + 1, kb, vb);
        __builtin_amdgcn_sched_barrier(0);
        compute(s, ka, va);
        if (s + 1 < n_steps) {
            if (s + 2 < n_steps) load(s + 2, ka, va);
            __builtin_amdgcn_sched_barrier(0);
            compute(s + 1, kb, vb);
        }
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32);
    __syncthreads();                                    // everybody is done with the query fragments
    const SplitLds<D> sm(smem_raw, a.rows);
    if (valid_row) {
        float* po = sm.o + (wave * a.rows + n) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<f32x4*>(po + 32 * db + 8 * q4 + 4 * hg) =
                    f32x4{o_acc[db][4 * q4], o_acc[db][4 * q4 + 1], o_acc[db][4 * q4 + 2], o_acc[db][4 * q4 + 3]};
        if (hg == 0) {
            sm.m[wave * a.rows + n] = m_top > -INFINITY ? m_ref : -INFINITY;
            sm.l[wave * a.rows + n] = l_tot;
        }
    }
    __syncthreads();
    merge_waves<D>(sm, a, ((int64_t(b) * a.n_kv_heads + h) * nc + c) * a.rows);
}
// LDS of a workgroup: the loop's part (queries, rotations) and the merge's share the space
inline size_t split32_lds_bytes(int rows, int q_len, int d) {
    const size_t loop = size_t(d / 16) * 64 * 16 + size_t(q_len) * (d / 2) * sizeof(float2), merge = split_lds_bytes(rows, d);
    return loop > merge ? loop : merge;
}

// Variant for q_len * G <= 16 query rows (the one-token decode step): the same scheme on v_mfma_f32_16x16x32_bf16.
// A wave takes 32 tokens (two pages) per step with two first-product MFMAs X and Y whose 16 key
// rows are chosen so that afterwards quarter-wave g4 (lanes 16 g4 .. 16 g4 + 15) holds, for its
// query column, the 8 CONSECUTIVE slots 8 (g4 % 2) .. + 7 of page g4 / 2: X gives slots +0..3,
// Y gives slots +4..7.  Those 8 probabilities are exactly one B operand of the second product,
// whose A operand (V^T) is then one contiguous 16-byte load.  All loads are unconditional (page
// ids are clamped into the pool); what lies beyond the visible length is removed afterwards by
// index: scores by select, V by bit mask.
// 32 sequences of 2K + 1K to 6K tokens, 16 / 8 heads of 128 dims, the new token stored in the same launch, with the merge of
// the partial results: 130 us per layer with one wave per unit, 125 us with four (5.8 TB/s; a copy of that size runs at 4.9).
// One step of the 16-row kernels: 32 tokens (two pages), 8 key loads and 8 value loads of 16 bytes per lane at D = 128.
template <int D>
struct Tokens16 {
    u32x4 kx[D / 32], ky[D / 32], vv[D / 16];
};

// A wave's steps of one cache: every `stride`-th step from token tok0 on.  Under load a memory round trip takes microseconds,
// so what precedes the first keys is kept to one: the page ids of all the wave's steps (one per lane, 32 steps at most) are
// asked for without waiting for the cache's length; pages past the end are read like any other (ids clamped into the pool)
// and removed by index.
// K: lane (m = n, g4) reads d-chunk 4 j + g4 of key row m; row m lives in page m / 8, slot m % 8 for X and + 8 for Y --
//    the 64 lanes of one load instruction take whole 128-byte lines (eight slots of a d-chunk), none shared with another
// V: lane (m = n, g4) reads slots 8 (g4 % 2) .. + 7 of row d = 16 db + m in page g4 / 2
template <int D, bool STREAM_KEYS>
struct Pages16 {
    static constexpr int KS = D / 32, DB = D / 16, KCH = D / 8;
    int my_page;
    const uint16_t *k_pool, *v_pool;
    int k_lane, v_lane;                  // this lane's place in a page (the pools are uniform: a lane keeps no address)
    int64_t page_k, page_v;
    __device__ __forceinline__ Pages16(const CacheView& cv, int b, int h, int lane, int tok0, int stride) {
        const int n = lane & 15, g4 = lane >> 4;
        const int page = tok0 / kPage + 2 * stride * (lane >> 1) + (lane & 1);
        const int id = cv.page_table[int64_t(b) * cv.max_pages + min(page, cv.max_pages - 1)];
        k_pool = cv.k_pool + int64_t(h) * KCH * (kPage * 8);
        v_pool = cv.v_pool + int64_t(h) * D * kPage;
        k_lane = g4 * (kPage * 8) + (n & 7) * 8;
        v_lane = n * kPage + 8 * (g4 & 1);
        page_k = int64_t(cv.n_kv_heads) * KCH * (kPage * 8);
        page_v = int64_t(cv.n_kv_heads) * D * kPage;
        my_page = min(max(id, 0), cv.n_pages - 1);
    }
    // step s of this cache, or of the other one where a wave walks both: their pages are alike, the pools and ids are not
    __device__ __forceinline__ void load(int s, Tokens16<D>& t32) const { load(s, t32, my_page, k_pool, v_pool); }
    __device__ __forceinline__ void load(int s, Tokens16<D>& t32, int page, const uint16_t* k_of, const uint16_t* v_of) const {
        const int lane = int(threadIdx.x & 63);
        const int id0 = __builtin_amdgcn_readlane(page, 2 * s), id1 = __builtin_amdgcn_readlane(page, 2 * s + 1);
        const uint16_t* kp = k_of + (int64_t(lane & 8 ? id1 : id0) * page_k + k_lane);
        const uint16_t* vp = v_of + (int64_t(lane & 32 ? id1 : id0) * page_v + v_lane);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            t32.kx[j] = key_load<STREAM_KEYS>(kp + 4 * j * (kPage * 8));
            t32.ky[j] = key_load<STREAM_KEYS>(kp + 4 * j * (kPage * 8) + 8 * 8);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) t32.vv[db] = stream_load(vp + db * 16 * kPage);
    }
};

// The running state of a query column (lane (n, g4): column n), in base-2 exponent units: m_ref is the column's reference
// exponent (the same in its four lanes); it starts at 0 with has_ref = false and is moved, out of line, only when a step brings
// an exponent more than kLazyRise above it (or the first finite score): the common step then needs no exchange between lanes
// and no rescale of the accumulator -- probabilities are bounded by 2^kLazyRise instead of 1, which fp32 and bf16 do not mind,
// and whoever finishes the row divides by l anyway.
template <int D>
struct State16 {
    static constexpr int KS = D / 32, DB = D / 16;
    static constexpr float kLazyRise = 8.f;
    bf16x8 qf[KS];
    f32x4 o_acc[DB];
    float m_ref = 0.f, l_run = 0.f;
    bool has_ref = false;
    __device__ __forceinline__ State16() {
#pragma unroll
        for (int db = 0; db < DB; ++db) o_acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // value of the three other lanes of a query column folded in (lanes n, n + 16, n + 32, n + 48):
    // v_permlane16_swap / v_permlane32_swap exchange 16- / 32-lane rows between their two operands; with
    // both operands set to x, every lane finds x of lane ^ 16 (^ 32) in one of the two results
    static __device__ __forceinline__ float column_max(float x) {
        float a1 = x, b1 = x;
        asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a1), "+v"(b1));
        float a2 = fmaxf(a1, b1), b2 = a2;
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a2), "+v"(b2));
        return fmaxf(a2, b2);
    }
    // one step: 32 tokens from token `tok` of a cache of `len` visible tokens, of which this lane's row sees [0, limit) and every
    // row [0, limit_min)
    __device__ __forceinline__ void step(Tokens16<D>& t32, int tok, int len, int limit, int limit_min, float scale_log2) {
        u32x4 (&kx)[KS] = t32.kx;
        u32x4 (&ky)[KS] = t32.ky;
        u32x4 (&vv)[DB] = t32.vv;
        const int g4 = int(threadIdx.x & 63) >> 4;
        bf16x2 ones2;
        ones2[0] = (__bf16)1.f;
        ones2[1] = (__bf16)1.f;
        const int first = tok + 8 * g4;       // token of this lane's first VALUE slot
        // scores of this lane: X rows 4 g4 .. + 3 and the Y rows eight slots further on
        const int first_k = tok + 16 * (g4 >> 1) + 4 * (g4 & 1);
        f32x4 sx = {0.f, 0.f, 0.f, 0.f}, sy = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kx[j]), qf[j], sx, 0, 0, 0);
            sy = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ky[j]), qf[j], sy, 0, 0, 0);
        }
        float t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = fmaf(e < 4 ? sx[e] : sy[e - 4], scale_log2, -m_ref);
        if (tok + 32 > limit_min) {           // uniform: a step that reaches some row's limit
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = first_k + (e & 3) + 8 * (e >> 2) < limit ? t[e] : -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, t[e]);
        if (__any(mx > kLazyRise || (!has_ref && mx > -INFINITY))) {
            // out of line: move the reference of the rows that need it, rescale what they have accumulated
            const float rise = column_max(mx);
            const bool move = has_ref ? rise > 0.f : rise > -INFINITY;
            const float shift = move ? rise : 0.f;
            const float alpha = has_ref ? __builtin_amdgcn_exp2f(-shift) : 1.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] -= shift;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) o_acc[db][i] *= alpha;
            m_ref += shift;
            has_ref = has_ref || move;
        }
        u32x4 pw;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            bf16x2 p2;
            p2[0] = (__bf16)__builtin_amdgcn_exp2f(t[e]);
            p2[1] = (__bf16)__builtin_amdgcn_exp2f(t[e + 1]);
            l_run = __builtin_amdgcn_fdot2_f32_bf16(p2, ones2, l_run, false);
            pw[e / 2] = __builtin_bit_cast(uint32_t, p2);
        }
        // The value operand of lane group g4 holds slots 8 (g4 % 2) .. + 7 of page g4 / 2, in order; the weights
        // of those slots sit half in this lane (X for even, Y for odd groups) and half in the lane of group g4 ^ 1:
        // one exchange of 16-lane rows per register pair (odd rows of the X words against even rows of the Y words)
        // leaves every lane with the eight weights of its value slots, in slot order.
#pragma unroll
        for (int r = 0; r < 2; ++r)
            asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(pw[r]), "+v"(pw[2 + r]));
        const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
        if (tok + 32 > len) {                 // uniform: only the step that holds the end of the cache
            u32x4 keep;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                keep[e] = (first + 2 * e < len ? 0x0000ffffu : 0u) | (first + 2 * e + 1 < len ? 0xffff0000u : 0u);
#pragma unroll
            for (int db = 0; db < DB; ++db) vv[db] &= keep;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
            o_acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv[db]), pb, o_acc[db], 0, 0, 0);
    }
};

template <int D, bool STREAM_KEYS>
__global__ __launch_bounds__(64 * kSplitWaves, 2) void decode_split16_kernel(DecodeArgs a) {
    constexpr int KS = D / 32, DB = D / 16, KCH = D / 8;
    // (cos, sin) of the q_len query positions; after the loop: SplitLds
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float2* s_rot = reinterpret_cast<float2*>(smem_raw);
    const WaveStamp stamp(a);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nc = a.ncs + a.ncr + a.append;             // (append: one more slot per sequence and head, the new token's)
    const unsigned bh = blockIdx.x / unsigned(nc);       // (sequence, KV head)
    const int c = unit_of(blockIdx.x, nc);
    const int h = int(bh % unsigned(a.n_kv_heads));
    const int b = int(bh / unsigned(a.n_kv_heads));
    const bool is_src = c < a.ncs;
    const bool is_tok = c == a.ncs + a.ncr;
    const CacheView& cv = is_src ? a.src : a.rsn;
    const int cc = is_src ? c : c - a.ncs;
    const int unit0 = is_tok ? 0 : cc * a.chunk;
    const int n = lane & 15, g4 = lane >> 4;
    const bool valid_row = n < a.rows;
    const int nr = min(n, a.rows - 1);                  // rows past the end repeat the last one (never stored)
    const int t_row = nr / a.group;
    const int hq = h * a.group + nr % a.group;
    // asked for at once: the page ids, the queries, a rotation frequency (rope_table_to_lds), the lengths
    const Pages16<D, STREAM_KEYS> pages(cv, b, h, lane, unit0 + 32 * wave, kSplitWaves);
    State16<D> st;
    {
        const uint16_t* qp = a.q + ((int64_t(b) * a.q_len + t_row) * a.n_q_heads + hq) * D + 8 * g4;
#pragma unroll
        for (int j = 0; j < KS; ++j) st.qf[j] = *reinterpret_cast<const bf16x8*>(qp + 32 * j);
    }
    const int len_all = min(max(is_src ? a.src_len[b] : a.rsn_len[b], 0), cv.max_pages * kPage);
    const int len = (a.append && !is_src && len_all > 0) ? len_all - 1 : len_all;     // cached tokens to walk
    if (is_tok ? len_all == 0 : unit0 >= len) return;
    // this wave's steps: every fourth one of the unit's
    const int n_steps = is_tok ? 0 : (min(len - unit0, a.chunk) - 32 * wave + 32 * kSplitWaves - 1) / (32 * kSplitWaves);
    const int limit = is_src ? len : min(max(len - a.q_len + t_row + 1, 0), len);
    const int limit_min = is_src ? len : min(max(len - a.q_len + 1, 0), len);         // the smallest limit of any row (row 0's)
    Tokens16<D> ta, tb;
    if (n_steps > 0) pages.load(0, ta);
    if (a.rope) {
        const int len_r = min(max(a.rsn_len[b], 0), a.rsn.max_pages * kPage);
        rope_table_to_lds<D>(s_rot, len_r - a.q_len, a.q_len, rope_frequency<D>(a.freq), 64 * kSplitWaves);
        lds_barrier();
        rotate_fragments<KS, 32>(st.qf, 8 * g4, s_rot + t_row * (D / 2));
    }
    if (is_tok && wave > 0) {
        // (the new token is one wave's work; the others hold nothing)
    } else if (is_tok) {
        // the new token: key fragments in the query's layout (piece 4 j + g4 of the row), rotated by the token's index
        const int idx = len_all - 1;
        bf16x8 kf[KS];
        const uint16_t* kp = a.k_new + (int64_t(b) * a.n_kv_heads + h) * D + 8 * g4;
#pragma unroll
        for (int j = 0; j < KS; ++j) kf[j] = *reinterpret_cast<const bf16x8*>(kp + 32 * j);
        if (a.rope) rotate_fragments<KS, 32>(kf, 8 * g4, s_rot);         // (q_len = 1: the query's position)
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < KS; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf(float(st.qf[j][e]), float(kf[j][e]), dot);
        dot += __shfl_xor(dot, 16);
        dot += __shfl_xor(dot, 32);
        st.m_ref = dot * a.scale_log2;
        st.has_ref = true;
        st.l_run = g4 == 0 ? 1.f : 0.f;                                  // (summed over the four lanes of a row below)
        const uint16_t* vp = a.v_new + (int64_t(b) * a.n_kv_heads + h) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) st.o_acc[db][i] = bf16_bits_to_f32(vp[16 * db + 4 * g4 + i]);
        // into the cache: this head's key and value at index idx; the workgroup of head 0 writes the new length
        const int id = a.rsn.page_table[int64_t(b) * a.rsn.max_pages + idx / kPage];
        const int slot_in_page = idx % kPage;
        if (id >= 0 && id < a.rsn.n_pages) {                          // never write outside the pool
            if (n == 0) {
                uint16_t* kdst = a.rsn.k_pool + (int64_t(id) * a.n_kv_heads + h) * KCH * (kPage * 8) + slot_in_page * 8;
#pragma unroll
                for (int j = 0; j < KS; ++j) *reinterpret_cast<bf16x8*>(kdst + (4 * j + g4) * (kPage * 8)) = kf[j];
            }
            uint16_t* vdst = a.rsn.v_pool + (int64_t(id) * a.n_kv_heads + h) * (D * kPage) + slot_in_page;
            for (int d0 = lane; d0 < D; d0 += 64) vdst[d0 * kPage] = vp[d0];
        }
        if (h == 0 && lane == 0) a.rsn.appended_len[b] = len_all;
    } else {
        // The loads of step x + 1 are issued before step x is computed (two register sets, used in turn): a wave has up to two
        // steps' worth of bytes in flight, and a load's latency is covered by the step before it.
        const int tok0 = unit0 + 32 * wave;
        for (int x = 0; x < n_steps; x += 2) {
            if (x + 1 < n_steps) pages.load(x + 1, tb);
            __builtin_amdgcn_sched_barrier(0);
            st.step(ta, tok0 + 32 * kSplitWaves * x, len, limit, limit_min, a.scale_log2);
            if (x + 1 < n_steps) {
                if (x + 2 < n_steps) pages.load(x + 2, ta);
                __builtin_amdgcn_sched_barrier(0);
                st.step(tb, tok0 + 32 * kSplitWaves * (x + 1), len, limit, limit_min, a.scale_log2);
            }
        }
    }

    float l_tot = st.l_run + __shfl_xor(st.l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    __syncthreads();                                    // everybody is done with the rotations
    const SplitLds<D> sm(smem_raw, a.rows);
    if (valid_row) {
        // lane (n, g4), block db, register i  <->  d = 16 db + 4 g4 + i
        float* po = sm.o + (wave * a.rows + n) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(po + 16 * db + 4 * g4) = st.o_acc[db];
        if (g4 == 0) {
            sm.m[wave * a.rows + n] = st.has_ref ? st.m_ref : -INFINITY;
            sm.l[wave * a.rows + n] = l_tot;
        }
    }
    __syncthreads();
    merge_waves<D>(sm, a, ((int64_t(b) * a.n_kv_heads + h) * nc + c) * a.rows);
}
// LDS of a workgroup: the rotations and the merge share the space
inline size_t split16_lds_bytes(int rows, int q_len, int d) {
    const size_t loop = size_t(q_len) * (d / 2) * sizeof(float2), merge = split_lds_bytes(rows, d);
    return loop > merge ? loop : merge;
}

// Short caches (the streaming session of one listener: a hundred source tokens, a few hundred reasoning tokens): one
// workgroup per (sequence, KV head) does everything -- no partial results in memory, no merge kernel, one launch per
// layer and token instead of two.  Such a step is bound by the chain of memory round trips a wave makes walking its
// tokens, so the tokens of BOTH caches are dealt out in steps of 32 to the waves of the workgroup (reasoning steps from the
// first wave up, source steps from the last one down -- who takes what is known before the lengths are), and the waves' states
// meet in LDS, where all threads merge them (log-sum-exp, fixed order) and write the finished rows.
// Two workgroups per compute unit, which takes 128 registers (with 134 from 257 workgroups on the second half waited for the
// first: 48 sequences, 32 / 8 heads of 128 dims, 128 tokens 9.9 -> 8.0 us, 640 tokens 26.1 -> 24.2).
constexpr int kSmallWaves = 8, kTokenWave = 4;

// APPEND (one new token per sequence, q_len = 1): k_new / v_new [batch][Hkv][D] is the token at index
// rsn_len[b] - 1 of the reasoning stream.  The workgroup of (sequence, KV head) stores its head's key (rotated by
// that index if a.rope) and value in the reasoning cache, folds the token in from registers -- score in fp32 from
// the bf16 operands, as the matrix instruction would -- and walks the cache only up to the token before it; the
// workgroup of head 0 writes the new length.  Nobody in this launch reads what it writes.
template <int D, bool APPEND>
__global__ __launch_bounds__(64 * kSmallWaves, 4) void decode_small16_kernel(DecodeArgs a, uint16_t* __restrict__ out, float* __restrict__ lse,
                                                                          const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new) {
    constexpr int KS = D / 32, DB = D / 16, KCH = D / 8;
    constexpr int W = kSmallWaves;
    constexpr int WP = APPEND ? W + 1 : W;            // states to merge: the waves' and the new token's
    extern __shared__ __align__(16) unsigned char smem_raw[];
    // [WP][rows][D] partial outputs, [WP][rows] reference exponents and sums, [q_len][D/2] (cos, sin)
    float* sm_o = reinterpret_cast<float*>(smem_raw);
    float2* sm_ml = reinterpret_cast<float2*>(sm_o + WP * a.rows * D);
    float2* sm_rot = sm_ml + WP * a.rows;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = int(blockIdx.x % unsigned(a.n_kv_heads));
    const int b = int(blockIdx.x / unsigned(a.n_kv_heads));
    const int n = lane & 15, g4 = lane >> 4;
    const bool valid_row = n < a.rows;
    const int nr = min(n, a.rows - 1);
    const int t_row = nr / a.group;
    const int hq = h * a.group + nr % a.group;
    // asked for at once: the page ids of both caches, the queries, the new token (wave kTokenWave), a rotation frequency, the
    // lengths
    const Pages16<D, false> pages_s(a.src, b, h, lane, 32 * (W - 1 - wave), W), pages_r(a.rsn, b, h, lane, 32 * wave, W);
    State16<D> st;
    {
        const uint16_t* qp = a.q + ((int64_t(b) * a.q_len + t_row) * a.n_q_heads + hq) * D + 8 * g4;
#pragma unroll
        for (int j = 0; j < KS; ++j) st.qf[j] = *reinterpret_cast<const bf16x8*>(qp + 32 * j);
    }
    const bool token_wave = APPEND && wave == kTokenWave;
    bf16x8 kf[KS];                                   // key fragments in the query's layout (piece 4 j + g4 of the row)
    uint16_t vf[D / 64];                             // value elements lane, lane + 64
    if (token_wave) {
        const uint16_t* kp = k_new + (int64_t(b) * a.n_kv_heads + h) * D + 8 * g4;
#pragma unroll
        for (int j = 0; j < KS; ++j) kf[j] = *reinterpret_cast<const bf16x8*>(kp + 32 * j);
#pragma unroll
        for (int u = 0; u < D / 64; ++u) vf[u] = v_new[(int64_t(b) * a.n_kv_heads + h) * D + 64 * u + lane];
    }
    const double freq = a.rope ? rope_frequency<D>(a.freq) : 0.0;
    const int len_s = min(max(a.src_len[b], 0), a.src.max_pages * kPage);
    const int len_all = min(max(a.rsn_len[b], 0), a.rsn.max_pages * kPage);
    const bool add = APPEND && len_all > 0;          // (rsn_len 0: an idle sequence, nothing to store)
    const int len_r = add ? len_all - 1 : len_all;   // cached reasoning tokens to walk
    // this wave's steps of 32 tokens: reasoning steps from wave 0 up, then source steps from the last wave down
    const int steps_s = (len_s - 32 * (W - 1 - wave) + 32 * W - 1) / (32 * W), steps_r = (len_r - 32 * wave + 32 * W - 1) / (32 * W);
    const int n_steps = steps_r + steps_s;
    auto load = [&](int x, Tokens16<D>& t) {
        const bool r = x < steps_r;
        pages_r.load(r ? x : x - steps_r, t, r ? pages_r.my_page : pages_s.my_page, r ? pages_r.k_pool : pages_s.k_pool, r ? pages_r.v_pool : pages_s.v_pool);
    };
    // the source slice is seen whole; reasoning token j by rows t with j <= len_all - q_len + t
    const int limit = min(max(len_all - a.q_len + t_row + 1, 0), len_r), limit_min = min(max(len_all - a.q_len + 1, 0), len_r);
    auto step = [&](int x, Tokens16<D>& t) {
        const bool r = x < steps_r;
        st.step(t, r ? 32 * (wave + W * x) : 32 * (W - 1 - wave + W * (x - steps_r)), r ? len_r : len_s, r ? limit : len_s, r ? limit_min : len_s,
                a.scale_log2);
    };
    const int new_page = token_wave && add ? a.rsn.page_table[int64_t(b) * a.rsn.max_pages + (len_all - 1) / kPage] : -1;
    if (a.rope) {
        rope_table_to_lds<D>(sm_rot, len_all - a.q_len, a.q_len, freq, 64 * W);
        lds_barrier();
        rotate_fragments<KS, 32>(st.qf, 8 * g4, sm_rot + t_row * (D / 2));
    }
    if (token_wave && add) {
        // the new token: the same key for every row; its value row is its partial output
        if (a.rope) rotate_fragments<KS, 32>(kf, 8 * g4, sm_rot);
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < KS; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf(float(st.qf[j][e]), float(kf[j][e]), dot);
        dot += __shfl_xor(dot, 16);
        dot += __shfl_xor(dot, 32);
        if (valid_row && g4 == 0) {
            sm_ml[W * a.rows + n] = float2{dot * a.scale_log2, 1.f};
        }
        for (int r = 0; r < a.rows; ++r)
#pragma unroll
            for (int u = 0; u < D / 64; ++u) sm_o[(W * a.rows + r) * D + 64 * u + lane] = bf16_bits_to_f32(vf[u]);
        // into the cache: page of index len_all - 1, this head
        const int slot = (len_all - 1) % kPage;
        if (new_page >= 0 && new_page < a.rsn.n_pages) {         // never write outside the pool
            if (n == 0) {
                uint16_t* kdst = a.rsn.k_pool + (int64_t(new_page) * a.n_kv_heads + h) * KCH * (kPage * 8) + slot * 8;
#pragma unroll
                for (int j = 0; j < KS; ++j) *reinterpret_cast<bf16x8*>(kdst + (4 * j + g4) * (kPage * 8)) = kf[j];
            }
            uint16_t* vdst = a.rsn.v_pool + (int64_t(new_page) * a.n_kv_heads + h) * (D * kPage) + slot;
#pragma unroll
            for (int u = 0; u < D / 64; ++u) vdst[(64 * u + lane) * kPage] = vf[u];
        }
        if (h == 0 && lane == 0) a.rsn.appended_len[b] = len_all;
    }
    for (int x = 0; x < n_steps; ++x) {
        Tokens16<D> t;
        load(x, t);
        step(x, t);
    }
    if (token_wave && !add && lane < a.rows) {
        sm_ml[W * a.rows + lane] = float2{-INFINITY, 0.f};
    }
    float l_tot = st.l_run + __shfl_xor(st.l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    if (valid_row) {
        // lane (n, g4), block db, register i  <->  d = 16 db + 4 g4 + i
        float* po = sm_o + (wave * a.rows + n) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(po + 16 * db + 4 * g4) = st.o_acc[db];
        if (g4 == 0) {
            sm_ml[wave * a.rows + n] = float2{st.has_ref ? st.m_ref : -INFINITY, l_tot};
        }
    }
    __syncthreads();
    // Merge: a thread takes one dim of a row, two or four where the rows have more than the threads; everything it needs is read at once, and
    // all waves take part.  (State by state, each with a branch, by the threads that had four dims: 2,900 of the workgroup's 15,800 cycles
    // with 4 rows of 128 dims, now 2,000; 36 layers of one token, 32 / 8 heads, 400 cached tokens 298.5 -> 291.5 us.)
    auto merge = [&](auto width) {
        constexpr int N = decltype(width)::value;
        for (int e = int(threadIdx.x) * N; e < a.rows * D; e += 64 * W * N) {
            const int row = e / D, d0 = e % D;
            float mw[WP], lw[WP], o[WP][N], m_all = -INFINITY;
#pragma unroll
            for (int w = 0; w < WP; ++w) {
                const float2 ml = sm_ml[w * a.rows + row];
                mw[w] = ml.x;
                lw[w] = ml.y;
                const float* po = sm_o + (w * a.rows + row) * D + d0;
                if constexpr (N == 4) {
                    const f32x4 x = *reinterpret_cast<const f32x4*>(po);
#pragma unroll
                    for (int i = 0; i < N; ++i) o[w][i] = x[i];
                } else {
                    const f32x2 x = N == 2 ? *reinterpret_cast<const f32x2*>(po) : f32x2{po[0], 0.f};
#pragma unroll
                    for (int i = 0; i < N; ++i) o[w][i] = x[i];
                }
            }
#pragma unroll
            for (int w = 0; w < WP; ++w) m_all = fmaxf(m_all, mw[w]);
            float acc[N], den = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = 0.f;
#pragma unroll
            for (int w = 0; w < WP; ++w) {
                // (a state that holds nothing may hold anything in its output)
                const bool skip = m_all == -INFINITY || holds_nothing(mw[w], lw[w]);
                const float wt = skip ? 0.f : __builtin_amdgcn_exp2f(mw[w] - m_all);
                den = skip ? den : fmaf(wt, lw[w], den);
#pragma unroll
                for (int i = 0; i < N; ++i) acc[i] = skip ? acc[i] : fmaf(wt, o[w][i], acc[i]);
            }
            const float inv = den > 0.f ? 1.f / den : 0.f;           // a row that sees nothing: out = 0, lse = -inf
            const int t = a.q_len == 1 ? 0 : row / a.group, hq_row = h * a.group + (row - t * a.group);
            uint16_t* dst = out + ((int64_t(b) * a.q_len + t) * a.n_q_heads + hq_row) * D + d0;
            if constexpr (N == 4) {
                bf16x4 o4;
#pragma unroll
                for (int i = 0; i < 4; ++i) o4[i] = (__bf16)(acc[i] * inv);
                *reinterpret_cast<bf16x4*>(dst) = o4;
            } else if constexpr (N == 2) {
                bf16x2 o2;
                o2[0] = (__bf16)(acc[0] * inv);
                o2[1] = (__bf16)(acc[1] * inv);
                *reinterpret_cast<bf16x2*>(dst) = o2;
            } else {
                *reinterpret_cast<__bf16*>(dst) = (__bf16)(acc[0] * inv);
            }
            if (lse && d0 == 0)
                lse[(int64_t(b) * a.q_len + t) * a.n_q_heads + hq_row] = den > 0.f ? (m_all + __builtin_amdgcn_logf(den)) * kLn2 : -INFINITY;
        }
    };
    if (a.rows * D <= 64 * W) merge(std::integral_constant<int, 1>{});
    else if (a.rows * D <= 64 * W * 2) merge(std::integral_constant<int, 2>{});
    else merge(std::integral_constant<int, 4>{});
}

// The 16-row kernel over 8-bit caches (E4M3 codes, one power-of-two fp32 scale per key row and per value
// row): half the bytes per token.  Codes become bf16 in registers (exact: 3 mantissa bits) and feed the same
// two bf16 products; the key scale multiplies the score (folded into the softmax scale factor), the value
// scale multiplies the probability before the second product -- both exact, the scales being powers of two.
// Pool layouts [page][head][D/16][slot][16] and [page][head][D][slot] bytes keep the loads contiguous:
//   K: lane (m, g4) reads the 16 bytes d = 64 jj + 16 g4 .. + 15 of key row m: two k-steps' worth (the query
//      fragments use the same assignment of head dims to k-steps)
//   V: lane (m, g4) reads the 16 bytes (all slots) of row d = 16 db + m in page g4: two k-steps' worth
//   scales: the 16 + 16 floats of page g4.
__device__ __forceinline__ bf16x8 e4m3x8_to_bf16(uint32_t lo, uint32_t hi) {
    const bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.f, false), b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.f, true);
    const bf16x2 c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.f, false), d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.f, true);
    bf16x8 r;
    r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
    r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
    return r;
}

template <int D>
__global__ __launch_bounds__(64 * kSplitWaves, 3) void decode_split16_fp8_kernel(DecodeArgs a) {
    constexpr int KS = D / 32, KP = D / 64, DB = D / 16, C16 = D / 16;
    // (cos, sin) of the q_len query positions; after the loop: SplitLds
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float2* s_rot = reinterpret_cast<float2*>(smem_raw);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nc = a.ncs + a.ncr;
    const unsigned bh = blockIdx.x / unsigned(nc);       // (sequence, KV head)
    const int c = unit_of(blockIdx.x, nc);
    const int h = int(bh % unsigned(a.n_kv_heads));
    const int b = int(bh / unsigned(a.n_kv_heads));
    const bool is_src = c < a.ncs;
    const CacheView& cv = is_src ? a.src : a.rsn;
    const int cc = is_src ? c : c - a.ncs;
    const int unit0 = cc * a.chunk;
    // With half the bytes per token, a wave takes 64 tokens (four pages) per step to keep as many bytes in flight
    // as the bf16 kernel does with 32; wave w takes steps w, w + 4, ...  Page ids (four lanes per step, 16 steps at most)
    // are asked for before the length is known, as in Pages16.
    int my_page = cv.page_table[int64_t(b) * cv.max_pages + min(unit0 / kPage + 4 * (kSplitWaves * (lane >> 2) + wave) + (lane & 3), cv.max_pages - 1)];
    my_page = min(max(my_page, 0), cv.n_pages - 1);
    const int len = min(max(is_src ? a.src_len[b] : a.rsn_len[b], 0), cv.max_pages * kPage);
    if (unit0 >= len) return;
    const int n_steps = (min(len - unit0, a.chunk) - 64 * wave + 64 * kSplitWaves - 1) / (64 * kSplitWaves);
    const int tok0 = unit0 + 64 * wave;

    const int n = lane & 15, g4 = lane >> 4;
    const bool valid_row = n < a.rows;
    const int nr = min(n, a.rows - 1);
    const int t_row = nr / a.group;
    const int hq = h * a.group + nr % a.group;
    const int limit = is_src ? len : max(len - a.q_len + t_row + 1, 0);
    const int limit_min = is_src ? len : max(len - a.q_len + 1, 0);
    bf16x2 ones2;
    ones2[0] = (__bf16)1.f;
    ones2[1] = (__bf16)1.f;

    // query fragments: k-step j = 2 jj + u holds head dims 64 jj + 16 g4 + 8 u + e
    bf16x8 qf[KS];
    {
        const uint16_t* qp = a.q + ((int64_t(b) * a.q_len + t_row) * a.n_q_heads + hq) * D;
        if (a.rope) {
            const int len_r = min(max(a.rsn_len[b], 0), a.rsn.max_pages * kPage);
            rope_table_to_lds<D>(s_rot, len_r - a.q_len, a.q_len, rope_frequency<D>(a.freq), 64 * kSplitWaves);
            lds_barrier();
        }
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            const int d0 = 64 * (j >> 1) + 16 * g4 + 8 * (j & 1);
            qf[j] = *reinterpret_cast<const bf16x8*>(qp + d0);
            if (a.rope) {
                // rotation pair of head dim d: (d, d + D/2); both halves come straight from memory
                const bool upper = d0 >= D / 2;
                const bf16x8 other = *reinterpret_cast<const bf16x8*>(qp + (upper ? d0 - D / 2 : d0 + D / 2));
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float2 r = s_rot[t_row * (D / 2) + (upper ? d0 - D / 2 : d0) + e];
                    const float x = float(qf[j][e]), y = float(other[e]);
                    qf[j][e] = (__bf16)(upper ? x * r.x + y * r.y : x * r.x - y * r.y);
                }
            }
        }
    }
    f32x4 o_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o_acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr float kLazyRise = 8.f;
    float m_ref = 0.f, l_run = 0.f;
    bool has_ref = false;

    const int64_t page_k = int64_t(cv.n_kv_heads) * C16 * (kPage * 16);      // bytes
    const int64_t page_v = int64_t(cv.n_kv_heads) * D * kPage;
    const int64_t page_s = int64_t(cv.n_kv_heads) * kPage;                   // floats
    // K: four 16-key sets per step; in set s, key row m = 4 gq + i is slot 4 s + i of page gq, so that afterwards
    //    lane group g4 holds all 16 slots of page g4 (set s, register i -> slot 4 s + i).  Lane (m = n, g4) reads
    //    the 16 bytes d = 64 jj + 16 g4 .. + 15 of its row.
    const int k_page_sel = n >> 2;
    const uint8_t* k_lane = reinterpret_cast<const uint8_t*>(cv.k_pool) + int64_t(h) * C16 * (kPage * 16) + g4 * (kPage * 16) + (n & 3) * 16;
    // V: lane (m = n, g4) reads the whole 16-slot row d = 16 db + m of page g4: slots 0..7 feed the first, 8..15 the
    //    second matrix instruction of the block
    const uint8_t* v_lane = reinterpret_cast<const uint8_t*>(cv.v_pool) + int64_t(h) * D * kPage + n * kPage;
    const int s_lane = h * kPage;

    auto column_max = [&](float x) {
        float a1 = x, b1 = x;
        asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a1), "+v"(b1));
        float a2 = fmaxf(a1, b1), b2 = a2;
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a2), "+v"(b2));
        return fmaxf(a2, b2);
    };

    for (int s = 0; s < n_steps; ++s) {
        int id[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) id[u] = __builtin_amdgcn_readlane(my_page, 4 * s + u);
        const int id_k = k_page_sel == 0 ? id[0] : k_page_sel == 1 ? id[1] : k_page_sel == 2 ? id[2] : id[3];
        const int id_g = g4 == 0 ? id[0] : g4 == 1 ? id[1] : g4 == 2 ? id[2] : id[3];
        const uint8_t* kp = k_lane + int64_t(id_k) * page_k;
        const uint8_t* vp = v_lane + int64_t(id_g) * page_v;
        const int64_t sp = int64_t(id_g) * page_s + s_lane;
        u32x4 k8[4][KP], v8[DB];
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int jj = 0; jj < KP; ++jj) k8[st][jj] = *reinterpret_cast<const u32x4*>(kp + 4 * jj * (kPage * 16) + 4 * st * 16);
#pragma unroll
        for (int db = 0; db < DB; ++db) v8[db] = stream_load(vp + db * 16 * kPage);
        f32x4 ks[4], vs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ks[u] = *reinterpret_cast<const f32x4*>(cv.k_scale + sp + 4 * u);
            vs[u] = *reinterpret_cast<const f32x4*>(cv.v_scale + sp + 4 * u);
        }

        const int first = tok0 + 64 * kSplitWaves * s + 16 * g4;      // token of this lane's slot 0
        f32x4 sc[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            sc[st] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int jj = j >> 1, u = j & 1;
                sc[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e4m3x8_to_bf16(k8[st][jj][2 * u], k8[st][jj][2 * u + 1]), qf[j], sc[st], 0, 0, 0);
            }
        }
        const bool reaches_limit = tok0 + 64 * kSplitWaves * s + 64 > limit_min;      // uniform
        float t[16], vsc[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {                  // slot e = 4 set + register
            t[e] = fmaf(sc[e >> 2][e & 3], ks[e >> 2][e & 3] * a.scale_log2, -m_ref);
            vsc[e] = vs[e >> 2][e & 3];
        }
        if (reaches_limit) {
            // slots past the visible length hold anything (scales included): remove them by index
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                t[e] = first + e < limit ? t[e] : -INFINITY;
                vsc[e] = first + e < len ? vsc[e] : 0.f;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, t[e]);
        if (__any(mx > kLazyRise || (!has_ref && mx > -INFINITY))) {
            const float rise = column_max(mx);
            const bool move = has_ref ? rise > 0.f : rise > -INFINITY;
            const float shift = move ? rise : 0.f;
            const float alpha = has_ref ? __builtin_amdgcn_exp2f(-shift) : 1.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) t[e] -= shift;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) o_acc[db][i] *= alpha;
            m_ref += shift;
            has_ref = has_ref || move;
        }
        bf16x8 pb[2];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const float p0 = __builtin_amdgcn_exp2f(t[e]), p1 = __builtin_amdgcn_exp2f(t[e + 1]);
            bf16x2 p2;
            p2[0] = (__bf16)p0;
            p2[1] = (__bf16)p1;
            l_run = __builtin_amdgcn_fdot2_f32_bf16(p2, ones2, l_run, false);
            pb[e >> 3][e & 7] = (__bf16)(p0 * vsc[e]);
            pb[e >> 3][(e & 7) + 1] = (__bf16)(p1 * vsc[e + 1]);
        }
        u32x4 keep[2];
        keep[0] = keep[1] = u32x4{0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
        if (tok0 + 64 * kSplitWaves * s + 64 > len) {
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    keep[hf][e] = (first + 8 * hf + 2 * e < len ? 0x0000ffffu : 0u) | (first + 8 * hf + 2 * e + 1 < len ? 0xffff0000u : 0u);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const u32x4 vb = __builtin_bit_cast(u32x4, e4m3x8_to_bf16(v8[db][2 * hf], v8[db][2 * hf + 1])) & keep[hf];
                o_acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vb), pb[hf], o_acc[db], 0, 0, 0);
            }
    }

    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    __syncthreads();                                    // everybody is done with the rotations
    const SplitLds<D> sm(smem_raw, a.rows);
    if (valid_row) {
        // lane (n, g4), block db, register i  <->  d = 16 db + 4 g4 + i
        float* po = sm.o + (wave * a.rows + n) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(po + 16 * db + 4 * g4) = o_acc[db];
        if (g4 == 0) {
            sm.m[wave * a.rows + n] = has_ref ? m_ref : -INFINITY;
            sm.l[wave * a.rows + n] = l_tot;
        }
    }
    __syncthreads();
    merge_waves<D>(sm, a, ((int64_t(b) * a.n_kv_heads + h) * nc + c) * a.rows);
}

// Merge of a row's partial results (both merge kernels): log-sum-exp in a fixed order, run-to-run identical.  D / 4 lanes take a
// row, four head dims each, and fetch kMergeBatch partials per memory round trip; a row's partials are dealt out to `splits`
// such groups of the workgroup (merge_splits), whose states meet in LDS.  Bound by the bytes of the partials and by the rate at
// which workgroups start -- a wave per row, fetching 32 (8) partials whether there were that many or not, took 31 us for 16,384
// rows of about 5 partials and 42 us for 65,536 rows of 1 to 3; so 11 and 23.
constexpr int kMergeThreads = 256, kMergeBatch = 8;
template <int D>
struct MergeRow {
    static constexpr int LANES = D / 4, GROUPS = kMergeThreads / LANES;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, den = 0.f;
    // another state of the row: weight 0 for one that holds nothing
    __device__ __forceinline__ void add(float w, float l, const f32x4& o) {
        den = fmaf(w, l, den);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(w, o[e], acc[e]);
    }
    __device__ __forceinline__ bool raise(float to) {
        if (to == -INFINITY) return false;                               // nothing visible so far
        const float alpha = __builtin_amdgcn_exp2f(m - to);
        m = to;
        den *= alpha;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= alpha;
        return true;
    }
    // partials first, first + stride, ... below n_tot; row_of(i): index of partial i's row
    template <typename RowOf>
    __device__ __forceinline__ void fold(const DecodeArgs& a, int first, int stride, int n_tot, int d0, RowOf row_of) {
        for (int i0 = first; i0 < n_tot; i0 += kMergeBatch * stride) {
            f32x2 ml[kMergeBatch];
            f32x4 o[kMergeBatch];
#pragma unroll
            for (int u = 0; u < kMergeBatch; ++u) {
                ml[u] = f32x2{-INFINITY, 0.f};
                o[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (i0 + u * stride < n_tot) {
                    const int64_t row = row_of(i0 + u * stride);
                    ml[u] = *reinterpret_cast<const f32x2*>(a.part_ml + row * 2);
                    o[u] = *reinterpret_cast<const f32x4*>(a.part_o + row * D + d0);
                }
            }
            float top = m;
#pragma unroll
            for (int u = 0; u < kMergeBatch; ++u) top = fmaxf(top, ml[u][0]);
            if (!raise(top)) continue;
#pragma unroll
            for (int u = 0; u < kMergeBatch; ++u) add(__builtin_amdgcn_exp2f(ml[u][0] - top), ml[u][1], o[u]);
        }
    }
    // the states of `splits` neighbouring groups into the first one's (called by every thread of the workgroup)
    __device__ __forceinline__ void meet(int splits) {
        __shared__ f32x4 s_acc[kMergeThreads];
        __shared__ f32x2 s_ml[GROUPS];
        const int group = int(threadIdx.x) / LANES, lane = int(threadIdx.x) % LANES;
        s_acc[threadIdx.x] = acc;
        if (lane == 0) s_ml[group] = f32x2{m, den};
        __syncthreads();
        if (group % splits != 0) return;
        float top = m;
        for (int s = 1; s < splits; ++s) top = fmaxf(top, s_ml[group + s][0]);
        if (!raise(top)) return;
        for (int s = 1; s < splits; ++s)
            add(__builtin_amdgcn_exp2f(s_ml[group + s][0] - top), s_ml[group + s][1], s_acc[(group + s) * LANES + lane]);
    }
    __device__ __forceinline__ void store(uint16_t* out, float* lse, int64_t row, int d0) const {
        const float inv = den > 0.f ? 1.f / den : 0.f;
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (__bf16)(acc[e] * inv);
        *reinterpret_cast<bf16x4*>(out + row * D + d0) = r;
        if (lse && d0 == 0) lse[row] = den > 0.f ? (m + __builtin_amdgcn_logf(den)) * kLn2 : -INFINITY;
    }
};
// Groups per row: as few (a power of two, at most the 8 that a workgroup has at 128 dims) as fetch a row's partials in one round
// trip; a single short unit of a long cache leaves hundreds of partials for a handful of rows.
inline int merge_splits(int n_partials) {
    int splits = 1;
    while (splits < 8 && splits * kMergeBatch < n_partials) splits *= 2;
    return splits;
}
inline int64_t merge_workgroups(int64_t rows, int d, int splits) {
    const int per = kMergeThreads / (d / 4) / splits;
    return (rows + per - 1) / per;
}

template <int D>
__global__ __launch_bounds__(kMergeThreads) void decode_combine_kernel(DecodeArgs a, uint16_t* __restrict__ out,
                                                                       float* __restrict__ lse, int splits) {
    using Row = MergeRow<D>;
    const int group = int(threadIdx.x) / Row::LANES, d0 = int(threadIdx.x) % Row::LANES * 4;
    const int64_t n_rows = int64_t(a.batch) * a.q_len * a.n_q_heads;
    const int64_t mine = int64_t(blockIdx.x) * (Row::GROUPS / splits) + group / splits;
    const unsigned row = unsigned(min(mine, n_rows - 1));
    const int hq = int(row % unsigned(a.n_q_heads));
    const int t = int((row / unsigned(a.n_q_heads)) % unsigned(a.q_len));
    const int b = int(row / (unsigned(a.n_q_heads) * unsigned(a.q_len)));
    const int h = hq / a.group, n = t * a.group + hq % a.group;
    const int nc = a.ncs + a.ncr + a.append;
    const int len_s = min(max(a.src_len[b], 0), a.src.max_pages * kPage);
    const int len_all = min(max(a.rsn_len[b], 0), a.rsn.max_pages * kPage);
    const int n_tok = (a.append && len_all > 0) ? 1 : 0;            // the new token's own partial (slot ncs + ncr)
    const int len_r = len_all - n_tok;                               // what the split kernel walked
    const int n_s = min((len_s + a.chunk - 1) / a.chunk, a.ncs), n_r = min((len_r + a.chunk - 1) / a.chunk, a.ncr);
    const int64_t base = (int64_t(b) * a.n_kv_heads + h) * nc;
    Row r;
    // partial i of the row -> slot: source units, reasoning units, then the token
    r.fold(a, group % splits, splits, n_s + n_r + n_tok, d0, [&](int i) {
        return (base + (i < n_s ? i : i < n_s + n_r ? a.ncs + (i - n_s) : a.ncs + a.ncr)) * a.rows + n;
    });
    if (splits > 1) r.meet(splits);
    if (group % splits == 0 && mine < n_rows) r.store(out, lse, row, d0);
}

// Source-chunk prefill (Alg. 1, prefill loop) with the cache pages SHARED through LDS: one workgroup per
// (sequence, KV head, group of 128 query rows, work unit of the source cache: chunk_units), wave w = the w-th block of
// 32 (token, head) rows.  Per step the four waves copy four pages (64 tokens) of K and of V -- 4 KB each at
// D = 128, verbatim, with asynchronous global -> LDS copies, one step ahead -- and every wave takes its matrix
// operands from there, so a page is fetched from L2 once per workgroup and not once per row block.  The pool
// layout of K is conflict-free as it is (16 slots x 16 bytes contiguous per 8-dim chunk); the 32-byte rows of V
// are not, so the copy swaps the two halves of every second group of 8 rows (by choosing what each lane fetches).
// Softmax as in the prefill kernel (prescaled queries, reference parked in the last score block, no running maximum);
// partial results [B][Hkv][row block][unit][32 rows],
// merged by chunk_combine_kernel.
// Work units of one sequence's source cache: as few as keep a unit within `target` tokens, all of the same length
// (a multiple of 64 tokens) -- equal units finish together, a long one beside a short remainder does not.
struct ChunkUnits {
    int len;      // tokens of the cache
    int size;     // tokens per unit
    int count;    // units
};
__device__ __forceinline__ ChunkUnits chunk_units(int len, int target) {
    ChunkUnits u;
    u.len = len;
    u.count = max((len + target - 1) / target, 1);
    u.size = ((len + u.count - 1) / u.count + 63) & ~63;
    return u;
}
constexpr int kChunkRankMax = 256;

template <int D, int STAGES, int TOK>
struct ChunkSmem {
    uint16_t k[STAGES][TOK * D];
    uint16_t v[STAGES][TOK * D];
};

// TOK tokens (TOK / 16 pages) per step, STAGES buffers of one step each, copies STAGES - 1 steps ahead.
template <int D, int STAGES, int TOK>
__global__ __launch_bounds__(256, 2) void chunk_split_lds_kernel(DecodeArgs a) {
    constexpr int KS = D / 16, DB = D / 32;
    constexpr int PAGE = D * kPage;                   // elements of one page of one head, K or V
    constexpr int NL = PAGE * 2 / 1024;               // 1 KB copies per page
    constexpr int PG = TOK / kPage;                   // pages per step
    constexpr int SBN = TOK / 32;                     // 32-key blocks per step
    constexpr int PER_WAVE = 2 * PG / 4;              // page copies (K or V) per wave and step
    static_assert(TOK == 32 || TOK == 64, "32 or 64 tokens per step");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    ChunkSmem<D, STAGES, TOK>& sm = *reinterpret_cast<ChunkSmem<D, STAGES, TOK>*>(smem_raw);

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rb_groups = (a.row_blocks + 3) / 4;
    const CacheView& cv = a.src;
    // Which unit: the workgroups of a launch are handed out in index order and a unit keeps its compute unit for as
    // long as it has tokens, so the LONGEST units go first -- workgroup index / (heads x row groups) is a rank in the
    // order of decreasing unit length over all (sequence, unit) pairs (ties by index), worked out by every
    // workgroup from the lengths themselves (one entry per thread and pass; kChunkRankMax entries at most, beyond
    // that the units go in index order).
    __shared__ __align__(16) int s_unit_len[kChunkRankMax];
    __shared__ int s_pick;
    const int per_rank = a.n_kv_heads * rb_groups;
    const int rank = int(blockIdx.x / unsigned(per_rank));
    const int hr = int(blockIdx.x % unsigned(per_rank));
    const int h = hr / rb_groups, rbg = hr % rb_groups;
    const int n_entries = a.batch * a.ncs;
    int entry = rank;
    if (n_entries <= kChunkRankMax) {
        const int padded = (n_entries + 3) & ~3;     // (entries past the end: -1, behind every real one)
        for (int e = threadIdx.x; e < padded; e += 256) {
            int tokens = -1;
            if (e < n_entries) {
                const int bb = e / a.ncs, cc = e % a.ncs;
                const ChunkUnits u = chunk_units(min(max(a.src_len[bb], 0), cv.max_pages * kPage), a.chunk);
                tokens = max(min(u.len - cc * u.size, u.size), 0);
            }
            s_unit_len[e] = tokens;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < n_entries; e += 256) {
            const int mine = s_unit_len[e];
            int before = 0;
            for (int o = 0; o < padded; o += 4) {
                const int4 other = *reinterpret_cast<const int4*>(&s_unit_len[o]);
                before += (other.x > mine || (other.x == mine && o < e)) ? 1 : 0;
                before += (other.y > mine || (other.y == mine && o + 1 < e)) ? 1 : 0;
                before += (other.z > mine || (other.z == mine && o + 2 < e)) ? 1 : 0;
                before += (other.w > mine || (other.w == mine && o + 3 < e)) ? 1 : 0;
            }
            if (before == rank) s_pick = e;          // exactly one entry has this rank
        }
        __syncthreads();
        entry = s_pick;
    }
    const int b = __builtin_amdgcn_readfirstlane(entry / a.ncs), c = __builtin_amdgcn_readfirstlane(entry % a.ncs);
    const int len = min(max(a.src_len[b], 0), cv.max_pages * kPage);
    const ChunkUnits units_b = chunk_units(len, a.chunk);
    const int tok0 = c * units_b.size;
    if (tok0 >= len) return;
    const int q_len = min(min(max(a.n_new ? a.n_new[b] : a.max_new, 0), a.max_new), len);
    const int n_rows = q_len * a.group;
    if (rbg * 128 >= n_rows) return;
    // the group's last row sees the most: a chunk past its limit holds nothing for any of its blocks
    const int group_last_t = min(q_len - 1, (rbg * 128 + 127) / a.group);
    if (tok0 >= len - q_len + group_last_t + 1) return;
    const int tok_end = min(len, tok0 + units_b.size);
    const int n_steps = (tok_end - tok0 + TOK - 1) / TOK;

    const int n = lane & 31, hg = lane >> 5;
    const int rb = rbg * 4 + wave;
    const int r = rb * 32 + n;
    const bool valid_row = r < n_rows;
    const int t_row = min(r, n_rows - 1) / a.group;
    const int hq = h * a.group + min(r, n_rows - 1) % a.group;
    // this wave's block: anything to do in this chunk?  (uniform; the wave still copies and meets the barriers)
    const int block_last_t = min(q_len - 1, (rb * 32 + 31) / a.group);
    const bool wave_works = rb * 32 < n_rows && tok0 < len - q_len + block_last_t + 1;
    const int limit = valid_row ? len - q_len + t_row + 1 : 0;                   // row sees tokens [0, limit)
    const int block_first_t = min(q_len - 1, (rb * 32) / a.group);
    const int limit_min = len - q_len + block_first_t + 1;                       // smallest limit of the block's valid rows

    bf16x8 qf[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j)
        qf[j] = *reinterpret_cast<const bf16x8*>(a.q + ((int64_t(b) * a.max_new + t_row) * a.n_q_heads + hq) * D + 16 * j + 8 * hg);
    if (a.rope) {
        // the positions of the group's 128 rows, at most 128 of them: they fit the (still unused) tile buffers exactly
        static_assert(sizeof(ChunkSmem<D, STAGES, TOK>) >= 128 * (D / 2) * sizeof(float2), "rotation table over the tile buffers");
        float2* s_rot = reinterpret_cast<float2*>(smem_raw);
        const int t_first = rbg * 128 / a.group;
        rope_table_to_lds<D>(s_rot, len - q_len + t_first, group_last_t - t_first + 1, rope_frequency<D>(a.freq), 256);
        __syncthreads();
        // (rows past the group's end repeat the last row of the sequence: it is this group's last or a later one)
        rotate_fragments<KS, 16>(qf, 8 * hg, s_rot + (min(t_row, group_last_t) - t_first) * (D / 2));
        __syncthreads();                             // read by everybody before the first copies land
    }
    // queries times scale * log2(e), rounded to bf16 again: K q' is the exponent of the softmax weight
#pragma unroll
    for (int j = 0; j < KS; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[j][e] = (__bf16)(float(qf[j][e]) * a.scale_log2);
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        u32x4 t = __builtin_bit_cast(u32x4, qf[j]);
        asm volatile("" : "+v"(t));
        qf[j] = __builtin_bit_cast(bf16x8, t);
    }

    // Copies.  A step is PG pages of K and PG pages of V; the four waves share them out, PER_WAVE page copies each:
    // copy number x = wave * PER_WAVE + u is page x % PG of K (x < PG) or of V.
    const int32_t* table = cv.page_table + int64_t(b) * cv.max_pages;
    const int last_page = (tok_end - 1) / kPage;                                 // last page that holds visible tokens
    const int64_t page_stride = int64_t(cv.n_kv_heads) * PAGE;
    const uint16_t* k_src = cv.k_pool + int64_t(h) * PAGE;                       // (+ 16 bytes per lane)
    // V rows are 32 bytes: read as they lie, lanes d and d + 8 of a 16-lane group would meet in the same banks.  A copy
    // places lane l's 16 bytes at position l, but WHICH 16 bytes a lane fetches is free: position 2 d + x holds the
    // half x ^ bit 3 of d of row d, and the readers below undo that.
    const int v_perm = (lane & ~1) | ((lane & 1) ^ ((lane >> 4) & 1));           // chunk fetched by this lane (same for every 1 KB piece: 32 rows)
    const uint16_t* v_src = cv.v_pool + int64_t(h) * PAGE;                       // (+ 16 bytes per fetched chunk)
    const uint32_t k_lane_off = uint32_t(lane) * 16u, v_lane_off = uint32_t(v_perm) * 16u;
    const uint32_t lds_k = uint32_t(uintptr_t(&sm.k[0][0])), lds_v = uint32_t(uintptr_t(&sm.v[0][0]));
    // the page ids of the whole unit, fetched once (up to 256 pages: four per lane): a load per step would make
    // every step wait for a round trip to memory, and for all copies in flight with it
    int my_pages[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int id = table[min(tok0 / kPage + 64 * u + lane, last_page)];
        my_pages[u] = min(max(id, 0), cv.n_pages - 1);
    }
    auto issue = [&](int s, int stage) {
        s = min(s, n_steps - 1);                                                 // past the last step: the same pages again, never used
#pragma unroll
        for (int w = 0; w < PER_WAVE; ++w) {
            const int x = wave * PER_WAVE + w;                                   // (uniform)
            const bool is_v = x >= PG;
            const int pg = is_v ? x - PG : x;
            const int pl = min(PG * s + pg, last_page - tok0 / kPage);          // pages past the end: the last one again (masked)
            const int quarter = pl >> 6;
            const int held = quarter == 0 ? my_pages[0] : quarter == 1 ? my_pages[1] : quarter == 2 ? my_pages[2] : my_pages[3];
            const int id = __builtin_amdgcn_readlane(held, pl & 63);
            const uint16_t* src = (is_v ? v_src : k_src) + int64_t(id) * page_stride;
            const uint32_t dst = (is_v ? lds_v : lds_k) + uint32_t(stage) * (TOK * D * 2) + uint32_t(pg) * (PAGE * 2);
            async_copy_rows_nt<NL>(src, is_v ? v_lane_off : k_lane_off, dst);        // read once: 2 % faster with the hint
        }
    };
    // The chunk streams from HBM (about 125 flop per byte: below the ridge of this machine), so the bytes in flight
    // matter: copies run STAGES - 1 steps ahead.  Every iteration issues exactly one step's copies (clamped at the
    // end), which keeps the count the waits rely on.
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s, s);

    f32x16 o_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[db][i] = 0.f;
    constexpr float kRise = 16777216.f;               // 2^24
    float m_ref = 0.f, l_run = 0.f;
    bool has_ref = false;
    // operand addresses inside a stage (elements): K lane (m = n, hg): page n / 16 of the 32-key block, slot
    // swap23(n % 16), chunk 2 j + hg; V lane (m = n, hg): row 32 db + n, slots 8 hg .. + 7 of page t (halves swapped
    // for every second group of 8 rows, see above)
    const int k_off = (n >> 4) * PAGE + swap23(n & 15) * 8 + hg * (kPage * 8);
    const int v_off = n * kPage + 8 * (hg ^ ((n >> 3) & 1));
    // Score blocks of a step.  Between steps the LAST one holds -m_ref of this lane's row in all sixteen registers:
    // the first matrix instruction of every block takes it as its accumulator input (the last block in place, after
    // the others have read it), so the scores come out relative to the reference without a subtraction.
    f32x16 s_acc[SBN];
#pragma unroll
    for (int i = 0; i < 16; ++i) s_acc[SBN - 1][i] = 0.f;

    int stage = 0;
    for (int s = 0; s < n_steps; ++s) {
        wait_vmcnt<(STAGES - 2) * PER_WAVE * NL>();   // step s has landed (the STAGES - 2 younger ones may still fly) ...
        __syncthreads();                              // ... for every wave; and everybody is done with step s - 1,
        issue(s + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);              // whose buffer the next copies take
        const uint16_t* kb = &sm.k[stage][0];
        const uint16_t* vb = &sm.v[stage][0];
        stage = stage == STAGES - 1 ? 0 : stage + 1;
        const int tok = tok0 + TOK * s;
        if (!wave_works || tok >= len - q_len + block_last_t + 1) continue;      // (uniform) nothing for this block here
        // operands leave LDS ahead of the matrix instructions that take them: all key fragments now, all value
        // fragments before the exponentials (scheduling barriers keep the compiler from moving them back)
        bf16x8 fk[SBN * KS];
#pragma unroll
        for (int f = 0; f < SBN * KS; ++f)
            fk[f] = *reinterpret_cast<const bf16x8*>(kb + 2 * (f % SBN) * PAGE + k_off + 2 * (f / SBN) * (kPage * 8));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < SBN * KS; ++f)
            s_acc[f % SBN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[f], qf[f / SBN], f < SBN ? s_acc[SBN - 1] : s_acc[f % SBN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        u32x4 fv[PG * DB];
        auto load_v = [&](int f0, int f1) {
#pragma unroll
            for (int f = f0; f < f1; ++f)
                fv[f] = *reinterpret_cast<const u32x4*>(vb + (f / DB) * PAGE + 32 * (f % DB) * kPage + v_off);
        };
        load_v(0, PG * DB / 2);
        __builtin_amdgcn_sched_barrier(0);
        // block sb, register i  <->  token tok + 32 sb + 16 (i/8) + 8 hg + i%8.  The scores leave the matrix pipe as
        // exponents relative to the row's reference (queries prescaled, -m_ref where the accumulators start).
        const bool masked = tok + TOK > limit_min || !valid_row;                 // (uniform up to the row validity)
        if (masked) {
#pragma unroll
            for (int sb = 0; sb < SBN; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    s_acc[sb][i] = tok + 32 * sb + 16 * (i >> 3) + 8 * hg + (i & 7) < limit ? s_acc[sb][i] : -INFINITY;
        }
        bf16x8 pb[PG];
        float psum;
        auto weights = [&]() {
            psum = 0.f;
#pragma unroll
            for (int sb = 0; sb < SBN; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float p = __builtin_amdgcn_exp2f(s_acc[sb][i]);
                    psum += p;
                    pb[2 * sb + (i >> 3)][i & 7] = (__bf16)p;
                }
        };
        // No running maximum: the reference only moves when a row has none yet, or when a step's weights say that
        // the scores have risen far above it (their sum beyond 2^24, overflow included).
        bool slow = __any(!has_ref && limit > tok);
        if (!slow) {
            weights();
            slow = __any(!(psum <= kRise));
        }
        if (slow) {
            // out of line: move the reference of the rows that need it (a row lives in lanes n and n + 32)
            float mx = -INFINITY;
#pragma unroll
            for (int sb = 0; sb < SBN; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s_acc[sb][i]);
            const float rise = fmaxf(mx, __shfl_xor(mx, 32));
            const bool move = has_ref ? rise > 0.f : rise > -INFINITY;
            const float shift = move ? rise : 0.f;
            const float alpha = has_ref ? __builtin_amdgcn_exp2f(-shift) : 1.f;
#pragma unroll
            for (int sb = 0; sb < SBN; ++sb)
#pragma unroll
                for (int i = 0; i < 16; ++i) s_acc[sb][i] -= shift;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o_acc[db][i] *= alpha;
            m_ref += shift;
            has_ref = has_ref || move;
            weights();
        }
        __builtin_amdgcn_sched_barrier(0);
        load_v(PG * DB / 2, PG * DB);
        __builtin_amdgcn_sched_barrier(0);
        // the last score block is where the next step's accumulators start: -m_ref again
#pragma unroll
        for (int i = 0; i < 16; ++i) s_acc[SBN - 1][i] = -m_ref;
        l_run += psum;
        if (tok + TOK > len) {                                                   // (uniform) the step that holds the end of the cache
            // slots past the visible length may hold anything (0 x NaN): remove them by bit mask
#pragma unroll
            for (int t4 = 0; t4 < PG; ++t4) {
                u32x4 keep;
                const int first = tok + 16 * t4 + 8 * hg;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    keep[e] = (first + 2 * e < len ? 0x0000ffffu : 0u) | (first + 2 * e + 1 < len ? 0xffff0000u : 0u);
#pragma unroll
                for (int db = 0; db < DB; ++db) fv[t4 * DB + db] &= keep;
            }
        }
#pragma unroll
        for (int t4 = 0; t4 < PG; ++t4)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fv[t4 * DB + db]), pb[t4], o_acc[db], 0, 0, 0);
    }
    wait_vmcnt<0>();
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (!valid_row || !wave_works) return;
    const int64_t slot = (((int64_t(b) * a.n_kv_heads + h) * a.row_blocks + rb) * a.ncs + c) * 32 + n;
    float* po = a.part_o + slot * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            f32x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = o_acc[db][4 * q4 + e];
            *reinterpret_cast<f32x4*>(po + 32 * db + 8 * q4 + 4 * hg) = o4;
        }
    if (hg == 0) {
        a.part_ml[slot * 2] = has_ref ? m_ref : -INFINITY;
        a.part_ml[slot * 2 + 1] = l_tot;
    }
}

// Merge for the source-chunk prefill; rows past n_new[b] are left untouched.
template <int D>
__global__ __launch_bounds__(kMergeThreads) void chunk_combine_kernel(DecodeArgs a, uint16_t* __restrict__ out,
                                                                      float* __restrict__ lse, int splits) {
    using Row = MergeRow<D>;
    const int group = int(threadIdx.x) / Row::LANES, d0 = int(threadIdx.x) % Row::LANES * 4;
    const int64_t n_rows = int64_t(a.batch) * a.max_new * a.n_q_heads;
    const int64_t mine = int64_t(blockIdx.x) * (Row::GROUPS / splits) + group / splits;
    const unsigned row = unsigned(min(mine, n_rows - 1));
    const int hq = int(row % unsigned(a.n_q_heads));
    const int t = int((row / unsigned(a.n_q_heads)) % unsigned(a.max_new));
    const int b = int(row / (unsigned(a.n_q_heads) * unsigned(a.max_new)));
    const int len = min(max(a.src_len[b], 0), a.src.max_pages * kPage);
    const int q_len = min(min(max(a.n_new ? a.n_new[b] : a.max_new, 0), a.max_new), len);
    const int h = hq / a.group;
    const int rr = t * a.group + hq % a.group, rb = rr / 32, n = rr % 32;
    const int last_t = min(q_len - 1, (rb * 32 + 31) / a.group);
    const int unit_size = chunk_units(len, a.chunk).size;
    // units the split kernel wrote for this block
    const int n_tot = t < q_len ? min((len - q_len + last_t + 1 + unit_size - 1) / unit_size, a.ncs) : 0;
    const int64_t base = ((int64_t(b) * a.n_kv_heads + h) * a.row_blocks + rb) * a.ncs;
    Row r;
    r.fold(a, group % splits, splits, n_tot, d0, [&](int i) { return (base + i) * 32 + n; });
    if (splits > 1) r.meet(splits);
    if (group % splits == 0 && mine < n_rows && t < q_len) r.store(out, lse, row, d0);
}

static inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
static inline int chunks_of(int len) { return (len + kChunk - 1) / kChunk; }

// Partial results of a decode step cut into `unit`-token work units.
static inline size_t decode_partial_bytes(int unit, int64_t batch, int hkv, int rows, int d, int max_src, int max_rsn) {
    const size_t nc = size_t((max_src + unit - 1) / unit) + size_t((max_rsn + unit - 1) / unit) + 1;   // + the appended token's slot
    const size_t slots = size_t(batch) * hkv * nc * rows;
    return align256(slots * d * sizeof(float)) + align256(slots * 2 * sizeof(float)) + 256;
}
// Short caches: one workgroup per (sequence, KV head) does everything (no partial results, no merge launch).  With heads of 64 dims
// that wins up to 1,024 tokens at every batch (one sequence, 16 / 8 heads, 900 tokens: 6.9 us against 7.8 replayed from a graph,
// 7.7 against 10.2 launched one by one).  With heads of 128 a wave's chain of steps is longer, and up to 40 workgroups leave the
// chip idle: there the split and its second launch win from some 832 tokens on (32 / 8 heads, 4 sequences: 640 tokens 8.1 here,
// 11.0 split; 832 tokens 11.0, 10.9; 1,024 tokens 12.6, 11.2; launched one by one 8.4 / 12.1, 10.9 / 11.9, 12.3 / 12.0); from 48
// workgroups on they don't (6 sequences, 1,024 tokens 12.5 / 12.9; 16: 16.0 / 21.4).
static inline bool small_decode(int64_t batch, int hkv, int d, int max_src, int max_rsn) {
    return max_src + max_rsn <= (d == 128 && batch * hkv <= 40 ? 832 : kSmallDecodeTokens);
}

// Tokens per work unit of a split kernel's workgroup.  Every unit pays a prologue (a chain of memory round trips, microseconds
// each under load) and a partial result, so a unit is as long as still leaves enough of them to fill the chip (512 workgroups
// at a time) and to end evenly: the longest of 4,096 .. 1,024 tokens that gives, with the length BOUNDS (about half the units
// they give are real), 2,048 units -- us per layer, 16 / 8 heads of 128 dims: 64 sequences of up to 24K tokens 622 with 2,048
// against 777 with 512; 16 of up to 16K 134 with 1,024 against 141 with 512; 48 of 2K 73 with 512 against 91 with 1,024.  Where
// a partial result weighs more or a token less, fewer units are enough: 384 with 9 to 16 query rows (24 sequences of 2K + 2K
// tokens, 32 / 8 heads of 128 dims 68 with 2,048 against 76 with 512), 768 for 8-bit caches (32 sequences of up to 8K tokens 82 with 2,048
// against 88 with 512), 192 of 4,096 tokens with 17 to 32 rows (8 sequences of up to 12K tokens 63 against 67 with 512; 32 of
// them 214 against 264).  And one whose workgroups are alike: the units of a head together (none counted longer than the longer
// cache) no more than a fifth longer than its caches.  A cache a little longer than a unit, or than the other cache, makes a
// long and a short workgroup, and the launch ends with the long ones -- 64 sequences of 5K + 5K tokens, 8 heads of 128 dims
// 455 with 4,096, 398 with 1,024; 8-bit, 32 / 8 heads 271 and 228; 20 of 3,000 + 900 tokens, 16 rows 78 with 4,096, 60 with 1,024;
// but 64 of 700 + 700, 16 rows 85 with 512, 69 with a unit for each cache.  (Only the bounds are known here: a few long caches among
// many short ones would take longer units, 128 of 300 tokens with one of 12,000 72 with 4,096 against 97.)
// A few sequences are bound by the walk over a unit and not by bandwidth: 256 tokens up to 256 units of 512 (one sequence of 4K
// tokens: 13.5 against 15.3), 128 up to 32 units (2K tokens: 11.7 against 15.3).
static inline int decode_unit_tokens(int64_t batch, int hkv, int rows, int max_src, int max_rsn, int pinned, bool fp8 = false) {
    if (pinned) return pinned;               // the caller's choice (st_dual_lens::unit_tokens)
    auto per_head = [&](int unit) { return int64_t((max_src + unit - 1) / unit) + (max_rsn + unit - 1) / unit; };
    auto units = [&](int unit) { return batch * hkv * per_head(unit); };
    auto even = [&](int unit) { return 5 * per_head(unit) * std::min(unit, std::max(max_src, max_rsn)) <= 6 * (int64_t(max_src) + max_rsn); };
    if (rows > 16 && units(kChunkLong) >= 192) return kChunkLong;
    const int64_t enough = rows > 8 ? 384 : fp8 ? 768 : 2048;
    for (int unit = kChunkLong; unit > kChunk; unit /= 2)
        if (units(unit) >= enough && even(unit)) return unit;
    return units(kChunk) > 256 ? kChunk : units(kChunk) > 32 ? kChunk / 2 : kChunkMin;
}

}  // namespace st

using namespace st;

static inline bool valid_unit(int tokens) { return tokens == 0 || tokens == 128 || tokens == 256 || tokens == 512 || tokens == 1024; }

extern "C" size_t st_decode_workspace_bytes(int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                            int32_t q_len, int32_t max_src_len, int32_t max_rsn_len, int32_t unit_tokens) {
    if (batch <= 0 || n_q_heads <= 0 || n_kv_heads <= 0 || q_len <= 0 || head_dim <= 0 || max_src_len < 0 || max_rsn_len < 0 ||
        !valid_unit(unit_tokens))
        return 0;
    const int rows = q_len * (n_q_heads / n_kv_heads);
    // enough for 512-token units whatever the bounds of a later call, and for the unit this very call would use
    const size_t base = decode_partial_bytes(kChunk, batch, n_kv_heads, rows, head_dim, max_src_len, max_rsn_len);
    // (few sequences: for the shortest unit, which shorter caches than these may get in a later call)
    int unit = decode_unit_tokens(batch, n_kv_heads, rows, max_src_len, max_rsn_len, unit_tokens);
    if (!unit_tokens && unit < kChunk) unit = kChunkMin;
    const size_t own = decode_partial_bytes(unit, batch, n_kv_heads, rows, head_dim, max_src_len, max_rsn_len);
    return base > own ? base : own;
}

// ---- the decode step for callers that cannot allocate: partial results in a device array of the library ----
// One copy of `scratch` exists on every GPU the library's code object is loaded on, at an address of its own; in host
// code the array's NAME is only a stand-in for it, so its device address is looked up once per device
// (hipGetSymbolAddress, with that device current) and only that pointer is ever handed to kernels.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the CURRENT device (looked up at the first call on that device).
static st_status static_scratch(void** ptr) {
    int dev = -1;
    ST_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual_static: device index %d (0 .. %d)", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        ST_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return fail(ST_ERR_RUNTIME, "st_attn_decode_dual_static: bad address of the scratch array");
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return ST_OK;
}

static st_status decode_dual_impl(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                  const st_dual_lens* lens, int32_t batch, int32_t n_q_heads, float scale, bool rotate,
                                  double theta_base, void* workspace, size_t workspace_bytes, void* hip_stream,
                                  const void* k_new = nullptr, const void* v_new = nullptr, bool append = false, bool no_alloc = false) {
    if (!out || !q || !caches || !lens) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: null pointer");
    if (append) {
        if (!k_new || !v_new) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_append: null pointer");
        if (!aligned16(k_new) || !aligned16(v_new)) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_append: k_new / v_new must be 16-byte aligned");
        if (lens->q_len != 1) return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual_append: one token per step (q_len %d)", lens->q_len);
        if (caches->source.dtype != ST_BF16 || caches->reasoning.dtype != ST_BF16)
            return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual_append: bf16 caches only");
        if (!caches->reasoning.appended_len) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_append: appended_len is null");
    }
    if (!lens->src_visible_len || !lens->rsn_len) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: null length vector");
    if (!aligned16(out) || !aligned16(q)) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: q / out must be 16-byte aligned");
    st_status r = check_cache(caches->source, "st_attn_decode_dual", "source", true);
    if (r != ST_OK) return r;
    r = check_cache(caches->reasoning, "st_attn_decode_dual", "reasoning", true);
    if (r != ST_OK) return r;
    const st_kv_cache& cs = caches->source;
    const st_kv_cache& cr = caches->reasoning;
    if (cs.n_kv_heads != cr.n_kv_heads || cs.head_dim != cr.head_dim)
        return fail(ST_ERR_SHAPE, "st_attn_decode_dual: the two caches differ in head geometry");
    if (cs.dtype != cr.dtype) return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual: the two caches differ in dtype");
    const bool fp8 = cs.dtype == ST_FP8_E4M3;
    const int hkv = cs.n_kv_heads, d = cs.head_dim;
    if (batch <= 0 || n_q_heads <= 0 || n_q_heads % hkv != 0)
        return fail(ST_ERR_SHAPE, "st_attn_decode_dual: n_q_heads %d must be a positive multiple of n_kv_heads %d", n_q_heads, hkv);
    const int group = n_q_heads / hkv;
    if (lens->q_len <= 0 || lens->q_len * group > 32)
        return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual: q_len %d x group %d must be in 1..32", lens->q_len, group);
    if (fp8 && lens->q_len * group > 16)
        return fail(ST_ERR_UNSUPPORTED, "st_attn_decode_dual: 8-bit caches take q_len %d x group %d up to 16", lens->q_len, group);
    if (lens->max_src_len < 0 || lens->max_rsn_len < 0) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: negative length bound");
    if (!valid_unit(lens->unit_tokens)) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: unit_tokens %d (0, 128, 256, 512 or 1024)", lens->unit_tokens);
    if (int64_t(lens->max_src_len) > int64_t(cs.max_pages_per_seq) * kPage || int64_t(lens->max_rsn_len) > int64_t(cr.max_pages_per_seq) * kPage)
        return fail(ST_ERR_CAPACITY, "st_attn_decode_dual: length bound exceeds the page table");
    const size_t need = decode_partial_bytes(kChunk, batch, hkv, lens->q_len * group, d, lens->max_src_len, lens->max_rsn_len);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual: workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < need) return fail(ST_ERR_CAPACITY, "st_attn_decode_dual: workspace has %zu bytes, needs %zu", workspace_bytes, need);
    if (scale <= 0.f) scale = 1.f / sqrtf(float(d));

    DecodeArgs a;
    a.src = cache_view(cs);
    a.rsn = cache_view(cr);
    a.src_len = lens->src_visible_len;
    a.rsn_len = lens->rsn_len;
    a.q = static_cast<const uint16_t*>(q);
    a.batch = batch;
    a.q_len = lens->q_len;
    a.n_q_heads = n_q_heads;
    a.n_kv_heads = hkv;
    a.group = group;
    a.rows = lens->q_len * group;
    // Work unit: see decode_unit_tokens; a workspace sized for other length bounds may only hold longer units.
    a.chunk = decode_unit_tokens(batch, hkv, a.rows, lens->max_src_len, lens->max_rsn_len, lens->unit_tokens, fp8);
    while (a.chunk < kChunk && decode_partial_bytes(a.chunk, batch, hkv, a.rows, d, lens->max_src_len, lens->max_rsn_len) > workspace_bytes)
        a.chunk *= 2;
    a.ncs = (lens->max_src_len + a.chunk - 1) / a.chunk;
    a.ncr = (lens->max_rsn_len + a.chunk - 1) / a.chunk;
    a.scale_log2 = scale * kLog2e;
    a.n_new = nullptr;
    a.max_new = lens->q_len;
    a.row_blocks = 1;
    a.rope = rotate ? 1 : 0;
    a.freq = rotate ? make_rope_freq(theta_base, d) : RopeFreq{};
    // long caches: the 16-row split kernel stores the token itself (one more slot per sequence and head); the
    // 32-row kernel does not, the token then goes in with a launch of its own
    const bool fuse_token = append && !fp8 && a.rows <= 16;
    a.append = fuse_token ? 1 : 0;
    a.k_new = static_cast<const uint16_t*>(k_new);
    a.v_new = static_cast<const uint16_t*>(v_new);
    {
        const WaveTrace wt = no_alloc ? WaveTrace{nullptr, 0} : prof_wave_trace();
        a.trace = wt.buf;
        a.trace_cap = wt.capacity;
    }
    const size_t slots = size_t(batch) * hkv * size_t(a.ncs + a.ncr + a.append) * a.rows;
    a.part_o = static_cast<float*>(workspace);
    a.part_ml = reinterpret_cast<float*>(static_cast<char*>(workspace) + align256(slots * d * sizeof(float)));

    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (!fp8 && a.rows <= 16 && small_decode(batch, hkv, d, lens->max_src_len, lens->max_rsn_len) && int64_t(batch) * hkv <= 0x7fffffff) {
        const size_t smem = (size_t(kSmallWaves + (append ? 1 : 0)) * a.rows * (d + 2) + size_t(a.q_len) * d) * sizeof(float);
        auto launch = [&](auto kernel) -> st_status {
            if (smem > 64 * 1024)                       // beyond the default limit (16 rows of 128 dims only)
                ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem)));
            hipLaunchKernelGGL(kernel, dim3((unsigned)(batch * hkv)), dim3(64 * kSmallWaves), smem, s, a, static_cast<uint16_t*>(out), lse,
                               static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new));
            return ST_OK;
        };
        const st_status lr = d == 64 ? (append ? launch(decode_small16_kernel<64, true>) : launch(decode_small16_kernel<64, false>))
                                     : (append ? launch(decode_small16_kernel<128, true>) : launch(decode_small16_kernel<128, false>));
        if (lr != ST_OK) return lr;
        ST_LAUNCH_CHECK("decode_small16_kernel");
        return ST_OK;
    }
    if (append && !fuse_token) {
        // the token goes in with a launch of its own, then the step below reads it like any other
        const st_status ar = append_token_at(cr, k_new, v_new, lens->rsn_len, batch, rotate, theta_base, s);
        if (ar != ST_OK) return ar;
    }
    const int64_t units = int64_t(batch) * hkv * (a.ncs + a.ncr + a.append);
    const int64_t out_units = int64_t(batch) * a.q_len * n_q_heads;
    if (units > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_decode_dual: grid too large");
    if (units > 0) {
        // (bytes of the launch from the length bounds: about half are real)
        const double bound_bytes = double(batch) * hkv * (double(lens->max_src_len) + lens->max_rsn_len) * 4.0 * d;
        const bool stream_keys = bound_bytes <= 4.0e9;
        auto go = [&](void (*kern)(DecodeArgs), size_t smem) {
            hipLaunchKernelGGL(kern, dim3((unsigned)units), dim3(64 * kSplitWaves), smem, s, a);
        };
        if (a.rows <= 16) {
            if (!no_alloc) prof_begin(kProfDecodeSplit, s);      // (the timing hooks create events)
            for (int rep = 0, n_rep = no_alloc ? 1 : prof_repeat(); rep < n_rep; ++rep)
            if (fp8) go(d == 64 ? decode_split16_fp8_kernel<64> : decode_split16_fp8_kernel<128>, split16_lds_bytes(a.rows, a.q_len, d));
            else if (d == 64) go(stream_keys ? decode_split16_kernel<64, true> : decode_split16_kernel<64, false>, split16_lds_bytes(a.rows, a.q_len, d));
            else go(stream_keys ? decode_split16_kernel<128, true> : decode_split16_kernel<128, false>, split16_lds_bytes(a.rows, a.q_len, d));
            if (!no_alloc) prof_end(kProfDecodeSplit, s);
        } else {
            const size_t smem = split32_lds_bytes(a.rows, a.q_len, d);
            auto kern = d == 64 ? (stream_keys ? decode_split32_kernel<64, true> : decode_split32_kernel<64, false>)
                                : (stream_keys ? decode_split32_kernel<128, true> : decode_split32_kernel<128, false>);
            if (smem > 64 * 1024)                       // beyond the default limit (32 rows of 128 dims)
                ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem)));
            go(kern, smem);
        }
        ST_LAUNCH_CHECK("decode_split_kernel");
    }
    if (out_units > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_decode_dual: grid too large");
    const int splits = merge_splits(a.ncs + a.ncr + a.append);
    const dim3 merge_grid((unsigned)merge_workgroups(out_units, d, splits));
    if (d == 64) hipLaunchKernelGGL((decode_combine_kernel<64>), merge_grid, dim3(kMergeThreads), 0, s, a, static_cast<uint16_t*>(out), lse, splits);
    else hipLaunchKernelGGL((decode_combine_kernel<128>), merge_grid, dim3(kMergeThreads), 0, s, a, static_cast<uint16_t*>(out), lse, splits);
    ST_LAUNCH_CHECK("decode_combine_kernel");
    return ST_OK;
}

extern "C" st_status st_attn_decode_dual(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                         const st_dual_lens* lens, int32_t batch, int32_t n_q_heads, float scale,
                                         void* workspace, size_t workspace_bytes, void* hip_stream) {
    return decode_dual_impl(out, lse, q, caches, lens, batch, n_q_heads, scale, false, 0.0, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t st_decode_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" st_status st_attn_decode_dual_static(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                                const st_dual_lens* lens, int32_t batch, int32_t n_q_heads, float scale,
                                                void* hip_stream) {
    if (!caches || !lens) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_static: null pointer");
    const int hkv = caches->source.n_kv_heads, d = caches->source.head_dim;
    if (batch <= 0 || n_q_heads <= 0 || hkv <= 0 || d <= 0 || n_q_heads % hkv != 0 || lens->q_len <= 0 || lens->max_src_len < 0 || lens->max_rsn_len < 0)
        return fail(ST_ERR_SHAPE, "st_attn_decode_dual_static: bad sizes");
    // what st_attn_decode_dual asks of a workspace for these bounds (partials of 512-token units) must fit the array
    const size_t need = decode_partial_bytes(kChunk, batch, hkv, lens->q_len * (n_q_heads / hkv), d, lens->max_src_len, lens->max_rsn_len);
    if (need > kStaticScratchBytes)
        return fail(ST_ERR_CAPACITY, "st_attn_decode_dual_static: the step needs %zu bytes of partial results, the library's array holds %zu; use st_attn_decode_dual with a workspace", need, kStaticScratchBytes);
    void* ws = nullptr;
    const st_status r = static_scratch(&ws);
    if (r != ST_OK) return r;
    // Nothing in the array has to start at zero: the split kernel writes every partial the merge kernel reads in the
    // same call (both walk the same units of the same lengths), so what an earlier call left is never looked at.
    return decode_dual_impl(out, lse, q, caches, lens, batch, n_q_heads, scale, false, 0.0, ws, kStaticScratchBytes, hip_stream,
                            nullptr, nullptr, false, /*no_alloc=*/true);
}

extern "C" st_status st_attn_decode_dual_rope(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                              const st_dual_lens* lens, int32_t batch, int32_t n_q_heads, float scale,
                                              double theta_base, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!(theta_base > 0.0)) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_rope: theta_base must be positive");
    return decode_dual_impl(out, lse, q, caches, lens, batch, n_q_heads, scale, true, theta_base, workspace, workspace_bytes,
                            hip_stream);
}

extern "C" st_status st_attn_decode_dual_append(void* out, float* lse, const void* q, const void* k_new, const void* v_new,
                                                const st_dual_cache* caches, const st_dual_lens* lens, int32_t batch,
                                                int32_t n_q_heads, float scale, double theta_base, void* workspace,
                                                size_t workspace_bytes, void* hip_stream) {
    if (theta_base < 0.0 || theta_base != theta_base) return fail(ST_ERR_INVALID_ARG, "st_attn_decode_dual_append: theta_base must be positive, or 0 for rotated inputs");
    return decode_dual_impl(out, lse, q, caches, lens, batch, n_q_heads, scale, theta_base > 0.0, theta_base, workspace, workspace_bytes,
                            hip_stream, k_new, v_new, true);
}

extern "C" size_t st_source_chunk_workspace_bytes(int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                                  int32_t max_new, int32_t max_src_len) {
    if (batch <= 0 || n_q_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0 || max_new <= 0 || max_src_len < 0) return 0;
    const size_t rb = (size_t(max_new) * (n_q_heads / n_kv_heads) + 31) / 32;
    const size_t slots = size_t(batch) * n_kv_heads * rb * size_t(chunks_of(max_src_len)) * 32;
    return align256(slots * head_dim * sizeof(float)) + align256(slots * 2 * sizeof(float)) + 256;
}

static st_status source_chunk_impl(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                   const int32_t* src_len, const int32_t* n_new, int32_t max_new,
                                   int32_t max_src_len, int32_t batch, int32_t n_q_heads, float scale, bool rotate,
                                   double theta_base, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!out || !q || !caches || !src_len) return fail(ST_ERR_INVALID_ARG, "st_attn_source_chunk: null pointer");
    if (!aligned16(out) || !aligned16(q)) return fail(ST_ERR_INVALID_ARG, "st_attn_source_chunk: q / out must be 16-byte aligned");
    st_status r = check_cache(caches->source, "st_attn_source_chunk", "source");
    if (r != ST_OK) return r;
    const st_kv_cache& cs = caches->source;
    const int hkv = cs.n_kv_heads, d = cs.head_dim;
    if (batch <= 0 || n_q_heads <= 0 || n_q_heads % hkv != 0)
        return fail(ST_ERR_SHAPE, "st_attn_source_chunk: n_q_heads %d must be a positive multiple of n_kv_heads %d", n_q_heads, hkv);
    if (max_new <= 0 || max_src_len < 0) return fail(ST_ERR_INVALID_ARG, "st_attn_source_chunk: bad sizes");
    if (int64_t(max_src_len) > int64_t(cs.max_pages_per_seq) * kPage)
        return fail(ST_ERR_CAPACITY, "st_attn_source_chunk: length bound exceeds the page table");
    const size_t need = st_source_chunk_workspace_bytes(batch, n_q_heads, hkv, d, max_new, max_src_len);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return fail(ST_ERR_INVALID_ARG, "st_attn_source_chunk: workspace must be non-null and 256-byte aligned");
    if (workspace_bytes < need) return fail(ST_ERR_CAPACITY, "st_attn_source_chunk: workspace has %zu bytes, needs %zu", workspace_bytes, need);
    if (scale <= 0.f) scale = 1.f / sqrtf(float(d));

    DecodeArgs a;
    a.src = cache_view(cs);
    a.rsn = a.src;                       // unused: there are no reasoning chunk slots
    a.src_len = src_len;
    a.rsn_len = src_len;
    a.q = static_cast<const uint16_t*>(q);
    a.batch = batch;
    a.q_len = max_new;
    a.n_q_heads = n_q_heads;
    a.n_kv_heads = hkv;
    a.group = n_q_heads / hkv;
    a.rows = 32;
    // Work unit: 512 tokens of the cache; longer ones when that still leaves a thousand workgroups or more --
    // a unit's partial result (128 rows x D floats) is written and merged once per unit.  (The workspace is
    // sized for the smallest unit.)
    a.chunk = kChunk;
    {
        const int64_t groups = int64_t(batch) * hkv * ((int64_t(max_new) * (n_q_heads / hkv) + 127) / 128);
        for (int unit = 8 * kChunk; unit > kChunk; unit /= 2)
            if (groups * ((max_src_len + unit - 1) / unit) >= 1024) {
                a.chunk = unit;
                break;
            }
    }
    a.ncs = (max_src_len + a.chunk - 1) / a.chunk;
    a.ncr = 0;
    a.append = 0;
    a.k_new = a.v_new = nullptr;
    a.trace = nullptr;
    a.trace_cap = 0;
    a.scale_log2 = scale * kLog2e;
    a.n_new = n_new;
    a.max_new = max_new;
    a.row_blocks = (max_new * a.group + 31) / 32;
    a.rope = rotate ? 1 : 0;
    a.freq = rotate ? make_rope_freq(theta_base, d) : RopeFreq{};
    const size_t slots = size_t(batch) * hkv * a.row_blocks * size_t(a.ncs) * 32;
    a.part_o = static_cast<float*>(workspace);
    a.part_ml = reinterpret_cast<float*>(static_cast<char*>(workspace) + align256(slots * d * sizeof(float)));

    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int64_t units = int64_t(batch) * hkv * a.row_blocks * a.ncs;
    const int64_t out_units = int64_t(batch) * max_new * n_q_heads;
    if (units / 4 + 1 > 0x7fffffff || out_units > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_source_chunk: grid too large");
    if (units > 0) {
        const int64_t wgs = int64_t(batch) * hkv * ((a.row_blocks + 3) / 4) * a.ncs;
        auto launch = [&](auto dtag) -> st_status {
            constexpr int HD = decltype(dtag)::value;
            constexpr int STAGES = 2, TOK = 64;      // (measured: three to five stages of 32 tokens, or four of 64 with one workgroup per compute unit, are no faster)
            const size_t smem = sizeof(ChunkSmem<HD, STAGES, TOK>);
            ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&chunk_split_lds_kernel<HD, STAGES, TOK>), hipFuncAttributeMaxDynamicSharedMemorySize, int(smem)));
            prof_begin(kProfSourceChunk, s);
            for (int rep = 0; rep < prof_repeat(); ++rep)
                hipLaunchKernelGGL((chunk_split_lds_kernel<HD, STAGES, TOK>), dim3((unsigned)wgs), dim3(256), smem, s, a);
            prof_end(kProfSourceChunk, s);
            return ST_OK;
        };
        const st_status lr = d == 64 ? launch(std::integral_constant<int, 64>{}) : launch(std::integral_constant<int, 128>{});
        if (lr != ST_OK) return lr;
        ST_LAUNCH_CHECK("chunk_split_lds_kernel");
    }
    const int splits = merge_splits(a.ncs);
    const dim3 merge_grid((unsigned)merge_workgroups(out_units, d, splits));
    if (d == 64) hipLaunchKernelGGL((chunk_combine_kernel<64>), merge_grid, dim3(kMergeThreads), 0, s, a, static_cast<uint16_t*>(out), lse, splits);
    else hipLaunchKernelGGL((chunk_combine_kernel<128>), merge_grid, dim3(kMergeThreads), 0, s, a, static_cast<uint16_t*>(out), lse, splits);
    ST_LAUNCH_CHECK("chunk_combine_kernel");
    return ST_OK;
}

extern "C" st_status st_attn_source_chunk(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                          const int32_t* src_len, const int32_t* n_new, int32_t max_new,
                                          int32_t max_src_len, int32_t batch, int32_t n_q_heads, float scale,
                                          void* workspace, size_t workspace_bytes, void* hip_stream) {
    return source_chunk_impl(out, lse, q, caches, src_len, n_new, max_new, max_src_len, batch, n_q_heads, scale, false, 0.0,
                             workspace, workspace_bytes, hip_stream);
}

extern "C" st_status st_attn_source_chunk_rope(void* out, float* lse, const void* q, const st_dual_cache* caches,
                                               const int32_t* src_len, const int32_t* n_new, int32_t max_new,
                                               int32_t max_src_len, int32_t batch, int32_t n_q_heads, float scale,
                                               double theta_base, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!(theta_base > 0.0)) return fail(ST_ERR_INVALID_ARG, "st_attn_source_chunk_rope: theta_base must be positive");
    return source_chunk_impl(out, lse, q, caches, src_len, n_new, max_new, max_src_len, batch, n_q_heads, scale, true, theta_base,
                             workspace, workspace_bytes, hip_stream);
}
