// Streaming-mask attention in fp32 on the matrix cores: forward and backward (the fp32 side of st_attn_prefill and
// st_attn_prefill_bwd; Sec. 3.2, Eq. 2).
//
// v_mfma_f32_32x32x2_f32 multiplies fp32 operands and accumulates in fp32 -- no precision is given up -- at twice the
// rate of the vector ALUs and leaves them free for the exponentials.  With two k-values per instruction the operand
// layouts are so simple that no shuffle is ever needed:
//   * first-type products (S^T = K Q^T and the like, contraction over the head dims): step (jj, e) contracts the dims
//     8 jj + e (lanes 0-31) and 8 jj + 4 + e (lanes 32-63), so a lane's operands of four steps are ONE 16-byte load of a
//     row as it lies in memory;
//   * accumulator register i of a lane holds row r(i) = 8 (i / 4) + 4 (lane / 32) + i % 4 of the result's 32 rows -- and
//     that is exactly the B operand of step i of a second-type product (O^T = V^T P^T and the like) whose k-values are
//     those rows; its A operand is element (row r(i), dim 32 db + lane % 32): 128 contiguous bytes per half wave.
// So every operand comes straight from the caller's tensors through the caches (rows gathered by token index): no packed
// copies, no workspace for the forward, and no LDS in the loops beyond the 32 rows a workgroup shares.
//
// Work: a workgroup owns 32 rows (query rows; keys for dK / dV) of a work item and one head; its FOUR WAVES take the
// 32-row blocks of the other side in turn and their results meet in LDS at the end.  A wave's chain of blocks is a
// quarter of the row's -- what a small problem is bound by -- and the waves never wait for each other inside the loop.
// Bound by those chains: one block of 32 x 32 x 128 is 128 instructions of 64 cycles in the forward, and the next block's
// operands are requested a phase ahead, but a wave has few blocks, the backward's registers leave one wave per SIMD, and the
// workgroups end in two uneven rounds -- the matrix pipe (fp32: 157 TFLOP/s) is busy 30 to 37 % of the cycles.
// Two sequences of about 900 tokens, 16 / 8 heads of 128 dims: forward 2.86 ms (one thread per row, vector ALUs) -> 0.090 ms
// (58 TFLOP/s of unmasked flop), gradients 19.8 -> 0.35 ms; 128 tokens, 2 heads of 64 dims: 200 -> 8 us.
#include <math.h>

#include <type_traits>

#include "st_plan.h"

namespace st {

constexpr int kF32Waves = 4, kF32Rows = 32;

// accumulator register i <-> row of the 32-row block
__device__ __forceinline__ int acc_row(int i, int hg) { return 8 * (i >> 2) + 4 * hg + (i & 3); }

// the rows a workgroup owns: 32-row part `sub` of a work item
struct OwnRows {
    int first, count;        // first row relative to the row's stream, rows (<= 32)
};
__device__ __forceinline__ OwnRows own_rows(const WorkItem& it, int sub) {
    return OwnRows{it.row0 + kF32Rows * sub, min(kF32Rows, it.n_rows - kF32Rows * sub)};
}

// [32][D] block of rows in LDS; four floats of padding send 16 consecutive rows to 16 different 16-byte columns
template <int D>
struct RowsLds {
    float x[kF32Rows][D + 4];
};

// What the four waves of a workgroup merge at the end
template <int D>
struct MergeLds {
    float o[kF32Waves][kF32Rows][D + 4];
};

// accumulator blocks (lane = row, dims along the registers) -> LDS rows
template <int D>
__device__ __forceinline__ void park(float (&rows)[kF32Rows][D + 4], const f32x16 (&acc)[D / 32], int n, int hg) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<f32x4*>(&rows[n][32 * db + 8 * q4 + 4 * hg]) =
                f32x4{acc[db][4 * q4], acc[db][4 * q4 + 1], acc[db][4 * q4 + 2], acc[db][4 * q4 + 3]};
}

// Masked pairs and values that are not finite.  A matrix instruction multiplies an operand row with the weights of all 32 columns of
// the block, 0 for the pairs that the mask forbids, and 0 x Inf is NaN: a bad value of a token would reach rows that do not see
// it.  A NaN stays, so the kernels walk their blocks without a look at this and check what comes out: a workgroup whose result
// is not finite throws it away and walks again with care -- in blocks with masked pairs the operand rows that hold such
// a value leave the product and are added to the columns that see them alone.  (Looking at the operands in every such block cost 4 %
// of the forward and 4 to 14 % of the gradients, most of it in registers; looking at the result costs 1 %, 0.2 us of the
// smallest forward.)

// (z stays 0 as long as what is folded into it is finite: 0 x Inf = 0 x NaN = NaN)
__device__ __forceinline__ float fold_finite(float z, const f32x4& x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) z = fmaf(x[e], 0.f, z);
    return z;
}
// bad[w], written by wave w before a barrier: does any wave report something?
__device__ __forceinline__ bool any_wave(const int (&bad)[kF32Waves]) {
    int any = 0;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) any |= bad[w];
    return any != 0;
}
// Sets the rows of an operand that hold a value that is not finite to zero; returned: bit r, row r of the block (x[g] holds row acc_row(g, hg)).
template <int DB>
__device__ __forceinline__ uint32_t take_out(float (&x)[16][DB], int hg) {
    uint32_t rows = 0u;
#pragma unroll
    for (int g = 0; g < 16; ++g) {
        float z = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) z = fmaf(x[g][db], 0.f, z);
        const unsigned long long lanes = __ballot(z != z);
        const bool lower = uint32_t(lanes) != 0u, upper = uint32_t(lanes >> 32) != 0u;
        rows |= (lower ? 1u << acc_row(g, 0) : 0u) | (upper ? 1u << acc_row(g, 1) : 0u);
#pragma unroll
        for (int db = 0; db < DB; ++db) x[g][db] = (hg ? upper : lower) ? 0.f : x[g][db];
    }
    return rows;
}
// weight x row r (uniform; `row` points at its dim 4 hg) added to the columns that see it; w: the block's weights
template <int D>
__device__ __forceinline__ void add_row(f32x16 (&acc)[D / 32], const f32x16& w, const float* row, int r, int n, bool seen) {
    float weight = w[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) weight = i == 4 * (r >> 3) + (r & 3) ? w[i] : weight;
    weight = __shfl(weight, n + 32 * ((r >> 2) & 1));
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 x = *reinterpret_cast<const f32x4_a4*>(row + 32 * db + 8 * q4);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[db][4 * q4 + c] = seen ? fmaf(weight, x[c], acc[db][4 * q4 + c]) : acc[db][4 * q4 + c];
        }
}

// --------------------------------------------------------------------------
// Forward
// --------------------------------------------------------------------------
template <int D>
struct FwdF32Smem {
    MergeLds<D> merge;
    float m[kF32Waves][kF32Rows], l[kF32Waves][kF32Rows];
    int bad[kF32Waves];
};

// false: the result is not finite, nothing has been stored
template <int D, bool CAREFUL>
__device__ __forceinline__ bool prefill_f32_walk(unsigned block, float* __restrict__ out, float* __restrict__ lse,
                                                 const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                 PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    constexpr int JJ = D / 8, DB = D / 32;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    FwdF32Smem<D>& sm = *reinterpret_cast<FwdF32Smem<D>*>(smem_raw);
    const unsigned per_item = unsigned(n_q_heads) * unsigned(pv.parts32);
    const int rank = int(block / per_item);
    const unsigned rest = block % per_item;
    const int hh = int(rest % unsigned(n_q_heads)), sub = int(rest / unsigned(n_q_heads));
    const int hk = hh % n_kv_heads, hq = hk * (n_q_heads / n_kv_heads) + hh / n_kv_heads;     // consecutive workgroups -> consecutive KV heads
    const WorkItem it = pv.sorted[rank];
    const OwnRows own = own_rows(it, sub);
    if (own.count <= 0) return true;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hg = lane >> 5;
    const int my_row = own.first + min(n, own.count - 1), last_row = own.first + own.count - 1;
    const int my_vis = pv.vis[it.a_base + my_row];
    const int64_t my_tok = pv.perm[it.a_base + my_row];
    // 32-column blocks of the two runs: the own stream up to the last row, for reasoning rows the source prefix it sees
    const int blocks_a = last_row / kF32Rows + 1;
    const int blocks_b = it.kind == ST_SOURCE ? 0 : (pv.vis[it.a_base + last_row] + kF32Rows - 1) / kF32Rows;
    const int first_vis = pv.vis[it.a_base + own.first];
    const int n_blocks = blocks_a + blocks_b;

    // token of this lane's key row in block t (columns past the end of the stream: the last one, masked below)
    auto key_token = [&](int t) {
        t = min(t, n_blocks - 1);
        const bool in_a = t < blocks_a;
        const int col = min((in_a ? t : t - blocks_a) * kF32Rows + n, (in_a ? it.n_stream : it.n_src) - 1);
        return pv.perm[(in_a ? it.a_base : it.b_base) + col];
    };
    const int64_t stride = int64_t(n_kv_heads) * D;
    const float* k_lane = k + int64_t(hk) * D + 4 * hg;
    const float* v_lane = v + int64_t(hk) * D + n;
    const int row = threadIdx.x >> 3, part = threadIdx.x & 7;              // of the merge: eight threads per row
    f32x4 qf[JJ];
    {
        const float* qp = q + (my_tok * n_q_heads + hq) * D + 4 * hg;
#pragma unroll
        for (int jj = 0; jj < JJ; ++jj) qf[jj] = *reinterpret_cast<const f32x4*>(qp + 8 * jj);
    }
    f32x16 o_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[db][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    f32x4 kf[JJ];
    int tok = 0;
    if (wave < n_blocks) {
        tok = key_token(wave);
        const float* kp = k_lane + tok * stride;
#pragma unroll
        for (int jj = 0; jj < JJ; ++jj) kf[jj] = *reinterpret_cast<const f32x4*>(kp + 8 * jj);
    }
    for (int t = wave; t < n_blocks; t += kF32Waves) {
        const int tok_next = key_token(t + kF32Waves);
        // ---- S^T = K Q^T; the value rows of the block are requested beside it ----
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
        float vf[16][DB];
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const float* vp = v_lane + __shfl(tok, acc_row(g, hg)) * stride;
#pragma unroll
            for (int db = 0; db < DB; ++db) vf[g][db] = vp[32 * db];
#pragma unroll
            for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj)
#pragma unroll
                for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[jj][e], qf[jj][e], s, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- softmax over the block: lane = query row, register i = column acc_row(i, hg) ----
        const bool in_a = t < blocks_a;
        const int c0 = (in_a ? t : t - blocks_a) * kF32Rows;
        const int limit = in_a ? my_row + 1 : my_vis;                      // columns < limit are visible
        const int limit_min = in_a ? own.first + 1 : first_vis;            // ... to every row
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] *= scale;
        if (c0 + kF32Rows > limit_min) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = c0 + acc_row(i, hg) < limit ? s[i] : -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;              // (a row that sees nothing yet)
        if (__any(m_new > m_run)) {
            const float alpha = expf(m_run - m_use);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o_acc[db][i] *= alpha;
        }
        m_run = m_new;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = expf(s[i] - m_use);
            l_run += s[i];
        }
        if (CAREFUL && c0 + kF32Rows > limit_min) {
            for (uint32_t rows = take_out<DB>(vf, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<D>(o_acc, s, v + __shfl(tok, r) * stride + int64_t(hk) * D + 4 * hg, r, n, c0 + r < limit);
            }
        }
        // ---- O^T += V^T P^T; the next block's keys are requested beside it ----
        tok = tok_next;
        const float* kp = k_lane + tok * stride;
#pragma unroll
        for (int g = 0; g < 16; ++g) {
#pragma unroll
            for (int db = 0; db < DB; ++db) o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[g][db], s[g], o_acc[db], 0, 0, 0);
#pragma unroll
            for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) kf[jj] = *reinterpret_cast<const f32x4*>(kp + 8 * jj);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // ---- merge of the four waves' states ----
    bool bad = false;
    if (!CAREFUL) {
        float z = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) z = fmaf(o_acc[db][i], 0.f, z);
        bad = __any(z != z);
    }
    park<D>(sm.merge.o[wave], o_acc, n, hg);
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (hg == 0) {
        sm.m[wave][n] = m_run;
        sm.l[wave][n] = l_tot;
    }
    if (!CAREFUL && lane == 0) sm.bad[wave] = bad;
    __syncthreads();
    if (!CAREFUL && any_wave(sm.bad)) return false;
    const int64_t rowhead = int64_t(pv.perm[it.a_base + own.first + min(row, own.count - 1)]) * n_q_heads + hq;
    float m_all = -INFINITY, wt[kF32Waves], den = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) m_all = fmaxf(m_all, sm.m[w][row]);           // finite: column 0 of the own stream is visible
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
        wt[w] = expf(sm.m[w][row] - m_all);                                // (0 for a wave that saw nothing)
        den = fmaf(wt[w], sm.l[w][row], den);
    }
    const float inv = 1.f / den;
    f32x4 a[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        a[db] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(&sm.merge.o[w][row][4 * part + 32 * db]);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[db][e] = fmaf(wt[w], x[e], a[db][e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) a[db][e] *= inv;
    }
    if (row < own.count) {
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(out + rowhead * D + 4 * part + 32 * db) = a[db];
        if (lse && part == 0) lse[rowhead] = m_all + logf(den);
    }
    return true;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 2) void prefill_f32_kernel(float* __restrict__ out, float* __restrict__ lse,
                                                                        const float* __restrict__ q, const float* __restrict__ k,
                                                                        const float* __restrict__ v, PlanView pv, int n_q_heads,
                                                                        int n_kv_heads, float scale) {
    unsigned block = blockIdx.x;
    if (prefill_f32_walk<D, false>(block, out, lse, q, k, v, pv, n_q_heads, n_kv_heads, scale)) return;
    asm volatile("" : "+s"(block));               // (nothing of the first walk is kept for the second: the registers are full)
    prefill_f32_walk<D, true>(block, out, lse, q, k, v, pv, n_q_heads, n_kv_heads, scale);
}

// --------------------------------------------------------------------------
// Backward, query side: delta_i = dO_i . O_i, dQ_i = scale sum_j dS_ij K_j
// --------------------------------------------------------------------------
template <int D>
struct DqF32Smem {
    union {                       // the rows are read in the loop, the merge comes after it
        struct {
            RowsLds<D> q, d_out;
        };
        MergeLds<D> merge;
    };
    float lse[kF32Rows], delta[kF32Rows];
    int bad[kF32Waves];
};

// false: the result is not finite, nothing but delta has been stored
template <int D, bool CAREFUL>
__device__ __forceinline__ bool bwd_dq_f32_walk(unsigned block, float* __restrict__ dq, float* __restrict__ delta_out,
                                                const float* __restrict__ d_out, const float* __restrict__ q, const float* __restrict__ k,
                                                const float* __restrict__ v, const float* __restrict__ out, const float* __restrict__ lse,
                                                PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    constexpr int JJ = D / 8, DB = D / 32;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    DqF32Smem<D>& sm = *reinterpret_cast<DqF32Smem<D>*>(smem_raw);
    const unsigned per_item = unsigned(n_q_heads) * unsigned(pv.parts32);
    const int rank = int(block / per_item);
    const unsigned rest = block % per_item;
    const int hh = int(rest % unsigned(n_q_heads)), sub = int(rest / unsigned(n_q_heads));
    const int hk = hh % n_kv_heads, hq = hk * (n_q_heads / n_kv_heads) + hh / n_kv_heads;
    const WorkItem it = pv.sorted[rank];
    const OwnRows own = own_rows(it, sub);
    if (own.count <= 0) return true;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hg = lane >> 5;
    const int my_row = own.first + min(n, own.count - 1), last_row = own.first + own.count - 1;
    const int my_vis = pv.vis[it.a_base + my_row];
    const int blocks_a = last_row / kF32Rows + 1;
    const int blocks_b = it.kind == ST_SOURCE ? 0 : (pv.vis[it.a_base + last_row] + kF32Rows - 1) / kF32Rows;
    const int first_vis = pv.vis[it.a_base + own.first];
    const int n_blocks = blocks_a + blocks_b;

    const int row = threadIdx.x >> 3, part = threadIdx.x & 7;
    const int64_t rowhead = int64_t(pv.perm[it.a_base + own.first + min(row, own.count - 1)]) * n_q_heads + hq;
    auto key_token = [&](int t) {
        t = min(t, n_blocks - 1);
        const bool in_a = t < blocks_a;
        const int col = min((in_a ? t : t - blocks_a) * kF32Rows + n, (in_a ? it.n_stream : it.n_src) - 1);
        return pv.perm[(in_a ? it.a_base : it.b_base) + col];
    };
    const int64_t stride = int64_t(n_kv_heads) * D;
    const float* k_rows = k + int64_t(hk) * D + 4 * hg;
    const float* v_rows = v + int64_t(hk) * D + 4 * hg;
    const float* k_cols = k + int64_t(hk) * D + n;
    // the workgroup's rows of q and dO into LDS (operands of every wave), their delta on the way
    {
        float dl = 0.f;
#pragma unroll
        for (int d = 4 * part; d < D; d += 32) {
            const f32x4 a = *reinterpret_cast<const f32x4_a4*>(d_out + rowhead * D + d), o = *reinterpret_cast<const f32x4_a4*>(out + rowhead * D + d);
            *reinterpret_cast<f32x4*>(&sm.q.x[row][d]) = *reinterpret_cast<const f32x4_a4*>(q + rowhead * D + d);
            *reinterpret_cast<f32x4*>(&sm.d_out.x[row][d]) = a;
#pragma unroll
            for (int e = 0; e < 4; ++e) dl = fmaf(a[e], o[e], dl);
        }
        dl += __shfl_xor(dl, 1);
        dl += __shfl_xor(dl, 2);
        dl += __shfl_xor(dl, 4);
        if (part == 0) {
            sm.lse[row] = lse[rowhead];
            sm.delta[row] = dl;
            if (row < own.count) delta_out[rowhead] = dl;
        }
    }
    __syncthreads();
    const float my_lse = sm.lse[n], my_delta = sm.delta[n];

    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;
    f32x4 kf[JJ], vf[JJ];
    int tok = 0;
    if (wave < n_blocks) {
        tok = key_token(wave);
#pragma unroll
        for (int jj = 0; jj < JJ; ++jj) kf[jj] = *reinterpret_cast<const f32x4_a4*>(k_rows + tok * stride + 8 * jj);
#pragma unroll
        for (int jj = 0; jj < JJ; ++jj) vf[jj] = *reinterpret_cast<const f32x4_a4*>(v_rows + tok * stride + 8 * jj);
    }
    for (int t = wave; t < n_blocks; t += kF32Waves) {
        const int tok_next = key_token(t + kF32Waves);
        // ---- S^T = K Q^T, dP^T = V dO^T; K as the second product's operand is requested beside them ----
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
        float kt[16][DB];
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const float* kp = k_cols + __shfl(tok, acc_row(g, hg)) * stride;
#pragma unroll
            for (int db = 0; db < DB; ++db) kt[g][db] = kp[32 * db];
#pragma unroll
            for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) {
                const f32x4 qv = *reinterpret_cast<const f32x4*>(&sm.q.x[n][8 * jj + 4 * hg]);
                const f32x4 ov = *reinterpret_cast<const f32x4*>(&sm.d_out.x[n][8 * jj + 4 * hg]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[jj][e], qv[e], s, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[jj][e], ov[e], dp, 0, 0, 0);
                }
            }
        }
        const bool in_a = t < blocks_a;
        const int c0 = (in_a ? t : t - blocks_a) * kF32Rows;
        const int limit = in_a ? my_row + 1 : my_vis, limit_min = in_a ? own.first + 1 : first_vis;
        const bool partial = c0 + kF32Rows > limit_min;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float p = expf(s[i] * scale - my_lse);
            if (partial) p = c0 + acc_row(i, hg) < limit ? p : 0.f;
            s[i] = p * (dp[i] - my_delta) * scale;
            if (CAREFUL) s[i] = c0 + acc_row(i, hg) < limit ? s[i] : 0.f;
        }
        if (CAREFUL && partial) {
            for (uint32_t rows = take_out<DB>(kt, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<D>(acc, s, k_rows + __shfl(tok, r) * stride, r, n, c0 + r < limit);
            }
        }
        // ---- dQ^T += K^T dS^T; the next block's rows are requested beside it ----
        tok = tok_next;
#pragma unroll
        for (int g = 0; g < 16; ++g) {
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(kt[g][db], s[g], acc[db], 0, 0, 0);
#pragma unroll
            for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) {
                kf[jj] = *reinterpret_cast<const f32x4_a4*>(k_rows + tok * stride + 8 * jj);
                vf[jj] = *reinterpret_cast<const f32x4_a4*>(v_rows + tok * stride + 8 * jj);
            }
        }
    }
    __syncthreads();
    park<D>(sm.merge.o[wave], acc, n, hg);
    __syncthreads();
    f32x4 a[DB];
    float z = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        a[db] = *reinterpret_cast<const f32x4*>(&sm.merge.o[0][row][4 * part + 32 * db]);
#pragma unroll
        for (int w = 1; w < kF32Waves; ++w) a[db] += *reinterpret_cast<const f32x4*>(&sm.merge.o[w][row][4 * part + 32 * db]);
        z = fold_finite(z, a[db]);
    }
    if (!CAREFUL) {
        const bool bad = __any(z != z);
        if (lane == 0) sm.bad[wave] = bad;
        __syncthreads();
        if (any_wave(sm.bad)) return false;
    }
    if (row < own.count) {
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4_a4*>(dq + rowhead * D + 4 * part + 32 * db) = a[db];
    }
    return true;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 2) void bwd_dq_f32_kernel(float* __restrict__ dq, float* __restrict__ delta_out,
                                                                       const float* __restrict__ d_out, const float* __restrict__ q,
                                                                       const float* __restrict__ k, const float* __restrict__ v,
                                                                       const float* __restrict__ out, const float* __restrict__ lse,
                                                                       PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    unsigned block = blockIdx.x;
    if (bwd_dq_f32_walk<D, false>(block, dq, delta_out, d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale)) return;
    asm volatile("" : "+s"(block));               // (nothing of the first walk is kept for the second: the registers are full)
    bwd_dq_f32_walk<D, true>(block, dq, delta_out, d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale);
}

// --------------------------------------------------------------------------
// Backward, key side: dV_j = sum_i P_ij dO_i, dK_j = scale sum_i dS_ij Q_i over the query rows i that see key j, summed
// over the query heads of the KV head.  A workgroup owns 32 keys of one KV head; the (32-row query block, query head)
// pairs are dealt out to its four waves.  parts > 1: the query heads of a KV head are dealt out to `parts` workgroups (a divisor
// of the group), which leave their sums in `partial` ([2: dK, dV][parts][N][n_kv_heads][D]) for bwd_dkv_sum_f32_kernel.
// Products not transposed (S = Q K^T): a lane owns a key, rows run along the accumulator registers.
// --------------------------------------------------------------------------
template <int D>
struct DkvF32Smem {
    union {                       // the rows are read in the loop, the merge comes after it
        struct {
            RowsLds<D> k, v;
        };
        MergeLds<D> merge;
    };
    int bad[kF32Waves];
};

// false: the result is not finite, nothing has been stored
template <int D, bool CAREFUL>
__device__ __forceinline__ bool bwd_dkv_f32_walk(unsigned block, float* __restrict__ dk, float* __restrict__ dv,
                                                 const float* __restrict__ delta, const float* __restrict__ d_out,
                                                 const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                 const float* __restrict__ lse, PlanView pv, int n_q_heads, int n_kv_heads, float scale,
                                                 int parts, float* __restrict__ partial, int64_t partial_stride) {
    constexpr int JJ = D / 8, DB = D / 32;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    DkvF32Smem<D>& sm = *reinterpret_cast<DkvF32Smem<D>*>(smem_raw);
    const unsigned per_item = unsigned(n_kv_heads) * unsigned(pv.parts32) * unsigned(parts);
    // (early keys are seen by the most rows: the table, sorted by the forward's cost, is walked backwards)
    const int rank = pv.m_max - 1 - int(block / per_item);
    const unsigned rest = block % per_item;
    const int hk = int(rest % unsigned(n_kv_heads)), part_of = int(rest / unsigned(n_kv_heads)) % parts, sub = int(rest / (unsigned(n_kv_heads) * unsigned(parts)));
    const int group = n_q_heads / n_kv_heads / parts, hq0 = (hk * parts + part_of) * group;      // this workgroup's query heads
    const WorkItem it = pv.sorted[rank];
    const OwnRows own = own_rows(it, sub);
    if (own.count <= 0) return true;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hg = lane >> 5;
    const int my_key = own.first + min(n, own.count - 1), last_key = own.first + own.count - 1;

    const int row = threadIdx.x >> 3, part = threadIdx.x & 7;
    const int64_t keyhead = int64_t(pv.perm[it.a_base + own.first + min(row, own.count - 1)]) * n_kv_heads + hk;
    // the rows that see the block's first key: the own stream from it on; for source keys also the reasoning rows from the
    // first one whose visible-source count exceeds it (counts do not decrease along the stream)
    const int S = it.n_src;
    const bool src = it.kind == ST_SOURCE;
    const int rsn_base = it.b_base + S;
    const int n_rsn = src ? pv.cu[it.seq + 1] - pv.cu[it.seq] - S : it.n_stream;
    int rsn_first = 0;
    if (src) {
        // searched by the whole wave: every lane tests the end of one 64th of the range
        int lo = 0, hi = n_rsn;                                 // the answer lies in [lo, hi]; hi == n_rsn: no such row
        while (lo < hi) {
            const int span = hi - lo, step = (span + 63) >> 6;
            const int last = min(span - 1, lane * step + step - 1);                              // end of this lane's piece
            const unsigned long long seen = __ballot(pv.vis[rsn_base + lo + last] > own.first);  // (monotone along the lanes)
            if (seen == 0ull) {
                lo = hi;
            } else {
                const int first = __ffsll((long long)seen) - 1;
                hi = lo + min(span - 1, first * step + step - 1);                                // this row exceeds it ...
                lo = lo + first * step;                                                          // ... and none before this piece does
            }
            lo = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
        }
        rsn_first = lo;
    }
    const int blocks_a = (it.n_stream - own.first + kF32Rows - 1) / kF32Rows;
    const int blocks_b = src ? (n_rsn - rsn_first + kF32Rows - 1) / kF32Rows : 0;
    const int n_iter = (blocks_a + blocks_b) * group;

    // iteration x: query head x % group, block x / group
    struct Iter { int base, row0, end, hq; bool rs; };
    auto iter_at = [&](int x) {
        x = min(x, n_iter - 1);
        const int t = x / group;
        Iter r;
        r.hq = hq0 + x % group;
        r.rs = t >= blocks_a;                                    // (rows of the other stream: visible by their source count)
        r.base = r.rs ? rsn_base : it.a_base;
        r.row0 = r.rs ? rsn_first + (t - blocks_a) * kF32Rows : own.first + t * kF32Rows;
        r.end = r.rs ? n_rsn : it.n_stream;
        return r;
    };
#pragma unroll
    for (int d = 4 * part; d < D; d += 32) {
        *reinterpret_cast<f32x4*>(&sm.k.x[row][d]) = *reinterpret_cast<const f32x4_a4*>(k + keyhead * D + d);
        *reinterpret_cast<f32x4*>(&sm.v.x[row][d]) = *reinterpret_cast<const f32x4_a4*>(v + keyhead * D + d);
    }
    __syncthreads();

    f32x16 dk_acc[DB], dv_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dk_acc[db][i] = dv_acc[db][i] = 0.f;
    f32x4 qf[JJ], of[JJ];
    Iter cur = iter_at(wave);
    int tok = 0, lim = 0;                                        // of this lane's row: token, keys it sees (index below lim)
    float l_row = 0.f, d_row = 0.f;
    auto row_info = [&](const Iter& r) {
        const int i = min(r.row0 + n, r.end - 1);
        tok = pv.perm[r.base + i];
        lim = r.row0 + n < r.end ? (r.rs ? pv.vis[r.base + i] : i + 1) : 0;          // rows past the end see nothing
        const int64_t rh = int64_t(tok) * n_q_heads + r.hq;
        l_row = lse[rh];
        d_row = delta[rh];
    };
    auto load_rows = [&](const Iter& r, int jj0, int jj1) {
        const int64_t off = (int64_t(tok) * n_q_heads + r.hq) * D + 4 * hg;
#pragma unroll
        for (int jj = jj0; jj < jj1; ++jj) {
            qf[jj] = *reinterpret_cast<const f32x4_a4*>(q + off + 8 * jj);
            of[jj] = *reinterpret_cast<const f32x4_a4*>(d_out + off + 8 * jj);
        }
    };
    if (wave < n_iter) {
        row_info(cur);
        load_rows(cur, 0, JJ);
    }
    for (int x = wave; x < n_iter; x += kF32Waves) {
        // ---- S = Q K^T, dP = dO V^T; Q and dO as the second products' operands are requested beside them ----
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
        float qt[16][DB], ot[16][DB];
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int64_t off = (int64_t(__shfl(tok, acc_row(g, hg))) * n_q_heads + cur.hq) * D + n;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                qt[g][db] = q[off + 32 * db];
                ot[g][db] = d_out[off + 32 * db];
            }
#pragma unroll
            for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) {
                const f32x4 kv = *reinterpret_cast<const f32x4*>(&sm.k.x[n][8 * jj + 4 * hg]);
                const f32x4 vv = *reinterpret_cast<const f32x4*>(&sm.v.x[n][8 * jj + 4 * hg]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(qf[jj][e], kv[e], s, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x2f32(of[jj][e], vv[e], dp, 0, 0, 0);
                }
            }
        }
        // register i <-> row acc_row(i, hg) of the block
        const bool full = __builtin_amdgcn_readfirstlane(lim) > last_key && cur.row0 + kF32Rows <= cur.end;    // (limits do not decrease along the rows)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = acc_row(i, hg);
            float p = expf(s[i] * scale - __shfl(l_row, r));
            if (!full) p = my_key < __shfl(lim, r) ? p : 0.f;
            s[i] = p;
            dp[i] = p * (dp[i] - __shfl(d_row, r)) * scale;
            if (CAREFUL && !full) dp[i] = my_key < __shfl(lim, r) ? dp[i] : 0.f;
        }
        if (CAREFUL && !full) {
            auto row_of = [&](const float* x, int r) { return x + (int64_t(__shfl(tok, r)) * n_q_heads + cur.hq) * D + 4 * hg; };
            for (uint32_t rows = take_out<DB>(ot, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<D>(dv_acc, s, row_of(d_out, r), r, n, my_key < __shfl(lim, r));
            }
            for (uint32_t rows = take_out<DB>(qt, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<D>(dk_acc, dp, row_of(q, r), r, n, my_key < __shfl(lim, r));
            }
        }
        // ---- dV^T += dO^T P, dK^T += Q^T dS; the next rows are requested beside them ----
        cur = iter_at(x + kF32Waves);
        row_info(cur);
#pragma unroll
        for (int g = 0; g < 16; ++g) {
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                dv_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(ot[g][db], s[g], dv_acc[db], 0, 0, 0);
                dk_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(qt[g][db], dp[g], dk_acc[db], 0, 0, 0);
            }
            load_rows(cur, g * JJ / 16, (g + 1) * JJ / 16);
        }
    }
    // ---- sums of the four waves, in a fixed order: dV, then dK ----
    f32x4 a[2][DB];
    float z = 0.f;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        __syncthreads();
        park<D>(sm.merge.o[wave], which == 0 ? dv_acc : dk_acc, n, hg);
        __syncthreads();
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            a[which][db] = *reinterpret_cast<const f32x4*>(&sm.merge.o[0][row][4 * part + 32 * db]);
#pragma unroll
            for (int w = 1; w < kF32Waves; ++w) a[which][db] += *reinterpret_cast<const f32x4*>(&sm.merge.o[w][row][4 * part + 32 * db]);
            z = fold_finite(z, a[which][db]);
        }
    }
    if (!CAREFUL) {
        const bool bad = __any(z != z);
        if (lane == 0) sm.bad[wave] = bad;
        __syncthreads();
        if (any_wave(sm.bad)) return false;
    }
    if (row < own.count) {
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            float* dst = (parts > 1 ? partial + ((which == 0 ? parts : 0) + part_of) * partial_stride : which == 0 ? dv : dk) + keyhead * D;
#pragma unroll
            for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4_a4*>(dst + 4 * part + 32 * db) = a[which][db];
        }
    }
    return true;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 1) void bwd_dkv_f32_kernel(float* __restrict__ dk, float* __restrict__ dv,
                                                                        const float* __restrict__ delta, const float* __restrict__ d_out,
                                                                        const float* __restrict__ q, const float* __restrict__ k,
                                                                        const float* __restrict__ v, const float* __restrict__ lse,
                                                                        PlanView pv, int n_q_heads, int n_kv_heads, float scale, int parts,
                                                                        float* __restrict__ partial, int64_t partial_stride) {
    unsigned block = blockIdx.x;
    if (bwd_dkv_f32_walk<D, false>(block, dk, dv, delta, d_out, q, k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride)) return;
    asm volatile("" : "+s"(block));               // (nothing of the first walk is kept for the second: the registers are full)
    bwd_dkv_f32_walk<D, true>(block, dk, dv, delta, d_out, q, k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride);
}

// dK (blockIdx.y = 0) or dV (1) from the partial sums of the key-side kernel, in a fixed order; n4 groups of four elements
__global__ __launch_bounds__(256) void bwd_dkv_sum_f32_kernel(float* __restrict__ dk, float* __restrict__ dv, const float* __restrict__ partial,
                                                              int64_t partial_stride, int parts, int64_t n4) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n4) return;
    const float* p = partial + blockIdx.y * parts * partial_stride + i * 4;
    f32x4 a = *reinterpret_cast<const f32x4*>(p);
    for (int x = 1; x < parts; ++x) a += *reinterpret_cast<const f32x4*>(p + x * partial_stride);
    *reinterpret_cast<f32x4_a4*>((blockIdx.y == 0 ? dk : dv) + i * 4) = a;
}

// ---- launches (arguments have been checked by the callers) ----
template <typename K>
static st_status with_smem(K kernel, size_t bytes) {
    ST_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)));
    return ST_OK;
}

st_status launch_prefill_f32(float* out, float* lse, const float* q, const float* k, const float* v, const PlanView& pv, int n_q_heads,
                             int n_kv_heads, int head_dim, float scale, hipStream_t s) {
    const int64_t blocks = int64_t(pv.m_max) * n_q_heads * pv.parts32;
    if (blocks > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_prefill: grid too large");
    auto run = [&](auto dtag) -> st_status {
        constexpr int D = decltype(dtag)::value;
        const st_status r = with_smem(&prefill_f32_kernel<D>, sizeof(FwdF32Smem<D>));
        if (r != ST_OK) return r;
        hipLaunchKernelGGL((prefill_f32_kernel<D>), dim3((unsigned)blocks), dim3(64 * kF32Waves), sizeof(FwdF32Smem<D>), s, out, lse, q, k, v, pv,
                           n_q_heads, n_kv_heads, scale);
        ST_LAUNCH_CHECK("prefill_f32_kernel");
        return ST_OK;
    };
    return head_dim == 64 ? run(std::integral_constant<int, 64>{}) : run(std::integral_constant<int, 128>{});
}

st_status launch_bwd_f32(float* dq, float* dk, float* dv, float* delta, const float* d_out, const float* q, const float* k, const float* v,
                         const float* out, const float* lse, const PlanView& pv, int n_q_heads, int n_kv_heads, int head_dim, float scale,
                         int64_t n_tokens, int parts, float* partial, hipStream_t s) {
    const int64_t qblocks = int64_t(pv.m_max) * n_q_heads * pv.parts32, kblocks = int64_t(pv.m_max) * n_kv_heads * parts * pv.parts32;
    const int64_t partial_stride = n_tokens * n_kv_heads * head_dim;
    if (qblocks > 0x7fffffff) return fail(ST_ERR_SHAPE, "st_attn_prefill_bwd: grid too large");
    auto run = [&](auto dtag) -> st_status {
        constexpr int D = decltype(dtag)::value;
        st_status r = with_smem(&bwd_dq_f32_kernel<D>, sizeof(DqF32Smem<D>));
        if (r != ST_OK) return r;
        r = with_smem(&bwd_dkv_f32_kernel<D>, sizeof(DkvF32Smem<D>));
        if (r != ST_OK) return r;
        hipLaunchKernelGGL((bwd_dq_f32_kernel<D>), dim3((unsigned)qblocks), dim3(64 * kF32Waves), sizeof(DqF32Smem<D>), s, dq, delta, d_out, q, k, v,
                           out, lse, pv, n_q_heads, n_kv_heads, scale);
        hipLaunchKernelGGL((bwd_dkv_f32_kernel<D>), dim3((unsigned)kblocks), dim3(64 * kF32Waves), sizeof(DkvF32Smem<D>), s, dk, dv, delta, d_out, q,
                           k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride);
        if (parts > 1) {
            const int64_t n4 = partial_stride / 4;
            hipLaunchKernelGGL(bwd_dkv_sum_f32_kernel, dim3((unsigned)((n4 + 255) / 256), 2), dim3(256), 0, s, dk, dv, partial, partial_stride, parts, n4);
        }
        ST_LAUNCH_CHECK("bwd_dq_f32_kernel / bwd_dkv_f32_kernel");
        return ST_OK;
    };
    return head_dim == 64 ? run(std::integral_constant<int, 64>{}) : run(std::integral_constant<int, 128>{});
}

}  // namespace st
