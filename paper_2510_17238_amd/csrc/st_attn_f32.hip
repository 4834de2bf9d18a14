// Streaming-mask attention in fp32 on the matrix cores: forward and backward (the fp32 side of st_attn_prefill and
// st_attn_prefill_bwd; Sec. 3.2, Eq. 2).
//
// Every fp32 operand is split into three bf16 terms (8 + 8 + 8 bits: all 24), and a product is six v_mfma_f32_32x32x16_bf16 instead of
// eight v_mfma_f32_32x32x2_f32 of twice the length: 192 cycles of the matrix pipe for 16 k-values where fp32 took 512.  The three products
// left out are below 2^-26 of the whole, the sums are fp32 as before and fewer; against 64 bits the error is 0.72 to 0.88 of what it was with the
// fp32 instructions, output and gradients, over 26 shapes of 54 to 1,200 tokens.  The operand layouts need no shuffle:
//   * first-type products (S^T = K Q^T and the like, contraction over the head dims): step j contracts 16 dims, of which a lane holds
//     16 j + 4 hg .. + 3 and 8 further on (hg = lane / 32): two 16-byte loads of a row as it lies in memory;
//   * accumulator register i of a lane holds row r(i) = 8 (i / 4) + 4 (lane / 32) + i % 4 of the result's 32 rows, and registers
//     8 st .. + 7 are the B operand of 16-row step st of a second-type product (O^T = V^T P^T and the like) whose k-values are
//     those rows; its A operand is element (row r(i), dim 32 db + lane % 32): 128 contiguous bytes per half wave.
// So every operand comes straight from the caller's tensors through the caches (rows gathered by token index): no packed
// copies, no workspace for the forward, and no LDS in the loops beyond the 32 rows a workgroup shares (split once).
//
// Work: a workgroup owns 32 rows (query rows; keys for dK / dV) of a work item and one head (query side with heads of 128 dims: two heads of
// a KV head, whose keys and values are then split once for both); its FOUR WAVES take the 32-row blocks of the other side in turn and
// their results meet in LDS at the end.  A wave's chain of blocks is a quarter of the row's -- what a small problem is bound by -- and
// the waves never wait for each other inside the loop.
// Bound by what a wave can issue: a block of 32 x 32 x 128 is 96 matrix instructions of 32 cycles in the forward beside 1,250 vector
// instructions, 900 of them splits; an operand that every wave split for itself is split again by the others.  The splits of the next step
// stand behind the matrix instructions of the present one (left to the compiler, the two ran one behind the other: key side 168 us
// against 147).  The workgroups end in two uneven rounds.
// Two sequences of about 900 tokens, 16 / 8 heads of 128 dims, us: forward 90 with the fp32 instructions -> 66, query side 137 -> 107,
// key side 212 -> 154; the training step with tables and rotation 432 -> 317.
#include <math.h>

#include <type_traits>

#include "st_plan.h"

namespace st {

constexpr int kF32Waves = 4, kF32Rows = 32;

// exp(x) = 2^n 2^f: x log2(e) = n + f with f in [-1/2, 1/2] exact but for its last bit, so that no rounding grows with x (2^(x log2(e)) of
// the rounded product is off by half a unit of it: 5e-7 at x = -8, 1.8e-6 at -32).  For every x what expf gives: 0.85e-7 at most against 64 bits (expf 0.82e-7)
// over [-32, 0], subnormal results, Inf and NaN included -- in eight instructions, expf's range checks left to one clamp (the training step
// above: 5 us more than the rounded product, expf 20).
__device__ __forceinline__ float exp_f32(float x) {
    constexpr float kHi = 1.4426950408889634f, kLo = 1.925963033500e-8f;                   // log2(e) in two terms
    const float n = __builtin_amdgcn_fmed3f(__builtin_rintf(x * kHi), -200.f, 200.f);
    return ldexpf(__builtin_amdgcn_exp2f(fmaf(x, kLo, fmaf(x, kHi, -n))), int(n));
}

// accumulator register i <-> row of the 32-row block
__device__ __forceinline__ int acc_row(int i, int hg) { return 8 * (i >> 2) + 4 * hg + (i & 3); }

// the rows a workgroup owns: 32-row part `sub` of a work item
struct OwnRows {
    int first, count;        // first row relative to the row's stream, rows (<= 32)
};
__device__ __forceinline__ OwnRows own_rows(const WorkItem& it, int sub) {
    return OwnRows{it.row0 + kF32Rows * sub, min(kF32Rows, it.n_rows - kF32Rows * sub)};
}

// what a workgroup of the forward or of the query side takes: the part `sub` of a work item, HB query heads of a KV head from hq on
struct HeadRows {
    int rank, sub, hk, hq;
    __device__ __forceinline__ HeadRows(unsigned block, int hb, const PlanView& pv, int n_q_heads, int n_kv_heads) {
        const unsigned sets = unsigned(n_q_heads / hb), per_item = sets * unsigned(pv.parts32), rest = block % per_item;
        rank = int(block / per_item);
        sub = int(rest / sets);
        const int hh = int(rest % sets);
        hk = hh % n_kv_heads;                      // consecutive workgroups -> consecutive KV heads
        hq = hk * (n_q_heads / n_kv_heads) + hb * (hh / n_kv_heads);
    }
    // before another walk, `step` heads on
    __device__ __forceinline__ void again(int step) {
        __syncthreads();                           // (the LDS of the walk before is still being read)
        hq += step;
        asm volatile("" : "+s"(rank), "+s"(sub));  // (nothing of a walk is kept for the next: the registers are full)
    }
};

// [32][D] block of rows in LDS; four floats of padding send 16 consecutive rows to 16 different 16-byte columns
template <int D>
struct RowsLds {
    float x[kF32Rows][D + 4];
};

// An fp32 operand as three bf16 terms of 2^24 x, each the rounded rest of the one before: 8 + 8 + 8 bits, so h + m + l is 2^24 x to the
// last bit for every finite x below 2^104 (2e31).  Unscaled, the last terms of an x below 2^-110 would be subnormal and lost: results
// 1e-3 to 9e-2 off with operands of 2^-118.  From 2^104 on a term is Inf, which shows in the result (see Walk).  Products come out as
// 2^48 of themselves.  (Two instructions on eleven per pair of values: 307 -> 317 us for the training step above.)
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;
struct Planes {
    bf16x8 h, m, l;
};
// Eight values of a lane (the k-values of an operand) on their way into planes, two of them at a time: pair w's first terms and what
// is left, then its other two.  slot(): the same in six pieces of 6 to 14 instructions, one behind a matrix instruction each.
struct Split8 {
    u32x4 h, m, l;
    f32x4 r0, r1;
    static __device__ __forceinline__ uint32_t pack(float a, float b) {
        bf16x2 r;
        r[0] = (__bf16)a;
        r[1] = (__bf16)b;
        uint32_t w = __builtin_bit_cast(uint32_t, r);
        asm("" : "+v"(w));              // (taken apart again below: else every half would be converted a second time, by itself)
        return w;
    }
    static __device__ __forceinline__ float lower(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
    static __device__ __forceinline__ float upper(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
    __device__ __forceinline__ void first(int w, float x0, float x1) {
#pragma clang fp contract(off)          // (x0 may be a product: fused with the difference it would be split unrounded, here but not there)
        const float y0 = x0 * kUp, y1 = x1 * kUp;
        const uint32_t word = pack(y0, y1);
        h[w] = word;
        r0[w] = y0 - lower(word);
        r1[w] = y1 - upper(word);
    }
    __device__ __forceinline__ void second(int w) {
#pragma clang fp contract(off)
        const uint32_t word = pack(r0[w], r1[w]);
        m[w] = word;
        l[w] = pack(r0[w] - lower(word), r1[w] - upper(word));
    }
    template <typename X>               // x(e), e = 0 .. 7: the values
    __device__ __forceinline__ void slot(int i, X x) {
        const int b = i < 3 ? 0 : 2;
        if (i % 3 == 0) {
            first(b, x(2 * b), x(2 * b + 1));
            first(b + 1, x(2 * b + 2), x(2 * b + 3));
        } else {
            second(b + i % 3 - 1);
        }
    }
    __device__ __forceinline__ Planes planes() const {
        return Planes{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
    }
};
template <typename X>
__device__ __forceinline__ Planes split8(X x) {
    Split8 t;
#pragma unroll
    for (int i = 0; i < 6; ++i) t.slot(i, x);
    return t.planes();
}
// Instruction i of acc += A B over 16 k-values: the small terms first (m l, l m and l l are below 2^-26 of the product).  The scores are
// summed in the same order in all kernels, with K as A or as B (KEYS_IN_B): a score of the backward is the forward's bit for bit, and
// its error leaves the weight exp(s - lse) where the row has few keys.
template <bool KEYS_IN_B = false>
__device__ __forceinline__ void mma3(f32x16& acc, const Planes& a, const Planes& b, int i) {
    const Planes &k = KEYS_IN_B ? b : a, &q = KEYS_IN_B ? a : b;
    const bf16x8 x = i == 0 ? k.l : i == 2 || i == 3 ? k.m : k.h, y = i == 1 ? q.l : i == 2 || i == 4 ? q.m : q.h;
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(KEYS_IN_B ? y : x, KEYS_IN_B ? x : y, acc, 0, 0, 0);
}
// Two such products in turn, slot(i), i = 0 .. 11, behind instruction i -- in this order: left to the compiler, all of a group's matrix
// instructions stand before its vector instructions and neither runs beside the other.
template <bool KEYS_IN_B = false, typename Slot>
__device__ __forceinline__ void mma3_pair(f32x16& acc0, const Planes& a0, const Planes& b0, f32x16& acc1, const Planes& a1, const Planes& b1, Slot slot) {
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        if (i % 2 == 0) mma3<KEYS_IN_B>(acc0, a0, b0, i / 2);
        else mma3<KEYS_IN_B>(acc1, a1, b1, i / 2);
        slot(i);
        __builtin_amdgcn_sched_barrier(0);
    }
}
// A lane's operand of 16-dim step j out of its row as loaded (f[jj]: dims 8 jj + 4 hg .. + 3): dims 16 j + 4 hg .. + 3 and 8 further on
template <int JJ>
__device__ __forceinline__ auto of_row(const f32x4 (&f)[JJ], int j) {
    return [&f, j](int e) { return f[2 * j + (e >> 2)][e & 3]; };
}
template <int JJ>
__device__ __forceinline__ Planes split_row(const f32x4 (&f)[JJ], int j) { return split8(of_row(f, j)); }
// The 32 rows that a workgroup shares, split, in LDS: per term [32][D], a row's eight values of (step, hg) in one 16-byte piece;
// eight bf16 of padding send 16 consecutive rows to 16 different 16-byte columns.
template <int D>
struct PlanesLds {
    uint16_t x[3][kF32Rows][D + 8];
    // dims d .. d + 3 (d a multiple of 4) of a row
    __device__ __forceinline__ void put(int row, int d, const f32x4& v) {
        const int at = (d & ~15) + 8 * ((d >> 2) & 1) + 4 * ((d >> 3) & 1);
        Split8 t;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            t.first(w, v[2 * w], v[2 * w + 1]);
            t.second(w);
        }
        *reinterpret_cast<u32x2*>(&x[0][row][at]) = u32x2{t.h[0], t.h[1]};
        *reinterpret_cast<u32x2*>(&x[1][row][at]) = u32x2{t.m[0], t.m[1]};
        *reinterpret_cast<u32x2*>(&x[2][row][at]) = u32x2{t.l[0], t.l[1]};
    }
    __device__ __forceinline__ Planes get(int row, int j, int hg) const {
        const int at = 16 * j + 8 * hg;
        return Planes{*reinterpret_cast<const bf16x8*>(&x[0][row][at]), *reinterpret_cast<const bf16x8*>(&x[1][row][at]),
                      *reinterpret_cast<const bf16x8*>(&x[2][row][at])};
    }
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
// a value leave the product and are added to the columns that see them alone.  What that leaves non-finite has seen such a value; as three terms
// an Inf is Inf and NaNs, so is a finite value from 2^104 on (Planes), and a product beyond 2^80 overflows: those entries are taken from a third
// walk, on fp32 instructions.
// (Looking at the operands in every such block cost 4 % of the forward and 4 to 14 % of the gradients, most of it in registers; looking
// at the result costs 1 %, 0.2 us of the smallest forward.)
enum class Walk { kFast, kCareful, kFp32 };
// A walk's result; the last walk fills in what the one before left non-finite (same thread, same elements).
template <bool FILL>
__device__ __forceinline__ void put(float* dst, const f32x4& x) {
    if (!FILL) {
        *reinterpret_cast<f32x4_a4*>(dst) = x;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (!isfinite(dst[e])) dst[e] = x[e];
    }
}

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
// Sets the rows of an operand that hold a value that is not finite, or not as bf16 terms (SPLIT), to zero; returned: bit r, row r
// of the block (x[g] holds row acc_row(g, hg)).
template <bool SPLIT, int DB>
__device__ __forceinline__ uint32_t take_out(float (&x)[16][DB], int hg) {
    constexpr float kLimit = SPLIT ? kUp * 1.00390625f : 1.f;      // (a value that is rounded up to 2^104 overflows with this)
    uint32_t rows = 0u;
#pragma unroll
    for (int g = 0; g < 16; ++g) {
        float z = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) z = fmaf(x[g][db] * kLimit, 0.f, z);
        const unsigned long long lanes = __ballot(z != z);
        const bool lower = uint32_t(lanes) != 0u, upper = uint32_t(lanes >> 32) != 0u;
        rows |= (lower ? 1u << acc_row(g, 0) : 0u) | (upper ? 1u << acc_row(g, 1) : 0u);
#pragma unroll
        for (int db = 0; db < DB; ++db) x[g][db] = (hg ? upper : lower) ? 0.f : x[g][db];
    }
    return rows;
}
// weight x row r (uniform; `row` points at its dim 4 hg) added to the columns that see it; w: the block's weights; SPLIT: acc is 2^48 of the sum
template <bool SPLIT, int D>
__device__ __forceinline__ void add_row(f32x16 (&acc)[D / 32], const f32x16& w, const float* row, int r, int n, bool seen) {
    float weight = w[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) weight = i == 4 * (r >> 3) + (r & 3) ? w[i] : weight;
    weight = __shfl(weight, n + 32 * ((r >> 2) & 1)) * (SPLIT ? 1.f / kDown : 1.f);
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
    union {                       // the rows are read in the loop, the merge comes after it
        PlanesLds<D> q;
        MergeLds<D> merge;
    };
    float m[kF32Waves][kF32Rows], l[kF32Waves][kF32Rows];
    int bad[kF32Waves];
};

// false: the result is not finite, nothing has been stored
template <int D, Walk WALK>
__device__ __forceinline__ bool prefill_f32_walk(const HeadRows& at, float* __restrict__ out, float* __restrict__ lse,
                                                 const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                 PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    constexpr int JJ = D / 8, DB = D / 32, KS = D / 16;
    constexpr bool CAREFUL = WALK != Walk::kFast, FP32 = WALK == Walk::kFp32;
    constexpr float kUnit = FP32 ? 1.f : kDown;              // a product's unit
    const float s_scale = scale * kUnit;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    FwdF32Smem<D>& sm = *reinterpret_cast<FwdF32Smem<D>*>(smem_raw);
    const int hk = at.hk, hq = at.hq;
    const WorkItem it = pv.sorted[at.rank];
    const OwnRows own = own_rows(it, at.sub);
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
    const int64_t rowhead = int64_t(pv.perm[it.a_base + own.first + min(row, own.count - 1)]) * n_q_heads + hq;
    f32x4 qf[FP32 ? JJ : 1];
    if constexpr (FP32) {
        const float* qp = q + (my_tok * n_q_heads + hq) * D + 4 * hg;
#pragma unroll
        for (int jj = 0; jj < JJ; ++jj) qf[jj] = *reinterpret_cast<const f32x4*>(qp + 8 * jj);
    } else {
#pragma unroll
        for (int d = 4 * part; d < D; d += 32) sm.q.put(row, d, *reinterpret_cast<const f32x4*>(q + rowhead * D + d));
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
    if constexpr (!FP32) __syncthreads();
    for (int t = wave; t < n_blocks; t += kF32Waves) {
        const int tok_next = key_token(t + kF32Waves);
        // ---- S^T = K Q^T; the value rows of the block are requested beside it ----
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
        float vf[16][DB];
        auto load_v = [&](int g) {
            const float* vp = v_lane + __shfl(tok, acc_row(g, hg)) * stride;
#pragma unroll
            for (int db = 0; db < DB; ++db) vf[g][db] = vp[32 * db];
        };
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                load_v(g);
#pragma unroll
                for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj)
#pragma unroll
                    for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[jj][e], qf[jj][e], s, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            Planes a = split_row(kf, 0);
#pragma unroll
            for (int j = 0; j < KS; ++j) {
#pragma unroll
                for (int g = j * 16 / KS; g < (j + 1) * 16 / KS; ++g) load_v(g);
                const Planes b = sm.q.get(n, j, hg);
                Split8 next;
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    mma3(s, a, b, i);
                    if (j + 1 < KS) next.slot(i, of_row(kf, j + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (j + 1 < KS) a = next.planes();
            }
        }
        // ---- softmax over the block: lane = query row, register i = column acc_row(i, hg) ----
        const bool in_a = t < blocks_a;
        const int c0 = (in_a ? t : t - blocks_a) * kF32Rows;
        const int limit = in_a ? my_row + 1 : my_vis;                      // columns < limit are visible
        const int limit_min = in_a ? own.first + 1 : first_vis;            // ... to every row
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] *= s_scale;
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
            s[i] = exp_f32(s[i] - m_use);
            l_run += s[i];
        }
        if (CAREFUL && c0 + kF32Rows > limit_min) {
            for (uint32_t rows = take_out<!FP32>(vf, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<!FP32, D>(o_acc, s, v + __shfl(tok, r) * stride + int64_t(hk) * D + 4 * hg, r, n, c0 + r < limit);
            }
        }
        // ---- O^T += V^T P^T; the next block's keys are requested beside it ----
        tok = tok_next;
        const float* kp = k_lane + tok * stride;
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
#pragma unroll
                for (int db = 0; db < DB; ++db) o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[g][db], s[g], o_acc[db], 0, 0, 0);
#pragma unroll
                for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) kf[jj] = *reinterpret_cast<const f32x4*>(kp + 8 * jj);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            auto v_step = [&](int x) { return [&vf, x](int e) { return vf[8 * (x / DB) + e][x % DB]; }; };      // x: (16 keys, 32 dims)
            Planes a0 = split8(v_step(0)), a1 = split8(v_step(1)), p = split8([&](int e) { return s[e]; });
            Split8 p_next;
#pragma unroll
            for (int x = 0; x < 2 * DB; x += 2) {
#pragma unroll
                for (int jj = 2 * x; jj < 2 * x + 4; ++jj) kf[jj] = *reinterpret_cast<const f32x4*>(kp + 8 * jj);
                if (x == DB) p = p_next.planes();
                Split8 next0, next1;
                mma3_pair(o_acc[x % DB], a0, p, o_acc[(x + 1) % DB], a1, p, [&](int i) {
                    if (x + 2 < 2 * DB) {
                        if (i < 6) next0.slot(i, v_step(x + 2));
                        else next1.slot(i - 6, v_step(x + 3));
                    }
                    if (x == DB - 2 && i % 2 == 1) p_next.slot(i / 2, [&](int e) { return s[8 + e]; });
                });
                if (x + 2 < 2 * DB) {
                    a0 = next0.planes();
                    a1 = next1.planes();
                }
            }
        }
    }
    // ---- merge of the four waves' states ----
    bool bad = false;
    if (!FP32) {
        float z = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) z = fmaf(o_acc[db][i], 0.f, z);
        bad = __any(z != z);
    }
    if constexpr (!FP32) __syncthreads();                                  // (the rows of q lie where the states meet)
    park<D>(sm.merge.o[wave], o_acc, n, hg);
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (hg == 0) {
        sm.m[wave][n] = m_run;
        sm.l[wave][n] = l_tot;
    }
    if (!FP32 && lane == 0) sm.bad[wave] = bad;
    __syncthreads();
    const bool finite = FP32 || !any_wave(sm.bad);
    if (!CAREFUL && !finite) return false;
    float m_all = -INFINITY, wt[kF32Waves], den = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) m_all = fmaxf(m_all, sm.m[w][row]);           // finite: column 0 of the own stream is visible
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
        wt[w] = expf(sm.m[w][row] - m_all);                                // (0 for a wave that saw nothing)
        den = fmaf(wt[w], sm.l[w][row], den);
    }
    const float inv = kUnit / den;
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
        for (int db = 0; db < DB; ++db) put<FP32>(out + rowhead * D + 4 * part + 32 * db, a[db]);
        if (lse && part == 0 && !(FP32 && isfinite(lse[rowhead]))) lse[rowhead] = m_all + logf(den);
    }
    return finite;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 2) void prefill_f32_kernel(float* __restrict__ out, float* __restrict__ lse,
                                                                        const float* __restrict__ q, const float* __restrict__ k,
                                                                        const float* __restrict__ v, PlanView pv, int n_q_heads,
                                                                        int n_kv_heads, float scale) {
    HeadRows at(blockIdx.x, 1, pv, n_q_heads, n_kv_heads);
    if (prefill_f32_walk<D, Walk::kFast>(at, out, lse, q, k, v, pv, n_q_heads, n_kv_heads, scale)) return;
    at.again(0);
    if (prefill_f32_walk<D, Walk::kCareful>(at, out, lse, q, k, v, pv, n_q_heads, n_kv_heads, scale)) return;
    at.again(0);
    prefill_f32_walk<D, Walk::kFp32>(at, out, lse, q, k, v, pv, n_q_heads, n_kv_heads, scale);
}

// --------------------------------------------------------------------------
// Backward, query side: delta_i = dO_i . O_i, dQ_i = scale sum_j dS_ij K_j
// --------------------------------------------------------------------------
template <int D, int HB>
struct DqF32Smem {
    union {                       // the rows are read in the loop, the merge comes after it
        struct {
            PlanesLds<D> q3[HB], d_out3[HB];
        };
        struct {                  // (the careful walk)
            RowsLds<D> q, d_out;
        };
        MergeLds<D> merge;
    };
    float lse[HB][kF32Rows], delta[HB][kF32Rows];
    int bad[kF32Waves];
};

// false: the result is not finite, nothing but delta has been stored
template <int D, int HB, Walk WALK>
__device__ __forceinline__ bool bwd_dq_f32_walk(const HeadRows& at, float* __restrict__ dq, float* __restrict__ delta_out,
                                                const float* __restrict__ d_out, const float* __restrict__ q, const float* __restrict__ k,
                                                const float* __restrict__ v, const float* __restrict__ out, const float* __restrict__ lse,
                                                PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    constexpr int JJ = D / 8, DB = D / 32, KS = D / 16;
    constexpr bool CAREFUL = WALK != Walk::kFast, FP32 = WALK == Walk::kFp32;
    constexpr float kUnit = FP32 ? 1.f : kDown;              // a product's unit
    const float s_scale = scale * kUnit;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    DqF32Smem<D, HB>& sm = *reinterpret_cast<DqF32Smem<D, HB>*>(smem_raw);
    const int hk = at.hk, hq = at.hq;
    const WorkItem it = pv.sorted[at.rank];
    const OwnRows own = own_rows(it, at.sub);
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
#pragma unroll
    for (int h = 0; h < HB; ++h) {
        const int64_t rh = rowhead + h;
        float dl = 0.f;
#pragma unroll
        for (int d = 4 * part; d < D; d += 32) {
            const f32x4 a = *reinterpret_cast<const f32x4_a4*>(d_out + rh * D + d), o = *reinterpret_cast<const f32x4_a4*>(out + rh * D + d);
            const f32x4 x = *reinterpret_cast<const f32x4_a4*>(q + rh * D + d);
            if constexpr (FP32) {
                *reinterpret_cast<f32x4*>(&sm.q.x[row][d]) = x;
                *reinterpret_cast<f32x4*>(&sm.d_out.x[row][d]) = a;
            } else {
                sm.q3[h].put(row, d, x);
                sm.d_out3[h].put(row, d, a);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) dl = fmaf(a[e], o[e], dl);
        }
        dl += __shfl_xor(dl, 1);
        dl += __shfl_xor(dl, 2);
        dl += __shfl_xor(dl, 4);
        if (part == 0) {
            sm.lse[h][row] = lse[rh];
            sm.delta[h][row] = dl;
            if (row < own.count) delta_out[rh] = dl;
        }
    }
    __syncthreads();
    float my_lse[HB], my_delta[HB];
    f32x16 acc[HB][DB];
#pragma unroll
    for (int h = 0; h < HB; ++h) {
        my_lse[h] = sm.lse[h][n];
        my_delta[h] = sm.delta[h][n];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[h][db][i] = 0.f;
    }
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
        f32x16 s[HB], dp[HB];
#pragma unroll
        for (int h = 0; h < HB; ++h)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[h][i] = dp[h][i] = 0.f;
        float kt[16][DB];
        auto load_kt = [&](int g) {
            const float* kp = k_cols + __shfl(tok, acc_row(g, hg)) * stride;
#pragma unroll
            for (int db = 0; db < DB; ++db) kt[g][db] = kp[32 * db];
        };
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                load_kt(g);
#pragma unroll
                for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) {
                    const f32x4 qv = *reinterpret_cast<const f32x4*>(&sm.q.x[n][8 * jj + 4 * hg]);
                    const f32x4 ov = *reinterpret_cast<const f32x4*>(&sm.d_out.x[n][8 * jj + 4 * hg]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        s[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[jj][e], qv[e], s[0], 0, 0, 0);
                        dp[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[jj][e], ov[e], dp[0], 0, 0, 0);
                    }
                }
            }
        } else {
            Planes a0 = split_row(kf, 0), a1 = split_row(vf, 0);
#pragma unroll
            for (int j = 0; j < KS; ++j) {
#pragma unroll
                for (int g = j * 16 / KS; g < (j + 1) * 16 / KS; ++g) load_kt(g);
                Split8 next0, next1;
                auto keys = [&](int i) {
                    if (j + 1 < KS) next0.slot(i, of_row(kf, j + 1));
                };
                auto values = [&](int i) {
                    if (j + 1 < KS) next1.slot(i, of_row(vf, j + 1));
                };
                if constexpr (HB == 2) {
                    mma3_pair(s[0], a0, sm.q3[0].get(n, j, hg), s[1], a0, sm.q3[1].get(n, j, hg), [&](int i) { if (i % 2 == 0) keys(i / 2); });
                    mma3_pair(dp[0], a1, sm.d_out3[0].get(n, j, hg), dp[1], a1, sm.d_out3[1].get(n, j, hg), [&](int i) { if (i % 2 == 0) values(i / 2); });
                } else {
                    mma3_pair(s[0], a0, sm.q3[0].get(n, j, hg), dp[0], a1, sm.d_out3[0].get(n, j, hg), [&](int i) { i < 6 ? keys(i) : values(i - 6); });
                }
                if (j + 1 < KS) {
                    a0 = next0.planes();
                    a1 = next1.planes();
                }
            }
        }
        const bool in_a = t < blocks_a;
        const int c0 = (in_a ? t : t - blocks_a) * kF32Rows;
        const int limit = in_a ? my_row + 1 : my_vis, limit_min = in_a ? own.first + 1 : first_vis;
        const bool partial = c0 + kF32Rows > limit_min;
#pragma unroll
        for (int h = 0; h < HB; ++h)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float p = exp_f32(fmaf(s[h][i], s_scale, -my_lse[h]));
                if (partial) p = c0 + acc_row(i, hg) < limit ? p : 0.f;
                s[h][i] = p * fmaf(dp[h][i], kUnit, -my_delta[h]) * scale;
                if (CAREFUL) s[h][i] = c0 + acc_row(i, hg) < limit ? s[h][i] : 0.f;
            }
        if (CAREFUL && partial) {
            for (uint32_t rows = take_out<!FP32>(kt, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<!FP32, D>(acc[0], s[0], k_rows + __shfl(tok, r) * stride, r, n, c0 + r < limit);
            }
        }
        // ---- dQ^T += K^T dS^T; the next block's rows are requested beside it ----
        tok = tok_next;
        auto load_rows = [&](int jj) {
            kf[jj] = *reinterpret_cast<const f32x4_a4*>(k_rows + tok * stride + 8 * jj);
            vf[jj] = *reinterpret_cast<const f32x4_a4*>(v_rows + tok * stride + 8 * jj);
        };
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
#pragma unroll
                for (int db = 0; db < DB; ++db) acc[0][db] = __builtin_amdgcn_mfma_f32_32x32x2f32(kt[g][db], s[0][g], acc[0][db], 0, 0, 0);
#pragma unroll
                for (int jj = g * JJ / 16; jj < (g + 1) * JJ / 16; ++jj) load_rows(jj);
            }
        } else {
            auto k_step = [&](int x) { return [&kt, x](int e) { return kt[8 * (x / DB) + e][x % DB]; }; };      // x: (16 keys, 32 dims)
            Planes a0 = split8(k_step(0)), a1 = split8(k_step(1)), ds[HB];
            Split8 ds_next[HB];
#pragma unroll
            for (int h = 0; h < HB; ++h) ds[h] = split8([&](int e) { return s[h][e]; });
#pragma unroll
            for (int x = 0; x < 2 * DB; x += 2) {
#pragma unroll
                for (int jj = 2 * x; jj < 2 * x + 4; ++jj) load_rows(jj);
#pragma unroll
                for (int h = 0; h < HB; ++h)
                    if (x == DB) ds[h] = ds_next[h].planes();
                Split8 next0, next1;
                auto rows = [&](int i) {                    // the operands of the next two steps, i = 0 .. 11
                    if (x + 2 < 2 * DB) {
                        if (i < 6) next0.slot(i, k_step(x + 2));
                        else next1.slot(i - 6, k_step(x + 3));
                    }
                };
                auto weights = [&](int i, int h) {          // dS of the other 16 keys, i = 0 .. 5
                    if (x == DB - 2) ds_next[h].slot(i, [&](int e) { return s[h][8 + e]; });
                };
                if constexpr (HB == 2) {
#pragma unroll
                    for (int y = 0; y < 2; ++y)
                        mma3_pair(acc[0][(x + y) % DB], y ? a1 : a0, ds[0], acc[1][(x + y) % DB], y ? a1 : a0, ds[1], [&](int i) {
                            if (i % 2 == 0) rows(6 * y + i / 2);
                            else weights(i / 2, y);
                        });
                } else {
                    mma3_pair(acc[0][x % DB], a0, ds[0], acc[0][(x + 1) % DB], a1, ds[0], [&](int i) {
                        rows(i);
                        if (i % 2 == 1) weights(i / 2, 0);
                    });
                }
                if (x + 2 < 2 * DB) {
                    a0 = next0.planes();
                    a1 = next1.planes();
                }
            }
        }
    }
    f32x4 a[HB][DB];
    float z = 0.f;
#pragma unroll
    for (int h = 0; h < HB; ++h) {
        __syncthreads();
        park<D>(sm.merge.o[wave], acc[h], n, hg);
        __syncthreads();
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            a[h][db] = *reinterpret_cast<const f32x4*>(&sm.merge.o[0][row][4 * part + 32 * db]);
#pragma unroll
            for (int w = 1; w < kF32Waves; ++w) a[h][db] += *reinterpret_cast<const f32x4*>(&sm.merge.o[w][row][4 * part + 32 * db]);
            z = fold_finite(z, a[h][db]);
            a[h][db] *= kUnit;
        }
    }
    bool finite = true;
    if (!FP32) {
        const bool bad = __any(z != z);
        if (lane == 0) sm.bad[wave] = bad;
        __syncthreads();
        finite = !any_wave(sm.bad);
        if (!CAREFUL && !finite) return false;
    }
    if (row < own.count) {
#pragma unroll
        for (int h = 0; h < HB; ++h)
#pragma unroll
            for (int db = 0; db < DB; ++db) put<FP32>(dq + (rowhead + h) * D + 4 * part + 32 * db, a[h][db]);
    }
    return finite;
}

template <int D, int HB>
__global__ __launch_bounds__(64 * kF32Waves, HB == 2 ? 1 : 2) void bwd_dq_f32_kernel(float* __restrict__ dq, float* __restrict__ delta_out,
                                                                                     const float* __restrict__ d_out, const float* __restrict__ q,
                                                                                     const float* __restrict__ k, const float* __restrict__ v,
                                                                                     const float* __restrict__ out, const float* __restrict__ lse,
                                                                                     PlanView pv, int n_q_heads, int n_kv_heads, float scale) {
    HeadRows at(blockIdx.x, HB, pv, n_q_heads, n_kv_heads);
    if (bwd_dq_f32_walk<D, HB, Walk::kFast>(at, dq, delta_out, d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale)) return;
    for (int h = 0; h < HB; ++h) {
        at.again(h);
        if (!bwd_dq_f32_walk<D, 1, Walk::kCareful>(at, dq, delta_out, d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale)) {
            at.again(0);
            bwd_dq_f32_walk<D, 1, Walk::kFp32>(at, dq, delta_out, d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale);
        }
    }
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
            PlanesLds<D> k3, v3;
        };
        struct {                  // (the careful walk)
            RowsLds<D> k, v;
        };
        MergeLds<D> merge;
    };
    int bad[kF32Waves];
};

// false: the result is not finite, nothing has been stored
template <int D, Walk WALK>
__device__ __forceinline__ bool bwd_dkv_f32_walk(unsigned block, float* __restrict__ dk, float* __restrict__ dv,
                                                 const float* __restrict__ delta, const float* __restrict__ d_out,
                                                 const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                 const float* __restrict__ lse, PlanView pv, int n_q_heads, int n_kv_heads, float scale,
                                                 int parts, float* __restrict__ partial, int64_t partial_stride) {
    constexpr int JJ = D / 8, DB = D / 32, KS = D / 16;
    constexpr bool CAREFUL = WALK != Walk::kFast, FP32 = WALK == Walk::kFp32;
    constexpr float kUnit = FP32 ? 1.f : kDown;              // a product's unit
    const float s_scale = scale * kUnit;
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
        const f32x4 kx = *reinterpret_cast<const f32x4_a4*>(k + keyhead * D + d), vx = *reinterpret_cast<const f32x4_a4*>(v + keyhead * D + d);
        if constexpr (FP32) {
            *reinterpret_cast<f32x4*>(&sm.k.x[row][d]) = kx;
            *reinterpret_cast<f32x4*>(&sm.v.x[row][d]) = vx;
        } else {
            sm.k3.put(row, d, kx);
            sm.v3.put(row, d, vx);
        }
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
        int row_tok[16];
#pragma unroll
        for (int g = 0; g < 16; ++g) row_tok[g] = __shfl(tok, acc_row(g, hg));
        auto load_cols = [&](int g) {
            const int64_t off = (int64_t(row_tok[g]) * n_q_heads + cur.hq) * D + n;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                qt[g][db] = q[off + 32 * db];
                ot[g][db] = d_out[off + 32 * db];
            }
        };
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                load_cols(g);
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
        } else {
            Planes a0 = split_row(qf, 0), a1 = split_row(of, 0), b0 = sm.k3.get(n, 0, hg), b1 = sm.v3.get(n, 0, hg);
#pragma unroll
            for (int j = 0; j < KS; ++j) {
#pragma unroll
                for (int g = j * 16 / KS; g < (j + 1) * 16 / KS; ++g) load_cols(g);
                const Planes k_next = sm.k3.get(n, min(j + 1, KS - 1), hg), v_next = sm.v3.get(n, min(j + 1, KS - 1), hg);
                Split8 next0, next1;
                mma3_pair<true>(s, a0, b0, dp, a1, b1, [&](int i) {
                    if (j + 1 < KS) {
                        if (i < 6) next0.slot(i, of_row(qf, j + 1));
                        else next1.slot(i - 6, of_row(of, j + 1));
                    }
                });
                b0 = k_next;
                b1 = v_next;
                if (j + 1 < KS) {
                    a0 = next0.planes();
                    a1 = next1.planes();
                }
            }
        }
        // register i <-> row acc_row(i, hg) of the block
        const bool full = __builtin_amdgcn_readfirstlane(lim) > last_key && cur.row0 + kF32Rows <= cur.end;    // (limits do not decrease along the rows)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = acc_row(i, hg);
            float p = exp_f32(fmaf(s[i], s_scale, -__shfl(l_row, r)));
            if (!full) p = my_key < __shfl(lim, r) ? p : 0.f;
            s[i] = p;
            dp[i] = p * fmaf(dp[i], kUnit, -__shfl(d_row, r)) * scale;
            if (CAREFUL && !full) dp[i] = my_key < __shfl(lim, r) ? dp[i] : 0.f;
        }
        if (CAREFUL && !full) {
            auto row_of = [&](const float* x, int r) { return x + (int64_t(__shfl(tok, r)) * n_q_heads + cur.hq) * D + 4 * hg; };
            for (uint32_t rows = take_out<!FP32>(ot, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<!FP32, D>(dv_acc, s, row_of(d_out, r), r, n, my_key < __shfl(lim, r));
            }
            for (uint32_t rows = take_out<!FP32>(qt, hg); rows != 0u; rows &= rows - 1u) {
                const int r = __ffs(rows) - 1;
                add_row<!FP32, D>(dk_acc, dp, row_of(q, r), r, n, my_key < __shfl(lim, r));
            }
        }
        // ---- dV^T += dO^T P, dK^T += Q^T dS; the next rows are requested beside them ----
        cur = iter_at(x + kF32Waves);
        row_info(cur);
        if constexpr (FP32) {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    dv_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(ot[g][db], s[g], dv_acc[db], 0, 0, 0);
                    dk_acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(qt[g][db], dp[g], dk_acc[db], 0, 0, 0);
                }
                load_rows(cur, g * JJ / 16, (g + 1) * JJ / 16);
            }
        } else {
            auto o_step = [&](int x) { return [&ot, x](int e) { return ot[8 * (x / DB) + e][x % DB]; }; };      // x: (16 rows, 32 dims)
            auto q_step = [&](int x) { return [&qt, x](int e) { return qt[8 * (x / DB) + e][x % DB]; }; };
            Planes a0 = split8(o_step(0)), a1 = split8(q_step(0)), p = split8([&](int e) { return s[e]; }), ds = split8([&](int e) { return dp[e]; });
            Split8 p_next, ds_next;
#pragma unroll
            for (int x = 0; x < 2 * DB; ++x) {
                load_rows(cur, 2 * x, 2 * x + 2);
                if (x == DB) {
                    p = p_next.planes();
                    ds = ds_next.planes();
                }
                Split8 next0, next1;
                mma3_pair(dv_acc[x % DB], a0, p, dk_acc[x % DB], a1, ds, [&](int i) {
                    if (x + 1 < 2 * DB) {
                        if (i < 6) next0.slot(i, o_step(x + 1));
                        else next1.slot(i - 6, q_step(x + 1));
                    }
                    if (x == DB - 2 && i % 2 == 1) p_next.slot(i / 2, [&](int e) { return s[8 + e]; });
                    if (x == DB - 1 && i % 2 == 1) ds_next.slot(i / 2, [&](int e) { return dp[8 + e]; });
                });
                if (x + 1 < 2 * DB) {
                    a0 = next0.planes();
                    a1 = next1.planes();
                }
            }
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
            a[which][db] *= kUnit;
        }
    }
    bool finite = true;
    if (!FP32) {
        const bool bad = __any(z != z);
        if (lane == 0) sm.bad[wave] = bad;
        __syncthreads();
        finite = !any_wave(sm.bad);
        if (!CAREFUL && !finite) return false;
    }
    if (row < own.count) {
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            float* dst = (parts > 1 ? partial + ((which == 0 ? parts : 0) + part_of) * partial_stride : which == 0 ? dv : dk) + keyhead * D;
#pragma unroll
            for (int db = 0; db < DB; ++db) put<FP32>(dst + 4 * part + 32 * db, a[which][db]);
        }
    }
    return finite;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, 1) void bwd_dkv_f32_kernel(float* __restrict__ dk, float* __restrict__ dv,
                                                                        const float* __restrict__ delta, const float* __restrict__ d_out,
                                                                        const float* __restrict__ q, const float* __restrict__ k,
                                                                        const float* __restrict__ v, const float* __restrict__ lse,
                                                                        PlanView pv, int n_q_heads, int n_kv_heads, float scale, int parts,
                                                                        float* __restrict__ partial, int64_t partial_stride) {
    unsigned block = blockIdx.x;
    if (bwd_dkv_f32_walk<D, Walk::kFast>(block, dk, dv, delta, d_out, q, k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride)) return;
    asm volatile("" : "+s"(block));               // (nothing of a walk is kept for the next: the registers are full)
    if (bwd_dkv_f32_walk<D, Walk::kCareful>(block, dk, dv, delta, d_out, q, k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride)) return;
    asm volatile("" : "+s"(block));
    bwd_dkv_f32_walk<D, Walk::kFp32>(block, dk, dv, delta, d_out, q, k, v, lse, pv, n_q_heads, n_kv_heads, scale, parts, partial, partial_stride);
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
        auto query_side = [&](auto htag) -> st_status {
            constexpr int HB = decltype(htag)::value;
            const st_status r = with_smem(&bwd_dq_f32_kernel<D, HB>, sizeof(DqF32Smem<D, HB>));
            if (r != ST_OK) return r;
            hipLaunchKernelGGL((bwd_dq_f32_kernel<D, HB>), dim3((unsigned)(qblocks / HB)), dim3(64 * kF32Waves), sizeof(DqF32Smem<D, HB>), s, dq, delta,
                               d_out, q, k, v, out, lse, pv, n_q_heads, n_kv_heads, scale);
            return ST_OK;
        };
        st_status r = with_smem(&bwd_dkv_f32_kernel<D>, sizeof(DkvF32Smem<D>));
        if (r != ST_OK) return r;
        // Two query heads of a KV head per workgroup, one wave per SIMD, with heads of 128 dims: keys and values are split once for both
        // (2 x 1,000 tokens, 16 / 8 heads, gradients 254 -> 217 us).  With heads of 64 two waves of a head each fit a SIMD and are the faster
        // (8 / 4 heads, 90 against 92; 1 x 1,200 92 against 99).
        if constexpr (D == 128) r = n_q_heads / n_kv_heads % 2 == 0 ? query_side(std::integral_constant<int, 2>{}) : query_side(std::integral_constant<int, 1>{});
        else r = query_side(std::integral_constant<int, 1>{});
        if (r != ST_OK) return r;
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
