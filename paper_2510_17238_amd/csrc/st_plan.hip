// Segment-table builder: turns per-token (stream, segment, position) ids into the
// tables that replace the dense additive mask of Eq. 2 (Sec. 3.2; Appendix E.1).
//
// Attention is indifferent to the order of keys, and the streaming mask is a pure
// function of the ids, so everything is expressed in "grouped stream-compact
// order": per sequence, the source tokens by position, then the reasoning tokens
// by position -- the paper's own training layout.  There the mask is two causal
// triangles (source x source, reasoning x reasoning) plus a staircase rectangle
// (reasoning rows x a prefix of the source stream), and a reasoning row needs just
// one number: how many source tokens it sees.
//
// All tables are built by two small integer kernels (one workgroup per sequence; the order of the work items), no host
// round trip.
#include <limits.h>

#include <algorithm>
#include <new>
#include <type_traits>

#include "st_plan.h"

namespace st {

static inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

static int32_t m_max_bound(int32_t batch, int64_t n_tokens) { return int32_t(n_tokens / kTileM) + 2 * batch; }

struct WsLayout {
    size_t cu, n_src, n_rsn, pairs, flag, perm, seg_c, vis, cost, items, sorted, tiles, total;
};

static WsLayout ws_layout(int32_t batch, int64_t n_tokens) {
    WsLayout L;
    const size_t m = size_t(m_max_bound(batch, n_tokens));
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    L.cu = take(sizeof(int32_t) * (batch + 1));
    L.n_src = take(sizeof(int32_t) * batch);
    L.n_rsn = take(sizeof(int32_t) * batch);
    L.pairs = take(sizeof(unsigned long long) * batch);
    L.flag = take(sizeof(int32_t));
    L.perm = take(sizeof(int32_t) * n_tokens);
    L.seg_c = take(sizeof(int32_t) * n_tokens);
    L.vis = take(sizeof(int32_t) * n_tokens);
    L.cost = take(sizeof(int32_t) * m);
    L.items = take(sizeof(WorkItem) * m);
    L.sorted = take(sizeof(WorkItem) * m);
    L.tiles = take(sizeof(TileInfo) * size_t(n_tokens / kTileN + 2 * batch));
    L.total = off;
    return L;
}

constexpr int kPlanThreads = 1024;
constexpr int kPre = 16;                 // tokens of a sequence that a thread keeps in registers through all passes (16,384 a sequence)
constexpr int kSegLds = 8192;            // source tokens of a sequence whose segment ids are searched in LDS
constexpr int kAloneMax = 256;           // work items up to which the workgroup of a single sequence orders them itself
constexpr int kSmallTable = 64, kLargeTable = 512;      // up to this batch cu_seqlens travels as a kernel argument

template <int CAP>
struct HostOffsets {                     // cu_seqlens, batch + 1 entries
    int32_t v[CAP + 1];
};

// ---- fill kernel that clears the validation flag (a kernel, so that the build can be recorded into a HIP graph) ----
__global__ void plan_clear_kernel(int32_t* flag) {
    if (threadIdx.x == 0) *flag = 0;
}

__device__ __forceinline__ int item_slots(int n) { return (n + kTileM - 1) / kTileM + 1; }      // work items of a sequence of n tokens, one spare
__device__ __forceinline__ int tile_slots(int n) { return (n + kTileN - 1) / kTileN + 1; }      // packed key tiles: ceil(S / 64) + ceil(R / 64) at most

__device__ __forceinline__ int full_tiles(int limit, int n_cols) {
    // key tiles whose in-range columns are all < limit
    return n_cols <= limit ? (n_cols + kTileN - 1) / kTileN : limit / kTileN;
}

struct PlanOut {                         // the tables of the workspace
    int32_t *cu, *n_src, *n_rsn, *perm, *seg_c, *vis, *flag, *cost;
    unsigned long long* pairs;
    WorkItem *items, *sorted;
    TileInfo* tiles;
};

// ---- kernel 1: one workgroup per sequence ------------------------------------------------------
// (1) rank every token inside its stream -> perm / seg_c in grouped compact order, stream sizes;
// (2) per compact row the number of visible source tokens (binary search over the source segment
//     ids), the visible-pair count of the sequence, and the optional ordering checks;
// (3) the sequence's work items and their sort keys, and what the packing kernels need to know of its key tiles.
// The ids of the first kPre chunks of 1,024 tokens are fetched once, up front, and stay in registers; the segment ids of the
// source stream go to LDS as they are ranked: up to 16K tokens the tables are written and not read back but for the items'
// few rows, and all chunks are ranked with three barriers.  Both kernels together, with a pass over memory for each of (1) and
// (2), a barrier per chunk and the items in one workgroup, before -> now: 4 x 4K tokens 22.6 -> 16.2 us, 8 x 16K 102 -> 30,
// 96 sequences of 60 to 900 tokens (whose offsets went over in three copies) 47 -> 16.
template <int CAP>
__global__ __launch_bounds__(kPlanThreads) void plan_sequence_kernel(const int32_t* __restrict__ stream_ids,
                                                                     const int32_t* __restrict__ segment_ids,
                                                                     const int32_t* __restrict__ positions, PlanOut o, int validate,
                                                                     int seq_major, int batch, HostOffsets<CAP> offsets) {
    constexpr int WAVES = kPlanThreads / 64;
    static_assert(kPre * WAVES == 256, "the counts of all chunks and waves are scanned by four waves");
    __shared__ int s_cnt[kPre * WAVES], s_sum[4], s_tail[2][WAVES], s_before[2];
    __shared__ unsigned long long s_pairs[WAVES];
    __shared__ int s_seg[kSegLds];            // segment ids of the source stream, then INT_MAX: the bisection below stays in LDS
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // CAP > 0: cu_seqlens travels as a kernel argument (no separate launch to publish it), and workgroup 0 writes the device
    // copy that later kernels use.  CAP = 0: it was copied to o.cu beforehand.
    auto cu_at = [&](int i) { return CAP > 0 ? offsets.v[CAP > 0 ? i : 0] : o.cu[i]; };
    const int t0 = cu_at(b), t1 = cu_at(b + 1), n = t1 - t0;

    int pre_stream[kPre], pre_seg[kPre], pre_rank[kPre];
#pragma unroll
    for (int j = 0; j < kPre; ++j) {
        const int t = t0 + j * kPlanThreads + threadIdx.x;
        pre_stream[j] = t < t1 ? stream_ids[t] : -1;
        pre_seg[j] = t < t1 ? segment_ids[t] : 0;
    }
    if (CAP > 0 && b == 0)
        for (int i = threadIdx.x; i <= batch; i += kPlanThreads) o.cu[i] = cu_at(i);
    if (wave == WAVES - 1) {
        // work item slots and packed tiles of the sequences before this one
        int slots = 0, tiles = 0;
        for (int i = lane; i < b; i += 64) {
            const int len = cu_at(i + 1) - cu_at(i);
            slots += item_slots(len);
            tiles += tile_slots(len);
        }
        for (int d = 32; d > 0; d >>= 1) {
            slots += __shfl_xor(slots, d);
            tiles += __shfl_xor(tiles, d);
        }
        if (lane == 0) {
            s_before[0] = slots;
            s_before[1] = tiles;
        }
    }

    // Ranks.  Sources of (chunk j, wave w), counted by ballots and scanned in that order: the number of sources before a token
    // is the scanned count plus the ballot's lower lanes.
    unsigned long long below[kPre];
#pragma unroll
    for (int j = 0; j < kPre; ++j) {
        const int t = t0 + j * kPlanThreads + threadIdx.x;
        if (t < t1 && pre_stream[j] != ST_SOURCE && pre_stream[j] != ST_REASONING) atomicOr(o.flag, 1);
        const unsigned long long mask = __ballot(pre_stream[j] == ST_SOURCE);
        below[j] = mask;
        if (lane == 0) s_cnt[j * WAVES + wave] = __popcll(mask);
    }
    int tail_sources = 0;                                       // (tokens beyond the registers)
    for (int t = t0 + kPre * kPlanThreads + threadIdx.x; t - int(threadIdx.x) < t1; t += kPlanThreads) {
        const int s = t < t1 ? stream_ids[t] : -1;
        if (t < t1 && s != ST_SOURCE && s != ST_REASONING) atomicOr(o.flag, 1);
        tail_sources += __popcll(__ballot(s == ST_SOURCE));     // (the wave's)
    }
    if (lane == 0) s_tail[0][wave] = tail_sources;
    __syncthreads();
    int scanned = 0, own = 0;
    if (wave < 4) {
        own = scanned = s_cnt[threadIdx.x];
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(scanned, d);
            scanned += lane >= d ? v : 0;
        }
        if (lane == 63) s_sum[wave] = scanned;
    }
    __syncthreads();
    if (wave < 4) {
        for (int w = 0; w < wave; ++w) scanned += s_sum[w];
        s_cnt[threadIdx.x] = scanned - own;                     // sources before (chunk, wave)
    }
    const int pre_sources = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    int S = pre_sources;
    if (n > kPre * kPlanThreads)
        for (int w = 0; w < WAVES; ++w) S += s_tail[0][w];
    const int R = n - S;
    const bool seg_in_lds = S < kSegLds;      // (a dozen dependent loads per row otherwise go to global memory)
    __syncthreads();
    if (threadIdx.x == 0) {
        o.n_src[b] = S;
        o.n_rsn[b] = R;
    }
    auto place = [&](int t, int src_rank, bool is_src, int seg) {
        const int r = is_src ? src_rank : S + ((t - t0) - src_rank);
        o.perm[t0 + r] = t;
        o.seg_c[t0 + r] = seg;
        if (is_src && seg_in_lds) s_seg[r] = seg;
        return r;
    };
    const unsigned long long lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < kPre; ++j) {
        const int t = t0 + j * kPlanThreads + threadIdx.x;
        pre_rank[j] = 0;
        if (t < t1) pre_rank[j] = place(t, s_cnt[j * WAVES + wave] + __popcll(below[j] & lower), pre_stream[j] == ST_SOURCE, pre_seg[j]);
    }
    // (tokens beyond the registers, a chunk and a barrier at a time)
    int total_before = pre_sources;
    for (int base = t0 + kPre * kPlanThreads, j = 1; base < t1; base += kPlanThreads, ++j) {
        const int t = base + threadIdx.x;
        const bool is_src = t < t1 && stream_ids[t] == ST_SOURCE;
        const unsigned long long mask = __ballot(is_src);
        if (lane == 0) s_tail[j & 1][wave] = __popcll(mask);
        __syncthreads();
        int before = total_before, all = 0;
        for (int w = 0; w < WAVES; ++w) {
            const int c = s_tail[j & 1][w];
            before += w < wave ? c : 0;
            all += c;
        }
        if (t < t1) place(t, before + __popcll(mask & lower), is_src, segment_ids[t]);
        total_before += all;
    }
    const int steps = 32 - __clz(S);                            // the answers 0 .. S take this many bits
    if (seg_in_lds)
        for (int i = S + threadIdx.x; i < (1 << steps); i += kPlanThreads) s_seg[i] = INT_MAX;
    __threadfence_block();      // perm / seg_c of this sequence are read back below by other threads
    __syncthreads();

    // visible source count of every row (source row r: r + 1; reasoning row: sources whose segment id is at most its own, by
    // bisection) and the visible pairs.  The bisections of a thread's rows run side by side.
    unsigned long long mine = 0ull;
    auto finish_row = [&](int r, int v) {
        mine += (unsigned long long)v + (r >= S ? (unsigned long long)(r - S + 1) : 0ull);
        o.vis[t0 + r] = v;
    };
    auto bisect_rows = [&](auto count_tag, int j0) {
        constexpr int N = decltype(count_tag)::value;
        int pos[N];
#pragma unroll
        for (int u = 0; u < N; ++u) pos[u] = 0;
        for (int half = 1 << steps >> 1; half > 0; half >>= 1) {
#pragma unroll
            for (int u = 0; u < N; ++u) pos[u] += s_seg[pos[u] + half - 1] <= pre_seg[j0 + u] ? half : 0;
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (t0 + (j0 + u) * kPlanThreads + int(threadIdx.x) < t1)
                finish_row(pre_rank[j0 + u], pre_rank[j0 + u] < S ? pre_rank[j0 + u] + 1 : min(pos[u], S));
    };
    static_assert(kPre % 4 == 0, "rows go four at a time");
    if (seg_in_lds) {
        if (n <= kPlanThreads) {
            bisect_rows(std::integral_constant<int, 1>{}, 0);
        } else {
#pragma unroll
            for (int j = 0; j < kPre; j += 4)
                if (t0 + j * kPlanThreads < t1) bisect_rows(std::integral_constant<int, 4>{}, j);          // (uniform)
        }
    }
    if (!seg_in_lds || n > kPre * kPlanThreads)
        for (int r = threadIdx.x; r < n; r += kPlanThreads)
            if (!seg_in_lds || o.perm[t0 + r] >= t0 + kPre * kPlanThreads) {
                int lo = 0, hi = S;
                const int g = o.seg_c[t0 + r];
                while (r >= S && lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (o.seg_c[t0 + mid] <= g) lo = mid + 1; else hi = mid;
                }
                finish_row(r, r < S ? r + 1 : lo);
            }
    if (validate)
        for (int r = threadIdx.x; r < n; r += kPlanThreads) {
            const int c = t0 + r;
            // neighbours inside one stream: positions strictly increase, segment ids do not decrease
            const bool has_next = (r + 1 < n) && ((r < S) == (r + 1 < S));
            if (has_next) {
                const int p0 = positions[o.perm[c]], p1 = positions[o.perm[c + 1]];
                if (!(p0 < p1) || o.seg_c[c] > o.seg_c[c + 1]) atomicOr(o.flag, 2);
            }
            if (positions[o.perm[c]] < 0 || o.seg_c[c] < 0) atomicOr(o.flag, 4);
        }
    for (int d = 32; d > 0; d >>= 1) mine += __shfl_xor(mine, d);
    if (lane == 0) s_pairs[wave] = mine;
    __threadfence_block();      // vis of this sequence is read back below
    __syncthreads();
    const int slots_before = s_before[0], tiles_before = s_before[1];
    if (threadIdx.x == 0) {
        unsigned long long tot = 0ull;
        for (int w = 0; w < WAVES; ++w) tot += s_pairs[w];
        o.pairs[b] = tot;
    }

    // work items: the 128-row query tiles of the source stream, then those of the reasoning stream; spare slots are empty
    const bool alone = batch == 1 && item_slots(n) <= kAloneMax;
    const int ts = (S + kTileM - 1) / kTileM, tr = (R + kTileM - 1) / kTileM;
    const int ps = (S + kTileN - 1) / kTileN, pr = (R + kTileN - 1) / kTileN;
    for (int local = threadIdx.x; local < item_slots(n); local += kPlanThreads) {
        WorkItem it = {};
        int cost = 0;
        if (local < ts + tr) {
            const bool src = local < ts;
            const int n_stream = src ? S : R;
            it.seq = b;
            it.kind = src ? ST_SOURCE : ST_REASONING;
            it.row0 = (src ? local : local - ts) * kTileM;
            it.n_rows = min(kTileM, n_stream - it.row0);
            const int last = it.row0 + it.n_rows - 1;
            it.a_total = last / kTileN + 1;
            it.a_full = full_tiles(it.row0 + 1, n_stream);
            it.a_base = t0 + (src ? 0 : S);
            it.b_base = t0;
            it.n_stream = n_stream;
            it.n_src = S;
            it.tile_b0 = tiles_before;
            it.tile_a0 = tiles_before + (src ? 0 : ps);
            if (!src) {
                const int vmin = o.vis[it.a_base + it.row0], vmax = o.vis[it.a_base + last];
                it.b_total = (vmax + kTileN - 1) / kTileN;
                it.b_full = full_tiles(vmin, S);
            }
            cost = it.a_total + it.b_total;
            // sort key: the cost, or -- sequence by sequence, longest first inside each -- the sequence in the high bits
            if (seq_major) cost = ((batch - 1 - b) << 20) + min(cost, (1 << 20) - 1);
        }
        o.items[slots_before + local] = it;
        if (alone) s_seg[local] = cost;                         // (the segment ids are done with)
        else o.cost[slots_before + local] = cost;
    }
    // packed key tiles: the source tiles, then the reasoning tiles; spare ones hold no rows
    for (int local = threadIdx.x; local < tile_slots(n); local += kPlanThreads) {
        const bool src = local < ps;
        const int row = (src ? local : local - ps) * kTileN;
        o.tiles[tiles_before + local] = local < ps + pr ? TileInfo{t0 + (src ? 0 : S) + row, min(kTileN, (src ? S : R) - row)} : TileInfo{0, 0};
    }
    if (alone) {
        // the only sequence: its workgroup orders the items itself (as plan_order_kernel does), no second launch
        __threadfence_block();
        __syncthreads();
        const int m = item_slots(n);
        for (int i = threadIdx.x; i < m; i += kPlanThreads) {
            const int ci = s_seg[i];
            int rank = 0;
#pragma unroll 8
            for (int k = 0; k < m; ++k) rank += int(s_seg[k] > ci || (s_seg[k] == ci && k < i));
            o.sorted[rank] = o.items[i];
        }
    }
}

// ---- kernel 2: the items longest first (stable rank by counting; unused slots have key 0 and come last) ----
// A workgroup ranks 64 items, a quarter of the comparisons per wave, four keys per LDS read and several reads in flight (one key
// at a time the walk is a chain of LDS latencies: 14 us for 133 items; 1,032 items in one workgroup of their own took 58 us).
__global__ __launch_bounds__(256) void plan_order_kernel(const int32_t* __restrict__ cost, int m_max,
                                                         const WorkItem* __restrict__ items,
                                                         WorkItem* __restrict__ sorted) {
    constexpr int CHUNK = 2048;
    __shared__ __align__(16) int s_cost[CHUNK];
    __shared__ int s_rank[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    const int ci = i < m_max ? cost[i] : 0;
    int rank = 0;
    for (int base = 0; base < m_max; base += CHUNK) {
        const int n = min(CHUNK, m_max - base), quads = (n + 3) / 4, per_wave = (quads + 3) / 4;
        __syncthreads();
        for (int j = threadIdx.x; j < 4 * quads; j += 256) s_cost[j] = j < n ? cost[base + j] : -1;      // (padding: behind every key)
        __syncthreads();
        const int end = min(quads, per_wave * (wave + 1));
#pragma unroll 8
        for (int k = per_wave * wave; k < end; ++k) {
            const int4 c = *reinterpret_cast<const int4*>(&s_cost[4 * k]);
            const int at = base + 4 * k;
            rank += int(c.x > ci || (c.x == ci && at < i)) + int(c.y > ci || (c.y == ci && at + 1 < i)) +
                    int(c.z > ci || (c.z == ci && at + 2 < i)) + int(c.w > ci || (c.w == ci && at + 3 < i));
        }
    }
    s_rank[wave][lane] = rank;
    __syncthreads();
    if (wave == 0 && i < m_max) sorted[s_rank[0][lane] + s_rank[1][lane] + s_rank[2][lane] + s_rank[3][lane]] = items[i];
}

}  // namespace st

using namespace st;

extern "C" size_t st_plan_workspace_bytes(int32_t batch, int64_t n_tokens) {
    if (batch <= 0 || n_tokens < 0) return 0;
    return ws_layout(batch, n_tokens).total;
}

extern "C" st_status st_plan_create(st_plan** plan_out, const int32_t* segment_ids, const int32_t* stream_ids,
                                    const int32_t* positions, const int32_t* cu_seqlens_host, int32_t batch,
                                    void* workspace, size_t workspace_bytes, int32_t validate, void* hip_stream) {
    if (!plan_out) return fail(ST_ERR_INVALID_ARG, "st_plan_create: plan is null");
    *plan_out = nullptr;
    if (!segment_ids || !stream_ids || !positions || !cu_seqlens_host)
        return fail(ST_ERR_INVALID_ARG, "st_plan_create: null pointer");
    if (batch <= 0) return fail(ST_ERR_INVALID_ARG, "st_plan_create: batch must be positive");
    if (cu_seqlens_host[0] != 0) return fail(ST_ERR_LAYOUT, "st_plan_create: cu_seqlens[0] must be 0");
    for (int b = 0; b < batch; ++b)
        if (cu_seqlens_host[b + 1] < cu_seqlens_host[b])
            return fail(ST_ERR_LAYOUT, "st_plan_create: cu_seqlens must be non-decreasing (entry %d)", b + 1);
    const int64_t n_tokens = cu_seqlens_host[batch];
    const WsLayout L = ws_layout(batch, n_tokens);
    if (workspace) {
        if (reinterpret_cast<uintptr_t>(workspace) & 255u)
            return fail(ST_ERR_INVALID_ARG, "st_plan_create: workspace must be 256-byte aligned");
        if (workspace_bytes < L.total)
            return fail(ST_ERR_CAPACITY, "st_plan_create: workspace has %zu bytes, needs %zu", workspace_bytes, L.total);
    }
    st_plan* p = new (std::nothrow) st_plan();
    if (!p) return fail(ST_ERR_RUNTIME, "st_plan_create: out of host memory");
    p->batch = batch;
    p->n_tokens = n_tokens;
    p->stream = static_cast<hipStream_t>(hip_stream);
    p->cu_host.assign(cu_seqlens_host, cu_seqlens_host + batch + 1);
    p->slot_base_host.resize(batch + 1);
    p->slot_base_host[0] = 0;
    for (int b = 0; b < batch; ++b) {
        const int n = p->cu_host[b + 1] - p->cu_host[b];
        p->slot_base_host[b + 1] = p->slot_base_host[b] + (n + kTileM - 1) / kTileM + 1;
        p->longest = std::max(p->longest, n);
        p->squared_tokens += double(n) * n;
    }
    p->m_max = p->slot_base_host[batch];   // <= m_max_bound(batch, n_tokens)
    // key tiles of the packed K / V^T buffers: ceil(S / 64) + ceil(R / 64) <= ceil(N / 64) + 1 per sequence
    p->pack_tiles = 0;
    for (int b = 0; b < batch; ++b) p->pack_tiles += (p->cu_host[b + 1] - p->cu_host[b] + kTileN - 1) / kTileN + 1;
    if (workspace) {
        p->ws = workspace;
    } else {
        hipError_t e = hipMalloc(&p->ws, L.total);
        if (e != hipSuccess) {
            delete p;
            return fail(ST_ERR_RUNTIME, "st_plan_create: hipMalloc(%zu) failed: %s", L.total, hipGetErrorString(e));
        }
        p->owns_ws = true;
    }
    char* w = static_cast<char*>(p->ws);
    p->cu = reinterpret_cast<int32_t*>(w + L.cu);
    p->n_src = reinterpret_cast<int32_t*>(w + L.n_src);
    p->n_rsn = reinterpret_cast<int32_t*>(w + L.n_rsn);
    p->pairs = reinterpret_cast<unsigned long long*>(w + L.pairs);
    p->flag = reinterpret_cast<int32_t*>(w + L.flag);
    p->perm = reinterpret_cast<int32_t*>(w + L.perm);
    p->seg_c = reinterpret_cast<int32_t*>(w + L.seg_c);
    p->vis = reinterpret_cast<int32_t*>(w + L.vis);
    p->cost = reinterpret_cast<int32_t*>(w + L.cost);
    p->items = reinterpret_cast<WorkItem*>(w + L.items);
    p->sorted = reinterpret_cast<WorkItem*>(w + L.sorted);
    p->tiles = reinterpret_cast<TileInfo*>(w + L.tiles);

    hipStream_t s = p->stream;
    auto bail = [&](hipError_t e, const char* what) {
        st_status r = fail(ST_ERR_RUNTIME, "st_plan_create: %s failed: %s", what, hipGetErrorString(e));
        st_plan_destroy(p);
        return r;
    };
    hipError_t e;
    // (the validation flag is only read back when validation is asked for: cleared then)
    if (validate) hipLaunchKernelGGL(plan_clear_kernel, dim3(1), dim3(64), 0, s, p->flag);
    // Order of the work items.  Small batches: longest first over the whole batch (best balance at the end of the
    // launch).  From 32K tokens on: sequence by sequence, longest first inside a sequence -- the workgroups running at
    // any time then stream the key / value tiles of ONE sequence, which stay in the caches (on 8 x 16K tokens the
    // attention kernel's HBM fetch falls from 18 GB to 3.5 GB per launch and it runs 7 to 9 % faster; four sequences
    // of 4K tokens lose 2 to 6 % to the worse balance, hence the threshold).
    const bool seq_major = n_tokens >= 32768 && batch > 1 && batch < 2048;
    const PlanOut o{p->cu, p->n_src, p->n_rsn, p->perm, p->seg_c, p->vis, p->flag, p->cost, p->pairs, p->items, p->sorted, p->tiles};
    auto sequences = [&](auto cap_tag) {
        constexpr int CAP = decltype(cap_tag)::value;
        HostOffsets<CAP> h;
        if (CAP > 0) std::copy(p->cu_host.begin(), p->cu_host.end(), h.v);
        hipLaunchKernelGGL((plan_sequence_kernel<CAP>), dim3(batch), dim3(kPlanThreads), 0, s, stream_ids, segment_ids, positions, o,
                           validate ? 1 : 0, seq_major ? 1 : 0, batch, h);
    };
    if (batch <= kSmallTable) {
        sequences(std::integral_constant<int, kSmallTable>{});
    } else if (batch <= kLargeTable) {
        sequences(std::integral_constant<int, kLargeTable>{});
    } else {
        // the host vector lives as long as the plan, so the asynchronous copy may read it later
        if ((e = hipMemcpyAsync(p->cu, p->cu_host.data(), sizeof(int32_t) * (batch + 1), hipMemcpyHostToDevice, s)) != hipSuccess)
            return bail(e, "copy of cu_seqlens");
        sequences(std::integral_constant<int, 0>{});
    }
    if (batch > 1 || p->m_max > kAloneMax)
        hipLaunchKernelGGL(plan_order_kernel, dim3((p->m_max + 63) / 64), dim3(256), 0, s, p->cost, p->m_max, p->items, p->sorted);
    if ((e = hipGetLastError()) != hipSuccess) return bail(e, "launch of plan kernels");
    // calls that use the plan on another stream wait for this point
    if ((e = hipEventCreateWithFlags(&p->built, hipEventDisableTiming)) != hipSuccess) return bail(e, "hipEventCreateWithFlags");
    if ((e = hipEventRecord(p->built, s)) != hipSuccess) return bail(e, "hipEventRecord");
    if (validate) {
        int32_t flag = 0;
        if ((e = hipMemcpyAsync(&flag, p->flag, sizeof(flag), hipMemcpyDeviceToHost, s)) != hipSuccess)
            return bail(e, "copy of validation flag");
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return bail(e, "hipStreamSynchronize");
        if (flag) {
            st_plan_destroy(p);
            return fail(ST_ERR_LAYOUT,
                        "st_plan_create: malformed token metadata (%s%s%s)", (flag & 1) ? "stream id outside {0,1}; " : "",
                        (flag & 2) ? "positions not strictly increasing or segment ids decreasing inside a stream; " : "",
                        (flag & 4) ? "negative id" : "");
        }
    }
    *plan_out = p;
    return ST_OK;
}

extern "C" void st_plan_destroy(st_plan* plan) {
    if (!plan) return;
    if (plan->owns_ws && plan->ws) (void)hipFree(plan->ws);
    if (plan->built) (void)hipEventDestroy(plan->built);
    delete plan;
}

extern "C" st_status st_plan_heads_per_workgroup(st_plan* plan, int32_t heads) {
    if (!plan) return fail(ST_ERR_INVALID_ARG, "st_plan_heads_per_workgroup: null plan");
    if (heads < 0 || heads > 2) return fail(ST_ERR_INVALID_ARG, "st_plan_heads_per_workgroup: %d (0 = by problem size, 1 or 2)", heads);
    plan->heads_per_workgroup = heads;
    return ST_OK;
}

extern "C" st_status st_plan_tile_shape(const st_plan* plan, int32_t* tile_m, int32_t* tile_n) {
    if (!plan || !tile_m || !tile_n) return fail(ST_ERR_INVALID_ARG, "st_plan_tile_shape: null pointer");
    *tile_m = kTileM;
    *tile_n = kTileN;
    return ST_OK;
}

static st_status fetch(const st_plan* plan, void* dst, const void* src, size_t bytes) {
    if (bytes == 0) return ST_OK;
    ST_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, plan->stream));
    ST_HIP(hipStreamSynchronize(plan->stream));
    return ST_OK;
}

extern "C" st_status st_plan_stream_counts(const st_plan* plan, int32_t* n_src_host, int32_t* n_rsn_host) {
    if (!plan || !n_src_host || !n_rsn_host) return fail(ST_ERR_INVALID_ARG, "st_plan_stream_counts: null pointer");
    st_status r = fetch(plan, n_src_host, plan->n_src, sizeof(int32_t) * plan->batch);
    if (r != ST_OK) return r;
    return fetch(plan, n_rsn_host, plan->n_rsn, sizeof(int32_t) * plan->batch);
}

extern "C" st_status st_plan_compact_index(const st_plan* plan, int32_t* index_host) {
    if (!plan || !index_host) return fail(ST_ERR_INVALID_ARG, "st_plan_compact_index: null pointer");
    return fetch(plan, index_host, plan->perm, sizeof(int32_t) * plan->n_tokens);
}

extern "C" st_status st_plan_visible_source(const st_plan* plan, int32_t* vis_host) {
    if (!plan || !vis_host) return fail(ST_ERR_INVALID_ARG, "st_plan_visible_source: null pointer");
    return fetch(plan, vis_host, plan->vis, sizeof(int32_t) * plan->n_tokens);
}

extern "C" st_status st_plan_visible_pairs(const st_plan* plan, uint64_t* pairs_host) {
    if (!plan || !pairs_host) return fail(ST_ERR_INVALID_ARG, "st_plan_visible_pairs: null pointer");
    return fetch(plan, pairs_host, plan->pairs, sizeof(uint64_t) * plan->batch);
}

extern "C" st_status st_plan_tile_classes(const st_plan* plan, int32_t seq, int32_t block, uint8_t* classes_host,
                                          int32_t* n_q_tiles, int32_t* n_k_tiles) {
    if (!plan || !n_q_tiles || !n_k_tiles) return fail(ST_ERR_INVALID_ARG, "st_plan_tile_classes: null pointer");
    if (seq < 0 || seq >= plan->batch) return fail(ST_ERR_INVALID_ARG, "st_plan_tile_classes: seq %d out of range", seq);
    if (block != ST_BLOCK_SS && block != ST_BLOCK_RS && block != ST_BLOCK_RR)
        return fail(ST_ERR_INVALID_ARG, "st_plan_tile_classes: block %d", block);
    int32_t S = 0, R = 0;
    st_status r = fetch(plan, &S, plan->n_src + seq, sizeof(int32_t));
    if (r != ST_OK) return r;
    r = fetch(plan, &R, plan->n_rsn + seq, sizeof(int32_t));
    if (r != ST_OK) return r;
    const int ts = (S + kTileM - 1) / kTileM, tr = (R + kTileM - 1) / kTileM;
    const int tq = block == ST_BLOCK_SS ? ts : tr;
    const int tk = ((block == ST_BLOCK_RR ? R : S) + kTileN - 1) / kTileN;
    *n_q_tiles = tq;
    *n_k_tiles = tk;
    if (!classes_host || tq == 0) return ST_OK;
    std::vector<WorkItem> items(tq);
    const int first = plan->slot_base_host[seq] + (block == ST_BLOCK_SS ? 0 : ts);
    r = fetch(plan, items.data(), plan->items + first, sizeof(WorkItem) * tq);
    if (r != ST_OK) return r;
    for (int a = 0; a < tq; ++a) {
        const int full = block == ST_BLOCK_RS ? items[a].b_full : items[a].a_full;
        const int total = block == ST_BLOCK_RS ? items[a].b_total : items[a].a_total;
        for (int c = 0; c < tk; ++c)
            classes_host[size_t(a) * tk + c] = c < full ? ST_TILE_FULL : (c < total ? ST_TILE_PARTIAL : ST_TILE_SKIP);
    }
    return ST_OK;
}
