// Device-resident segment tables of one packed batch (internal view of st_plan).
#pragma once
#include <algorithm>
#include <vector>

#include "st_internal.h"

namespace st {

// One query tile of one stream of one sequence, in stream-compact coordinates.
// Block A is the causal block over the row's own stream (SS for source rows, RR
// for reasoning rows); block B is the rectangular source prefix of reasoning rows
// (RS) and is empty for source rows.  Key tiles [0, full) of a block need no mask,
// [full, total) are compared element-wise, the rest is never visited.
struct WorkItem {
    int32_t seq;
    int32_t kind;     // ST_SOURCE / ST_REASONING
    int32_t row0;     // first row, relative to the start of the row's stream
    int32_t n_rows;   // 0 marks an unused slot
    int32_t a_full, a_total;
    int32_t b_full, b_total;
    // everything else a kernel needs about the item's sequence, so that one 64-byte load suffices
    int32_t a_base;   // compact row of column 0 of block A (start of the row's own stream)
    int32_t b_base;   // compact row of column 0 of block B (start of the source stream)
    int32_t n_stream; // tokens of the row's own stream
    int32_t n_src;    // source tokens of the sequence
    int32_t tile_a0;  // packed key tile of column 0 of block A
    int32_t tile_b0;  // packed key tile of column 0 of block B
    int32_t pad0, pad1;
};
static_assert(sizeof(WorkItem) == 64, "WorkItem is one 64-byte record");

// A packed key tile: compact row of its first row, rows (0: a spare tile, never read).
struct TileInfo {
    int32_t base, valid;
};

struct PlanView {  // what kernels need
    const int32_t* cu;       // [B+1] token offsets
    const int32_t* n_src;    // [B]
    const int32_t* perm;     // [N] compact row -> token index
    const int32_t* vis;      // [N] visible source count per compact row
    const WorkItem* sorted;  // [m_max] work items, longest first (unused slots last)
    int32_t m_max;
    // Packed K / V^T buffers (bf16 path): key tiles of kTileN rows each -- per sequence first ceil(S / kTileN) source tiles,
    // then the reasoning tiles, then spare ones.
    const TileInfo* tiles;     // [pack_tiles]
    int32_t pack_tiles;
    // 32-row parts of a work item that some sequence has rows for: 4, fewer where no sequence has more than 96 tokens.  A kernel whose
    // workgroups take a part each launches no more of them -- one that finds no row still waits for its item in a place on the
    // chip: 300 sequences of 33 tokens, 32 / 8 heads of 64 dims in bf16 128 us with four parts, 75 with two; 64 sequences of one
    // token, 16 / 8 heads of 128 in fp32 39 with four, 18 with one.
    int32_t parts32;
};

// fp32 attention (st_attn_f32.hip); the callers have checked the arguments and ordered `s` behind the plan
st_status launch_prefill_f32(float* out, float* lse, const float* q, const float* k, const float* v, const PlanView& pv, int n_q_heads,
                             int n_kv_heads, int head_dim, float scale, hipStream_t s);
st_status launch_bwd_f32(float* dq, float* dk, float* dv, float* delta, const float* d_out, const float* q, const float* k, const float* v,
                         const float* out, const float* lse, const PlanView& pv, int n_q_heads, int n_kv_heads, int head_dim, float scale,
                         int64_t n_tokens, int parts, float* partial, hipStream_t s);

}  // namespace st

struct st_plan {
    int32_t batch = 0;
    int64_t n_tokens = 0;
    int32_t m_max = 0;
    int32_t heads_per_workgroup = 0;   // bf16 attention kernel: 0 = chosen by problem size, 1, 2 (st_plan_heads_per_workgroup)
    std::vector<int32_t> cu_host, slot_base_host;
    int32_t longest = 0;               // tokens of the longest sequence
    double squared_tokens = 0;         // sum over the sequences of tokens^2
    int32_t pack_tiles = 0;
    void* ws = nullptr;
    bool owns_ws = false;
    hipStream_t stream = nullptr;
    hipEvent_t built = nullptr;        // recorded on `stream` behind the kernels that build the tables
    int32_t *cu = nullptr, *n_src = nullptr, *n_rsn = nullptr;
    int32_t *perm = nullptr, *seg_c = nullptr, *vis = nullptr, *cost = nullptr, *flag = nullptr;
    unsigned long long* pairs = nullptr;
    st::WorkItem* items = nullptr;    // slot order (sequence by sequence)
    st::WorkItem* sorted = nullptr;   // longest first
    st::TileInfo* tiles = nullptr;    // packed key tiles

    // Orders `s` behind the build of the tables (nothing to do on the stream that built them).
    hipError_t wait_built(hipStream_t s) const { return (s == stream || !built) ? hipSuccess : hipStreamWaitEvent(s, built, 0); }

    st::PlanView view() const { return st::PlanView{cu, n_src, perm, vis, sorted, m_max, tiles, pack_tiles, std::max((std::min(longest, st::kTileM) + 31) / 32, 1)}; }
};
