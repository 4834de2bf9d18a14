// 64-row operand tiles and their way into LDS, shared by the forward and the backward attention kernels.
//
// A "row tile" holds 64 rows of a stream (stream-compact order) of one head: [64 rows][D], rows parked in the order the first-type MFMA
// wants, 16-byte chunks XOR-swizzled.  The forward's one-head form (K and V) and the gradients (K, V, Q, dO) gather row tiles straight from the tensors into LDS (RowGather).  Packed
// ones (pack_rows; 16 KB each at D = 128, contiguous, so that a tile is a plain linear copy) are read by the two-head form, by the one-head
// form on long sequences and of rotated keys, and by both directions where a tensor cannot be gathered: too large, written over by a
// result, in the gradients also not aligned to 16 bytes.  Transposed operands come out of a row tile with transposing LDS reads (TrOffsets
// below); the packed V of the forward is a "transposed tile" ([D][64 rows], swizzled).
#pragma once
#include "st_plan.h"

namespace st {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// One wave-wide asynchronous copy global -> LDS: lane l's 16 bytes at `g` land at LDS byte offset
// lds_off + 16 l (lds_off must be wave-uniform).  Completion is counted by vmcnt like any load.
__device__ __forceinline__ void async_copy16(const void* g, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_off) : "memory", "m0");
}
// The same at base + off (one 32-bit offset per lane), `kb` KB further on both sides: the instruction's immediate offset moves the
// global address and the LDS address alike.  (kb, 0 .. 3, is a constant once the caller's loop is unrolled.)
__device__ __forceinline__ void async_copy_1k(const void* base, uint32_t off, uint32_t lds_off, int kb) {
#define ST_COPY_1K(IMM) asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" IMM ::"v"(off), "s"(base), "s"(lds_off) : "memory", "m0")
    if (kb == 0) ST_COPY_1K("");
    else if (kb == 1) ST_COPY_1K(" offset:1024");
    else if (kb == 2) ST_COPY_1K(" offset:2048");
    else ST_COPY_1K(" offset:3072");
#undef ST_COPY_1K
}
// NL wave-wide 16-byte copies global -> LDS, 1 KB apart on both sides: the instruction's immediate offset moves
// the global address and the LDS address alike, so the LDS base goes into m0 once.
template <int NL>
__device__ __forceinline__ void async_copy_rows(const void* base, uint32_t lane_off, uint32_t lds_off) {
    static_assert(NL == 2 || NL == 4, "tile sizes of head_dim 64 and 128");
    if constexpr (NL == 4)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072"
                     ::"v"(lane_off), "s"(base), "s"(lds_off) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024"
                     ::"v"(lane_off), "s"(base), "s"(lds_off) : "memory", "m0");
}

// NL such copies 1 KB apart on both sides, read-once bytes: the instruction's immediate offset moves the global and
// the LDS address alike, so the LDS base goes into m0 once
template <int NL>
__device__ __forceinline__ void async_copy_rows_nt(const void* base, uint32_t lane_off, uint32_t lds_off) {
    static_assert(NL == 2 || NL == 4, "pages of head_dim 64 and 128");
    if constexpr (NL == 4)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024 nt\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048 nt\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072 nt"
                     ::"v"(lane_off), "s"(base), "s"(lds_off) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024 nt"
                     ::"v"(lane_off), "s"(base), "s"(lds_off) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// LDS tiles of the MFMA kernel: no padding; inside every row the 16-byte chunks are stored at
// position chunk ^ key(row).  The LDS has 64 four-byte banks, so a 16-byte operand read serves 16
// lanes (16 consecutive rows) per cycle, and the key must send those 16 rows to 16 different
// 16-byte columns of the 256-byte bank line: for 256-byte rows the key is row % 16 with its two
// 2-bit halves exchanged -- any one-to-one key serves the 16-byte reads, and this one also sends
// four CONSECUTIVE rows to four different 64-byte quarters of the bank line, which is what the
// transposing reads below (four rows x 64 bytes per pass) need; (row / 2) % 8 for 128-byte rows
// (two rows per bank line).  The packed global tiles already have this arrangement, so a tile
// travels global -> LDS as a plain linear copy.
template <int ROW_BYTES>
__device__ __forceinline__ int swizzle_key(int row) {
    return ROW_BYTES == 256 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((row >> 1) & 7);
}

// A transposed operand fragment straight out of a ROW tile ([64 rows][D], rows parked in swap23 order, chunks
// swizzled as above): ds_read_b64_tr_b16 gives lane l of a 16-lane group, as its element j, the (l % 4)-th 16-bit
// value of the 8 bytes that lane 4 j + l / 4 of the group points at.  With lane i of a group pointing at row
// i / 4, columns 4 (i % 4) .. + 3 of a 4-row x 16-column block, every lane receives one COLUMN of the block: two
// such reads (rows 0-3 and 4-7 of an 8-row group) are the eight k-values of an A operand whose M index runs
// along the tile's columns.  TrOffsets holds a lane's element offsets inside a 16-row step for the two reads
// and every 32-column block; the step's first row (a multiple of 16) is added as a constant.
template <int D>
struct TrOffsets {
    int off[2][D / 32];
    __device__ __forceinline__ explicit TrOffsets(int lane) {
        const int l16 = lane & 15, mg = (lane >> 4) & 1, hg = lane >> 5;
        const int j = l16 >> 2, cm = 2 * mg + ((l16 & 3) >> 1);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // logical row 8 hg + 4 t + j of the step sits at position 8 t + 4 hg + j (bits 2 and 3 swapped)
            const int lr = 8 * t + 4 * hg + j;
#pragma unroll
            for (int u = 0; u < D / 32; ++u) off[t][u] = lr * D + ((4 * u + cm) ^ swizzle_key<2 * D>(lr)) * 8 + 4 * (l16 & 1);
        }
    }
    // columns 32 u .. 32 u + 31 (M index = lane % 32), rows 16 step .. + 15 (k index 8 (lane / 32) .. + 7) of `tile`
    __device__ __forceinline__ bf16x8 fragment(const uint16_t* tile, int step, int u) const {
        typedef __bf16 lds_bf16x4 __attribute__((ext_vector_type(4), address_space(3)));
        const uint16_t* p = tile + step * 16 * D;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + off[0][u]));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + off[1][u]));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// swap bits 2 and 3: the row order in which K is parked in LDS, so that after the
// first MFMA each half-wave holds 8 CONSECUTIVE keys per 16-key step
__host__ __device__ __forceinline__ int swap23(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

// A row tile gathered straight out of the caller's tensor: each of the four waves of a workgroup copies 16 of the tile's rows, D / 32
// copies of 1 KB, and a lane names the address of its own 16 bytes -- the row order and the chunk swizzle of the tile come from
// which bytes a lane asks for.  (One head's rows lie a token apart: the L2 serves such rows as fast as packed ones, 30 TB/s over the chip either
// way.)  The tokens of the rows come the same way, 64 bytes per wave and tile, copied into LDS well ahead (copy_tokens) and turned into byte
// offsets of the lane's pieces by offsets(); tensors of one stride share them.
template <int D>
struct RowGather {
    static constexpr int NL = D / 32;                // copies of a wave per tile
    static constexpr int kAreas = 4;                 // tiles whose tokens may be under way or in use
    static constexpr int kBytes = 4 * kAreas * 256;  // LDS of a workgroup's four waves (a copy writes 4 bytes per lane)
    uint32_t stride, lds;                            // row bytes; the wave's token areas (LDS address), both uniform
    const unsigned char* area;                       // ... as a pointer
    // bits 0-7 byte / 16 of the lane's piece of its row (copy 0), 8-15 the row whose token this lane fetches, 16-23 byte of its rows' tokens
    // in an area: one register through the kernel instead of three (taken apart where it is used, see part())
    uint32_t lane_parts;
    __device__ __forceinline__ uint32_t part(int i) const {
        uint32_t x = lane_parts;
        asm volatile("" : "+v"(x));                  // (here, not once and for all)
        return (x >> (8 * i)) & 255u;
    }
    __device__ __forceinline__ RowGather(unsigned char* smem, int wave, int lane, uint32_t row_bytes) {
        // copy i of a wave fills positions R i .. of its 16: lane group g takes position R i + g, which holds row swap23(position)
        constexpr int R = 16 / NL;
        const int g = lane / (D / 8), chunk = lane & (D / 8 - 1), slot = lane & 15;
        stride = row_bytes;
        lane_parts = uint32_t(chunk ^ swizzle_key<2 * D>(g)) | uint32_t(16 * wave + swap23(R * (slot % NL) + slot / NL)) << 8        // (slot NL g + i: copy i's row of group g)
                     | uint32_t(4 * NL * g) << 16;
        lds = uint32_t(uintptr_t(smem)) + uint32_t(wave) * (kAreas * 256);
        area = smem + wave * (kAreas * 256);
    }
    // the tokens of the wave's rows of a tile: rows row0 + .. of the list `perm`, the last one (row `last`) in place of rows past it
    __device__ __forceinline__ void copy_tokens(const int32_t* perm, int row0, int last, int tile) const {
        const uint32_t off = uint32_t(min(row0 + int(part(1)), last)) * 4u;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(perm), "s"(lds + uint32_t(tile % kAreas) * 256u) : "memory", "m0");
    }
    // the tokens of the lane's pieces of a tile, out of LDS
    __device__ __forceinline__ void tokens(uint32_t (&tok)[NL], int tile) const {
        const unsigned char* p = area + (tile % kAreas) * 256 + part(2);
        if constexpr (NL == 4) {
            const u32x4 x = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
            for (int i = 0; i < NL; ++i) tok[i] = x[i];
        } else {
            const u32x2 x = *reinterpret_cast<const u32x2*>(p);
#pragma unroll
            for (int i = 0; i < NL; ++i) tok[i] = x[i];
        }
    }
    // their byte offsets (in place), for copies from base(): the copies' immediate offsets move LDS and global address alike, which is taken
    // back here, with a base (NL - 1) KB below the tensor's
    __device__ __forceinline__ void form(uint32_t (&off)[NL]) const {
        const uint32_t piece = part(0) * 16;
#pragma unroll
        for (int i = 0; i < NL; ++i) off[i] = off[i] * stride + (piece ^ (uint32_t(NL == 4 ? i : 4 * i) * 16)) + 1024u * uint32_t(NL - 1 - i);
    }
    __device__ __forceinline__ void offsets(uint32_t (&off)[NL], int tile) const {
        tokens(off, tile);
        form(off);
    }
    static __device__ __forceinline__ const void* base(const uint16_t* tensor) { return reinterpret_cast<const unsigned char*>(tensor) - (NL - 1) * 1024; }
    // copy i alone, and all of them
    static __device__ __forceinline__ void copy_one(const void* base, const uint32_t (&off)[NL], uint32_t lds_off, int i) { async_copy_1k(base, off[i], lds_off, i); }
    static __device__ __forceinline__ void copy(const void* base, const uint32_t (&off)[NL], uint32_t lds_off) {
        if constexpr (NL == 4)
            asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %4\n\tglobal_load_lds_dwordx4 %1, %4 offset:1024\n\t"
                         "global_load_lds_dwordx4 %2, %4 offset:2048\n\tglobal_load_lds_dwordx4 %3, %4 offset:3072"
                         ::"v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "s"(lds_off) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                         ::"v"(off[0]), "v"(off[1]), "s"(base), "s"(lds_off) : "memory", "m0");
    }
};

// A gathered row's byte offset and the 3 KB that take the immediate offsets back have to fit 32 bits together: true of every tensor but one
// within 4 KB of 4 GiB, which is packed instead.
inline bool gather_fits(int64_t n_tokens, int n_heads, int head_dim) { return n_tokens * n_heads * head_dim * 2 <= int64_t(0xffffffff) - 4096; }

// parts of kTileM / head_waves rows of an item that a launch has workgroups for
__host__ __device__ inline int item_parts(const PlanView& pv, int head_waves) { return (pv.parts32 * head_waves + 3) / 4; }
// Rows [sub * part_rows, + part_rows) of a work item as an item of their own, with the extents as the plan builds them
// (n_rows <= 0: no such rows).
__device__ __forceinline__ WorkItem item_part(WorkItem it, const PlanView& pv, int sub, int part_rows) {
    it.row0 += sub * part_rows;
    it.n_rows = min(part_rows, it.n_rows - sub * part_rows);
    if (it.n_rows <= 0) return it;
    const int last = it.row0 + it.n_rows - 1;
    it.a_total = last / kTileN + 1;
    it.a_full = it.n_stream <= it.row0 + 1 ? (it.n_stream + kTileN - 1) / kTileN : (it.row0 + 1) / kTileN;
    if (it.kind != ST_SOURCE) {
        const int vmin = pv.vis[it.a_base + it.row0], vmax = pv.vis[it.a_base + last];
        it.b_total = (vmax + kTileN - 1) / kTileN;
        it.b_full = it.n_src <= vmin ? (it.n_src + kTileN - 1) / kTileN : vmin / kTileN;
    }
    return it;
}

// The rows of one tile and head, gathered by a workgroup of 256 threads into a row tile: parked in the row order the first MFMA
// wants (bits 2 and 3 of the row swapped), with the chunk swizzle of the LDS tile; rows past the end of the stream are zero
// (they are masked, but must be finite).  each(row, element offset of the piece, piece) sees every 16-byte piece on the way:
// D / 8 neighbouring lanes hold a row.
template <int D, typename Each>
__device__ __forceinline__ void pack_rows(uint16_t* dst, const uint16_t* src, const int32_t* perm, int valid, uint32_t row_stride,
                                          uint32_t head, Each each) {
    constexpr int CH = D / 8;
#pragma unroll
    for (int u = 0; u < kTileN * CH / 256; ++u) {
        const int c = int(threadIdx.x) + 256 * u;
        const int row = c / CH, ch = c % CH;
        u32x4 val = {0u, 0u, 0u, 0u};
        uint32_t at = 0;
        if (row < valid) {
            at = uint32_t(perm[row]) * row_stride + head * D + ch * 8;
            val = *reinterpret_cast<const u32x4_a2*>(src + at);
        }
        each(row, at, val);
        const int lr = swap23(row);                                    // row position in the tile
        *reinterpret_cast<u32x4*>(dst + lr * D + (ch ^ swizzle_key<2 * D>(lr)) * 8) = val;
    }
}

}  // namespace st
