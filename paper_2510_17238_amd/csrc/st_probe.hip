// Machine probes for the benchmark: what this GPU sustains for the access pattern of the decode kernel and for
// the instruction the prefill kernel lives on, so that a roofline fraction can be read against a measured ceiling
// and not only against the data-sheet peak.  They compute nothing of the method.
//   probe_paged_read_kernel  one wave per workgroup; per step a wave reads two 4 KB "key
//                            pages" and two 4 KB "value pages" at pseudo-random page indices with the decode
//                            kernel's per-lane addressing (16 loads of 16 bytes per lane), and folds them with XOR.
//   probe_mfma_kernel        4 waves per workgroup; every wave issues independent v_mfma_f32_32x32x16_bf16 on
//                            register operands with random mantissas, nothing else in the loop.
#include "st_internal.h"
#include "st_probe.h"

namespace st {

__global__ __launch_bounds__(64, 4) void probe_paged_read_kernel(const unsigned char* __restrict__ pool, uint32_t page_mask,
                                                                int steps, uint32_t salt, uint32_t* __restrict__ sink) {
    const int lane = threadIdx.x;
    const int n = lane & 15, g4 = lane >> 4;
    const uint64_t wave = blockIdx.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int s = 0; s < steps; ++s) {
        // four distinct pseudo-random pages per step; a "page" is 4 KB: 16 tokens x 128 dims x 2 bytes of one head
        const uint64_t base = (wave * steps + s) * 4;
        size_t pg[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pg[u] = size_t(uint32_t((base + u) * 2654435761ull + 12345u + salt) & page_mask) * 4096;
        const unsigned char* kp = pool + pg[n >> 3] + g4 * 256 + (8 * ((n >> 2) & 1) + (n & 3)) * 16;
        const unsigned char* vp = pool + pg[2 + (g4 >> 1)] + n * 32 + 16 * (g4 & 1);
        u32x4 t[16];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            t[2 * j] = *reinterpret_cast<const u32x4*>(kp + j * 1024);
            t[2 * j + 1] = *reinterpret_cast<const u32x4*>(kp + j * 1024 + 64);
        }
#pragma unroll
        for (int db = 0; db < 8; ++db) t[8 + db] = *reinterpret_cast<const u32x4*>(vp + db * 512);
#pragma unroll
        for (int u = 0; u < 16; ++u) acc ^= t[u];
    }
    const uint32_t r = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
    if (r == 0x9e3779b9u) sink[0] = r;           // keeps the loads alive; practically never taken
}

__device__ __forceinline__ uint32_t probe_hash(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352dU; x ^= x >> 15; x *= 0x846ca68bU; x ^= x >> 16;
    return x;
}
// two bf16 values of magnitude in [0.5, 2) with random sign and mantissa
__device__ __forceinline__ uint32_t probe_bf16_pair(uint32_t h) {
    const uint32_t lo = (h & 0x80FFu) | 0x3F00u | ((h >> 4) & 0x0080u);
    const uint32_t hi = ((h >> 16) & 0x80FFu) | 0x3F00u | ((h >> 20) & 0x0080u);
    return lo | (hi << 16);
}

__global__ __launch_bounds__(256) void probe_mfma_kernel(float* __restrict__ sink, int iterations) {
    bf16x8 a[8], b[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        u32x4 x, y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t h1 = probe_hash(threadIdx.x * 131u + s * 17u + i + blockIdx.x * 7919u), h2 = probe_hash(h1 + 12345u);
            x[i] = probe_bf16_pair(h1);
            y[i] = probe_bf16_pair(h2);
        }
        a[s] = __builtin_bit_cast(bf16x8, x);
        b[s] = __builtin_bit_cast(bf16x8, y);
    }
    f32x16 c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 16; ++i) c[u][i] = 0.f;
    for (int it = 0; it < iterations; ++it) {
#pragma unroll
        for (int s = 0; s < 8; ++s) c[s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], b[s], c[s & 3], 0, 0, 0);
        if ((it & 1023) == 1023) {               // keep the accumulators finite
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 16; ++i) c[u][i] *= 1e-3f;
        }
    }
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 16; ++i) s += c[u][i];
    if (s == 12345.678f) sink[0] = s;
}

}  // namespace st

using namespace st;

extern "C" int32_t st_probe_paged_read(const void* pool, size_t pool_bytes, int32_t n_waves, int32_t steps_per_wave, uint32_t salt,
                                       uint32_t* sink, void* hip_stream) {
    if (!pool || !sink) return fail(ST_ERR_INVALID_ARG, "st_probe_paged_read: null pointer");
    if (!aligned16(pool)) return fail(ST_ERR_INVALID_ARG, "st_probe_paged_read: pool must be 16-byte aligned");
    if (pool_bytes < 4096 || (pool_bytes & (pool_bytes - 1)) != 0 || pool_bytes > (size_t(1) << 43))
        return fail(ST_ERR_INVALID_ARG, "st_probe_paged_read: pool_bytes must be a power of two in [4 KiB, 8 TiB]");
    if (n_waves <= 0 || steps_per_wave <= 0) return fail(ST_ERR_INVALID_ARG, "st_probe_paged_read: bad sizes");
    hipLaunchKernelGGL(probe_paged_read_kernel, dim3((unsigned)n_waves), dim3(64), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const unsigned char*>(pool), uint32_t(pool_bytes / 4096 - 1), steps_per_wave, salt * 0x9E3779B1u, sink);
    ST_LAUNCH_CHECK("probe_paged_read_kernel");
    return ST_OK;
}

extern "C" int32_t st_probe_mfma_bf16(int32_t n_workgroups, int32_t iterations, float* sink, void* hip_stream) {
    if (!sink) return fail(ST_ERR_INVALID_ARG, "st_probe_mfma_bf16: null pointer");
    if (n_workgroups <= 0 || iterations <= 0) return fail(ST_ERR_INVALID_ARG, "st_probe_mfma_bf16: bad sizes");
    hipLaunchKernelGGL(probe_mfma_kernel, dim3((unsigned)n_workgroups), dim3(256), 0, static_cast<hipStream_t>(hip_stream), sink,
                       iterations);
    ST_LAUNCH_CHECK("probe_mfma_kernel");
    return ST_OK;
}
