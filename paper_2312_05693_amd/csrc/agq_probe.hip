// Measurement aid for bench.py and the tests' view of the library's dispatch rules, built as its own small library
// (libagq_probe.so): not part of the product and not linked into libagq.so.  Two kernels that bound what one launch of a weight-streaming kernel can reach on
// the device at hand: a plain read of a buffer with the access pattern of the decode kernels (one coalesced
// 16-byte load per lane and KiB, every load of a workgroup requested before the first is used), and an empty
// kernel (the cost of a launch inside a replayed graph).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <chrono>

#include "agq_internal.h"

namespace {

typedef unsigned int probe_u4 __attribute__((ext_vector_type(4)));
constexpr int kLoads = 4;        // 16-byte loads in flight per lane
constexpr int kThreads = 512;    // 32 KiB per workgroup: the weights of one 16-channel tile at K = 4096

__global__ __launch_bounds__(kThreads) void probe_read_kernel(const probe_u4 *src, size_t n16, uint32_t *sink) {
    const size_t base = (size_t)blockIdx.x * (kThreads * kLoads) + threadIdx.x;
    probe_u4 v[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const size_t at = base + (size_t)i * kThreads;
        v[i] = src[at < n16 ? at : n16 - 1];
    }
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) acc ^= v[i][0] ^ v[i][1] ^ v[i][2] ^ v[i][3];
    // every lane's loads are needed by a store the compiler cannot rule out (it happens for one bit pattern)
    if (acc == 0x9e3779b9u) sink[threadIdx.x & 63] = acc;
}

__global__ void probe_empty_kernel() {}

// An int8 matrix instruction with no memory traffic at all: every lane loads four pairs of operand registers once (4 x 16 bytes
// each from `a` and `b`, the same 16 KiB for every workgroup) and then issues MFMAs, every one with another pair than the one
// before it, as in a GEMM: 16 x 16 x 64 (the tiled kernel's), eight independent ones a round, or 32 x 32 x 32 (WIDE), four of twice
// the operations.  What this measures is the rate the matrix cores sustain for given operand VALUES (the instruction
// stream is the same for all of them).
typedef int probe_v4i __attribute__((ext_vector_type(4)));

template <bool WIDE>
__global__ __launch_bounds__(256) void probe_mfma_kernel(const probe_v4i *a, const probe_v4i *b, int reps, uint32_t *sink) {
    constexpr int kAcc = WIDE ? 4 : 8, kRegs = WIDE ? 16 : 4;
    typedef int acc_t __attribute__((ext_vector_type(kRegs)));
    probe_v4i av[4], bv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        av[j] = a[j * 256 + threadIdx.x];
        bv[j] = b[j * 256 + threadIdx.x];
    }
    acc_t acc[kAcc];
#pragma unroll
    for (int j = 0; j < kAcc; ++j)
#pragma unroll
        for (int r = 0; r < kRegs; ++r) acc[j][r] = 0;
    for (int it = 0; it < reps; it += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < kAcc; ++j) {
                const probe_v4i x = av[j & 3], y = bv[(j + u + (j >> 2)) & 3];
                // (as assembly: around the builtins the compiler copied the accumulators once a turn, a fifth of the rate of the small form)
                if constexpr (WIDE) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc[j]) : "v"(x), "v"(y));
                else asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(acc[j]) : "v"(x), "v"(y));
            }
    }
#pragma unroll
    for (int j = 0; j < kAcc; ++j) asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[j]));    // the last results, before they are read
    uint32_t x = 0;
#pragma unroll
    for (int j = 0; j < kAcc; ++j)
#pragma unroll
        for (int r = 0; r < kRegs; ++r) x ^= (uint32_t)acc[j][r];
    if (x == 0x9e3779b9u) sink[threadIdx.x & 63] = x;   // never, but the compiler cannot rule it out
}

}  // namespace

// src: device buffer of `bytes` bytes (a multiple of 16, at least 16), 16-byte aligned; sink: device, 256 bytes.
extern "C" int agq_probe_read(const void *src, size_t bytes, void *sink, void *stream) {
    if (!src || !sink || bytes < 16 || (bytes % 16) != 0) return -1;
    const size_t n16 = bytes / 16;
    const size_t per_wg = (size_t)kThreads * kLoads;
    probe_read_kernel<<<(unsigned)((n16 + per_wg - 1) / per_wg), kThreads, 0, (hipStream_t)stream>>>(
        (const probe_u4 *)src, n16, (uint32_t *)sink);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

extern "C" int agq_probe_empty(void *stream) {
    probe_empty_kernel<<<1, 64, 0, (hipStream_t)stream>>>();
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

// `a`, `b`: 16 KiB each (4 x 256 lanes x 16 bytes of int8 operand values, device memory); `workgroups` of 256
// threads (four wavefronts, one per SIMD of a CU); `reps` (a multiple of four) rounds of 8 x 32^3 operations per wavefront;
// wide: 32 x 32 x 32 instead of 16 x 16 x 64 MFMAs.
extern "C" int agq_probe_mfma_i8(const void *a, const void *b, int workgroups, int reps, int wide, void *sink, void *stream) {
    if (!a || !b || !sink || workgroups < 1 || reps < 4 || (reps & 3)) return -1;
    const auto kernel = wide ? probe_mfma_kernel<true> : probe_mfma_kernel<false>;
    kernel<<<(unsigned)workgroups, 256, 0, (hipStream_t)stream>>>((const probe_v4i *)a, (const probe_v4i *)b, reps, (uint32_t *)sink);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Host only: the kernel that a linear layer of x [M,K] and blobs [N[p], K] takes with a workspace of that size: an
// AgqTiledVariant (agq_internal.h), or -1 for the weight-streaming kernel.  n_extra: -1 for plain blobs.
extern "C" int agq_probe_gemm_route(int x_kind, int64_t M, int64_t K, const int64_t *N, int count, int n_extra, size_t workspace_bytes) {
    const AgqRoute r = agq_gemm_route(x_kind, M, K, N, count, n_extra, workspace_bytes);
    return r.tiles ? (int)r.choice.variant : -1;
}

// Host only: the workgroup tile of that call, 100 nt + 10 jt + kg of AgqTiledChoice, plus 1000 times the slices of a K split;
// -1 for the weight-streaming kernel.
extern "C" int agq_probe_gemm_tile(int x_kind, int64_t M, int64_t K, const int64_t *N, int count, int n_extra, size_t workspace_bytes) {
    const AgqRoute r = agq_gemm_route(x_kind, M, K, N, count, n_extra, workspace_bytes);
    if (!r.tiles) return -1;
    return (r.choice.variant == TILED_SPLIT ? 1000 * r.choice.splits : 0) + 100 * r.choice.nt + 10 * r.choice.jt + r.choice.kg;
}

// Host only: token tiles that the walk over tiles of 16 nt tokens, kg groups, takes together, for M tokens and n_sum channels in all.
extern "C" int agq_probe_tiled_band(int64_t M, int64_t n_sum, int nt, int kg) { return agq_tiled_band(M, n_sum, nt, kg); }

// Host only: nanoseconds that the host takes for that choice, fp16 input on plain blobs, on average over `reps` of them.
extern "C" double agq_probe_gemm_route_ns(int64_t M, int64_t K, const int64_t *N, int count, size_t workspace_bytes, int reps) {
    const auto t0 = std::chrono::steady_clock::now();
    volatile int64_t rows = M, taken = 0;                // (read and written every time, so that no choice is left out)
    for (int i = 0; i < reps; ++i) taken = taken + agq_gemm_route(0, rows, K, N, count, -1, workspace_bytes).tiles;
    return std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now() - t0).count() / reps;
}

// Host only: whether 5 to 16 rows of fp16 input on plain blobs [N[p], K] run with two channel tiles per workgroup of the
// per-tile kernel (1 / 0).
extern "C" int agq_probe_decode_pairs(int64_t M, int64_t K, const int64_t *N, int count) {
    int64_t tiles = 0, tile_pairs = 0;
    for (int p = 0; p < count; ++p) {
        tiles += (N[p] + 15) / 16;
        tile_pairs += (N[p] + 31) / 32;
    }
    return agq_decode_pairs(0, false, M, agq_k_tiles(K), tiles, tile_pairs);
}
