// Batched device-to-device copies: one launch moves many (src, dst, len)
// pieces, where one copy call per piece would queue thousands of small
// launches.  The table of pieces is in device memory, or, for a host table,
// in the kernel arguments (COPY_ARG_PIECES per launch).
//
// What bounds a copy of this kind is latency: requests lie packed, so source and
// destination mostly disagree modulo 16, and a piece may be a megabyte.  The moves
// are therefore 16 bytes wide whatever the source's alignment (the destination is brought
// to 16 bytes; unaligned 16-byte loads are one instruction here), four are in flight
// per thread, and COPY_SPLIT workgroups share a piece, in turns of 16 KiB.  400 requests
// of 22 MB in one launch: 1.8 ms with a workgroup per piece and single bytes where the alignments
// differ, 11 us now (2 TB/s); the serving burst of that size in 44.6 ms, 46.5 before.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace lz {
namespace {

constexpr int COPY_WG = 256;

constexpr int COPY_SPLIT = 8;      // workgroups per piece
constexpr int COPY_UNROLL = 4;     // 16-byte moves in flight per thread
constexpr uint64_t COPY_TURN = (uint64_t)COPY_WG * COPY_UNROLL;  // 16-byte units of one turn

// 16 bytes in device memory, at any address and at a multiple of 16
typedef uint32_t Unit __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) Unit Unit16;
typedef Unit UnitAny __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) UnitAny Unit1;

// Part `part` of COPY_SPLIT of a piece.  Every byte is read and written once, within [src, src + len).
__device__ __forceinline__ void copy_piece(const CopyPiece &p, uint32_t part) {
    const uint8_t *s = p.src;
    uint8_t *d = p.dst;
    const uint64_t len = p.len;
    uint64_t head = (16 - ((uintptr_t)d & 15)) & 15;
    if (head > len) head = len;
    const uint64_t nv = (len - head) / 16;
    const uint64_t tail = head + nv * 16;
    if (part == 0) {  // the ends, fewer than 16 bytes each
        if (threadIdx.x < head) d[threadIdx.x] = s[threadIdx.x];
        if (tail + threadIdx.x < len) d[tail + threadIdx.x] = s[tail + threadIdx.x];
    }
    const Unit1 *sv = (const Unit1 *)(s + head);
    Unit16 *dv = (Unit16 *)(d + head);
    uint64_t t = part * COPY_TURN;
    for (; t + COPY_TURN <= nv; t += COPY_SPLIT * COPY_TURN) {  // no test between the loads: all in flight at once
        Unit v[COPY_UNROLL];
#pragma unroll
        for (int q = 0; q < COPY_UNROLL; ++q) v[q] = sv[t + q * COPY_WG + threadIdx.x];
#pragma unroll
        for (int q = 0; q < COPY_UNROLL; ++q) dv[t + q * COPY_WG + threadIdx.x] = v[q];
    }
    // at most one turn is left, of fewer than COPY_TURN units, and in one part only
    for (uint64_t j = t + threadIdx.x; j < nv && j < t + COPY_TURN; j += COPY_WG) dv[j] = sv[j];
}

__global__ __launch_bounds__(COPY_WG) void copy_many_kernel(const CopyPiece *pieces, uint32_t n) {
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) copy_piece(pieces[i], blockIdx.y);
}

// the pieces in the kernel's arguments: nothing to upload first
struct CopyArgs {
    CopyPiece p[COPY_ARG_PIECES];
    uint32_t n;
};

__global__ __launch_bounds__(COPY_WG) void copy_args_kernel(const CopyArgs a) {
    for (uint32_t i = blockIdx.x; i < a.n; i += gridDim.x) copy_piece(a.p[i], blockIdx.y);
}

}  // namespace

hipError_t launch_copy_many(const CopyPiece *pieces, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const unsigned grid = n < 4096 ? n : 4096;
    hipLaunchKernelGGL(copy_many_kernel, dim3(grid, COPY_SPLIT), dim3(COPY_WG), 0, s, pieces, n);
    return hipGetLastError();
}

hipError_t launch_copy_pieces_host(const CopyPiece *pieces, uint32_t n, hipStream_t s) {
    for (uint32_t i = 0; i < n; i += COPY_ARG_PIECES) {
        CopyArgs a;
        a.n = n - i < COPY_ARG_PIECES ? n - i : COPY_ARG_PIECES;
        for (uint32_t j = 0; j < a.n; ++j) a.p[j] = pieces[i + j];
        hipLaunchKernelGGL(copy_args_kernel, dim3(a.n, COPY_SPLIT), dim3(COPY_WG), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lz
