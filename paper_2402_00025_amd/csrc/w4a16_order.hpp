// Gather of the activations for weights in activation order on gfx950: A_work[i][t] = A[i][perm[t]], moved as they are.
//
// An element fetched on its own costs a cache line of the unit's memory pipe, 64 of them per instruction: nothing for a
// decode step, whose gather is the latency of two loads, but 1.1 TB/s for a prompt.  There a workgroup reads whole rows
// into LDS, in order, and picks its elements from there.  us, buffers new to the caches (m x k), element by element with a
// 64-bit division each -> now: 16 x 4096: 2.23 -> 2.12, 64 x 4096: 2.74 -> 2.40, 333 x 4096: 5.98 -> 3.75,
// 1024 x 8192: 32.0 -> 9.4, 2048 x 8192: 61.5 -> 15.2 (4.4 TB/s, reads and writes together; a large copy moves 4.75),
// 1500 x 28672: 185 -> 48.  Four rows a workgroup: 14.6 at 2048 x 8192, but 3.8-4.3 at 333 x 4096, and half the widths.
#pragma once
#include "w4a16_device.hpp"

namespace w4a16 {

constexpr int kOrderRows = 2;          // rows that a workgroup stages in LDS
constexpr int kOrderThreads = 512;     // of such a workgroup
constexpr int kOrderCols = 4;          // columns per thread and pass: 8 bytes of a row
constexpr int kOrderMaxK = 160 * 1024 / (2 * kOrderRows);
constexpr int kOrderFewThreads = 128;  // of a workgroup that does not

// Entries of perm outside [0, k) are clamped, so that the kernels stay inside A whatever it holds.
__device__ __forceinline__ int order_source(int src, int k) { return src < 0 ? 0 : (src >= k ? k - 1 : src); }

// Few rows, and what the other kernel does not take: a thread per E columns (k % E == 0; E = 2: perm on 8 bytes).
// Written through (sc1): no dirty line is left for the end of the launch.
template <int E>
__global__ void __launch_bounds__(kOrderFewThreads)
actorder_gather_few_kernel(const _Float16* __restrict__ A, const int32_t* __restrict__ perm, _Float16* __restrict__ A_work, int m, int k)
{
    const unsigned t = (blockIdx.x * kOrderFewThreads + threadIdx.x) * E;
    if (t >= (unsigned)k) return;
    int src[E];
    if constexpr (E == 2) {
        const int2 both = *(const int2*)(perm + t);
        src[0] = order_source(both.x, k);
        src[1] = order_source(both.y, k);
    } else {
        src[0] = order_source(perm[t], k);
    }
    for (int i = blockIdx.y; i < m; i += gridDim.y) {
        const _Float16* row = A + (size_t)i * k;
        const rsrc_t rs = make_rsrc(A_work + (size_t)i * k, (uint32_t)k * 2u);
        if constexpr (E == 2)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, half2_t{row[src[0]], row[src[1]]}), rs, t * 2u, 0, 16);
        else
            __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, row[src[0]]), rs, t * 2u, 0, 16);
    }
}

// Many rows: a workgroup reads two rows into LDS, the two values of a column side by side, and writes its share
// (blockIdx.y of gridDim.y) of their columns, so that one LDS read and one look into perm serve two elements.
// A on 8 bytes, perm and A_work on 16, k a multiple of 4 up to kOrderMaxK.
__global__ void __launch_bounds__(kOrderThreads)
actorder_gather_rows_kernel(const _Float16* __restrict__ A, const int32_t* __restrict__ perm, _Float16* __restrict__ A_work, int m, int k)
{
    typedef _Float16 column_t __attribute__((ext_vector_type(kOrderRows)));
    typedef _Float16 piece_t __attribute__((ext_vector_type(kOrderCols)));
    extern __shared__ __attribute__((aligned(16))) char order_lds[];
    column_t* const cols = (column_t*)order_lds;
    const int r0 = blockIdx.x * kOrderRows, rows = m - r0 < kOrderRows ? m - r0 : kOrderRows;
    const _Float16* const from = A + (size_t)r0 * k;
    _Float16* const to = A_work + (size_t)r0 * k;
#pragma unroll 4
    for (int c = (int)threadIdx.x * kOrderCols; c < k; c += kOrderThreads * kOrderCols) {
        piece_t in[kOrderRows];
#pragma unroll
        for (int r = 0; r < kOrderRows; ++r) in[r] = *(const piece_t*)(from + (size_t)(r < rows ? r : rows - 1) * k + c);
#pragma unroll
        for (int e = 0; e < kOrderCols; ++e) {
            column_t col;
#pragma unroll
            for (int r = 0; r < kOrderRows; ++r) col[r] = in[r][e];
            cols[c + e] = col;
        }
    }
    const int share = ((k / kOrderCols + (int)gridDim.y - 1) / (int)gridDim.y) * kOrderCols;
    const int begin = (int)blockIdx.y * share, end = begin + share < k ? begin + share : k;
    __syncthreads();
#pragma unroll 2
    for (int t = begin + (int)threadIdx.x * kOrderCols; t < end; t += kOrderThreads * kOrderCols) {
        const int4 src = *(const int4*)(perm + t);
        const column_t v[kOrderCols] = {cols[order_source(src.x, k)], cols[order_source(src.y, k)], cols[order_source(src.z, k)],
                                        cols[order_source(src.w, k)]};
#pragma unroll
        for (int r = 0; r < kOrderRows; ++r)
            if (r < rows) *(piece_t*)(to + (size_t)r * k + t) = piece_t{v[0][r], v[1][r], v[2][r], v[3][r]};
    }
}

// k is a multiple of 32.
static inline hipError_t launch_gather(const void* A, const void* perm, void* A_work, int m, int k, hipStream_t stream)
{
    const _Float16* a = (const _Float16*)A;
    const int32_t* p = (const int32_t*)perm;
    // Whole rows pay from 48 rows and 160 K elements on.  us, element by element and whole rows: 160 x 1024: 2.35, 2.11,
    // 48 x 4096: 2.48, 2.32, 48 x 14336: 4.75, 4.21; below, 96 x 1024: 1.76, 2.06, 32 x 14336: 3.77, 4.11 (although 32 x 28672:
    // 6.05, 5.44).  The columns of two rows go to as many workgroups as make 256 of them, up to 8 (64 x 28672: 7.4 with
    // two shares, 5.8 with 8; 333 x 14336: 10.1 with one, 9.0 with two; 2048 x 8192: 15.2 with one, 19.5 with two).
    if (m >= 48 && (size_t)m * (size_t)k >= 160 * 1024 && k <= kOrderMaxK && (uintptr_t)A % 8 == 0 && (uintptr_t)perm % 16 == 0) {
        const size_t lds = (size_t)k * kOrderRows * 2;
        if (lds > 64 * 1024) {
            const hipError_t e = hipFuncSetAttribute((const void*)actorder_gather_rows_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     kOrderMaxK * kOrderRows * 2);
            if (e != hipSuccess) return e;
        }
        const unsigned pairs = ((unsigned)m + kOrderRows - 1) / kOrderRows;
        const unsigned even = (256 + pairs / 2) / pairs, shares = even < 1 ? 1 : even < 8 ? even : 8;
        hipLaunchKernelGGL(actorder_gather_rows_kernel, dim3(pairs, shares), dim3(kOrderThreads), lds, stream, a, p, (_Float16*)A_work, m, k);
        return hipGetLastError();
    }
    const unsigned rows = m < 65535 ? (unsigned)m : 65535u;
    if ((uintptr_t)perm % 8 == 0)
        hipLaunchKernelGGL(actorder_gather_few_kernel<2>, dim3(((unsigned)k / 2 + kOrderFewThreads - 1) / kOrderFewThreads, rows),
                           dim3(kOrderFewThreads), 0, stream, a, p, (_Float16*)A_work, m, k);
    else
        hipLaunchKernelGGL(actorder_gather_few_kernel<1>, dim3(((unsigned)k + kOrderFewThreads - 1) / kOrderFewThreads, rows),
                           dim3(kOrderFewThreads), 0, stream, a, p, (_Float16*)A_work, m, k);
    return hipGetLastError();
}

}  // namespace w4a16
