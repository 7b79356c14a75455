// Launches of the many-row kernel (see w4a16_rows.hpp).
#include "w4a16_rows.hpp"

namespace w4a16 {

template <int MB, bool SPLIT>
static hipError_t launch_rows_one(const RowsArgs& a, hipStream_t stream)
{
    auto kern = gemm_rows_kernel<MB, 4, 4, SPLIT>;
    constexpr int lds_bytes = kRowsLdsBytes<MB, 4>;
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.tiles_m * a.tiles_n * a.split_k)), dim3(64 * kRowsStrips), lds_bytes, stream, a);
    return hipGetLastError();
}

hipError_t launch_rows(const RowsArgs& a, int row_blocks, hipStream_t stream)
{
    if (row_blocks == 8) return a.split_k > 1 ? launch_rows_one<8, true>(a, stream) : launch_rows_one<8, false>(a, stream);
    return a.split_k > 1 ? launch_rows_one<4, true>(a, stream) : launch_rows_one<4, false>(a, stream);
}

}  // namespace w4a16
