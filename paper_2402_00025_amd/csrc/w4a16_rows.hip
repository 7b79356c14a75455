// Launches of the many-row kernel (see w4a16_rows.hpp).
#include "w4a16_rows.hpp"

namespace w4a16 {

template <int MB, int BITS, int IPG>
static hipError_t launch_rows_one(const RowsArgs& a, int workers, hipStream_t stream)
{
    auto kern = gemm_rows_kernel<MB, BITS, IPG>;
    constexpr int lds_bytes = kRowsLdsBytes<MB, BITS>;
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)workers), dim3(64 * kRowsStrips), lds_bytes, stream, a);
    return hipGetLastError();
}

template <int BITS>
static hipError_t launch_rows_width(const RowsArgs& a, int ipg, int row_blocks, int workers, hipStream_t stream)
{
    if (row_blocks == 8 && rows_tall_ok(ipg)) return launch_rows_one<8, BITS, 4>(a, workers, stream);
    switch (ipg) {
    case 1: return launch_rows_one<4, BITS, 1>(a, workers, stream);
    case 2: return launch_rows_one<4, BITS, 2>(a, workers, stream);
    default: return launch_rows_one<4, BITS, 4>(a, workers, stream);
    }
}

hipError_t launch_rows(const RowsArgs& a, int bits, int ipg, int row_blocks, int workers, hipStream_t stream)
{
    switch (bits) {
    case 8: return launch_rows_width<8>(a, ipg, row_blocks, workers, stream);
    case 3: return launch_rows_width<3>(a, ipg, row_blocks, workers, stream);
    case 2: return launch_rows_width<2>(a, ipg, row_blocks, workers, stream);
    default: return launch_rows_width<4>(a, ipg, row_blocks, workers, stream);
    }
}

}  // namespace w4a16
