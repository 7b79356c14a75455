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
    if (ipg == 4) {
        switch (row_blocks) {
        case 3: return launch_rows_one<3, BITS, 4>(a, workers, stream);
        case 5: return launch_rows_one<5, BITS, 4>(a, workers, stream);
        case 6: return launch_rows_one<6, BITS, 4>(a, workers, stream);
        case 7: return launch_rows_one<7, BITS, 4>(a, workers, stream);
        case 8: return launch_rows_one<8, BITS, 4>(a, workers, stream);
        default: return launch_rows_one<4, BITS, 4>(a, workers, stream);
        }
    }
    if (ipg == 2) return row_blocks == 3 ? launch_rows_one<3, BITS, 2>(a, workers, stream) : launch_rows_one<4, BITS, 2>(a, workers, stream);
    return row_blocks == 3 ? launch_rows_one<3, BITS, 1>(a, workers, stream) : launch_rows_one<4, BITS, 1>(a, workers, stream);
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
