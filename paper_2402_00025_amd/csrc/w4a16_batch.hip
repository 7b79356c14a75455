// Launches of the kernel for up to 64 rows (see w4a16_batch.hpp).
#include "w4a16_batch.hpp"

namespace w4a16 {

template <int MT, int BITS, int IPG, int STRIPS>
static hipError_t launch_batch_one(const BatchArgs& a, hipStream_t stream)
{
    auto kern = gemm_batch_kernel<MT, BITS, IPG, STRIPS>;
    if constexpr (kBatchLdsBytes<MT> > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kBatchLdsBytes<MT>);
        if (e != hipSuccess) return e;
    }
    const int packed = a.m | a.param_shift << 7 | (int)((unsigned)a.chunks_base << 9);
    const BatchRest rest{a.flags, a.counts, a.errors, a.err_host, a.fixed, a.spin_limit, a.probe_delay};
    hipLaunchKernelGGL(kern, dim3((unsigned)a.split_k, (unsigned)a.tiles), dim3(64 * kBatchWaves), kBatchLdsBytes<MT>, stream, a.A,
                       a.qweight, a.scales, a.qzeros, a.C, packed, a.n, a.k, a.split_k | a.chunks_rem << 16, rest);
    return hipGetLastError();
}

template <int MT, int BITS, int IPG>
static hipError_t launch_batch_strips(const BatchArgs& a, hipStream_t stream)
{
    return a.strips == 2 ? launch_batch_one<MT, BITS, IPG, 2>(a, stream) : launch_batch_one<MT, BITS, IPG, 1>(a, stream);
}

template <int BITS, int IPG>
static hipError_t launch_batch_rows(const BatchArgs& a, hipStream_t stream)
{
    switch ((a.m + 15) / 16) {
    case 1:
        // (groups of 128: the per-wave and the streaming kernel are faster, by 5 to 15 % on average)
        if constexpr (IPG < 4) return launch_batch_strips<1, BITS, IPG>(a, stream);
        return hipErrorInvalidValue;
    case 2: return launch_batch_strips<2, BITS, IPG>(a, stream);
    case 3: return launch_batch_strips<3, BITS, IPG>(a, stream);
    case 4: return launch_batch_strips<4, BITS, IPG>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

template <int BITS>
static hipError_t launch_batch_width(const BatchArgs& a, int ipg, hipStream_t stream)
{
    switch (ipg) {
    case 1: return launch_batch_rows<BITS, 1>(a, stream);
    case 2: return launch_batch_rows<BITS, 2>(a, stream);
    default: return launch_batch_rows<BITS, 4>(a, stream);
    }
}

hipError_t launch_batch(const BatchArgs& a, int bits, int ipg, hipStream_t stream)
{
    switch (bits) {
    case 8: return launch_batch_width<8>(a, ipg, stream);
    case 3: return launch_batch_width<3>(a, ipg, stream);
    case 2: return launch_batch_width<2>(a, ipg, stream);
    default: return launch_batch_width<4>(a, ipg, stream);
    }
}

}  // namespace w4a16
