// The compression kernels for tensors of one data block (see enec_single.hpp), one instance per element format and group
// length.
#include "enec_single.hpp"

namespace enec {

template <int DT>
static SingleFn single_for(unsigned L)
{
    if (L == 8) return &compress_single_kernel<DT, 1>;
    if (L == 32) return &compress_single_kernel<DT, 4>;
    return L == 16 ? &compress_single_kernel<DT, 2> : nullptr;
}

SingleFn pick_compress_single(int dtype, unsigned L)
{
    if (dtype == DT_FP16) return single_for<DT_FP16>(L);
    if (dtype == DT_FP32) return single_for<DT_FP32>(L);
    return dtype == DT_BF16 ? single_for<DT_BF16>(L) : nullptr;
}

}  // namespace enec
