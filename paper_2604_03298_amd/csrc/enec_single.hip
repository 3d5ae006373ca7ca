// The compression kernels for tensors of one data block (see enec_single.hpp), one instance per element format, group
// length and size of the arguments.
#include "enec_single.hpp"

namespace enec {

template <class Args, int DT>
static void (*single_for(unsigned L))(const Args)
{
    if (L == 8) return &compress_single_kernel<DT, 1, Args>;
    if (L == 32) return &compress_single_kernel<DT, 4, Args>;
    return L == 16 ? &compress_single_kernel<DT, 2, Args> : nullptr;
}

template <class Args>
static void (*single_of(int dtype, unsigned L))(const Args)
{
    if (dtype == DT_FP16) return single_for<Args, DT_FP16>(L);
    if (dtype == DT_FP32) return single_for<Args, DT_FP32>(L);
    return dtype == DT_BF16 ? single_for<Args, DT_BF16>(L) : nullptr;
}

SingleFn pick_compress_single(int dtype, unsigned L) { return single_of<SingleArgs>(dtype, L); }
SingleFewFn pick_compress_single_few(int dtype, unsigned L) { return single_of<SingleFewArgs>(dtype, L); }

}  // namespace enec
