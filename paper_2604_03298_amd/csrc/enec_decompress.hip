// The decompression kernels (see enec_decompress.hpp), one instance per element format and group length.
#include "enec_decompress.hpp"

namespace enec {

template <int DT>
static DecompressFn decompress_for(unsigned L)
{
    if (L == 8) return &decompress_kernel<DT, 1>;
    if (L == 32) return &decompress_kernel<DT, 4>;
    return L == 16 ? &decompress_kernel<DT, 2> : nullptr;
}

DecompressFn pick_decompress(int dtype, unsigned L)
{
    if (dtype == DT_FP16) return decompress_for<DT_FP16>(L);
    if (dtype == DT_FP32) return decompress_for<DT_FP32>(L);
    return dtype == DT_BF16 ? decompress_for<DT_BF16>(L) : nullptr;
}

}  // namespace enec
