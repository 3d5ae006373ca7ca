// The decompression kernels (see enec_decompress.hpp): per element format and group length one instance for one stream, one for
// several of one block size and one for several block sizes.
#include "enec_decompress.hpp"

namespace enec {

template <int DT, bool MIXED, bool ONE>
static DecompressFn decompress_for(unsigned L)
{
    if (L == 8) return &decompress_kernel<DT, 1, MIXED, ONE>;
    if (L == 32) return &decompress_kernel<DT, 4, MIXED, ONE>;
    return L == 16 ? &decompress_kernel<DT, 2, MIXED, ONE> : nullptr;
}

template <int DT>
static DecompressFn decompress_of(unsigned L, bool mixed_block_sizes, bool one_stream)
{
    if (mixed_block_sizes) return decompress_for<DT, true, false>(L);
    return one_stream ? decompress_for<DT, false, true>(L) : decompress_for<DT, false, false>(L);
}

DecompressFn pick_decompress(int dtype, unsigned L, bool mixed_block_sizes, bool one_stream)
{
    if (dtype == DT_FP16) return decompress_of<DT_FP16>(L, mixed_block_sizes, one_stream);
    if (dtype == DT_FP32) return decompress_of<DT_FP32>(L, mixed_block_sizes, one_stream);
    return dtype == DT_BF16 ? decompress_of<DT_BF16>(L, mixed_block_sizes, one_stream) : nullptr;
}

}  // namespace enec
