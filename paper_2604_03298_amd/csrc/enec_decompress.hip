// The decompression kernels (see enec_decompress.hpp): per element format and group length one instance for one block
// size and one for several.
#include "enec_decompress.hpp"

namespace enec {

template <int DT, bool MIXED>
static DecompressFn decompress_for(unsigned L)
{
    if (L == 8) return &decompress_kernel<DT, 1, MIXED>;
    if (L == 32) return &decompress_kernel<DT, 4, MIXED>;
    return L == 16 ? &decompress_kernel<DT, 2, MIXED> : nullptr;
}

DecompressFn pick_decompress(int dtype, unsigned L, bool mixed_block_sizes)
{
    if (dtype == DT_FP16) return mixed_block_sizes ? decompress_for<DT_FP16, true>(L) : decompress_for<DT_FP16, false>(L);
    if (dtype == DT_FP32) return mixed_block_sizes ? decompress_for<DT_FP32, true>(L) : decompress_for<DT_FP32, false>(L);
    if (dtype != DT_BF16) return nullptr;
    return mixed_block_sizes ? decompress_for<DT_BF16, true>(L) : decompress_for<DT_BF16, false>(L);
}

}  // namespace enec
