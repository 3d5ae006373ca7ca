// The decompression kernels (see enec_decompress.hpp), per element format and group length.  Compiled twice: with -DENEC_ONE=1 the
// instances for one stream, with -DENEC_ONE=0 those for several, of one block size and of several block sizes.  (A process's first
// decompression loads all instances of a unit: 1.55 ms for all 27, 1.13 for the 18 for several streams, 0.64 for the nine for one.)
#include "enec_decompress.hpp"

#ifndef ENEC_ONE
#error "compile with -DENEC_ONE=0|1"
#endif

namespace enec {

template <int DT, bool MIXED>
static DecompressFn decompress_for(unsigned L)
{
    if (L == 8) return &decompress_kernel<DT, 1, MIXED, ENEC_ONE>;
    if (L == 32) return &decompress_kernel<DT, 4, MIXED, ENEC_ONE>;
    return L == 16 ? &decompress_kernel<DT, 2, MIXED, ENEC_ONE> : nullptr;
}

#if ENEC_ONE
DecompressFn pick_decompress_one(int dtype, unsigned L)
{
    if (dtype == DT_FP16) return decompress_for<DT_FP16, false>(L);
    if (dtype == DT_FP32) return decompress_for<DT_FP32, false>(L);
    return dtype == DT_BF16 ? decompress_for<DT_BF16, false>(L) : nullptr;
}
#else
DecompressFn pick_decompress(int dtype, unsigned L, bool mixed_block_sizes)
{
    if (dtype == DT_FP16) return mixed_block_sizes ? decompress_for<DT_FP16, true>(L) : decompress_for<DT_FP16, false>(L);
    if (dtype == DT_FP32) return mixed_block_sizes ? decompress_for<DT_FP32, true>(L) : decompress_for<DT_FP32, false>(L);
    if (dtype != DT_BF16) return nullptr;
    return mixed_block_sizes ? decompress_for<DT_BF16, true>(L) : decompress_for<DT_BF16, false>(L);
}
#endif

}  // namespace enec
