// The compression kernels for one tuple per data block (see enec_per_block.hpp), one instance per element
// format and group length.  Compiled twice, because the kernel with deferred stores wants different choices of the compiler:
// with -DENEC_FP32=1 its fp32 instances, with -DENEC_FP32=0 everything else.
#include "enec_per_block.hpp"

#ifndef ENEC_FP32
#error "compile with -DENEC_FP32=0|1"
#endif

namespace enec {

#if !ENEC_FP32
template <int DT>
static PbCompressFn compress_for(unsigned L)
{
    if (L == 8) return &compress_per_block_kernel<DT, 1>;
    if (L == 32) return &compress_per_block_kernel<DT, 4>;
    return L == 16 ? &compress_per_block_kernel<DT, 2> : nullptr;
}

#endif

template <int DT>
static CompressFn stream_for(unsigned L)
{
    if (L == 8) return &compress_per_block_stream_kernel<DT, 1>;
    if (L == 32) return &compress_per_block_stream_kernel<DT, 4>;
    return L == 16 ? &compress_per_block_stream_kernel<DT, 2> : nullptr;
}

#if ENEC_FP32
CompressFn pick_compress_per_block_stream_fp32(unsigned L) { return stream_for<DT_FP32>(L); }
#else
PbCompressFn pick_compress_per_block(int dtype, unsigned L)
{
    if (dtype == DT_FP16) return compress_for<DT_FP16>(L);
    if (dtype == DT_FP32) return compress_for<DT_FP32>(L);
    return dtype == DT_BF16 ? compress_for<DT_BF16>(L) : nullptr;
}

CompressFn pick_compress_per_block_stream(int dtype, unsigned L)
{
    if (dtype == DT_FP16) return stream_for<DT_FP16>(L);
    if (dtype == DT_FP32) return pick_compress_per_block_stream_fp32(L);
    return dtype == DT_BF16 ? stream_for<DT_BF16>(L) : nullptr;
}
#endif

}  // namespace enec
