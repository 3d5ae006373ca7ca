// Compression of tensors of one data block each (norm vectors, biases) with a given tuple, in a launch of their own: a workgroup
// takes one tensor (compress_one_block of enec_device.hpp, which compress_kernel's launches run too where they take such tensors
// along).
#pragma once
#include "enec_kernels.hpp"

namespace enec {

template <int DT, int LPG, class Args>
__global__ void __launch_bounds__(SINGLE_THREADS) compress_single_kernel(const Args p)
{
    extern __shared__ __align__(16) uint8_t smem[];
    compress_one_block<DT, LPG, DT == DT_FP32 ? 2 : 4>(p.item[blockIdx.x], smem, SINGLE_THREADS);
}

}  // namespace enec
