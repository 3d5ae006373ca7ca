// Compression of tensors of one data block each (norm vectors, biases) with a given tuple, in a launch of their own
// (compress_one_block of enec_device.hpp, which compress_kernel's launches run too where they take such tensors along).
//
// Bound: the latency of a launch.  Such a tensor has no earlier block to wait for and nobody waits for it, so none of what
// compress_kernel does for the order of blocks is needed here: control record, ticket, scan words and the look at them are
// four trips to memory one after the other, and its stores wait for them.  A workgroup takes one tensor; its raw bytes are
// stored as soon as they are split.  The widths and the block size are run-time values, looked up with the tensor, so that
// tensors share a launch whatever their tuples and lengths.
//
// A thread takes eight adjacent elements at a time, not the eight rows of eight columns of the other kernels: a block of
// 4096 elements has eight waves' worth of such vectors and one wave's worth of columns.  The transformed bytes meet in LDS,
// in element order, and Alg. 2's bit map is a table that is read at run time: each byte of a plane is the OR of up to eight
// rotated and masked bytes.  So the code is short, which matters to a kernel that runs each instruction once or twice.
// Two norm vectors of 4096 elements: kernel 4.1 -> 3.2 us (call 6.9 either way, which is the host's time), layer of 405 MB
// 131.8 -> 130.9.
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
