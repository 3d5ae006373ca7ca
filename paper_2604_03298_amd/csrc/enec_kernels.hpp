// Kernel tables of libenec.  Compression with one tuple per tensor has one function per element format, group
// length and kind of block size (the default one as a constant, or any as an argument) that maps a tuple
// (m, a = n - m) to the kernel instance built for it (nullptr if there is none); each of the eighteen is compiled as
// a translation unit of its own (enec_kernels.hip with -DENEC_DT=<format 0|1|2> -DENEC_LPG=<lanes per group 1|2|4>
// -DENEC_LOGB=<14|0>), so that the build runs in parallel and a process loads what it uses: the runtime loads a
// unit's code when the first of its kernels is asked for.
// The other kernels know the widths at run time only and exist once per element format and group length.
#pragma once
#include "enec_device.hpp"

namespace enec {

using CompressFn = void (*)(const CompressArgs);
constexpr uint32_t DEFAULT_LOGB = 14;       // log2 of the default data-block size, which has instances of its own (the _b14 tables)

#define ENEC_TABLES(dt)                                                                             \
    CompressFn pick_compress_##dt##_lpg1_b14(int m, int a), pick_compress_##dt##_lpg1_b0(int m, int a); \
    CompressFn pick_compress_##dt##_lpg2_b14(int m, int a), pick_compress_##dt##_lpg2_b0(int m, int a); \
    CompressFn pick_compress_##dt##_lpg4_b14(int m, int a), pick_compress_##dt##_lpg4_b0(int m, int a);
ENEC_TABLES(dt0)
ENEC_TABLES(dt1)
ENEC_TABLES(dt2)
#undef ENEC_TABLES

// Decompression (enec_decompress.hpp, compiled in enec_decompress.hip).  One launch takes up to MAX_BATCH
// streams of one element format and group length, whatever their tuples.
struct DecompressItem {
    const uint8_t *in;
    void *out;
    uint64_t n_elems;
    uint64_t tuples_at;         // byte offset in the stream of the first block's tuple: the tuple table, or header byte 24
    uint64_t tail_base;         // fp32: where the lower halves of the elements are
    uint64_t payload_base;
    uint64_t payload_bytes;     // total_bytes - payload_base
    uint32_t *status;           // device-accessible or null: set to 7 (format error) when a block is left undecoded
    uint32_t tuple_stride;      // bytes from a block's tuple to the next one's: 4, or 0 if one tuple holds for all
    uint32_t logB;              // log2 of the data-block size
    uint32_t hdr[11];           // the header the launch was configured from
};

struct DecompressArgs {
    uint32_t first[MAX_BATCH];  // number of each stream's first data block among the blocks of the launch
    uint32_t B, logB;           // the block size if all streams have the same
    uint32_t turn_at;           // fp32: byte offset in the dynamic LDS where upper halves change lanes (behind the packed part)
    DecompressItem item[MAX_BATCH];
};

using DecompressFn = void (*)(const DecompressArgs);
DecompressFn pick_decompress(int dtype, unsigned L, bool mixed_block_sizes), pick_decompress_one(int dtype, unsigned L);

// Compression with one tuple per data block (enec_per_block.hpp, compiled in enec_per_block.hip).
// LDS copies of the block histogram in the compress kernel, and their distance in words
constexpr uint32_t PB_HIST_COPIES = 16, PB_HIST_STRIDE = 257;   // words; 16 * 257 * 4 bytes of LDS

// Data blocks are handed out by tickets (see the compress kernel): PB_TICKET_CLASSES counters,
// PB_TICKET_STRIDE 32-bit words apart (a cache line each)
constexpr uint32_t PB_TICKET_CLASSES = 8, PB_TICKET_STRIDE = 16;

struct PbCompressItem {         // one tensor of a launch
    const void *in;
    uint8_t *out;
    unsigned long long *out_bytes;
    uint64_t *words;            // nb look-back words, zero at launch
    uint64_t n_elems;
    uint64_t tuples_at;         // byte offset of the tuple table in the stream
    uint64_t tail_base;         // fp32: where the lower halves go
    uint64_t payload_base;
    uint32_t nb;
    uint32_t first;             // number of its first data block; the blocks of a call are numbered through
};

struct PbCompressArgs {
    PbCompressItem item[MAX_BATCH];
    uint32_t *ticket;           // PB_TICKET_CLASSES counters, zero before the call's first launch
    uint32_t n_items;
    uint32_t first_block;       // this launch codes blocks first_block .. first_block + n_blocks - 1
    uint32_t n_blocks;
    uint32_t B, logB, spin_limit;
    uint32_t park_at;           // byte offset in the dynamic LDS where raw bytes wait (behind the image)
};
constexpr int PB_SM_REG_ROWS = 4;               // rows of a thread's raw bytes kept in registers; the other rows wait in LDS

using PbCompressFn = void (*)(const PbCompressArgs);
PbCompressFn pick_compress_per_block(int dtype, unsigned L);
// the same for blocks of the default size, with deferred stores (its arguments are those of the one-tuple kernels)
constexpr uint32_t pb_image_bytes(uint32_t L) { return (1u << DEFAULT_LOGB) / (8u * L) + (1u << DEFAULT_LOGB); }
CompressFn pick_compress_per_block_stream(int dtype, unsigned L), pick_compress_per_block_stream_fp32(unsigned L);

// Compression of tensors of one data block each (enec_single.hpp, compiled in enec_single.hip), whatever their tuples and
// block sizes: workgroup i takes tensor i.
// A launch of few has arguments of its own: they lie in device memory, where the host writes them over the link (256 bytes
// instead of 1 KB: one, two and four vectors of 4096 elements 6.15, 7.25 and 8.54 us with the long ones, 5.95, 7.04 and 8.35 with these).
constexpr int SINGLE_FEW = 4;
struct SingleArgs {
    SingleItem item[MAX_BATCH];
};
struct SingleFewArgs {
    SingleItem item[SINGLE_FEW];
};

constexpr uint32_t SINGLE_THREADS = 512;
// its dynamic LDS: the transformed bytes in element order (y; fp16: with the three left-over mantissa bits in bits 5..7) | mask | high records
constexpr uint32_t single_lds_bytes(uint32_t B, uint32_t L, uint32_t a) { return B + B / (8u * L) + a * B / 8u; }
using SingleFn = void (*)(const SingleArgs);
using SingleFewFn = void (*)(const SingleFewArgs);
SingleFn pick_compress_single(int dtype, unsigned L);
SingleFewFn pick_compress_single_few(int dtype, unsigned L);

}  // namespace enec
