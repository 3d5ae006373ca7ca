// Device code of libenec: the ENEC codec (bf16, fp16, fp32 tensors) on CDNA4 (gfx950), wave64.
//
// Thread mapping (both directions).  A data block of B elements is seen as 8 rows of
// C = B/8 columns: element c + t*C is row t, column c.  Alg. 2 (hierarchical halving
// bit-packing, Sec. V-B) over a whole block only ever combines elements of one column,
// and the a bytes it produces for a column do not depend on B: its "normalized bytes"
// are a planes of C bytes, plane-major.  So a thread that owns 8 adjacent columns
//   * reads / writes, for each row, one 128-bit vector of 8 bf16 (fully coalesced),
//   * packs its 8 columns in registers with byte-lane SIMD-within-a-register
//     arithmetic (4 columns per 32-bit register),
//   * owns half of a group of 16 consecutive elements per row; the two halves sit in
//     adjacent lanes and are combined with one DPP operation.  (Template parameter LPG =
//     lanes per group: 1, 2 or 4 for group lengths 8, 16, 32; Eq. 4 searches the length.)
// A workgroup has B/64 threads (256 for the default B = 16384) and handles one block.
//
// Element formats (template parameter DT).  Only the exponent field is coded (Sec. VI-B);
// every format is first split into an exponent byte X and the raw byte sign<<7 | first seven
// mantissa bits, after which the three formats share all code:
//   DT_BF16  1|8|7   nothing is left over
//   DT_FP16  1|5|10  the last three mantissa bits ride on top of the m low bits of y in the low
//                    plane, which is therefore m + 3 bits wide
//   DT_FP32  1|8|23  the upper half of an element is a bf16 word; the lower halves are copied
//                    to a region between the offset table and the payloads, at positions that
//                    do not depend on any compressed size
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

// Three waves per SIMD for the compression kernel: the register budget (168) that lets three
// workgroups of 256 threads share a CU.  The 16-bit formats fit it once the waiting block's
// sign/mantissa bytes are parked in LDS (all group lengths; the layer with L = 8: 0.177 -> 0.154 ms,
// with L = 32: 0.207 -> 0.181 ms against two waves with the bytes in registers).  The fp32 instances
// (twice the row registers) spill at that budget and run faster with two.
#ifndef ENEC_COMPRESS_OCCUPANCY
#define ENEC_COMPRESS_WAVES (DT != DT_FP32 ? 3 : 2)
#define ENEC_COMPRESS_OCCUPANCY __attribute__((amdgpu_waves_per_eu(ENEC_COMPRESS_WAVES, ENEC_COMPRESS_WAVES)))
#endif

namespace enec {

constexpr int DT_BF16 = 0, DT_FP16 = 1, DT_FP32 = 2;
constexpr int low_plane_bits(int m, int dt) { return m + (dt == DT_FP16 ? 3 : 0); }
constexpr uint32_t exponent_bits(int dt) { return dt == DT_FP16 ? 5u : 8u; }
// The compress instances whose waiting sign/mantissa bytes lie in LDS.  fp32 with a run-time block size has the
// registers for them (two waves per SIMD) and is faster that way (45e6 elements in blocks of 32768: 84.4 against
// 86.9 us; in default blocks, with everything constant, LDS is faster: 78.3 against 80.6).
constexpr bool compress_sm_in_lds(int dt, bool default_block) { return dt != DT_FP32 || default_block; }

// ---------------------------------------------------------------------------------
// Compile-time bit map of Alg. 2 for one column (8 values of W bits -> W bytes).
// A "field" says: bits of row t land in byte `plane` at a constant bit offset.
// ---------------------------------------------------------------------------------
struct HHTable {
    int count;
    int plane[64];
    int row[64];
    int shift[64];        // destination bit - source bit (may be negative)
    unsigned dmask[64];   // destination bits inside the byte
    bool clean[64];       // whole W-bit value fits without spilling into the next byte
};

template <int W>
constexpr HHTable make_hh_table()
{
    HHTable T{};
    int lab[8][16] = {};
    for (int i = 0; i < 8; ++i)
        for (int k = 0; k < 16; ++k) lab[i][k] = (k < W) ? i * 8 + k : -1;
    int width = W, length = 8, planes = 0, n = 0;
    while (width > 0) {
        while (length > 1 && width < 8) {
            length /= 2;
            for (int i = 0; i < length; ++i)
                for (int k = 0; k < width; ++k) lab[i][width + k] = lab[i + length][k];
            width *= 2;
        }
        for (int j = 0; j < length; ++j) {
            for (int t = 0; t < 8; ++t) {
                int shift = 0;
                unsigned dmask = 0, smask = 0;
                for (int k = 0; k < 8; ++k)
                    if (lab[j][k] >= 0 && lab[j][k] / 8 == t) {
                        int sb = lab[j][k] % 8;
                        shift = k - sb;
                        dmask |= 1u << k;
                        smask |= 1u << sb;
                    }
                if (dmask) {
                    T.plane[n] = planes + j;
                    T.row[n] = t;
                    T.shift[n] = shift;
                    T.dmask[n] = dmask;
                    T.clean[n] = (smask == ((1u << W) - 1u)) && shift >= 0 && shift + W <= 8;
                    ++n;
                }
            }
            for (int k = 0; k < 8; ++k) lab[j][k] = lab[j][k + 8];
            for (int k = 8; k < 16; ++k) lab[j][k] = -1;
        }
        planes += length;
        width -= 8;
    }
    T.count = n;
    return T;
}

template <int W> struct HH { static constexpr HHTable table = make_hh_table<W>(); };

__device__ __forceinline__ uint32_t shl_or_shr(uint32_t v, int s)
{
    return s >= 0 ? (v << s) : (v >> (-s));
}

// ---------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------
// Tensors and payloads are read once and written once, so they pass the caches as streaming
// (non-temporal) accesses.  It takes both sides: a copy of 896 MB with blocks of 32 KB runs at 5.4 TB/s
// with plain accesses, at 5.5 / 5.6 with only the loads / only the stores streaming, at 6.2 with both.
// Streaming loads leave nothing in the 256 MB Infinity Cache, so they don't push out what others have just written
// there, and they gain nothing from what lies there.  A 134 MB bf16 tensor, us, streaming / plain loads / the
// kernels before, which had plain accesses on both sides:
//   caches full of another kernel's output   compress 55 / 74 / 76   decompress 44 / 63 / 63
//   input written by the kernel before       compress 54 / 51 / 55   decompress 49 / 38 / 41
//   input brought by a copy from the host                            decompress 45 / 64 / 64
//   the same data again and again            compress 52 / 47 / 58   decompress 40 / 36 / 51
// The last line is for two sets of 232 MB in turn.  Where both sets fit into the cache (67 MB tensors), streaming
// loses to both others: compress 32 / 28 / 30, decompress 22 / 20 / 21, one tuple per block 22 / 19 / 19.  Weights lie in
// memory until their layer comes up and arrive over the host link, which are the first and the third line.
typedef uint32_t vec2u __attribute__((ext_vector_type(2)));
typedef uint32_t vec4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const uint4 *p)
{
    const vec4u v = __builtin_nontemporal_load(reinterpret_cast<const vec4u *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 ld_stream(const uint2 *p)
{
    const vec2u v = __builtin_nontemporal_load(reinterpret_cast<const vec2u *>(p));
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ void st_stream(uint4 *p, uint4 v)
{
    __builtin_nontemporal_store(vec4u{v.x, v.y, v.z, v.w}, reinterpret_cast<vec4u *>(p));
}
__device__ __forceinline__ void st_stream(uint2 *p, uint2 v)
{
    __builtin_nontemporal_store(vec2u{v.x, v.y}, reinterpret_cast<vec2u *>(p));
}
// 16 bytes per lane from memory to LDS without a register in between: lane i's bytes land at `lds` + 16 i
// (`lds` is the same for the whole wave; lanes that are switched off move nothing).  Streaming, as above.
__device__ __forceinline__ void load_to_lds(const uint8_t *p, uint8_t *lds)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 2 /* non-temporal */);
}
// all loads of this wave have arrived (in LDS too; a barrier after it makes them visible to the workgroup), all its stores
// and atomics have been made
__device__ __forceinline__ void wait_accesses()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    // selector byte i picks output byte i: 0-3 = bytes of lo, 4-7 = bytes of hi
    return __builtin_amdgcn_perm(hi, lo, sel);
}

__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b)
{
    return (a & mask) | (b & ~mask);
}

// per-byte (a - b) mod 256 without borrows between bytes
__device__ __forceinline__ uint32_t bytesub_safe(uint32_t a, uint32_t b)
{
    const uint32_t H = 0x80808080u;
    return ((a | H) - (b & ~H)) ^ ((a ^ ~b) & H);
}

// value of the neighbouring lane (lane ^ 1), one DPP move
__device__ __forceinline__ uint32_t swap_pair(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, false);
}

// OR over the four lanes of a quad, two DPP moves
__device__ __forceinline__ uint32_t quad_or(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E /* quad_perm [2,3,0,1] */, 0xF, 0xF, false);
    return v;
}

// v_writelane_b32 (this compiler has no builtin for it; the declaration names LLVM's intrinsic)
extern "C" __device__ int enec_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// a3: the wave's mask bits of the eight rows go into the block's mask (one bit per group, group order = row-major).
// flagged[t] = ballot of "this lane's group of row t needs a record"; the LPG lanes of a group agree, so every LPG-th bit
// counts.  Lane 2t + h takes half h of row t's ballot, and the sixteen lanes squeeze their 32 bits to 32 / LPG and store
// them with one instruction.  (The same on the scalar unit, row after row, was 130 dependent instructions.)
template <int LPG>
__device__ __forceinline__ void put_mask_bits(const uint64_t (&flagged)[8], uint8_t *mask, uint32_t logC, uint32_t wave, uint32_t lane)
{
    uint32_t x = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        x = (uint32_t)enec_writelane((int)(uint32_t)flagged[t], 2 * t, (int)x);
        x = (uint32_t)enec_writelane((int)(uint32_t)(flagged[t] >> 32), 2 * t + 1, (int)x);
    }
    const uint32_t t = lane >> 1, h = lane & 1u;
    // a row's mask is 2^(logC - 3) / LPG bits; the wave's share starts 64 / LPG bits after the one before.  A block of
    // 2048 elements (logC = 8) has half a wave per row: its upper half holds no group.
    const bool mine = lane < 16u && (logC > 8u || h == 0);
    const uint32_t bit = (t << (logC - 3u)) + 64u * wave + 32u * h;      // first lane of the half row, over all rows
    if constexpr (LPG == 1) {
        if (mine) *reinterpret_cast<uint32_t *>(mask + (bit >> 3)) = x;
    } else if constexpr (LPG == 2) {
        x &= 0x55555555u;
        x = (x | (x >> 1)) & 0x33333333u;
        x = (x | (x >> 2)) & 0x0F0F0F0Fu;
        x = (x | (x >> 4)) & 0x00FF00FFu;
        x = x | (x >> 8);
        if (mine) *reinterpret_cast<uint16_t *>(mask + (bit >> 4)) = (uint16_t)x;
    } else {
        x &= 0x11111111u;
        x = (x | (x >> 3)) & 0x03030303u;
        x = (x | (x >> 6)) & 0x000F000Fu;
        x = x | (x >> 12);
        if (mine) mask[bit >> 5] = (uint8_t)x;
    }
}

// inclusive prefix sum over the 64 lanes with data-parallel-primitive moves: four shifts inside
// each row of 16 lanes, then the last lane of a row is broadcast into the next row (rows 1 and 3)
// and the last lane of the lower half into the upper half.  Six dependent VALU operations; the
// same through ds_bpermute (__shfl_up) is six round trips to the LDS crossbar.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, uint32_t /*lane*/)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111 /* row_shr:1 */, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112 /* row_shr:2 */, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114 /* row_shr:4 */, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142 /* row_bcast:15 */, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143 /* row_bcast:31 */, 0xC, 0xF, false);
    return v;
}

// Value of `v` in lane `idx`.  A thread's group of row t lies in mask word (index of the group) / 32;
// for groups of 16 and 32 elements that word index is the same for all lanes of a wave (it depends
// on t and on the wave's number only), so one v_readlane with a scalar index fetches it; for groups
// of 8 the two halves of a wave look at different words and the LDS crossbar is asked.
template <int LPG>
__device__ __forceinline__ uint32_t mask_word_lane(uint32_t v, uint32_t idx)
{
    if constexpr (LPG == 1) return (uint32_t)__shfl((int)v, (int)idx, 64);
    else return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)__builtin_amdgcn_readfirstlane((int)idx));
}

// sum over the 64 lanes of values whose total fits 32 bits, in every lane
__device__ __forceinline__ uint32_t wave_sum32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v, 0), 63);
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)v, d, 64);
        const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), d, 64);
        v += ((uint64_t)hi << 32) | lo;
    }
    return v;
}

// ---------------------------------------------------------------------------------
// Inter-block scan (Fig. 4: prefix sums of per-block compressed sizes) and work distribution.
//
// Scan state.  Block and group words are self-contained: [63:24] tag of the call that wrote it,
// [23] range error, [22:0] a size in units of 16 bytes.  Relaxed device-scope loads and stores
// are enough, no fence is needed, and they are never cleared: a word whose tag is not the
// current call's tag is simply "not published yet".
//   block word k   size of data block k, stored as soon as the block's mask is known
//   group word g   sum of the sizes of the GROUP blocks of group g
//   accumulator g  [63:48] blocks counted, [47:32] of them with a range error, [31:0] sum of
//                  their sizes; zero between calls.  Every block adds itself with one atomic; the
//                  workgroup whose addition completes the group stores the group word and zeroes
//                  the accumulator.  So a group word appears as soon as its last block is known
//                  and no workgroup ever waits for blocks of its own generation (a designated
//                  owner polling the other blocks of its group turned the loop latency-bound as
//                  soon as the blocks took equal time and the workgroups ran in lockstep).
// The start of block k is the sum of the group words below its group plus the block words of the
// earlier blocks of its own group: few words, read by one wave.
//
// Work distribution.  The grid is persistent (at most as many workgroups as the device holds at
// once).  Data blocks are dealt into `ncls` classes, block k belongs to class k mod ncls, and
// class c is served only by the workgroups with blockIdx mod ncls == c, which draw its blocks
// in increasing order from the class's ticket counter.  A workgroup therefore holds blocks in
// increasing order and publishes a block's size before it waits for anything, so the lowest
// unpublished block is always held by (or next in line for) a workgroup that is not waiting for
// it: the scan cannot deadlock.  Eight classes keep the rate of atomics on one address (about
// 12 ns each on MI355X) far below the block rate.
//
// Pipelining.  A workgroup stores block i-1 only while it is working on block i: by then the
// sizes of all earlier blocks were published an iteration ago, so the reads of the scan state
// succeed at the first attempt and nobody spins on hot cache lines in the steady state.
//
// Control record of class c (WS_STRIDE words apart): [0] ticket counter, never reset; [1] value
// of the counter when the current call started; [2..3] tag of the last finished call; class 0 also
// [4..5] tag of the last call in which a workgroup gave up waiting for the scan: whoever writes a
// header looks at it, so that a give-up anywhere in the launch turns every header of the launch
// into status ENEC_E_HIP (the block that gave up was stored at a start computed from a partial sum).  A class
// with L blocks and W workgroups sees exactly L + W draws per call (every workgroup draws until
// its first draw beyond L), so the workgroup that receives draw number L + W - 1 knows that
// nobody will touch the record again in this call and writes the next call's base and tag.
// ---------------------------------------------------------------------------------
constexpr uint64_t ST_ERR = 1ull << 23;
constexpr uint64_t ST_VALUE = (1ull << 23) - 1;
constexpr uint32_t SPIN_LIMIT = 1u << 20;      // default of CompressArgs::spin_limit: seconds, far beyond any real wait
constexpr uint32_t NO_BLOCK = 0xFFFFFFFFu;
constexpr uint32_t WS_STRIDE = 32;            // control records sit 128 bytes apart
constexpr uint32_t WS_CLASSES = 8;
// blocks per scan group: with G blocks a start costs G - 1 block words plus (blocks in flight) / G
// group words, and G additions meet on one accumulator at about 12 ns each
constexpr uint32_t GROUP_LOG = 3, GROUP = 1u << GROUP_LOG;

__device__ __forceinline__ uint64_t ld_state(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_state(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void spin_pause(uint32_t spins)
{
    if (spins < 4) __builtin_amdgcn_s_sleep(4);
    else if (spins < 16) __builtin_amdgcn_s_sleep(16);
    else __builtin_amdgcn_s_sleep(64);
}

// One launch handles up to MAX_BATCH tensors that share (m, n - m, block size): their data blocks
// form one global sequence (tensor after tensor), item[i].first is the global index of tensor i's
// first block.
constexpr int MAX_BATCH = 16;

struct CompressItem {
    const uint16_t *in;
    uint8_t *out;
    uint64_t *out_bytes;    // device-accessible or null
    uint64_t *ws_block;     // nb block words
    uint64_t *ws_group;     // ceil(nb / GROUP) group words
    uint64_t *ws_acc;       // ceil(nb / GROUP) group accumulators, zero between calls
    uint64_t n_elems;
    uint64_t payload_base;
    uint32_t nb, first;
    uint32_t b, mode;       // mode 0: window clear of 0 and 255; 1: n = exponent width; 2: window touches an end
    uint64_t tail_base;     // fp32: where the lower halves of the elements go
};

// a tensor of one data block
struct SingleItem {
    const uint16_t *in;
    uint8_t *out;
    uint64_t *out_bytes;        // device-accessible or null
    uint64_t n_elems;
    uint32_t payload_base, tail_base;
    uint32_t logB, b, n, m, mode;       // mode as in CompressItem
};
// Arguments lie in device memory, where the host writes them over the link for every launch, so what few launches have must
// not make them longer for all: a launch's tensors of one block lie behind its items, from the end of their array down.
struct CompressArgs {
    uint32_t *ws_ctl;       // WS_CLASSES control records
    uint32_t B, logB;
    uint32_t total;         // data blocks of all items
    uint32_t wgs;           // workgroups that code them: the grid without n_single.  (Asked of the runtime, gridDim.x lies behind
                            // all arguments: 256 bytes more of them, and a trip to memory of its own for the first workgroups)
    uint32_t ncls;          // number of block classes = min(8, wgs)
    uint32_t n_items;
    uint32_t spin_limit;    // polls of the scan state after which a workgroup gives up (status ENEC_E_HIP)
    uint16_t lookahead;     // draw the next ticket while working on the current block
    uint16_t n_single;      // tensors of one block that the launch takes along (takes_singles): its first workgroups
    static constexpr uint32_t SINGLES = MAX_BATCH * sizeof(CompressItem) / sizeof(SingleItem);
    union {
        CompressItem item[MAX_BATCH];
        SingleItem behind[SINGLES];
    };
    __host__ __device__ SingleItem &single(uint32_t i) { return behind[SINGLES - 1u - i]; }
    __host__ __device__ const SingleItem &single(uint32_t i) const { return behind[SINGLES - 1u - i]; }
    bool takes_another_single() const
    {
        return n_single < (uint32_t)MAX_BATCH && n_items * sizeof(CompressItem) + (n_single + 1u) * sizeof(SingleItem) <= sizeof item;
    }
};

// ---------------------------------------------------------------------------------
// a5: one record per masked group (Sec. V-B: the high n - m bits of a group that needs them, packed by
// Alg. 2 with N = L), written into the LDS image at the group's rank among the block's masked groups.
// HI[t][h] = high parts of this thread's eight elements of row t in byte lanes; my_word / my_excl = the
// wave's copy of the mask words and of their exclusive popcount prefix.  Shared by the kernels for one
// tuple per tensor and for one tuple per data block.
// ---------------------------------------------------------------------------------
template <int A, int LPG>
__device__ __forceinline__ void pack_records(const uint32_t (&HI)[8][2], uint32_t my_word, uint32_t my_excl,
                                             uint8_t *img_high, uint32_t logC, uint32_t tid, bool active)
{
    constexpr HHTable TH = HH<A>::table;
    constexpr uint32_t RB = A * LPG;                     // bytes of one record: (n - m) L / 8
    if constexpr (LPG == 1) {
        // A group is this lane's 8 elements of a row, and Alg. 2 with N = 8 is the column map
        // itself.  The lane's 8 x 8 bytes (row = group, byte = element) are transposed, so that
        // one register holds the same element of four groups and the eight groups are packed at
        // once in byte lanes; A normalized bytes per group are then joined (byte i with byte
        // i + ceil(A/2)), the pad byte of an odd count is dropped.
        constexpr int HALF = (A + 1) / 2;
        uint32_t T[8][2];                 // T[element][k]: groups 4k .. 4k+3
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t r0 = HI[4 * k][h], r1 = HI[4 * k + 1][h], r2 = HI[4 * k + 2][h], r3 = HI[4 * k + 3][h];
                const uint32_t lo01 = byte_perm(r1, r0, 0x05010400u), hi01 = byte_perm(r1, r0, 0x07030602u);
                const uint32_t lo23 = byte_perm(r3, r2, 0x05010400u), hi23 = byte_perm(r3, r2, 0x07030602u);
                T[4 * h][k] = byte_perm(lo23, lo01, 0x05040100u);
                T[4 * h + 1][k] = byte_perm(lo23, lo01, 0x07060302u);
                T[4 * h + 2][k] = byte_perm(hi23, hi01, 0x05040100u);
                T[4 * h + 3][k] = byte_perm(hi23, hi01, 0x07060302u);
            }
        uint32_t P[A + 1][2];            // normalized byte q of groups 4k .. 4k+3 (P[A] = the pad)
#pragma unroll
        for (int q = 0; q <= A; ++q) P[q][0] = P[q][1] = 0;
#pragma unroll
        for (int f = 0; f < TH.count; ++f)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                P[TH.plane[f]][k] |= shl_or_shr(T[TH.row[f]][k], TH.shift[f]) & (TH.dmask[f] * 0x01010101u);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t g = ((uint32_t)t << (logC - 3)) + tid;
            const uint32_t wv = mask_word_lane<LPG>(my_word, g >> 5);
            const uint32_t pre = mask_word_lane<LPG>(my_excl, g >> 5);
            if (active && ((wv >> (g & 31u)) & 1u)) {
                const uint32_t rank = pre + __popc(wv & ((1u << (g & 31u)) - 1u));
                uint8_t *dst = img_high + RB * rank;
#pragma unroll
                for (int j = 0; j < A; ++j)
                    dst[j] = (uint8_t)(P[(j & 1) ? (j >> 1) + HALF : (j >> 1)][t >> 2] >> (8 * (t & 3)));
            }
        }
    } else if constexpr (LPG == 2) {
        const uint32_t par = tid & 1u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // even lanes pack the group of row 2u, odd lanes the group of row 2u+1
            const uint32_t own0 = par ? HI[2 * u + 1][0] : HI[2 * u][0];
            const uint32_t own1 = par ? HI[2 * u + 1][1] : HI[2 * u][1];
            const uint32_t snd0 = par ? HI[2 * u][0] : HI[2 * u + 1][0];
            const uint32_t snd1 = par ? HI[2 * u][1] : HI[2 * u + 1][1];
            const uint32_t rcv0 = swap_pair(snd0);
            const uint32_t rcv1 = swap_pair(snd1);
            uint32_t F[4];
            F[0] = par ? rcv0 : own0;
            F[1] = par ? rcv1 : own1;
            F[2] = par ? own0 : rcv0;
            F[3] = par ? own1 : rcv1;
            const uint32_t g = ((2u * u + par) << (logC - 4)) + (tid >> 1);
            // even and odd lanes look at the groups of two rows: two wave-uniform word indices
            const uint32_t w_even = (((2u * u) << (logC - 4)) + (tid >> 1)) >> 5;
            const uint32_t w_odd = (((2u * u + 1u) << (logC - 4)) + (tid >> 1)) >> 5;
            const uint32_t wv_e = mask_word_lane<LPG>(my_word, w_even), wv_o = mask_word_lane<LPG>(my_word, w_odd);
            const uint32_t pre_e = mask_word_lane<LPG>(my_excl, w_even), pre_o = mask_word_lane<LPG>(my_excl, w_odd);
            const uint32_t wv = par ? wv_o : wv_e;
            const uint32_t pre = par ? pre_o : pre_e;
            const uint32_t bit = (wv >> (g & 31u)) & 1u;
            if (active && bit) {
                const uint32_t rank = pre + __popc(wv & ((1u << (g & 31u)) - 1u));
                // the group's 16 values are 2 columns of 8 rows: row r = bytes (2r, 2r+1)
                uint32_t P[A];
#pragma unroll
                for (int q = 0; q < A; ++q) P[q] = 0;
#pragma unroll
                for (int f = 0; f < TH.count; ++f) {
                    const int r = TH.row[f];
                    const uint32_t s = shl_or_shr(F[r >> 1], TH.shift[f] - 16 * (r & 1));
                    P[TH.plane[f]] |= s & (TH.dmask[f] * 0x0101u);
                }
                // normalized byte j = byte (j & 1) of P[j >> 1]; stream word i = nb[i] | nb[i + A] << 8
                uint16_t *dst = reinterpret_cast<uint16_t *>(img_high + 2u * A * rank);
#pragma unroll
                for (int i = 0; i < A; ++i) {
                    const uint32_t lo = (P[i >> 1] >> (8 * (i & 1))) & 0xFFu;
                    const uint32_t hi = (P[(i + A) >> 1] >> (8 * ((i + A) & 1))) & 0xFFu;
                    dst[i] = (uint16_t)(lo | (hi << 8));
                }
            }
        }
    } else {
        // a group is the 32 elements of a quad: seen as 8 rows of 4 columns (element i = row i / 4,
        // column i % 4) Alg. 2's folds again stay inside a column; lane j holds rows 2j and 2j+1
        const uint32_t j = tid & 3u;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t g = ((uint32_t)t << (logC - 5)) + (tid >> 2);
            const uint32_t wv = mask_word_lane<LPG>(my_word, g >> 5);
            const uint32_t pre = mask_word_lane<LPG>(my_excl, g >> 5);
            if (active && ((wv >> (g & 31u)) & 1u)) {
                const uint32_t rank = pre + __popc(wv & ((1u << (g & 31u)) - 1u));
                uint32_t P[A];
#pragma unroll
                for (int q = 0; q < A; ++q) P[q] = 0;
#pragma unroll
                for (int f = 0; f < TH.count; ++f) {
                    const int r = TH.row[f];
                    const uint32_t c = shl_or_shr(HI[t][r & 1], TH.shift[f]) & (TH.dmask[f] * 0x01010101u);
                    P[TH.plane[f]] |= ((uint32_t)(r >> 1) == j) ? c : 0u;
                }
#pragma unroll
                for (int q = 0; q < A; ++q) P[q] = quad_or(P[q]);
                if (j == 0) {
                    // normalized byte 4q + c = byte c of P[q]; stream word i = nb[i] | nb[i + 2A] << 8
                    uint32_t *dst = reinterpret_cast<uint32_t *>(img_high + RB * rank);
#pragma unroll
                    for (int k = 0; k < A; ++k) {
                        const int i0 = 2 * k, i1 = 2 * k + 1, h0 = i0 + 2 * A, h1 = i1 + 2 * A;
                        const uint32_t b0 = (P[i0 >> 2] >> (8 * (i0 & 3))) & 0xFFu;
                        const uint32_t b1 = (P[h0 >> 2] >> (8 * (h0 & 3))) & 0xFFu;
                        const uint32_t b2 = (P[i1 >> 2] >> (8 * (i1 & 3))) & 0xFFu;
                        const uint32_t b3 = (P[h1 >> 2] >> (8 * (h1 & 3))) & 0xFFu;
                        dst[k] = b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
                    }
                }
            }
        }
    }
}

// d3: the inverse for row t: the high parts of this thread's eight elements (zero if the group has no record)
template <int A, int LPG>
__device__ __forceinline__ void unpack_record_row(const uint8_t *img_high, uint32_t my_word, uint32_t my_excl,
                                                  uint32_t logC, uint32_t tid, int t, uint32_t &h0, uint32_t &h1)
{
    constexpr HHTable TH = HH<A>::table;
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    constexpr uint32_t RB = A * LPG;
    h0 = h1 = 0;
    const uint32_t g = ((uint32_t)t << (logC - 3 - LOG_LPG)) + (tid >> LOG_LPG);
    const uint32_t wv = mask_word_lane<LPG>(my_word, g >> 5);
    const uint32_t pre = mask_word_lane<LPG>(my_excl, g >> 5);
    if ((wv >> (g & 31u)) & 1u) {
        const uint32_t rank = pre + __popc(wv & ((1u << (g & 31u)) - 1u));
        const uint8_t *rec8 = img_high + RB * rank;
        if constexpr (LPG == 1) {
            // this lane's 8 elements are the group: stream byte j is normalized byte j/2
            // (even j) or j/2 + ceil(A/2) (odd j), the dropped pad byte is zero
            constexpr int HALF = (A + 1) / 2;
            uint32_t P[A + 1];
#pragma unroll
            for (int q = 0; q <= A; ++q) P[q] = 0;
#pragma unroll
            for (int j = 0; j < A; ++j) P[(j & 1) ? (j >> 1) + HALF : (j >> 1)] = rec8[j];
            uint32_t h[2] = {0u, 0u};
#pragma unroll
            for (int f = 0; f < TH.count; ++f) {
                const int r = TH.row[f];
                const uint32_t smask = TH.shift[f] >= 0 ? (TH.dmask[f] >> TH.shift[f])
                                                        : (TH.dmask[f] << (-TH.shift[f]));
                h[r >> 2] |= (shl_or_shr(P[TH.plane[f]], -TH.shift[f]) & smask) << (8 * (r & 3));
            }
            h0 = h[0];
            h1 = h[1];
        } else if constexpr (LPG == 2) {
            const uint32_t par = tid & 1u;
            const uint16_t *rec = reinterpret_cast<const uint16_t *>(rec8);
            uint32_t nbyte[2 * A];
#pragma unroll
            for (int i = 0; i < A; ++i) {
                const uint32_t w = rec[i];
                nbyte[i] = w & 0xFFu;
                nbyte[i + A] = w >> 8;
            }
            uint32_t P[A];
#pragma unroll
            for (int q = 0; q < A; ++q) P[q] = 0;
#pragma unroll
            for (int j = 0; j < 2 * A; ++j) P[j >> 1] |= nbyte[j] << (8 * (j & 1));
            uint32_t E[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) E[r] = 0;
#pragma unroll
            for (int f = 0; f < TH.count; ++f) {
                const uint32_t smask = (TH.shift[f] >= 0 ? (TH.dmask[f] >> TH.shift[f])
                                                        : (TH.dmask[f] << (-TH.shift[f]))) * 0x0101u;
                E[TH.row[f]] |= shl_or_shr(P[TH.plane[f]], -TH.shift[f]) & smask;
            }
            // this lane's 8 elements are rows 4*par .. 4*par+3 of the two-column view
            h0 = par ? (E[4] | (E[5] << 16)) : (E[0] | (E[1] << 16));
            h1 = par ? (E[6] | (E[7] << 16)) : (E[2] | (E[3] << 16));
        } else {
            // the quad's group as 8 rows of 4 columns: stream word i = normalized byte i |
            // normalized byte i + 2A << 8, normalized byte 4q + c = byte c of plane q
            const uint32_t *rec = reinterpret_cast<const uint32_t *>(rec8);
            uint32_t nbyte[4 * A];
#pragma unroll
            for (int k = 0; k < A; ++k) {
                const uint32_t w = rec[k];
                nbyte[2 * k] = w & 0xFFu;
                nbyte[2 * k + 2 * A] = (w >> 8) & 0xFFu;
                nbyte[2 * k + 1] = (w >> 16) & 0xFFu;
                nbyte[2 * k + 1 + 2 * A] = w >> 24;
            }
            uint32_t P[A];
#pragma unroll
            for (int q = 0; q < A; ++q)
                P[q] = nbyte[4 * q] | (nbyte[4 * q + 1] << 8) | (nbyte[4 * q + 2] << 16) | (nbyte[4 * q + 3] << 24);
            uint32_t E[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) E[r] = 0;
#pragma unroll
            for (int f = 0; f < TH.count; ++f) {
                const uint32_t smask = (TH.shift[f] >= 0 ? (TH.dmask[f] >> TH.shift[f])
                                                        : (TH.dmask[f] << (-TH.shift[f]))) * 0x01010101u;
                E[TH.row[f]] |= shl_or_shr(P[TH.plane[f]], -TH.shift[f]) & smask;
            }
            // lane j of the quad holds rows 2j and 2j+1
            const uint32_t j = tid & 3u;
            h0 = j == 0 ? E[0] : (j == 1 ? E[2] : (j == 2 ? E[4] : E[6]));
            h1 = j == 0 ? E[1] : (j == 1 ? E[3] : (j == 2 ? E[5] : E[7]));
        }
    }
}

// a1: 128-bit loads of the 8 rows of data block k (pad elements beyond the tensor's end); a
// thread's 8 elements of a row are one vector (16-bit formats) or two (fp32).
// WHOLE: the tensor's last block, shorter than B, is read with whole vectors; false: element by element (16-bit formats
// only), for kernels that have no registers left for the former.
template <int DT, bool WHOLE = true, class Item>
__device__ __forceinline__ void load_block_rows(const Item &p, uint32_t B, uint32_t logB, uint32_t k,
                                                uint32_t tid, bool active, uint32_t logC,
                                                uint4 (&raw)[DT == DT_FP32 ? 16 : 8])
{
    const uint64_t blk0 = (uint64_t)k << logB;
    // a pad element has exponent b and nothing else: y = 0, raw byte 0, no left-over bits
    const uint32_t padw = DT == DT_FP32 ? (p.b << 23) : (p.b << (DT == DT_FP16 ? 10 : 7)) * 0x00010001u;
    if constexpr (DT == DT_FP32) {
        // plain loads: the two vectors of a thread are halves of the same lines, which streaming loads fetch twice
        // (134e6 elements 202.5 us with streaming loads, 183.4 with plain ones; 45e6 77.6 and 71.8)
        const uint32_t *in = reinterpret_cast<const uint32_t *>(p.in);
        if (blk0 + B <= p.n_elems) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint4 *src = reinterpret_cast<const uint4 *>(in + blk0 + ((uint64_t)t << logC) + 8u * tid);
                raw[2 * t] = active ? src[0] : make_uint4(padw, padw, padw, padw);
                raw[2 * t + 1] = active ? src[1] : make_uint4(padw, padw, padw, padw);
            }
            return;
        }
        const uint32_t left = (uint32_t)(p.n_elems - blk0);       // the tensor's last block, shorter than B
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t at = ((uint32_t)t << logC) + 8u * tid;
            const uint4 *src = reinterpret_cast<const uint4 *>(in + blk0 + at);
            const bool whole = active && at + 8u <= left;
            raw[2 * t] = whole ? src[0] : make_uint4(padw, padw, padw, padw);
            raw[2 * t + 1] = whole ? src[1] : make_uint4(padw, padw, padw, padw);
        }
        if (const uint32_t end = left & ~7u, rest = left & 7u; rest && active && (end & ((1u << logC) - 1u)) == 8u * tid) {
            const uint32_t *src = in + blk0 + end;
            uint32_t d[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = src[(uint32_t)i < rest ? i : 0];
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = (uint32_t)i < rest ? d[i] : padw;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if ((uint32_t)t == end >> logC) {
                    raw[2 * t] = make_uint4(d[0], d[1], d[2], d[3]);
                    raw[2 * t + 1] = make_uint4(d[4], d[5], d[6], d[7]);
                }
        }
    } else {
        if (blk0 + B <= p.n_elems) {               // whole block inside the tensor: no per-row tests
#pragma unroll
            for (int t = 0; t < 8; ++t)
                raw[t] = active ? ld_stream(reinterpret_cast<const uint4 *>(p.in + blk0 + ((uint64_t)t << logC) + 8u * tid))
                                : make_uint4(padw, padw, padw, padw);
            return;
        }
        if constexpr (!WHOLE) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint64_t e0 = blk0 + ((uint64_t)t << logC) + 8u * tid;
                uint32_t d[4] = {padw, padw, padw, padw};
                if (active && e0 < p.n_elems) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (e0 + i < p.n_elems) {
                            const uint32_t v = p.in[e0 + i];
                            d[i >> 1] = (i & 1) ? ((d[i >> 1] & 0x0000FFFFu) | (v << 16))
                                                : ((d[i >> 1] & 0xFFFF0000u) | v);
                        }
                }
                raw[t] = make_uint4(d[0], d[1], d[2], d[3]);
            }
            return;
        }
        // the tensor's last block, shorter than B: whole vectors as ever, and the lane in whose vector the tensor ends
        // asks for those elements together.  (All elements of all eight rows one by one, each under a branch and waited
        // for before the next, made every tensor wait for its last block: three of 8388609 elements 26.8 us, now 24.0.)
        const uint32_t left = (uint32_t)(p.n_elems - blk0);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t at = ((uint32_t)t << logC) + 8u * tid;
            raw[t] = active && at + 8u <= left ? ld_stream(reinterpret_cast<const uint4 *>(p.in + blk0 + at))
                                               : make_uint4(padw, padw, padw, padw);
        }
        if (const uint32_t end = left & ~7u, rest = left & 7u; rest && active && (end & ((1u << logC) - 1u)) == 8u * tid) {
            const uint16_t *src = p.in + blk0 + end;
            uint32_t d[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = src[(uint32_t)i < rest ? i : 0];
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = (uint32_t)i < rest ? d[i] : padw & 0xFFFFu;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if ((uint32_t)t == end >> logC)
                    raw[t] = make_uint4(d[0] | (d[1] << 16), d[2] | (d[3] << 16), d[4] | (d[5] << 16), d[6] | (d[7] << 16));
        }
    }
}

// ---------------------------------------------------------------------------------
// compression of a tensor of one data block by one workgroup (of at most `most` threads): compress_single_kernel, and the
// first workgroups of a compress_kernel launch that has such tensors beside it.  Q: vectors of a thread whose loads travel together
//
// Bound: the latency of a launch.  Such a tensor has no earlier block to wait for and nobody waits for it, so none of what
// compress_kernel does for the order of blocks is needed here: control record, ticket, scan words and the look at them are
// four trips to memory one after the other, and its stores wait for them.  The raw bytes are stored as soon as they are split.
// The widths and the block size are run-time values, looked up with the tensor, so that tensors share a launch whatever their
// tuples and lengths.
//
// A thread takes eight adjacent elements at a time, not the eight rows of eight columns of the other kernels: a block of
// 4096 elements has eight waves' worth of such vectors and one wave's worth of columns.  The transformed bytes meet in LDS,
// in element order, and Alg. 2's bit map is a table that is read at run time: each byte of a plane is the OR of up to eight
// rotated and masked bytes.  So the code is short, which matters to a kernel that runs each instruction once or twice.
// Two norm vectors of 4096 elements in a launch of their own, with columns / vectors: kernel 4.8 / 3.5 us (the call takes 6.9
// either way, which is the host's time).
// ---------------------------------------------------------------------------------
// Alg. 2's bit map for W-bit values (HHTable) by planes: the entries of plane q, unused ones zero.
// Bits 0-2 row, 3-7 rotation to the right, 8-15 destination bits.
struct HHPlanes {
    uint32_t entry[8][8][8];
};
template <int W>
constexpr void hh_planes_of(HHPlanes &p)
{
    constexpr HHTable t = make_hh_table<W>();
    int used[8] = {};
    for (int f = 0; f < t.count; ++f) {
        const int q = t.plane[f];
        p.entry[W - 1][q][used[q]++] = (uint32_t)t.row[f] | ((uint32_t)(-t.shift[f]) & 31u) << 3 | (uint32_t)t.dmask[f] << 8;
    }
    if constexpr (W < 8) hh_planes_of<W + 1>(p);
}
constexpr HHPlanes make_hh_planes()
{
    HHPlanes p{};
    hh_planes_of<1>(p);
    return p;
}
static __device__ const HHPlanes hh_planes = make_hh_planes();

template <int DT, int LPG, int Q>
__device__ __forceinline__ void compress_one_block(const SingleItem &it, uint8_t *smem, uint32_t most)
{
    __shared__ uint32_t s_tab[128], s_err[8];
    constexpr uint32_t E = exponent_bits(DT);
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t logB = it.logB, B = 1u << logB, logC = logB - 3u, nvec = B >> 3, threads = nvec < most ? nvec : most;
    if (tid >= threads) return;                          // whole waves that the launch's larger blocks need
    const uint32_t b = it.b, n = it.n, m = it.m, a = n - m, mode = it.mode;
    const uint32_t lm = m + (DT == DT_FP16 ? 3u : 0u);
    const uint32_t n_elems = (uint32_t)it.n_elems;
    const uint32_t mask_bytes = B >> (6 + LOG_LPG);                   // B / (8 L)
    uint8_t *img_mask = smem + B, *img_high = img_mask + mask_bytes;
    uint8_t *dst = it.out + it.payload_base;
    const uint32_t crep = ((b + (1u << (n - 1))) & 0xFFu) * 0x01010101u;
    const uint32_t srep = (1u << (n - 1)) * 0x01010101u;
    const uint32_t nrep = ((1u << n) - 1u) * 0x01010101u;
    const uint32_t lrep = ((1u << m) - 1u) * 0x01010101u;
    const uint32_t arep = ((1u << a) - 1u) * 0x01010101u;
    const uint32_t xlo = b + 1u > (1u << (n - 1)) ? b + 1u - (1u << (n - 1)) : 0u;
    const uint32_t xhi = b + (1u << (n - 1)) < 255u ? b + (1u << (n - 1)) : 255u;
    // a pad element has exponent b and nothing else: y = 0, raw byte 0, no left-over bits
    const uint32_t padw = DT == DT_FP32 ? (b << 23) : (b << (DT == DT_FP16 ? 10 : 7)) * 0x00010001u;

    uint32_t tab = 0;
    if (tid < 128u) {
        const uint32_t w = tid < 64u ? lm : a;
        if (w) tab = (&hh_planes.entry[w - 1u][0][0])[tid & 63u];
    }

    // ---- a1 split, a2 transform, a3 group test ----
    uint32_t out_of = 0;
    for (uint32_t v0 = tid; v0 < nvec; v0 += Q * threads) {           // (whole waves: nvec and threads are multiples of 64)
        uint4 raw[Q][DT == DT_FP32 ? 2 : 1];
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const uint32_t e = 8u * (v0 + u * threads);
            if (DT == DT_FP32) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(it.in) + e;
                raw[u][0] = raw[u][DT == DT_FP32] = make_uint4(padw, padw, padw, padw);
                if (e + 8u <= n_elems && e < B) {
                    raw[u][0] = reinterpret_cast<const uint4 *>(src)[0];
                    raw[u][DT == DT_FP32] = reinterpret_cast<const uint4 *>(src)[1];
                } else if (e < n_elems) {
                    uint32_t d[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) d[i] = e + i < n_elems ? src[e + i < n_elems ? i : 0] : padw;
                    raw[u][0] = make_uint4(d[0], d[1], d[2], d[3]);
                    raw[u][DT == DT_FP32] = make_uint4(d[4], d[5], d[6], d[7]);
                }
            } else {
                const uint16_t *src = it.in + e;
                raw[u][0] = make_uint4(padw, padw, padw, padw);
                if (e + 8u <= n_elems && e < B) {
                    raw[u][0] = ld_stream(reinterpret_cast<const uint4 *>(src));
                } else if (e < n_elems) {
                    uint32_t d[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) d[i] = src[e + i < n_elems ? i : 0];
#pragma unroll
                    for (int i = 0; i < 8; ++i) d[i] = e + i < n_elems ? d[i] : padw & 0xFFFFu;
                    raw[u][0] = make_uint4(d[0] | (d[1] << 16), d[2] | (d[3] << 16), d[4] | (d[5] << 16), d[6] | (d[7] << 16));
                }
            }
        }
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const uint32_t v = v0 + u * threads;
            if (v >= nvec) break;                                     // (uniform over the wave)
            uint4 r16;
            if constexpr (DT == DT_FP32) {
                const uint4 x = raw[u][0], y = raw[u][1];
                r16 = make_uint4(byte_perm(x.y, x.x, 0x07060302u), byte_perm(x.w, x.z, 0x07060302u),
                                 byte_perm(y.y, y.x, 0x07060302u), byte_perm(y.w, y.z, 0x07060302u));
                if (8u * v < n_elems)
                    st_stream(reinterpret_cast<uint4 *>(it.out + it.tail_base + 16u * v),
                              make_uint4(byte_perm(x.y, x.x, 0x05040100u), byte_perm(x.w, x.z, 0x05040100u),
                                         byte_perm(y.y, y.x, 0x05040100u), byte_perm(y.w, y.z, 0x05040100u)));
            } else {
                r16 = raw[u][0];
            }
            uint32_t sm[2], Y[2], gor = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d0 = h ? r16.z : r16.x, d1 = h ? r16.w : r16.y;
                const uint32_t Lb = byte_perm(d1, d0, 0x06040200u);
                const uint32_t Hb = byte_perm(d1, d0, 0x07050301u);
                uint32_t X, T3 = 0;
                if constexpr (DT == DT_FP16) {
                    sm[h] = (Hb & 0x80808080u) | ((Hb & 0x03030303u) << 5) | ((Lb >> 3) & 0x1F1F1F1Fu);
                    X = (Hb >> 2) & 0x1F1F1F1Fu;
                    T3 = (Lb & 0x07070707u) << 5;
                } else {
                    sm[h] = bfi(0x7F7F7F7Fu, Lb, Hb);
                    X = bfi(0xFEFEFEFEu, Hb << 1, Lb >> 7);
                }
                const uint32_t Z = bytesub_safe(crep, X);
                if (mode == 2) {                   // (a difference modulo 256 could lie in the window by wrapping)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t xb = (X >> (8 * i)) & 0xFFu;
                        out_of |= (uint32_t)((xb < xlo) | (xb > xhi));
                    }
                } else if (mode == 0) {
                    out_of |= Z & ~nrep;
                }
                const uint32_t y = (Z ^ srep) & nrep;
                gor |= (y >> m) & arep;
                Y[h] = y | T3;
            }
            st_stream(reinterpret_cast<uint2 *>(dst + 8u * v), make_uint2(sm[0], sm[1]));
            *reinterpret_cast<uint2 *>(smem + 8u * v) = make_uint2(Y[0], Y[1]);
            if constexpr (LPG == 2) gor |= swap_pair(gor);
            if constexpr (LPG == 4) gor = quad_or(gor);
            // adjacent lanes hold adjacent groups: every LPG-th bit of the ballot, squeezed together
            uint64_t x = __builtin_amdgcn_ballot_w64(gor != 0);
            if constexpr (LPG == 2) {
                x &= 0x5555555555555555ull;
                x = (x | (x >> 1)) & 0x3333333333333333ull;
                x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
                x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
                x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
                x = x | (x >> 16);
            } else if constexpr (LPG == 4) {
                x &= 0x1111111111111111ull;
                x = (x | (x >> 3)) & 0x0303030303030303ull;
                x = (x | (x >> 6)) & 0x000F000F000F000Full;
                x = (x | (x >> 12)) & 0x000000FF000000FFull;
                x = x | (x >> 24);
            }
            if (lane == 0) {
                uint8_t *to = img_mask + (v >> (3 + LOG_LPG));
                if constexpr (LPG == 1) *reinterpret_cast<uint64_t *>(to) = x;
                else if constexpr (LPG == 2) *reinterpret_cast<uint32_t *>(to) = (uint32_t)x;
                else *reinterpret_cast<uint16_t *>(to) = (uint16_t)x;
            }
        }
    }
    const uint64_t any = __builtin_amdgcn_ballot_w64(out_of != 0);
    if (lane == 0) s_err[wave] = any != 0;
    if (tid < 128u) s_tab[tid] = tab;
    __syncthreads();

    // ---- a5 positions: exclusive popcount prefix over the mask words (a wave scan per wave) ----
    const uint32_t nwords = mask_bytes >> 2;                          // at most 64
    const uint32_t my_word = lane < nwords ? reinterpret_cast<const uint32_t *>(img_mask)[lane] : 0u;
    const uint32_t my_pc = __popc(my_word);
    const uint32_t my_incl = wave_incl_scan(my_pc, lane);
    const uint32_t my_excl = my_incl - my_pc;
    const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)my_incl, 63);
    const uint32_t fixed = B + mask_bytes + ((lm * B) >> 3);
    const uint32_t hbytes = (uint32_t)LPG * a * cnt, S = (fixed + hbytes + 15u) & ~15u;

    // ---- a5 one record per masked group: the group's bytes are 8 rows of LPG columns ----
    if (cnt != 0) {
        const uint32_t half = ((uint32_t)LPG * a + 1u) >> 1;          // stream byte 2i = normalized byte i, 2i + 1 = normalized byte i + half
        for (uint32_t g = tid; g < nvec >> LOG_LPG; g += threads) {   // (whole waves but for the last: B / L groups)
            const uint32_t wv = (uint32_t)__shfl((int)my_word, (int)(g >> 5), 64), pre = (uint32_t)__shfl((int)my_excl, (int)(g >> 5), 64);
            if (!((wv >> (g & 31u)) & 1u)) continue;
            uint8_t *rec = img_high + (uint32_t)LPG * a * (pre + __popc(wv & ((1u << (g & 31u)) - 1u)));
            const uint8_t *src = smem + 8u * LPG * g;
            for (uint32_t q = 0; q < a; ++q) {
                uint32_t P = 0;
#pragma unroll
                for (int f = 0; f < 8; ++f) {
                    const uint32_t e = s_tab[64u + 8u * q + f];
                    uint32_t x;
                    if constexpr (LPG == 1) x = src[e & 7u];
                    else if constexpr (LPG == 2) x = *reinterpret_cast<const uint16_t *>(src + 2u * (e & 7u));
                    else x = *reinterpret_cast<const uint32_t *>(src + 4u * (e & 7u));
                    x >>= m;                                          // (bits of the neighbouring byte are masked away)
                    P |= __builtin_amdgcn_alignbit(x, x, (e >> 3) & 31u) & ((e >> 8) * 0x01010101u);
                }
#pragma unroll
                for (uint32_t c = 0; c < (uint32_t)LPG; ++c) {
                    const uint32_t i = (uint32_t)LPG * q + c;
                    rec[i < half ? 2u * i : 2u * (i - half) + 1u] = (uint8_t)(P >> (8u * c));
                }
            }
        }
    }

    // ---- a4 low plane, straight to its place: stream byte 2i = normalized byte i, 2i + 1 = normalized byte i + T/2 ----
    const uint32_t nlow = (lm * B) >> 7, T2 = (lm * B) >> 4;
    for (uint32_t j = tid; j < nlow; j += threads) {
        uint2 part[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t at = 8u * j + (i ? T2 : 0u), q = at >> logC, col = at & ((1u << logC) - 1u);
            uint32_t P0 = 0, P1 = 0;
#pragma unroll
            for (int f = 0; f < 8; ++f) {
                const uint32_t e = s_tab[8u * q + f], r = (e >> 3) & 31u, d = (e >> 8) * 0x01010101u;
                uint2 x = *reinterpret_cast<const uint2 *>(smem + ((e & 7u) << logC) + col);
                if constexpr (DT == DT_FP16) {
                    x.x = (x.x & lrep) | (((x.x >> 5) & 0x07070707u) << m);
                    x.y = (x.y & lrep) | (((x.y >> 5) & 0x07070707u) << m);
                }
                P0 |= __builtin_amdgcn_alignbit(x.x, x.x, r) & d;
                P1 |= __builtin_amdgcn_alignbit(x.y, x.y, r) & d;
            }
            part[i] = make_uint2(P0, P1);
        }
        st_stream(reinterpret_cast<uint4 *>(dst + B + mask_bytes) + j,
                  make_uint4(byte_perm(part[1].x, part[0].x, 0x05010400u), byte_perm(part[1].x, part[0].x, 0x07030602u),
                             byte_perm(part[1].y, part[0].y, 0x05010400u), byte_perm(part[1].y, part[0].y, 0x07030602u)));
    }
    if (tid < mask_bytes >> 4)
        st_stream(reinterpret_cast<uint4 *>(dst + B) + tid, reinterpret_cast<const uint4 *>(img_mask)[tid]);
    if (cnt != 0) {
        __syncthreads();
        for (uint32_t v = tid; 16u * v < hbytes; v += threads) {
            const uint4 o = reinterpret_cast<const uint4 *>(img_high)[v];
            uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {                             // zero the padding behind the last record
                const uint32_t at = 16u * v + 4u * i;
                if (at >= hbytes) w[i] = 0;
                else if (at + 4u > hbytes) w[i] &= (1u << (8u * (hbytes - at))) - 1u;
            }
            st_stream(reinterpret_cast<uint4 *>(dst + fixed) + v, make_uint4(w[0], w[1], w[2], w[3]));
        }
    }
    if (tid == 0) {
        uint32_t err = 0;
        for (uint32_t w = 0; w < threads >> 6; ++w) err |= s_err[w];
        const uint32_t status = err ? 6u : 0u;
        const uint64_t total = status ? 0ull : it.payload_base + S;
        uint64_t *table = reinterpret_cast<uint64_t *>(it.out + 64);
        table[0] = 0;
        table[1] = S;
        uint32_t *h = reinterpret_cast<uint32_t *>(it.out);
        h[0] = 0x43454E45u;                              // "ENEC"
        h[1] = 1u | ((uint32_t)DT << 16) | ((8u * LPG) << 24);   // version, dtype, L
        h[2] = n_elems; h[3] = 0;
        h[4] = B; h[5] = 1;
        h[6] = b | (n << 8) | (m << 16) | (E << 24);
        h[7] = status;
        h[8] = (uint32_t)total; h[9] = 0;
#pragma unroll
        for (int i = 10; i < 16; ++i) h[i] = 0;
        if (it.out_bytes) *it.out_bytes = total;
    }
}

// ---------------------------------------------------------------------------------
// compression: split, transform, group test, packing, inter-block scan, store
// (Sec. V-A compression path; Sec. V-B; Sec. V-C; Fig. 4)
// ---------------------------------------------------------------------------------
// Which instances take tensors of one block along: those of the default block size (2^14) for the tuples that the search returns for
// matrices (bf16 and fp32 n = 5 to 8, fp16 n = 4 and 5, m >= 2 and n - m = 1 to 3, for Gaussian, uniform and heavy-tailed
// weights, with outliers, a scale per row or zeros among them).  compress_one_block does not depend on the widths, and a
// process's first compression loads all instances of a unit: in each of the 44 of bf16, and with four vectors in flight, it made
// their code 1.38 MB instead of 0.98 and that call 2.13 ms instead of 1.90, and it took fp32's instance for (m, n) = (5, 5) over
// the step from three waves per SIMD to two; in these 15, and with one vector, 1.06 MB and 1.98 ms against 1.94.
constexpr bool takes_singles(unsigned m, unsigned a, unsigned logb) { return logb == 14u && m >= 2u && a >= 1u && a <= 3u; }

// LOGB: log2 of the block size where it is a constant, 0 = it is p.B.  The default block size has instances of its
// own: with run-time sizes 50 scalar registers of shifts and offsets are spilled into vector lanes and read back in
// every block; as constants they cost nothing (layer of 405 MB 151.2 -> 147.7 us, 470 MB matrices 312.7 -> 301.6,
// fp16 107.0 -> 104.7, groups of eight 52.9 -> 51.5).
template <int M, int A, int DT, int LPG, uint32_t LOGB>
__global__ void __launch_bounds__(LOGB ? (1 << LOGB) / 64 : 512) ENEC_COMPRESS_OCCUPANCY compress_kernel(const CompressArgs p)
{
    constexpr int N = M + A;
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    constexpr uint32_t RB = A * LPG;                     // bytes of one high record: (n - m) L / 8
    constexpr int LM = low_plane_bits(M, DT);            // width of the low plane
    constexpr uint32_t NMASK = ((1u << N) - 1u) * 0x01010101u;
    constexpr uint32_t LMASK = ((1u << M) - 1u) * 0x01010101u;
    constexpr uint32_t AMASK = ((1u << A) - 1u) * 0x01010101u;
    constexpr uint32_t SREP = (1u << (N - 1)) * 0x01010101u;
    constexpr int MP = LM > 0 ? LM : 1;
    constexpr int AP = A > 0 ? A : 1;
    constexpr int RW = DT == DT_FP32 ? 16 : 8;           // 128-bit vectors of one block per thread
    constexpr bool FULL = N == (int)exponent_bits(DT);   // the window is the whole exponent range (mode 1)
    // With a run-time block size the 16-bit formats have no registers left for two forms of the transform (bf16) and the
    // ragged block in whole vectors: 22 to 34 were spilled, and 67e6 elements took, in blocks of 8192 and groups of 32,
    // 76.4 us (bf16) and 72.5 (fp16) against 61.1 and 60.0 like this; groups of 16 59.9 and 64.7 against 55.2 and 58.1,
    // groups of 8 60.4 and 64.5 against 54.9 and 58.1; three ragged tensors of 1e6 elements in blocks of 2048 15.6 and 15.5
    // against 13.2 and 13.7.  fp32 (two waves per SIMD) and the constant block size have them.
    constexpr bool WHOLE = LOGB != 0 || DT == DT_FP32;
    constexpr bool MODE_PER_STEP = LOGB == 0 && DT == DT_BF16 && !FULL;

    // two LDS images of the packed part of a payload: mask | low plane (as normalized bytes,
    // interleaved on the way out) | high records
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t s_k[2];                // block index of this / the next iteration
    __shared__ unsigned long long s_tag;       // tag of this call
    __shared__ unsigned long long s_off;       // start of the block being stored, bytes
    __shared__ uint32_t s_status;              // header status found by the scan for that block
    __shared__ uint32_t s_err[2];              // range error in the block of image 0 / 1

    constexpr bool TAKES_SINGLES = takes_singles(M, A, LOGB);
    const uint32_t n_single = TAKES_SINGLES ? p.n_single : 0u, wg = blockIdx.x - n_single;
    if constexpr (TAKES_SINGLES)
        if (__builtin_expect((int32_t)wg < 0, 0)) {
            compress_one_block<DT, LPG, 1>(p.single(blockIdx.x), smem, (1u << LOGB) / 64u);
            return;
        }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t B = LOGB ? 1u << LOGB : p.B, logB = LOGB ? LOGB : p.logB, logC = logB - 3u;
    const uint32_t nact = B >> 6, threads = nact < 64u ? 64u : nact;
    const bool active = LOGB || tid < nact;                 // (a constant block has a whole number of waves)
    const uint32_t acc_tid = threads > 64u ? 64u : 0u;      // the lane that talks to the group accumulators
    const uint32_t mask_bytes = (B >> 6) >> LOG_LPG;                  // B / (8 L)
    const uint32_t img_bytes = mask_bytes + (((uint32_t)(LM + A) * B) >> 3);
    const uint32_t fixed = B + mask_bytes + ((LM * B) >> 3);

    // ---- control record of this workgroup's class (thread 0) ---------------------------
    const uint32_t home = wg % p.ncls;
    uint32_t *ctl = p.ws_ctl + WS_STRIDE * home;
    const uint32_t class_blocks = home < p.total ? (p.total - home + p.ncls - 1u) / p.ncls : 0u;
    const uint32_t class_wgs = (p.wgs - home + p.ncls - 1u) / p.ncls;
    uint32_t ticket_base = 0, zero = 0;
    uint64_t tag0 = 0;
    bool drawing = true;
    // decode a draw; the last draw of the class hands the record over to the next call
    auto decode_draw = [&](uint32_t raw) -> uint32_t {
        const uint32_t t = raw - ticket_base;
        if (t == class_blocks + class_wgs - 1u) {
            ctl[1] = raw + 1u;
            for (uint32_t c = home; c < WS_CLASSES; c += p.ncls)
                *reinterpret_cast<uint64_t *>(p.ws_ctl + WS_STRIDE * c + 2) = tag0;
        }
        if (t >= class_blocks) { drawing = false; return NO_BLOCK; }
        return t * p.ncls + home;
    };
    uint32_t slot = 0;
    // tensor that global block kg belongs to, searching upwards from item c
    auto item_of = [&](uint32_t kg, uint32_t c) -> uint32_t {
        while (c + 1u < p.n_items && kg >= p.item[c + 1u].first) ++c;
        return c;
    };
    // Every block is drawn, also the first one: a workgroup that is dispatched late (the device may
    // be shared with other kernels) must not own a block that running workgroups wait for.  When all
    // workgroups start together, workgroup w draws block w, so its rows are requested on that guess
    // while the control record and the draw are still travelling.
    const uint32_t guess = wg;                       // the grid never exceeds the number of blocks
    uint32_t ci = item_of(guess, 0);
    uint4 raw[RW];
    load_block_rows<DT, WHOLE>(p.item[ci], B, logB, guess - p.item[ci].first, tid, active, logC, raw);
    if (tid == 0) {
        ticket_base = ctl[1];
        tag0 = *reinterpret_cast<const uint64_t *>(ctl + 2) + 1u;
        // the record must have been read before this workgroup's first draw can be counted
        zero = ticket_base ^ (uint32_t)tag0;
        asm volatile("v_and_b32 %0, 0, %0" : "+v"(zero));
        s_k[0] = decode_draw(atomicAdd(ctl + zero, 1u));
        s_tag = tag0;
        s_err[0] = s_err[1] = 0;
        s_status = 0;
    }
    __syncthreads();
    uint32_t k = __builtin_amdgcn_readfirstlane(s_k[0]);     // global block index
    if (k != guess && k != NO_BLOCK) {                       // the guess was wrong: ask again
        ci = item_of(k, 0);
        load_block_rows<DT, WHOLE>(p.item[ci], B, logB, k - p.item[ci].first, tid, active, logC, raw);
    }
    const uint64_t tag = (uint64_t)s_tag << 24;
    constexpr HHTable TL = HH<MP>::table;

    // wave 0 carries the scan of one tensor: sum of its group words [0, groups_summed) and what
    // went wrong so far (bit 1 range error in an earlier block, bit 2 gave up waiting)
    uint64_t groups_sum = 0;
    uint32_t groups_summed = 0, scan_flags = 0, scan_item = NO_BLOCK;

    // sum of the (valid) words base[0 .. count), count <= 64, one word per lane; `v` may hold a
    // copy read earlier (have = true), words that were not valid yet are read again until they are
    auto sum_words = [&](const uint64_t *base, uint32_t count, bool have, uint64_t v, uint32_t &flags) -> uint64_t {
        const bool need = lane < count;
        bool ok = !need || (have && (v & ~0xFFFFFFull) == tag);
        uint32_t spins = 0;
        while (__builtin_amdgcn_ballot_w64(!ok) != 0) {
            if (!ok) {
                v = ld_state(base + lane);
                ok = (v & ~0xFFFFFFull) == tag;
            }
            if (__builtin_amdgcn_ballot_w64(!ok) == 0) break;
            if (++spins > p.spin_limit) {                                      // never hang
                flags |= 4u;
                v = 0;
                if (lane == 0) st_state(reinterpret_cast<uint64_t *>(p.ws_ctl + 4), tag);
                break;
            }
            spin_pause(spins);
        }
        if (__builtin_amdgcn_ballot_w64(need && (v & ST_ERR))) flags |= 2u;
        // at most 64 sizes below 2^23 units of 16 bytes: the sum fits 32 bits
        return wave_sum32(need ? (uint32_t)(v & ST_VALUE) : 0u);
    };
    // start of block kb (wave 0; early_g / early_b = copies of the first needed group words / of
    // the earlier block words of its group, read ahead of time)
    auto block_start = [&](const CompressItem &it, uint32_t kb, bool early, uint64_t early_g, uint64_t early_b) -> uint64_t {
        const uint32_t g = kb >> GROUP_LOG;
        while (groups_summed < g) {
            const uint32_t c = g - groups_summed < 64u ? g - groups_summed : 64u;
            groups_sum += sum_words(it.ws_group + groups_summed, c, early, early_g, scan_flags);
            groups_summed += c;
            early = false;
        }
        const uint64_t own_group = sum_words(it.ws_block + ((uint64_t)g << GROUP_LOG), kb & (GROUP - 1u), early_b != 0, early_b, scan_flags);
        return (groups_sum + own_group) << 4;
    };

    // the block waiting to be stored
    uint32_t pend = NO_BLOCK, pend_item = 0, pend_cnt = 0, pend_S = 0, pend_err = 0;   // pend: index inside its tensor
    // its sign/mantissa bytes wait in LDS behind the two images, in element order (in registers they were
    // what the compiler spilled), or in registers
    constexpr bool SM_IN_LDS = compress_sm_in_lds(DT, LOGB != 0);
    uint32_t SMp[SM_IN_LDS ? 1 : 8][2];
    uint8_t *sm_wait = smem + 2u * img_bytes;

    // stores block `kb` whose packed part sits in image `img` and whose sign/mantissa bytes sit in sm_wait
    auto store_block = [&](const CompressItem &it, uint32_t kb, uint32_t cnt, uint32_t S, const uint8_t *img,
                           uint32_t err_own) {
        const uint64_t off = s_off;
        uint8_t *dst = it.out + it.payload_base + off;
        // The payload leaves as one run of 16-byte vectors, sign/mantissa plane | mask | low plane | high
        // records.  Payloads start at multiples of 16 bytes, lines are 128: the vectors are dealt to the lanes
        // so that a wave's kilobyte begins at a line, because a streaming store of part of a line costs more
        // than its bytes (64-byte pieces: 3.7 instead of 6.0 TB/s in a plain copy).  Against the same run dealt from
        // the payload's start it writes 1.6 % less (470 MB matrices 343.2 against 349.0 MB per launch) and is worth
        // 1 to 2 % in batches (16 x 34 MB 179.8 against 183.2 us, 7 x 34 MB 85.8 / 87.1) and 1 to 5 % for blocks of
        // 2048; nothing on one large tensor (537 MB 174.5 / 174.6); one small tensor loses 2 % (34 MB 21.1 / 20.7).
        const uint32_t shift = (uint32_t)((uintptr_t)dst >> 4) & 7u;     // vectors of the first line that are not ours
        const uint32_t nsm = B >> 4, nmask = mask_bytes >> 4, nlow = (LM * B) >> 7;
        const uint32_t hbytes = RB * cnt, nall = S >> 4;
        // vector j of the low plane: stream byte 2i = normalized byte i, stream byte 2i+1 = normalized byte i + T/2
        auto low_vector = [&](uint32_t j) -> uint4 {
            const uint32_t T2 = (LM * B) >> 4;                           // half of the plane's length
            const uint8_t *ilow = img + mask_bytes + 8u * j;
            const uint2 a = *reinterpret_cast<const uint2 *>(ilow);
            const uint2 c = *reinterpret_cast<const uint2 *>(ilow + T2);
            return make_uint4(byte_perm(c.x, a.x, 0x05010400u), byte_perm(c.x, a.x, 0x07030602u),
                              byte_perm(c.y, a.y, 0x05010400u), byte_perm(c.y, a.y, 0x07030602u));
        };
        // vector u of the packed part, behind the low plane: the padding behind the last record is zero
        auto high_vector = [&](uint32_t u) -> uint4 {
            const uint4 o = *reinterpret_cast<const uint4 *>(img + 16u * u);
            const uint32_t at = 16u * (u - nmask - nlow);
            if (at + 16u <= hbytes) return o;
            uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (at + 4u * i >= hbytes) w[i] = 0;
                else if (at + 4u * i + 4u > hbytes) w[i] &= (1u << (8u * (hbytes - at - 4u * i))) - 1u;
            }
            return make_uint4(w[0], w[1], w[2], w[3]);
        };
        auto packed_vector = [&](uint32_t u) -> uint4 {
            if (LM > 0 && u - nmask < nlow) return low_vector(u - nmask);            // (wraps for a mask vector)
            if (A == 0 || u < nmask) return *reinterpret_cast<const uint4 *>(img + 16u * u);
            return high_vector(u);
        };
        int32_t v = (int32_t)tid - (int32_t)shift;
        if constexpr (LOGB != 0) {
            // Constant sizes: round i stores vectors i threads - 7 .. i threads + threads - 1, so all but the rounds in
            // which one region ends and the next begins know at compile time what they store.
            constexpr int T = (1 << LOGB) / 64, NSM = (1 << LOGB) / 16, NLO = NSM + (1 << LOGB) / (1024 * LPG), NHI = NLO + (LM << LOGB) / 128;
            constexpr int ROUNDS = (NHI + 7 + T - 1) / T;                // rounds that reach below NHI
#pragma unroll
            for (int i = 0; i < ROUNDS; ++i) {
                const int first = i * T - 7, last = i * T + T - 1;
                const int32_t w = v + i * T;
                if ((first < 0 && w < 0) || (last >= NHI && w >= (int32_t)nall)) continue;
                uint4 o;
                if (last < NSM || (first < NSM && w < NSM)) o = reinterpret_cast<const uint4 *>(sm_wait)[w];
                else if (LM > 0 && first >= NLO && last < NHI) o = low_vector((uint32_t)w - NLO);
                else o = packed_vector((uint32_t)w - NSM);
                st_stream(reinterpret_cast<uint4 *>(dst) + w, o);
            }
            if constexpr (A > 0)
                for (v += ROUNDS * T; v < (int32_t)nall; v += T) st_stream(reinterpret_cast<uint4 *>(dst) + v, high_vector((uint32_t)v - NSM));
        } else {
            if constexpr (!SM_IN_LDS) {
                if (active) {
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        st_stream(reinterpret_cast<uint2 *>(dst + ((size_t)t << logC) + 8u * tid), make_uint2(SMp[t][0], SMp[t][1]));
                }
                while (v < (int32_t)nsm) v += (int32_t)threads;
            }
            for (; v < (int32_t)nsm; v += (int32_t)threads)
                if (v >= 0)
                    st_stream(reinterpret_cast<uint4 *>(dst) + v, reinterpret_cast<const uint4 *>(sm_wait)[v]);
            for (; v < (int32_t)nall; v += (int32_t)threads)
                st_stream(reinterpret_cast<uint4 *>(dst) + v, packed_vector((uint32_t)v - nsm));
        }
        if (tid == 0) {
            uint64_t *table = reinterpret_cast<uint64_t *>(it.out + 64);
            table[kb] = off;
            if (kb == it.nb - 1u) {
                const uint64_t end = off + S;
                uint32_t fl = s_status | err_own;
                if (ld_state(reinterpret_cast<const uint64_t *>(p.ws_ctl + 4)) == tag) fl |= 4u;   // somebody gave up
                const uint32_t status = (fl & 4u) ? 8u : ((fl & 3u) ? 6u : 0u);
                const uint64_t total = status ? 0ull : it.payload_base + end;
                table[it.nb] = end;
                if (((uint64_t)(it.nb + 1u) & 1ull)) table[it.nb + 1u] = 0;   // pad up to the payload base
                uint32_t *h = reinterpret_cast<uint32_t *>(it.out);
                h[0] = 0x43454E45u;                              // "ENEC"
                h[1] = 1u | ((uint32_t)DT << 16) | ((8u * LPG) << 24);   // version, dtype, L
                h[2] = (uint32_t)it.n_elems; h[3] = (uint32_t)(it.n_elems >> 32);
                h[4] = B; h[5] = it.nb;
                h[6] = it.b | ((uint32_t)N << 8) | ((uint32_t)M << 16) | (exponent_bits(DT) << 24);
                h[7] = status;
                h[8] = (uint32_t)total; h[9] = (uint32_t)(total >> 32);
#pragma unroll
                for (int i = 10; i < 16; ++i) h[i] = 0;
                if (it.out_bytes) *it.out_bytes = total;
            }
        }
    };

    while (k != NO_BLOCK) {
        uint8_t *img = smem + slot * img_bytes;
        uint32_t *img_maskw = reinterpret_cast<uint32_t *>(img);
        uint8_t *img_low = img + mask_bytes;
        uint8_t *img_high = img_low + (((size_t)LM * B) >> 3);

        // wave 0 reads the scan state for the block stored in this iteration now and uses it
        // after the arithmetic: published an iteration ago, it is normally all there
        const CompressItem &it = p.item[ci];
        const uint32_t kl = k - it.first;                    // index of the block inside its tensor
        const uint32_t crep = ((it.b + (1u << (N - 1))) & 0xFFu) * 0x01010101u;
        const uint32_t xlo = it.b + 1u > (1u << (N - 1)) ? it.b + 1u - (1u << (N - 1)) : 0u;
        const uint32_t xhi = it.b + (1u << (N - 1)) < 255u ? it.b + (1u << (N - 1)) : 255u;
        const uint32_t mode = it.mode;
        uint64_t early_g = 0, early_b = 0;
        if (wave == 0 && pend != NO_BLOCK) {
            if (scan_item != pend_item) { scan_item = pend_item; groups_sum = 0; groups_summed = 0; scan_flags = 0; }
            const CompressItem &pit = p.item[pend_item];
            const uint32_t pg = pend >> GROUP_LOG;
            if (groups_summed + lane < pg) early_g = ld_state(pit.ws_group + groups_summed + lane);
            if (lane < (pend & (GROUP - 1u))) early_b = ld_state(pit.ws_block + ((uint64_t)pg << GROUP_LOG) + lane);
        }

        // the ticket for the following block is drawn now and looked at after the arithmetic
        uint32_t next_raw = 0;
        const bool draw_now = tid == 0 && p.lookahead && drawing;
        if (draw_now) next_raw = atomicAdd(ctl + zero, 1u);

        uint32_t SMc[8][2], HI[8][2], accP[MP][2];
        uint64_t flagged[8];
        uint32_t err_acc = 0;
        bool bad = false;
#pragma unroll
        for (int q = 0; q < MP; ++q) accP[q][0] = accP[q][1] = 0;

        const uint64_t row0 = ((uint64_t)kl << logB) + 8u * tid;   // this thread's first element of row 0
        // WRAP: the bytes are subtracted without borrows between them, and where the window is not the whole exponent
        // range every exponent is compared with it.  Two straight runs of code and one branch: a branch on the mode at
        // each of the sixteen subtractions (MODE_PER_STEP) cuts the transform into pieces that nothing is scheduled across.
        auto transform = [&](auto wrap) {
        constexpr bool WRAP = decltype(wrap)::value;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint32_t gor = 0;
            uint4 r16;                           // the row's eight 16-bit words
            if constexpr (DT == DT_FP32) {
                // upper halves go on as bf16 words, lower halves leave at once
                const uint4 u = raw[2 * t], v = raw[2 * t + 1];
                r16 = make_uint4(byte_perm(u.y, u.x, 0x07060302u), byte_perm(u.w, u.z, 0x07060302u),
                                 byte_perm(v.y, v.x, 0x07060302u), byte_perm(v.w, v.z, 0x07060302u));
                const uint64_t e0 = row0 + ((uint64_t)t << logC);
                if (active && e0 < it.n_elems)   // elements past the end are pads with zero lower halves
                    st_stream(reinterpret_cast<uint4 *>(it.out + it.tail_base + 2u * e0),
                              make_uint4(byte_perm(u.y, u.x, 0x05040100u), byte_perm(u.w, u.z, 0x05040100u),
                                         byte_perm(v.y, v.x, 0x05040100u), byte_perm(v.w, v.z, 0x05040100u)));
            } else {
                r16 = raw[t];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d0 = h ? r16.z : r16.x;
                const uint32_t d1 = h ? r16.w : r16.y;
                // a1 split: low / high bytes of four 16-bit words
                const uint32_t Lb = byte_perm(d1, d0, 0x06040200u);
                const uint32_t Hb = byte_perm(d1, d0, 0x07050301u);
                uint32_t X, T3 = 0;
                if constexpr (DT == DT_FP16) {
                    SMc[t][h] = (Hb & 0x80808080u) | ((Hb & 0x03030303u) << 5) | ((Lb >> 3) & 0x1F1F1F1Fu);
                    X = (Hb >> 2) & 0x1F1F1F1Fu;
                    T3 = Lb & 0x07070707u;
                } else {
                    SMc[t][h] = bfi(0x7F7F7F7Fu, Lb, Hb);
                    X = bfi(0xFEFEFEFEu, Hb << 1, Lb >> 7);
                }
                // a2 transform: z = (b + 2^(n-1) - x) mod 256 per byte, y = z with the sign bit flipped
                uint32_t Z;
                if constexpr (MODE_PER_STEP) {
                    if (mode == 0) {
                        Z = crep - X;
                        err_acc |= Z;
                    } else {
                        Z = bytesub_safe(crep, X);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t xb = (X >> (8 * i)) & 0xFFu;
                            bad |= (xb < xlo) | (xb > xhi);
                        }
                    }
                } else if constexpr (!WRAP) {
                    Z = crep - X;
                    err_acc |= Z;
                } else {
                    Z = bytesub_safe(crep, X);
                    if constexpr (!FULL) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t xb = (X >> (8 * i)) & 0xFFu;
                            bad |= (xb < xlo) | (xb > xhi);
                        }
                    }
                }
                uint32_t Y = Z ^ SREP;
                if (N < 8) Y &= NMASK;
                // a3: high parts decide the group; a4: low parts go to the column packer
                const uint32_t hi = A > 0 ? ((Y >> M) & AMASK) : 0u;
                HI[t][h] = hi;
                gor |= hi;
                if (LM > 0) {
                    const uint32_t low = (Y & LMASK) | (T3 << M);
#pragma unroll
                    for (int f = 0; f < TL.count; ++f)
                        if (TL.row[f] == t) {
                            uint32_t s = shl_or_shr(low, TL.shift[f]);
                            if (!TL.clean[f]) s &= TL.dmask[f] * 0x01010101u;
                            accP[TL.plane[f]][h] |= s;
                        }
                }
            }
            // a3: OR over the lanes that share a group, one mask bit per group
            if constexpr (LPG == 2) gor |= swap_pair(gor);
            if constexpr (LPG == 4) gor = quad_or(gor);
            flagged[t] = __builtin_amdgcn_ballot_w64(gor != 0);
        }
        };
        if constexpr (FULL) {
            transform(std::true_type{});
        } else if constexpr (MODE_PER_STEP) {
            transform(std::true_type{});
            if (mode == 0) bad = (err_acc & ~NMASK) != 0;
        } else if (DT == DT_FP16 || mode == 0) {
            transform(std::false_type{});
            bad = (err_acc & ~NMASK) != 0;
        } else {
            transform(std::true_type{});
        }
        if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) atomicOr(&s_err[slot], 1u);

        if (64u * wave < nact) put_mask_bits<LPG>(flagged, img, logC, wave, lane);
        if (LM > 0 && active) {
#pragma unroll
            for (int q = 0; q < LM; ++q)
                *reinterpret_cast<uint2 *>(img_low + ((size_t)q << logC) + 8u * tid) =
                    make_uint2(accP[q][0], accP[q][1]);
        }
        if (tid == 0) s_k[slot ^ 1u] = draw_now ? decode_draw(next_raw) : NO_BLOCK;
        __syncthreads();                                                     // barrier 1

        // ---- a5 (positions): exclusive popcount prefix over the block's mask words; every wave
        // computes it for itself (a wave scan of at most 64 words) -----------------------
        const uint32_t nwords = (B >> 8) >> LOG_LPG;          // 32-bit words of the mask (at most 64)
        const uint32_t my_word = lane < nwords ? img_maskw[lane] : 0u;
        const uint32_t my_pc = __popc(my_word);
        const uint32_t my_incl = wave_incl_scan(my_pc, lane);
        const uint32_t my_excl = my_incl - my_pc;
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)my_incl, 63);
        const uint32_t own_err = s_err[slot] & 1u;
        const uint32_t S = (fixed + RB * cnt + 15u) & ~15u;

        // ---- a6: publish this block's size at once, and add it to its group's accumulator
        // [blocks:16 | blocks with a range error:16 | sum of sizes:32]; what the addition returns
        // is looked at after barrier 2, when it has had time to travel ---------------------
        if (tid == 0) st_state(it.ws_block + kl, tag | (own_err ? ST_ERR : 0ull) | (uint64_t)(S >> 4));
        // (a group of one block, e.g. a tensor of one block, is complete with its only member)
        const uint32_t grp = kl >> GROUP_LOG;
        const uint32_t members = it.nb - (grp << GROUP_LOG) < GROUP ? it.nb - (grp << GROUP_LOG) : GROUP;
        uint64_t acc_old = 0;
        if (tid == acc_tid && members > 1u)
            acc_old = __hip_atomic_fetch_add(it.ws_acc + grp, (1ull << 48) | ((uint64_t)own_err << 32) | (uint64_t)(S >> 4),
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // ---- a5: one record per masked group ------------------------------------------
        if constexpr (A > 0) pack_records<A, LPG>(HI, my_word, my_excl, img_high, logC, tid, active);

        // ---- a6 (wave 0): the start of the block stored in this iteration -----------------
        if (wave == 0 && pend != NO_BLOCK) {
            const uint64_t off = block_start(p.item[pend_item], pend, true, early_g, early_b);
            if (lane == 0) { s_off = off; s_status = scan_flags; }
        }
        __syncthreads();                                                     // barrier 2
        if (tid == 0) s_err[slot] = 0;          // read by everybody before barrier 2; next use in two iterations

        // ---- a6: whoever completes a group publishes its word and clears the accumulator for
        // the next call; nobody ever waits for blocks of its own generation ------------------
        if (tid == acc_tid) {
            if ((uint32_t)(acc_old >> 48) == members - 1u) {
                const uint64_t sum = (acc_old & 0xFFFFFFFFull) + (S >> 4);
                const bool any_err = ((acc_old >> 32) & 0xFFFFull) != 0 || own_err;
                st_state(it.ws_group + grp, tag | (any_err ? ST_ERR : 0ull) | sum);
                if (members > 1u) st_state(it.ws_acc + grp, 0ull);
            }
        }

        // the following block's rows start to travel while the previous block is stored
        const uint32_t knext = __builtin_amdgcn_readfirstlane(s_k[slot ^ 1u]);
        uint32_t cnext = ci;
        if (knext != NO_BLOCK) {
            cnext = item_of(knext, ci);
            load_block_rows<DT, WHOLE>(p.item[cnext], B, logB, knext - p.item[cnext].first, tid, active, logC, raw);
        }

        // ---- a7: stores of the previous block ----------------------------------------------
        if (pend != NO_BLOCK)
            store_block(p.item[pend_item], pend, pend_cnt, pend_S, smem + (slot ^ 1u) * img_bytes, pend_err);
        __syncthreads();                                                     // barrier 3: other image free

        // this block becomes the pending one
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if constexpr (SM_IN_LDS) {
                if (active)
                    *reinterpret_cast<uint2 *>(sm_wait + ((size_t)t << logC) + 8u * tid) = make_uint2(SMc[t][0], SMc[t][1]);
            } else {
                SMp[t][0] = SMc[t][0];
                SMp[t][1] = SMc[t][1];
            }
        }
        pend = kl; pend_item = ci; pend_cnt = cnt; pend_S = S; pend_err = own_err;
        slot ^= 1u;
        k = knext;
        ci = cnext;
        if (k == NO_BLOCK && !p.lookahead) {           // without lookahead the next ticket is drawn only now
            if (tid == 0) s_k[slot] = drawing ? decode_draw(atomicAdd(ctl + zero, 1u)) : NO_BLOCK;
            __syncthreads();
            k = __builtin_amdgcn_readfirstlane(s_k[slot]);
            if (k != NO_BLOCK) {
                ci = item_of(k, ci);
                load_block_rows<DT, WHOLE>(p.item[ci], B, logB, k - p.item[ci].first, tid, active, logC, raw);
            }
        }
    }

    // ---- drain: the last block of this workgroup ---------------------------------------------
    if (pend != NO_BLOCK) {
        if (wave == 0) {
            if (scan_item != pend_item) { scan_item = pend_item; groups_sum = 0; groups_summed = 0; scan_flags = 0; }
            const uint64_t off = block_start(p.item[pend_item], pend, false, 0, 0);
            if (lane == 0) { s_off = off; s_status = scan_flags; }
        }
        __syncthreads();
        store_block(p.item[pend_item], pend, pend_cnt, pend_S, smem + (slot ^ 1u) * img_bytes, pend_err);
    }
}

// ---------------------------------------------------------------------------------
// exponent histogram (Sec. V-E phase 1), of the whole tensor (every = 1) or of a sample of it
// ---------------------------------------------------------------------------------
constexpr uint32_t SAMPLE_CHUNK = 4096;     // elements; the sample is taken in whole chunks

struct HistogramItem {          // one tensor of a launch
    const void *in;
    uint64_t n_elems;
    unsigned long long *hist;   // 256 counters, zero at launch and again at the end
    uint32_t first, count;      // its workgroups: first .. first + count - 1
};
struct HistogramArgs {
    HistogramItem item[MAX_BATCH];
    uint32_t n_items, every;
    uint32_t *done;             // workgroups that have added their counts, zero at launch and again at the end
    unsigned long long *counts; // all histograms of the call, one behind the other
    unsigned long long *host;   // pinned memory: where they go
    uint32_t *arrived;          // pinned memory: set to 1 (0 when the kernel has ended: nobody was last, see enec_tune_batch)
    uint32_t n_counts, wgs;     // wgs: the grid
};

// Bound: HBM, with the LDS atomics (7.2 lanes per clock and CU: 46 us for a layer of 202e6 elements) not far behind.
// One workgroup per CU: each ends with a global atomic per exponent value it has seen, on addresses that all of its
// tensor's workgroups share, 12 ns apiece.  Eight waves with four vectors each in flight and the next four asked for
// before the present ones are counted: 202e6 elements 61 us (6.6 TB/s); without asking ahead, 512 workgroups of four
// waves, 70.  Whole calls, us, 512 threads x 256 workgroups against 512 x 512 / 1024 x 256 / 256 x 1024: layer
// 99.4 against 101.3 / 103.2 / 103.2, 268e6 elements 107.7 / 117.0 / 112.1 / 124.9, 17e6 41.0 / 44.4 / 40.7 / 53.0;
// six or eight vectors in flight are slower again (layer 103.5, 103.9).
// The workgroup that adds its counts last hands all of them over and leaves the counters zero for the next call.  With a kernel
// before this one that cleared them and one behind it that handed them over a call took, for the layer / twenty tensors of
// 262144 elements / one of 1e6, 85.4 / 56.6 / 25.6 us, now 83.3 / 53.9 / 22.7; with one count of a thread after the other, each
// waited for, and sums on the host beside the search 84.3 / 57.8 / 23.3.
constexpr uint32_t HIST_THREADS = 512, HIST_WORKGROUPS = 256;

template <int DT>
__global__ void __launch_bounds__(HIST_THREADS) histogram_kernel(const HistogramArgs p)
{
    uint32_t ti = 0;
    for (uint32_t i = 1; i < p.n_items; ++i)
        if (blockIdx.x >= p.item[i].first) ti = i;
    const void *in_ = p.item[ti].in;
    const uint64_t n_elems = p.item[ti].n_elems;
    unsigned long long *hist = p.item[ti].hist;
    const uint32_t every = p.every;
    const uint32_t wg = blockIdx.x - p.item[ti].first, wgs = p.item[ti].count;    // this tensor's share of the grid
    // 32 copies of the histogram, lane i of every wave counts into copy i mod 32: lanes with equal
    // exponents, the normal case, would otherwise queue up on one LDS word; the copies are 257 words
    // apart, which puts the same bin of all copies into different banks.  (Measured on this machine:
    // LDS atomics run at 7.2 lanes per clock and CU when no two lanes of an instruction share a bank
    // beyond the two that must, 4.6 with sixteen copies and Gaussian weights, 0.5 on one address.)
    constexpr uint32_t COPIES = 32, STRIDE = 257;
    __shared__ uint32_t s_h[COPIES * STRIDE];
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < COPIES * STRIDE; i += HIST_THREADS) s_h[i] = 0;
    __syncthreads();
    uint32_t *mine = s_h + (tid & (COPIES - 1u)) * STRIDE;
    constexpr uint32_t PER_VEC = DT == DT_FP32 ? 4u : 8u;        // elements in 16 bytes
    const uint64_t nvec = n_elems / PER_VEC;
    const uint64_t stride = (uint64_t)wgs * HIST_THREADS;
    // the LDS counters cannot overflow: the workgroups are shared out over the launch's tensors by size, a tensor gets at least
    // half of its exact share of HIST_WORKGROUPS (rounded down, but not below one), so a workgroup counts at most twice the
    // launch's sixteen times 2^34 elements / 256 = 2^31
    // the sample: chunks of SAMPLE_CHUNK elements whose number is a multiple of `every`
    constexpr uint32_t LOG_VPC = DT == DT_FP32 ? 10u : 9u;      // 16-byte vectors in a chunk
    const uint64_t chunks = (nvec + (1u << LOG_VPC) - 1u) >> LOG_VPC;
    const uint64_t picked = ((chunks + every - 1u) / every) << LOG_VPC;
    auto count = [&](const uint4 q) {
        const uint32_t d[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (DT == DT_FP32) {
                atomicAdd(&mine[(d[i] >> 23) & 0xFFu], 1u);
            } else if constexpr (DT == DT_FP16) {
                atomicAdd(&mine[(d[i] >> 10) & 0x1Fu], 1u);
                atomicAdd(&mine[(d[i] >> 26) & 0x1Fu], 1u);
            } else {
                atomicAdd(&mine[(d[i] >> 7) & 0xFFu], 1u);
                atomicAdd(&mine[(d[i] >> 23) & 0xFFu], 1u);
            }
        }
    };
    auto vec_of = [&](uint64_t sv) { return (((sv >> LOG_VPC) * every) << LOG_VPC) + (sv & ((1u << LOG_VPC) - 1u)); };
    constexpr int Q = 4;                                 // vectors of a thread that travel together
    uint4 q[Q];
    bool ok[Q];
    auto ask = [&](uint64_t sv) {
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const uint64_t v = vec_of(sv + u * stride);
            ok[u] = sv + u * stride < picked && v < nvec;
            if (ok[u]) q[u] = ld_stream(reinterpret_cast<const uint4 *>(in_) + v);
        }
    };
    uint64_t sv = (uint64_t)wg * HIST_THREADS + tid;
    ask(sv);
    while (__builtin_amdgcn_ballot_w64(ok[0])) {
        uint4 now[Q];
        bool has[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) { now[u] = q[u]; has[u] = ok[u]; }
        sv += Q * stride;
        ask(sv);
#pragma unroll
        for (int u = 0; u < Q; ++u)
            if (has[u]) count(now[u]);
    }
    if (wg == 0 && tid < (uint32_t)(n_elems % PER_VEC) && ((nvec * PER_VEC) / SAMPLE_CHUNK) % every == 0) {
        const uint64_t e = nvec * PER_VEC + tid;
        uint32_t x;
        if constexpr (DT == DT_FP32) x = (reinterpret_cast<const uint32_t *>(in_)[e] >> 23) & 0xFFu;
        else if constexpr (DT == DT_FP16) x = (reinterpret_cast<const uint16_t *>(in_)[e] >> 10) & 0x1Fu;
        else x = (reinterpret_cast<const uint16_t *>(in_)[e] >> 7) & 0xFFu;
        atomicAdd(&mine[x], 1u);
    }
    __syncthreads();
    uint32_t c = 0;
    if (tid < 256u) {
#pragma unroll
        for (uint32_t i = 0; i < COPIES; ++i) c += s_h[i * STRIDE + tid];
    }
    if (c) atomicAdd(&hist[tid], (unsigned long long)c);
    // What passes from one workgroup to another is an atomic of the device's scope, which no cache keeps back, so waiting for this
    // wave's own accesses is enough; a release would write the L2 back, 40 us of a layer's 86.
    wait_accesses();
    __syncthreads();
    if (tid == 0) s_h[0] = __hip_atomic_fetch_add(p.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_h[0] != p.wgs - 1u) return;
    // (all counts of a thread travel together.  The host reads when the kernel has ended, so nothing here waits for anything else.)
    constexpr uint32_t R = MAX_BATCH * 256u / 2u / HIST_THREADS;
    unsigned long long lo[R], hi[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = 2u * (r * HIST_THREADS + tid);
        if (i >= p.n_counts) break;
        lo[r] = __hip_atomic_load(p.counts + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hi[r] = __hip_atomic_load(p.counts + i + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = 2u * (r * HIST_THREADS + tid);
        if (i >= p.n_counts) break;
        *reinterpret_cast<uint4 *>(p.host + i) = make_uint4((uint32_t)lo[r], (uint32_t)(lo[r] >> 32), (uint32_t)hi[r], (uint32_t)(hi[r] >> 32));
        *reinterpret_cast<uint4 *>(p.counts + i) = make_uint4(0, 0, 0, 0);
    }
    if (tid == 0) {
        *p.done = 0;
        *p.arrived = 1;
    }
}

}  // namespace enec
