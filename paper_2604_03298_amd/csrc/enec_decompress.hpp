// Decompression: offset lookup, mask prefix, unpack, inverse transform, recombine (Sec. V-A decompression
// path; Alg. 1 decompression part), for streams with one tuple and with one tuple per data block.
//
// Bound: HBM.  One workgroup per data block, as many as the grid needs, none of them persistent: blocks are
// independent, and a workgroup that starts when another ends keeps the accesses of the device in stream
// order.  A kernel that only moves the bytes of a block (24.8 KB in, 32 KB out) reaches 5.9 TB/s that way
// and 5.75 with a persistent grid and the next block prefetched, which this kernel replaced.  What a
// block waits for (table entry, then its payload) is hidden by the other workgroups of the CU.  For the 16-bit
// formats these are the workgroups of 65536 elements, four at the default block size: the registers and the LDS
// would let twice as many, but then more of the device's accesses are in flight than its memory likes (405 MB
// layer: 124.7 us with eight, 123.2 with five, 120.0 with four, 121.2 with three; 470 MB matrices 273.8, 270.1,
// 271.9, 268.5).  The host holds the rest back with LDS that nobody uses (decompress_lds_floor), because a limit
// on the waves per SIMD would count the idle lanes of blocks of 2048 elements, half of each wave, as well: with
// four waves per SIMD 537 MB in such blocks take 174 us instead of 153, 268 MB with one tuple per block 87 instead
// of 78 (83 with the kernel that came before).
//
// The widths (m, n) are run-time values, uniform over the workgroup: the unpackers are reached through a
// switch over eight low-plane widths and eight record widths.  So the streams of a call that differ only in
// their tuples share a launch (sixteen vectors of 100001 elements with tuples of their own: 7 instead of 16 us).
// A launch has the threads and the LDS of its largest block size; the blocks of streams with smaller ones join it as
// long as they are few (enec_decompress_batch), for each takes the place of a large one while it runs.  So the norm
// vectors of a decoder layer, whose default block size is their length, need no launch of 4 us of their own.
//
// The decoded elements leave as streaming stores, whatever their number.  Alone that is faster at every size; a reader
// right behind finds less of them in the caches.  Decode and reader together, streaming / plain stores / the kernel
// before (us, caches full of other data): 34 MB and a copy 36.6 / 29.5 / 33.9, and a product with 16 rows
// 35.6 / 37.1 / 41.6; 90 MB and a copy 84.5 / 64.6 / 77.2, 16 rows 87.1 / 84.3 / 98.2, 256 rows 103.8 / 94.8 / 105.8;
// 470 MB and a copy 336 / 339 / 361, 16 rows 283 / 261 / 287, 256 rows 501 / 505 / 519.
#pragma once
#include "enec_kernels.hpp"

namespace enec {

// d3: plane values of the thread's 8 rows from the stream's low plane (already joined pairwise by
// Alg. 2's last step: stream byte 2i = normalized byte i, 2i+1 = normalized byte i + T/2)
template <int LM>
__device__ __forceinline__ void unpack_low(const uint8_t *img_low, uint32_t B, uint32_t logC, uint32_t tid,
                                           uint32_t (&LOW)[8][2])
{
    constexpr HHTable TL = HH<LM>::table;
    uint32_t Pl[LM][2];
    const uint32_t T2 = (LM * B) >> 4;
#pragma unroll
    for (int q = 0; q < LM; ++q) {
        const uint32_t i = ((uint32_t)q << logC) + 8u * tid;
        const bool even = i < T2;
        const uint4 sp = *reinterpret_cast<const uint4 *>(img_low + 2u * (even ? i : i - T2));
        const uint32_t sel = even ? 0x06040200u : 0x07050301u;
        Pl[q][0] = byte_perm(sp.y, sp.x, sel);
        Pl[q][1] = byte_perm(sp.w, sp.z, sel);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) LOW[t][0] = LOW[t][1] = 0;
#pragma unroll
    for (int f = 0; f < TL.count; ++f) {
        const uint32_t smask = (TL.shift[f] >= 0 ? (TL.dmask[f] >> TL.shift[f]) : (TL.dmask[f] << (-TL.shift[f]))) * 0x01010101u;
#pragma unroll
        for (int h = 0; h < 2; ++h) LOW[TL.row[f]][h] |= shl_or_shr(Pl[TL.plane[f]][h], -TL.shift[f]) & smask;
    }
}

template <int A, int LPG>
__device__ __forceinline__ void unpack_records(const uint8_t *img_high, uint32_t my_word, uint32_t my_excl,
                                               uint32_t logC, uint32_t tid, uint32_t (&HI)[8][2])
{
#pragma unroll
    for (int t = 0; t < 8; ++t) unpack_record_row<A, LPG>(img_high, my_word, my_excl, logC, tid, t, HI[t][0], HI[t][1]);
}

// Between LDS accesses of different lanes of one wave.  The wave barrier alone accesses no memory, so it would let the
// optimiser move a lane's accesses across it wherever it can prove that this lane's own addresses differ; the
// wavefront-scope fences forbid that and cost no instruction.
__device__ __forceinline__ void exchange_in_wave()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Zero, known when all fields of the item are: has them loaded together.  Left to itself the compiler asks for each where it
// is used, and the first workgroups of a launch, whose arguments are in no cache yet, wait for memory three times before they
// know where their stream is.  us, each where it is used / together: one matrix of 4e6 elements 6.09 / 5.99, 45e6 in fp32 58.9 /
// 57.1, sixteen streams of 4e6 40.4 / 39.9.
__device__ __forceinline__ uint32_t loaded(const DecompressItem &it)
{
    uint32_t zero, zero2;
    asm("s_mov_b32 %0, 0" : "=s"(zero) : "s"(it.in), "s"(it.out), "s"(it.n_elems), "s"(it.tuples_at), "s"(it.tail_base), "s"(it.payload_base),
        "s"(it.payload_bytes), "s"(it.status), "s"(it.tuple_stride), "s"(it.logB));
    asm("s_mov_b32 %0, 0" : "=s"(zero2) : "s"(it.hdr[0]), "s"(it.hdr[1]), "s"(it.hdr[2]), "s"(it.hdr[3]), "s"(it.hdr[4]), "s"(it.hdr[5]),
        "s"(it.hdr[6]), "s"(it.hdr[7]), "s"(it.hdr[8]), "s"(it.hdr[9]), "s"(it.hdr[10]));
    return zero | zero2;
}

// fp32: three waves per SIMD, whose blocks are 115 KB of traffic and need the registers (45e6 elements: 66.8 us with
// four, four registers spilled; 61.1 with three; 66.6 with two); the 16-bit formats: at least what their LDS allows
#define DEC_WAVES_MIN (DT == DT_FP32 ? 3 : 4)
#define DEC_WAVES_MAX (DT == DT_FP32 ? 3 : 8)

// MIXED: the streams' block sizes differ.  (In the instances for one block size it stays an argument: looked up with the
// stream, it cost fp32 1 to 2 % and the 16-bit formats the eighth wave per SIMD, 12 % in blocks of 2048.)
// ONE: the launch has one stream, so a block need not look for its own, nor wait for fields that only launches of several need
// (us, without / with: 4e6 elements 5.98 / 5.81, 45e6 in fp32 58.4 / 58.1, 67e6 in blocks of 4096 40.3 / 40.2).
template <int DT, int LPG, bool MIXED, bool ONE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(DEC_WAVES_MIN, DEC_WAVES_MAX))) decompress_kernel(const DecompressArgs p)
{
    constexpr uint32_t E = exponent_bits(DT);
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    extern __shared__ __align__(16) uint8_t smem[];      // the packed part as it is in the stream
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    // the stream this block belongs to (the blocks of the launch's streams are numbered through; `first` of
    // the entries that are not used is beyond every block)
    DecompressItem it = p.item[0];
    uint32_t zero, ti = 0, first = 0;
    if constexpr (ONE) {
        zero = loaded(it);
    } else {
        // The next streams' fields are on their way by then: two words bring the next 256 bytes.  (Without them a launch of two
        // streams waits for the first one's fields and then as long again for the second's: 128 blocks of two streams 5.50 us against
        // 5.39 where no field is loaded early, 5.29 like this.  Bringing all sixteen streams' costs every launch 4 to 6 %.  Finding
        // the stream before any field is asked for makes seven streams of 1e6 elements 1 to 2 % faster, sixteen of 4e6 1.4 % slower.)
        uint32_t next;
        asm("s_mov_b32 %0, 0" : "=s"(next) : "s"(p.item[1].status), "s"(p.item[2].tuple_stride));
        zero = loaded(it) | next;
#pragma unroll
        for (int i = 1; i < MAX_BATCH; ++i)
            if (blockIdx.x + zero >= p.first[i]) { ti = i; first = p.first[i]; }
        if (ti != 0) {
            it = p.item[ti];
            zero = loaded(it);
        }
    }
    const uint32_t k = blockIdx.x - first + zero;
    const uint32_t logB = MIXED ? it.logB : p.logB, B = MIXED ? 1u << logB : p.B, logC = logB - 3u;
    const uint32_t nact = B >> 6, threads = MIXED ? blockDim.x : nact < 64u ? 64u : nact;     // those that unpack / that load
    const bool active = tid < nact;
    const uint32_t mask_bytes = (B >> 6) >> LOG_LPG;                  // B / (8 L)

    // d1: header as configured, tuple (in the tuple table, or in the header), offsets
    const uint32_t *hd = reinterpret_cast<const uint32_t *>(it.in);
    const uint64_t *table = reinterpret_cast<const uint64_t *>(it.in + 64);
    const uint64_t t0 = table[k], t1 = table[k + 1];
    const uint32_t tup = *reinterpret_cast<const uint32_t *>(it.in + it.tuples_at + (uint64_t)it.tuple_stride * k);
    uint32_t differ = (hd[10] ^ it.hdr[10]) & (0u - (it.tuple_stride >> 2));     // byte 40 ff.: only with a tuple table
#pragma unroll
    for (int i = 0; i < 10; ++i) differ |= hd[i] ^ it.hdr[i];
    const uint32_t b = tup & 0xFFu, n = (tup >> 8) & 0xFFu, m = (tup >> 16) & 0xFFu;
    // a block that is skipped (damaged header, tuple or table entry) leaves its part of the output
    // untouched: the caller is told through the status word
    const uint32_t a = n - m, lm = m + (DT == DT_FP16 ? 3u : 0u);
    const uint32_t fixed = B + mask_bytes + ((lm * B) >> 3);
    const uint64_t sz = t1 - t0;
    const uint64_t room = it.payload_bytes - t0;
    if ((differ != 0) | (n < 1u) | (n > E) | (m > n) | (b >= (1u << E)) |
        (sz < fixed) | (sz > fixed + (uint32_t)LPG * a * ((B >> 3) >> LOG_LPG) + 15u) | (((sz | t0) & 15u) != 0) |
        (t0 > it.payload_bytes) | (sz > room)) {
        if (tid == 0 && it.status) *it.status = 7u;
        return;
    }

    // Everything the block needs is requested at once.  The packed part (mask | low plane | high records)
    // goes from memory to LDS without passing through registers, 16 bytes per lane to the wave's base + 16
    // lane; the sizes are whole 16-byte vectors.
    const uint8_t *src = it.in + it.payload_base + t0;
    const uint32_t nvec = ((uint32_t)sz - B) >> 4;
    for (uint32_t v0 = __builtin_amdgcn_readfirstlane(tid & ~63u); v0 < nvec; v0 += threads)
        if (v0 + lane < nvec) load_to_lds(src + B + 16u * (v0 + lane), smem + 16u * v0);
    uint2 smv[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
        smv[t] = active ? ld_stream(reinterpret_cast<const uint2 *>(src + ((size_t)t << logC) + 8u * tid)) : make_uint2(0, 0);
    // fp32: lower halves, straight from the stream (region padded to 16 bytes).  A wave's 512 elements of a row
    // are 2 KB of output.  Stored by the threads that unpack them, 2 x 16 bytes per lane, every streaming store
    // would write half of each 128-byte line it touches, which a plain copy shows at 3.4 instead of 6.0 TB/s.  So
    // the upper halves change lanes through LDS, and lane i stores elements 4 i .. 4 i + 3 of the first, then of
    // the second 256 elements; it loads the lower halves of those.
    const uint64_t blk0 = (uint64_t)k << logB;
    uint2 tl[DT == DT_FP32 ? 16 : 1];
    const uint32_t col4 = 8u * (tid & ~63u) + 4u * lane;                  // its column in the first of the two
    if constexpr (DT == DT_FP32) {
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const uint32_t c = col4 + 256u * (t & 1);
            const uint64_t e = blk0 + ((uint64_t)(t >> 1) << logC) + c;
            tl[t] = c < (1u << logC) && e < it.n_elems ? ld_stream(reinterpret_cast<const uint2 *>(it.in + it.tail_base + 2u * e))
                                                       : make_uint2(0, 0);
        }
    }
    wait_accesses();
    __syncthreads();
    // (a wave of fp32 stays whole, its lanes exchange what they have)
    if (DT == DT_FP32 ? MIXED && (tid & ~63u) >= nact : !active) return;

    // d2: mask words and their exclusive popcount prefix (a wave scan per wave)
    const uint8_t *img_low = smem + mask_bytes;
    const uint8_t *img_high = img_low + ((lm * B) >> 3);
    const uint32_t nwords = (B >> 8) >> LOG_LPG;
    const uint32_t my_word = lane < nwords ? reinterpret_cast<const uint32_t *>(smem)[lane] : 0u;
    const uint32_t my_pc = __popc(my_word);
    const uint32_t my_excl = wave_incl_scan(my_pc, lane) - my_pc;

    // d3: low-plane values and high bits of the thread's 8 x 8 elements
    uint32_t LOW[8][2], HI[8][2];
    switch (lm) {
    case 1: unpack_low<1>(img_low, B, logC, tid, LOW); break;
    case 2: unpack_low<2>(img_low, B, logC, tid, LOW); break;
    case 3: unpack_low<3>(img_low, B, logC, tid, LOW); break;
    case 4: unpack_low<4>(img_low, B, logC, tid, LOW); break;
    case 5: unpack_low<5>(img_low, B, logC, tid, LOW); break;
    case 6: unpack_low<6>(img_low, B, logC, tid, LOW); break;
    case 7: unpack_low<7>(img_low, B, logC, tid, LOW); break;
    case 8: unpack_low<8>(img_low, B, logC, tid, LOW); break;
    default:
#pragma unroll
        for (int t = 0; t < 8; ++t) LOW[t][0] = LOW[t][1] = 0;
        break;
    }
    switch (a) {
    case 1: unpack_records<1, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 2: unpack_records<2, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 3: unpack_records<3, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 4: unpack_records<4, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 5: unpack_records<5, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 6: unpack_records<6, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 7: unpack_records<7, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    case 8: unpack_records<8, LPG>(img_high, my_word, my_excl, logC, tid, HI); break;
    default:
#pragma unroll
        for (int t = 0; t < 8; ++t) HI[t][0] = HI[t][1] = 0;
        break;
    }

    const uint32_t crep = ((b + (1u << (n - 1))) & 0xFFu) * 0x01010101u;
    const uint32_t srep = (1u << (n - 1)) * 0x01010101u;
    const uint32_t lrep = ((1u << m) - 1u) * 0x01010101u;
    const uint32_t erep = ((1u << E) - 1u) * 0x01010101u;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint64_t e0 = blk0 + ((uint64_t)t << logC) + 8u * tid;
        uint32_t o[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t Y = (LOW[t][h] & lrep) | (HI[t][h] << m);
            // d4: x = b - sext_n(y) = (b + 2^(n-1)) - (y ^ 2^(n-1)), modulo the exponent field
            const uint32_t Xv = bytesub_safe(crep, Y ^ srep) & erep;
            const uint32_t sm = h ? smv[t].y : smv[t].x;
            uint32_t Hi, Lo;
            if constexpr (DT == DT_FP16) {
                const uint32_t T3 = (LOW[t][h] >> m) & 0x07070707u;
                Hi = (sm & 0x80808080u) | (Xv << 2) | ((sm >> 5) & 0x03030303u);
                Lo = ((sm & 0x1F1F1F1Fu) << 3) | T3;
            } else {
                Hi = bfi(0x7F7F7F7Fu, Xv >> 1, sm);
                Lo = bfi(0x7F7F7F7Fu, sm, Xv << 7);
            }
            o[2 * h] = byte_perm(Hi, Lo, 0x05010400u);
            o[2 * h + 1] = byte_perm(Hi, Lo, 0x07030602u);
        }
        if constexpr (DT == DT_FP32) {
            // the wave's 1 KB of upper halves in element order (a wave's LDS accesses are executed in order, the
            // kilobyte is its own; exchange_in_wave keeps the compiler to that order)
            uint8_t *turn = smem + p.turn_at + 16u * (tid & ~63u);
            *reinterpret_cast<uint4 *>(turn + 16u * lane) = make_uint4(o[0], o[1], o[2], o[3]);
            exchange_in_wave();
            uint32_t *out32 = reinterpret_cast<uint32_t *>(it.out);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint2 up = *reinterpret_cast<const uint2 *>(turn + 512u * i + 8u * lane), lo = tl[2 * t + i];
                const uint32_t c = col4 + 256u * i;
                const uint64_t e = blk0 + ((uint64_t)t << logC) + c;
                // element = lower half | bf16 word << 16
                const uint32_t w[4] = {byte_perm(up.x, lo.x, 0x05040100u), byte_perm(up.x, lo.x, 0x07060302u),
                                       byte_perm(up.y, lo.y, 0x05040100u), byte_perm(up.y, lo.y, 0x07060302u)};
                if (c < (1u << logC)) {
                    if (e + 4 <= it.n_elems) {
                        st_stream(reinterpret_cast<uint4 *>(out32 + e), make_uint4(w[0], w[1], w[2], w[3]));
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (e + j < it.n_elems) out32[e + j] = w[j];
                    }
                }
            }
            exchange_in_wave();                  // the next row is written over what other lanes have read
        } else {
            uint16_t *out16 = reinterpret_cast<uint16_t *>(it.out);
            if (e0 + 8 <= it.n_elems) {
                st_stream(reinterpret_cast<uint4 *>(out16 + e0), make_uint4(o[0], o[1], o[2], o[3]));
            } else if (e0 < it.n_elems) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (e0 + i < it.n_elems) out16[e0 + i] = (uint16_t)(o[i >> 1] >> (16 * (i & 1)));
            }
        }
    }
}

}  // namespace enec
