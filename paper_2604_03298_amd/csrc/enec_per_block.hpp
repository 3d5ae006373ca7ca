// ENEC streams with one (b, n, m) per data block: the search of Sec. V-E (Eq. 1-4) runs inside the
// compress kernel on the exponents of each block's own elements, so a tensor whose blocks differ
// (zeros, constants, weights of several scales, noise) is coded block by block with the tuple
// that fits.  Compression only: enec_decompress.hpp reads these streams like any other.  One pass over the tensor:
//   ticket -> rows -> split -> LDS histogram -> (b, n) by Eq. 1-3 -> m by Eq. 4 -> transform ->
//   group test -> size (published) -> packing (Alg. 2, widths chosen at run time from the template
//   instances) -> sum of the earlier blocks' sizes -> stores.
// The widths are run-time values here, so the packers are reached through a switch; the kernel
// of enec_device.hpp, which knows its widths at compile time, stays the fast path for one tuple
// per tensor.
// Two kernels: compress_per_block_stream_kernel for the default block size (persistent grid, stores deferred by a block)
// and compress_per_block_kernel for the others (one workgroup per block, which places its block at once).
#pragma once
#include "enec_kernels.hpp"

namespace enec {

// look-back word of a block: zero = nothing yet
constexpr uint64_t PB_PREFIX = 1ull << 63;     // [60:0] = end of this block's payload (inclusive prefix), / 16
constexpr uint64_t PB_SIZE = 1ull << 62;       // [60:0] = size of this block's payload, / 16
constexpr uint64_t PB_GAVE_UP = 1ull << 61;    // somebody before (or this block) stopped waiting
constexpr uint64_t PB_VALUE = (1ull << 61) - 1;
constexpr int PB_WINDOW = 256;                  // blocks one look-back step covers (4 words per lane)

// Eq. 1: bits needed for the window [l, h] around b, capped by the exponent field
__device__ __forceinline__ uint32_t pb_width_for(uint32_t b, uint32_t l, uint32_t h, uint32_t E)
{
    const uint32_t pos = 32u - __clz(b - l);                          // bit length, 0 for 0
    const uint32_t neg = h > b ? 32u - __clz(h - b - 1u) : 0u;
    const uint32_t w = (pos > neg ? pos : neg) + 1u;
    return w < E ? w : E;
}

// a1: the 8 rows of data block k as 128-bit vectors (a thread's 8 elements of a row are one vector,
// two for fp32); elements beyond the tensor's end read as zero words
template <int DT>
__device__ __forceinline__ void pb_load_rows(const void *src, uint64_t n_elems, uint32_t B, uint32_t logB, uint32_t k, uint32_t tid, bool active,
                                             uint32_t logC, uint4 (&raw)[DT == DT_FP32 ? 16 : 8])
{
    const uint64_t blk0 = (uint64_t)k << logB;
    const uint32_t real = n_elems - blk0 < B ? (uint32_t)(n_elems - blk0) : B;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint32_t at = ((uint32_t)t << logC) + 8u * tid;         // first element of the thread in this row
        if constexpr (DT == DT_FP32) {
            uint4 u = make_uint4(0, 0, 0, 0), v = make_uint4(0, 0, 0, 0);
            if (active && at < real) {
                const uint32_t *in = reinterpret_cast<const uint32_t *>(src) + blk0 + at;
                if (at + 8u <= real) {
                    u = *reinterpret_cast<const uint4 *>(in);               // plain: see load_block_rows
                    v = *reinterpret_cast<const uint4 *>(in + 4);
                } else {
                    uint32_t d[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (at + i < real) d[i] = in[i];
                    u = make_uint4(d[0], d[1], d[2], d[3]);
                    v = make_uint4(d[4], d[5], d[6], d[7]);
                }
            }
            raw[2 * t] = u;
            raw[2 * t + 1] = v;
        } else {
            uint4 r = make_uint4(0, 0, 0, 0);
            if (active && at < real) {
                const uint16_t *in = reinterpret_cast<const uint16_t *>(src) + blk0 + at;
                if (at + 8u <= real) {
                    r = ld_stream(reinterpret_cast<const uint4 *>(in));
                } else {
                    uint32_t d[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (at + i < real) d[i >> 1] |= (uint32_t)in[i] << (16 * (i & 1));
                    r = make_uint4(d[0], d[1], d[2], d[3]);
                }
            }
            raw[t] = r;
        }
    }
}

// Alg. 2 over the low plane of the thread's 8 rows, taken straight from the transformed bytes Y (bits
// below m; fp16 adds the three left-over mantissa bits kept in bits 5..7 of Y's bytes): the plane
// value of a row exists only while that row is folded into the normalized bytes
template <int LM, int DT>
__device__ __forceinline__ void pb_pack_low_from_y(const uint32_t (&Y)[8][2], uint32_t lrep, uint32_t m,
                                                   uint8_t *img_low, uint32_t logC, uint32_t tid)
{
    constexpr HHTable TL = HH<LM>::table;
    uint32_t acc[LM][2];
#pragma unroll
    for (int q = 0; q < LM; ++q) acc[q][0] = acc[q][1] = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t low = Y[t][h] & lrep;
            if constexpr (DT == DT_FP16) low |= ((Y[t][h] >> 5) & 0x07070707u) << m;
#pragma unroll
            for (int f = 0; f < TL.count; ++f)
                if (TL.row[f] == t) {
                    uint32_t s = shl_or_shr(low, TL.shift[f]);
                    if (!TL.clean[f]) s &= TL.dmask[f] * 0x01010101u;
                    acc[TL.plane[f]][h] |= s;
                }
        }
#pragma unroll
    for (int q = 0; q < LM; ++q)
        *reinterpret_cast<uint2 *>(img_low + ((size_t)q << logC) + 8u * tid) = make_uint2(acc[q][0], acc[q][1]);
}

template <int A, int LPG>
__device__ __forceinline__ void pb_pack_records_from_y(const uint32_t (&Y)[8][2], uint32_t m, uint32_t arep,
                                                       uint32_t my_word, uint32_t my_excl, uint8_t *img_high,
                                                       uint32_t logC, uint32_t tid, bool active)
{
    uint32_t HI[8][2];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        HI[t][0] = (Y[t][0] >> m) & arep;
        HI[t][1] = (Y[t][1] >> m) & arep;
    }
    pack_records<A, LPG>(HI, my_word, my_excl, img_high, logC, tid, active);
}

// minimum over the 64 lanes, in every lane
__device__ __forceinline__ uint32_t wave_min32(uint32_t v)
{
    auto mn = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x111 /* row_shr:1 */, 0xF, 0xF, false));
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x112 /* row_shr:2 */, 0xF, 0xF, false));
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x114 /* row_shr:4 */, 0xF, 0xF, false));
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x118 /* row_shr:8 */, 0xF, 0xF, false));
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142 /* row_bcast:15 */, 0xA, 0xF, false));
    v = mn(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143 /* row_bcast:31 */, 0xC, 0xF, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Phases 2 and 3 of Sec. V-E for one block, from the counts of its exponents (s_hist) and the values that occur
// (s_present): s_best = n << 8 | b, s_m = m, visible to all waves on return.  s_best must be all ones before.
template <int DT, int LPG>
__device__ __forceinline__ void pb_search(const uint32_t *s_hist, const unsigned long long *s_present, unsigned long long &s_best, uint32_t &s_m,
                                          uint32_t real)
{
    constexpr uint32_t E = exponent_bits(DT);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t xl = 255u, xh = 0u;
#pragma unroll
    for (int c = 3; c >= 0; --c) {
        const uint64_t z = s_present[c];
        if (z) xl = 64u * c + (uint32_t)__builtin_ctzll(z);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint64_t z = s_present[c];
        if (z) xh = 64u * c + 63u - (uint32_t)__builtin_clzll(z);
    }
    xl = __builtin_amdgcn_readfirstlane(xl);
    xh = __builtin_amdgcn_readfirstlane(xh);
    // Eq. 4 for every m (lane m holds the count of elements whose y fits m bits) with the group length
    // the block is coded with, 1/L + n + (m - n) p^L, in IEEE double, p^L by three to five squarings;
    // the smallest value wins, ties go to the smaller m (one wave)
    auto choose_m = [&](uint32_t cnt, uint32_t n) -> uint32_t {
        // (a whole block has a power of two of elements, which needs no division)
        const double q = (real & (real - 1u)) == 0 ? __builtin_ldexp((double)cnt, -(int)__builtin_ctz(real)) : (double)cnt / (double)real;
        const double q2 = q * q, q4 = q2 * q2;
        double qL = q4 * q4;                                   // p^8
        if constexpr (LPG >= 2) qL = qL * qL;                  // p^16
        if constexpr (LPG == 4) qL = qL * qL;                  // p^32
        double least = (1.0 / (double)(8 * LPG) + (double)n) + ((double)lane - (double)n) * qL;
        if (lane > n) least = __builtin_inf();
        uint32_t at = lane;
        // the first minimum of lanes 0 .. 15 travels to lane 15; of two equal ones the lower lane's stays
        auto fold = [&](auto ctrl) {
            constexpr int C = decltype(ctrl)::value;
            const unsigned long long bits = (unsigned long long)__double_as_longlong(least);
            const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)bits, (int)bits, C, 0xF, 0xF, false);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(bits >> 32), (int)(bits >> 32), C, 0xF, 0xF, false);
            const uint32_t from = (uint32_t)__builtin_amdgcn_update_dpp((int)at, (int)at, C, 0xF, 0xF, false);
            const double other = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
            if (other <= least) { least = other; at = from; }
        };
        fold(std::integral_constant<int, 0x111 /* row_shr:1 */>{});
        fold(std::integral_constant<int, 0x112 /* row_shr:2 */>{});
        fold(std::integral_constant<int, 0x114 /* row_shr:4 */>{});
        fold(std::integral_constant<int, 0x118 /* row_shr:8 */>{});
        return (uint32_t)__builtin_amdgcn_readlane((int)at, 15);
    };
    if (xh - xl < 64u) {
        // The usual case, at most 64 values between the lowest and the highest: wave 0 does the whole
        // search in registers.  Lane j holds the count of value xl + j and is candidate b = xl + j.
        if (wave == 0) {
            const uint32_t R = xh - xl + 1u;
            const bool valid = lane < R;
            const uint32_t v = valid ? s_hist[xl + lane] : 0u;
            // every b with Eq. 1's n and Eq. 3's cost; ties: smaller n, then smaller b
            const uint32_t nb_ = pb_width_for(xl + lane, xl, xh, E);
            // Eq. 1's n makes 2^n exceed every distance inside the window, so with P_j = the counts of values xl .. xl + j
            //   D_j = sum_i v_i ((j - i) mod 2^n) = j N - sum_i i v_i + 2^n (N - P_j):
            // a prefix sum and a sum in place of a pass over the values (23 bits, exact as before).
            const uint32_t P = wave_incl_scan(v, lane);
            const uint32_t D = lane * real + ((real - P) << nb_) - wave_sum32(lane * v);
            const uint32_t Dmin = wave_min32(valid ? D : 0xFFFFFFFFu);
            const uint32_t pick = wave_min32(valid && D == Dmin ? (nb_ << 8) | (xl + lane) : 0xFFFFFFFFu);
            const uint32_t b = pick & 0xFFu, n = pick >> 8;
            // phase 3: lane m counts the elements whose y fits m bits: those down to 2^m - 1 below b, and above b those
            // from 2^n - 2^m + 1 on (there y = 2^n - (x - b))
            const uint32_t pos = b - xl, p2 = 1u << (lane < n ? lane : n);
            const uint32_t below = (uint32_t)__shfl((int)P, (int)(pos - p2), 64);
            const uint32_t top = pos + (1u << n) - p2;
            const uint32_t above = (uint32_t)__shfl((int)P, (int)(top < 63u ? top : 63u), 64);
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)P, (int)pos) - (pos >= p2 ? below : 0u) + (real - above);
            const uint32_t best_m = choose_m(cnt, n);
            if (lane == 0) {
                s_best = ((unsigned long long)n << 8) | b;
                s_m = best_m;
            }
        }
        __syncthreads();
    } else {
        // A block whose exponents spread over more than 64 values.  Lane j of a wave holds the counts of
        // the values j, 64 + j, 128 + j and 192 + j; wave w takes the candidates b = xl + 64 w + j (and
        // further ones if the workgroup has fewer than four waves); the waves' best meet in s_best.
        // Eq. 1 gives n = 7 or 8 for every b of such a block (the wider side of the window has at least
        // 32 values).  With n fixed, Eq. 3's cost D_n(b) = sum_x count[x] ((b - x) mod 2^n) obeys
        //   D_n(b + 1) - D_n(b) = N - 2^n H_n[(b + 1) mod 2^n],   H_n = the counts folded modulo 2^n,
        // (every term grows by one, the ones that wrap fall by 2^n - 1), so the 64 costs of a wave come
        // from D_n of its first candidate, a sum over the lanes, and a prefix sum of H_n over the lanes.
        uint32_t hv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) hv[c] = s_hist[64 * c + lane];
        for (uint32_t b0 = xl + 64u * wave; b0 <= xh; b0 += blockDim.x) {
            const uint32_t bb = b0 + lane;
            const bool valid = bb <= xh;
            const uint32_t nb_ = pb_width_for(bb, xl, xh, E);
            const uint32_t h0 = s_hist[bb & 255u], h1 = s_hist[(bb + 128u) & 255u];
            uint32_t D = 0xFFFFFFFFu;                         // costs are at most 2^15 elements * 255
#pragma unroll
            for (uint32_t nn = 7; nn <= 8; ++nn) {
                const uint32_t mask = (1u << nn) - 1u;
                uint32_t t = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) t += __umul24(hv[c], (b0 - (64u * c + lane)) & mask);
                const uint32_t first = wave_sum32(t);                       // D_nn(b0)
                const uint32_t g = nn == 8 ? h0 : h0 + h1;                  // H_nn[b mod 2^nn]
                const uint32_t upto = wave_incl_scan(g, lane) - (uint32_t)__builtin_amdgcn_readlane((int)g, 0);
                if (nb_ == nn) D = first + lane * real - (upto << nn);
            }
            const uint32_t Dmin = wave_min32(valid ? D : 0xFFFFFFFFu);
            const uint32_t pick = wave_min32(valid && D == Dmin ? (nb_ << 8) | bb : 0xFFFFFFFFu);
            if (lane == 0) atomicMin(&s_best, ((unsigned long long)Dmin << 16) | pick);   // ties: smaller n, then smaller b
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t b = (uint32_t)s_best & 0xFFu, n = ((uint32_t)s_best >> 8) & 0xFFu;
            uint32_t ybits[4];                                     // y < 2^m  <=>  ybits <= m
#pragma unroll
            for (int c = 0; c < 4; ++c) ybits[c] = 32u - (uint32_t)__clz((b - (64u * c + lane)) & ((1u << n) - 1u));
            uint32_t cnt = 0;
            for (uint32_t j = 0; j <= n; ++j) {
                uint32_t t = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) t += ybits[c] <= j ? hv[c] : 0u;
                const uint32_t s = wave_sum32(t);
                if (lane == j) cnt = s;
            }
            const uint32_t best_m = choose_m(cnt, n);
            if (lane == 0) s_m = best_m;
        }
        __syncthreads();
    }
}

// waves per SIMD the compress kernel is built for: six where the instance fits 80 registers without
// spilling (fp16, and bf16 with groups of 16), five elsewhere: a spill here parks raw bytes in scratch
// memory, and they are reloaded when the block is stored, after they have left the L2
#define PB_COMPRESS_WAVES ((DT == DT_FP32 || (DT == DT_BF16 && LPG != 2)) ? 5 : 6)

template <int DT, int LPG>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(PB_COMPRESS_WAVES, PB_COMPRESS_WAVES)))
compress_per_block_kernel(const PbCompressArgs p)
{
    constexpr uint32_t E = exponent_bits(DT);
    constexpr int RW = DT == DT_FP32 ? 16 : 8;
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;

    extern __shared__ __align__(16) uint8_t smem[];      // mask | low plane (normalized bytes) | high records
    __shared__ uint32_t s_hist[256];
    __shared__ unsigned long long s_best;                // Eq. 3 cost << 16 | n << 8 | b of the best candidate
    __shared__ uint32_t s_ticket, s_m, s_flags;
    __shared__ unsigned long long s_present[4];          // exponent values that occur, one bit each
    __shared__ unsigned long long s_off;

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t B = p.B, logC = p.logB - 3u;
    const uint32_t nact = B >> 6;
    const bool active = tid < nact;
    const uint32_t mask_bytes = (B >> 6) >> LOG_LPG;                  // B / (8 L)

    // Blocks are taken in the order in which workgroups start (tickets), not by blockIdx: a block then
    // only waits for blocks that running workgroups hold or that the next workgroups to start will
    // draw, and every workgroup publishes its size before it waits for anything, so the look-back
    // makes progress whatever part of the grid is resident (every wait is bounded by the spin limit
    // as well).  There are PB_TICKET_CLASSES counters: the blocks of a call's launches are numbered
    // through, workgroup w of a launch draws from counter (the launch's first block + w) mod 8, the
    // t-th draw from counter c is block 8 t + c, and every launch has as many workgroups of a class
    // as blocks of it (the counters go on counting from one launch of the call to the next).
    // Returning atomics on one address are serialised at the memory side; with eight addresses the
    // kernel measured 5 % faster than with one.
    const uint32_t cls = (p.first_block + blockIdx.x) & (PB_TICKET_CLASSES - 1u);
    uint32_t ticket = 0;
    if (tid == 0) {
        ticket = atomicAdd(p.ticket + PB_TICKET_STRIDE * cls, 1u);
        s_best = ~0ull;
        s_flags = 0u;
    }
    // Phase 1 counts into PB_HIST_COPIES copies of the histogram (lane i uses copy i mod 16), so that
    // lanes with equal exponents, the normal case, do not queue up on one LDS word; the copies are
    // PB_HIST_STRIDE words apart, which spreads one bin of all copies over the banks.  They share
    // the dynamic LDS with the payload image, which is written only after the search.  They are
    // cleared while the ticket travels.
    uint32_t *hcopy = reinterpret_cast<uint32_t *>(smem);
    for (uint32_t i = tid; i < PB_HIST_COPIES * PB_HIST_STRIDE / 4u; i += blockDim.x)
        reinterpret_cast<uint4 *>(hcopy)[i] = make_uint4(0, 0, 0, 0);
    if (tid == 0) s_ticket = ticket;
    __syncthreads();
    // the tensor this block belongs to (the blocks of the call's tensors are numbered through)
    const uint32_t kg = __builtin_amdgcn_readfirstlane(s_ticket * PB_TICKET_CLASSES + cls);
    if (kg - p.first_block >= p.n_blocks) return;        // (never: a class has as many workgroups as blocks)
    uint32_t ti = 0;
    for (uint32_t i = 1; i < p.n_items; ++i)
        if (kg >= p.item[i].first) ti = i;
    const PbCompressItem &it = p.item[ti];
    const uint32_t k = kg - it.first;
    uint4 raw[RW];
    pb_load_rows<DT>(it.in, it.n_elems, B, p.logB, k, tid, active, logC, raw);
    uint32_t *mine = hcopy + (lane & (PB_HIST_COPIES - 1u)) * PB_HIST_STRIDE;
    const uint64_t blk0 = (uint64_t)k << p.logB;
    const uint32_t real = it.n_elems - blk0 < B ? (uint32_t)(it.n_elems - blk0) : B;   // elements that are not pads
    const bool full = real == B && nact >= 64u;          // no pads and no idle lanes (uniform)

    // ---- a1: rows, split into exponent bytes X and raw bytes SM; fp16's three left-over mantissa bits
    // travel in bits 5..7 of X's bytes (its exponents have five bits) ----
    uint32_t X[8][2], SM[PB_SM_REG_ROWS][2];
    // The raw bytes wait for the block's offset from here to the very end.  Rows PB_SM_REG_ROWS .. 7
    // wait in LDS behind the image (8 bytes per thread and row), the others in registers: with all
    // eight in registers the kernel needs 90 of them, five workgroups fit a CU; with four parked it
    // needs 77 and six fit (LDS: 16.4 KB of image + 8 KB), which measured 5 to 14 % faster.
    uint8_t *sm_park = smem + p.park_at;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint32_t at = ((uint32_t)t << logC) + 8u * tid;         // first element of the thread in this row
        uint4 r16;
        if constexpr (DT == DT_FP32) {
            const uint4 u = raw[2 * t], v = raw[2 * t + 1];
            r16 = make_uint4(byte_perm(u.y, u.x, 0x07060302u), byte_perm(u.w, u.z, 0x07060302u),
                             byte_perm(v.y, v.x, 0x07060302u), byte_perm(v.w, v.z, 0x07060302u));
            // the lower halves leave at once (pads have zero lower halves; the region is padded to 16 bytes)
            if (active && at < real)
                st_stream(reinterpret_cast<uint4 *>(it.out + it.tail_base + 2u * (blk0 + at)),
                          make_uint4(byte_perm(u.y, u.x, 0x05040100u), byte_perm(u.w, u.z, 0x05040100u),
                                     byte_perm(v.y, v.x, 0x05040100u), byte_perm(v.w, v.z, 0x05040100u)));
        } else {
            r16 = raw[t];
        }
        uint32_t sm2[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t d0 = h ? r16.z : r16.x;
            const uint32_t d1 = h ? r16.w : r16.y;
            const uint32_t Lb = byte_perm(d1, d0, 0x06040200u);
            const uint32_t Hb = byte_perm(d1, d0, 0x07050301u);
            uint32_t x;
            if constexpr (DT == DT_FP16) {
                sm2[h] = (Hb & 0x80808080u) | ((Hb & 0x03030303u) << 5) | ((Lb >> 3) & 0x1F1F1F1Fu);
                x = (Hb >> 2) & 0x1F1F1F1Fu;
                X[t][h] = x | ((Lb & 0x07070707u) << 5);
            } else {
                sm2[h] = bfi(0x7F7F7F7Fu, Lb, Hb);
                x = bfi(0xFEFEFEFEu, Hb << 1, Lb >> 7);
                X[t][h] = x;
            }
            // ---- Sec. V-E phase 1: exponent counts of the block's own elements ----
            if (full) {
                if (active) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) atomicAdd(&mine[(x >> (8 * i)) & 0xFFu], 1u);
                }
            } else if (active) {
                const uint32_t e = at + 4u * h;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e + i < real) atomicAdd(&mine[(x >> (8 * i)) & 0xFFu], 1u);
            }
        }
        if (t < PB_SM_REG_ROWS) { SM[t % PB_SM_REG_ROWS][0] = sm2[0]; SM[t % PB_SM_REG_ROWS][1] = sm2[1]; }
        else *reinterpret_cast<uint2 *>(sm_park + (((uint32_t)(t - PB_SM_REG_ROWS) * blockDim.x + tid) << 3)) = make_uint2(sm2[0], sm2[1]);
    }
    __syncthreads();

    // ---- phase 2: the counts of the 256 exponent values, lowest and highest value present ----
    for (uint32_t x = tid; x < 256u; x += blockDim.x) {
        uint32_t c = 0;
#pragma unroll 8
        for (uint32_t i = 0; i < PB_HIST_COPIES; ++i) c += hcopy[i * PB_HIST_STRIDE + x];
        s_hist[x] = c;
        const uint64_t present = __builtin_amdgcn_ballot_w64(c != 0);       // x / 64 is the same for the whole wave
        if (lane == 0) s_present[x >> 6] = present;
    }
    __syncthreads();
    pb_search<DT, LPG>(s_hist, s_present, s_best, s_m, real);
    const uint32_t b = (uint32_t)s_best & 0xFFu, n = ((uint32_t)s_best >> 8) & 0xFFu;
    const uint32_t m = s_m, a = n - m;
    const uint32_t lm = m + (DT == DT_FP16 ? 3u : 0u);

    uint8_t *img = smem;
    uint32_t *img_maskw = reinterpret_cast<uint32_t *>(img);
    uint8_t *img_low = img + mask_bytes;
    uint8_t *img_high = img_low + ((lm * B) >> 3);
    const uint32_t fixed = B + mask_bytes + ((lm * B) >> 3);

    // ---- a2 transform (in place: X becomes y, fp16 keeps its three bits above), a3 group test ----
    const uint32_t crep = ((b + (1u << (n - 1))) & 0xFFu) * 0x01010101u;
    const uint32_t brep = b * 0x01010101u;
    const uint32_t srep = (1u << (n - 1)) * 0x01010101u;
    const uint32_t nrep = ((1u << n) - 1u) * 0x01010101u;
    const uint32_t lrep = ((1u << m) - 1u) * 0x01010101u;
    const uint32_t arep = ((1u << a) - 1u) * 0x01010101u;
    uint64_t flagged[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        uint32_t gor = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t x = X[t][h];
            if constexpr (DT == DT_FP16) x &= 0x1F1F1F1Fu;
            if (!full) {      // pads behave like exponent b: y = 0
                const int32_t left = (int32_t)real - (int32_t)(((uint32_t)t << logC) + 8u * tid + 4u * h);
                const uint32_t padm = !active || left <= 0 ? 0xFFFFFFFFu : (left >= 4 ? 0u : 0xFFFFFFFFu << (8 * left));
                x = bfi(padm, brep, x);
            }
            const uint32_t Y = (bytesub_safe(crep, x) ^ srep) & nrep;
            gor |= (Y >> m) & arep;
            if constexpr (DT == DT_FP16) X[t][h] = Y | (X[t][h] & 0xE0E0E0E0u);
            else X[t][h] = Y;
        }
        // a3: OR over the lanes that share a group, one mask bit per group
        if constexpr (LPG == 2) gor |= swap_pair(gor);
        if constexpr (LPG == 4) gor = quad_or(gor);
        flagged[t] = __builtin_amdgcn_ballot_w64(gor != 0);
    }
    if (64u * wave < nact) put_mask_bits<LPG>(flagged, img, logC, wave, lane);
    __syncthreads();

    // ---- a5 positions: exclusive popcount prefix over the mask words (a wave scan per wave) ----
    const uint32_t nwords = (B >> 8) >> LOG_LPG;          // 32-bit words of the mask (at most 64)
    const uint32_t my_word = lane < nwords ? img_maskw[lane] : 0u;
    const uint32_t my_pc = __popc(my_word);
    const uint32_t my_incl = wave_incl_scan(my_pc, lane);
    const uint32_t my_excl = my_incl - my_pc;
    const uint32_t cnt = __shfl(my_incl, 63, 64);
    const uint32_t S = (fixed + (uint32_t)LPG * a * cnt + 15u) & ~15u;
    // ---- a6: the size is known: publish it before anything else ----
    if (tid == 0) st_state(it.words + k, PB_SIZE | (uint64_t)(S >> 4));

    // ---- a4 low plane ----
    if (active) {
        switch (lm) {
        case 1: pb_pack_low_from_y<1, DT>(X, lrep, m, img_low, logC, tid); break;
        case 2: pb_pack_low_from_y<2, DT>(X, lrep, m, img_low, logC, tid); break;
        case 3: pb_pack_low_from_y<3, DT>(X, lrep, m, img_low, logC, tid); break;
        case 4: pb_pack_low_from_y<4, DT>(X, lrep, m, img_low, logC, tid); break;
        case 5: pb_pack_low_from_y<5, DT>(X, lrep, m, img_low, logC, tid); break;
        case 6: pb_pack_low_from_y<6, DT>(X, lrep, m, img_low, logC, tid); break;
        case 7: pb_pack_low_from_y<7, DT>(X, lrep, m, img_low, logC, tid); break;
        case 8: pb_pack_low_from_y<8, DT>(X, lrep, m, img_low, logC, tid); break;
        default: break;
        }
    }
    switch (a) {
    case 1: pb_pack_records_from_y<1, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 2: pb_pack_records_from_y<2, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 3: pb_pack_records_from_y<3, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 4: pb_pack_records_from_y<4, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 5: pb_pack_records_from_y<5, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 6: pb_pack_records_from_y<6, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 7: pb_pack_records_from_y<7, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 8: pb_pack_records_from_y<8, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    default: break;
    }

    // ---- a6 (wave 0): look back over the earlier blocks, PB_WINDOW at a time (lane i reads blocks
    // top - i, top - 64 - i, ...), until one of them carries its inclusive prefix.  A lower block is held
    // by a workgroup that publishes its size before it waits for anything (see above), so every wait
    // ends; the spin limit is a safety net. ----
    if (wave == 0) {
        uint64_t sum = 0;
        uint32_t flags = 0;
        int64_t top = (int64_t)k - 1;                    // highest block of the current window
        while (top >= 0) {
            uint64_t v[PB_WINDOW / 64];
            bool ok[PB_WINDOW / 64];
#pragma unroll
            for (int w = 0; w < PB_WINDOW / 64; ++w) { v[w] = 0; ok[w] = top - 64 * w - (int64_t)lane < 0; }
            uint32_t spins = 0, first_w = PB_WINDOW / 64, first_lane = 64;
            for (;;) {
#pragma unroll
                for (int w = 0; w < PB_WINDOW / 64; ++w)
                    if (!ok[w]) v[w] = ld_state(it.words + (top - 64 * w - (int64_t)lane));
                // the nearest block with a prefix; everything above it must be there
                bool missing = false;
                first_w = PB_WINDOW / 64;
                first_lane = 64;
#pragma unroll
                for (int w = 0; w < PB_WINDOW / 64; ++w) {
                    if (!ok[w]) ok[w] = v[w] != 0;
                    if (first_w == PB_WINDOW / 64) {
                        const uint64_t stop = __builtin_amdgcn_ballot_w64((v[w] & PB_PREFIX) != 0);
                        const uint64_t need = stop ? ((stop & (~stop + 1ull)) << 1) - 1ull : ~0ull;
                        if (__builtin_amdgcn_ballot_w64(!ok[w]) & need) missing = true;
                        if (stop) { first_w = w; first_lane = (uint32_t)__builtin_ctzll(stop); }
                    }
                }
                if (!missing) break;
                if (++spins > p.spin_limit) { flags |= 4u; break; }
                spin_pause(spins);
            }
            if (flags & 4u) break;
            uint64_t part = 0;
            bool gave_up = false;
#pragma unroll
            for (int w = 0; w < PB_WINDOW / 64; ++w) {
                const bool use = top - 64 * w - (int64_t)lane >= 0 &&
                                 ((uint32_t)w < first_w || ((uint32_t)w == first_w && lane <= first_lane));
                if (use) { part += v[w] & PB_VALUE; gave_up |= (v[w] & PB_GAVE_UP) != 0; }
            }
            if (__builtin_amdgcn_ballot_w64(gave_up)) flags |= 4u;
            sum += wave_sum(part);
            if (first_w != PB_WINDOW / 64) break;
            top -= PB_WINDOW;
        }
        if (lane == 0) {
            s_off = sum << 4;
            s_flags = flags;
            st_state(it.words + k, PB_PREFIX | ((flags & 4u) ? PB_GAVE_UP : 0ull) | (sum + (S >> 4)));
        }
    }
    __syncthreads();

    // ---- a7: stores ----
    // Streaming although each region starts at any 16 bytes, so that its ends are parts of lines: that writes 3.6 %
    // more than plain stores do (layer 313 against 302 MB), which the caches join, and is faster all the same
    // (67e6 elements of mixed blocks 81.8 against 82.5 us, 134e6 146.8 / 151.4, 34e6 53.0 / 54.4; blocks of 2048
    // equal).  One run dealt along lines, as in the one-tuple kernel, was not tried here.
    const uint64_t off = s_off;
    uint8_t *dst = it.out + it.payload_base + off;
    if (active) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            // pads have zero raw bytes already (their words were loaded as zero)
            const uint2 sm = t < PB_SM_REG_ROWS ? make_uint2(SM[t % PB_SM_REG_ROWS][0], SM[t % PB_SM_REG_ROWS][1])
                                                : *reinterpret_cast<const uint2 *>(sm_park + (((uint32_t)(t - PB_SM_REG_ROWS) * blockDim.x + tid) << 3));
            st_stream(reinterpret_cast<uint2 *>(dst + ((size_t)t << logC) + 8u * tid), sm);
        }
    }
    for (uint32_t v = tid; v < (mask_bytes >> 4); v += blockDim.x)
        st_stream(reinterpret_cast<uint4 *>(dst + B + 16u * v), *reinterpret_cast<const uint4 *>(img + 16u * v));
    if (lm > 0) {
        uint8_t *dlow = dst + B + mask_bytes;
        const uint32_t T2 = (lm * B) >> 4;               // half of the plane's length
        for (uint32_t v = tid; v < (T2 >> 3); v += blockDim.x) {
            const uint2 lo = *reinterpret_cast<const uint2 *>(img_low + 8u * v);
            const uint2 hi = *reinterpret_cast<const uint2 *>(img_low + 8u * v + T2);
            uint4 o;   // stream byte 2i = normalized byte i, stream byte 2i+1 = normalized byte i + T/2
            o.x = byte_perm(hi.x, lo.x, 0x05010400u);
            o.y = byte_perm(hi.x, lo.x, 0x07030602u);
            o.z = byte_perm(hi.y, lo.y, 0x05010400u);
            o.w = byte_perm(hi.y, lo.y, 0x07030602u);
            st_stream(reinterpret_cast<uint4 *>(dlow + 16u * v), o);
        }
    }
    if (a > 0) {
        uint8_t *dhigh = dst + fixed;
        const uint32_t hbytes = (uint32_t)LPG * a * cnt;
        for (uint32_t v = tid; 16u * v < hbytes; v += blockDim.x) {
            const uint4 o = *reinterpret_cast<const uint4 *>(img_high + 16u * v);
            uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {                // zero the padding behind the last record
                const uint32_t at = 16u * v + 4u * i;
                if (at >= hbytes) w[i] = 0;
                else if (at + 4u > hbytes) w[i] &= (1u << (8u * (hbytes - at))) - 1u;
            }
            st_stream(reinterpret_cast<uint4 *>(dhigh + 16u * v), make_uint4(w[0], w[1], w[2], w[3]));
        }
    }
    if (tid == 0) {
        uint64_t *table = reinterpret_cast<uint64_t *>(it.out + 64);
        table[k] = off;
        *reinterpret_cast<uint32_t *>(it.out + it.tuples_at + 4u * k) = b | (n << 8) | (m << 16);
        if (k == it.nb - 1u) {
            const uint64_t end = off + S;
            const uint32_t status = (s_flags & 4u) ? 8u : 0u;
            const uint64_t total = status ? 0ull : it.payload_base + end;
            table[it.nb] = end;
            if (((uint64_t)(it.nb + 1u) & 1ull)) table[it.nb + 1u] = 0;          // pad up to the tuple table
            for (uint32_t i = it.nb; i < ((it.nb + 3u) & ~3u); ++i)              // pad behind the tuple table
                *reinterpret_cast<uint32_t *>(it.out + it.tuples_at + 4u * i) = 0;
            uint32_t *h = reinterpret_cast<uint32_t *>(it.out);
            h[0] = 0x43454E45u;                                                // "ENEC"
            h[1] = 1u | ((uint32_t)DT << 16) | ((8u * LPG) << 24);             // version, dtype, L
            h[2] = (uint32_t)it.n_elems; h[3] = (uint32_t)(it.n_elems >> 32);
            h[4] = B; h[5] = it.nb;
            h[6] = E << 24;                                                    // (b, n, m) = 0: see the tuple table
            h[7] = status;
            h[8] = (uint32_t)total; h[9] = (uint32_t)(total >> 32);
            h[10] = 1u;                                                        // one tuple per block
#pragma unroll
            for (int i = 11; i < 16; ++i) h[i] = 0;
            if (it.out_bytes) *it.out_bytes = total;
        }
    }
}


// ---------------------------------------------------------------------------------
// The same streams for blocks of the default size, from a persistent grid with deferred stores: the tickets, scan words and
// their rules are those of compress_kernel (see "Inter-block scan" in enec_device.hpp).
//
// Bound: the in-order placement, then the chain of steps of a block.  A workgroup that places its block at once waits 8 us
// of 23 for the slowest of the blocks before it, 2 for its ticket and 3 for its rows.  Here the ticket and the rows of the
// next block travel while a block is worked on, and a block is stored an iteration after its size was published.  Three
// workgroups per CU (50 KB of LDS: two images of the worst case and the waiting block's raw bytes).  An iteration takes 12 us: rows
// and split 0.6, counting 1.9, sums and search 1.4, transform 0.7, packing 1.6, start of the waiting block 1.8, loads
// and stores 3.0, rest 0.9.  us per call, one workgroup per block with the former search -> this kernel:
//   before the waves' priority (below): 67e6 elements of mixed blocks 79.3 -> 60.3, 34e6 Gaussian 50.7 -> 34.8, 134e6
//   143.3 -> 119.8, fp16 34e6 52.5 -> 37.8, fp32 62.7 -> 56.8, 1e6 13.1 -> 10.5
//   a layer of Gaussian matrices, seven tensors of 405 MB: 210 -> 174, with the priority 154 (with two norm vectors, which take
//   the other kernel: 220 -> 185 -> 165); one with a scale per row and outliers, nine tensors: 234 -> 205 -> 191
// Looking up the start during the search and storing then, by the other three waves, was slower than all of these (mixed
// blocks 76): the blocks before have not published by then, and the wait for them grows from 1.8 to 5 us.
// The unit is compiled without the hoisting of constants out of loops: the sixteen packers' constants, kept in registers
// over the whole loop, cost the 16-bit formats 12 to 15 spilled registers (34e6 elements: bf16 38.3 against 36.1 us with
// groups of 16, 40.4 / 35.8 of 8, 41.8 / 39.1 of 32; fp16 41.4 / 38.9, 41.1 / 40.0, 43.9 / 41.7).  fp32 has twice the rows in
// flight, runs two waves per SIMD, spills neither way and loses by it, so its instances are compiled with the hoisting (34e6
// elements, without / with: groups of 16 57.5 / 55.1, of 8 59.4 / 54.8, of 32 61.7 / 56.8; 67e6 97.8 / 92.9).  compress_per_block_kernel, which has no loop over blocks, is the same either way: equal registers and
// times within 0.5 % in blocks of 2048 to 32768.
// ---------------------------------------------------------------------------------
#define PB_STREAM_WAVES (DT == DT_FP32 ? 2 : 3)

template <int DT, int LPG>
__global__ void __launch_bounds__((1 << DEFAULT_LOGB) / 64) __attribute__((amdgpu_waves_per_eu(PB_STREAM_WAVES, PB_STREAM_WAVES)))
compress_per_block_stream_kernel(const CompressArgs p)
{
    constexpr uint32_t E = exponent_bits(DT), logB = DEFAULT_LOGB, B = 1u << logB, logC = logB - 3u, T = B / 64u;
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    constexpr int RW = DT == DT_FP32 ? 16 : 8;
    constexpr uint32_t MASK_BYTES = (B >> 6) >> LOG_LPG, IMG = pb_image_bytes(8 * LPG);
    static_assert(IMG >= PB_HIST_COPIES * PB_HIST_STRIDE * 4 && IMG % 16 == 0, "the histogram copies lie where the image will be");

    // two images (mask | low plane as normalized bytes | high records), the waiting block's raw bytes in element order
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t s_hist[256];
    __shared__ unsigned long long s_present[4], s_best, s_tag, s_off;
    __shared__ uint32_t s_k[2], s_m, s_status;
    uint8_t *sm_wait = smem + 2u * IMG;

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;

    const uint32_t home = blockIdx.x % p.ncls;
    uint32_t *ctl = p.ws_ctl + WS_STRIDE * home;
    const uint32_t class_blocks = home < p.total ? (p.total - home + p.ncls - 1u) / p.ncls : 0u;
    const uint32_t class_wgs = (p.wgs - home + p.ncls - 1u) / p.ncls;
    uint32_t ticket_base = 0, zero = 0;
    uint64_t tag0 = 0;
    bool drawing = true;
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
    auto item_of = [&](uint32_t kg, uint32_t c) -> uint32_t {
        while (c + 1u < p.n_items && kg >= p.item[c + 1u].first) ++c;
        return c;
    };
    const uint32_t guess = blockIdx.x;
    uint32_t ci = item_of(guess, 0);
    uint4 raw[RW];
    load_block_rows<DT>(p.item[ci], B, logB, guess - p.item[ci].first, tid, true, logC, raw);
    auto clear_counts = [&](uint8_t *img) {
        for (uint32_t i = tid; i < PB_HIST_COPIES * PB_HIST_STRIDE / 4u; i += T) reinterpret_cast<uint4 *>(img)[i] = make_uint4(0, 0, 0, 0);
    };
    clear_counts(smem);
    if (tid == 0) {
        ticket_base = ctl[1];
        tag0 = *reinterpret_cast<const uint64_t *>(ctl + 2) + 1u;
        // the record must have been read before this workgroup's first draw can be counted
        zero = ticket_base ^ (uint32_t)tag0;
        asm volatile("v_and_b32 %0, 0, %0" : "+v"(zero));
        s_k[0] = decode_draw(atomicAdd(ctl + zero, 1u));
        s_tag = tag0;
        s_status = 0;
    }
    __syncthreads();
    uint32_t k = __builtin_amdgcn_readfirstlane(s_k[0]);
    if (k != guess && k != NO_BLOCK) {
        ci = item_of(k, 0);
        load_block_rows<DT>(p.item[ci], B, logB, k - p.item[ci].first, tid, true, logC, raw);
    }
    const uint64_t tag = (uint64_t)s_tag << 24;

    // wave 1 carries the scan of one tensor
    uint64_t groups_sum = 0;
    uint32_t groups_summed = 0, scan_flags = 0, scan_item = NO_BLOCK;
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
        return wave_sum32(need ? (uint32_t)(v & ST_VALUE) : 0u);
    };
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

    uint32_t pend = NO_BLOCK, pend_item = 0, pend_cnt = 0, pend_S = 0, pend_tuple = 0;
    auto store_block = [&](const CompressItem &it, uint32_t kb, const uint8_t *img) {
        const uint32_t n = (pend_tuple >> 8) & 0xFFu, m = pend_tuple >> 16;
        const uint32_t lm = m + (DT == DT_FP16 ? 3u : 0u);
        const uint64_t off = s_off;
        const uint64_t tuples = (64ull + 8ull * ((uint64_t)it.nb + 1u) + 15u) & ~15ull;
        uint8_t *dst = it.out + it.payload_base + off;
        const uint32_t shift = (uint32_t)((uintptr_t)dst >> 4) & 7u;     // vectors of the first line that are not ours
        constexpr uint32_t NSM = B >> 4, NMASK = MASK_BYTES >> 4;
        const uint32_t nlow = lm << (logB - 7u), hbytes = (uint32_t)LPG * (n - m) * pend_cnt, nall = pend_S >> 4;
        const uint32_t T2 = lm << (logB - 4u);                           // half of the low plane's length
        auto packed_vector = [&](uint32_t u) -> uint4 {
            const uint32_t j = u - NMASK;                                // vector of the low plane (wraps for a mask vector)
            if (j < nlow) {
                const uint2 a = *reinterpret_cast<const uint2 *>(img + MASK_BYTES + 8u * j);
                const uint2 c = *reinterpret_cast<const uint2 *>(img + MASK_BYTES + 8u * j + T2);
                return make_uint4(byte_perm(c.x, a.x, 0x05010400u), byte_perm(c.x, a.x, 0x07030602u),
                                  byte_perm(c.y, a.y, 0x05010400u), byte_perm(c.y, a.y, 0x07030602u));
            }
            const uint4 o = *reinterpret_cast<const uint4 *>(img + 16u * u);
            const uint32_t at = 16u * (j - nlow);                        // (huge for the mask)
            if (u < NMASK || at + 16u <= hbytes) return o;
            uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {                                // zero the padding behind the last record
                if (at + 4u * i >= hbytes) w[i] = 0;
                else if (at + 4u * i + 4u > hbytes) w[i] &= (1u << (8u * (hbytes - at - 4u * i))) - 1u;
            }
            return make_uint4(w[0], w[1], w[2], w[3]);
        };
        int32_t v = (int32_t)tid - (int32_t)shift;
#pragma unroll
        for (int i = 0; i < (int)(NSM / T); ++i)                         // ends at most at vector NSM - 1
            if (i > 0 || v >= 0)
                st_stream(reinterpret_cast<uint4 *>(dst) + v + i * (int)T, reinterpret_cast<const uint4 *>(sm_wait)[v + i * (int)T]);
        v += (int32_t)NSM;
        if (v < (int32_t)NSM) {                                          // the raw bytes' last vectors
            st_stream(reinterpret_cast<uint4 *>(dst) + v, reinterpret_cast<const uint4 *>(sm_wait)[v]);
            v += (int32_t)T;
        }
        for (; v < (int32_t)nall; v += (int32_t)T) st_stream(reinterpret_cast<uint4 *>(dst) + v, packed_vector((uint32_t)v - NSM));
        if (tid == 0) {
            uint64_t *table = reinterpret_cast<uint64_t *>(it.out + 64);
            table[kb] = off;
            *reinterpret_cast<uint32_t *>(it.out + tuples + 4ull * kb) = pend_tuple;
            if (kb == it.nb - 1u) {
                const uint64_t end = off + pend_S;
                uint32_t fl = s_status;
                if (ld_state(reinterpret_cast<const uint64_t *>(p.ws_ctl + 4)) == tag) fl |= 4u;   // somebody gave up
                const uint32_t status = (fl & 4u) ? 8u : 0u;
                const uint64_t total = status ? 0ull : it.payload_base + end;
                table[it.nb] = end;
                if (((uint64_t)(it.nb + 1u) & 1ull)) table[it.nb + 1u] = 0;          // pad up to the tuple table
                for (uint32_t i = it.nb; i < ((it.nb + 3u) & ~3u); ++i)              // pad behind the tuple table
                    *reinterpret_cast<uint32_t *>(it.out + tuples + 4u * i) = 0;
                uint32_t *h = reinterpret_cast<uint32_t *>(it.out);
                h[0] = 0x43454E45u;                                                // "ENEC"
                h[1] = 1u | ((uint32_t)DT << 16) | ((8u * LPG) << 24);             // version, dtype, L
                h[2] = (uint32_t)it.n_elems; h[3] = (uint32_t)(it.n_elems >> 32);
                h[4] = B; h[5] = it.nb;
                h[6] = E << 24;                                                    // (b, n, m) = 0: see the tuple table
                h[7] = status;
                h[8] = (uint32_t)total; h[9] = (uint32_t)(total >> 32);
                h[10] = 1u;                                                        // one tuple per block
#pragma unroll
                for (int i = 11; i < 16; ++i) h[i] = 0;
                if (it.out_bytes) *it.out_bytes = total;
            }
        }
    };

    uint32_t slot = 0;
    while (k != NO_BLOCK) {
        uint8_t *img = smem + slot * IMG;
        const CompressItem &it = p.item[ci];
        const uint32_t kl = k - it.first;

        uint32_t next_raw = 0;
        const bool draw_now = tid == 0 && p.lookahead && drawing;
        if (draw_now) next_raw = atomicAdd(ctl + zero, 1u);

        // ---- a1: split; fp16's three left-over mantissa bits travel in bits 5..7 of X's bytes ----
        const uint64_t blk0 = (uint64_t)kl << logB;
        const uint32_t real = it.n_elems - blk0 < B ? (uint32_t)(it.n_elems - blk0) : B;   // elements that are not pads
        const bool full = real == B;
        uint32_t X[8][2], SM[8][2];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint4 r16;
            if constexpr (DT == DT_FP32) {
                const uint4 u = raw[2 * t], v = raw[2 * t + 1];
                const uint32_t at = ((uint32_t)t << logC) + 8u * tid;
                r16 = make_uint4(byte_perm(u.y, u.x, 0x07060302u), byte_perm(u.w, u.z, 0x07060302u),
                                 byte_perm(v.y, v.x, 0x07060302u), byte_perm(v.w, v.z, 0x07060302u));
                if (at < real)
                    st_stream(reinterpret_cast<uint4 *>(it.out + it.tail_base + 2u * (blk0 + at)),
                              make_uint4(byte_perm(u.y, u.x, 0x05040100u), byte_perm(u.w, u.z, 0x05040100u),
                                         byte_perm(v.y, v.x, 0x05040100u), byte_perm(v.w, v.z, 0x05040100u)));
            } else {
                r16 = raw[t];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t d0 = h ? r16.z : r16.x, d1 = h ? r16.w : r16.y;
                const uint32_t Lb = byte_perm(d1, d0, 0x06040200u);
                const uint32_t Hb = byte_perm(d1, d0, 0x07050301u);
                if constexpr (DT == DT_FP16) {
                    SM[t][h] = (Hb & 0x80808080u) | ((Hb & 0x03030303u) << 5) | ((Lb >> 3) & 0x1F1F1F1Fu);
                    X[t][h] = ((Hb >> 2) & 0x1F1F1F1Fu) | ((Lb & 0x07070707u) << 5);
                } else {
                    SM[t][h] = bfi(0x7F7F7F7Fu, Lb, Hb);
                    X[t][h] = bfi(0xFEFEFEFEu, Hb << 1, Lb >> 7);
                }
            }
        }
        if (tid == 0) s_best = ~0ull;
        __syncthreads();                                                     // the copies are clear

        // ---- Sec. V-E phase 1: exponent counts of the block's own elements ----
        uint32_t *mine = reinterpret_cast<uint32_t *>(img) + (lane & (PB_HIST_COPIES - 1u)) * PB_HIST_STRIDE;
        if (full) {
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) atomicAdd(&mine[(X[t][h] >> (8 * i)) & (DT == DT_FP16 ? 0x1Fu : 0xFFu)], 1u);
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (((uint32_t)t << logC) + 8u * tid + i < real)
                        atomicAdd(&mine[(X[t][i >> 2] >> (8 * (i & 3))) & (DT == DT_FP16 ? 0x1Fu : 0xFFu)], 1u);
        }
        __syncthreads();
        {   // phase 2: the counts of the 256 exponent values, and which occur
            uint32_t c = 0;
#pragma unroll
            for (uint32_t i = 0; i < PB_HIST_COPIES; ++i) c += reinterpret_cast<const uint32_t *>(img)[i * PB_HIST_STRIDE + tid];
            s_hist[tid] = c;
            const uint64_t present = __builtin_amdgcn_ballot_w64(c != 0);
            if (lane == 0) s_present[wave] = present;
        }
        __syncthreads();
        pb_search<DT, LPG>(s_hist, s_present, s_best, s_m, real);
        const uint32_t b = (uint32_t)s_best & 0xFFu, n = ((uint32_t)s_best >> 8) & 0xFFu;
        const uint32_t m = s_m, a = n - m;
        const uint32_t lm = m + (DT == DT_FP16 ? 3u : 0u);
        uint32_t *img_maskw = reinterpret_cast<uint32_t *>(img);
        uint8_t *img_low = img + MASK_BYTES;
        uint8_t *img_high = img_low + (lm << (logB - 3u));
        const uint32_t fixed = B + MASK_BYTES + (lm << (logB - 3u));

        // ---- a2 transform (in place: X becomes y, fp16 keeps its three bits above), a3 group test ----
        const uint32_t crep = ((b + (1u << (n - 1))) & 0xFFu) * 0x01010101u;
        const uint32_t brep = b * 0x01010101u;
        const uint32_t srep = (1u << (n - 1)) * 0x01010101u;
        const uint32_t nrep = ((1u << n) - 1u) * 0x01010101u;
        const uint32_t lrep = ((1u << m) - 1u) * 0x01010101u;
        const uint32_t arep = ((1u << a) - 1u) * 0x01010101u;
        if (!full) {                               // pads behave like exponent b: y = 0
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int32_t left = (int32_t)real - (int32_t)(((uint32_t)t << logC) + 8u * tid + 4u * h);
                    const uint32_t padm = left <= 0 ? 0xFFFFFFFFu : (left >= 4 ? 0u : 0xFFFFFFFFu << (8 * left));
                    X[t][h] = bfi(padm, brep, X[t][h]);
                }
        }
        uint64_t flagged[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint32_t gor = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t x = X[t][h];
                if constexpr (DT == DT_FP16) x &= 0x1F1F1F1Fu;
                const uint32_t Y = (bytesub_safe(crep, x) ^ srep) & nrep;
                gor |= (Y >> m) & arep;
                if constexpr (DT == DT_FP16) X[t][h] = Y | (X[t][h] & 0xE0E0E0E0u);
                else X[t][h] = Y;
            }
            if constexpr (LPG == 2) gor |= swap_pair(gor);
            if constexpr (LPG == 4) gor = quad_or(gor);
            flagged[t] = __builtin_amdgcn_ballot_w64(gor != 0);
        }
        put_mask_bits<LPG>(flagged, img, logC, wave, lane);
        if (tid == 0) s_k[slot ^ 1u] = draw_now ? decode_draw(next_raw) : NO_BLOCK;
        __syncthreads();
        // From here to the end of the stores a block has what others wait for (its size, its place) and what travels (rows,
        // stores): these waves go before those of the CU's other workgroups, which count or search.  67e6 elements of mixed
        // blocks 61.0 -> 57.6 us.  (In compress_kernel, whose waves spend their time alike, it gave 0.6 % of the layer and of
        // 470 MB matrices and took 0.2 to 0.4 % from fp16 and groups of eight: left out.)
        __builtin_amdgcn_s_setprio(2);

        // wave 1 reads the scan state for the waiting block now and uses it after the packing
        uint64_t early_g = 0, early_b = 0;
        if (wave == 1 && pend != NO_BLOCK) {
            if (scan_item != pend_item) { scan_item = pend_item; groups_sum = 0; groups_summed = 0; scan_flags = 0; }
            const CompressItem &pit = p.item[pend_item];
            const uint32_t pg = pend >> GROUP_LOG;
            if (groups_summed + lane < pg) early_g = ld_state(pit.ws_group + groups_summed + lane);
            if (lane < (pend & (GROUP - 1u))) early_b = ld_state(pit.ws_block + ((uint64_t)pg << GROUP_LOG) + lane);
        }
        // ---- a5 positions, a6: publish this block's size at once ----
        constexpr uint32_t NWORDS = (B >> 8) >> LOG_LPG;          // 32-bit words of the mask (at most 64)
        const uint32_t my_word = lane < NWORDS ? img_maskw[lane] : 0u;
        const uint32_t my_pc = __popc(my_word);
        const uint32_t my_incl = wave_incl_scan(my_pc, lane);
        const uint32_t my_excl = my_incl - my_pc;
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)my_incl, 63);
        const uint32_t S = (fixed + (uint32_t)LPG * a * cnt + 15u) & ~15u;
        if (tid == 0) st_state(it.ws_block + kl, tag | (uint64_t)(S >> 4));
        const uint32_t grp = kl >> GROUP_LOG;
        const uint32_t members = it.nb - (grp << GROUP_LOG) < GROUP ? it.nb - (grp << GROUP_LOG) : GROUP;
        uint64_t acc_old = 0;
        if (tid == 64u && members > 1u)
            acc_old = __hip_atomic_fetch_add(it.ws_acc + grp, (1ull << 48) | (uint64_t)(S >> 4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // ---- a4 low plane, a5 one record per masked group ----
        switch (lm) {
        case 1: pb_pack_low_from_y<1, DT>(X, lrep, m, img_low, logC, tid); break;
        case 2: pb_pack_low_from_y<2, DT>(X, lrep, m, img_low, logC, tid); break;
        case 3: pb_pack_low_from_y<3, DT>(X, lrep, m, img_low, logC, tid); break;
        case 4: pb_pack_low_from_y<4, DT>(X, lrep, m, img_low, logC, tid); break;
        case 5: pb_pack_low_from_y<5, DT>(X, lrep, m, img_low, logC, tid); break;
        case 6: pb_pack_low_from_y<6, DT>(X, lrep, m, img_low, logC, tid); break;
        case 7: pb_pack_low_from_y<7, DT>(X, lrep, m, img_low, logC, tid); break;
        case 8: pb_pack_low_from_y<8, DT>(X, lrep, m, img_low, logC, tid); break;
        default: break;
        }
        switch (a) {
        case 1: pb_pack_records_from_y<1, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 2: pb_pack_records_from_y<2, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 3: pb_pack_records_from_y<3, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 4: pb_pack_records_from_y<4, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 5: pb_pack_records_from_y<5, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 6: pb_pack_records_from_y<6, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 7: pb_pack_records_from_y<7, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        case 8: pb_pack_records_from_y<8, LPG>(X, m, arep, my_word, my_excl, img_high, logC, tid, true); break;
        default: break;
        }

        // ---- a6: whoever completes a group publishes its word and clears the accumulator for the next call ----
        if (tid == 64u && (uint32_t)(acc_old >> 48) == members - 1u) {
            st_state(it.ws_group + grp, tag | ((acc_old & 0xFFFFFFFFull) + (S >> 4)));
            if (members > 1u) st_state(it.ws_acc + grp, 0ull);
        }
        // ---- a6 (wave 1): the start of the waiting block ----
        if (wave == 1 && pend != NO_BLOCK) {
            const uint64_t off = block_start(p.item[pend_item], pend, true, early_g, early_b);
            if (lane == 0) { s_off = off; s_status = scan_flags; }
        }
        __syncthreads();

        // the following block's rows start to travel while the previous block is stored
        const uint32_t knext = __builtin_amdgcn_readfirstlane(s_k[slot ^ 1u]);
        uint32_t cnext = ci;
        if (knext != NO_BLOCK) {
            cnext = item_of(knext, ci);
            load_block_rows<DT>(p.item[cnext], B, logB, knext - p.item[cnext].first, tid, true, logC, raw);
        }
        // ---- a7: stores of the previous block ----
        if (pend != NO_BLOCK) store_block(p.item[pend_item], pend, smem + (slot ^ 1u) * IMG);
        __syncthreads();                                                     // the other image and sm_wait are free

        // this block becomes the waiting one
#pragma unroll
        for (int t = 0; t < 8; ++t)
            *reinterpret_cast<uint2 *>(sm_wait + ((size_t)t << logC) + 8u * tid) = make_uint2(SM[t][0], SM[t][1]);
        clear_counts(smem + (slot ^ 1u) * IMG);
        __builtin_amdgcn_s_setprio(0);
        pend = kl; pend_item = ci; pend_cnt = cnt; pend_S = S; pend_tuple = b | (n << 8) | (m << 16);
        slot ^= 1u;
        k = knext;
        ci = cnext;
        if (k == NO_BLOCK && !p.lookahead) {           // without lookahead the next ticket is drawn only now
            if (tid == 0) s_k[slot] = drawing ? decode_draw(atomicAdd(ctl + zero, 1u)) : NO_BLOCK;
            __syncthreads();
            k = __builtin_amdgcn_readfirstlane(s_k[slot]);
            if (k != NO_BLOCK) {
                ci = item_of(k, ci);
                load_block_rows<DT>(p.item[ci], B, logB, k - p.item[ci].first, tid, true, logC, raw);
            }
        }
    }

    // ---- drain: the last block of this workgroup ----
    if (pend != NO_BLOCK) {
        if (wave == 1) {
            if (scan_item != pend_item) { scan_item = pend_item; groups_sum = 0; groups_summed = 0; scan_flags = 0; }
            const uint64_t off = block_start(p.item[pend_item], pend, false, 0, 0);
            if (lane == 0) { s_off = off; s_status = scan_flags; }
        }
        __syncthreads();
        store_block(p.item[pend_item], pend, smem + (slot ^ 1u) * IMG);
    }
}

}  // namespace enec
