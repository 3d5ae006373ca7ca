// Compression of tensors of one data block each (norm vectors, biases) with a given tuple.
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

template <int DT, int LPG>
__device__ __forceinline__ void compress_one_block(const SingleItem &it, uint8_t *smem, uint32_t (&s_tab)[128], uint32_t (&s_err)[8],
                                                   uint32_t threads)
{
    constexpr uint32_t E = exponent_bits(DT);
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    constexpr int Q = DT == DT_FP32 ? 2 : 4;             // vectors of a thread whose loads travel together
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t logB = it.logB, B = 1u << logB, logC = logB - 3u, nvec = B >> 3;
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

template <int DT, int LPG>
__global__ void __launch_bounds__(SINGLE_THREADS) compress_single_kernel(const SingleArgs p)
{
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t s_tab[128], s_err[8];
    const SingleItem &it = p.item[blockIdx.x];
    const uint32_t nvec = 1u << (it.logB - 3u), threads = nvec < SINGLE_THREADS ? nvec : SINGLE_THREADS;
    if (threadIdx.x >= threads) return;                  // whole waves that the launch's larger blocks need
    compress_one_block<DT, LPG>(it, smem, s_tab, s_err, threads);
}

}  // namespace enec
