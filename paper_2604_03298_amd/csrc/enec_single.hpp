// Compression of tensors of one data block each (norm vectors, biases) with a given tuple.
//
// Bound: the latency of a launch.  Such a tensor has no earlier block to wait for and nobody waits for it, so none of what
// compress_kernel does for the order of blocks is needed here: control record, ticket, scan words and the look at them are
// four trips to memory one after the other, and its stores wait for them.  A workgroup takes one tensor; its raw bytes are
// stored as soon as they are split.  The widths and the block size are run-time values, looked up with the tensor, so that
// tensors share a launch whatever their tuples and lengths.
#pragma once
#include "enec_per_block.hpp"

namespace enec {

template <int DT, int LPG>
__global__ void __launch_bounds__(512) compress_single_kernel(const SingleArgs p)
{
    constexpr uint32_t E = exponent_bits(DT);
    constexpr int LOG_LPG = LPG == 4 ? 2 : LPG - 1;
    constexpr int RW = DT == DT_FP32 ? 16 : 8;
    extern __shared__ __align__(16) uint8_t smem[];      // mask | low plane (normalized bytes) | high records
    __shared__ uint32_t s_err;

    const SingleItem &it = p.item[blockIdx.x];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t logB = it.logB, B = 1u << logB, logC = logB - 3u, nact = B >> 6, threads = nact < 64u ? 64u : nact;
    if (tid >= threads) return;                          // whole waves that the launch's larger blocks need
    const bool active = tid < nact;
    uint4 raw[RW];
    load_block_rows<DT>(it, B, logB, 0u, tid, active, logC, raw);
    if (tid == 0) s_err = 0;

    const uint32_t b = it.b, n = it.n, m = it.m, a = n - m;
    const uint32_t lm = m + (DT == DT_FP16 ? 3u : 0u);
    const uint32_t mask_bytes = nact >> LOG_LPG;                      // B / (8 L)
    const uint32_t fixed = B + mask_bytes + ((lm * B) >> 3);
    uint8_t *img_low = smem + mask_bytes, *img_high = img_low + ((lm * B) >> 3);
    uint8_t *dst = it.out + it.payload_base;
    const uint32_t crep = ((b + (1u << (n - 1))) & 0xFFu) * 0x01010101u;
    const uint32_t srep = (1u << (n - 1)) * 0x01010101u;
    const uint32_t nrep = ((1u << n) - 1u) * 0x01010101u;
    const uint32_t lrep = ((1u << m) - 1u) * 0x01010101u;
    const uint32_t arep = ((1u << a) - 1u) * 0x01010101u;
    const uint32_t xlo = b + 1u > (1u << (n - 1)) ? b + 1u - (1u << (n - 1)) : 0u;
    const uint32_t xhi = b + (1u << (n - 1)) < 255u ? b + (1u << (n - 1)) : 255u;

    // ---- a1 split, a2 transform, a3 group test ----
    uint32_t Y[8][2];                    // fp16: the three left-over mantissa bits in bits 5..7
    uint64_t flagged[8];
    uint32_t out_of = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint32_t at = ((uint32_t)t << logC) + 8u * tid;
        uint4 r16;
        if constexpr (DT == DT_FP32) {
            const uint4 u = raw[2 * t], v = raw[2 * t + 1];
            r16 = make_uint4(byte_perm(u.y, u.x, 0x07060302u), byte_perm(u.w, u.z, 0x07060302u),
                             byte_perm(v.y, v.x, 0x07060302u), byte_perm(v.w, v.z, 0x07060302u));
            if (active && at < it.n_elems)
                st_stream(reinterpret_cast<uint4 *>(it.out + it.tail_base + 2u * at),
                          make_uint4(byte_perm(u.y, u.x, 0x05040100u), byte_perm(u.w, u.z, 0x05040100u),
                                     byte_perm(v.y, v.x, 0x05040100u), byte_perm(v.w, v.z, 0x05040100u)));
        } else {
            r16 = raw[t];
        }
        uint32_t sm[2], gor = 0;
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
            if (it.mode == 2) {                    // (a difference modulo 256 could lie in the window by wrapping)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t xb = (X >> (8 * i)) & 0xFFu;
                    out_of |= (uint32_t)((xb < xlo) | (xb > xhi));
                }
            } else if (it.mode == 0) {
                out_of |= Z & ~nrep;
            }
            const uint32_t y = (Z ^ srep) & nrep;
            gor |= (y >> m) & arep;
            Y[t][h] = y | T3;
        }
        if (active) st_stream(reinterpret_cast<uint2 *>(dst + ((size_t)t << logC) + 8u * tid), make_uint2(sm[0], sm[1]));
        if constexpr (LPG == 2) gor |= swap_pair(gor);
        if constexpr (LPG == 4) gor = quad_or(gor);
        flagged[t] = __builtin_amdgcn_ballot_w64(gor != 0);
    }
    put_mask_bits<LPG>(flagged, smem, logC, wave, lane);
    __syncthreads();
    if (__builtin_amdgcn_ballot_w64(out_of != 0) != 0 && lane == 0) atomicOr(&s_err, 1u);

    // ---- a5 positions, a4 low plane, a5 one record per masked group ----
    const uint32_t nwords = (B >> 8) >> LOG_LPG;
    const uint32_t my_word = lane < nwords ? reinterpret_cast<const uint32_t *>(smem)[lane] : 0u;
    const uint32_t my_pc = __popc(my_word);
    const uint32_t my_incl = wave_incl_scan(my_pc, lane);
    const uint32_t my_excl = my_incl - my_pc;
    const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)my_incl, 63);
    const uint32_t hbytes = (uint32_t)LPG * a * cnt, S = (fixed + hbytes + 15u) & ~15u;
    if (active) {
        switch (lm) {
        case 1: pb_pack_low_from_y<1, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 2: pb_pack_low_from_y<2, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 3: pb_pack_low_from_y<3, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 4: pb_pack_low_from_y<4, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 5: pb_pack_low_from_y<5, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 6: pb_pack_low_from_y<6, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 7: pb_pack_low_from_y<7, DT>(Y, lrep, m, img_low, logC, tid); break;
        case 8: pb_pack_low_from_y<8, DT>(Y, lrep, m, img_low, logC, tid); break;
        default: break;
        }
    }
    switch (a) {
    case 1: pb_pack_records_from_y<1, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 2: pb_pack_records_from_y<2, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 3: pb_pack_records_from_y<3, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 4: pb_pack_records_from_y<4, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 5: pb_pack_records_from_y<5, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 6: pb_pack_records_from_y<6, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 7: pb_pack_records_from_y<7, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    case 8: pb_pack_records_from_y<8, LPG>(Y, m, arep, my_word, my_excl, img_high, logC, tid, active); break;
    default: break;
    }
    __syncthreads();

    // ---- a7: mask | low plane, joined | high records, zero padding ----
    dst += B;
    const uint32_t nmask = mask_bytes >> 4, nlow = (lm * B) >> 7, T2 = (lm * B) >> 4;
    for (uint32_t v = tid; v < (S - B) >> 4; v += threads) {
        const uint32_t j = v - nmask;                    // vector of the low plane (wraps for a mask vector)
        uint4 o;
        if (j < nlow) {
            const uint2 c = *reinterpret_cast<const uint2 *>(img_low + 8u * j);
            const uint2 d = *reinterpret_cast<const uint2 *>(img_low + 8u * j + T2);
            o = make_uint4(byte_perm(d.x, c.x, 0x05010400u), byte_perm(d.x, c.x, 0x07030602u),
                           byte_perm(d.y, c.y, 0x05010400u), byte_perm(d.y, c.y, 0x07030602u));
        } else {
            o = *reinterpret_cast<const uint4 *>(smem + 16u * v);
            const uint32_t at = 16u * (j - nlow);
            if (v >= nmask && at + 16u > hbytes) {
                uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (at + 4u * i >= hbytes) w[i] = 0;
                    else if (at + 4u * i + 4u > hbytes) w[i] &= (1u << (8u * (hbytes - at - 4u * i))) - 1u;
                }
                o = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        st_stream(reinterpret_cast<uint4 *>(dst + 16u * v), o);
    }
    if (tid == 0) {
        const uint32_t status = s_err ? 6u : 0u;
        const uint64_t total = status ? 0ull : it.payload_base + S;
        uint64_t *table = reinterpret_cast<uint64_t *>(it.out + 64);
        table[0] = 0;
        table[1] = S;
        uint32_t *h = reinterpret_cast<uint32_t *>(it.out);
        h[0] = 0x43454E45u;                              // "ENEC"
        h[1] = 1u | ((uint32_t)DT << 16) | ((8u * LPG) << 24);   // version, dtype, L
        h[2] = (uint32_t)it.n_elems; h[3] = 0;
        h[4] = B; h[5] = 1;
        h[6] = b | (n << 8) | (m << 16) | (E << 24);
        h[7] = status;
        h[8] = (uint32_t)total; h[9] = 0;
#pragma unroll
        for (int i = 10; i < 16; ++i) h[i] = 0;
        if (it.out_bytes) *it.out_bytes = total;
    }
}

}  // namespace enec
