// Output side of the many-token kernels: a wavefront's finished sums to memory, without a barrier.
//
// A wavefront owns WM blocks of 16 tokens x WN bands of 16 channels; a lane holds channel lane % 16 of every band, tokens
// 4 (lane / 16) .. + 3 of every block.  It turns a block (several, where their rows are short) into row-major order in an
// LDS slab of its own -- a wavefront's LDS accesses run in order, so there is no wait beyond the one for the data -- and
// stores 16 bytes per lane, whole row segments.
#pragma once
#include "w4a8_device.hpp"

#include <utility>

namespace w4a8 {

// the value of the neighbouring lane (lane ^ 1), and of the lane two further (lane ^ 2)
__device__ __forceinline__ uint32_t from_pair_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1 /* quad_perm [1, 0, 3, 2] */, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t from_next_pair_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E /* quad_perm [2, 3, 0, 1] */, 0xF, 0xF, true);
}

// Lane q of four neighbouring lanes comes with bytes (row 0 .. 3) of column q and leaves with bytes (column 0 .. 3) of row q.
__device__ __forceinline__ uint32_t transpose_bytes_in_quad(uint32_t v, int lane) {
    const bool odd = (lane & 1) != 0, high = (lane & 2) != 0;
    // v_perm_b32(S0, S1, sel): selector 0..3 -> bytes of S1, 4..7 -> bytes of S0
    const uint32_t p = from_pair_lane(v);
    v = __builtin_amdgcn_perm(v, p, odd ? 0x07030501u : 0x02060004u);    // even: v0 p0 v2 p2, odd: p1 v1 p3 v3
    const uint32_t n = from_next_pair_lane(v);
    return __builtin_amdgcn_perm(v, n, high ? 0x07060302u : 0x01000504u);   // low: v0 v1 n0 n1, high: n2 n3 v2 v3
}

// two float32 -> two bf16 (round to nearest even) in one dword
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    const b2 c = __builtin_convertvector(v, b2);
    return *reinterpret_cast<const uint32_t*>(&c);
}

// Writes blocks F0 .. F1 - 1 of acc.  slab: the wavefront's own, SlabBytes<OutT, WN>::value.  m_wave: token of block 0's first row;
// n_wave: channel of band 0's first column (of N; the rows of a SiluFp8 output have N / 2 bytes).  scale: s_x, or what the
// partial sums of a K range are stored with; OUT_SCALED: times w_out[n] (w_out[0] when per_channel is 0).  q: FP8 outputs.
template <typename OutT, int WN> struct OutLayout {
    static constexpr bool SILU = OutKind<OutT>::SILU, FP8 = sizeof(OutT) == 1;
    static constexpr int EB = FP8 ? 1 : (int)sizeof(OutT);       // bytes per output
    static constexpr int ROW_B = (SILU ? 8 : 16) * WN * EB;      // bytes of a wavefront's row
    static constexpr int SEGS = ROW_B / 16;                      // 16-byte pieces of it
    static constexpr int BLOCKS = SEGS < 4 ? 4 / SEGS : 1;       // blocks per round: 64 pieces at least
    static constexpr int STRIDE = ROW_B + 16;
    static constexpr int SLAB_BYTES = 16 * BLOCKS * STRIDE;
};
template <typename OutT, int WM, int WN, bool OUT_SCALED, int F0, int F1>
__device__ __forceinline__ void store_tile(const v4f (&acc)[WM][WN], uint8_t* slab, int m_wave, int n_wave, int M, int N, OutT* y, int64_t ldy,
                                           float scale, const float* w_out, int per_channel, const StaticQuantizer& q, int lane) {
    using L = OutLayout<OutT, WN>;
    constexpr int EB = L::EB, RSB = L::STRIDE, SEGS = L::SEGS, ROWS_PER_STORE = 64 / SEGS, STORES = 16 * L::BLOCKS / ROWS_PER_STORE;
    static_assert((F1 - F0) % L::BLOCKS == 0, "whole rounds");
    const int i = lane & 15, kq = lane >> 4;
    const int seg = lane % SEGS, srow = lane / SEGS;
    const int n_first = L::SILU ? n_wave / 2 : n_wave, n_end = L::SILU ? N / 2 : N;
    float so[WN];                                                // output scale of the lane's channel of band j
#pragma unroll
    for (int j = 0; j < WN; ++j) so[j] = OUT_SCALED ? scale * w_out[per_channel ? min(n_wave + j * 16 + i, N - 1) : 0] : scale;
    const bool odd = (i & 1) != 0;
    const uint32_t sel_lo = odd ? 0x05040100u : 0x01000504u, sel_hi = odd ? 0x07060302u : 0x03020706u;
    auto lo = [](uint32_t pair) { return __uint_as_float(pair << 16); };
    auto hi = [](uint32_t pair) { return __uint_as_float(pair & 0xFFFF0000u); };
#pragma unroll
    for (int f = F0; f < F1; f += L::BLOCKS) {
        wave_lds_fence();                                        // the round before has read its rows
#pragma unroll
        for (int b = 0; b < L::BLOCKS; ++b) {
            const v4f(&a)[WN] = acc[f + b];
            uint8_t* const rows = slab + b * 16 * RSB;
            if constexpr (L::SILU) {
#pragma unroll
                for (int j = 0; j < WN; j += 2) {                // band j: gate rows, band j + 1: the up rows of the same channels
                    const uint32_t g01 = bf16_pair(scale * a[j][0], scale * a[j][1]), g23 = bf16_pair(scale * a[j][2], scale * a[j][3]);
                    const uint32_t u01 = bf16_pair(scale * a[j + 1][0], scale * a[j + 1][1]), u23 = bf16_pair(scale * a[j + 1][2], scale * a[j + 1][3]);
                    const uint32_t h01 = bf16_pair(silu_mul_bf16_gate(lo(g01), lo(u01)), silu_mul_bf16_gate(hi(g01), hi(u01)));
                    const uint32_t h23 = bf16_pair(silu_mul_bf16_gate(lo(g23), lo(u23)), silu_mul_bf16_gate(hi(g23), hi(u23)));
                    const uint32_t w = transpose_bytes_in_quad(q.four(lo(h01), hi(h01), lo(h23), hi(h23)), lane);
                    *reinterpret_cast<uint32_t*>(rows + (4 * kq + (i & 3)) * RSB + (j / 2) * 16 + (i & ~3)) = w;
                }
            } else if constexpr (L::FP8) {
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    const uint32_t v01 = bf16_pair(scale * a[j][0], scale * a[j][1]), v23 = bf16_pair(scale * a[j][2], scale * a[j][3]);
                    const uint32_t w = transpose_bytes_in_quad(q.four(lo(v01), hi(v01), lo(v23), hi(v23)), lane);
                    *reinterpret_cast<uint32_t*>(rows + (4 * kq + (i & 3)) * RSB + j * 16 + (i & ~3)) = w;
                }
            } else if constexpr (EB == 2) {
                // even lanes keep tokens 0, 1 and take the odd neighbour's, odd lanes keep tokens 2, 3: a lane then holds
                // channels {i & ~1, i | 1} of two tokens
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    const uint32_t v01 = bf16_pair(so[j] * a[j][0], so[j] * a[j][1]), v23 = bf16_pair(so[j] * a[j][2], so[j] * a[j][3]);
                    const uint32_t own = odd ? v23 : v01, nb = from_pair_lane(odd ? v01 : v23);
                    uint8_t* p = rows + (4 * kq + (odd ? 2 : 0)) * RSB + (j * 16 + (i & ~1)) * 2;
                    *reinterpret_cast<uint32_t*>(p) = __builtin_amdgcn_perm(own, nb, sel_lo);
                    *reinterpret_cast<uint32_t*>(p + RSB) = __builtin_amdgcn_perm(own, nb, sel_hi);
                }
            } else {
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) *reinterpret_cast<float*>(rows + (4 * kq + r) * RSB + (j * 16 + i) * 4) = so[j] * a[j][r];
            }
        }
        wave_lds_fence();
#pragma unroll
        for (int h = 0; h < STORES; ++h) {
            const int row = h * ROWS_PER_STORE + srow;
            const uint4 w = *reinterpret_cast<const uint4*>(slab + row * RSB + seg * 16);
            const int m = m_wave + f * 16 + row, n = n_first + seg * (16 / EB);
            if (m < M && n < n_end) {
                OutT* dst = y + (int64_t)m * ldy + n;
                if (n + 16 / EB <= n_end) {
                    store_16_unaligned(dst, w);
                } else {
                    const uint32_t e4[4] = {w.x, w.y, w.z, w.w};
                    for (int e = 0; e < 16 / EB && n + e < n_end; ++e) {
                        if constexpr (EB == 1) reinterpret_cast<uint8_t*>(dst)[e] = (uint8_t)(e4[e / 4] >> (8 * (e % 4)));
                        else if constexpr (EB == 2) dst[e] = (uint16_t)(e4[e / 2] >> (16 * (e % 2)));
                        else dst[e] = __uint_as_float(e4[e]);
                    }
                }
            }
        }
    }
}

}  // namespace w4a8
