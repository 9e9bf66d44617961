// Offline calibration: the Hessian of the layer-wise objective, H += X^T X for one batch of calibration activations
// X [T, K] (Eq. 5, App. A.2), on the matrix units.
//
// H is symmetric, so only the tiles on and below the diagonal are multiplied; a tile off the diagonal is added at both of
// its places.  A workgroup of four wavefronts owns a TILE x TILE tile, a wavefront (TILE / 2)^2 of it in 32 x 32 blocks,
// and walks over all tokens; a slice of tokens is staged in LDS (double buffered, the next slice's loads in flight in
// registers while this one is multiplied).
//   - bf16 activations: 32x32x16 bf16 MFMA.  An operand lane holds eight tokens of one feature, X holds the features of a
//     token side by side: a thread loads two features of eight tokens (a dword each) and transposes them in registers
//     on the way to LDS.  Products of bf16 are exact; the unit adds the eight of an octet with 24 bits below the largest
//     and rounds each octet's sum into the float32 accumulator to nearest, an eighth of the roundings of one float32 FMA
//     per token: at 8192 tokens x 4096 features the relative error against float64 (2-norm) is 3.9e-7, with the FMA
//     chain this replaces 3.8e-6.
//   - float32 activations: 32x32x2 float32 MFMA, which takes its two products in order, each one a correctly rounded
//     FMA -- the same chain per element, and the same bits, as a scalar loop over the tokens.
// Measured at 8192 tokens x 4096 features, against 64 x 64 tiles of scalar FMAs over both triangles: bf16 4190 -> 292 us
// (LDS reads of the operands bound it: two 16-byte reads per MFMA pair), float32 4040 -> 1410 us (the float32 matrix
// unit's rate, 153 TFLOP/s measured, takes 900).  The finer tiles even out the load where there are few: a launch is done
// when the compute unit with the most tiles is.  bf16 takes 128 x 128 tiles from 400 of them on (276 of them at 2944
// features 279 us, where 64 x 64 take about 220; 528 of them at 4096 features 339 us, now 292, 64 x 64 about 430), float32 always 64 x 64.
// On few tokens reading and writing H is most of the time, which the finer tiles spread better: up to 512 tokens 64 x 64 (128 x
// 128 / 64 x 64 tiles: 16 tokens x 5120 features 69 / 39 us, 512 tokens 92 / 64, 4096 features 54 / 48, 14336 features 696 / 637);
// rows that are not aligned for 4-byte loads up to 32 tokens only (32 tokens x 4096 features 42 / 41, 64 tokens 46 / 47).
#include "w4a8_device.hpp"
#include "w4a8_internal.hpp"

#include <math.h>

namespace w4a8 {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// How one thread brings its share of a slice from global memory to LDS, per input type.  load() takes any slice, with zeros for what is
// past the ends.  load_whole() (bf16, 128 x 128 tiles, aligned rows) takes a slice of existing tokens with one offset per lane (place())
// on top of a uniform row address, so that a load is one instruction; features past the end repeat the last ones, whose products belong
// to no element of H.  Range checks and 64-bit addresses for every load kept the vector unit busier than the matrix unit: 8192 tokens x
// 4096 features 351 -> 292 us, x 14336 features 3.06 -> 2.55 ms.  64 x 64 tiles, which run where tokens are few, gain 4 % by it on many
// tokens and lose 3 to 7 % on few; float32 ones are bound by the matrix unit.
template <typename InT, int TILE> struct Slice;

template <int TILE> struct Slice<float, TILE> {
    static constexpr int TOKENS = 16;
    static constexpr int STRIDE = TILE + 32;                     // floats per token: the two tokens of an operand lie 32 banks apart
    static constexpr int BYTES = TOKENS * STRIDE * 4;            // one operand
    static constexpr int UNITS = TOKENS * TILE / 4 / 256;        // four features of a token per unit
    float4 r[UNITS];
    // features f0 .. f0 + TILE - 1 of tokens t0 ..; zeros past the ends
    template <bool VEC>
    __device__ __forceinline__ void load(const float* x, int64_t T, int64_t K, int64_t ldx, int64_t t0, int64_t f0, int tid) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int id = tid + u * 256, t = id / (TILE / 4), f = (id % (TILE / 4)) * 4;
            const float* p = x + (t0 + t) * ldx + f0 + f;
            const bool row_ok = t0 + t < T;
            if (VEC) {
                r[u] = (row_ok && f0 + f < K) ? *reinterpret_cast<const float4*>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                r[u].x = (row_ok && f0 + f < K) ? p[0] : 0.f;
                r[u].y = (row_ok && f0 + f + 1 < K) ? p[1] : 0.f;
                r[u].z = (row_ok && f0 + f + 2 < K) ? p[2] : 0.f;
                r[u].w = (row_ok && f0 + f + 3 < K) ? p[3] : 0.f;
            }
        }
    }
    __device__ __forceinline__ void store(uint8_t* lds, int tid) const {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int id = tid + u * 256, t = id / (TILE / 4), f = (id % (TILE / 4)) * 4;
            *reinterpret_cast<float4*>(lds + (t * STRIDE + f) * 4) = r[u];
        }
    }
    template <int NB>
    static __device__ __forceinline__ void multiply(const uint8_t* a, const uint8_t* b, int fa, int fb, int lane, v16f (&acc)[NB][NB]) {
        const float* pa = reinterpret_cast<const float*>(a) + (lane >> 5) * STRIDE + fa + (lane & 31);
        const float* pb = reinterpret_cast<const float*>(b) + (lane >> 5) * STRIDE + fb + (lane & 31);
#pragma unroll
        for (int s = 0; s < TOKENS / 2; ++s) {
            float av[NB], bv[NB];
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                av[e] = pa[2 * s * STRIDE + e * 32];
                bv[e] = pb[2 * s * STRIDE + e * 32];
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
};

template <int TILE> struct Slice<uint16_t, TILE> {
    static constexpr int TOKENS = 32;
    static constexpr int BYTES = TOKENS * TILE * 2;              // one operand: octet o of feature f at (o * TILE + f) * 16
    static constexpr int UNITS = (TOKENS / 8) * (TILE / 2) / 256;    // two features of eight tokens per unit
    static constexpr int SPLIT = UNITS == 0 ? 2 : 1;             // 64 x 64 tiles: half of the threads per operand
    static constexpr int REGS = UNITS == 0 ? 1 : UNITS;
    uint32_t r[REGS][8];
    uint32_t at[REGS];
    __device__ __forceinline__ void place(int64_t K, int64_t ldx, int64_t f0, int tid) {
#pragma unroll
        for (int u = 0; u < REGS; ++u) {
            const int id = (tid & (256 / SPLIT - 1)) + u * 256, o = id / (TILE / 2), f = (id % (TILE / 2)) * 2;
            at[u] = (uint32_t)(o * 8 * ldx + min((int64_t)f, K - 2 - f0));
        }
    }
    // the slice that begins at the uniform address p (feature f0 of its first token)
    __device__ __forceinline__ void load_whole(const uint16_t* p, int64_t ldx) {
#pragma unroll
        for (int u = 0; u < REGS; ++u)
#pragma unroll
            for (int t = 0; t < 8; ++t) r[u][t] = *reinterpret_cast<const uint32_t*>(p + t * ldx + at[u]);
    }
    template <bool VEC>
    __device__ __forceinline__ void load(const uint16_t* x, int64_t T, int64_t K, int64_t ldx, int64_t t0, int64_t f0, int tid) {
#pragma unroll
        for (int u = 0; u < REGS; ++u) {
            const int id = (tid & (256 / SPLIT - 1)) + u * 256, o = id / (TILE / 2), f = (id % (TILE / 2)) * 2;
            const uint16_t* p = x + (t0 + o * 8) * ldx + f0 + f;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const bool row_ok = t0 + o * 8 + t < T;
                if (VEC) {
                    r[u][t] = (row_ok && f0 + f < K) ? *reinterpret_cast<const uint32_t*>(p + t * ldx) : 0u;
                } else {
                    const uint32_t lo = (row_ok && f0 + f < K) ? p[t * ldx] : 0u, hi = (row_ok && f0 + f + 1 < K) ? p[t * ldx + 1] : 0u;
                    r[u][t] = lo | (hi << 16);
                }
            }
        }
    }
    __device__ __forceinline__ void store(uint8_t* lds, int tid) const {
#pragma unroll
        for (int u = 0; u < REGS; ++u) {
            const int id = (tid & (256 / SPLIT - 1)) + u * 256, o = id / (TILE / 2), f = (id % (TILE / 2)) * 2;
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                lo[t] = __builtin_amdgcn_perm(r[u][2 * t + 1], r[u][2 * t], 0x05040100u);   // the first feature of both tokens
                hi[t] = __builtin_amdgcn_perm(r[u][2 * t + 1], r[u][2 * t], 0x07060302u);
            }
            uint8_t* p = lds + (o * TILE + f) * 16;
            *reinterpret_cast<uint4*>(p) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<uint4*>(p + 16) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        }
    }
    template <int NB>
    static __device__ __forceinline__ void multiply(const uint8_t* a, const uint8_t* b, int fa, int fb, int lane, v16f (&acc)[NB][NB]) {
        const uint8_t* pa = a + ((lane >> 5) * TILE + fa + (lane & 31)) * 16;
        const uint8_t* pb = b + ((lane >> 5) * TILE + fb + (lane & 31)) * 16;
#pragma unroll
        for (int s = 0; s < TOKENS / 16; ++s) {
            v8bf av[NB], bv[NB];
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                av[e] = *reinterpret_cast<const v8bf*>(pa + (2 * s * TILE + e * 32) * 16);
                bv[e] = *reinterpret_cast<const v8bf*>(pb + (2 * s * TILE + e * 32) * 16);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
};

constexpr int64_t MAX_LDX = int64_t(1) << 24;   // 32 rows of it below 2^32 bytes

// 128 x 128 tiles: three workgroups to a compute unit, so that the 528 tiles of 4096 features run at the same time
template <typename InT, int TILE, bool VEC>
__global__ void __launch_bounds__(256, TILE == 128 ? 3 : 1) hessian_accumulate_kernel(const InT* __restrict__ x, int64_t T, int64_t K, int64_t ldx,
                                                                 float* __restrict__ h, int h_vec) {
    using S = Slice<InT, TILE>;
    constexpr int NB = TILE / 64;                                // 32 x 32 blocks of a wavefront in each direction
    constexpr bool HALVES = sizeof(InT) == 2 && TILE == 64;      // each half of the threads stages one operand
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][2 * S::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // tile (bi, bj), bj <= bi, of the lower triangle, row by row
    const int b = blockIdx.x;
    int bi = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
    while ((int64_t)bi * (bi + 1) / 2 > b) --bi;
    while ((int64_t)(bi + 1) * (bi + 2) / 2 <= b) ++bi;
    const int bj = b - (int)((int64_t)bi * (bi + 1) / 2);
    const int64_t i0 = (int64_t)bi * TILE, j0 = (int64_t)bj * TILE;

    v16f acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    S sa, sb;
    constexpr bool WHOLE = sizeof(InT) == 2 && TILE == 128 && VEC;
    const bool near = WHOLE && ldx <= MAX_LDX;                   // offsets inside a slice fit 32 bits
    if constexpr (WHOLE) {
        if (near) {
            sa.place(K, ldx, i0, tid);
            sb.place(K, ldx, j0, tid);
        }
    }
    auto load = [&](int64_t t0) {
        if constexpr (WHOLE) {
            if (near && t0 + S::TOKENS <= T) {
                sa.load_whole(x + t0 * ldx + i0, ldx);
                sb.load_whole(x + t0 * ldx + j0, ldx);
                return;
            }
        }
        if (HALVES) {
            sa.template load<VEC>(x, T, K, ldx, t0, tid < 128 ? i0 : j0, tid);
        } else {
            sa.template load<VEC>(x, T, K, ldx, t0, i0, tid);
            sb.template load<VEC>(x, T, K, ldx, t0, j0, tid);
        }
    };
    const int fa = (wave >> 1) * (TILE / 2), fb = (wave & 1) * (TILE / 2);
    load(0);
    int buf = 0;
    for (int64_t t0 = 0; t0 < T; t0 += S::TOKENS, buf ^= 1) {
        if (HALVES) {
            sa.store(lds[buf] + (tid < 128 ? 0 : S::BYTES), tid);
        } else {
            sa.store(lds[buf], tid);
            sb.store(lds[buf] + S::BYTES, tid);
        }
        __syncthreads();                                         // also: everyone is done with the stage the next slice goes to
        if (t0 + S::TOKENS < T) load(t0 + S::TOKENS);
        S::template multiply<NB>(lds[buf], lds[buf] + S::BYTES, fa, fb, lane, acc);
    }
    // result lane: column lane % 32 of a block, rows 8 (v / 4) + 4 (lane / 32) + v % 4
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int64_t gj = j0 + fb + j * 32 + (lane & 31);
            if (gj >= K) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t gi = i0 + fa + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (gi < K) h[gi * K + gj] += acc[i][j][v];
            }
            if (bi != bj) {                                      // the mirrored tile: four neighbouring columns per lane
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t gi = i0 + fa + i * 32 + 8 * q + 4 * (lane >> 5);
                    float* p = h + gj * K + gi;
                    if (h_vec && gi + 3 < K) {
                        float4 w = *reinterpret_cast<const float4*>(p);
                        w.x += acc[i][j][4 * q];
                        w.y += acc[i][j][4 * q + 1];
                        w.z += acc[i][j][4 * q + 2];
                        w.w += acc[i][j][4 * q + 3];
                        *reinterpret_cast<float4*>(p) = w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (gi + e < K) p[e] += acc[i][j][4 * q + e];
                    }
                }
            }
        }
}

template <typename InT, int TILE>
int launch_tile(const InT* x, int64_t T, int64_t K, int64_t ldx, bool vec, float* h, hipStream_t st) {
    const int64_t n = (K + TILE - 1) / TILE;
    const dim3 grid((unsigned)(n * (n + 1) / 2));
    const int h_vec = K % 4 == 0 && reinterpret_cast<uintptr_t>(h) % 16 == 0;   // the mirrored tile is added through float4
    if (vec) hipLaunchKernelGGL((hessian_accumulate_kernel<InT, TILE, true>), grid, dim3(256), 0, st, x, T, K, ldx, h, h_vec);
    else hipLaunchKernelGGL((hessian_accumulate_kernel<InT, TILE, false>), grid, dim3(256), 0, st, x, T, K, ldx, h, h_vec);
    return launch_status();
}

}  // namespace

int launch_hessian_accumulate(const void* x, w4a8_dtype dt, int64_t T, int64_t K, int64_t ldx, float* h, hipStream_t st) {
    const uintptr_t addr = reinterpret_cast<uintptr_t>(x);
    if (dt == W4A8_F32) {
        const bool vec = addr % 16 == 0 && ldx % 4 == 0 && K % 4 == 0;
        return launch_tile<float, 64>(static_cast<const float*>(x), T, K, ldx, vec, h, st);
    }
    const bool vec = addr % 4 == 0 && ldx % 2 == 0 && K % 2 == 0;
    const int64_t n = (K + 127) / 128;
    if (n * (n + 1) / 2 >= 400 && T > (vec ? 512 : 32)) return launch_tile<uint16_t, 128>(static_cast<const uint16_t*>(x), T, K, ldx, vec, h, st);
    return launch_tile<uint16_t, 64>(static_cast<const uint16_t*>(x), T, K, ldx, vec, h, st);
}

}  // namespace w4a8
