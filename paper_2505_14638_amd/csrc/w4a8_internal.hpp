// Host-side declarations shared by the kernel files and the C-ABI front end.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/w4a8.h"
#include "../../include/w4a8_tuning.h"
#include "launch_choice.hpp"

namespace w4a8 {

inline int hip_status(hipError_t e) { return e == hipSuccess ? W4A8_OK : W4A8_ERR_HIP; }
inline int launch_status() { return hip_status(hipGetLastError()); }

// What the launchers of the tiled-layout linear kernels pass down to a launch: the operands of w4a8_linear after
// validation.
struct LinearArgs {
    const uint8_t* x8;
    int M;
    int64_t ldx8;
    const float* s_x;
    const uint8_t* packed;
    const float* scales;
    int N, n_tiles, C, cpg, NG;      // channels, 16-row bands, 128-deep chunks, chunks per group, groups per row
    void* y;
    int64_t ldy;
    const float* w_out;
    int per_channel;
    int mode;                        // a WeightMode
    const float* y_scale;            // FP8 output only: the static scale the output is quantized with (Eq. 13)
    int xq = 0;                      // skinny kernel: x8 is the float32 (1) / bf16 (2) activation matrix, quantized in the kernel
    uint8_t* x8_out = nullptr;       // ... and where its codes go as well (row stride K), or null
};

// Output type beyond the public w4a8_dtype values, for the launchers: E4M3 bytes, the bf16 result quantized with the
// next layer's static activation scale (code-exact mode only).
constexpr int YDT_E4M3 = 2;
// The gate|up layer with SiLU*mul and the next quantization folded in (see SiluFp8): y is E4M3 bytes [M, N / 2].
constexpr int YDT_SILU_E4M3 = 3;

int launch_quantize_act(const void* x, w4a8_dtype dt, int64_t M, int64_t K, int64_t ldx, const float* scale,
                        uint8_t* x8, int64_t ldx8, hipStream_t st);
int launch_act_amax(const void* x, w4a8_dtype dt, int64_t M, int64_t K, int64_t ldx, float* amax, hipStream_t st);
int launch_act_scale(const float* amax, float* scale, hipStream_t st);
int launch_pack_weights(const void* src, w4a8_src kind, const float* src_scales, int64_t N, int64_t K, int32_t G,
                        w4a8_layout layout, uint8_t* packed, float* scales, hipStream_t st);
// asymmetric format (tiled storage): src = float32 weights (W4A8_SRC_F32_RTN) or unsigned codes with their scales and
// zero-points; params = the 80-byte records
int launch_pack_weights_asym(const void* src, w4a8_src kind, const float* src_scales, const uint8_t* src_zeros,
                             int64_t N, int64_t K, int32_t G, uint8_t* packed, uint8_t* params, hipStream_t st);
// tiled layout only: scales8 != nullptr: the two-level bytes nearest_E4M3(code * s8[n,g]); asym_params != nullptr: the
// asymmetric format's bytes nearest_E4M3(code - zero_point[n,g]), or with asym_two_level its two-level bytes
// nearest_E4M3((code - zero_point[n,g]) * s8[n,g])
int launch_dequant_weights(const uint8_t* packed, int64_t N, int64_t K, w4a8_layout layout, uint8_t* w8,
                           const float* scales8, const uint8_t* asym_params, int asym_two_level, int32_t G,
                           hipStream_t st);
int launch_linear_canonical(const uint8_t* x8, int64_t M, int64_t K, int64_t ldx8, const float* s_x,
                            const uint8_t* packed, const float* scales, int64_t N, int32_t G, void* y,
                            w4a8_dtype ydt, int64_t ldy, hipStream_t st);
// nt / waves / depth = 0: chosen from the shape.  mode: a WeightMode; w_out and per_channel count in MODE_TWO_LEVEL.
int launch_linear_skinny(const uint8_t* x8, int64_t M, int64_t K, int64_t ldx8, const float* s_x,
                         const uint8_t* packed, const float* scales, int64_t N, int32_t G, void* y, w4a8_dtype ydt,
                         int64_t ldy, int nt, int waves, int depth, const float* w_out, int per_channel, int mode,
                         const float* y_scale, hipStream_t st, int xq = 0, uint8_t* x8_out = nullptr);
// The launch shapes the launchers choose by themselves (requested values other than 0 are kept); false: not built.
bool skinny_launch_shape(int64_t M, int64_t K, int64_t N, int ydt, int mode, int xq, int& nt, int& waves, int& depth);
bool mfma_launch_shape(int64_t M, int64_t K, int64_t N, int mode, int& mf, int& ks, int& tpw, int& cfg2d);
// mf = 16-token blocks per workgroup, ks = K-split groups per workgroup, tpw = weight bands per wavefront; 0: chosen
int launch_linear_mfma_tiled(const uint8_t* x8, int64_t M, int64_t K, int64_t ldx8, const float* s_x,
                             const uint8_t* packed, const float* scales, int64_t N, int32_t G, void* y,
                             w4a8_dtype ydt, int64_t ldy, int mf, int ks, int tpw, const float* w_out, int per_channel,
                             int mode, const float* y_scale, hipStream_t st);
// Second tiling of the many-token kernel (2-D grid of wavefronts, expansion shared through LDS, persistent workgroups).
// cfg: a tile of mfma2d_tile; group_m = token blocks per super-column of the block order (0: chosen); workgroups = size of
// the persistent grid (0: one per compute unit); mode: a WeightMode, the two-level ones with w_out and per_channel as in the
// first tiling (float32 / bf16 outputs, no split of K); ksplit > 1: K is multiplied in that
// many ranges by different workgroups, their float32 partial sums go through `workspace` (mfma2d_splitk_bytes).
bool mfma2d_tile(int cfg, int& bm, int& bn);

int launch_linear_mfma2d(const uint8_t* x8, int64_t M, int64_t K, int64_t ldx8, const float* s_x, const uint8_t* packed,
                         const float* scales, int64_t N, int32_t G, void* y, w4a8_dtype ydt, int64_t ldy, int cfg,
                         int group_m, int workgroups, int mode, const float* y_scale, hipStream_t st, int ksplit = 1,
                         void* workspace = nullptr, const float* w_out = nullptr, int per_channel = 0);
void launch_linear_pipe(const LinearArgs& a, int cfg, int ydt, dim3 grid, int grid_m, int grid_n, int group_m, int ksplit, int cps,
                        int64_t split_stride, hipStream_t st);
int launch_hessian_accumulate(const void* x, w4a8_dtype dt, int64_t T, int64_t K, int64_t ldx, float* h, hipStream_t st);
int launch_gar_permutation(const float* hdiag, int64_t K, int32_t G, int32_t* perm, hipStream_t st);
// U = upper Cholesky factor of the inverse dampened (and reordered) Hessian; workspace: hessian_factor_workspace_bytes(K)
size_t hessian_factor_workspace_bytes(int64_t K);
int launch_hessian_inverse_factor(const float* h, int64_t K, double damp, const int32_t* perm, void* workspace, float* u,
                                  int32_t* info, hipStream_t st);
// workspace: N * K floats, the current weights
int launch_dpq_calibrate(const float* w, const float* u, const float* s_w, int per_channel, const int32_t* perm,
                         int64_t N, int64_t K, int32_t G, uint8_t* codes, float* scales, uint8_t* zeros, void* workspace,
                         int mse_grid, float mse_max_shrink, hipStream_t st);
// q_scale != nullptr: h is E4M3 bytes, the bf16 result quantized with *q_scale (Eq. 13)
int launch_silu_mul(const void* gu, int64_t M, int64_t F, int64_t ldgu, void* h, int64_t ldh, const float* q_scale,
                    hipStream_t st);

}  // namespace w4a8
