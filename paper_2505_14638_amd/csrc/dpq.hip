// Offline calibration: Dual Precision Quantization (Alg. 1, Eq. 5-12) and the Group-Aware Reordering permutation
// (Sec. 3.2, App. A.3).
//
// Alg. 1 walks along a row: quantize one weight (FP8, then INT4, Eq. 7-9), dequantize it the way inference will
// (Eq. 10-11), and push the error onto every later weight of the row through the Hessian factor U (Eq. 12; U is the
// upper Cholesky factor of the inverse Hessian, Sec. 3.3).  Rows are independent, columns strictly sequential.  The
// work is arranged in blocks of 128 columns: inside a block four lanes own a row; the columns right of the block receive
// the block's 128 errors afterwards, tile by tile.  Every weight still sees the same float32 operations in the same order
// as in the plain column-by-column statement (w <- w - err_q * U[q, v] for q ascending, product and difference rounded
// separately), so the integer decisions are reproducible bit for bit; only the time at which an update is applied moves.
// That rules out the matrix unit (a product there is not rounded by itself): the updates take a multiplication and a
// subtraction each on the vector unit, 1.75 ms for 4096 x 4096 weights.
#include "w4a8_device.hpp"
#include "w4a8_internal.hpp"

namespace w4a8 {
namespace {

constexpr int DPQ_BLOCK = 128;      // columns per block

// val(nearest_Z(t)): the E4M3 value nearest to t (ties to even, saturating), as a float32
__device__ __forceinline__ float fp8_value(float t) {
    const int b = __builtin_amdgcn_cvt_pk_fp8_f32(sat448(t), 0.0f, 0, false);
    return __builtin_amdgcn_cvt_f32_fp8(b, 0);
}

// position i of the reordered tensor holds original column perm[i]: inside a group by descending diagonal, groups
// by descending maximum; ties keep the lower original index first.  One thread per column; the maxima of the groups come
// from the workgroup together, MAXIMA groups at a time (every thread for itself, all K values one after the other: 185 us at
// K = 4096; together 25).  A maximum is kept as an unsigned integer that orders like the floats, 0 for "nothing but
// NaN", which no comparison below is true for.
constexpr int MAXIMA = 1024;
__global__ void __launch_bounds__(256) gar_permutation_kernel(const float* __restrict__ d, int K, int G, int32_t* __restrict__ perm) {
    __shared__ uint32_t top[MAXIMA];
    auto value_of = [](uint32_t key) {
        return key == 0u ? __uint_as_float(0x7FC00000u) : __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
    };
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const bool mine_exists = c < K;
    const int g = (mine_exists ? c : 0) / G, NG = K / G;
    const float mine = d[mine_exists ? c : 0];
    int inside = 0;
    float gmax = d[(int64_t)g * G];
#pragma unroll 16
    for (int j = 0; j < G; ++j) {
        const float v = d[g * G + j];
        inside += (v > mine) || (v == mine && g * G + j < c);
        gmax = fmaxf(gmax, v);
    }
    int rank = 0;
    for (int h0 = 0; h0 < NG; h0 += MAXIMA) {
        const int count = min(MAXIMA, NG - h0);
        for (int h = threadIdx.x; h < count; h += 256) top[h] = 0u;
        __syncthreads();
        for (int e = threadIdx.x; e < count * G; e += 256) {                    // the 64 values of a wavefront lie in one group
            const float v = d[h0 * G + e];
            const uint32_t b = __float_as_uint(v);
            uint32_t key = (v != v) ? 0u : (b & 0x80000000u) ? ~b : b | 0x80000000u;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) key = max(key, (uint32_t)__shfl_xor((int)key, m));
            if ((threadIdx.x & 63) == 0) atomicMax(&top[e / G], key);
        }
        __syncthreads();
        for (int h = 0; h < count; ++h) {
            const float m = value_of(top[h]);
            rank += (m > gmax) || (m == gmax && h0 + h < g);
        }
        __syncthreads();
    }
    if (mine_exists) perm[rank * G + inside] = c;
}

struct DpqArgs {
    const float* w;               // [N, K] the weights, original column order
    float* work;                  // [N, K] current weights, reordered columns; a finished block's columns hold its errors
    const float* u;               // [K, K] upper factor, reordered columns
    const float* s_w;
    int per_channel;
    const int32_t* perm;          // or nullptr
    int N, K, G;
    uint8_t* codes;               // [N, K], original column order
    float* scales;                // [N, K / G], original group order
    uint8_t* zeros;               // [N, K / G]
    int mse_grid;                 // candidates of the scale search (Sec. 3.3); <= 1: none
    float shrink_step;            // max_shrink / mse_grid
};

// Eq. 8 for a range [lo, hi] that contains zero: s = (hi - lo) / 15 (1 for an empty range), z = round(-lo / s)
__device__ __forceinline__ void group_params(float lo, float hi, float& s, float& z) {
    const float span = __fsub_rn(hi, lo);
    s = (span == 0.0f) ? 1.0f : __fdiv_rn(span, 15.0f);
    z = fminf(fmaxf(rintf(__fdiv_rn(-lo, s)), 0.0f), 15.0f);
}

// a / b, correctly rounded, from y = RN(1 / b): the estimate a * y is at most two units off, one correction makes it
// faithful, and a second one rounds it correctly (Markstein's theorem on the final step of a division by a correctly
// rounded reciprocal).  Five operations, where the general division takes about ten and several mode switches; valid while
// neither the residuals nor the quotient leave the normal range, which the callers' range checks see to (a zero's sign may
// differ, which nothing here depends on).
__device__ __forceinline__ float div_by(float a, float b, float y) {
    float q = __fmul_rn(a, y);
    q = __fmaf_rn(__fmaf_rn(-b, q, a), y, q);
    return __fmaf_rn(__fmaf_rn(-b, q, a), y, q);
}
constexpr float DIV_LO = 0x1p-30f, DIV_HI = 0x1p30f;            // divisors
constexpr uint32_t NUM_LO = 0x21800000u, NUM_SPAN = 0x5D800000u - 0x21800000u;   // bits of 2^-60, up to 2^60: weights
__device__ __forceinline__ bool plain_divisor(float b) { return fabsf(b) >= DIV_LO && fabsf(b) <= DIV_HI; }

// fp8_value for a finite t
__device__ __forceinline__ float fp8_value_finite(float t) {
    return __builtin_amdgcn_cvt_f32_fp8(__builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(t, -448.0f, 448.0f), 0.0f, 0, false), 0);
}

// score += the squared error of DPQ_BLOCK FP8 values at `v` quantized with (s, z) and reconstructed (Eq. 9 with clipping, Eq. 10),
// one after the other.  plain: s is a plain divisor and no value is NaN; a value is then zero or between 2^-9 and 448, and
// everything here stays finite.
__device__ __forceinline__ void add_squared_error(const float* v, float s, float z, bool plain, float& score) {
    if (plain) {
        const float y = __fdiv_rn(1.0f, s);
        auto add = [&](float w8) {
            const float uq = __builtin_amdgcn_fmed3f(rintf(__fadd_rn(div_by(w8, s, y), z)), 0.0f, 15.0f);
            const float d = __fsub_rn(w8, fp8_value_finite(__fmul_rn(__fsub_rn(uq, z), s)));
            score = __fadd_rn(score, __fmul_rn(d, d));
        };
#pragma unroll 2
        for (int j = 0; j < DPQ_BLOCK; j += 4) {
            const float4 t = *reinterpret_cast<const float4*>(v + j);
            add(t.x);
            add(t.y);
            add(t.z);
            add(t.w);
        }
    } else {
        for (int j = 0; j < DPQ_BLOCK; ++j) {
            const float uq = fminf(fmaxf(rintf(__fadd_rn(__fdiv_rn(v[j], s), z)), 0.0f), 15.0f);
            const float d = __fsub_rn(v[j], fp8_value(__fmul_rn(__fsub_rn(uq, z), s)));
            score = __fadd_rn(score, __fmul_rn(d, d));
        }
    }
}

template <int P>
__device__ __forceinline__ float quad_broadcast(float v) {       // lane P of the lane's group of four
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), P * 0x55, 0xF, 0xF, true));
}

constexpr int ROWS = 64;             // rows of a workgroup's tile; four lanes each inside a block
constexpr int SEG = 32;              // columns of a block whose rows of U are staged at a time
constexpr int TILE_STRIDE = DPQ_BLOCK + 4;
constexpr int PART = 36;             // staged U: [column q][lane p of the row][slot]: U[q, 4 * (q / 4 + slot) + p]
constexpr int SEG_FLOATS = SEG * 4 * PART;
constexpr int SLICE_FLOATS = SEG * (ROWS + DPQ_BLOCK);           // one slice of the update: errors and U
constexpr int DPQ_LDS = 2 * SEG_FLOATS > ROWS * TILE_STRIDE ? 2 * SEG_FLOATS : ROWS * TILE_STRIDE;
static_assert(SLICE_FLOATS <= DPQ_LDS, "the update's slice fits");

struct RowState {
    float w[32];                  // the lane's columns of the block that are left: slot j = column 4 (done + j) + p
    float sw, y_sw, s, y_s, z;
    uint32_t span;                // NUM_SPAN, or 0 when a divisor of this row asks for the general division
};

// One weight: column q of the block, U[q, v] for the lane's columns v from q's slot on at `u`, U[q, q] and its reciprocal
// in `d`.  Q = q % 4 is the lane of the row that owns it, in slot 0 of R.w; LEFT the slots in R.w.
template <int Q, int LEFT>
__device__ __forceinline__ void dpq_weight(RowState& R, const float* u, float2 d, bool diag_plain, int p, float& code) {
    float4 v[LEFT / 4];
#pragma unroll
    for (int j = 0; j < LEFT / 4; ++j) v[j] = *reinterpret_cast<const float4*>(u + 4 * j);   // back by the time e is there
    const float w = quad_broadcast<Q>(R.w[0]);
    const bool plain = (__float_as_uint(w) & 0x7FFFFFFFu) - NUM_LO < R.span && diag_plain;
    const float w8 = fp8_value_finite(div_by(w, R.sw, R.y_sw));                           // Eq. 7
    const float t = __fadd_rn(div_by(w8, R.s, R.y_s), R.z);
    float uq = __builtin_amdgcn_fmed3f(rintf(t), 0.0f, 15.0f);                            // Eq. 9
    const float w8_hat = fp8_value_finite(__fmul_rn(__fsub_rn(uq, R.z), R.s));            // Eq. 10
    float e = div_by(__fsub_rn(w, __fmul_rn(w8_hat, R.sw)), d.x, d.y);                    // Eq. 11
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!plain) != 0, 0)) {                  // zeros, extreme values: the general division
        const float g8 = fp8_value(__fdiv_rn(w, R.sw));
        uq = fminf(fmaxf(rintf(__fadd_rn(__fdiv_rn(g8, R.s), R.z)), 0.0f), 15.0f);
        const float g8_hat = fp8_value(__fmul_rn(__fsub_rn(uq, R.z), R.s));
        e = __fdiv_rn(__fsub_rn(w, __fmul_rn(g8_hat, R.sw)), d.x);
    }
#pragma unroll
    for (int j = 0; j < LEFT; ++j) {                                                      // Eq. 12 inside the block
        const float next = __fsub_rn(R.w[j], __fmul_rn(e, j % 4 == 0 ? v[j / 4].x : j % 4 == 1 ? v[j / 4].y : j % 4 == 2 ? v[j / 4].z : v[j / 4].w));
        // in the weight's own slot: lanes behind it are updated, its own lane keeps the error, those before it theirs
        R.w[j] = j > 0 ? next : p > Q ? next : p == Q ? e : R.w[j];
        asm volatile("" : "+v"(R.w[j]));                         // here, not where the column is next read: the products would pile up
    }
    if (p == Q) code = uq;
}

// The 32 columns of a segment, LEFT slots in R.w at its start: slot by slot, the codes and errors going out and R.w moving on.
// A loop of four weights (the whole block unrolled is 70 KB of instructions that every launch fetches anew, 80 us a block).
template <int LEFT>
__device__ __forceinline__ void dpq_segment(RowState& R, const DpqArgs& a, const float* u, const float2* diag, const int* cols, bool diag_plain,
                                            int64_t n, bool row_ok, int c, int p) {
    u += p * PART;
#pragma unroll 1
    for (int t = 0; t < SEG / 4; ++t, u += 16 * PART, diag += 4) {
        float code = 0.0f;
        const int col = cols[4 * t + p];
        dpq_weight<0, LEFT>(R, u, diag[0], diag_plain, p, code);
        dpq_weight<1, LEFT>(R, u + 4 * PART, diag[1], diag_plain, p, code);
        dpq_weight<2, LEFT>(R, u + 8 * PART, diag[2], diag_plain, p, code);
        dpq_weight<3, LEFT>(R, u + 12 * PART, diag[3], diag_plain, p, code);
        if (row_ok) {
            a.work[n * a.K + c + 4 * t + p] = R.w[0];
            a.codes[n * a.K + col] = (uint8_t)code;
        }
#pragma unroll
        for (int j = 0; j + 1 < LEFT; ++j) R.w[j] = R.w[j + 1];
    }
}

// What becomes of the first column block's tiles: written to `work` like the others, or quantized with the group's parameters,
// formed from the tile (groups of one block) or found in the outputs (where dpq_group_kernel put them).
enum BlockStep { NO_BLOCK = 0, PARAMS_HERE = 1, PARAMS_GIVEN = 2 };

// One launch of the walk.  Workgroups own tiles of 64 rows x 128 columns of the columns from c_first on, the tiles of the
// first column block coming first:
//   gather:  the tile comes from the original weights, reordered; otherwise from `work`;
//   update:  it receives the errors of the block at c_err (Eq. 12 for the columns right of a block: for every column q of
//            that block, ascending, w <- w - err[n, q] * U[c_err + q, v]);
//   block:   the tiles of the first column block are then quantized, column by column, the others written to `work`;
//   ready:   a launch before has brought that many column blocks up to date: the first is only quantized, the other ones skipped.
// With groups of 128 one launch does the first three: the next block is quantized by the workgroups that bring it up to date
// while the others update the rest, so the serial part (60 us a block, the update of its own columns included) hides behind
// the updates for as long as there are many.  With a scale search in a launch of its own the block's columns are brought up
// to date in a launch before that.  Wider groups need all of their columns up to date before the first is quantized: an
// update and a block launch each.
// Update: a thread owns 8 x 4 outputs; per error column three 16-byte LDS reads feed 64 vector operations, which bound it
// (4096 rows x 3968 columns: 112 us, with 4 x 4 outputs and a pass of its own 219; the vector unit needs 107).
// Block: lane p of a row's four holds the columns v with v % 4 == p in registers; every lane takes the (identical)
// quantization step and applies the error to its own columns.  The row of U comes from LDS, 32 columns staged at a time.  32
// lanes per row, with the weights in LDS, spent most instructions on repeating the quantization step (89 us a block).
// Measured at 4096 x 4096: 6.7 -> 2.3 ms; at 256 x 4096, where the serial part is all, 3.9 -> 1.9.
// Three workgroups to a compute unit leave 168 registers, which spills 47 of them, all outside the loops over columns: once
// per launch and 32 columns.  With two and no spills 256 x 4096 takes 1.79 ms instead of 1.90 and 4096 x 4096 2.32 instead of
// 2.26, 16384 x 4096 7.13 instead of 6.38.
__global__ void __launch_bounds__(256, 3) dpq_step_kernel(DpqArgs a, int c_first, int c_err, int row_blocks, int gather, int update, int block,
                                                          int ready) {
    __shared__ __attribute__((aligned(16))) float lds[DPQ_LDS];
    __shared__ float2 diag[2][SEG];
    __shared__ int cols[DPQ_BLOCK];                              // original columns of the block
    __shared__ int general[2];                                   // a diagonal entry of the staged segment asks for the general division
    const int tid = threadIdx.x;
    const int rb = blockIdx.x % row_blocks, cb = blockIdx.x / row_blocks;
    if (ready > 0 && cb == 0) gather = update = 0;
    const int r0 = rb * ROWS, v0 = c_first + (ready > 0 && cb > 0 ? cb + ready - 1 : cb) * DPQ_BLOCK;
    const int tr = (tid >> 5) * 8, tc = (tid & 31) * 4;          // K is a multiple of 128: the columns of a tile all exist
    float w[8][4];
    {
        int64_t col[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) col[j] = (gather && a.perm) ? a.perm[v0 + tc + j] : v0 + tc + j;
        const float* src = gather ? a.w : a.work;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t n = min(r0 + tr + i, a.N - 1);         // rows past the end repeat the last one; not stored
#pragma unroll
            for (int j = 0; j < 4; ++j) w[i][j] = src[n * a.K + col[j]];
        }
    }
    if (update) {
        float* el = lds;                                         // el[q * 64 + r]: error q of row r of the tile
        float* ul = lds + SEG * ROWS;                            // ul[q * 128 + c]: U[c_err + q, column c of the tile]
        const float* erow = a.work + (int64_t)min(r0 + (tid & 63), a.N - 1) * a.K + c_err + (tid >> 6) * 4;
        const float* urow = a.u + (int64_t)(c_err + (tid >> 5)) * a.K + v0 + tc;
        float e4[2][4], u4[4][4];
        auto load = [&](int q0) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) e4[h][j] = erow[q0 + h * 16 + j];
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) u4[h][j] = urow[(int64_t)(q0 + h * 8) * a.K + j];
        };
        load(0);
        for (int q0 = 0; q0 < DPQ_BLOCK; q0 += SEG) {
            __syncthreads();                                     // everyone is done with the slice before
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) el[((tid >> 6) * 4 + h * 16 + j) * ROWS + (tid & 63)] = e4[h][j];
#pragma unroll
            for (int h = 0; h < 4; ++h)
                *reinterpret_cast<float4*>(ul + ((tid >> 5) + h * 8) * DPQ_BLOCK + tc) = make_float4(u4[h][0], u4[h][1], u4[h][2], u4[h][3]);
            __syncthreads();
            if (q0 + SEG < DPQ_BLOCK) load(q0 + SEG);
#pragma unroll 4
            for (int q = 0; q < SEG; ++q) {
                const float4 ea = *reinterpret_cast<const float4*>(el + q * ROWS + tr), eb = *reinterpret_cast<const float4*>(el + q * ROWS + tr + 4);
                const float4 uu = *reinterpret_cast<const float4*>(ul + q * DPQ_BLOCK + tc);
                const float ev[8] = {ea.x, ea.y, ea.z, ea.w, eb.x, eb.y, eb.z, eb.w}, uv[4] = {uu.x, uu.y, uu.z, uu.w};
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[i][j] = __fsub_rn(w[i][j], __fmul_rn(ev[i], uv[j]));
            }
        }
    }
    if (!block || cb != 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (r0 + tr + i < a.N) {
#pragma unroll
                for (int j = 0; j < 4; ++j) a.work[(int64_t)(r0 + tr + i) * a.K + v0 + tc + j] = w[i][j];
            }
        return;
    }

    // the block: lane p of row r of the tile
    __builtin_amdgcn_s_setprio(2);                               // ahead of the update's wavefronts on the same SIMD
    const int r = tid >> 2, p = tid & 3, c0 = c_first;
    const int64_t n = min(r0 + r, a.N - 1);
    const bool row_ok = r0 + r < a.N;
    // the rows of U of segment sg, columns from the segment's first on: thread -> 16 values of row tid / 8
    float us[16];
    const float* useg = a.u + (int64_t)(c0 + (tid >> 3)) * a.K + c0 + (tid & 7) * 16;
    float ud;                                                    // threads 0..31: U[q, q] of the segment's columns
    auto load_u = [&](int sg) {
        if (tid < SEG) ud = a.u[(int64_t)(c0 + sg * SEG + tid) * (a.K + 1)];
        if (sg * SEG + (tid & 7) * 16 < DPQ_BLOCK) {
#pragma unroll
            for (int j = 0; j < 16; ++j) us[j] = useg[(int64_t)sg * SEG * a.K + sg * SEG + j];
        }
    };
    load_u(0);
    __syncthreads();                                             // everyone is done with the update's last slice
#pragma unroll
    for (int i = 0; i < 8; ++i)
        *reinterpret_cast<float4*>(lds + (tr + i) * TILE_STRIDE + tc) = make_float4(w[i][0], w[i][1], w[i][2], w[i][3]);
    if (tid < 2) general[tid] = 0;
    if (tid < DPQ_BLOCK) cols[tid] = a.perm ? a.perm[c0 + tid] : c0 + tid;
    __syncthreads();
    RowState R;
    float* mine = lds + r * TILE_STRIDE;
#pragma unroll
    for (int j = 0; j < 32; ++j) R.w[j] = mine[4 * j + p];
    R.sw = a.s_w[a.per_channel ? n : 0];
    const int NG = a.K / a.G, g = c0 / a.G;
    const int og = a.perm ? a.perm[g * a.G] / a.G : g;           // the original group these columns belong to
    float s, z;
    if (block == PARAMS_HERE) {                                  // Eq. 8 on the group's current weights, which are the tile's
        float lo = 0.0f, hi = 0.0f;                              // minimum and maximum: any order gives the same result
        bool nan = false;
#pragma unroll 4
        for (int j = p; j < DPQ_BLOCK; j += 4) {
            const float w8 = fp8_value(__fdiv_rn(mine[j], R.sw));
            lo = fminf(lo, w8);
            hi = fmaxf(hi, w8);
            nan |= w8 != w8;
            mine[j] = w8;                                        // what the search below scores
        }
#pragma unroll
        for (int m = 1; m < 4; m <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, m));
            hi = fmaxf(hi, __shfl_xor(hi, m));
        }
        group_params(lo, hi, s, z);
        if (a.mse_grid > 1) {                                    // the search of dpq_group_kernel, a row's lanes sharing the candidates
            __builtin_amdgcn_wave_barrier();                     // a row's lanes lie in one wavefront, whose LDS accesses run in order
            float best = __builtin_inff(), bs = s, bz = z;
            int best_i = a.mse_grid;
            for (int i = p; i < a.mse_grid; i += 4) {
                const float shrink = __fsub_rn(1.0f, __fmul_rn((float)i, a.shrink_step));
                float si, zi, score = 0.0f;
                group_params(__fmul_rn(shrink, lo), __fmul_rn(shrink, hi), si, zi);
                add_squared_error(mine, si, zi, __builtin_amdgcn_ballot_w64(!plain_divisor(si) || nan) == 0, score);
                if (score < best) { best = score; best_i = i; bs = si; bz = zi; }
            }
#pragma unroll
            for (int m = 1; m < 4; m <<= 1) {
                const float ob = __shfl_xor(best, m), os = __shfl_xor(bs, m), oz = __shfl_xor(bz, m);
                const int oi = __shfl_xor(best_i, m);
                if (ob < best || (ob == best && oi < best_i)) { best = ob; best_i = oi; bs = os; bz = oz; }
            }
            s = bs;
            z = bz;
        }
        if (p == 0 && row_ok) {
            a.scales[n * NG + og] = s;
            a.zeros[n * NG + og] = (uint8_t)z;
        }
    } else {
        s = a.scales[n * NG + og];
        z = (float)a.zeros[n * NG + og];
    }
    R.s = s;
    R.z = z;
    R.y_sw = __fdiv_rn(1.0f, R.sw);
    R.y_s = __fdiv_rn(1.0f, s);
    R.span = plain_divisor(R.sw) && plain_divisor(s) ? NUM_SPAN : 0u;
    __syncthreads();                                             // the tile has been read by everyone

    auto stage_u = [&](int sg) {
        float* dst = lds + (sg & 1) * SEG_FLOATS;
        const int q = tid >> 3, first = (tid & 7) * 16, col = sg * SEG + first;
        if (col < DPQ_BLOCK) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {                       // what lies left of the row's own slot goes to a slot that nobody reads
                const int slot = (first + j) / 4 - q / 4;
                dst[(q * 4 + (j & 3)) * PART + (slot >= 0 ? slot : PART - 1)] = us[j];
            }
        }
        if (tid < SEG) {
            diag[sg & 1][tid] = make_float2(ud, __fdiv_rn(1.0f, ud));
            if (!plain_divisor(ud)) atomicOr(&general[sg & 1], 1);
        }
        // (slots past a row's last are read too, for columns of R.w that are done: values of no account)
    };
#define W4A8_DPQ_SEGMENT(SG)                                                                                        \
    {                                                                                                               \
        stage_u(SG);                                                                                                \
        __syncthreads();                                                                                            \
        if (SG < 3) load_u(SG + 1);                                                                                 \
        const bool diag_plain = general[SG & 1] == 0;                                                               \
        dpq_segment<32 - 8 * SG>(R, a, lds + (SG & 1) * SEG_FLOATS, diag[SG & 1], cols + SG * SEG, diag_plain, n, row_ok, c0 + SG * SEG, p); \
    }
    W4A8_DPQ_SEGMENT(0) W4A8_DPQ_SEGMENT(1) W4A8_DPQ_SEGMENT(2) W4A8_DPQ_SEGMENT(3)
#undef W4A8_DPQ_SEGMENT
}

// Group parameters of the group at columns c0 .. c0 + G - 1, which `work` holds up to date: Eq. 8 on the FP8 values, and with
// mse_grid > 1 the scale search of Sec. 3.3 (the paper names it, not its grid): candidate i shrinks the range by p_i = 1 - i *
// shrink_step and is scored by the squared error, on the FP8 values, of what inference will reconstruct; float32 sums over the
// group in visiting order; the smallest score wins, the lowest index among equals, and the whole range if no score is finite.
// A score is a serial sum, so the parallelism is in the rows and candidates: a workgroup takes `rows` rows and a thread one
// candidate of one of them, 128 columns in LDS as FP8 values at a time, converted once for all candidates.  With four lanes
// to a row, inside the walk, and for groups wider than 128 a conversion per candidate, 256 rows x 4096 features took 5.9 ms at
// 20 candidates in groups of 4096 and 20.6 ms at 100, now 2.3 and 2.2 (32 lanes to a row, a candidate each: 4.5 and 7.3).
constexpr int GROUP_ROWS = 32;
__global__ void __launch_bounds__(256) dpq_group_kernel(DpqArgs a, int c0, int rows) {
    __shared__ __attribute__((aligned(16))) float w8[GROUP_ROWS * TILE_STRIDE];
    __shared__ float lo[GROUP_ROWS], hi[GROUP_ROWS];
    __shared__ int has_nan[GROUP_ROWS];
    __shared__ unsigned long long best[GROUP_ROWS];              // score's bits, then candidate: squared errors order like their bits
    const int tid = threadIdx.x, lane = tid & 63;
    const int r0 = blockIdx.x * rows, count = min(rows, a.N - r0);
    const float* work = a.work + (int64_t)r0 * a.K + c0;
    auto fp8_of = [&](int r, int j) { return fp8_value(__fdiv_rn(work[(int64_t)r * a.K + j], a.s_w[a.per_channel ? r0 + r : 0])); };
    for (int r = tid >> 6; r < count; r += 4) {                  // the range, a wavefront per row
        float l = 0.0f, h = 0.0f;
        bool nan = false;
#pragma unroll 4
        for (int j = lane; j < a.G; j += 64) {
            const float v = fp8_of(r, j);
            nan |= v != v;
            l = fminf(l, v);
            h = fmaxf(h, v);
            if (a.G == DPQ_BLOCK) w8[r * TILE_STRIDE + j] = v;
        }
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            l = fminf(l, __shfl_xor(l, m));
            h = fmaxf(h, __shfl_xor(h, m));
        }
        const int any_nan = __builtin_amdgcn_ballot_w64(nan) != 0;
        if (lane == 0) {
            has_nan[r] = any_nan;
            lo[r] = l;
            hi[r] = h;
            best[r] = ~0ull;
        }
    }
    __syncthreads();
    auto candidate = [&](int r, int i, float& s, float& z) {
        const float shrink = __fsub_rn(1.0f, __fmul_rn((float)i, a.shrink_step));
        group_params(__fmul_rn(shrink, lo[r]), __fmul_rn(shrink, hi[r]), s, z);
    };
    for (int base = 0; a.mse_grid > 1 && base < count * a.mse_grid; base += 256) {
        const bool mine = base + tid < count * a.mse_grid;
        const int r = mine ? (base + tid) / a.mse_grid : 0, i = mine ? (base + tid) % a.mse_grid : 0;
        float s, z, score = 0.0f;
        candidate(r, i, s, z);
        const bool plain = __builtin_amdgcn_ballot_w64(!plain_divisor(s) || has_nan[r]) == 0;
        for (int j0 = 0; j0 < a.G; j0 += DPQ_BLOCK) {
            if (a.G > DPQ_BLOCK) {
                __syncthreads();                                 // everyone is done with the columns before
#pragma unroll 4
                for (int e = tid; e < count * DPQ_BLOCK; e += 256)
                    w8[(e >> 7) * TILE_STRIDE + (e & (DPQ_BLOCK - 1))] = fp8_of(e >> 7, j0 + (e & (DPQ_BLOCK - 1)));
                __syncthreads();
            }
            add_squared_error(w8 + r * TILE_STRIDE, s, z, plain, score);
        }
        if (mine && score < __builtin_inff())
            atomicMin(&best[r], ((unsigned long long)__float_as_uint(score) << 32) | (unsigned)i);
    }
    __syncthreads();
    if (tid < count) {
        const int NG = a.K / a.G, g = c0 / a.G;
        const int og = a.perm ? a.perm[c0] / a.G : g;
        float s, z;
        if (best[tid] == ~0ull) group_params(lo[tid], hi[tid], s, z);
        else candidate(tid, (int)(uint32_t)best[tid], s, z);
        a.scales[(int64_t)(r0 + tid) * NG + og] = s;
        a.zeros[(int64_t)(r0 + tid) * NG + og] = (uint8_t)z;
    }
}

}  // namespace

int launch_gar_permutation(const float* hdiag, int64_t K, int32_t G, int32_t* perm, hipStream_t st) {
    hipLaunchKernelGGL(gar_permutation_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, hdiag, (int)K, (int)G, perm);
    return launch_status();
}

int launch_dpq_calibrate(const float* w, const float* u, const float* s_w, int per_channel, const int32_t* perm,
                         int64_t N, int64_t K, int32_t G, uint8_t* codes, float* scales, uint8_t* zeros, void* workspace,
                         int mse_grid, float mse_max_shrink, hipStream_t st) {
    DpqArgs a;
    a.mse_grid = mse_grid;
    a.shrink_step = mse_grid > 1 ? mse_max_shrink / (float)mse_grid : 0.0f;
    a.w = w;
    a.work = static_cast<float*>(workspace);
    a.u = u; a.s_w = s_w; a.per_channel = per_channel; a.perm = perm;
    a.N = (int)N; a.K = (int)K; a.G = (int)G;
    a.codes = codes; a.scales = scales; a.zeros = zeros;
    const int row_blocks = (int)((N + ROWS - 1) / ROWS), nb = (int)(K / DPQ_BLOCK);
    auto step = [&](int c_first, int column_blocks, int c_err, int gather, int update, int block, int ready) {
        hipLaunchKernelGGL(dpq_step_kernel, dim3((unsigned)row_blocks * (unsigned)column_blocks), dim3(256), 0, st, a, c_first, c_err,
                           row_blocks, gather, update, block, ready);
        return launch_status();
    };
    auto group = [&](int c0) {                                   // the parameters of the group that starts there
        const int rows = mse_grid > 1 ? max(1, min(GROUP_ROWS, 256 / mse_grid)) : 4;
        hipLaunchKernelGGL(dpq_group_kernel, dim3((unsigned)((N + rows - 1) / rows)), dim3(256), 0, st, a, c0, rows);
        return launch_status();
    };
    // Groups of 128: a search over few candidates, or one whose passes hide behind the updates of many rows, stays with the walk;
    // otherwise the chip is idle meanwhile and a launch of its own over all rows and candidates pays for itself, at about
    // 15 us a block.  In place / in a launch of its own, ms: 4096 features, 4 candidates: 256 rows 2.06 / 2.51, 4096 rows
    // 2.39 / 3.04; 20: 256 rows 2.67 / 2.34, 2048 rows 2.75 / 2.55, 4096 rows 2.86 / 2.97, 8192 rows 3.96 / 4.41; 100: 256
    // rows 5.70 / 2.27, 8192 rows 6.30 / 5.65, 12288 rows 7.66 / 7.88, 16384 rows 9.02 / 10.1.  1024 features: 4096 rows and 20
    // candidates 0.67 / 0.62, 8192 rows 0.68 / 0.68, 16384 rows and 100 candidates 1.48 / 1.50.
    if (G == DPQ_BLOCK && (mse_grid <= 12 || N >= (int64_t)160 * mse_grid)) {
        if (int e = step(0, 1, 0, 1, 0, PARAMS_HERE, 0)) return e;
        for (int b = 1; b < nb; ++b)                             // the first update finds the other columns where they came from
            if (int e = step(b * DPQ_BLOCK, nb - b, (b - 1) * DPQ_BLOCK, b == 1, 1, PARAMS_HERE, 0)) return e;
        return W4A8_OK;
    }
    if (G == DPQ_BLOCK) {
        for (int b = 0; b < nb; ++b) {
            // the block's own columns first, with others up to 512 tiles of 64 x 128 (4096 x 4096, 20 candidates: 2.97 ms; 256
            // tiles 3.03, 768 3.08, the own columns alone 3.17); the rest beside the walk
            const int lead = b == 0 ? 1 : min(nb - b, max(1, 512 / row_blocks));
            const int c = b * DPQ_BLOCK, c_err = b > 0 ? c - DPQ_BLOCK : 0;
            if (int e = step(c, lead, c_err, b < 2, b > 0, NO_BLOCK, 0)) return e;
            if (int e = group(c)) return e;
            if (int e = step(c, b == 0 ? 1 : 1 + nb - b - lead, c_err, b < 2, b > 0, PARAMS_GIVEN, lead)) return e;
        }
        return W4A8_OK;
    }
    if (int e = step(0, nb, 0, 1, 0, NO_BLOCK, 0)) return e;
    for (int b = 0; b < nb; ++b) {
        if (b * DPQ_BLOCK % G == 0)
            if (int e = group(b * DPQ_BLOCK)) return e;
        if (int e = step(b * DPQ_BLOCK, 1, 0, 0, 0, PARAMS_GIVEN, 1)) return e;
        if (b + 1 < nb)
            if (int e = step((b + 1) * DPQ_BLOCK, nb - b - 1, b * DPQ_BLOCK, 0, 1, NO_BLOCK, 0)) return e;
    }
    return W4A8_OK;
}

}  // namespace w4a8
