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
// The products still come from the matrix unit: an outer product of one column and one row has a single term per element, added to
// an accumulator of zero, so each is rounded by itself, to nearest even, subnormal results included.  The vector
// unit is left with the subtractions: 4096 x 4096 weights 1.8 ms, with both operations there 2.3.
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

// div_by's range: weights; divisors are those of plain_divisor.  (A zero's sign, which it may turn, decides nothing here.)
constexpr uint32_t NUM_LO = 0x21800000u, NUM_SPAN = 0x5D800000u - 0x21800000u;   // bits of 2^-60, up to 2^60: weights

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

typedef float v32f __attribute__((ext_vector_type(32)));
typedef float v8f __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
constexpr int THREADS = 512;
constexpr int ROWS = 64;             // rows of a workgroup's tile; four lanes each in the chain of a block
constexpr int SEG = 32;              // columns of a block that are quantized at a stretch, and errors staged at a time
constexpr int TILE_STRIDE = DPQ_BLOCK + 4;
constexpr int PART = 12;             // staged U of a segment: [column q][lane p of the row][slot]: U[q, 4 * (q / 4 + slot) + p], 8 slots
constexpr int TILE_FLOATS = ROWS * TILE_STRIDE;
constexpr int SEG_U = SEG * 4 * PART, SEG_E = SEG * ROWS;        // U of a segment, its errors
constexpr int SLICE_FLOATS = SEG * (ROWS + DPQ_BLOCK);           // one slice of an update: errors and U
constexpr int STAGE_FLOATS = 2 * SEG_U + 2 * SEG_E > SLICE_FLOATS ? 2 * SEG_U + 2 * SEG_E : SLICE_FLOATS;

// Products of two error columns with the two rows of U that go with them, 32 x 32 each; every product is rounded by itself (an FMA with
// zero), which is what Eq. 12 asks for -- only the sign of a zero product may differ, which changes nothing but the sign of a
// weight that is zero.  a: lane l has row l % 32 of error column l / 32; b: column l % 32 of that row of U.  Registers 0 .. 15 belong
// to the first error column, 16 .. 31 to the second: row product_row, column l % 32.
__device__ __forceinline__ v32f products_32(float a, float b) { return __builtin_amdgcn_mfma_f32_32x32x1f32(a, b, v32f{}, 0, 0, 0); }
__device__ __forceinline__ int product_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
// The same for 16 rows x 32 columns: a: lane l has row l % 16 of error column l / 32, b: column 16 (l / 16 % 2) + l % 16 of that row of U.
// Registers 8 e .. 8 e + 7 belong to error column e: column 16 (v / 4 % 2) + l % 16, row 4 (l / 16) + v % 4.
__device__ __forceinline__ v16f products_16(float a, float b) { return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, v16f{}, 0, 0, 0); }

struct RowState {
    float w[8];                   // the lane's columns of the segment that are left: slot j = column 4 (done + j) + p
    float sw, y_sw, s, y_s, z;
    uint32_t span;                // NUM_SPAN, or 0 when a divisor of this row asks for the general division
};

// One weight: column q of the segment, U[q, v] for the lane's columns v from q's slot on at `u`, U[q, q] and its reciprocal
// in `d`.  Q = q % 4 is the lane of the row that owns it, in slot 0 of R.w.  For divisors and a weight in the range of div_by;
// `far` ends up at R.span or above if the weight is not.  The chain from one column to the next is thirty dependent operations; the
// updates of the slots behind the first, which the next three columns do not need, fill the gaps between them.
template <int Q>
__device__ __forceinline__ void dpq_weight(RowState& R, const float* u, float2 d, int p, float& code, uint32_t& far) {
    const float4 v0 = *reinterpret_cast<const float4*>(u), v1 = *reinterpret_cast<const float4*>(u + 4);
    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    const float w = quad_broadcast<Q>(R.w[0]);
    far = max(far, (__float_as_uint(w) & 0x7FFFFFFFu) - NUM_LO);
    const float w8 = fp8_value_finite(div_by(w, R.sw, R.y_sw));                           // Eq. 7
    const float t = __fadd_rn(div_by(w8, R.s, R.y_s), R.z);
    const float uq = __builtin_amdgcn_fmed3f(rintf(t), 0.0f, 15.0f);                      // Eq. 9
    const float w8_hat = fp8_value_finite(__fmul_rn(__fsub_rn(uq, R.z), R.s));            // Eq. 10
    const float e = div_by(__fsub_rn(w, __fmul_rn(w8_hat, R.sw)), d.x, d.y);              // Eq. 11
    // Eq. 12 inside the segment.  In the weight's own slot lanes behind it are updated, its own lane keeps the error, those before it theirs
    const float next = __fsub_rn(R.w[0], __fmul_rn(e, v[0]));
    R.w[0] = p > Q ? next : p == Q ? e : R.w[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) R.w[j] = __fsub_rn(R.w[j], __fmul_rn(e, v[j]));
    code = p == Q ? uq : code;
}

// The same for any values (zeros, extreme ones): the general division.
__device__ __forceinline__ void dpq_weight_general(RowState& R, int Q, const float* u, float d, int p, int lane, float& code) {
    const float w = __shfl(R.w[0], (lane & ~3) | Q);
    const float g8 = fp8_value(__fdiv_rn(w, R.sw));
    const float uq = fminf(fmaxf(rintf(__fadd_rn(__fdiv_rn(g8, R.s), R.z)), 0.0f), 15.0f);
    const float g8_hat = fp8_value(__fmul_rn(__fsub_rn(uq, R.z), R.s));
    const float e = __fdiv_rn(__fsub_rn(w, __fmul_rn(g8_hat, R.sw)), d);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float next = __fsub_rn(R.w[j], __fmul_rn(e, u[j]));
        R.w[j] = j > 0 ? next : p > Q ? next : p == Q ? e : R.w[j];
    }
    code = p == Q ? uq : code;
}

// What becomes of the first column block's tiles: written to `work` like the others, or quantized with the group's parameters,
// formed from the tile (groups of one block) or found in the outputs (where dpq_group_kernel put them).
enum BlockStep { NO_BLOCK = 0, PARAMS_HERE = 1, PARAMS_GIVEN = 2 };

// A slice of an update: 32 errors of the tile's rows from r0 on and the 32 rows of U that go with them, the tile's 128 columns, on their
// way to LDS.  el[q * 64 + r]: error q of row r; ul[q * 128 + c]: U[c_err + q, v0 + c].
struct Slice {
    float e[4], u[8];
    __device__ __forceinline__ void load(const DpqArgs& a, int r0, int c_err, int v0, int q0, int tid) {
        const float* er = a.work + (int64_t)min(r0 + (tid & 63), a.N - 1) * a.K + c_err + q0 + (tid >> 6) * 4;
        const float* ur = a.u + (int64_t)(c_err + q0 + (tid >> 4)) * a.K + v0 + (tid & 15) * 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] = er[j];
#pragma unroll
        for (int j = 0; j < 8; ++j) u[j] = ur[j];
    }
    __device__ __forceinline__ void store(float* el, float* ul, int tid) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) el[((tid >> 6) * 4 + j) * ROWS + (tid & 63)] = e[j];
        float* d = ul + (tid >> 4) * DPQ_BLOCK + (tid & 15) * 8;
        *reinterpret_cast<float4*>(d) = make_float4(u[0], u[1], u[2], u[3]);
        *reinterpret_cast<float4*>(d + 4) = make_float4(u[4], u[5], u[6], u[7]);
    }
};

// One launch of the walk.  Workgroups own tiles of 64 rows x 128 columns of the columns from c_first on, the tiles of the
// first column block coming first:
//   gather:  the tile comes from the original weights, reordered; otherwise from `work`;
//   update:  it receives the errors of the block at c_err (Eq. 12 for the columns right of a block: for every column q of
//            that block, ascending, w <- w - err[n, q] * U[c_err + q, v]);
//   block:   the tiles of the first column block are then quantized, column by column, the others written to `work`;
//   ready:   a launch before has brought that many column blocks up to date: the first is only quantized, the other ones skipped.
// With groups of 128 one launch does the first three: the next block is quantized by the workgroups that bring it up to date
// while the others update the rest, so the serial part hides behind the updates for as long as there are many.  With a scale search in a
// launch of its own the block's columns are brought up to date in a launch before that.  Wider groups need all of their columns up to
// date before the first is quantized: an update and a block launch each.
// Update: the products come from the matrix unit, one outer product per error column, so that the vector unit is left with the
// subtractions.  The first update of 4096 x 4096 (1984 tiles, 2.1 G products) takes 106 us, of which loading and storing the tiles is about a
// third; 112 us with both operations on the vector unit, where the serial part did not hide behind it.
// Block: 32 columns at a time.  Lane p of a row's four holds the columns v with v % 4 == p of a segment in registers; every lane takes the
// (identical) quantization step and applies the error to its own columns.  The columns of the later segments take the segment's 32
// errors afterwards, on the matrix unit: those of the next one before it begins, the others by the four wavefronts that have no rows, beside the
// chain.  A wavefront alone on its SIMD issues one vector operation every five cycles, so what a column costs is their number: 60,
// with all later columns of the block in registers 100 on average.  32 lanes per row, with the weights in LDS, spent most
// instructions on repeating the quantization step.  A launch whose updates are few takes 38 us (256 x 4096 in all 1.22 ms, before
// 1.89 ms); 4096 x 4096 takes 1.8 ms, before 2.3 ms, and 16384 x 4096 5.7 ms, before 6.4 ms.  Where weights or scales ask for the general division in
// every step of four (rows of zeros, rows at 1e-30) 4096 x 4096 takes 2.2 ms, before 2.4.
__global__ void __launch_bounds__(THREADS, 4) dpq_step_kernel(DpqArgs a, int c_first, int c_err, int row_blocks, int gather, int update, int block,
                                                              int ready) {
    __shared__ __attribute__((aligned(16))) float lds[TILE_FLOATS + STAGE_FLOATS];
    __shared__ float2 diag[2][SEG];
    __shared__ int cols[DPQ_BLOCK];                              // original columns of the block
    __shared__ int general[2];                                   // a diagonal entry of the staged segment asks for the general division
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, lc = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* const stage = lds + TILE_FLOATS;
    const int rb = blockIdx.x % row_blocks, cb = blockIdx.x / row_blocks;
    const bool quantize = block && cb == 0;
    if (quantize) __builtin_amdgcn_s_setprio(2);                 // ahead of the update's wavefronts on the same SIMD
    if (ready > 0 && cb == 0) gather = update = 0;
    const int r0 = rb * ROWS, v0 = c_first + (ready > 0 && cb > 0 ? cb + ready - 1 : cb) * DPQ_BLOCK, c0 = c_first;
    {
        // a wavefront has 32 rows x 32 columns of the tile
        const int wr = (wave >> 2) * 32, wc = (wave & 3) * 32, col = v0 + wc + lc;
        v16f w;
        const int64_t from = (gather && a.perm) ? a.perm[col] : col;
        const float* src = gather ? a.w : a.work;
#pragma unroll
        for (int v = 0; v < 16; ++v)                             // rows past the end repeat the last one; not stored
            w[v] = src[(int64_t)min(r0 + wr + product_row(v, lane), a.N - 1) * a.K + from];
        if (update) {
            float *el = stage, *ul = stage + SEG * ROWS;
            const float *ea = el + half * ROWS + wr + lc, *ua = ul + half * DPQ_BLOCK + wc + lc;
            Slice slice;
            slice.load(a, r0, c_err, v0, 0, tid);
            for (int q0 = 0; q0 < DPQ_BLOCK; q0 += SEG) {
                __syncthreads();                                 // everyone is done with the slice before
                slice.store(el, ul, tid);
                __syncthreads();
                if (q0 + SEG < DPQ_BLOCK) slice.load(a, r0, c_err, v0, q0 + SEG, tid);
                v32f p = products_32(ea[0], ua[0]);
#pragma unroll 4
                for (int q = 0; q < SEG; q += 2) {
                    const int qn = q + 2 < SEG ? q + 2 : q;      // the next products are formed while these are subtracted
                    v32f next = products_32(ea[qn * ROWS], ua[qn * DPQ_BLOCK]);
                    asm volatile("" : "+v"(next), "+v"(w)); // ... which keeps the order as written
#pragma unroll
                    for (int v = 0; v < 16; ++v) w[v] = __fsub_rn(w[v], p[v]);
#pragma unroll
                    for (int v = 0; v < 16; ++v) w[v] = __fsub_rn(w[v], p[16 + v]);
                    p = next;
                }
            }
        }
        if (!quantize) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int n = r0 + wr + product_row(v, lane);
                if (n < a.N) a.work[(int64_t)n * a.K + col] = w[v];
            }
            return;
        }
        if (update) __syncthreads();                             // the last slice has been read by everyone
#pragma unroll
        for (int v = 0; v < 16; ++v) lds[(wr + product_row(v, lane)) * TILE_STRIDE + wc + lc] = w[v];
    }
    float* const seg_u = stage;                                  // + (segment & 1) * SEG_U
    float* const seg_e = stage + 2 * SEG_U;                      // + (segment & 1) * SEG_E: [q][64 rows]
    // The rows of U of segment sg, columns of the segment, by 256 threads: four values each of row t / 8
    auto stage_u = [&](int sg, int t) {
        const int q = t >> 3, first = (t & 7) * 4;
        const float* ur = a.u + (int64_t)(c0 + sg * SEG + q) * a.K + c0 + sg * SEG + first;
        float* dst = seg_u + (sg & 1) * SEG_U;
        const int slot = (t & 7) - (q >> 2);                     // what lies left of the row's own slot goes to a slot that nobody reads
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(q * 4 + j) * PART + (slot >= 0 ? slot : PART - 1)] = ur[j];
        // (slots past a row's last are read too, for columns of R.w that are done: values of no account)
        if (t < SEG) {
            const float ud = a.u[(int64_t)(c0 + sg * SEG + t) * (a.K + 1)];
            diag[sg & 1][t] = make_float2(ud, __fdiv_rn(1.0f, ud));
            const bool odd_one = __builtin_amdgcn_ballot_w64(!plain_divisor(ud)) != 0;
            if (t == 0) general[sg & 1] = odd_one;
        }
    };
    // tile -= products of segment sg's errors, for the 32 columns of segment `to`, rows wr .. wr + 15, by one wavefront: U first, the rest when
    // the errors are there
    const int blk = (lane >> 4) & 1, l16 = lane & 15;
    float uv[SEG / 2];
    auto fetch_u = [&](int sg, int to) {
        const float* ur = a.u + (int64_t)(c0 + sg * SEG + half) * a.K + c0 + to * SEG + 16 * blk + l16;
#pragma unroll
        for (int q = 0; q < SEG / 2; ++q) uv[q] = ur[(int64_t)(2 * q) * a.K];
    };
    auto push_errors = [&](int sg, int to, int wr) {
        const float* el = seg_e + (sg & 1) * SEG_E + half * ROWS + wr + l16;
        float* t = lds + (wr + 4 * (lane >> 4)) * TILE_STRIDE + to * SEG + l16;
        v8f w;
#pragma unroll
        for (int v = 0; v < 8; ++v) w[v] = t[(v & 3) * TILE_STRIDE + 16 * (v >> 2)];
        v16f p = products_16(el[0], uv[0]);
#pragma unroll
        for (int q = 0; q < SEG / 2; ++q) {
            const int qn = q + 1 < SEG / 2 ? q + 1 : q;
            v16f next = products_16(el[2 * qn * ROWS], uv[qn]);
            asm volatile("" : "+v"(next), "+v"(w));         // keeps the order as written
#pragma unroll
            for (int v = 0; v < 8; ++v) w[v] = __fsub_rn(w[v], p[v]);
#pragma unroll
            for (int v = 0; v < 8; ++v) w[v] = __fsub_rn(w[v], p[8 + v]);
            p = next;
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) t[(v & 3) * TILE_STRIDE + 16 * (v >> 2)] = w[v];
    };
    // wavefronts 0 .. 3: lane p of row r; wavefronts 4 .. 7 prepare what comes next
    const bool chain = wave < 4;
    const int r = (tid >> 2) & (ROWS - 1), p = tid & 3;
    const int64_t n = min(r0 + r, a.N - 1);
    const bool row_ok = r0 + r < a.N;
    if (!chain) {
        stage_u(0, tid - 256);
    } else if (tid < DPQ_BLOCK) {
        cols[tid] = a.perm ? a.perm[c0 + tid] : c0 + tid;
    }
    __syncthreads();
    RowState R;
    float* mine = lds + r * TILE_STRIDE;
    if (chain) {
        R.sw = a.s_w[a.per_channel ? n : 0];
        const int NG = a.K / a.G, g = c0 / a.G;
        const int og = a.perm ? a.perm[g * a.G] / a.G : g;       // the original group these columns belong to
        float s, z;
        if (block == PARAMS_HERE) {                              // Eq. 8 on the group's current weights, which are the tile's
            float lo = 0.0f, hi = 0.0f;                          // minimum and maximum: any order gives the same result
            bool nan = false;
#pragma unroll 4
            for (int j = p; j < DPQ_BLOCK; j += 4) {
                const float w8 = fp8_value(__fdiv_rn(mine[j], R.sw));
                lo = fminf(lo, w8);
                hi = fmaxf(hi, w8);
                nan |= w8 != w8;
            }
#pragma unroll
            for (int m = 1; m < 4; m <<= 1) {
                lo = fminf(lo, __shfl_xor(lo, m));
                hi = fmaxf(hi, __shfl_xor(hi, m));
            }
            group_params(lo, hi, s, z);
            if (a.mse_grid > 1) {                                // the search of dpq_group_kernel, a row's lanes sharing the candidates
                float keep[32];                                  // the search scores FP8 values, which stand in the weights' place meanwhile
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    keep[j] = mine[4 * j + p];
                    mine[4 * j + p] = fp8_value(__fdiv_rn(keep[j], R.sw));
                }
                __builtin_amdgcn_wave_barrier();                 // a row's lanes lie in one wavefront, whose LDS accesses run in order
                float best = __builtin_inff(), bs = s, bz = z;
                int best_i = a.mse_grid;
                for (int i = p; i < a.mse_grid; i += 4) {
                    const float shrink = __fsub_rn(1.0f, __fmul_rn((float)i, a.shrink_step));
                    float si, zi, score = 0.0f;
                    group_params(__fmul_rn(shrink, lo), __fmul_rn(shrink, hi), si, zi);
                    add_squared_error(mine, si, zi, __builtin_amdgcn_ballot_w64(!plain_divisor(si) || nan) == 0, score);
                    if (score < best) { best = score; best_i = i; bs = si; bz = zi; }
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = 0; j < 32; ++j) mine[4 * j + p] = keep[j];
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
    }
    constexpr int SEGS = DPQ_BLOCK / SEG;
#pragma unroll 1
    for (int sg = 0; sg < SEGS; ++sg) {
        if (chain) {
            const float* u = seg_u + (sg & 1) * SEG_U + p * PART;
            const float2* d = diag[sg & 1];
            const bool diag_plain = general[sg & 1] == 0;
            float* el = seg_e + (sg & 1) * SEG_E;
#pragma unroll
            for (int j = 0; j < 8; ++j) R.w[j] = mine[sg * SEG + 4 * j + p];
            // a loop of four weights: unrolled, the code of a block takes longer to fetch than to run
#pragma unroll 1
            for (int t = 0; t < SEG / 4; ++t, u += 16 * PART, d += 4) {
                float code = 0.0f;
                const int col = cols[sg * SEG + 4 * t + p];
                const RowState before = R;
                uint32_t far = diag_plain ? 0u : ~0u;
                dpq_weight<0>(R, u, d[0], p, code, far);
                dpq_weight<1>(R, u + 4 * PART, d[1], p, code, far);
                dpq_weight<2>(R, u + 8 * PART, d[2], p, code, far);
                dpq_weight<3>(R, u + 12 * PART, d[3], p, code, far);
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(far >= R.span) != 0, 0)) {   // once more, by the general division
                    R = before;
                    code = 0.0f;
#pragma unroll 1
                    for (int q = 0; q < 4; ++q) dpq_weight_general(R, q, u + 4 * PART * q, d[q].x, p, lane, code);
                }
                el[(4 * t + p) * ROWS + r] = R.w[0];
                if (row_ok) {
                    a.work[n * a.K + c0 + sg * SEG + 4 * t + p] = R.w[0];
                    a.codes[n * a.K + col] = (uint8_t)code;
                }
#pragma unroll
                for (int j = 0; j + 1 < 8; ++j) R.w[j] = R.w[j + 1];
            }
        } else {
            if (sg + 1 < SEGS) stage_u(sg + 1, tid - 256);
            const int wr = (wave - 4) * 16;
            // the errors of the segment before this one, for the segments after this one
            if (sg > 0)
                for (int to = sg + 1; to < SEGS; ++to) {
                    fetch_u(sg - 1, to);
                    push_errors(sg - 1, to, wr);
                }
            if (sg + 1 < SEGS) fetch_u(sg, sg + 1);              // there when this segment's errors are
        }
        __syncthreads();
        if (sg + 1 < SEGS && !chain) push_errors(sg, sg + 1, (wave - 4) * 16);
        __syncthreads();
    }
}

// Group parameters of the group at columns c0 .. c0 + G - 1, which `work` holds up to date: Eq. 8 on the FP8 values, and with
// mse_grid > 1 the scale search of Sec. 3.3 (the paper names it, not its grid): candidate i shrinks the range by p_i = 1 - i *
// shrink_step and is scored by the squared error, on the FP8 values, of what inference will reconstruct; float32 sums over the
// group in visiting order; the smallest score wins, the lowest index among equals, and the whole range if no score is finite.
// A score is a serial sum, so the parallelism is in the rows and candidates: a workgroup takes `rows` rows and a thread one
// candidate of one of them, 128 columns in LDS as FP8 values at a time, converted once for all candidates.  With four lanes
// to a row, inside the walk, and for groups wider than 128 a conversion per candidate, 256 rows x 4096 features took 5.9 ms at
// 20 candidates in groups of 4096 and 20.6 ms at 100, now 1.5 and 1.4 (32 lanes to a row, a candidate each, on the walk before: 4.5 and 7.3, against 2.3 and 2.2).
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
        hipLaunchKernelGGL(dpq_step_kernel, dim3((unsigned)row_blocks * (unsigned)column_blocks), dim3(THREADS), 0, st, a, c_first, c_err,
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
    // 15 us a block.  In place / in a launch of its own, ms: 4096 features, 4 candidates: 256 rows 1.43 / 1.76; 12: 256 rows 1.72 / 1.71,
    // 4096 rows 2.12 / 2.38; 20: 256 rows 2.01 / 1.61, 2048 rows 2.16 / 1.79, 4096 rows 2.33 / 2.35, 8192 rows 3.45 / 3.72; 100: 256
    // rows 4.98 / 1.53, 8192 rows 5.64 / 4.96, 12288 rows 6.88 / 7.13, 16384 rows 8.63 / 9.32.  14336 features, 4096 rows, 20 candidates
    // 18.0 / 18.7.  1024 features: 4096 rows and 20 candidates 0.52 / 0.44, 8192 rows 0.54 / 0.50, 16384 rows and 100 candidates 1.34 / 1.36.
    if (G == DPQ_BLOCK && (mse_grid <= 12 || N >= (int64_t)160 * mse_grid)) {
        if (int e = step(0, 1, 0, 1, 0, PARAMS_HERE, 0)) return e;
        for (int b = 1; b < nb; ++b)                             // the first update finds the other columns where they came from
            if (int e = step(b * DPQ_BLOCK, nb - b, (b - 1) * DPQ_BLOCK, b == 1, 1, PARAMS_HERE, 0)) return e;
        return W4A8_OK;
    }
    if (G == DPQ_BLOCK) {
        for (int b = 0; b < nb; ++b) {
            // the block's own columns first, with others up to 256 tiles of 64 x 128 (4096 x 4096, 20 candidates: 2.35 ms; 512 tiles
            // 2.41, 768 2.49; 2048 rows 1.79, 1.92, 2.02); the rest beside the walk
            const int lead = b == 0 ? 1 : min(nb - b, max(1, 256 / row_blocks));
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
