// Offline calibration: from the Hessian H = X^T X of the layer-wise objective (Eq. 5, App. A.2) to the matrix U that
// carries the updates of Eq. 12 -- dampening and Cholesky factorization (Sec. 3.3).
//
// U is the upper-triangular factor of the inverse dampened Hessian, H_d^-1 = U^T U.  It is reached without forming
// H_d^-1: with J the index reversal, the lower Cholesky factor L of J H_d J gives H_d = R R^T with R = J L J upper
// triangular, hence H_d^-1 = (R^-1)^T R^-1 and U = R^-1 = J L^-1 J (the factor with positive diagonal is unique).
// So the work is one blocked Cholesky factorization and one triangular inversion, both in float64 on 64 x 64 tiles (the
// Hessian arrives as float32, and U leaves as float32), multiplied on the float64 matrix unit (16x16x4; its rate is that of
// the vector unit, but a wavefront's 32 x 32 share of a tile takes a third of the LDS reads of 4 x 4 outputs per thread):
//   factorization, for each pair of tile columns k, k + 1:  scale the tiles of column k by the inverse of its diagonal
//     factor;  subtract its outer product from column k + 1;  scale column k + 1;  subtract the outer product of both (128
//     deep: the trailing matrix is read and written once per pair) from every tile to the right.  What a step waits for is
//     the next diagonal tile, so the workgroup that updates it goes on to factor and invert it, while the others still
//     work on the rest of the matrix;
//   inversion X = L^-1, by forward substitution in the same launches, one pair of columns behind:  X[k, :] = L_kk^-1 R[k, :]
//     with R = I minus the products of the rows above.  Once X[k, :] and X[k + 1, :] are there, all rows of R below take their
//     products (128 deep) in the launch that updates the single column k + 3, which waits for its diagonal tile and
//     leaves the chip idle otherwise.
// Every step is one launch over independent tiles, so no kernel waits on another workgroup.
// 4096 features take 2.0 ms; before the present factor_tile, and with two workgroups to a unit instead of three (118 + 32 registers
// per lane in trailing_update_kernel), 2.5 ms.  The 46 GFLOP would
// take 1.05 ms at the 43 TFLOP/s that the float64 matrix unit reaches on the whole chip.  What a diagonal tile waits for: 5.5 us for its panel,
// 13 us (64 deep) or 16 us (128 deep) for the launch that updates, factors and inverts it, 1.3 ms over all.  The launches of the middle columns take 20 to 31 us for
// their products, those of the first up to 50 us; the others wait for the diagonal tile.
// (Tiles handed to the dies in compact regions, and a higher priority for the workgroup with the diagonal tile, gave nothing.)
#include "w4a8_device.hpp"
#include "w4a8_internal.hpp"

namespace w4a8 {
namespace {

constexpr int TB = 64;              // tile edge
constexpr int KS = 32;              // depth of one staged slice
constexpr int LDA = KS + 2;         // row stride of a slice [64][KS] (k contiguous): rows 4 banks apart, free of conflicts
constexpr int LDT = TB + 2;         // row stride of a whole tile, and of a slice [KS][64]

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

// LDS of a workgroup: two slices while it multiplies; then, if it factors, the tile
constexpr int SLICE = TB * LDA;
constexpr int LDS_DOUBLES = 2 * SLICE;
static_assert(TB * LDT <= LDS_DOUBLES, "the tile fits");

// scalars[0] = damp * mean(diag(H)); *info = 0.  One workgroup; a fixed summation order.
__global__ void __launch_bounds__(256) damp_term_kernel(const float* __restrict__ h, int n, double damp, double* __restrict__ scalars,
                                                        int32_t* __restrict__ info) {
    __shared__ double part[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += (double)h[(int64_t)i * n + i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        scalars[0] = damp * part[0] / (double)n;
        *info = 0;
    }
}

// a[i, j] = H_d[p(n-1-i), p(n-1-j)] for j <= i (the lower triangle of the reversed, reordered, dampened Hessian); one
// workgroup per row
__global__ void __launch_bounds__(256) gather_reversed_kernel(const float* __restrict__ h, const int32_t* __restrict__ perm, int n,
                                                              const double* __restrict__ scalars, double* __restrict__ a) {
    const int i = blockIdx.x;
    const int oi = perm ? perm[n - 1 - i] : n - 1 - i;
    for (int j = threadIdx.x; j <= i; j += 256) {
        const int oj = perm ? perm[n - 1 - j] : n - 1 - j;
        double v = (double)h[(int64_t)oi * n + oj];
        if (i == j) v += scalars[0];
        a[(int64_t)i * n + j] = v;
    }
}

// One lane's share of C(16 x 16) += A(16 x 16) B(16 x 16) on the float64 matrix unit.  Lane (i, g) = (lane % 16, lane / 16)
// gives A's row i and B's column i at four values of k, taken as two pairs of neighbours (the order of k is free as
// long as both operands agree), and holds C's column i, rows g + 4 r.
// a: A(i, k) = a[i * lda + k].  b: B(k, i) = b[i * ldb + k] (B_KFAST) or b[k * ldb + i].
template <bool B_KFAST>
__device__ __forceinline__ void block_mac(v4d& acc, const double* a, int lda, const double* b, int ldb, int lane) {
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int k = 8 * s + 2 * g;
        const v2d av = *reinterpret_cast<const v2d*>(a + i * lda + k);
        v2d bv;
        if (B_KFAST) bv = *reinterpret_cast<const v2d*>(b + i * ldb + k);
        else bv = v2d{b[k * ldb + i], b[(k + 1) * ldb + i]};
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[0], bv[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[1], bv[1], acc, 0, 0, 0);
    }
}

// 1 / sqrt(d) to within an ulp or two: the hardware's estimate (23 bits) and one third-order step.
// Not finite for d <= 0 and NaN.
__device__ __forceinline__ double inv_sqrt(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// 1 / d likewise
__device__ __forceinline__ double inverse(double d) {
    const double y = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// v of lane LANE of each 16 lanes.  What a lane permutation reads must have been written two wait states before; the compiler sees to
// that only between instructions of its own, so each of these begins with the wait.
template <int LANE>
__device__ __forceinline__ double row_broadcast(double v) {
    double r;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v), "n"(LANE));
    return r;
}

// d[Q + u] += d[J](lane Q + u of each 16) * m for u < COUNT
template <int J, int Q, int COUNT>
__device__ __forceinline__ void eliminate_columns(double (&d)[16], double m) {
#define FMA_ROW_BROADCAST(acc, source, lane) "v_fmac_f64_dpp " acc ", " source ", %[m] row_newbcast:" lane " row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (COUNT >= 4) {
        asm("s_nop 1\n\t" FMA_ROW_BROADCAST("%0", "%[s]", "%[l0]") FMA_ROW_BROADCAST("%1", "%[s]", "%[l1]") FMA_ROW_BROADCAST("%2", "%[s]", "%[l2]")
                FMA_ROW_BROADCAST("%3", "%[s]", "%[l3]")
            : "+&v"(d[Q]), "+&v"(d[Q + 1]), "+&v"(d[Q + 2]), "+&v"(d[Q + 3])
            : [s] "v"(d[J]), [m] "v"(m), [l0] "n"(Q), [l1] "n"(Q + 1), [l2] "n"(Q + 2), [l3] "n"(Q + 3));
        eliminate_columns<J, Q + 4, COUNT - 4>(d, m);
    } else if constexpr (COUNT > 0) {
        asm("s_nop 1\n\t" FMA_ROW_BROADCAST("%0", "%[s]", "%[l0]") : "+v"(d[Q]) : [s] "v"(d[J]), [m] "v"(m), [l0] "n"(Q));
        eliminate_columns<J, Q + 1, COUNT - 1>(d, m);
    }
}

// x[u] += x[u](lane J of each 16) * m
template <int J>
__device__ __forceinline__ void eliminate_identity(double (&x)[4], double m) {
    asm("s_nop 1\n\t" FMA_ROW_BROADCAST("%0", "%0", "%[l]") FMA_ROW_BROADCAST("%1", "%1", "%[l]") FMA_ROW_BROADCAST("%2", "%2", "%[l]")
            FMA_ROW_BROADCAST("%3", "%3", "%[l]")
        : "+&v"(x[0]), "+&v"(x[1]), "+&v"(x[2]), "+&v"(x[3])
        : [m] "v"(m), [l] "n"(J));
#undef FMA_ROW_BROADCAST
}

// Pivot J and those after it, of a 16 x 16 block in L~ D L~^T form: d[c] is column c of row i = lane % 16, x[u] column 4 (lane / 16) + u of L~^-1's row
// i, both rows being in every 16 lanes (d) or spread over them (x).  `pivot` receives the row's own pivot.
template <int J>
struct Eliminate {
    static __device__ __forceinline__ void run(double (&d)[16], double (&x)[4], double& pivot, int i) {
        const double p = row_broadcast<J>(d[J]);
        pivot = i == J ? p : pivot;
        const double m = i > J ? -(d[J] * inverse(p)) : 0.0;          // rows up to the pivot's stay as they are
        // the next pivot's column first, then whole fours
        eliminate_columns<J, J + 1, 1>(d, m);
        eliminate_columns<J, J + 2, 14 - J>(d, m);
        eliminate_identity<J>(x, m);
        Eliminate<J + 1>::run(d, x, pivot, i);
    }
};
template <>
struct Eliminate<15> {
    static __device__ __forceinline__ void run(double (&d)[16], double (&)[4], double& pivot, int i) {
        const double p = row_broadcast<15>(d[15]);
        pivot = i == 15 ? p : pivot;
    }
};

// Diagonal tile kb, whose lower triangle lies in `t` (row stride LDT): dinv[kb], row-major 64 x 64, and x[kb, kb] <- V = L^-1 with L its
// lower Cholesky factor (zeros above the diagonal; L itself is not needed).  A pivot that is not positive is
// reported through *info (1 + its index in the reversed order, first failure only); the results are then not finite.
// This is the serial part of the factorization: 64 pivots, each waiting for the one before.  16 at a time: one wavefront
// brings the 16 x 16 diagonal block up to date with the columns just finished and turns it into the inverse of its factor, the block's rows
// being in each 16 lanes, so that a pivot reaches the others as an operand of the multiply-add itself (a lane broadcast within
// 16 lanes): 22 vector operations a pivot, neither a barrier nor a trip through LDS.  The other three meanwhile apply
// the columns just finished to the rest of the tile, a row of blocks each, and form the rows of V, a block each.
// With P = V_pp A(r, p)^T = L(r, p)^T no product waits for a transposed operand: the matrix unit's result has the layout of
// both its operands.  Block (r, c) of the tile is A's, then V's for c <= r, and L(c, r)^T for c > r.
// 19 thousand cycles a tile, 8 us, half of them for the pivots (150 each); 40 thousand, 17 us, with panels of 64 rows factored by one wavefront, a
// row per lane and every value broadcast through scalar registers, and the inverse put together afterwards.
__device__ __forceinline__ void factor_tile(double* t, int n, int kb, double* __restrict__ dinv, double* __restrict__ x, int32_t* __restrict__ info) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    auto blk = [&](int r, int c) { return t + r * 16 * LDT + c * 16; };
    auto l_transposed = [&](int r, int p) {                      // P[k][r's row]: rows g + 4 e, column i
        v4d acc = {0.0, 0.0, 0.0, 0.0};
        block_mac<true>(acc, blk(p, p), LDT, blk(r, p), LDT, lane);
        return acc;
    };
    auto subtract_product = [&](int r, int c, const v4d& pr, const v4d& pc) {
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pr[e], pc[e], acc, 0, 0, 0);
        double* to = blk(r, c) + g * LDT + i;
#pragma unroll
        for (int e = 0; e < 4; ++e) to[4 * e * LDT] -= acc[e];
    };
    auto store_block = [&](int r, int c, const v4d& v, double sign) {
        double* to = blk(r, c) + g * LDT + i;
#pragma unroll
        for (int e = 0; e < 4; ++e) to[4 * e * LDT] = sign * v[e];
    };
    auto inverse_block = [&](int r, int c) {                     // V(r, c) = -V(r, r) sum over q of L(r, q) V(q, c)
        v4d m = {0.0, 0.0, 0.0, 0.0}, v = {0.0, 0.0, 0.0, 0.0};
        for (int q = c; q < r; ++q) {
            const double *l = blk(q, r) + g * LDT + i, *vq = blk(q, c) + g * LDT + i;
#pragma unroll
            for (int e = 0; e < 4; ++e) m = __builtin_amdgcn_mfma_f64_16x16x4f64(l[4 * e * LDT], vq[4 * e * LDT], m, 0, 0, 0);
        }
        const double* vr = blk(r, r) + i * LDT + g;
#pragma unroll
        for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f64_16x16x4f64(vr[4 * e], m[e], v, 0, 0, 0);
        store_block(r, c, v, -1.0);
    };
    for (int jb = 0; jb <= 4; ++jb) {
        const int p = jb - 1;                                    // the columns just finished
        if (wave == 0 && jb < 4) {
            double* b = blk(jb, jb);
            if (p >= 0) {
                const v4d pj = l_transposed(jb, p);
                subtract_product(jb, jb, pj, pj);
                __builtin_amdgcn_wave_barrier();                 // LDS accesses of a wavefront run in order
            }
            double d[16], v[4], pivot = 0.0;
#pragma unroll
            for (int c = 0; c < 16; c += 2) {
                const v2d two = *reinterpret_cast<const v2d*>(b + i * LDT + c);
                d[c] = two[0];
                d[c + 1] = two[1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = i == 4 * g + u ? 1.0 : 0.0;
            Eliminate<0>::run(d, v, pivot, i);
            const double rs = inv_sqrt(pivot);
#pragma unroll
            for (int u = 0; u < 4; u += 2) *reinterpret_cast<v2d*>(b + i * LDT + 4 * g + u) = v2d{rs * v[u], rs * v[u + 1]};
            const uint32_t bad = (uint32_t)__builtin_amdgcn_ballot_w64(!(pivot > 0.0)) & 0xFFFFu;
            if (bad && lane == 0 && *info == 0) *info = kb * TB + jb * 16 + __builtin_ctz(bad) + 1;
        } else if (wave > 0 && p >= 0) {
            if (wave > p) {                                      // blocks (wave, p + 1 ..) of the tile; wavefront 0 has (p + 1, p + 1)
                const v4d pr = l_transposed(wave, p);
                for (int c = p + 1; c <= wave; ++c)
                    if (!(wave == p + 1 && c == p + 1)) subtract_product(wave, c, pr, l_transposed(c, p));
                store_block(p, wave, pr, 1.0);
            } else {
                inverse_block(p, wave - 1);
            }
        }
        __syncthreads();
    }
    // V, zeros above the diagonal
    double* dv = dinv + (int64_t)kb * TB * TB;
#pragma unroll
    for (int u = 0; u < TB * TB / 512; ++u) {
        const int idx = tid + u * 256, r = idx >> 5, c = (idx & 31) * 2;
        const v2d v = (c >> 4) <= (r >> 4) ? *reinterpret_cast<const v2d*>(t + r * LDT + c) : v2d{0.0, 0.0};
        *reinterpret_cast<v2d*>(dv + r * TB + c) = v;
        *reinterpret_cast<v2d*>(x + ((int64_t)kb * TB + r) * n + (int64_t)kb * TB + c) = v;
    }
}

// acc (a wavefront's 2 x 2 blocks of 16 x 16: rows 32 (wave / 2).., columns 32 (wave % 2)..) += A B for a 64 x 64 tile.
// A(r, k) = ap[r * ars + k].  B(k, c): bp(k0) is the address of the slice k0 .. k0 + KS - 1, B(k0 + k, c) there at
// c * brs + k (B_KFAST) or k * brs + c.  depth is a multiple of KS.  A slice is loaded into registers while the one before
// is multiplied; last() may load what is needed after the product beside the last one, in the same
// registers.  Ends with a barrier after the last slice has been consumed: LDS and operand tiles may be overwritten.
template <bool B_KFAST, typename BP, typename LAST>
__device__ __forceinline__ void tile_mac(v4d (&acc)[2][2], const double* ap, int ars, BP&& bp, int brs, int depth, double* lds, LAST&& last) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    double* as = lds;
    double* bs = lds + SLICE;
    v2d ra[4], rb[4];
    // one offset per lane and operand, the rest of an address is uniform
    const uint32_t from_a = (uint32_t)((tid >> 4) * ars + (tid & 15) * 2);
    const uint32_t from_b = (uint32_t)(B_KFAST ? (tid >> 4) * brs + (tid & 15) * 2 : (tid >> 5) * brs + (tid & 31) * 2);
    auto load = [&](int k0) {
        const double* b = bp(k0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ra[u] = *reinterpret_cast<const v2d*>(ap + (int64_t)(16 * u) * ars + k0 + from_a);
            rb[u] = *reinterpret_cast<const v2d*>(b + (int64_t)((B_KFAST ? 16 : 8) * u) * brs + from_b);
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = tid + u * 256;
            *reinterpret_cast<v2d*>(as + (id >> 4) * LDA + (id & 15) * 2) = ra[u];
            if (B_KFAST) *reinterpret_cast<v2d*>(bs + (id >> 4) * LDA + (id & 15) * 2) = rb[u];
            else *reinterpret_cast<v2d*>(bs + (id >> 5) * LDT + (id & 31) * 2) = rb[u];
        }
    };
    auto multiply = [&]() {
        const double* pa = as + ((wave >> 1) * 32 + i) * LDA + 2 * g;
        const double* pb = B_KFAST ? bs + ((wave & 1) * 32 + i) * LDA + 2 * g : bs + 2 * g * LDT + (wave & 1) * 32 + i;
#pragma unroll
        for (int s = 0; s < KS / 8; ++s) {
            v2d av[2], bv[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                av[e] = *reinterpret_cast<const v2d*>(pa + e * 16 * LDA + 8 * s);
                if (B_KFAST) bv[e] = *reinterpret_cast<const v2d*>(pb + e * 16 * LDA + 8 * s);
                else bv[e] = v2d{pb[8 * s * LDT + e * 16], pb[(8 * s + 1) * LDT + e * 16]};
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x][h], bv[y][h], acc[x][y], 0, 0, 0);
        }
    };
    load(0);
    for (int k0 = KS; k0 < depth; k0 += KS) {
        store();
        __syncthreads();
        load(k0);
        multiply();
        __syncthreads();
    }
    store();
    __syncthreads();
    last();
    multiply();
    __syncthreads();
}
static_assert(KS * LDT <= SLICE, "a slice in either order fits");

// f(value, address) for every element this lane holds of a tile with row stride `stride` (n: tiles of the matrices): one offset per
// lane, the rest of the address is uniform
template <typename F>
__device__ __forceinline__ void each_element(v4d (&acc)[2][2], double* tile, int stride, F&& f) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
    const uint32_t mine = (uint32_t)(g * stride + i);
    double* part = tile + (wave >> 1) * 32 * (int64_t)stride + (wave & 1) * 32;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double v = acc[x][y][e];
                f(v, (part + (int64_t)(x * 16 + 4 * e) * stride + y * 16)[mine]);
                acc[x][y][e] = v;
            }
}

__device__ __forceinline__ void clear(v4d (&a)[2][2]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u >> 1][u & 1] = v4d{0.0, 0.0, 0.0, 0.0};
}

// acc = old - acc
__device__ __forceinline__ void subtract_from(const v4d (&old)[2][2], v4d (&acc)[2][2]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u >> 1][u & 1] = old[u >> 1][u & 1] - acc[u >> 1][u & 1];
}

// the first diagonal tile
__global__ void __launch_bounds__(256) factor_first_kernel(double* __restrict__ a, int n, double* __restrict__ dinv, double* __restrict__ x,
                                                           int32_t* __restrict__ info) {
    __shared__ __attribute__((aligned(16))) double lds[LDS_DOUBLES];
    for (int idx = threadIdx.x; idx < TB * TB; idx += 256) {
        const int r = idx >> 6, c = idx & 63;
        lds[r * LDT + c] = (c <= r) ? a[(int64_t)r * n + c] : 0.0;
    }
    __syncthreads();
    factor_tile(lds, n, 0, dinv, x, info);
}

// Workgroups 0 .. panel - 1: a[i, kb] <- a[i, kb] * (L_kk^-1)^T for the tiles i = kb + 1 + blockIdx.x below the diagonal tile.
// The others: X[kx, j] = L_kx,kx^-1 R[kx, j], j = 0, 1, .., in the place of R.
__global__ void __launch_bounds__(256) scale_panel_kernel(double* a, double* x, int n, int kb, int panel, int kx, const double* dinv) {
    __shared__ __attribute__((aligned(16))) double lds[2 * SLICE];
    const int b = blockIdx.x;
    v4d acc[2][2] = {};
    double* tile;
    if (b < panel) {
        tile = a + ((int64_t)(kb + 1 + b) * TB) * n + (int64_t)kb * TB;
        // B(k, c) = V(c, k) = dinv[c * 64 + k]
        const double* dv = dinv + (int64_t)kb * TB * TB;
        tile_mac<true>(acc, tile, n, [&](int k0) { return dv + k0; }, TB, TB, lds, [] {});
    } else {
        tile = x + ((int64_t)kx * TB) * n + (int64_t)(b - panel) * TB;
        tile_mac<false>(acc, dinv + (int64_t)kx * TB * TB, TB, [&](int k0) { return tile + (int64_t)k0 * n; }, n, TB, lds, [] {});
    }
    each_element(acc, tile, n, [](double v, double& m) { m = v; });
}

// Workgroups 0 .. trailing - 1: a[i, j] -= sum over q in [kb, kb + depth / 64) of a[i, q] a[j, q]^T.  columns = 1: the tiles
// i >= j0 of tile column j0; otherwise all tiles j0 <= j <= i.  Workgroup 0 has the tile (j0, j0), and factors it.
// The others: rows i0, i0 + 1, .. of the inversion, x_cols tiles each: R[i, j] -= sum over q in [xq, xq + xn) of L[i, q] X[q, j]
// (X[q, j] is zero for q < j; R[i, j] for j >= xq has not been touched before and starts at zero).
__global__ void __launch_bounds__(256) trailing_update_kernel(double* a, double* x, int n, int kb, int depth, int j0, int columns, int trailing,
                                                              int xq, int xn, int i0, int x_cols, double* dinv, int32_t* info) {
    __shared__ __attribute__((aligned(16))) double lds[LDS_DOUBLES];
    const int b = blockIdx.x;
    if (b >= trailing) {
        const int i = i0 + (b - trailing) / x_cols, j = (b - trailing) % x_cols, q = max(xq, j);
        double* tile = x + ((int64_t)i * TB) * n + (int64_t)j * TB;
        const double* bp = x + ((int64_t)q * TB) * n + (int64_t)j * TB;
        v4d acc[2][2] = {}, old[2][2];
        tile_mac<false>(acc, a + ((int64_t)i * TB) * n + (int64_t)q * TB, n, [&](int k0) { return bp + (int64_t)k0 * n; }, n,
                        (xq + xn - q) * TB, lds, [&] {
                            if (j < xq) each_element(old, tile, n, [](double& v, double& m) { v = m; });
                            else clear(old);
                        });
        subtract_from(old, acc);
        each_element(acc, tile, n, [](double v, double& m) { m = v; });
        return;
    }
    int ti = b, tj = 0;
    if (columns != 1) {                                          // row ti, column tj of the triangle of tiles, row by row
        ti = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
        while (ti * (ti + 1) / 2 > b) --ti;
        while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
        ti = __builtin_amdgcn_readfirstlane(ti);
        tj = b - ti * (ti + 1) / 2;
    }
    const int i = j0 + ti, j = j0 + tj;
    double* tile = a + ((int64_t)i * TB) * n + (int64_t)j * TB;
    const double* bp = a + ((int64_t)j * TB) * n + (int64_t)kb * TB;
    v4d acc[2][2] = {}, old[2][2];
    // B(k, c) = a[j, q](c, k)
    tile_mac<true>(acc, a + ((int64_t)i * TB) * n + (int64_t)kb * TB, n, [&](int k0) { return bp + k0; }, n, depth, lds,
                   [&] { each_element(old, tile, n, [](double& v, double& m) { v = m; }); });
    subtract_from(old, acc);
    if (b == 0) {
        each_element(acc, lds, LDT, [](double v, double& m) { m = v; });
        __syncthreads();
        factor_tile(lds, n, j0, dinv, x, info);
    } else {
        each_element(acc, tile, n, [](double v, double& m) { m = v; });
    }
}

// u[r, c] = X[n-1-r, n-1-c] for c >= r, 0 below the diagonal; one workgroup per row
__global__ void __launch_bounds__(256) write_factor_kernel(const double* __restrict__ x, int n, float* __restrict__ u) {
    const int r = blockIdx.x;
    for (int c = threadIdx.x; c < n; c += 256)
        u[(int64_t)r * n + c] = (c >= r) ? (float)x[(int64_t)(n - 1 - r) * n + (n - 1 - c)] : 0.0f;
}

}  // namespace

size_t hessian_factor_workspace_bytes(int64_t K) {
    return (size_t)(2 * K * K + K * TB + 2) * sizeof(double);
}

int launch_hessian_inverse_factor(const float* h, int64_t K, double damp, const int32_t* perm, void* workspace, float* u,
                                  int32_t* info, hipStream_t st) {
    const int n = (int)K, nb = n / TB;                           // nb is even: K is a multiple of 128
    double* a = static_cast<double*>(workspace);
    double* x = a + K * K;
    double* dinv = x + K * K;
    double* scalars = dinv + K * TB;
    hipLaunchKernelGGL(damp_term_kernel, dim3(1), dim3(256), 0, st, h, n, damp, scalars, info);
    hipLaunchKernelGGL(gather_reversed_kernel, dim3(n), dim3(256), 0, st, h, perm, n, scalars, a);
    hipLaunchKernelGGL(factor_first_kernel, dim3(1), dim3(256), 0, st, a, n, dinv, x, info);
    if (int e = launch_status()) return e;
    // panel of column kb (`panel` tiles); row kx of the inverse
    auto scale = [&](int kb, int panel, int kx) {
        if (panel + kx > 0) hipLaunchKernelGGL(scale_panel_kernel, dim3(panel + kx), dim3(256), 0, st, a, x, n, kb, panel, kx, dinv);
    };
    // `trailing` tiles from column j0 on; rows i0 .. i0 + rows - 1 of R, tiles 0 .. cols - 1, take the rows xq .. xq + xn - 1 of X
    auto update = [&](int kb, int depth, int j0, int columns, int trailing, int xq, int xn, int i0, int rows, int cols) {
        if (trailing + rows * cols > 0)
            hipLaunchKernelGGL(trailing_update_kernel, dim3(trailing + rows * cols), dim3(256), 0, st, a, x, n, kb, depth, j0, columns,
                               trailing, xq, xn, i0, cols, dinv, info);
    };
    for (int kb = 0; kb < nb; kb += 2) {
        const int below = nb - kb - 1, m = below - 1;            // tiles below column kb's diagonal tile, and column kb + 1's
        scale(kb, below, kb > 0 ? kb - 1 : 0);                   // and X[kb - 1, :], the second row of the pair before
        // and the products of that pair's rows of X, for all rows below it
        update(kb, TB, kb + 1, 1, below, kb - 2, 2, kb, kb > 0 ? nb - kb : 0, kb);
        scale(kb + 1, m, kb);                                    // and X[kb, :]
        update(kb, 2 * TB, kb + 2, m, m * (m + 1) / 2, kb, 1, kb + 1, 1, kb + 1);   // and its products for row kb + 1
        if (int e = launch_status()) return e;
    }
    scale(0, 0, nb - 1);                                         // X[nb - 1, :]
    hipLaunchKernelGGL(write_factor_kernel, dim3(n), dim3(256), 0, st, x, n, u);
    return launch_status();
}

}  // namespace w4a8
