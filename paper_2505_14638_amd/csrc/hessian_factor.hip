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
// Measured at 4096 features, against 64-deep updates on scalar FMAs, a diagonal tile in a launch of its own (112 us each) and
// an inversion row by row: 11.4 -> 2.75 ms; with the inversion inside the factorization's launches instead of after them
// (twelve launches that double the inverted blocks, 630 us): 2.41 ms (2.41 to 2.6 over the runs since).  The chain of diagonal tiles bounds it: 22 to 24 us to
// load, factor and invert one, in 64 launches that take 23 us at the least (38 with the rows of the inverse beside it, 59 with the
// largest trailing update), and 5.7 us for each panel.
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

// LDS of a workgroup: two slices while it multiplies; then, if it factors, the tile and the inverses of its four diagonal
// 16 x 16 blocks
constexpr int SLICE = TB * LDA;
constexpr int VD = 16 * 18;         // one such inverse, row stride 18
constexpr int LDS_DOUBLES = TB * LDT + 4 * VD;
static_assert(2 * SLICE <= LDS_DOUBLES, "both slices fit");

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

__device__ __forceinline__ double read_lane(double v, int lane) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// 1 / sqrt(d) to within an ulp or two: the hardware's estimate (23 bits) and one third-order step.
// Not finite for d <= 0 and NaN.
__device__ __forceinline__ double inv_sqrt(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Diagonal tile kb, whose lower triangle lies in `t` (row stride LDT): a[kb, kb] <- its lower Cholesky factor L (zeros
// above the diagonal); dinv[kb], row-major 64 x 64, and x[kb, kb] <- V = L^-1 (zeros above the diagonal).  A pivot that is not positive is
// reported through *info (1 + its index in the reversed order, first failure only); the results are then not finite.
// This is the serial part of the factorization: 64 pivots, each waiting for the one before.  Four panels of 16 columns;
// one wavefront factors a panel with a row per lane and its 16 columns in registers, the column just finished reaching
// the other lanes by v_readlane, so that a pivot costs neither a barrier nor a trip through LDS (112 us a tile
// with two barriers, a square root and a division per pivot, 22 to 24 now); the trailing blocks are then updated by all
// four on the matrix unit.  V is put together from the inverses of the four 16 x 16
// diagonal blocks, doubling twice; V's block (i, j) lies in the place of the tile's block (j, i), which L does not use.
__device__ __forceinline__ void factor_tile(double* t, double* vd, double* __restrict__ a, int n, int kb, double* __restrict__ dinv,
                                            double* __restrict__ x, int32_t* __restrict__ info) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    auto blk = [&](int r, int c) { return t + r * 16 * LDT + c * 16; };
    for (int jb = 0; jb < 4; ++jb) {
        if (wave == 0) {
            double c[16];
            double* row = t + lane * LDT + jb * 16;
#pragma unroll
            for (int j = 0; j < 16; j += 2) {
                const v2d v = *reinterpret_cast<const v2d*>(row + j);
                c[j] = v[0];
                c[j + 1] = v[1];
            }
            double d = read_lane(c[0], jb * 16);
            int bad = -1;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double rs = inv_sqrt(d);
                if (!(d > 0.0) && bad < 0) bad = j;
                double s = d * rs;
                s = fma(fma(-s, s, d), 0.5 * rs, s);             // sqrt(d)
                c[j] = (lane == jb * 16 + j) ? s : c[j] * rs;
                if (j + 1 < 16) {                                // the next pivot first
                    d = read_lane(fma(-c[j], c[j], c[j + 1]), jb * 16 + j + 1);
                }
#pragma unroll
                for (int q = j + 1; q < 16; ++q) c[q] = fma(-c[j], read_lane(c[j], jb * 16 + q), c[q]);
            }
            if (bad >= 0 && lane == 0 && *info == 0) *info = kb * TB + jb * 16 + bad + 1;
            // rows above the panel belong to finished columns, what lies above the diagonal is not part of L
            if (lane >= jb * 16) {
#pragma unroll
                for (int j = 0; j < 16; ++j) row[j] = (jb * 16 + j <= lane) ? c[j] : 0.0;
            }
        }
        __syncthreads();
        // trailing blocks (r, c), jb < c <= r < 4, numbered row by row
        int number = 0;
        for (int r = jb + 1; r < 4; ++r)
            for (int c = jb + 1; c <= r; ++c, ++number)
                if ((number & 3) == wave) {
                    v4d acc = {0.0, 0.0, 0.0, 0.0};
                    block_mac<true>(acc, blk(r, jb), LDT, blk(c, jb), LDT, lane);
                    double* p = blk(r, c) + g * LDT + i;
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[4 * e * LDT] -= acc[e];
                }
        __syncthreads();
    }
    double* tile = a + ((int64_t)kb * TB) * n + (int64_t)kb * TB;
    for (int idx = tid; idx < TB * TB; idx += 256) {
        const int r = idx >> 6, c = idx & 63;
        tile[(int64_t)r * n + c] = (c <= r) ? t[r * LDT + c] : 0.0;
    }
    // wavefront w inverts diagonal block w: lane = column (four copies of each)
    {
        const double* l = blk(wave, wave);
        double x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = (r == i) ? 1.0 : 0.0;
        // the reciprocals of the diagonal: one per lane, four copies
        const double rd = 1.0 / l[i * LDT + i];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] *= read_lane(rd, r);
#pragma unroll
            for (int q = r + 1; q < 16; ++q) x[q] = fma(-l[q * LDT + r], x[r], x[q]);
        }
        double* v = vd + wave * VD;
        if (g == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r * 18 + i] = (r >= i) ? x[r] : 0.0;
        }
    }
    __syncthreads();                                             // also: the tile has been copied out, its blocks may go
    auto store_block = [&](double* p, const v4d& v, double sign) {
#pragma unroll
        for (int e = 0; e < 4; ++e) p[(g + 4 * e) * LDT + i] = sign * v[e];
    };
    // V10 = -V11 (L10 V00), V32 = -V33 (L32 V22): L10 and L32 are not needed afterwards and take the inner products
    const int lo = (wave & 1) * 2;                               // wavefronts 0 and 1 (the others repeat the products, unstored)
    {
        v4d m = {0.0, 0.0, 0.0, 0.0};
        block_mac<false>(m, blk(lo + 1, lo), LDT, vd + lo * VD, 18, lane);
        __syncthreads();
        if (wave < 2) store_block(blk(lo + 1, lo), m, 1.0);
        __syncthreads();
        v4d w = {0.0, 0.0, 0.0, 0.0};
        block_mac<false>(w, vd + (lo + 1) * VD, 18, blk(lo + 1, lo), LDT, lane);
        if (wave < 2) store_block(blk(lo, lo + 1), w, -1.0);
        __syncthreads();
    }
    // the lower left quarter, one 16 x 16 block per wavefront: M = L[2..3, 0..1] V[0..1, 0..1], then -V[2..3, 2..3] M
    const int r = 2 + (wave >> 1), c = wave & 1;
    {
        v4d m = {0.0, 0.0, 0.0, 0.0};
        if (c == 0) {
            block_mac<false>(m, blk(r, 0), LDT, vd, 18, lane);
            block_mac<false>(m, blk(r, 1), LDT, blk(0, 1), LDT, lane);
        } else {
            block_mac<false>(m, blk(r, 1), LDT, vd + VD, 18, lane);
        }
        __syncthreads();
        store_block(blk(r, c), m, 1.0);
        __syncthreads();
        v4d w = {0.0, 0.0, 0.0, 0.0};
        if (r == 2) {
            block_mac<false>(w, vd + 2 * VD, 18, blk(2, c), LDT, lane);
        } else {
            block_mac<false>(w, blk(2, 3), LDT, blk(2, c), LDT, lane);
            block_mac<false>(w, vd + 3 * VD, 18, blk(3, c), LDT, lane);
        }
        store_block(blk(c, r), w, -1.0);
        __syncthreads();
    }
    double* dv = dinv + (int64_t)kb * TB * TB;
    for (int idx = tid; idx < TB * TB; idx += 256) {
        const int rr = idx >> 6, cc = idx & 63, br = rr >> 4, bc = cc >> 4;
        double v = 0.0;
        if (br == bc) v = vd[br * VD + (rr & 15) * 18 + (cc & 15)];
        else if (br > bc) v = blk(bc, br)[(rr & 15) * LDT + (cc & 15)];
        dv[idx] = v;
        x[((int64_t)kb * TB + rr) * n + (int64_t)kb * TB + cc] = v;
    }
}

// acc (a wavefront's 2 x 2 blocks of 16 x 16: rows 32 (wave / 2).., columns 32 (wave % 2)..) += A B for a 64 x 64 tile.
// A(r, k) = ap[r * ars + k].  B(k, c): bp(k0) is the address of the slice k0 .. k0 + KS - 1, B(k0 + k, c) there at
// c * brs + k (B_KFAST) or k * brs + c.  depth is a multiple of KS.  A slice is loaded into registers while the one before
// is multiplied.  Ends with a barrier after the last slice has been consumed: LDS and operand tiles may be overwritten.
template <bool B_KFAST, typename BP>
__device__ __forceinline__ void tile_mac(v4d (&acc)[2][2], const double* ap, int64_t ars, BP&& bp, int64_t brs, int depth, double* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    double* as = lds;
    double* bs = lds + SLICE;
    v2d ra[4], rb[4];
    auto load = [&](int k0) {
        const double* b = bp(k0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = tid + u * 256;
            ra[u] = *reinterpret_cast<const v2d*>(ap + (int64_t)(id >> 4) * ars + k0 + (id & 15) * 2);
            rb[u] = B_KFAST ? *reinterpret_cast<const v2d*>(b + (int64_t)(id >> 4) * brs + (id & 15) * 2)
                            : *reinterpret_cast<const v2d*>(b + (int64_t)(id >> 5) * brs + (id & 31) * 2);
        }
    };
    load(0);
    for (int k0 = 0; k0 < depth; k0 += KS) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = tid + u * 256;
            *reinterpret_cast<v2d*>(as + (id >> 4) * LDA + (id & 15) * 2) = ra[u];
            if (B_KFAST) *reinterpret_cast<v2d*>(bs + (id >> 4) * LDA + (id & 15) * 2) = rb[u];
            else *reinterpret_cast<v2d*>(bs + (id >> 5) * LDT + (id & 31) * 2) = rb[u];
        }
        __syncthreads();
        if (k0 + KS < depth) load(k0 + KS);
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
        __syncthreads();
    }
}
static_assert(KS * LDT <= SLICE, "a slice in either order fits");

// f(row, column, value) for every element of the tile this lane holds
template <typename F>
__device__ __forceinline__ void each_element(v4d (&acc)[2][2], F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double v = acc[x][y][e];
                f((wave >> 1) * 32 + x * 16 + g + 4 * e, (wave & 1) * 32 + y * 16 + i, v);
                acc[x][y][e] = v;
            }
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
    factor_tile(lds, lds + TB * LDT, a, n, 0, dinv, x, info);
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
        tile_mac<true>(acc, tile, n, [&](int k0) { return dv + k0; }, TB, TB, lds);
    } else {
        tile = x + ((int64_t)kx * TB) * n + (int64_t)(b - panel) * TB;
        tile_mac<false>(acc, dinv + (int64_t)kx * TB * TB, TB, [&](int k0) { return tile + (int64_t)k0 * n; }, n, TB, lds);
    }
    each_element(acc, [&](int r, int c, double v) { tile[(int64_t)r * n + c] = v; });
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
        v4d acc[2][2] = {}, old[2][2] = {};
        if (j < xq) each_element(old, [&](int r, int c, double& v) { v = tile[(int64_t)r * n + c]; });
        tile_mac<false>(acc, a + ((int64_t)i * TB) * n + (int64_t)q * TB, n, [&](int k0) { return bp + (int64_t)k0 * n; }, n,
                        (xq + xn - q) * TB, lds);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) acc[u][v] = old[u][v] - acc[u][v];
        each_element(acc, [&](int r, int c, double v) { tile[(int64_t)r * n + c] = v; });
        return;
    }
    int ti = b, tj = 0;
    if (columns != 1) {                                          // row ti, column tj of the triangle of tiles, row by row
        ti = (int)((sqrtf(8.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
        while (ti * (ti + 1) / 2 > b) --ti;
        while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
        tj = b - ti * (ti + 1) / 2;
    }
    const int i = j0 + ti, j = j0 + tj;
    double* tile = a + ((int64_t)i * TB) * n + (int64_t)j * TB;
    const double* bp = a + ((int64_t)j * TB) * n + (int64_t)kb * TB;
    v4d acc[2][2] = {}, old[2][2];                               // what the tile holds is on its way while the product is formed
    each_element(old, [&](int r, int c, double& v) { v = tile[(int64_t)r * n + c]; });
    // B(k, c) = a[j, q](c, k)
    tile_mac<true>(acc, a + ((int64_t)i * TB) * n + (int64_t)kb * TB, n, [&](int k0) { return bp + k0; }, n, depth, lds);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = old[u][v] - acc[u][v];
    if (b == 0) {
        each_element(acc, [&](int r, int c, double v) { lds[r * LDT + c] = (c <= r) ? v : 0.0; });
        __syncthreads();
        factor_tile(lds, lds + TB * LDT, a, n, j0, dinv, x, info);
    } else {
        each_element(acc, [&](int r, int c, double v) { tile[(int64_t)r * n + c] = v; });
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
