// Which kernel, tile and split of K the many-token layers run on, from the sizes alone (host code).
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/w4a8.h"

namespace w4a8 {

// How the tiled-layout linear kernels read the weights.
//   MODE_CODE_EXACT  signed codes, fp32 group scales applied to the partial sums
//   MODE_TWO_LEVEL   signed codes, `scales` = FP8-domain group scales, output scaled by s_x * w_out[n] (w_out[0] when
//                    per_channel is 0)
//   MODE_ASYM        unsigned codes, `scales` = the 80-byte records of group scales and zero-points
//   MODE_POW2        signed codes, power-of-two group scales applied by the matrix unit (block-scaled MFMA)
//   MODE_ASYM_TWO    unsigned codes and zero-points with FP8-domain group scales in the 80-byte records: the two-level
//                    reading of the asymmetric format; output scaled like MODE_TWO_LEVEL
enum WeightMode { MODE_CODE_EXACT = 0, MODE_TWO_LEVEL = 1, MODE_ASYM = 2, MODE_POW2 = 3, MODE_ASYM_TWO = 4 };

// Built workgroup shapes {token blocks, K-split groups, bands per wavefront}, in the launcher's order of preference
// (the last one is considered first, under its own condition).
#define W4A8_MFMA_SHAPES 7
#define W4A8_MFMA_SHAPE_LIST {{16, 1, 1}, {8, 1, 1}, {8, 2, 1}, {4, 1, 1}, {4, 2, 1}, {4, 4, 1}, {16, 1, 2}}

// Estimated microseconds, from which the launch of a layer is chosen: a launch, what every round of workgroups that run at the same time takes,
// what grows with the share of the chip that is taken, and the outputs (a million of them; more where their rows are not
// aligned for 16-byte stores).  x: rounds, c: 128-deep chunks of K, or passes.
struct Outputs {
    double million;
    bool ragged;
};
struct UnitTimes {                   // the second tiling, one workgroup per compute unit: a partly filled last round costs nearly a full one
    double launch, tile, chunk, tile_fill, chunk_fill, out, out_ragged;
    double cost(int64_t tiles, double c, Outputs o) const {
        const double x = (double)tiles / 256.0;
        return launch + ceil(x) * (tile + c * chunk) + x * (tile_fill + c * chunk_fill) + (out + (o.ragged ? out_ragged : 0.0)) * o.million;
    }
};
struct PairTimes {                   // two to a compute unit: alone on it, sharing it, and the last round's share after full ones
    double launch, alone, alone_c, shared, shared_c, tail, out, out_ragged;
    double cost(int64_t tiles, double c, Outputs o) const {
        const int64_t full = tiles / 512, rem = tiles % 512;
        const double s = shared + shared_c * c;
        // a last round of at most 256 workgroups starts while others still finish theirs, and has its units to itself
        const double last = rem == 0 ? 0.0 : rem > 256 ? s : full > 0 ? tail * s : alone + alone_c * c;
        return launch + (double)full * s + last + (out + (o.ragged ? out_ragged : 0.0)) * o.million;
    }
};
struct FirstTimes {                  // the first tiling, `places` workgroups at a time; tail: how much of a full round a partly filled one costs
    double launch, group, pass, group_fill, pass_fill, tail, out, out_ragged;
    double cost(int64_t groups, int places, double passes, Outputs o) const {
        const double x = (double)groups / places, rounds = x <= 1.0 ? 1.0 : (1.0 - tail) * x + tail * ceil(x);
        return launch + rounds * (group + passes * pass) + x * (group_fill + passes * pass_fill) + (out + (o.ragged ? out_ragged : 0.0)) * o.million;
    }
};
struct TileTimes {
    UnitTimes tall, square, half, half_short;   // the second tiling's 512 x 128, 256 x 256 and 256 x 128 tiles, the last also on the loop for few chunks
    PairTimes pair;                          // its 256 x 128 tiles of four wavefronts
    FirstTimes first[W4A8_MFMA_SHAPES - 1];  // the first tiling's shapes, in the order of their list
};
// Fitted to 2307 layers in each format, every tile and shape timed on all of them, on half of them with weights that come from HBM: random ones (65 ...
// 8192 tokens, 128 ... 28672 features, a fifth of them at most 1536, 360 ... 32768 channels, half of them no multiple of 128) and 16
// layers x 20 token counts.  What they choose is 0.6 ... 1.5 % slower than the best in the mean (0.8 ... 1.4 on the half that a fit has not
// seen), up to a third on single sizes (few chunks and ragged rows).
// PAIR_TIE, OTHER_TIE: between equals the four-wavefront tiles in the plain formats (3072 tokens of 4096 -> 6144, code-exact, 95 us, eight
// wavefronts 96.5), the eight-wavefront ones in the others (4096 tokens, asymmetric, 120.6, four 122.3).
// MARKED_RISK: groups that hold a -8, which nobody knows here, cost a layer on linear_pipe.hip 58 %, on the other tiles 28 and on the first tiling 11 to
// 22.  With it 8 of the 1274 layers take more than 10 % longer with -8 in every group than on the launches chosen before, without it
// 47; it costs the others 0.2 %.
constexpr double PAIR_TIE = 0.985, OTHER_TIE = 1.01, MARKED_RISK = 1.05;
constexpr TileTimes CODE_EXACT_TIMES = {{4.35, 3.13, 1.34, 0.648, 0.328, 0.0899, 0.161}, {3.89, 3.64, 1.45, 0.962, 0.24, 0.0491, 0.0874},
    {4, 3.03, 0.736, 0.356, 0.177, 0.142, 0.143}, {}, {5.84, 0.441, 1.22, 0.661, 1.72, 0.611, 0.309, 0.131},
    {{4.28, 0.864, 1.13, 2.24, 0.749, 0.968, 0.249, 0.0517}, {4.05, 0, 0.757, 3.28, 0.38, 1, 0.0756, 0.0382}, {3.8, 0, 0.874, 2.32, 0.48, 0.843, 0.163, 0.0727},
     {3.59, 0, 0.569, 3.45, 0.545, 0.574, 0, 0.0282}, {3.53, 0, 0.605, 2.65, 0.602, 0.728, 0, 0.0717}, {3.28, 0.142, 0.726, 1.32, 0.552, 0.884, 0.0123, 0.279}}};
constexpr TileTimes POW2_TIMES = {{}, {3.92, 3.48, 1.24, 1.47, 0.242, 0.0141, 0.119},
    {4.38, 1.54, 0.706, 0.897, 0.116, 0.127, 0.14}, {}, {5.4, 0.12, 1.07, 0.222, 1.52, 0.618, 0.271, 0.13},
    {{4.29, 0.637, 1.03, 1.97, 0.66, 0.956, 0.273, 0.0421}, {4.07, 0, 0.696, 2.42, 0.42, 0.917, 0.142, 0.0419}, {3.83, 0, 0.827, 1.61, 0.571, 0.758, 0.204, 0.0979},
     {3.51, 0, 0.584, 3.56, 0.521, 0.548, 0, 0.0403}, {3.46, 0, 0.623, 2.7, 0.583, 0.697, 0, 0.0903}, {3.34, 0, 0.746, 1.35, 0.545, 0.898, 0.0372, 0.309}}};
constexpr TileTimes TWO_LEVEL_TIMES = {{4.04, 2.86, 1.33, 0, 0.243, 0.142, 0.125}, {4.04, 3.68, 1.45, 1.28, 0.226, 0.0467, 0.101},
    {3.87, 2.78, 0.754, 0, 0.149, 0.172, 0.113}, {3.97, 1.25, 0.799, 0.326, 0.195, 0.182, 0.128}, {5.99, 0.99, 1.2, 0.852, 1.67, 0.624, 0.328, 0.114},
    {{5.46, 1.2, 0.674, 0, 1.04, 0.98, 0.342, 0.0395}, {4.74, 0, 0.551, 1.57, 0.51, 0.847, 0.296, 0.0512}, {4.62, 0, 0.671, 1.83, 0.539, 0.757, 0.295, 0.0937},
     {4.11, 0, 0.477, 2.84, 0.636, 0.436, 0.214, 0.0828}, {4.23, 0, 0.471, 3.21, 0.693, 0.576, 0, 0.104}, {3.65, 0.139, 0.664, 1.92, 0.457, 0.845, 0.0436, 0.219}}};
constexpr TileTimes ASYM_TIMES = {{4.05, 3.65, 1.5, 0, 0.285, 0.142, 0.126}, {3.89, 5.71, 1.75, 1.31, 0.252, 0.0317, 0.111},
    {3.83, 4.28, 0.867, 0.216, 0.167, 0.195, 0.109}, {4.28, 0.714, 1.11, 0.792, 0.0174, 0.206, 0.122}, {6.06, 1.83, 1.45, 2.48, 2, 0.63, 0.28, 0.11},
    {{5.59, 0.668, 1.03, 0.557, 1.08, 0.909, 0.364, 0.0412}, {4.89, 0, 0.638, 1.39, 0.582, 1, 0.313, 0.0335}, {4.57, 0, 0.749, 1.82, 0.644, 0.788, 0.3, 0.0789},
     {4.26, 0, 0.496, 1.73, 0.77, 0.607, 0.305, 0.0625}, {3.81, 0.0344, 0.603, 2.65, 0.303, 0.908, 0, 0.0526}, {3.55, 0.222, 0.732, 1.98, 0.464, 0.85, 0, 0.183}}};
constexpr TileTimes ASYM_TWO_TIMES = {{3.84, 2.79, 1.37, 0, 0.248, 0.153, 0.139}, {3.52, 4.58, 1.53, 1.37, 0.273, 0.0279, 0.108},
    {4.39, 2.14, 0.808, 0.0477, 0.147, 0.153, 0.113}, {3.95, 1.12, 0.893, 0.18, 0.172, 0.215, 0.137}, {5.87, 0.514, 1.27, 0.618, 1.74, 0.653, 0.344, 0.14},
    {{4.86, 1.69, 0.789, 0, 1, 1, 0.347, 0.0417}, {4.89, 0, 0.591, 1.15, 0.611, 0.935, 0.338, 0.0637}, {4.64, 0, 0.747, 1.74, 0.607, 0.778, 0.327, 0.102},
     {4.2, 0, 0.502, 1.96, 0.767, 0.635, 0.389, 0.0556}, {4.25, 0, 0.506, 3.13, 0.865, 0.652, 0.0134, 0.0945}, {3.66, 0.126, 0.761, 2.19, 0.441, 0.835, 0, 0.208}}};

// 512 x 128 tiles in place of 256 x 256 ones: for the code-exact format where the grid needs no more of them.  A
// 512 x 128 tile expands half as many bands per MFMA, which that format's FMAs leave no room for (8192 tokens of 4096 -> 28672:
// 844 us against 866, and 1 to 5 % less at each of fourteen sizes timed in turn); with power-of-two scales the expansion has room
// beside the MFMAs and the square's smaller panels win (779 / 764).
inline bool mfma2d_tall_instead(int64_t M, int64_t N, int mode) {
    return mode == MODE_CODE_EXACT && (M + 511) / 512 * ((N + 127) / 128) <= (M + 255) / 256 * ((N + 255) / 256);
}

// The first tiling's shape for a layer; requested values other than 0 are kept.  False: a combination that is not built.
inline bool first_tiling_shape(int64_t M, int64_t K, int64_t N, int& mf, int& ks, int& tpw) {
    static const int cand[W4A8_MFMA_SHAPES][3] = W4A8_MFMA_SHAPE_LIST;
    if (mf != 0 && ks != 0 && tpw != 0) return true;
    const int C = (int)(K / 128);
    const int n_tiles = (int)((N + 15) / 16);
    int pick = -1, fallback = -1;
    // 256 tokens x 256 channels (two bands per wavefront, half the LDS reads per MFMA, one workgroup per compute unit)
    // measured no faster than 256 x 128 at twice the occupancy on any swept shape: on request only.
    if (tpw == 2 && (mf == 0 || mf == 16) && (ks == 0 || ks == 1)) pick = W4A8_MFMA_SHAPES - 1;
    for (int q = 0; q < W4A8_MFMA_SHAPES - 1 && pick < 0; ++q) {
        const int mfv = cand[q][0], ksv = cand[q][1], tpv = cand[q][2];
        if ((mf && mf != mfv) || (ks && ks != ksv) || (tpw && tpw != tpv)) continue;
        fallback = q;                                            // the finest shape that matches the request
        if (mfv > 4 && 16 * mfv >= 2 * M + 64) continue;         // mostly padding
        if (ksv > 1 && C < 4 * ksv) continue;                    // too few chunks to split
        const int per_wg = (8 / ksv) * tpv;
        const int64_t groups = ((M + 16 * mfv - 1) / (16 * mfv)) * (int64_t)((n_tiles + per_wg - 1) / per_wg);
        if (groups >= 384) { pick = q; break; }
    }
    if (pick < 0) pick = fallback;
    if (pick < 0) return false;
    mf = cand[pick][0];
    ks = cand[pick][1];
    tpw = cand[pick][2];
    return true;
}

// 256 x 128 tiles of the formats with a table per channel on few chunks of K run on the loop of linear_mfma2d.hip: its start is shorter than that of
// linear_pipe.hip, which has three chunks on their way before it begins.  Time against linear_pipe.hip on 1 ... 2, 3 ... 4, 5 ... 6, 7 ... 8,
// 9 ... 12, 13 ... 20 chunks: asymmetric 0.76, 0.80, 0.84, 0.88, 0.92, 0.98, two-level 0.85, 0.87, 0.90, 0.92, 0.96, 0.99, asymmetric
// two-level 0.88, 0.91, 0.93, 0.95, 0.98, 1.02.  (The plain formats gain by it up to eight chunks too, but on sizes where the first tiling is faster still.)
inline bool mfma2d_few_chunks(int64_t C, int mode) { return C <= 12 && mode != MODE_CODE_EXACT && mode != MODE_POW2; }

// Launch shape of the many-token kernels for a layer; requested values of mf / ks / tpw other than 0 are kept
// (microseconds: the estimate, where all were 0).
// cfg2d >= 0 on return: the layer goes to the second tiling (linear_mfma2d.hip, linear_pipe.hip) with that workgroup tile.
//  - The second tiling (a 2-D grid of wavefronts, expansion shared through LDS, persistent workgroups) competes with the first on
//    estimated time; its tiles differ in what they ask of the vector unit and of memory per MFMA (large ones least) and
//    in how well a grid fills the chip.  Microseconds on 512 x 128 / 256 x 256 / 256 x 128 / four-wavefront 256 x 128 tiles / first
//    tiling, code-exact: 8192 tokens of 4096 -> 28672 848 / 903 / 965 / 954 / 968; 1024 tokens of 4096 -> 6144 55 / 57 / 35 / 45 / 39;
//    3072 tokens of 4096 -> 6144 113 / 112 / 96 / 96 / 109; 2048 tokens of 4096 -> 28672 227 / 231 / 236 / 221 / 248; 256
//    tokens of 4096 -> 4096 49 / 53 / 31 / 41 / 14.  128 x 128 tiles would be the fastest by more than 3 % on one size in thirty
//    (65 ... 128 tokens of very wide layers) and serve the split of K only.
//  - First tiling: tall token blocks amortize the nibble expansion over more MFMAs; K-splits shorten the dependent chain of
//    passes (each waits for the copies of the next) when the grid is too small to fill the chip, at the price of a wider activation
//    block to copy per pass.  On one to three chunks the four groups of (4, 4, 1) have too few for all, and are still the fastest of the
//    small grids (283 tokens of 384 -> 640 4.9 us, (4, 1, 1) 5.7).
inline bool choose_many_token_launch(int64_t M, int64_t K, int64_t N, int mode, int& mf, int& ks, int& tpw, int& cfg2d, double& microseconds) {
    static const int cand[W4A8_MFMA_SHAPES][3] = W4A8_MFMA_SHAPE_LIST;
    cfg2d = -1;
    const bool chosen = mf == 0 && ks == 0 && tpw == 0;
    if (!first_tiling_shape(M, K, N, mf, ks, tpw)) return false;
    microseconds = 0.0;
    if (!chosen) return true;
    const TileTimes& t = mode == MODE_ASYM        ? ASYM_TIMES
                         : mode == MODE_ASYM_TWO  ? ASYM_TWO_TIMES
                         : mode == MODE_TWO_LEVEL ? TWO_LEVEL_TIMES
                         : mode == MODE_POW2      ? POW2_TIMES
                                                  : CODE_EXACT_TIMES;
    const int64_t chunks = K / 128;
    const double c = (double)chunks;
    const Outputs o{(double)M * (double)N * 1e-6, N % 8 != 0};
    auto tiles = [&](int64_t bm, int64_t bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn); };
    double& best = microseconds;
    best = INFINITY;
    for (int q = 0; q < W4A8_MFMA_SHAPES - 1; ++q) {
        const int m = cand[q][0], k = cand[q][1];
        if (m > 4 && 16 * m >= 2 * M + 64) continue;             // mostly padding
        if (k == 2 && chunks < 2) continue;
        const int64_t per_wg = 8 / k, groups = (M + 16 * m - 1) / (16 * m) * (((N + 15) / 16 + per_wg - 1) / per_wg);
        // workgroups that run at the same time: two to a compute unit, three of the smallest shapes (registers)
        const int places = m == 4 && (k == 1 || (k == 2 && mode != MODE_ASYM)) ? 768 : 512;
        const double us = t.first[q].cost(groups, places, (double)((chunks + k - 1) / k), o);
        if (us < best) {
            best = us;
            mf = m;
            ks = k;
            tpw = cand[q][2];
        }
    }
    // by tile: 512 x 128 for the formats whose expansion is the longer one, and where it stands for 256 x 256; 256 x 256; 256 x 128
    // with eight wavefronts and with four
    const bool plain = mode == MODE_CODE_EXACT || mode == MODE_POW2, tall_instead = mfma2d_tall_instead(M, N, mode);
    const double e[5] = {plain && !tall_instead ? INFINITY : t.tall.cost(tiles(512, 128), c, o),
                         tall_instead ? INFINITY : t.square.cost(tiles(256, 256), c, o),
                         (mode == MODE_CODE_EXACT ? MARKED_RISK : 1.0) * (mfma2d_few_chunks(chunks, mode) ? t.half_short : t.half).cost(tiles(256, 128), c, o), INFINITY, (plain ? PAIR_TIE : OTHER_TIE) * t.pair.cost(tiles(256, 128), c, o)};
    for (int q = 0; q < 5; ++q) {
        if (e[q] < best) {
            best = e[q];
            cfg2d = q;
        }
    }
    return true;
}

// Row stride (floats) of a K range's partial sums in the workspace, and the bytes `ksplit` ranges take.
inline int64_t mfma2d_splitk_ldw(int64_t N) { return (N + 63) / 64 * 64; }
inline size_t mfma2d_splitk_bytes(int64_t M, int64_t N, int ksplit) {
    return ksplit > 1 ? (size_t)ksplit * (size_t)M * (size_t)mfma2d_splitk_ldw(N) * sizeof(float) : 0;
}

// The split of K this library uses for a layer of many-token shape when the caller provides a workspace: ksplit = 0 means
// none.  Few output tiles and a deep K (the down projection of a decoder block at 64...512 tokens): the tiles are multiplied
// in `ksplit` K ranges by different workgroups, about as many as it takes to give every compute unit one, and a second launch
// adds up the partial sums.  The tile is the one whose estimate is the lowest: fixed + time per chunk of a range, which grows with the share
// of the chip that is busy, + the partial sums, written and read once.  Fitted to 182 layers (41 ... 512 tokens, 8192 ... 28672
// features, 512 ... 16384 channels), errors -20 ... +28 %, less where it matters; what is chosen is 0.8 % slower than the best in the mean.  Against 128 x 256 tiles
// (128 x 128 where those are at most 16) everywhere: 512 tokens of 28672 -> 8192 144 -> 123 us, 256 tokens 80 -> 70, 512 tokens of
// 14336 -> 4096 49 -> 44, 164 of 21120 -> 5312 43 -> 38.  A layer whose estimate without ranges is lower stays whole (256 tokens of
// 8192 -> 4096 21.6 us, split 24.1 at best; 500 of 8192 -> 2048 23.1 / 24.5).
inline void mfma2d_choose_ksplit(int64_t M, int64_t K, int64_t N, int& cfg, int& ksplit) {
    struct Candidate {
        int cfg, bm, bn;
        double fixed, chunk, fill, per_mb;
    };
    static const Candidate candidates[3] = {{5, 128, 128, 13.2, 0.323, 0.221, 0.177}, {2, 256, 128, 13.7, 0.872, 0.0, 0.165}, {3, 128, 256, 14.0, 1.18, 0.0, 0.059}};
    cfg = 3;
    ksplit = 0;
    const int64_t C = K / 128;
    constexpr double CLEAR_GAIN = 0.87;
    if (M > 512 || K < 8192) return;
    int mf = 0, ks = 0, tpw = 0, cfg2d;
    double best;
    if (!choose_many_token_launch(M, K, N, MODE_CODE_EXACT, mf, ks, tpw, cfg2d, best)) return;
    const double whole = best;
    best *= 1.03;                                                // between equals the ranges (100 tokens of 8192 -> 2048 16.6 us, whole 17.0)
    int64_t cps = 0;
    auto ranges = [&](int64_t tiles) {                          // 0: none
        int64_t s = tiles > 128 ? 0 : 256 / tiles;
        if (s > C / 8) s = C / 8;
        if (s < 2) return (int64_t)0;
        cps = (C + s - 1) / s;
        s = (C + cps - 1) / cps;                                // no empty range
        return s < 2 ? (int64_t)0 : s;
    };
    // Scratch is bounded by the static workspace, or, on larger layers, by what ranges of 128 x 256 tiles (128 x 128 where those are
    // at most 16) would take: layers the static workspace serves under that rule are served under this one.
    const int64_t plane = M * mfma2d_splitk_ldw(N) * (int64_t)sizeof(float);
    const int64_t wide = (M + 127) / 128 * ((N + 255) / 256);
    int64_t most = ranges(wide <= 16 ? (M + 127) / 128 * ((N + 127) / 128) : wide);
    most = K < 12288 && most < 4 ? 0 : most * plane;             // (where that rule left the layer whole)
    if (most < (int64_t)W4A8_STATIC_WORKSPACE_BYTES) most = (int64_t)W4A8_STATIC_WORKSPACE_BYTES;
    for (const Candidate& q : candidates) {
        const int64_t tiles = (M + q.bm - 1) / q.bm * ((N + q.bn - 1) / q.bn), s = ranges(tiles);
        if (s == 0 || s * plane > most) continue;
        const double us = q.fixed + (double)cps * (q.chunk + q.fill * (double)(tiles * s) / 256.0) + q.per_mb * 4e-6 * (double)s * (double)M * (double)N;
        // more scratch than the static workspace has: for a clear gain only, so that layers close to equal stay with callers that have no more
        if (us < best && (s * plane <= (int64_t)W4A8_STATIC_WORKSPACE_BYTES || (K >= 12288 && us < CLEAR_GAIN * whole))) {
            best = us;
            cfg = q.cfg;
            ksplit = (int)s;
        }
    }
}

}  // namespace w4a8
