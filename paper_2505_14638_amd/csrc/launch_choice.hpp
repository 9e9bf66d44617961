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

// Estimated microseconds, from which the launch of a layer is chosen.  What a grid costs is its rounds -- workgroups that run at
// the same time -- times what a round takes, and the last, partly filled one costs nearly as much as a full one.
// C: 128-deep chunks of K.
struct UnitRound {
    double fixed, chunk, fill;       // one workgroup per compute unit: fixed + C (chunk + fill * share of the units that are busy)
    double cost(int64_t tiles, double c) const {
        const int64_t full = tiles / 256, rem = tiles % 256;
        return (double)full * (fixed + c * (chunk + fill)) + (rem == 0 ? 0.0 : fixed + c * (chunk + fill * (double)rem / 256.0));
    }
};
struct PairRound {                   // two to a compute unit: alone on it, sharing it, and the last round's share after full ones
    double alone, alone_c, shared, shared_c, tail;
    double cost(int64_t tiles, double c) const {
        const int64_t full = tiles / 512, rem = tiles % 512;
        const double s = shared + shared_c * c;
        // a last round of at most 256 workgroups starts while others still finish theirs, and has its units to itself
        return (double)full * s + (rem == 0 ? 0.0 : rem > 256 ? s : full > 0 ? tail * s : alone + alone_c * c);
    }
};
struct FirstRound {                  // the first tiling, two to a unit: fixed + passes (pass + fill * share of the 512 places that are taken)
    double fixed, pass, fill, tail;
    double cost(int64_t groups, double passes) const {
        const int64_t full = groups / 512, rem = groups % 512;
        const double s = fixed + passes * (pass + fill), last = fixed + passes * (pass + fill * (double)rem / 512.0);
        return (double)full * s + (rem == 0 ? 0.0 : full > 0 && rem <= 256 ? tail * s : last);
    }
};
struct TileTimes {
    UnitRound tall, square, half;            // the second tiling's 512 x 128, 256 x 256 and 256 x 128 tiles
    PairRound pair;                          // its 256 x 128 tiles of four wavefronts
    FirstRound first[W4A8_MFMA_SHAPES - 1];  // the first tiling's shapes, in the order of their list
};
// Fitted to 16 layers (1024 ... 28672 features, 1024 ... 28672 channels) x 19 token counts (65 ... 8192) on every tile and on the
// first tiling's own choice, in each format: what they choose is 0.2 % (the plain formats 0.8) slower than the best in the mean, 10 % at
// most.  The first tiling is taken unless an estimate is 4 % below its own, so that errors of the fit cost no time there.
// Shapes that a format's runs never met (the first tiling's tall ones) are priced at 1.25 times the code-exact times.
constexpr double PREFER_FIRST = 0.96, SWITCH_SHAPE = 0.85;
constexpr TileTimes CODE_EXACT_TIMES = {{5.88, 1.35, 0.331}, {6.34, 1.4, 0.302}, {4.61, 0.761, 0.158}, {7.6, 1.14, 7.11, 1.715, 0.572},
    {{7.05, 1.04, 0.867, 0.687}, {4.11, 0.715, 0.425, 0.716}, {4.06, 0.841, 0.476, 0.632}, {3.35, 0.611, 0.155, 0.412}, {1.87, 0.68, 0.265, 0.3}, {1.81, 0.733, 0.491, 0.679}}};
constexpr TileTimes POW2_TIMES = {{5.81, 1.22, 0.253}, {6.1, 1.2, 0.259}, {4.97, 0.722, 0.0877}, {6.82, 0.987, 5.69, 1.54, 0.582},
    {{8.95, 1.3, 1.08, 0.687}, {6.81, 0.704, 0.375, 0.495}, {5.63, 1.1, 0.217, 0.481}, {5.85, 0.764, 0.193, 0.412}, {4.93, 0.693, 0.203, 0.3}, {4.04, 0.475, 0.853, 0.424}}};
constexpr TileTimes TWO_LEVEL_TIMES = {{5.5, 1.26, 0.289}, {6.37, 1.4, 0.253}, {6.9, 0.763, 0.0966}, {7.58, 1.15, 7.65, 1.68, 0.597},
    {{8.95, 1.3, 1.08, 0.687}, {7.4, 0.457, 0.618, 0.6}, {7.19, 0.603, 0.61, 0.424}, {5.85, 0.764, 0.193, 0.412}, {6.36, 0.625, 0.209, 0.3}, {5.92, 0.414, 0.713, 0.375}}};
constexpr TileTimes ASYM_TIMES = {{6.26, 1.46, 0.324}, {8.41, 1.7, 0.258}, {7.3, 0.907, 0.126}, {7.81, 1.4, 8.31, 2.08, 0.62},
    {{8.95, 1.3, 1.08, 0.687}, {6.61, 0.894, 0.531, 0.716}, {6.86, 0.904, 0.511, 0.493}, {5.85, 0.764, 0.193, 0.412}, {6.32, 0.641, 0.273, 0.529}, {5.9, 0.499, 0.706, 0.412}}};
constexpr TileTimes ASYM_TWO_TIMES = {{5.76, 1.29, 0.3}, {6.98, 1.48, 0.291}, {5.63, 0.866, 0.0763}, {7.55, 1.2, 7.47, 1.76, 0.612},
    {{8.95, 1.3, 1.08, 0.687}, {8.22, 0.906, 0.227, 0.516}, {6.96, 0.76, 0.608, 0.469}, {5.85, 0.764, 0.193, 0.412}, {6.46, 0.666, 0.273, 0.357}, {6.27, 0.52, 0.673, 0.403}}};

// 512 x 128 tiles in place of 256 x 256 ones: for the code-exact format where the grid needs no more of them.  A
// 512 x 128 tile expands half as many bands per MFMA, which that format's FMAs leave no room for (8192 tokens of 4096 -> 28672:
// 840 us against 858); with power-of-two scales the expansion has room beside the MFMAs and the square's smaller panels win (779 / 764).
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
//    block to copy per pass.  The first shape, in the list's order, that gives about 1.5 workgroups per compute unit, unless the
//    estimates say that this costs an eighth (600 tokens of 1024 -> 8224: 17.7 us, now 15.9); they tell close shapes apart less well than
//    the rule does.
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
    const double c = (double)(K / 128);
    auto tiles = [&](int64_t bm, int64_t bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn); };
    // the first tiling's shape: the rule's, unless another one's estimate is well below its
    auto first_cost = [&](int q) {
        const int64_t per_wg = 8 / cand[q][1];
        return t.first[q].cost((M + 16 * cand[q][0] - 1) / (16 * cand[q][0]) * (((N + 15) / 16 + per_wg - 1) / per_wg),
                               (double)((K / 128 + cand[q][1] - 1) / cand[q][1]));
    };
    int shape = 0;
    while (cand[shape][0] != mf || cand[shape][1] != ks || cand[shape][2] != tpw) ++shape;   // one of the list's, chosen above
    const double rule = first_cost(shape);
    double lowest = SWITCH_SHAPE * rule;
    for (int q = 0; q < W4A8_MFMA_SHAPES - 1; ++q) {
        if (cand[q][0] > 4 && 16 * cand[q][0] >= 2 * M + 64) continue;   // mostly padding
        if (cand[q][1] > 1 && K / 128 < 4 * cand[q][1]) continue;        // too few chunks to split
        if (first_cost(q) < lowest) {
            lowest = first_cost(q);
            shape = q;
        }
    }
    mf = cand[shape][0];
    ks = cand[shape][1];
    tpw = cand[shape][2];
    double& best = microseconds;
    best = PREFER_FIRST * first_cost(shape);
    // by tile: 512 x 128 for the formats whose expansion is the longer one, and where it stands for 256 x 256; 256 x 256; 256 x 128
    // with eight wavefronts and with four
    const bool plain = mode == MODE_CODE_EXACT || mode == MODE_POW2, tall_instead = mfma2d_tall_instead(M, N, mode);
    const double e[5] = {plain && !tall_instead ? INFINITY : t.tall.cost(tiles(512, 128), c),
                         tall_instead ? INFINITY : t.square.cost(tiles(256, 256), c),
                         t.half.cost(tiles(256, 128), c), INFINITY, t.pair.cost(tiles(256, 128), c)};
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
// of the chip that is busy, + the partial sums, written and read once.  Fitted to 47 layers (41 ... 512 tokens, 8192 ... 28672
// features, 512 ... 16384 channels), errors -14 ... +11 %; against 128 x 256 tiles (128 x 128 where those are at most 16) everywhere:
// 512 tokens of 28672 -> 8192 144 -> 123 us, 256 tokens 80 -> 70, 512 tokens of 14336 -> 4096 49 -> 44, 164 of 21120 -> 5312
// 43 -> 38.  A layer whose estimate without ranges is lower stays whole (256 tokens of 8192 -> 4096 21.6 us, split
// 24.1 at best; 500 of 8192 -> 2048 23.1 / 24.5).
inline void mfma2d_choose_ksplit(int64_t M, int64_t K, int64_t N, int& cfg, int& ksplit) {
    struct Candidate {
        int cfg, bm, bn;
        double fixed, chunk, fill, per_mb;
    };
    static const Candidate candidates[3] = {{5, 128, 128, 12.9, 0.426, 0.118, 0.127}, {2, 256, 128, 13.2, 0.644, 0.138, 0.178}, {3, 128, 256, 9.34, 0.888, 0.141, 0.275}};
    cfg = 3;
    ksplit = 0;
    const int64_t C = K / 128;
    if (M > 512 || K < 8192) return;
    int mf = 0, ks = 0, tpw = 0, cfg2d;
    double best;
    if (!choose_many_token_launch(M, K, N, MODE_CODE_EXACT, mf, ks, tpw, cfg2d, best)) return;
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
    if (wide <= 16 && most >= 4) best = INFINITY;                // so few tiles: always
    most = K < 12288 && most < 4 ? 0 : most * plane;             // (where that rule left the layer whole)
    if (most < (int64_t)W4A8_STATIC_WORKSPACE_BYTES) most = (int64_t)W4A8_STATIC_WORKSPACE_BYTES;
    for (const Candidate& q : candidates) {
        const int64_t tiles = (M + q.bm - 1) / q.bm * ((N + q.bn - 1) / q.bn), s = ranges(tiles);
        if (s == 0 || s * plane > most) continue;
        const double us = q.fixed + (double)cps * (q.chunk + q.fill * (double)(tiles * s) / 256.0) + q.per_mb * 4e-6 * (double)s * (double)M * (double)N;
        if (us < best) {
            best = us;
            cfg = q.cfg;
            ksplit = (int)s;
        }
    }
}

}  // namespace w4a8
