// W4A8 linear layer for many tokens, second tiling, on tiles that leave registers for two chunks of operands: 256 x 128 and
// 128 x 128 (tokens x channels).  Layout, tile walk and expansion are those of linear_mfma2d.hip; the loop runs further ahead:
//   - MFMAs of a chunk read registers only.  Meanwhile the operands of the next chunk come from LDS into a second set, the nibbles of the
//     chunk after that are expanded and published, and the activations, scales and nibbles of later ones are on their way;
//   - everything from global memory goes to LDS (three activation stages, three slots each of nibbles, scales and records per
//     wavefront), so that one counted wait per chunk -- all copies but the ones issued in this chunk -- gives each of them at
//     least a whole chunk to arrive.  A wavefront issues the same number of copies in every chunk.  The last chunks, whose copies would lie
//     behind the end of K, run in a loop of their own: there those are copies of no lanes, which cost no traffic, and the count leaves
//     them out (pipe_copies.hpp).
// The copies are spread over the steps of a chunk: eight wavefronts that issue several at once wait for each other's at the one
// vector memory path of the compute unit, with their MFMAs behind them (two at a time 86 us where one at a time takes 69).
// Measured against the loop with operands read at the head of a chunk and one wait for everything at its end, in turn on one card, microseconds:
// 512 tokens of 14336 -> 4096, 256 x 128 tiles: code-exact 114 -> 93, powers of two 111 -> 85, two-level 104 -> 95, asymmetric 126 -> 109,
// asymmetric two-level 116 -> 100; 128 x 128 tiles 85 -> 66, 82 -> 64, 87 -> 75, 101 -> 85, 95 -> 79.  1024 tokens of 4096 -> 14336,
// 256 x 128 tiles 81 -> 73, 71 -> 60, 69 -> 69, 83 -> 79, 75 -> 69.  Its start is longer: on few chunks of K the formats with a table per channel
// stay with linear_mfma2d.hip (mfma2d_few_chunks), and the plain ones take 256 x 128 tiles 2 % longer at four chunks or 11 % (code-exact).
// What bounds a chunk (256 x 128; 1970 cycles with the time stamps and before the last chunks had a loop of their own): 1024 cycles of MFMAs, 32 of a
// SIMD's, and as many of the LDS port, one operand of 2 KB per MFMA and wavefront at 128 bytes a cycle, with the copies' and the expansion's
// writes on top; the copies' issue 200, the expansion and its LDS traffic 300, the barrier and its wait 150; the older wavefront of
// a SIMD runs through its steps in 1300 cycles, the younger one beside it in 1700.
// With -8 in every group the two-level format takes up to 5 % longer than on the loop this replaces (the operand is formed twice), and the plain formats 58 %
// longer than without: every wavefront of a tile's row puts the operand right in its registers.  To let the expanding wavefront do that takes 20 to
// 26 % off such layers and adds 2 to 5 % to all others.
#include "linear_epilogue.hpp"
#include "pipe_copies.hpp"
#include "w4a8_device.hpp"
#include "w4a8_internal.hpp"

#include <math.h>

#include <type_traits>
#include <utility>

namespace w4a8 {
namespace {

constexpr int XCDS_P = 8;

// All lanes if left > 0, none otherwise.
__device__ __forceinline__ uint64_t lanes_if(int left) {
    uint64_t m;
    asm("s_cmp_gt_i32 %1, 0\n\ts_cselect_b64 %0, -1, 0" : "=s"(m) : "s"(left) : "scc");
    return m;
}
// lds_dma_16 / lds_dma_4 for all lanes or for `lanes`, possibly none.  OFFSET counts in LDS and in memory.
template <int OFFSET> __device__ __forceinline__ void lds_dma_16_at(const uint8_t* base, uint32_t offset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
                 :
                 : "v"(offset), "s"(base), "s"(lds_addr), "i"(OFFSET)
                 : "memory", "m0");
}
template <int OFFSET> __device__ __forceinline__ void lds_dma_16_lanes(uint64_t lanes, const uint8_t* base, uint32_t offset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %0, %1 offset:%4\n\ts_mov_b64 exec, -1"
                 :
                 : "v"(offset), "s"(base), "s"(lds_addr), "s"(lanes), "i"(OFFSET)
                 : "memory", "m0");
}
__device__ __forceinline__ void lds_dma_4_lanes(uint64_t lanes, const uint8_t* base, uint32_t offset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dword %0, %1\n\ts_mov_b64 exec, -1"
                 :
                 : "v"(offset), "s"(base), "s"(lds_addr), "s"(lanes)
                 : "memory", "m0");
}

struct All {};                       // in the place of a mask: all lanes

// s_waitcnt vmcnt(N) lgkmcnt(0), known to the compiler
template <int N> __device__ __forceinline__ void wait_copies_but() {
    static_assert(N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}
// ... for all copies but those of a chunk that ends, one of the last.  One statement: branches of the compiler's own cost registers.
template <int NEAR, int FAR> __device__ __forceinline__ void wait_older_copies(int left) {
    constexpr int SOME = copies_that_may_be_left(NEAR, FAR, 4);
    static_assert(copies_that_may_be_left(NEAR, FAR, 3) == 0, "the last one below");
    wait_copies_but<copies_that_may_be_left(NEAR, FAR, 5)>();
    asm volatile("s_cmp_gt_i32 %0, 4\n\ts_cbranch_scc1 1f\n\ts_waitcnt vmcnt(%1)\n\ts_cmp_gt_i32 %0, 3\n\ts_cbranch_scc1 1f\n\t"
                 "s_waitcnt vmcnt(0)\n1:"
                 :
                 : "s"(left), "i"(SOME)
                 : "memory", "scc");
}

template <typename OutT, int WGM, int WGN, int WM, int WN, int MODE>
__global__ void __launch_bounds__(64 * WGM * WGN, 2) linear_pipe_kernel(
    const uint8_t* __restrict__ x8, int M, int64_t ldx8, const float* __restrict__ s_x,
    const uint8_t* __restrict__ packed, const float* __restrict__ scales, int N, int n_tiles, int C, int cpg, int NG,
    OutT* __restrict__ y, int64_t ldy, int grid_m, int grid_n, int group_m, const float* __restrict__ y_scale, int ksplit,
    int cps, int64_t split_stride, const float* __restrict__ w_out, int per_channel) {
    constexpr int WAVES = WGM * WGN;
    static_assert(WAVES == 8 && WN % WGM == 0 && WN % 2 == 0, "eight wavefronts; every one expands whole bands of its own");
    constexpr bool POW2 = MODE == MODE_POW2, TWO = MODE == MODE_TWO_LEVEL, ASYM2 = MODE == MODE_ASYM_TWO, ASYM = MODE == MODE_ASYM || ASYM2;
    constexpr bool OUT_SCALED = TWO || ASYM2;                    // the operand carries the group scale
    constexpr bool SUM_IN_MFMA = POW2 || OUT_SCALED;             // no FMAs in the loop
    constexpr bool NEED_S = !OUT_SCALED, NEED_E = OUT_SCALED || ASYM;
    constexpr int REC = ASYM ? ASYM_RECORD_BYTES : 64;           // bytes of scales (and zero-points) per band and group
    constexpr int BM = 16 * WM * WGM, BN = 16 * WN * WGN, NBAND = WN * WGN, EPW = WN / WGM;
    static_assert(EPW == 1, "one expanded band per wavefront");
    constexpr int A_STAGE = BM * 128, B_STAGE = NBAND * 2048;
    // LDS: activations 0, 1, weight operands 0, activations 2, weight operands 1 (the last two also hold the epilogue's slabs),
    // three slots each of raw nibbles, group scales and records per wavefront
    constexpr int B0 = 2 * A_STAGE, A2 = B0 + B_STAGE, B1 = A2 + A_STAGE, RAW = B1 + B_STAGE, RAW_SLOT = WAVES * 1024;
    constexpr int SC = RAW + 3 * RAW_SLOT, SC_SLOT = NEED_S ? WAVES * 256 : 0;
    constexpr int EC = SC + 3 * SC_SLOT, EC_SLOT = NEED_E ? WAVES * REC : 0;
    constexpr int LDS_BYTES = EC + 3 * EC_SLOT;
    static_assert(LDS_BYTES <= 160 * 1024, "one workgroup per compute unit");
    constexpr int DPW = BM / (8 * WAVES);                        // 1 KiB activation pages a wavefront copies per chunk
    constexpr int NEAR = DPW + (NEED_S ? 1 : 0), FAR = 1 + (NEED_E ? 1 : 0);   // copies a wavefront issues per chunk
    constexpr int COPIES = NEAR + FAR;
    constexpr int STEPS = WM * WN;                               // MFMAs per chunk and wavefront
    constexpr int E_FIRST = WN == 2 ? 1 : 2, E_LAST = STEPS - 3;               // steps E_FIRST .. E_LAST share the expansion
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int kq = lane >> 4, i = lane & 15;

    // This workgroup's tiles, as in linear_mfma2d_kernel: (K range, tile) units of the XCD's contiguous share of the block order
    const int tiles = grid_m * grid_n;
    const int total = tiles * ksplit;
    const int nx = gridDim.x / XCDS_P;
    const int per_xcd = (total + XCDS_P - 1) / XCDS_P;
    const int v_end = min(total, (int)(blockIdx.x % XCDS_P + 1) * per_xcd);
    int v = (int)(blockIdx.x % XCDS_P) * per_xcd + (int)(blockIdx.x / XCDS_P);
    if (v >= v_end) return;

    int m0 = 0, bn = 0, split = 0, c_begin = 0, c_end = C;
    const uint8_t* xrow0 = x8;
    uint32_t xoff[DPW];                                          // lane's offset of page q from the tile's first row
    uint32_t eoff = 0, soff = 0, roff = 0;                       // ... of the expanded band's nibbles, the bands' scales, the expanded band's record
    auto set_tile = [&](int unit) {
        split = unit / tiles;
        const int vt = unit - split * tiles;
        c_begin = split * cps;
        c_end = min(C, c_begin + cps);
        const int group = vt / (group_m * grid_n);
        const int first_m = group * group_m;
        const int rows_in_group = min(group_m, grid_m - first_m);
        const int in_group = vt - group * group_m * grid_n;
        const int bm = first_m + in_group % rows_in_group;
        bn = in_group / rows_in_group;
        m0 = bm * BM;
        // bands past the end reload the last one; not stored
        const int te = min(bn * NBAND + wn * WN + wm, n_tiles - 1);
        eoff = (uint32_t)te * (uint32_t)C * 1024u + lane * 16;
        roff = (uint32_t)te * (uint32_t)(NG * REC) + (uint32_t)min(lane, REC / 4 - 1) * 4;
        const int ts = min(bn * NBAND + wn * WN + (WN == 2 ? (kq & 1) : kq), n_tiles - 1);
        soff = (uint32_t)ts * (uint32_t)(NG * REC) + i * 4;
        xrow0 = x8 + (int64_t)m0 * ldx8 - (DPW - 1) * 1024;          // (the lanes' offsets make up for it)
#pragma unroll
        for (int q = 0; q < DPW; ++q) {
            const int d = wave * DPW + q, r = (d & 1) * 8 + (lane >> 3);
            const int row = min(m0 + (d >> 1) * 16 + r, M - 1) - m0;   // rows past the end reload the last row; not stored
            xoff[q] = (uint32_t)row * (uint32_t)ldx8 + (uint32_t)(((lane & 7) ^ (r & 7) ^ (r >> 3)) * 16) + (uint32_t)(DPW - 1 - q) * 1024;
        }
    };
    // activation stages are laid out in LDS as in linear_mfma2d_kernel
    const uint32_t xa_off = (uint32_t)((wm * WM) * 2048 + (i >> 3) * 1024 + ((i & 7) * 8 + ((2 * kq) ^ ((i & 7) ^ (i >> 3)))) * 16);
    const uint32_t xc_off = (uint32_t)((wm * WM) * 2048 + (i >> 3) * 1024 + ((i & 7) * 8 + ((2 * kq + 1) ^ ((i & 7) ^ (i >> 3)))) * 16);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const uint8_t* sbytes = reinterpret_cast<const uint8_t*>(scales);

    auto stage_a = [](int s) { return s * A_STAGE + (s == 2 ? B_STAGE : 0); };
    // copies of chunk c, by `lanes`: page q of the activations to the stage at `at`, the scales and the nibbles and records to slot s
    auto copy_page = [&](int c, int at, auto Q, auto lanes) {
        constexpr int q = decltype(Q)::value;
        if constexpr (std::is_same_v<decltype(lanes), All>) lds_dma_16_at<q * 1024>(xrow0 + (int64_t)c * 128, xoff[q], lds0 + (uint32_t)at + (uint32_t)(wave * DPW) * 1024);
        else lds_dma_16_lanes<q * 1024>(lanes, xrow0 + (int64_t)c * 128, xoff[q], lds0 + (uint32_t)at + (uint32_t)(wave * DPW) * 1024);
    };
    auto copy_all_pages = [&](int c, int at, auto lanes) {
        static_for(std::make_integer_sequence<int, DPW>{}, [&](auto Q) { copy_page(c, at, Q, lanes); });
    };
    auto copy_scales = [&](int g, int s, auto lanes) {
        if constexpr (NEED_S && std::is_same_v<decltype(lanes), All>) lds_dma_4(sbytes + (int64_t)g * REC, soff, lds0 + SC + (uint32_t)(s * SC_SLOT + wave * 256));
        else if constexpr (NEED_S) lds_dma_4_lanes(lanes, sbytes + (int64_t)g * REC, soff, lds0 + SC + (uint32_t)(s * SC_SLOT + wave * 256));
    };
    auto copy_raw = [&](int c, int s, auto lanes) {
        if constexpr (std::is_same_v<decltype(lanes), All>) lds_dma_16_at<0>(packed + (int64_t)c * 1024, eoff, lds0 + RAW + (uint32_t)(s * RAW_SLOT + wave * 1024));
        else lds_dma_16_lanes<0>(lanes, packed + (int64_t)c * 1024, eoff, lds0 + RAW + (uint32_t)(s * RAW_SLOT + wave * 1024));
    };
    auto copy_record = [&](int g, int s, auto lanes) {
        constexpr uint64_t record = (1ull << (REC / 4)) - 1;
        uint64_t some = record;
        if constexpr (!std::is_same_v<decltype(lanes), All>) some &= lanes;
        if constexpr (NEED_E) lds_dma_4_lanes(some, sbytes + (int64_t)g * REC, roff, lds0 + EC + (uint32_t)(s * EC_SLOT + wave * REC));
    };
    auto publish = [&](int stage, int h, uint32_t a, uint32_t b, uint32_t c2, uint32_t d) {
        *reinterpret_cast<uint4*>(lds + (stage ? B1 : B0) + (wn * WN + wm) * 2048 + h * 1024 + lane * 16) = make_uint4(a, b, c2, d);
    };

    struct Ops {
        v8i b[WN], x[WM];
        float s[WN];
    };
    auto read_weights = [&](Ops& O, int stage, int j) {
        const uint8_t* src = lds + (stage ? B1 : B0) + (wn * WN + j) * 2048 + lane * 16;
        const uint4 lo = *reinterpret_cast<const uint4*>(src), hi = *reinterpret_cast<const uint4*>(src + 1024);
        O.b[j] = v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    };
    auto read_tokens = [&](Ops& O, int at, int f) {
        const uint4 lo = *reinterpret_cast<const uint4*>(lds + at + xa_off + f * 2048), hi = *reinterpret_cast<const uint4*>(lds + at + xc_off + f * 2048);
        O.x[f] = v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    };
    auto read_scale = [&](Ops& O, int s, int j) {
        if constexpr (NEED_S) O.s[j] = *reinterpret_cast<const float*>(lds + SC + s * SC_SLOT + wave * 256 + j * 64 + i * 4);
    };
    v4f acc[WM][WN];
    v4f p_prev, p_prev2;
    auto fold = [&](const Ops& O, auto FP, auto JP, const v4f& p) {
        constexpr int fp = decltype(FP)::value, jp = decltype(JP)::value;
        const float sc = fabsf(O.s[jp]);
        acc[fp][jp][0] = fmaf(sc, p[0], acc[fp][jp][0]);
        acc[fp][jp][1] = fmaf(sc, p[1], acc[fp][jp][1]);
        acc[fp][jp][2] = fmaf(sc, p[2], acc[fp][jp][2]);
        acc[fp][jp][3] = fmaf(sc, p[3], acc[fp][jp][3]);
    };
    auto expand_all = [&](u32x4 raw, uint32_t z, float s8) {
        const uint4 r = make_uint4(raw[0], raw[1], raw[2], raw[3]);
        return TWO     ? slot_to_operand_two_level<true>(r, two_level_table(s8))
               : ASYM2 ? slot_to_operand_asym(r, asym_two_level_table_shared(z, s8, kq))
               : ASYM  ? slot_to_operand_asym(r, asym_table_shared(z, kq))
                       : slot_to_operand<false>(r);
    };
    auto publish_all = [&](int stage, const v8i& o) {
        publish(stage, 0, (uint32_t)o[0], (uint32_t)o[1], (uint32_t)o[2], (uint32_t)o[3]);
        publish(stage, 1, (uint32_t)o[4], (uint32_t)o[5], (uint32_t)o[6], (uint32_t)o[7]);
    };
    int s0 = 0, s1 = 1, s2 = 2;                                  // c % 3, (c + 1) % 3, (c + 2) % 3, c counted from the unit's first chunk
    int g3 = 0, left3 = 0;                                       // group of chunk c + 3, and its chunks from c + 3 on

    // Multiplies chunk c (in cur) and meanwhile reads chunk c + 1 into nxt, expands the nibbles of chunk c + 2 into the stage that chunk c was
    // read from, and copies the activations and scales of chunk c + 3 and the nibbles of chunk c + 4.  PAR: parity of c - c_begin.  LAST: in the
    // loop of the last four chunks (with a fifth or sixth where their number asks for it).
    auto chunk = [&](int c, Ops& cur, Ops& nxt, auto PAR, auto LAST) {
        constexpr int par = decltype(PAR)::value;
        constexpr bool last = decltype(LAST)::value;
        const int at1 = stage_a(s1), at0 = stage_a(s0);
        u32x4 raw = *reinterpret_cast<const u32x4*>(lds + RAW + s2 * RAW_SLOT + wave * 1024 + lane * 16);
        float es = 0.0f;
        uint32_t ez = 0u;
        if (OUT_SCALED) es = *reinterpret_cast<const float*>(lds + EC + s2 * EC_SLOT + wave * REC + i * 4);
        if (ASYM) ez = lds[EC + s2 * EC_SLOT + wave * REC + 64 + i];
        if (!OUT_SCALED && !ASYM) {
            uint32_t marks = 0u;
#pragma unroll
            for (int j = 0; j < WN; ++j) marks |= __float_as_uint(cur.s[j]);
            if (any_marked(__uint_as_float(marks))) {            // wave-uniform, rare: a group that holds a -8
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    if (any_marked(cur.s[j])) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) cur.b[j][e] = (int)sm_fix_minus_eight((uint32_t)cur.b[j][e]);
                    }
                }
            }
        }
        using Lanes = std::conditional_t<last, uint64_t, All>;
        Lanes lanes_a, lanes_w;
        if constexpr (last) {
            lanes_a = lanes_if(c_end - c - 3);
            lanes_w = lanes_if(c_end - c - 4);
        }
        const int g4 = left3 > 1 ? g3 : g3 + 1;
        MagTable tab = {0u, 0u, 0u};
        AsymTable atab = {{0u, 0u, 0u, 0u}};
        uint32_t eop[8];
        static_for(std::make_integer_sequence<int, STEPS>{}, [&](auto ST) {
            constexpr int st = decltype(ST)::value, f = st / WN, j = st % WN;
            if (POW2) acc[f][j] = mfma_16x16x128_e4m3_scaled(cur.x[f], cur.b[j], acc[f][j], E8M0_ONE, e8m0_of(cur.s[j]));
            if (OUT_SCALED) acc[f][j] = mfma_16x16x128_e4m3(cur.x[f], cur.b[j], acc[f][j]);
            const v4f p = SUM_IN_MFMA ? v4f{0.f, 0.f, 0.f, 0.f} : mfma_16x16x128_e4m3(cur.x[f], cur.b[j], v4f{0.f, 0.f, 0.f, 0.f});
            // the next chunk's operands
            constexpr bool RB = st < WN, RS = NEED_S && st >= 2 && st < 2 + WN, RX = f > 0 && j == 0, RL = st == (WN == 2 ? 5 : (WM - 1) * WN + 1);
            if constexpr (RB) read_weights(nxt, par ^ 1, st);
            if constexpr (RS) read_scale(nxt, s1, st - 2);
            if constexpr (RX) read_tokens(nxt, at1, f - 1);
            if constexpr (RL) read_tokens(nxt, at1, WM - 1);
            // copies
            constexpr int D0 = st * COPIES / STEPS, D1 = (st + 1) * COPIES / STEPS;
            static_for(std::make_integer_sequence<int, D1 - D0>{}, [&](auto DI) {
                constexpr int d = D0 + decltype(DI)::value;
                if constexpr (d < DPW) copy_page(c + 3, at0, std::integral_constant<int, d>{}, lanes_a);
                else if constexpr (d == DPW) copy_raw(c + 4, s1, lanes_w);
                else if constexpr (d == DPW + 1 && NEED_S) copy_scales(g3, s0, lanes_a);
                else copy_record(g4, s1, lanes_w);
            });
            if constexpr (!SUM_IN_MFMA) {
                constexpr int sp = (st + STEPS - 2) % STEPS;
                fold(st < 2 ? nxt : cur, std::integral_constant<int, sp / WN>{}, std::integral_constant<int, sp % WN>{}, p_prev2);
                keep_here(acc[sp / WN][sp % WN]);
            }
            p_prev2 = p_prev;
            p_prev = p;
            if constexpr (st == E_FIRST) {
                if (TWO) tab = two_level_table(es);
                if (ASYM) atab = ASYM2 ? asym_two_level_table_shared(ez, es, kq) : asym_table_shared(ez, kq);
            }
            constexpr int SPAN = E_LAST - E_FIRST + 1, se = st - E_FIRST;
            constexpr bool EX = se >= 0 && se < SPAN;
            constexpr int E0 = EX ? se * 8 / SPAN : 0, E1 = EX ? (se + 1) * 8 / SPAN : 0;
            static_for(std::make_integer_sequence<int, E1 - E0>{}, [&](auto EI) {
                constexpr int e = E0 + decltype(EI)::value, d = e >> 1;
                uint32_t o;
                if (TWO) o = (e & 1) ? two_level_half_fast<4>(raw[d], tab) : two_level_half_fast<0>(raw[d], tab);
                else if (ASYM) o = (e & 1) ? asym_half<4>(raw[d], atab) : asym_half<0>(raw[d], atab);
                else o = (e & 1) ? sm_half_to_e4m3_fast<4>(raw[d]) : sm_half_to_e4m3_fast<0>(raw[d]);
                keep_here(o);
                eop[e] = o;
                if (e == 3) publish(par, 0, eop[0], eop[1], eop[2], eop[3]);
                if (e == 7) publish(par, 1, eop[4], eop[5], eop[6], eop[7]);
            });
            constexpr int ALU = (SUM_IN_MFMA ? 0 : 4) + (E1 - E0) * (ASYM ? 7 : 4), WRITES = (E0 <= 3 && E1 > 3 ? 1 : 0) + (E0 <= 7 && E1 > 7 ? 1 : 0);
            constexpr int READS = (RB ? 2 : 0) + (RS ? 1 : 0) + (RX ? 2 : 0) + (RL ? 2 : 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // this step's MFMA
            if constexpr (READS > 0) __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, ALU, 0);                          // ALU work independent of it
            if constexpr (WRITES > 0) __builtin_amdgcn_sched_group_barrier(0x200, WRITES, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (TWO) {
            if (any_marked(es)) publish_all(par, slot_to_operand_two_level<true>(make_uint4(raw[0], raw[1], raw[2], raw[3]), tab));
        }
        const int t = s0;
        s0 = s1;
        s1 = s2;
        s2 = t;
        left3 = left3 > 1 ? left3 - 1 : cpg;
        g3 = g4;
        if (last) wait_older_copies<NEAR, FAR>(c_end - c);       // all but this chunk's copies have landed, reads and writes are done
        else wait_copies_but<COPIES>();
        __syncthreads();
    };

    // A tile's start.  Before the epilogue of the tile before it: chunks 0 and 1, whose nibbles come through registers, and the nibbles of
    // chunk 2; they stay clear of the slabs.  After it: the rest of what the loop expects to be on its way, and the operands of chunk 0.
    u32x4 raw0, raw1;
    float es0 = 0.0f, es1 = 0.0f;
    uint32_t ez0 = 0u, ez1 = 0u;
    auto start_issue = [&]() {
        const int c1 = min(c_begin + 1, c_end - 1);
        raw0 = *reinterpret_cast<const u32x4*>(packed + (int64_t)c_begin * 1024 + eoff);
        raw1 = *reinterpret_cast<const u32x4*>(packed + (int64_t)c1 * 1024 + eoff);
        const uint32_t rbase = roff - (uint32_t)min(lane, REC / 4 - 1) * 4;
        if (OUT_SCALED) {
            es0 = *reinterpret_cast<const float*>(sbytes + (int64_t)(c_begin / cpg) * REC + rbase + i * 4);
            es1 = *reinterpret_cast<const float*>(sbytes + (int64_t)(c1 / cpg) * REC + rbase + i * 4);
        }
        if (ASYM) {
            ez0 = sbytes[(int64_t)(c_begin / cpg) * REC + rbase + 64 + i];
            ez1 = sbytes[(int64_t)(c1 / cpg) * REC + rbase + 64 + i];
        }
        copy_all_pages(c_begin, stage_a(0), All{});
        copy_scales(c_begin / cpg, 0, All{});
        const uint64_t lanes1 = lanes_if(c_end - c_begin - 1), lanes2 = lanes_if(c_end - c_begin - 2);
        copy_all_pages(c_begin + 1, stage_a(1), lanes1);
        copy_scales((c_begin + 1) / cpg, 1, lanes1);
        copy_raw(c_begin + 2, 2, lanes2);
        copy_record((c_begin + 2) / cpg, 2, lanes2);
    };
    Ops oa, ob;
    auto start_finish = [&]() {
        publish_all(0, expand_all(raw0, ez0, es0));
        publish_all(1, expand_all(raw1, ez1, es1));
        const uint64_t lanes2 = lanes_if(c_end - c_begin - 2), lanes3 = lanes_if(c_end - c_begin - 3);
        copy_all_pages(c_begin + 2, stage_a(2), lanes2);
        copy_scales((c_begin + 2) / cpg, 2, lanes2);
        copy_raw(c_begin + 3, 0, lanes3);
        copy_record((c_begin + 3) / cpg, 0, lanes3);
        wait_older_copies<NEAR, FAR>(c_end - c_begin + 1);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            read_weights(oa, 0, j);
            read_scale(oa, 0, j);
            ob.s[j] = 0.0f;
        }
#pragma unroll
        for (int f = 0; f < WM; ++f) read_tokens(oa, 0, f);
        g3 = (c_begin + 3) / cpg;
        left3 = cpg - (c_begin + 3) % cpg;
        s0 = 0;
        s1 = 1;
        s2 = 2;
        p_prev = p_prev2 = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < WM; ++f)
#pragma unroll
            for (int j = 0; j < WN; ++j) acc[f][j] = v4f{0.f, 0.f, 0.f, 0.f};
        __syncthreads();                                         // everybody's reads are done
    };

    const float sx = ksplit > 1 ? 1.0f : *s_x;

    using Out = OutLayout<OutT, WN>;
    static_assert(WAVES * Out::SLAB_BYTES <= A_STAGE + B_STAGE, "the wavefronts' slabs fit");
    const StaticQuantizer quantizer(sizeof(OutT) == 1 ? *y_scale : 1.0f);   // FP8 output: the next layer's activation scale

    set_tile(v);
    start_issue();
    for (;;) {
        start_finish();
        __builtin_amdgcn_s_setprio(1);
        int c = c_begin;
        for (; c + 5 < c_end; c += 2) {
            chunk(c, oa, ob, std::integral_constant<int, 0>{}, std::false_type{});
            chunk(c + 1, ob, oa, std::integral_constant<int, 1>{}, std::false_type{});
        }
        for (; c < c_end; c += 2) {
            chunk(c, oa, ob, std::integral_constant<int, 0>{}, std::true_type{});
            if (c + 1 < c_end) chunk(c + 1, ob, oa, std::integral_constant<int, 1>{}, std::true_type{});
        }
        __builtin_amdgcn_s_setprio(0);
        if (!SUM_IN_MFMA) {
            const bool odd = ((c_end - c_begin) & 1) != 0;
            Ops last;
#pragma unroll
            for (int j = 0; j < WN; ++j) last.s[j] = odd ? oa.s[j] : ob.s[j];
            fold(last, std::integral_constant<int, (STEPS - 2) / WN>{}, std::integral_constant<int, (STEPS - 2) % WN>{}, p_prev2);
            fold(last, std::integral_constant<int, WM - 1>{}, std::integral_constant<int, WN - 1>{}, p_prev);
        }
        const int em0 = m0, ebn = bn, esplit = split;
        v += nx;
        const bool more = v < v_end;
        if (more) {
            set_tile(v);
            start_issue();
        }
        store_tile<OutT, WM, WN, OUT_SCALED, 0, WM>(acc, lds + A2 + wave * Out::SLAB_BYTES, em0 + wm * WM * 16, ebn * BN + wn * WN * 16, M, N,
                                                    y + (int64_t)esplit * split_stride, ldy, sx, w_out, per_channel, quantizer, lane);
        if (!more) break;
        __syncthreads();                                         // everybody is done with the slabs
    }
}

template <int WGM, int WGN, int WM, int WN, int MODE>
void launch_mode(const LinearArgs& a, int ydt, dim3 grid, int grid_m, int grid_n, int group_m, int ksplit, int cps, int64_t stride, hipStream_t st) {
#define W4A8_PIPE(T)                                                                                                           \
    hipLaunchKernelGGL((linear_pipe_kernel<T, WGM, WGN, WM, WN, MODE>), grid, dim3(64 * WGM * WGN), 0, st, a.x8, a.M, a.ldx8, \
                       a.s_x, a.packed, a.scales, a.N, a.n_tiles, a.C, a.cpg, a.NG, static_cast<T*>(a.y), a.ldy, grid_m,       \
                       grid_n, group_m, a.y_scale, ksplit, cps, stride, a.w_out, a.per_channel)
    if (ydt == W4A8_F32) {
        W4A8_PIPE(float);
    } else if (ydt == W4A8_BF16) {
        W4A8_PIPE(uint16_t);
    } else if constexpr (MODE == MODE_CODE_EXACT) {              // FP8 output exists for the code-exact mode only
        if (ydt == YDT_SILU_E4M3) W4A8_PIPE(SiluFp8);
        else W4A8_PIPE(uint8_t);
    }
}

template <int WGM, int WGN, int WM, int WN>
void launch_cfg(const LinearArgs& a, int ydt, dim3 grid, int grid_m, int grid_n, int group_m, int ksplit, int cps, int64_t stride, hipStream_t st) {
    if (a.mode == MODE_POW2) launch_mode<WGM, WGN, WM, WN, MODE_POW2>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
    else if (a.mode == MODE_TWO_LEVEL) launch_mode<WGM, WGN, WM, WN, MODE_TWO_LEVEL>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
    else if (a.mode == MODE_ASYM) launch_mode<WGM, WGN, WM, WN, MODE_ASYM>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
    else if (a.mode == MODE_ASYM_TWO) launch_mode<WGM, WGN, WM, WN, MODE_ASYM_TWO>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
    else launch_mode<WGM, WGN, WM, WN, MODE_CODE_EXACT>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
}

}  // namespace

void launch_linear_pipe(const LinearArgs& a, int cfg, int ydt, dim3 grid, int grid_m, int grid_n, int group_m, int ksplit, int cps, int64_t stride, hipStream_t st) {
    if (cfg == 2) launch_cfg<4, 2, 4, 4>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
    else launch_cfg<2, 4, 4, 2>(a, ydt, grid, grid_m, grid_n, group_m, ksplit, cps, stride, st);
}

}  // namespace w4a8
