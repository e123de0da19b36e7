// 17 to 144 rows: the W4A16 linear for a few draft blocks at once, CDNA4 (gfx950).
//
// Same layer as the other decode kernels (Sec. 2.1, 3.2, 3.3 of arXiv
// 2607.04244).  This file is compiled with matrix-core results kept in
// ordinary VGPRs, as tiled.hip is (see build.py).

#include "decode_common.h"

namespace qlin {

// The direct-to-LDS loads of x: rows of 128 k, or of 64 (HALF), 1 KiB a load.
template <bool HALF>
struct XLoads {
    static constexpr int kChunks = HALF ? 8 : 16, kRows = 64 / kChunks, kLoads = 16 / kRows;
    uint32_t at[kLoads], last[kLoads];        // byte offsets of this lane's chunk; in the last m-tile
    __device__ static inline int swizzle(int row, int c) { return HALF ? c ^ ((row >> 1) & 7) : c ^ (row & 15); }
    __device__ inline XLoads(int lane, uint32_t row_bytes, int last_row) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int r = kRows * i + lane / kChunks;
            const uint32_t c = (uint32_t)swizzle(r, lane % kChunks) * 16u;
            at[i] = (uint32_t)r * row_bytes + c;
            last[i] = (uint32_t)min(r, last_row) * row_bytes + c;
        }
    }
};

// A workgroup owns K chunk c (groups [g0, g0 + Kc)) of column tiles
// [t0, t0 + Tn), Tn <= TN, and all 16 MT rows: every weight of the launch is
// read and dequantized exactly once.  Its 8 waves cut the K range: in a round
// each takes one unit of K and there all of the workgroup's tiles, so the x
// it needs (16 MT rows of the unit) is read from LDS into registers once and
// serves Tn tiles; split by columns instead, every wave would read all of x
// and LDS bandwidth would bound the kernel from 32 rows on.  A unit is a group
// (128 k) up to 64 rows and half a group beyond, where the x of a whole one
// would take 32 MT of a lane's registers.  With whole groups a last round of
// up to four gives each to two waves, 64 k each; where it is the only round they
// load no more than they use: every other tile each or, of one tile, 64 k.  Of
// five or six groups in the only round the last ones are divided by tiles over waves
// 4 to 7, as each of these shares a SIMD with one of the first four: 640 x 19456 at
// 17 / 32 / 48 rows 6.8 / 7.1 / 7.9 -> 6.1 / 6.45 / 7.2 us, 768 x 16384 6.2 / 6.45 /
// 7.1 -> 5.8 / 6.1 / 6.9 (seven divided that way were 3 to 7% slower).
//
// The waves share nothing before the end: a wave stages its unit's x in LDS
// of its own with direct-to-LDS loads (LDS only turns rows into operand
// order), its weight blocks arrive in registers, and both are requested one
// round ahead, as soon as the round's own x has gone from LDS to registers: no
// workgroup barrier in the walk.
//
// Measured (graph replays over rotating weights, us a launch; before: the
// staged kernel of 16 rows and fewer with up to four m-tiles, whose x chunk
// fitted LDS only for K splits of 5 to 26): 2560 x 19456 at 32 / 48 / 64 rows
// 12.9 / 14.5 / 16.8 (34 / 35 / 61 before, 17.6 / 18.4 / 18.5 as 64 x 128
// blocks of the tiled kernel), 9728 x 2560 10.9 / 12.4 / 14.0 (21 / 22 / 37;
// tiled 16.4 / 16.6 / 16.7).  At 64 rows of 2560 x 19456 half of the time goes
// to the loads (every workgroup reads all of x, 327 KB, mostly from L2, beside
// its weights), a fifth to products that the loads do not cover and a quarter
// to the sums and stores.  Requesting the weights two rounds ahead (two copies of the
// walk's body) was 0.6 to 1.4 us slower; a workgroup-wide pipeline of 4-group
// steps, two waves a group, with a barrier a step took 15.3 us at 32 rows.
// Beyond 64 rows, against the tiled kernel: 2560 x 6144 at 65 / 96 / 129 rows
// 10.8 / 12.8 / 14.9 (14.1 / 14.1 / 17.1), 2560 x 12288 at 65 / 90 rows
// 13.3 / 15.5 (17.7 / 18.0), 512 x 2048 at 65 / 128 rows 4.3 / 5.2 (5.9 / 5.9).
//
// At the end the waves' sums are added in LDS in a fixed order: wave w + 4 to
// wave w, then the four sums in order; of a single round of groups shared by tile
// each pair of waves is one of the four.  LDS bandwidth bounds this end, 16 KB a
// tile and m-tile.  With sums in row order (four lanes to a bank), every wave's
// sums of every tile, and both waves of a pair loading all of a shared group,
// 512 x 19456 at 17 / 48 / 64 rows took 6.6 / 7.8 / 8.3 us, now 5.5 / 6.4 / 7.0,
// 512 x 4096 at 64 rows 5.2, now 4.8.  Longer walks are one loop: a last round as
// code of its own behind it takes 9.3 us for 2560 x 12288 at 17 rows, not 8.3.
//
// x of a wave in LDS: 16-byte chunk c (k = 8 c) of row r at slot
// 16 r + (c ^ (r & 15)), as in the tiled kernel, or, with half-group units,
// 8 r + (c ^ ((r >> 1) & 7)): coalesced fills and operand reads without bank
// conflicts.
template <int MT, int TN, bool SYM>
__global__ void __launch_bounds__(kThreads) k_mid(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool HG = MT > 4;                      // a wave's unit of K: half a group
    constexpr int KJ = HG ? 2 : 4;                   // 32-wide steps of k in a unit
    constexpr bool kShareTiles = !HG && TN > 1;      // what the two waves of a shared last group divide
    constexpr int ROWS = 16 * MT, kHalf = kWaves / 2;
    constexpr uint32_t kWaveX = ROWS * KJ * 64;      // LDS bytes of a wave's x
    constexpr int NS = (TN + 3) / 4;                 // scale loads per group: four tiles each
    constexpr int kSzBlk = kTileN * (SYM ? kSzBytesSym : kSzBytesAsym);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4;
    const WgWork w = wg_work<kRouteMixed>(a, blockIdx.x);
    // work of this wave: rounds of 8 units, then its part of the last ones
    const int units = HG ? 2 * w.Kc : w.Kc;
    const int full = units / kWaves, rem = units % kWaves;
    const bool paired = !HG && rem <= kHalf;
    const bool alone = kShareTiles && full == 0 && rem < 7;   // one round of shared groups is all
    // the unit of a wave in it, and its tiles t, with (t & mask) == pick: up to four
    // groups by pairs of waves; of five or six, one each to waves 0 .. 3 and the
    // rest divided over waves 4 .. 7, each on a SIMD with one of the first
    struct Part1 {
        int unit, mask, pick;
    };
    auto part_of = [&](int wv) -> Part1 {
        if (rem <= kHalf) return {wv >> 1, 1, wv & 1};
        if (wv < kHalf) return {wv, 0, 0};
        if (rem == 5) return {4, 3, wv & 3};
        return {4 + (wv & 1), 1, wv >> 1 & 1};
    };
    const Part1 part = part_of(wave);
    const int tail = alone ? part.unit : paired ? wave >> 1 : wave;   // its unit among the last ones
    const int last = tail < rem ? 1 : 0;             // takes part in the last round
    auto other = [&](int t) { return (t & part.mask) != part.pick; };   // a tile of another wave
    auto group_of = [&](int u) { return HG ? u >> 1 : u; };
    auto half_of = [&](int u) { return HG ? (uint32_t)(u & 1) : 0u; };

    // what a wave loads for a round: its unit, every other tile of a shared group
    // (and its x), or 64 k of one
    enum Share { kWhole, kTiles, kHalves };
    // x of a unit (or, in half-group rows, of a half): load (mt, i) fills rows
    // 16 mt + kRows i + lane / kChunks; rows >= M (only in the last m-tile) are
    // copies of row M - 1 and feed no stored output
    const uint32_t row_bytes = (uint32_t)a.K * 2u;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)((uint32_t)a.M * row_bytes), kRsrcFlags);
    const uint32_t lds_x = lds_addr(smem) + wave * kWaveX;
    const XLoads<HG> xl(lane, row_bytes, a.M - 1 - 16 * (MT - 1));
    const XLoads<true> xh(lane, row_bytes, a.M - 1 - 16 * (MT - 1));   // unused but for kHalves
    auto load_x = [&](auto share, int u) {
        constexpr bool kHalf64 = share == kHalves;
        const auto &x = [&]() -> const auto & {
            if constexpr (kHalf64) return xh;
            else return xl;
        }();
        const uint32_t off = (uint32_t)(w.g0 + group_of(u)) * 256u + (kHalf64 ? wave & 1 : half_of(u)) * 128u;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < x.kLoads; ++i)
                load_lds_buf16(rx, mt == MT - 1 ? x.last[i] : x.at[i], off + mt * 16 * row_bytes,
                               lds_x + (mt * x.kLoads + i) * 1024u);
    };
    // weights and scales of group kb; lane (lg, lm) of scale load i holds column lm of tile 4 i + lg
    const size_t base = (size_t)w.t0 * a.Kb + w.g0;
    const int span = w.Tn * a.Kb;
    const __amdgpu_buffer_rsrc_t rc =
        __builtin_amdgcn_make_buffer_rsrc((void *)(w.codes + base * 64), 0, span * 1024, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)w.sz + base * kSzBlk), 0, span * kSzBlk, kRsrcFlags);
    uint32_t sv[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i)
        sv[i] = (uint32_t)(min(4 * i + lg, w.Tn - 1) * a.Kb) * kSzBlk + sz_offset_bytes<SYM>(lm);
    typedef uint32_t words_t __attribute__((ext_vector_type(KJ)));
    struct Unit {
        words_t c[TN];
        uint32_t s[NS];
    };
    auto load_w = [&](auto share, Unit &g, int u) {
        const int kb = group_of(u);
#pragma unroll
        for (int i = 0; i < NS; ++i) g.s[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, sv[i], kb * kSzBlk, kWeightPolicy);
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            if (share == kTiles && other(t)) continue;
            const uint32_t soff = (uint32_t)(min(t, w.Tn - 1) * a.Kb + kb) * 1024u;
            if constexpr (HG) {
                g.c[t] = __builtin_amdgcn_raw_buffer_load_b64(rc, lane * 16 + half_of(u) * 8, soff, kWeightPolicy);
            } else if constexpr (share == kHalves) {
                const v2u c = __builtin_amdgcn_raw_buffer_load_b64(rc, lane * 16 + (wave & 1) * 8, soff, kWeightPolicy);
                g.c[t][0] = c[0];
                g.c[t][1] = c[1];
            } else {
                g.c[t] = __builtin_amdgcn_raw_buffer_load_b128(rc, lane * 16, soff, kWeightPolicy);
            }
        }
    };
    v4f acc[TN][MT];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[t][mt] = v4f{0, 0, 0, 0};
    const uint4 *xs = (const uint4 *)(smem + wave * kWaveX);

    auto walk = [&](auto route) {
        constexpr bool F16 = decltype(route)::value;
        const ExtractConsts<F16> kx;
        const DeqSel<SYM, F16> dsel(lane);
        Unit g;
        auto request = [&](auto share, int u) {
            load_x(share, u);
            load_w(share, g, u);
        };
        // one round on what is in flight; `next` requests the round after it.  Of
        // a whole unit the wave takes its first 64 k, its second or both
        auto round = [&](auto share, auto next, bool lo, bool hi) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this round's x is in LDS
            const Unit cur = g;
            constexpr int kSteps = share == kHalves ? 2 : KJ;
            using X = XLoads<HG || share == kHalves>;
            v8bf xf[kSteps][MT];
#pragma unroll
            for (int j = 0; j < kSteps; ++j)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    xf[j][mt] = __builtin_bit_cast(v8bf, xs[(16 * mt + lm) * X::kChunks + X::swizzle(lm, 4 * j + lg)]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // and in registers: its LDS is free
            next();
            uint32_t sz[4 * NS];
#pragma unroll
            for (int i = 0; i < NS; ++i) {                       // each tile's words to all lanes of its column
                const auto h = __builtin_amdgcn_permlane32_swap(cur.s[i], cur.s[i], false, false);
                const auto e = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
                const auto o = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
                sz[4 * i] = e[0];
                sz[4 * i + 1] = e[1];
                sz[4 * i + 2] = o[0];
                sz[4 * i + 3] = o[1];
            }
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                if (t >= w.Tn || (share == kTiles && other(t))) continue;
                const MfmaDeq d = dsel.setup(sz[t]);
#pragma unroll
                for (int jj = 0; jj < kSteps; jj += 2) {
                    if (share == kWhole && !HG && !(jj ? hi : lo)) continue;
#pragma unroll
                    for (int j = jj; j < jj + 2; ++j) {
                        const v8bf wa = mfma_dequant<F16>(cur.c[t][j], d, kx);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, xf[j][mt], acc[t][mt], 0, 0, 0);
                    }
                }
            }
        };
        using Whole = std::integral_constant<Share, kWhole>;
        using Part = std::integral_constant<Share, kShareTiles ? kTiles : kHalves>;
        if constexpr (kShareTiles) {
            if (alone) {
                request(Part{}, tail);
                round(Part{}, [] {}, true, true);
                return;
            }
        } else if constexpr (!HG) {
            if (full == 0 || (full == 1 && (MT == 4 || rem == 0))) {
                auto request_last = [&] {
                    if (last && paired) request(Part{}, full * kWaves + tail);
                    else if (last) request(Whole{}, full * kWaves + tail);
                };
                if (full == 1) {
                    request(Whole{}, wave);
                    round(Whole{}, request_last, true, true);
                } else {
                    request_last();
                }
                if (last && paired) round(Part{}, [] {}, true, true);
                else if (last) round(Whole{}, [] {}, true, true);
                return;
            }
        }
        auto unit_of = [&](int r) { return r < full ? r * kWaves + wave : full * kWaves + tail; };
        request(Whole{}, unit_of(0));
        for (int r = 0; r < full + last; ++r) {
            const bool whole = r < full || !paired;
            round(Whole{}, [&] { if (r + 1 < full + last) request(Whole{}, unit_of(r + 1)); },
                  whole || (wave & 1) == 0, whole || (wave & 1) == 1);
        }
    };
    // Both routes in one kernel: with a route each the compiler copies the sums
    // between registers from round to round (1024 x 19456 at 17 rows 7.5 us, not 7.1).
    if (full + last > 0) on_route<kRouteMixed>(w.f16, walk);

    // sums: [set < 4][tile][row][16 columns] fp32 in LDS, over the x, in the order
    // of sums_unit().  D of the 16x16 op: lane l holds columns 4 (l >> 4) + v of row l & 15
    lds_barrier();
    float *sums = (float *)smem;
    auto at = [&](int set, int t, int mt) {
        return (v4f *)(sums + (size_t)(set * TN + t) * ROWS * 16 + 4 * sums_unit(16 * mt + lm, lg));
    };
    if (alone && rem <= kHalf) {
        // one round of shared groups: the pairs are the sets, each tile in one wave of a pair
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (t < w.Tn && !other(t)) *at(wave >> 1, t, mt) = acc[t][mt];
    } else if (alone) {
        // five or six groups: wave w + 4, in the tiles it has, to wave w
        const Part1 partner = part_of(wave | kHalf);
        const int set = wave & (kHalf - 1);
        if (wave >= kHalf) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (t < w.Tn && !other(t)) *at(set, t, mt) = acc[t][mt];
        }
        lds_barrier();
        if (wave < kHalf) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (t < w.Tn)
                        *at(set, t, mt) = (t & partner.mask) == partner.pick ? acc[t][mt] + *at(set, t, mt) : acc[t][mt];
        }
    } else {
        // wave w + 4 to wave w (no sums in waves past the last unit of a single round)
        auto busy = [&](int wv) { return full > 0 || (paired ? wv >> 1 : wv) < rem; };
        const int set = wave & (kHalf - 1);
        if (wave >= kHalf && busy(wave)) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (t < w.Tn) *at(set, t, mt) = acc[t][mt];
        }
        lds_barrier();
        if (wave < kHalf) {
            if (busy(wave + kHalf)) {
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        if (t < w.Tn) *at(set, t, mt) = acc[t][mt] + *at(set, t, mt);
            } else {
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        if (t < w.Tn) *at(set, t, mt) = acc[t][mt];
            }
        }
    }
    lds_barrier();
    write_sums<kHalf>(a, w, sums, TN, ROWS);
}

template <int MT, int TN, bool SYM>
static FwdKernel pick_mid_tiles(int tn) {
    if (tn == TN) return k_mid<MT, TN, SYM>;
    if constexpr (TN > 1) return pick_mid_tiles<MT, TN - 1, SYM>(tn);
    return nullptr;
}

template <int MT, bool SYM>
static FwdKernel pick_mid_rows(int mrows, int tn) {
    if (mrows == 16 * MT) return pick_mid_tiles<MT, mid_tiles_max(MT), SYM>(tn);
    if constexpr (MT < kMidTilesM) return pick_mid_rows<MT + 1, SYM>(mrows, tn);
    return nullptr;
}

FwdKernel pick_mid(int mrows, int tn, bool symmetric) {
    return symmetric ? pick_mid_rows<2, true>(mrows, tn) : pick_mid_rows<2, false>(mrows, tn);
}

}  // namespace qlin
