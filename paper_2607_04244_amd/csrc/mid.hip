// 17 to 64 rows: the W4A16 linear for a few draft blocks at once, CDNA4 (gfx950).
//
// Same layer as the other decode kernels (Sec. 2.1, 3.2, 3.3 of arXiv
// 2607.04244).  This file is compiled with matrix-core results kept in
// ordinary VGPRs, as tiled.hip is (see build.py).

#include "decode_common.h"

#include <type_traits>

namespace qlin {

// A workgroup owns K chunk c (groups [g0, g0 + Kc)) of column tiles
// [t0, t0 + Tn), Tn <= TN, and all 16 MT rows: every weight of the launch is
// read and dequantized exactly once.  Its 8 waves cut the K range: in a round
// each takes one whole group and there all of the workgroup's tiles, so the x
// it needs (16 MT rows x 128 k) is read from LDS into registers once and
// serves Tn tiles; split by columns instead, every wave would read all of x
// and LDS bandwidth would bound the kernel from 32 rows on.  A last round of
// up to four groups gives each group to two waves, 64 k each.
//
// The waves share nothing before the end: a wave stages its group's x in LDS
// of its own with direct-to-LDS loads (LDS only turns rows into operand
// order), its weight blocks arrive in registers, and both are requested one
// round ahead, right after the round's own have landed: no workgroup barrier
// in the walk.
//
// Measured (graph replays over rotating weights, us a launch; before: the
// staged kernel of 16 rows and fewer with up to four m-tiles, whose x chunk
// fitted LDS only for K splits of 5 to 26): 2560 x 19456 at 32 / 48 / 64 rows
// 12.5 / 14.6 / 16.7 (34 / 35 / 60 before, 17.4 / 17.6 / 18.1 as 64 x 128
// blocks of the tiled kernel), 9728 x 2560 10.3 / 12.3 / 13.9 (21 / 22 / 37;
// tiled 16.6 / 16.7 / 17.0).  Of the 16.7 us, 8.2 go to the loads (10.7 MB of
// x per row of workgroups besides the weights), 3.3 to products that the loads
// do not cover, 2.4 to the sums in LDS and 1.4 to the stores.  Requesting the
// weights two rounds ahead (two copies of the walk's body) was 0.6 to 1.4 us
// slower; a workgroup-wide pipeline of 4-group steps, two waves a group, with
// a barrier a step took 15.3 us at 32 rows.
//
// At the end the waves' sums are added in LDS in a fixed order: wave w + 4 to
// wave w, then the four sums in order.
//
// x of a wave in LDS: 16-byte chunk c (k = 8 c) of row r at slot
// 16 r + (c ^ (r & 15)), as in the tiled kernel: coalesced fills and operand
// reads without bank conflicts.
// Operand of s_waitcnt that waits until at most n vector-memory loads are in
// flight, and for nothing else.
constexpr int wait_vmcnt(int n) { return (n & 15) | (n >> 4) << 14 | 7 << 4 | 15 << 8; }

template <int MT, int TN, bool SYM>
__global__ void __launch_bounds__(kThreads) k_mid(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int ROWS = 16 * MT, kHalf = kWaves / 2;
    constexpr int NS = (TN + 3) / 4;                 // scale loads per group: four tiles each
    constexpr int kSzBlk = kTileN * (SYM ? kSzBytesSym : kSzBytesAsym);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4;
    const WgWork w = wg_work(a, blockIdx.x);
    // rounds of this wave: whole ones, then its part of the last Kc % 8 groups
    const int full = w.Kc / kWaves, rem = w.Kc % kWaves;
    const bool paired = rem <= kHalf;
    const int tail = paired ? wave >> 1 : wave;      // its group among the last ones
    const int nr = full + (tail < rem ? 1 : 0);

    // x: load (mt, i) fills rows 16 mt + 4 i + (lane >> 4); rows >= M (only in
    // the last m-tile) are copies of row M - 1 and feed no stored output
    const uint32_t row_bytes = (uint32_t)a.K * 2u;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)((uint32_t)a.M * row_bytes), kRsrcFlags);
    uint32_t xv[4], xl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 4 * i + lg;
        xv[i] = (uint32_t)r * row_bytes + (uint32_t)(lm ^ r) * 16u;
        xl[i] = (uint32_t)min(r, a.M - 1 - 16 * (MT - 1)) * row_bytes + (uint32_t)(lm ^ r) * 16u;
    }
    const uint32_t lds_x = lds_addr(smem) + wave * (ROWS * 256);
    auto load_x = [&](int kb) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                load_lds_buf16(rx, mt == MT - 1 ? xl[i] : xv[i], (uint32_t)(w.g0 + kb) * 256u + mt * 16 * row_bytes,
                               lds_x + (mt * 4 + i) * 1024u);
    };
    // weights and scales of group kb; lane (lg, lm) of scale load i holds column lm of tile 4 i + lg
    const size_t base = (size_t)w.t0 * a.Kb + w.g0;
    const int span = w.Tn * a.Kb;
    const __amdgpu_buffer_rsrc_t rc =
        __builtin_amdgcn_make_buffer_rsrc((void *)(w.codes + base * 64), 0, span * 1024, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)w.sz + base * kSzBlk), 0, span * kSzBlk, kRsrcFlags);
    const uint32_t cv = lane * 16;
    uint32_t sv[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i)
        sv[i] = (uint32_t)(min(4 * i + lg, w.Tn - 1) * a.Kb) * kSzBlk + sz_offset_bytes<SYM>(lm);
    struct Group {
        uint4 c[TN];
        uint32_t s[NS];
    };
    auto load_s = [&](Group &g, int i, int kb) {
        g.s[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, sv[i], kb * kSzBlk, kWeightPolicy);
    };
    auto load_c = [&](Group &g, int t, int kb) {
        g.c[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                               rc, cv, (min(t, w.Tn - 1) * a.Kb + kb) * 1024, kWeightPolicy));
    };
    auto load_w = [&](Group &g, int kb) {
#pragma unroll
        for (int i = 0; i < NS; ++i) load_s(g, i, kb);
#pragma unroll
        for (int t = 0; t < TN; ++t) load_c(g, t, kb);
    };
    auto group_of = [&](int r) { return r < full ? r * kWaves + wave : full * kWaves + tail; };

    v4f acc[TN][MT];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[t][mt] = v4f{0, 0, 0, 0};
    const uint4 *xb = (const uint4 *)smem + wave * (ROWS * 16) + lm * 16;

    // once per dequantization route (uniform in the workgroup: its tiles
    // belong to one member), the first loads included, so that none in flight
    // is copied between the routes' registers
    auto walk = [&](auto route) {
        constexpr bool F16 = decltype(route)::value;
        const ExtractConsts<F16> kx;
        const DeqSel<SYM, F16> dsel(lane);
        // round r with its weights in g, which it refills for round r + 2.
        // The loads of a round are issued in the order x (of the next
        // round), weights (of the one after), so when only the weights of
        // round r + 1 are left in flight, x and weights of round r are there.
        // The wait is the builtin and not inline assembly: the compiler takes
        // it into account and adds no waits of its own, which would count
        // the x loads it does not see as older than they are.
        auto round = [&](int r, Group &g) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const Group cur = g;
            v8bf xf[4][MT];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    xf[j][mt] = __builtin_bit_cast(v8bf, xb[mt * 256 + ((4 * j + lg) ^ lm)]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // x is in registers: its LDS is free
            if (r + 1 < nr) {
                load_x(group_of(r + 1));
                load_w(g, group_of(r + 1));
            }
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
            // all 128 k of the group, or this wave's 64 of a shared last group
            const bool lo = r < full || !paired || (wave & 1) == 0, hi = r < full || !paired || (wave & 1) == 1;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                if (t < w.Tn) {
                    const MfmaDeq d = dsel.setup(sz[t]);
                    auto word = [&](uint32_t P, int j) {
                        const v8bf wa = mfma_dequant<F16>(P, d, kx);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, xf[j][mt], acc[t][mt], 0, 0, 0);
                    };
                    if (lo) {
                        word(cur.c[t].x, 0);
                        word(cur.c[t].y, 1);
                    }
                    if (hi) {
                        word(cur.c[t].z, 2);
                        word(cur.c[t].w, 3);
                    }
                }
            }
        };
        Group g;
        load_x(group_of(0));
        load_w(g, group_of(0));
        for (int r = 0; r < nr; ++r) round(r, g);
    };
    if (nr > 0) {
        if (w.f16) walk(std::true_type{});
        else walk(std::false_type{});
    }

    // sums: [wave w < 4][tile][row][16 columns] fp32 in LDS, over the x.  D of
    // the 16x16 op: lane l holds columns 4 (l >> 4) + v of row l & 15
    lds_barrier();
    float *sums = (float *)smem;
    auto at = [&](int t, int mt) {
        return sums + ((size_t)((wave & (kHalf - 1)) * TN + t) * ROWS + 16 * mt + lm) * 16 + 4 * lg;
    };
    if (wave >= kHalf) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (t < w.Tn) *(v4f *)at(t, mt) = acc[t][mt];
    }
    lds_barrier();
    if (wave < kHalf) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (t < w.Tn) *(v4f *)at(t, mt) = acc[t][mt] + *(const v4f *)at(t, mt);
    }
    lds_barrier();
    write_sums<kHalf>(a, w, sums, TN, ROWS);
}

template <int MT, bool SYM>
static FwdKernel pick_mid_rows(int tn) {
    switch (tn) {
        case 1: return k_mid<MT, 1, SYM>;
        case 2: return k_mid<MT, 2, SYM>;
        case 3: return k_mid<MT, 3, SYM>;
        case 4: return k_mid<MT, 4, SYM>;
        case 5: return k_mid<MT, 5, SYM>;
    }
    if constexpr (mid_tiles_max(MT) >= 6)
        if (tn == 6) return k_mid<MT, 6, SYM>;
    if constexpr (mid_tiles_max(MT) >= 8) {
        if (tn == 7) return k_mid<MT, 7, SYM>;
        if (tn == 8) return k_mid<MT, 8, SYM>;
    }
    return nullptr;
}

FwdKernel pick_mid(int mrows, int tn, bool symmetric) {
    switch (mrows) {
        case 32: return symmetric ? pick_mid_rows<2, true>(tn) : pick_mid_rows<2, false>(tn);
        case 48: return symmetric ? pick_mid_rows<3, true>(tn) : pick_mid_rows<3, false>(tn);
        case 64: return symmetric ? pick_mid_rows<4, true>(tn) : pick_mid_rows<4, false>(tn);
    }
    return nullptr;
}

}  // namespace qlin
