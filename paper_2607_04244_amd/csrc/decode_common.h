// Device code shared by the decode kernels (kernels.hip, mid.hip; tiled.hip uses on_route): a
// workgroup's share of a launch, and the exchange of split-K partial sums.
#pragma once

#include "device_common.h"

#include <type_traits>

namespace qlin {

// Calls walk(std::bool_constant<f16 route>): for a mixed launch by the member's
// route (uniform in the workgroup: its tiles belong to one member).  A walk
// includes its first loads, so that none in flight is copied between the two
// routes' registers.
template <Route R, typename Walk>
__device__ inline void on_route(bool member_f16, const Walk &walk) {
    if constexpr (R == kRouteMixed) {
        if (member_f16) walk(std::true_type{});
        else walk(std::false_type{});
    } else {
        walk(std::bool_constant<R == kRouteF16>{});
    }
}

// Column range, member and K chunk of workgroup `bid`: chunk c, range jn
// (over all members), the member's tiles [t0, t0 + Tn) and groups
// [g0, g0 + Kc), and the member's weights and output.
struct WgWork {
    int c, jn, t0, Tn, g0, Kc;
    const uint4 *codes;
    const void *sz;
    uint16_t *y;
    int N;
    bool f16;
    float unscale;           // what the sums are multiplied by before their rounding (F16 route)
};
// Everything here is wave-uniform scalar work at the start of the kernel:
// the arguments arrive in one batch of scalar loads (the range starts are one
// contiguous array, every index static, and the chunk needs no division),
// then the member's fields in one more.
template <Route R>
__device__ inline WgWork wg_work(const FwdArgs &a, int bid) {
    WgWork w;
    w.c = gn_chunk(bid, a.Gn, a.inv_gn, a.gn_shift);
    w.jn = bid - w.c * a.Gn;
    int m = 0, g0 = 0;                        // the member owning range jn, its first range
#pragma unroll
    for (int i = 1; i < kMaxMembers; ++i)
        if (w.jn >= a.gn0[i]) {
            m = i;
            g0 = a.gn0[i];
        }
    // one scalar load of the member's fields at a computed offset (reading a
    // member at a fixed index as well would make the compiler copy the
    // whole argument block to scratch memory)
    const FwdMember &f = a.mem[m];
    w.codes = f.codes;
    w.sz = f.sz;
    w.y = f.y;
    w.N = f.N;
    w.f16 = R == kRouteMixed ? f.f16 != 0 : R == kRouteF16;
    w.unscale = w.f16 ? kF16Unscale : 1.0f;
    const int j = w.jn - g0;
    w.t0 = j * f.Nq + min(j, f.Nr);
    w.Tn = f.Nq + (j < f.Nr ? 1 : 0);
    w.g0 = w.c * a.Kq + min(w.c, a.Kr);
    w.Kc = a.Kq + (w.c < a.Kr ? 1 : 0);
    return w;
}

// Split-K partial sums travel between workgroups that may sit on different
// XCDs, whose L2 caches are not coherent with each other for ordinary
// accesses.  They are written and read with agent-scope (sc1) buffer
// accesses, which the hardware performs at the device coherence point; an
// agent-scope release/acquire fence instead would write back and invalidate
// the whole L2 of the XCD on every arrival.  Workgroup (c, jn) owns a
// contiguous region of TnMax * M * 16 fp32 at ((c * Gn + jn) * TnMax * M * 16),
// item it = (tile * M + m) * 2 + half at float offset 8 * it, so the 16-byte
// accesses of a wave are contiguous.

__device__ inline __amdgpu_buffer_rsrc_t ws_rsrc(const FwdArgs &a) {
    return __builtin_amdgcn_make_buffer_rsrc(a.ws, 0, (int)a.ws_bytes, kRsrcFlags);
}
__device__ inline uint32_t ws_region(const FwdArgs &a, int c, int jn) {      // byte offset
    return (uint32_t)((c * a.Gn + jn) * a.TnMax * a.M) * 64u;
}
// The four sums of quarter row `it` of the workgroup's output (row m,
// columns n .. n + 3): bf16 straight to y when the whole K range is covered,
// else fp32 partials to the workspace, quarter it at float offset 4 it of the
// region (half row h = (tile * M + m) * 2 + half is quarters 2h and 2h + 1).
__device__ inline void store_quarter(const FwdArgs &a, const WgWork &w, int it, int m, int n, const float s[4],
                                     bool direct) {
    if (direct) {
        const float u = w.unscale;
        *(uint2 *)(w.y + (size_t)m * w.N + n) =
            make_uint2(cvt_pk_bf16(s[0] * u, s[1] * u), cvt_pk_bf16(s[2] * u, s[3] * u));
    } else {
        const uint32_t off = ws_region(a, w.c, w.jn) + (uint32_t)it * 16u;
        __builtin_amdgcn_raw_buffer_store_b128(
            v4u{__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])},
            ws_rsrc(a), off, 0, kSc1);
    }
}

// The last of the S workgroups of a column range adds the S fp32 partials in
// chunk order (fixed order) and writes y.
__device__ inline void reduce_chunks(const FwdArgs &a, const WgWork &w) {
    const int tid = threadIdx.x;
    const int items = w.Tn * a.M * 2;
    // Every wave waits until its partial-sum stores have completed at the
    // device coherence point before the barrier; one relaxed atomic per
    // workgroup then counts the arrival.  The last arrival reads the other
    // workgroups' partials with agent-scope loads, which do not hit stale
    // cached copies.
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const uint32_t old = __hip_atomic_fetch_add(&a.counters[w.jn], 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        s_last = (old == (uint32_t)(a.S - 1));
    }
    __syncthreads();
    if (!s_last) return;
    const __amdgpu_buffer_rsrc_t r = ws_rsrc(a);
    const uint32_t inv_pt = 0xFFFFFFFFu / (uint32_t)(a.M * 2) + 1u;   // as in write_sums()
    for (int it = tid; it < items; it += kThreads) {
        const int tl = (int)__umulhi((uint32_t)it, inv_pt);
        const int rem = it - tl * a.M * 2;
        const int m = rem >> 1, hh = rem & 1;
        const size_t n = (size_t)(w.t0 + tl) * kTileN + 8 * hh;
        // partials of kBatch chunks are loaded together (one memory round
        // trip per batch, not per chunk), then added in chunk order
        constexpr int kBatch = 8;
        float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int c0 = 0; c0 < a.S; c0 += kBatch) {
            v4u v[kBatch][2];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int cc = min(c0 + u, a.S - 1);      // unconditional load; extra ones are not added
                const uint32_t off = ws_region(a, cc, w.jn) + (uint32_t)it * 32u;
                v[u][0] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kSc1);
                v[u][1] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, kSc1);
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (c0 + u < a.S)
#pragma unroll
                    for (int i = 0; i < 8; ++i) s[i] += __uint_as_float(v[u][i >> 2][i & 3]);
        }
        const float un = w.unscale;
        uint4 o;
        o.x = cvt_pk_bf16(s[0] * un, s[1] * un);
        o.y = cvt_pk_bf16(s[2] * un, s[3] * un);
        o.z = cvt_pk_bf16(s[4] * un, s[5] * un);
        o.w = cvt_pk_bf16(s[6] * un, s[7] * un);
        *(uint4 *)(w.y + (size_t)m * w.N + n) = o;
    }
    if (tid == 0) __hip_atomic_store(&a.counters[w.jn], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Writes the workgroup's results from SETS partial sums per column tile in
// LDS: set i of tile tl from row (i * tiles + tl) * rows of 16 fp32 columns, in
// the order of sums_unit() (sets that hold nothing for a tile are zero).  The sets of an item are added
// in order; with the whole K range covered (S == 1) the sum goes to y as bf16,
// otherwise to the fp32 workspace, and the last of the S workgroups of this
// column range adds the S partials in chunk order and writes y.  Every sum
// runs in a fixed order, so results do not depend on timing: repeated calls
// give identical bits.
//
// The loop strides by the compile-time workgroup size: blockDim.x would be a
// scalar load of the dispatch's hidden arguments here, after the main loop,
// and that load misses the scalar cache and costs a memory round trip on the
// workgroup's critical path.
//
// An item's reads do not depend on each other: all SETS of them are issued
// before the first add.  Adding zero sets leaves a sum's bits unchanged (the
// sum starts at +0), so no test of which sets hold a tile is needed.
template <int SETS>
__device__ inline void write_sums(const FwdArgs &a, const WgWork &w, const float *sums, int tiles, int rows) {
    const int tid = threadIdx.x;
    const int per_tile = a.M * 4;                  // items (quarter rows of 4 columns) per tile
    const int items = w.Tn * per_tile;
    const bool direct = (a.S == 1);
    // tile of an item: a multiply-high by ceil(2^32 / per_tile), exact since
    // items and per_tile stay below 2^16
    const uint32_t inv_pt = 0xFFFFFFFFu / (uint32_t)per_tile + 1u;
    for (int it = tid; it < items; it += kThreads) {
        const int tl = (int)__umulhi((uint32_t)it, inv_pt);
        const int rem = it - tl * per_tile;
        const int m = rem >> 2, qq = rem & 3;
        float4 v[SETS];
#pragma unroll
        for (int i = 0; i < SETS; ++i)
            v[i] = *(const float4 *)(sums + (size_t)(i * tiles + tl) * rows * 16 + 4 * sums_unit(m, qq));
        float s[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < SETS; ++i) {
            s[0] += v[i].x;
            s[1] += v[i].y;
            s[2] += v[i].z;
            s[3] += v[i].w;
        }
        store_quarter(a, w, it, m, (w.t0 + tl) * kTileN + 4 * qq, s, direct);
    }
    if (!direct) reduce_chunks(a, w);
}

}  // namespace qlin
