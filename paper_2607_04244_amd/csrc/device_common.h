// Device-side building blocks shared by the kernels (kernels.hip, mid.hip,
// tiled.hip and, for its vector types and cross-lane helpers, attn.hip): vector
// types, the block layout, the nibble extraction and the two exact
// dequantization routes.  Header-only, inline.
#pragma once

#include "qlin_internal.h"

namespace qlin {

typedef __attribute__((address_space(3))) void lds_void_t;   // LDS, for direct-to-LDS loads
typedef __attribute__((address_space(1))) void glb_void_t;   // global memory

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ layout

// Column (within the tile) and k (within the group) of nibble p of word j of lane l.
__host__ __device__ inline void block_coord(int l, int j, int p, int &n16, int &k128) {
    const int r = 2 * (p & 1) + (p >> 2);
    const int h = (p >> 1) & 1;
    n16 = 4 * ((l >> 2) & 3) + r;
    k128 = 32 * j + 8 * (l >> 4) + 4 * h + (l & 3);
}

// Buffer-resource constants.  Cross-workgroup partial sums travel between
// workgroups that may sit on different XCDs, whose L2 caches are not coherent
// with each other for ordinary accesses: they are written and read with
// agent-scope (sc1) buffer accesses, which the hardware performs at the
// device coherence point.
constexpr int kSc1 = 16;                 // cache-policy operand of the buffer builtins: sc1 (agent scope)
constexpr int kRsrcFlags = 0x00020000;   // buffer descriptor word 3: 32-bit raw data

// ------------------------------------------------------------------ small helpers

__device__ inline uint32_t cvt_pk_bf16(float lo, float hi) {
    v2f f = {lo, hi};
    v2bf b = __builtin_convertvector(f, v2bf);   // round to nearest even
    return __builtin_bit_cast(uint32_t, b);
}

__device__ inline uint16_t cvt_bf16(float v) {
    __bf16 b = (__bf16)v;
    return __builtin_bit_cast(uint16_t, b);
}

__device__ inline float bf16_lo_to_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi_to_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Two exact routes turn a packed word into bf16 weights; a handle's scales
// decide at creation which one its s|z words are stored for.
//
// F16 = true (every scale in [2^-25, 2^4)): the codes enter the dequantizing
// product as f16 subnormals.  A nibble at bits 0-3 of a 16-bit half is the f16
// number q 2^-24 and one at bits 4-7 is q 2^-20, so a word needs one shift and
// four ANDs for its eight codes, and no exponent bits are OR-ed in.  The
// matrix op takes f16 subnormals exactly (checked over 2 million products of
// every code with scales across the range).  The scale is stored as
// s 2^kF16Exp in f16 (8 significant bits: exact), divided by 16 in the columns
// r >= 2 of a 4-column block, whose codes sit at bits 4-7.  All weights then
// come out multiplied by 2^(kF16Exp - 24), exactly, so they round to the same
// bf16 significands, and the sum is multiplied by kF16Unscale before its one
// rounding.  The matrix cores keep binary32's subnormals, so sums stay as exact
// as on the other route while products x w are above 2^-114; below, they are
// multiples of 2^-137 (not 2^-149), 1/16 of the smallest bf16 step: outputs in
// bf16's own subnormal range, below 2^-126, may be off by a step more (measured at
// 2^-128: relative error 7.2e-3 against 5.8e-3; from 2^-124 up no difference).
//
// F16 = false (any scale in [2^-100, 2^100]): 0x4300 | q is the bf16 number
// 128 + q: three shifts and four v_and_or_b32 per word.
//
// Measured per word (cycles a wave64 instruction holds a SIMD with 2 waves on
// it): v_and_b32 of two VGPRs and v_lshrrev_b32 2.7, v_and_or_b32 4.6,
// v_cvt_pk_bf16_f32 4.6, the 4x4x4 matrix op 8.2: 13.5 against 26.5 cycles of
// extraction per eight weights.
constexpr int kF16Exp = 12;
constexpr float kF16Unscale = 4096.0f;     // 2^(24 - kF16Exp)

struct Pairs { uint32_t a0, a1, a2, a3; };

// Masks of the extraction; in registers (gfx9 VOP3 takes no literal, and an
// AND with a scalar operand issues at half the rate of one with two vector
// operands), opaque to the optimizer so that they stay there.
template <bool F16>
struct ExtractConsts;
template <>
struct ExtractConsts<false> {
    uint32_t mask, magic;
    __device__ inline ExtractConsts() {
        mask = __builtin_amdgcn_readfirstlane(0x000F000Fu);
        magic = 0x43004300u;                        // bf16 128.0 in both halves
        asm volatile("" : "+v"(magic));
    }
    // the four "128 + q" bf16 pairs: pair i holds nibbles i (low half) and i + 4 (high half)
    __device__ inline Pairs pairs(uint32_t P) const {
        Pairs o;
        o.a0 = (P & mask) | magic;
        o.a1 = ((P >> 4) & mask) | magic;
        o.a2 = ((P >> 8) & mask) | magic;
        o.a3 = ((P >> 12) & mask) | magic;
        return o;
    }
};
template <>
struct ExtractConsts<true> {
    uint32_t lo, hi;
    __device__ inline ExtractConsts() {
        lo = 0x000F000Fu;
        hi = 0x00F000F0u;
        asm volatile("" : "+v"(lo), "+v"(hi));
    }
    // the same four pairs as f16 q 2^-24 (a0, a2) and q 2^-20 (a1, a3)
    __device__ inline Pairs pairs(uint32_t P) const {
        const uint32_t p8 = P >> 8;
        return Pairs{P & lo, P & hi, p8 & lo, p8 & hi};
    }
};

// One lane's 16 bytes of a weight block.
__device__ inline uint4 load_block(const uint4 *codes, size_t idx) { return codes[idx]; }

// Cache policy of the decode kernels' weight loads: non-temporal.  A forward
// reads every weight once, so streaming them with this hint keeps them from
// displacing x, y and the partial sums in L2 and the last-level cache (the
// tiled kernel keeps ordinary loads: the row blocks of a column block reuse
// its weights from L2).
constexpr int kWeightPolicy = 2;   // cache-policy operand of the buffer builtins: nt
__device__ inline uint4 load_block_nt(const uint4 *codes, size_t idx) {
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const v4u *)codes + idx));
}

// Per (column, group) dequantization word of lane l's column n16 = l & 15 of a
// tile.  What is stored, and loaded by load_sz:
//   F16 = false, zero-points: bf16 s in the low half, bf16 zc = -(128 + z) in
//     the high half (exact: an integer of 8 significant bits), so that
//     (128 + q) * s + zc * s = (q - z) * s;
//   F16 = true, zero-points: f16 s' (see above) in the half of the column's
//     parity (low for even columns, where the diagonal operand needs it), and
//     in the other half the f16 subnormal zc = -z 2^-24 (-z 2^-20 for columns
//     r >= 2), so that s' * zc is the offset of the scaled weights;
//   symmetric: 16 bits of s or s' per column; a lane loads the 32-bit pair of
//     columns that holds its own, and z = 8 is supplied by the kernel.
constexpr uint32_t kZcSymmetric = 0xC308u;      // bf16 -136
constexpr uint32_t kSzBytesSym = 2, kSzBytesAsym = 4;

// f16 zero-point offset of column n16 (z integer in [0, 15])
__host__ __device__ inline uint32_t f16_zc(uint32_t z, int n16) { return 0x8000u | ((n16 & 2) ? z << 4 : z); }

template <bool SYM>
__device__ inline uint32_t sz_offset_bytes(int n16) { return SYM ? (uint32_t)(n16 >> 1) * 4u : (uint32_t)n16 * 4u; }

template <bool SYM>
__device__ inline uint32_t load_sz(const void *sz, size_t block, int n16) {
    return *(const uint32_t *)((const char *)sz + block * (kTileN * (SYM ? kSzBytesSym : kSzBytesAsym)) +
                               sz_offset_bytes<SYM>(n16));
}
template <bool SYM>
__device__ inline uint32_t load_sz_nt(const void *sz, size_t block, int n16) {   // non-temporal, as load_block_nt
    return __builtin_nontemporal_load(
        (const uint32_t *)((const char *)sz + block * (kTileN * (SYM ? kSzBytesSym : kSzBytesAsym)) +
                           sz_offset_bytes<SYM>(n16)));
}

__device__ inline float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, a), __builtin_bit_cast(v2bf, b), c, false);
}

// --- matrix-core dequantization ------------------------------------------

struct MfmaDeq { v4s bdiag; v4f c4; };

// Per-lane constants (column l & 15) that turn a loaded dequantization word
// into B = diag(s) in the 4x4 block layout (lane l supplies B[r][l & 3],
// non-zero only for r = l & 3: element l & 3 of four 16-bit elements) and the
// offset C = zc * s.  Built once per kernel.
template <bool SYM, bool F16>
struct DeqSel;

template <bool SYM>
struct DeqSel<SYM, false> {
    uint32_t s0, s1, half;          // byte selectors (v_perm_b32)
    __device__ inline explicit DeqSel(int lane) {
        constexpr uint32_t kLo = 0x0C0C0100u, kHi = 0x01000C0Cu, kZero = 0x0C0C0C0Cu;
        const int r = lane & 3;
        s0 = r == 0 ? kLo : r == 1 ? kHi : kZero;
        s1 = r == 2 ? kLo : r == 3 ? kHi : kZero;
        half = (lane & 1) ? 0x05040302u : 0x05040100u;    // this column's half of the pair, zc above it
    }
    __device__ inline uint32_t word(uint32_t raw) const {
        if constexpr (SYM) return __builtin_amdgcn_perm(kZcSymmetric, raw, half);
        else return raw;
    }
    __device__ inline MfmaDeq setup(uint32_t raw) const {
        const uint32_t sz = word(raw);
        const float c = dot2(sz, sz >> 16, 0.0f);         // s * zc, exactly (one bf16 product, plus 0)
        MfmaDeq d;
        d.bdiag = __builtin_bit_cast(v4s, v2u{__builtin_amdgcn_perm(sz, sz, s0), __builtin_amdgcn_perm(sz, sz, s1)});
        d.c4 = v4f{c, c, c, c};
        return d;
    }
};

template <bool SYM>
struct DeqSel<SYM, true> {
    uint32_t m0, m1, own, zc;       // halves of the two dwords of B; this column's half of a pair; z = 8
    __device__ inline explicit DeqSel(int lane) {
        const int r = lane & 3;
        own = (r & 1) ? 0xFFFF0000u : 0x0000FFFFu;
        m0 = r < 2 ? own : 0u;
        m1 = r < 2 ? 0u : own;
        zc = f16_zc(8, r) << ((r & 1) ? 0 : 16);
    }
    __device__ inline MfmaDeq setup(uint32_t raw) const {
        const uint32_t sz = SYM ? ((raw & own) | zc) : raw;
        float c;                                          // s' * zc, exactly (12 significant bits)
        asm("v_fma_mix_f32 %0, %1, %1, 0 op_sel:[0,1,0] op_sel_hi:[1,1,0]" : "=v"(c) : "v"(sz));
        MfmaDeq d;
        d.bdiag = __builtin_bit_cast(v4s, v2u{raw & m0, raw & m1});
        d.c4 = v4f{c, c, c, c};
        return d;
    }
};

// Dequantize one packed word into the 8 bf16 A-operand values of
// v_mfma_f32_16x16x32_bf16 (row n = l & 15): element e holds
// w[n][32j + 8(l >> 4) + e] (times 2^(kF16Exp - 24) for F16).
template <bool F16>
__device__ inline v8bf mfma_dequant(uint32_t P, const MfmaDeq &d, const ExtractConsts<F16> &k) {
    const Pairs a = k.pairs(P);
    const v2u A0 = {a.a0, a.a1}, A1 = {a.a2, a.a3};
    v4f d0, d1;
    if constexpr (F16) {
        d0 = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(v4h, A0), __builtin_bit_cast(v4h, d.bdiag), d.c4, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(v4h, A1), __builtin_bit_cast(v4h, d.bdiag), d.c4, 0, 0, 0);
    } else {
        d0 = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(v4s, A0), d.bdiag, d.c4, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(v4s, A1), d.bdiag, d.c4, 0, 0, 0);
    }
    const v4u w = {cvt_pk_bf16(d0[0], d0[1]), cvt_pk_bf16(d0[2], d0[3]),
                   cvt_pk_bf16(d1[0], d1[1]), cvt_pk_bf16(d1[2], d1[3])};
    return __builtin_bit_cast(v8bf, w);
}

// --- vector-ALU dequantization -------------------------------------------

// Constants for the four columns n = 16 t + 4 * ((l >> 2) & 3) + r of lane l.
// The scales are the weights' own on either route: the vector unit flushes
// binary32's subnormals, so scaled sums would vanish 2^12 earlier.
struct ValuDeq { uint32_t sl[4], sh[4]; float c[4]; };

// v[r]: what a handle stores for column r (the 32-bit word, or for symmetric
// handles the 16 bits in the half of the column's parity).
template <bool SYM>
__device__ inline ValuDeq valu_setup(const uint32_t v[4], bool f16) {
    ValuDeq d;
    if (f16) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint16_t own = (uint16_t)((r & 1) ? v[r] >> 16 : v[r]);
            const float s = (float)__builtin_bit_cast(_Float16, own) * __builtin_ldexpf(1.0f, r >= 2 ? 4 - kF16Exp : -kF16Exp);
            d.sh[r] = __float_as_uint(s);          // 8 significant bits: the bf16 pair (0, s)
            d.sl[r] = d.sh[r] >> 16;               // bf16 pair (s, 0)
            if constexpr (SYM) {
                d.c[r] = s * -136.0f;
            } else {
                float p;                           // -z s, scaled as on the matrix-core route (DeqSel)
                asm("v_fma_mix_f32 %0, %1, %1, 0 op_sel:[0,1,0] op_sel_hi:[1,1,0]" : "=v"(p) : "v"(v[r]));
                d.c[r] = __builtin_fmaf(p, kF16Unscale, s * -128.0f);   // -(128 + z) * s, exactly
            }
        }
        return d;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t sz = SYM ? (((r & 1) ? v[r] >> 16 : v[r] & 0xFFFFu) | (kZcSymmetric << 16)) : v[r];
        d.c[r] = dot2(sz, sz >> 16, 0.0f);   // -(128 + z) * s
        d.sl[r] = sz & 0xFFFFu;      // bf16 pair (s, 0)
        d.sh[r] = sz << 16;          // bf16 pair (0, s)
    }
    return d;
}

// Dequantize one packed word: pr[r] = bf16 pair (w[n_r][k0], w[n_r][k0 + 4]) with
// k0 = 32j + 8(l >> 4) + (l & 3).
__device__ inline void valu_dequant(uint32_t P, const ValuDeq &d, const ExtractConsts<false> &k, uint32_t pr[4]) {
    const Pairs a = k.pairs(P);
    const float w00 = dot2(a.a0, d.sl[0], d.c[0]), w01 = dot2(a.a0, d.sh[1], d.c[1]);
    const float w02 = dot2(a.a1, d.sl[2], d.c[2]), w03 = dot2(a.a1, d.sh[3], d.c[3]);
    const float w10 = dot2(a.a2, d.sl[0], d.c[0]), w11 = dot2(a.a2, d.sh[1], d.c[1]);
    const float w12 = dot2(a.a3, d.sl[2], d.c[2]), w13 = dot2(a.a3, d.sh[3], d.c[3]);
    pr[0] = cvt_pk_bf16(w00, w10);
    pr[1] = cvt_pk_bf16(w01, w11);
    pr[2] = cvt_pk_bf16(w02, w12);
    pr[3] = cvt_pk_bf16(w03, w13);
}

// ------------------------------------------------------------------ LDS staging

// One direct-to-LDS 16-byte load per lane: lane l's 16 bytes from src land
// at lds_dst + 16 l (lds_dst uniform across the wave).  Issued as inline
// assembly so that the compiler does not track it: its wait-count pass
// handles direct-to-LDS writes coarsely and would drain every outstanding
// load before each later LDS read.  The caller waits for it explicitly
// (s_waitcnt vmcnt) before the barrier that publishes the data; loads the
// compiler does track and issues later are younger, so its own waits stay
// sufficient.  These statements set m0 themselves and list it as clobbered;
// the compiler warns that it may not preserve a reserved register across
// them, which matters only if it kept a value of its own in m0: the
// generated code of every kernel here has no other m0 access.
__device__ inline void load_lds_x16(const void *src, const uint4 *lds_dst) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(m0), "v"(src) : "memory", "m0");
}

// The same with the non-temporal hint, for data a call reads once.
__device__ inline void load_lds_x16_nt(const void *src, const uint4 *lds_dst) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off nt" :: "s"(m0), "v"(src) : "memory", "m0");
}

// The same with 4 bytes per lane: lane l's dword lands at lds_dst + 4 l.
__device__ inline void load_lds_x4(const void *src, const void *lds_dst) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" :: "s"(m0), "v"(src) : "memory", "m0");
}

// LDS byte address of p (wave-uniform), as a scalar.
__device__ inline uint32_t lds_addr(const void *p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p);
}

// Direct-to-LDS buffer loads: lane l's 16 (4) bytes at byte offset
// voff + soff of the resource land at LDS byte address lds + 16 l (4 l).
// Inline assembly for the same reason as load_lds_x16; lds and soff are
// scalars, so a load whose per-lane offset is fixed costs no vector work.
__device__ inline void load_lds_buf16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}
__device__ inline void load_lds_buf4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}

// Barrier for LDS hand-off only.  __syncthreads() also waits for every
// outstanding global load, which would drain the weight prefetch.
__device__ inline void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace qlin
