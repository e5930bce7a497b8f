// Device-side building blocks of the LUT build and correction kernels:
// the binary64 LUT entry, the XCD-aware tile order, and the correction tile
// with its three ways of reading the strip's LUT rows. Shared by the plain
// kernels (lut_build.hip, lut_apply.hip) and the persistent batch kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// The LUT entry is a fixed sequence of binary64 operations: no contraction
// into fused multiply-adds anywhere in this translation unit (the build also
// passes -ffp-contract=off).
#pragma clang fp contract(off)

namespace rc {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// LUT entry for integer level v (§I LUT generation, definition in rc.h):
// Horner from the cubic coefficient down, one rounding per operation, then
// round half away from zero and clamp to [0, L-1]; top is L-1.
// The rounding and clamp are done as r = cvt(acc + h) with h = 0.5 - 2^-54
// (the double just below 1/2) and v_cvt_u32_f64, which truncates, sends NaN,
// -Inf and every negative to 0 and +Inf and everything above 2^32 to 2^32 - 1,
// then min(r, L-1). For 0 <= acc < 2^52, trunc(fl(acc + h)) is
// round-half-away(acc): if frac(acc) >= 1/2 the exact sum is at least n -
// 2^-54 for n = ceil(acc), and it only falls below n when acc = n - 1/2, where
// n - 2^-54 rounds up to n (a tie to even at n = 1, nearer n above); if
// frac(acc) < 1/2 the exact sum is at most floor(acc) + 1 - ulp(acc) - 2^-54,
// more than half an ulp below floor(acc) + 1, so it cannot round up to it.
// With plain 1/2 instead of h, acc = 1/2 - 2^-54 would round to 1. For acc >=
// 2^52 both the rounded value and r exceed every L; for acc < 0 the sum is
// below 1, so r = 0.
__device__ __forceinline__ uint32_t lut_round(double a0, double a1, double a2, double a3,
                                              double x) {
    double acc = a3;
    acc = acc * x;
    acc = acc + a2;
    acc = acc * x;
    acc = acc + a1;
    acc = acc * x;
    acc = acc + a0;
    const double sum = acc + 0x1.fffffffffffffp-2;
    uint32_t r;
    // As an instruction: the C++ conversion is undefined out of range, and the
    // saturation replaces a maximum and a minimum in binary64.
    asm("v_cvt_u32_f64 %0, %1" : "=v"(r) : "v"(sum));
    return r;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Entries of two consecutive levels, packed: the conversion to 16 bits
// saturates, then one packed minimum with top in both halves.
__device__ __forceinline__ uint32_t lut_pair(double a0, double a1, double a2, double a3, double x0,
                                             double x1, uint32_t top2) {
    const uint32_t p = __builtin_bit_cast(
        uint32_t, __builtin_amdgcn_cvt_pk_u16(lut_round(a0, a1, a2, a3, x0),
                                              lut_round(a0, a1, a2, a3, x1)));
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_min(__builtin_bit_cast(u16x2, p),
                                                        __builtin_bit_cast(u16x2, top2)));
}

// The 8 entries of levels x[0] .. x[7], two per word.
__device__ __forceinline__ u32x4 lut_eight(double a0, double a1, double a2, double a3,
                                           const double (&x)[8], uint32_t top2) {
    return u32x4{lut_pair(a0, a1, a2, a3, x[0], x[1], top2),
                 lut_pair(a0, a1, a2, a3, x[2], x[3], top2),
                 lut_pair(a0, a1, a2, a3, x[4], x[5], top2),
                 lut_pair(a0, a1, a2, a3, x[6], x[7], top2)};
}

// Workgroups are dispatched round-robin over the XCDs (block i runs on XCD
// i mod X). Renumber them so that XCD x receives one contiguous range of
// logical tiles: neighbouring tiles then share that XCD's L2.
__device__ __forceinline__ int xcd_tile(int i, int G, int X) {
    if (X <= 1) return i;
    const int q = G / X, r = G - (G / X) * X;
    const int x = i % X, k = i / X;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// VEC pixels of one line held by one lane.
template <int VEC> struct Px;
template <> struct Px<1> { typedef unsigned short T; };
template <> struct Px<2> { typedef unsigned int T; };
template <> struct Px<4> { typedef u32x2 T; };
template <> struct Px<8> { typedef u32x4 T; };

template <int VEC> constexpr int log_vec() {
    return VEC == 1 ? 0 : (VEC == 2 ? 1 : (VEC == 4 ? 2 : 3));
}

// Applies f(k, dn_k) to the VEC 16-bit DNs held in w and packs the results.
template <int VEC, typename F>
__device__ __forceinline__ typename Px<VEC>::T map_px(typename Px<VEC>::T w, F f) {
    if constexpr (VEC == 1) {
        return (unsigned short)f(0, (uint32_t)w);
    } else if constexpr (VEC == 2) {
        return f(0, w & 0xffffu) | (f(1, w >> 16) << 16);
    } else if constexpr (VEC == 4) {
        u32x2 r;
        r.x = f(0, w.x & 0xffffu) | (f(1, w.x >> 16) << 16);
        r.y = f(2, w.y & 0xffffu) | (f(3, w.y >> 16) << 16);
        return r;
    } else {
        u32x4 r;
        r.x = f(0, w.x & 0xffffu) | (f(1, w.x >> 16) << 16);
        r.y = f(2, w.y & 0xffffu) | (f(3, w.y >> 16) << 16);
        r.z = f(4, w.z & 0xffffu) | (f(5, w.z >> 16) << 16);
        r.w = f(6, w.w & 0xffffu) | (f(7, w.w >> 16) << 16);
        return r;
    }
}

// As map_px, with a second set of VEC 16-bit values: f(k, a_k, b_k).
template <int VEC, typename F>
__device__ __forceinline__ typename Px<VEC>::T map_px2(typename Px<VEC>::T a,
                                                       typename Px<VEC>::T b, F f) {
    if constexpr (VEC == 1) {
        return (unsigned short)f(0, (uint32_t)a, (uint32_t)b);
    } else if constexpr (VEC == 2) {
        return f(0, a & 0xffffu, b & 0xffffu) | (f(1, a >> 16, b >> 16) << 16);
    } else {
        typename Px<VEC>::T r;
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i)
            r[i] = f(2 * i, a[i] & 0xffffu, b[i] & 0xffffu) |
                   (f(2 * i + 1, a[i] >> 16, b[i] >> 16) << 16);
        return r;
    }
}

// Raw buffer resource over `bytes` bytes from `base` (gfx9-family word 3:
// untyped 32-bit data). Buffer loads past `bytes` return 0 and stores past
// it are dropped, so a tile's last partial pass needs no per-line guard.
constexpr int kRsrcWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             kRsrcWord3);
}

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Image cache policy NT -> the cache-policy bits of the buffer loads and
// stores (gfx950: bit 0 sc0, bit 1 nt, bit 4 sc1):
//   0 default,  1 nt loads and stores,  2 nt stores,
//   3 sc0 loads + nt stores,  4 sc1 loads + nt stores,  5 sc0 loads.
constexpr int kPolicies = 6;
constexpr int ld_aux(int nt) { return nt == 1 ? 2 : (nt == 3 || nt == 5 ? 1 : (nt == 4 ? 16 : 0)); }
constexpr int st_aux(int nt) { return nt >= 1 && nt <= 4 ? 2 : 0; }

// VEC pixels of one line through a buffer resource: per-lane byte offset
// `vo` (VGPR) plus a wave-uniform line offset `so` (SGPR); NT is the image
// cache policy above.
template <int VEC, int NT> struct Buf;
template <int NT> struct Buf<1, NT> {
    static __device__ __forceinline__ unsigned short ld(__amdgpu_buffer_rsrc_t r, uint32_t vo,
                                                        uint32_t so) {
        return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)vo, (int)so,
                                                                    ld_aux(NT));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                              unsigned short v) {
        __builtin_amdgcn_raw_buffer_store_b16((short)v, r, (int)vo, (int)so, st_aux(NT));
    }
};
template <int NT> struct Buf<2, NT> {
    static __device__ __forceinline__ unsigned int ld(__amdgpu_buffer_rsrc_t r, uint32_t vo,
                                                      uint32_t so) {
        return (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so,
                                                                  ld_aux(NT));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                              unsigned int v) {
        __builtin_amdgcn_raw_buffer_store_b32((int)v, r, (int)vo, (int)so, st_aux(NT));
    }
};
template <int NT> struct Buf<4, NT> {
    static __device__ __forceinline__ u32x2 ld(__amdgpu_buffer_rsrc_t r, uint32_t vo,
                                               uint32_t so) {
        return (u32x2)__builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, ld_aux(NT));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                              u32x2 v) {
        __builtin_amdgcn_raw_buffer_store_b64((i32x2)v, r, (int)vo, (int)so, st_aux(NT));
    }
};
template <int NT> struct Buf<8, NT> {
    static __device__ __forceinline__ u32x4 ld(__amdgpu_buffer_rsrc_t r, uint32_t vo,
                                               uint32_t so) {
        return (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, (int)so, ld_aux(NT));
    }
    // A store of more than 8 bytes reads its data registers after issue; the
    // compiler only keeps the next VALU off them when soffset is not a
    // register (measured on gfx950: with the line offset in an SGPR, the loop
    // counter update right after the store overwrote its first dword). The
    // whole offset therefore goes in the VGPR, soffset is the constant 0.
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                              u32x4 v) {
        __builtin_amdgcn_raw_buffer_store_b128((i32x4)v, r, (int)(vo + so), 0, st_aux(NT));
    }
};

// Streams `passes` passes over a tile's lines. In each pass a lane handles
// its VEC pixels of UNROLL lines (line_stride bytes apart); consecutive
// passes start pass_adv bytes apart (0: UNROLL * line_stride, contiguous
// lines; a multiple of it when a tile takes every k-th pass). Software
// pipelined with two register sets used alternately: the loads of pass k+1
// are issued before pass k is gathered and stored, so a wave's memory
// latency overlaps its own gather work (no register copies between the sets,
// which would force a wait on the prefetched loads). The prefetch past the
// last pass falls outside the buffer range (loads of 0); offsets stay below
// 2^31 because tiles are sized with two passes of slack. emit(set, so)
// corrects and stores the UNROLL lines of a register set at line offset so.
template <int VEC, int UNROLL, int NT, typename E>
__device__ __forceinline__ void stream_sets(__amdgpu_buffer_rsrc_t rin, uint32_t vo,
                                            uint32_t line_stride, int passes, uint32_t pass_adv,
                                            E emit) {
    typedef typename Px<VEC>::T T;
    const uint32_t pass_bytes = pass_adv ? pass_adv : UNROLL * line_stride;
    T a[UNROLL], b[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) a[u] = Buf<VEC, NT>::ld(rin, vo, u * line_stride);
    uint32_t so = 0;  // wave-uniform line offset of the current pass
    for (int k = 0; k < passes; k += 2) {
        so = __builtin_amdgcn_readfirstlane(so);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            b[u] = Buf<VEC, NT>::ld(rin, vo, so + pass_bytes + u * line_stride);
        emit(a, so);
        if (k + 1 >= passes) break;
        so += pass_bytes;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            a[u] = Buf<VEC, NT>::ld(rin, vo, so + pass_bytes + u * line_stride);
        emit(b, so);
        so += pass_bytes;
    }
}

// stream_sets with one call gather(k, dn) per pixel k of the lane.
template <int VEC, int UNROLL, int NT, typename G>
__device__ __forceinline__ void stream_lines(__amdgpu_buffer_rsrc_t rin,
                                             __amdgpu_buffer_rsrc_t rout, uint32_t vo,
                                             uint32_t line_stride, int passes, G gather,
                                             uint32_t pass_adv = 0) {
    typedef typename Px<VEC>::T T;
    stream_sets<VEC, UNROLL, NT>(
        rin, vo, line_stride, passes, pass_adv, [&](const T (&w)[UNROLL], uint32_t so) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                Buf<VEC, NT>::st(rout, vo, so + u * line_stride, map_px<VEC>(w[u], gather));
        });
}

// ---- the three LUT access modes -------------------------------------------------------

// Raw LDS strip, level-major: tile[v * W + j] is detector j's entry for level
// v. With W a multiple of 64 entries, the 32 lanes of a half-wave that own
// consecutive detector pairs read 32 different banks whatever the levels.
__device__ __forceinline__ uint32_t g_raw(const uint16_t* tile, uint32_t dnv, uint32_t top,
                                          int logW, int j) {
    const uint32_t v = dnv < top ? dnv : top;
    return tile[(v << logW) + j];
}

// Global LUT row (the L2 path).
__device__ __forceinline__ uint32_t g_glb(const uint16_t* row, uint32_t dnv, uint32_t top) {
    const uint32_t v = dnv < top ? dnv : top;
    return row[v];
}

// Packed LDS strip. Every LUT row is cut into blocks of 32 levels; a block is
// stored as its first entry (16-bit base) and the 31 steps between
// consecutive entries, each in {0, 1, 2, 3}, as two 32-bit bit-planes (bit i
// of `lo`/`hi` = low/high bit of step i). Entry v of the row is then
//   base[v / 32] + popcount(lo & m) + 2 * popcount(hi & m),  m = 2^(v % 32) - 1,
// exactly. That is 2.5 bits per entry instead of 16, so strips 6.4x wider fit
// in LDS. Rows with a negative step or a step above 3 cannot be packed; the
// tile then falls back to global gathers. Layout: planes [NB][W] (u32x2)
// followed by bases [NB][W] (u16), detector j of the strip at position
// p = (j % VEC) * (W / VEC) + j / VEC, so the lanes of a wave read
// consecutive 8-byte plane words for each of their VEC pixels.
__device__ __forceinline__ uint32_t g_packed(const u32x2* planes, const uint16_t* bases,
                                             uint32_t dnv, uint32_t top, int logW, int p) {
    const uint32_t v = dnv < top ? dnv : top;
    const int idx = (int)((v >> 5) << logW) + p;
    const u32x2 q = planes[idx];
    const uint32_t m = (1u << (v & 31u)) - 1u;
    return (uint32_t)bases[idx] + (uint32_t)__builtin_popcount(q.x & m) +
           2u * (uint32_t)__builtin_popcount(q.y & m);
}

// Bytes of LDS a packed strip of W detectors needs for L levels.
__host__ __device__ constexpr size_t packed_lds_bytes(int W, int L) {
    return (size_t)((L + 31) / 32) * (size_t)W * 10;
}

// ---- dense LDS strip: one bit per step -------------------------------------------------
//
// A LUT row is cut into blocks of 64 levels. Within block `blk` the entries
// e_0..e_63 are stored as an unclamped staircase U_0..U_63 with
// clamp(U_i, 0, L-1) = e_i:
//   U_i = U_0 + s*i + sum_{t<i} b_t,   s in {0, 1},  b_t in {0, 1},
// i.e. each step U_{t+1} - U_t is s or s + 1. Where the row saturates
// (entries 0 before the first positive one, entries L-1 from the first L-1
// on) the staircase goes on below 0 / above L-1 in steps of s + 1 and the
// clamp restores the entries. The encoder takes s = max(0, largest step -
// 1), so a block whose only unsaturated step is 2 (a jump into or out of a
// saturated run) still fits.
//
// Stored form, chosen so that the decode is additive and needs no masks:
//   plane z: bit 63 - t = 1 - b_t (t = 0..62), bit 0 = s;
//   header H (int16) = U_0 + B - 63 - 64*(s+1)*blk - s,  B = sum_t b_t.
// Shifting z left by i keeps bits 0..63-i, i.e. the complemented steps
// t >= i and bit 0, so popcount(z << i) = (63 - i) - sum_{t>=i} b_t + s and,
// with m = s + 1 and level v = 64*blk + i,
//   U = H + m*v + popcount(z << (v mod 64))      (m*v = v << s),
// exactly. |H| < 16448 for L <= 8192, so H never equals kDenseBad, the
// header that marks a block the dense form cannot hold. 80 bits per 64
// entries (1.25 bits per entry): a 4096-level strip of 256 detectors fits
// 160 KiB. Encodable blocks: non-decreasing, with the steps between
// unsaturated entries within {s, s+1}, s <= 1 (calibration LUTs: gains
// below 2); other rows make the tile gather from the global LUT.
// Layout: planes [NB][W] (64-bit) from byte 0, then headers [NB][W] (int16)
// from byte NB * W * 8; detector j of the strip at position p = (j % VEC) *
// (W / VEC) + j / VEC, as the packed strip. A lane keeps 8p and its header
// base NB*W*8 + 2p, so each of the two addresses of a level is one shift-add
// of the block index. Requires L <= kDenseMaxLevels = 8192 (header range).
constexpr int16_t kDenseBad = -32768;

__host__ __device__ constexpr size_t dense_lds_bytes(int W, int L) {
    return (size_t)((L + 63) / 64) * (size_t)W * 10;
}

// LDS addressed from byte 0: the correction kernels have no static LDS, so
// their dynamic LDS starts at 0 (prepare_apply_kernels and
// prepare_batch_kernel check it on the host and refuse otherwise); with the
// base a known constant no address needs an add for it.
typedef __attribute__((address_space(3))) const uint64_t lds_u64;
typedef __attribute__((address_space(3))) const int16_t lds_i16;

// med3(x, 0, hi) in one instruction (the compiler forms it only for
// constant bounds); hi is wave-uniform.
__device__ __forceinline__ uint32_t clamp0(int x, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi));
    return (uint32_t)r;
}

// popcount(x) + acc in one instruction (the compiler would otherwise sum
// two popcounts with a separate three-way add).
__device__ __forceinline__ int bcnt_acc(uint32_t x, int acc) {
    int r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// p8 = 8p, h2 = NB*W*8 + 2p (the lane's position p in the plane and header
// arrays, in bytes from the start of LDS).
// hmin: lowered to the header read.
__device__ __forceinline__ uint32_t g_dense_min(uint32_t dnv, uint32_t top, int logW, uint32_t p8,
                                                uint32_t h2, int& hmin) {
    const uint32_t v = dnv < top ? dnv : top;
    const uint32_t blk = v >> 6;
    const uint64_t z = *(lds_u64*)(uintptr_t)((blk << (logW + 3)) + p8);
    const int h = *(lds_i16*)(uintptr_t)((blk << (logW + 1)) + h2);
    hmin = min(hmin, h);
    const uint64_t sh = z << (v & 63u);
    int u = (int)(v << ((uint32_t)z & 1u)) + h;
    u = bcnt_acc((uint32_t)(sh >> 32), u);
    u = bcnt_acc((uint32_t)sh, u);
    return clamp0(u, (int)top);
}

__device__ __forceinline__ uint32_t g_dense(uint32_t dnv, uint32_t top, int logW, uint32_t p8,
                                            uint32_t h2) {
    int unused = 0;
    return g_dense_min(dnv, top, logW, p8, h2, unused);
}

// As g_dense, for a strip with blocks the dense form cannot hold: a level of
// such a block (header kDenseBad) reads the LUT row in global memory.
__device__ __forceinline__ uint32_t g_dense_checked(uint32_t dnv, uint32_t top, int logW,
                                                    uint32_t p8, uint32_t h2,
                                                    const uint16_t* row) {
    const uint32_t v = dnv < top ? dnv : top;
    const uint32_t blk = v >> 6;
    const int h = *(lds_i16*)(uintptr_t)((blk << (logW + 1)) + h2);
    if (h == (int)kDenseBad) return row[v];
    const uint64_t z = *(lds_u64*)(uintptr_t)((blk << (logW + 3)) + p8);
    const uint64_t sh = z << (v & 63u);
    int u = (int)(v << ((uint32_t)z & 1u)) + h;
    u = bcnt_acc((uint32_t)(sh >> 32), u);
    u = bcnt_acc((uint32_t)sh, u);
    return clamp0(u, (int)top);
}

// Lane exchanges inside groups of 8 lanes as DPP moves (VALU, no LDS):
// quad_perm [1,0,3,2] and [2,3,0,1] swap with the lane at distance 1 and 2,
// row_half_mirror (lane i <-> 7 - i) with one of the other quad, and
// row_shl:1 reads the next lane of the 16-lane row.
constexpr int kDppQuadXor1 = 0xB1;
constexpr int kDppQuadXor2 = 0x4E;
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppRowShl1 = 0x101;

template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}

// Sum / OR over the 8 lanes of x's group, returned on all 8.
__device__ __forceinline__ uint32_t group8_add(uint32_t x) {
    x += (uint32_t)dpp_move<kDppQuadXor1>((int)x);
    x += (uint32_t)dpp_move<kDppQuadXor2>((int)x);
    return x + (uint32_t)dpp_move<kDppHalfMirror>((int)x);
}
__device__ __forceinline__ uint32_t group8_or(uint32_t x) {
    x |= (uint32_t)dpp_move<kDppQuadXor1>((int)x);
    x |= (uint32_t)dpp_move<kDppQuadXor2>((int)x);
    return x | (uint32_t)dpp_move<kDppHalfMirror>((int)x);
}

// ---- dense encoding of LUT rows by a wave ----------------------------------------------
//
// A wave takes 512 consecutive levels of a row per pass, 8 blocks of 64: lane
// 8g + q holds entries 8q .. 8q + 7 of block g, two per word, so a pass loads
// or stores 1 KiB of the row contiguously. The 8 lanes of a block decide its
// form together with DPP moves (VALU, no LDS).

// Both halves of a word at a time (16-bit entries, steps and flags).
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) -
                                                __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) +
                                                __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                        __builtin_bit_cast(u16x2, b)));
}
// (As an instruction: the compiler turns a minimum with 1 into a comparison
// per half.)
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The step bits x0 .. x3 of a lane (bit 0 of each half), as one byte.
__device__ __forceinline__ uint32_t step_byte(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                              int q) {
    const uint32_t y = x0 | (x1 << 2) | (x2 << 4) | (x3 << 6);
    return (y | (y >> 15)) & (q == 7 ? 0x7Fu : 0xFFu);
}

// Bit k of the steps of a packed block's four lanes q = 0 .. 3 (8 steps each,
// two per word), as the block's plane on all four.
__device__ __forceinline__ uint32_t quad_plane(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3,
                                               int k, int q) {
    constexpr uint32_t kOnes = 0x00010001u;
    const uint32_t y = ((d0 >> k) & kOnes) | (((d1 >> k) & kOnes) << 2) |
                       (((d2 >> k) & kOnes) << 4) | (((d3 >> k) & kOnes) << 6);
    uint32_t word = ((y | (y >> 15)) & 0xFFu) << (q << 3);
    word |= (uint32_t)dpp_move<kDppQuadXor1>((int)word);
    return word | (uint32_t)dpp_move<kDppQuadXor2>((int)word);
}

// Blocks (of a group of 8 lanes) in which no lane fails.
__device__ __forceinline__ bool group8_ok(bool fail, int lane) {
    const uint64_t f = __ballot(fail);
    return f == 0 || ((f >> (lane & 56)) & 0xFFu) == 0;
}

// One pass of one row: the plane word and header (kDenseBad if the block does
// not fit) of block blk, valid on lane q = 0. whole: the pass lies inside the
// row (wave-uniform). Bound by instruction issue, so it works on two entries
// per word, without a branch per entry: the 8 steps of a lane in 4 packed
// subtractions; a block's slope s is 1 if any of its steps has bit 1 set;
// every step minus s must then be 0 or 1 in both halves (a negative or larger
// step fails that), and those bits are the block's. The usual pass is whole
// with all entries in 1 .. L-2 (a lane's are if its first is not 0 or above
// L-1 and its last is below L-1, or it has a negative step and the block fails
// either way): about 45 instructions. The other kind masks the steps that say
// nothing about the slope (inside a run of 0 or of L-1, or past the row; they
// must be 0 and count as s + 1): about 100. With one entry per register and a
// branch per entry the two took 110 and 500, and the build with encoding 80 us
// on 3 x 6000 rows of 4096 levels against 52 us now.
__device__ __forceinline__ void encode_pass(const u32x4 w, int L, int blk, bool whole,
                                            uint64_t* z_out, int16_t* head_out) {
    constexpr uint32_t kOnes = 0x00010001u;
    const int lane = (int)(threadIdx.x & 63);
    const int q = lane & 7;
    const uint32_t top = (uint32_t)(L - 1);
    // Steps e_{k+1} - e_k, k = 2i and 2i + 1 in word i; b_i are the later entries.
    const uint32_t nx = (uint32_t)dpp_move<kDppRowShl1>((int)w.x);  // lane q + 1's (q < 7)
    const uint32_t b0 = __builtin_amdgcn_alignbit(w.y, w.x, 16);
    const uint32_t b1 = __builtin_amdgcn_alignbit(w.z, w.y, 16);
    const uint32_t b2 = __builtin_amdgcn_alignbit(w.w, w.z, 16);
    const uint32_t b3 = __builtin_amdgcn_alignbit(nx, w.w, 16);
    const uint32_t d0 = pk_sub(b0, w.x), d1 = pk_sub(b1, w.y), d2 = pk_sub(b2, w.z);
    const uint32_t d3 = pk_sub(b3, w.w);
    const uint32_t first = w.x & 0xffffu, last = w.w >> 16;
    int s, u0 = (int)first;  // lane q = 0: the block's first entry
    bool ok;
    uint32_t lo8;
    if (whole && !__any(first - 1u >= top || last >= top)) {
        // Lane q = 7 has no step 63: it repeats its step 62.
        const uint32_t e3 = __builtin_amdgcn_perm(d3, d3, q == 7 ? 0x01000100u : 0x03020100u);
        const uint32_t any = d0 | d1 | d2 | e3;
        const uint32_t two = group8_or((any | (any >> 16)) & 2u);
        s = (int)(two >> 1);
        const uint32_t ss = (two >> 1) | (two << 15);
        const uint32_t x0 = pk_sub(d0, ss), x1 = pk_sub(d1, ss), x2 = pk_sub(d2, ss);
        const uint32_t x3 = pk_sub(e3, ss);
        ok = group8_ok(((x0 | x1 | x2 | x3) & ~kOnes) != 0, lane);
        lo8 = step_byte(x0, x1, x2, x3, q);
    } else {
        // Valid steps of this lane (entries t and t + 1 both in the block).
        const int v = min(64, L - (blk << 6)) - 1 - (q << 3);
        auto valid = [&](int i) {
            return v >= 2 * i + 2 ? 0xFFFFFFFFu : (v == 2 * i + 1 ? 0xFFFFu : 0u);
        };
        const uint32_t b[4] = {b0, b1, b2, b3}, d[4] = {d0, d1, d2, d3};
        const uint32_t top2 = top * kOnes;
        uint32_t m[4], any = 0, zeros = 0, wrong = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t vm = valid(i);
            const uint32_t up = pk_min(b[i], kOnes);  // 1 where the later entry is not 0
            // All ones where the step tells the slope.
            m[i] = pk_sub(0u, up & pk_min(pk_sub(top2, w[i]), kOnes)) & vm;
            any |= d[i] & m[i];
            wrong |= d[i] & ~m[i] & vm;
            wrong |= pk_max(w[i], top2) ^ top2;  // an entry above L-1
            zeros = pk_add(zeros, (kOnes - up) & vm);
        }
        const uint32_t two = group8_or((any | (any >> 16)) & 2u);
        s = (int)(two >> 1);
        const uint32_t ss = (two >> 1) | (two << 15);
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = (pk_sub(d[i], ss) & m[i]) | (kOnes & ~m[i]);
            wrong |= x[i] & ~kOnes;
        }
        ok = group8_ok(wrong != 0, lane);
        lo8 = step_byte(x[0], x[1], x[2], x[3], q);
        // A block that opens with zeros: as many steps below 0 as steps end in 0.
        const int nz = (int)group8_add((zeros & 0xffffu) + (zeros >> 16));
        if (u0 == 0) u0 = -(s + 1) * nz;
    }
    // Plane word: bit 63 - t = 1 - b_t, bit 0 = s. Lane q holds steps 8q .. 8q
    // + 7: its byte, bit-reversed, belongs in the high word for q < 4 (byte 3 -
    // q), in the low one for q >= 4 (byte 7 - q); each quad ORs its word.
    uint32_t word = __builtin_bitreverse32(lo8) >> ((q & 3) << 3);
    word |= (uint32_t)dpp_move<kDppQuadXor1>((int)word);
    word |= (uint32_t)dpp_move<kDppQuadXor2>((int)word);
    const uint32_t hi = word, lo = (uint32_t)dpp_move<kDppHalfMirror>((int)word);  // q = 0
    const int H = u0 + __builtin_popcount(hi) + __builtin_popcount(lo) - 63 - ((s + 1) << 6) * blk -
                  s;
    if (H <= (int)kDenseBad || H > 32767) ok = false;
    const uint64_t z = ((uint64_t)~hi << 32) | (uint64_t)((~lo & ~1u) | (uint32_t)s);
    *z_out = ok ? z : 0;
    *head_out = ok ? (int16_t)H : kDenseBad;
}

// All blocks of R rows of L levels: fetch(r, v0, whole, w) gives every row's 8
// entries from level v0 of pass r (words past the row are ignored; several
// rows per pass keep several loads in flight), put(i, blk, plane, header)
// takes row i's block from lane q = 0. AHEAD: a pass's entries are fetched
// while the one before is encoded (for fetches that load). Every lane of the
// wave must call it.
template <int R, bool AHEAD, typename F, typename P>
__device__ __forceinline__ void encode_rows(int L, F fetch, P put) {
    const int NB = (L + 63) >> 6;
    const int lane = (int)(threadIdx.x & 63);
    const int rounds = (NB + 7) >> 3;
    u32x4 next[R];
    if (AHEAD) fetch(lane << 3, 512 <= L, next);
    for (int r = 0; r < rounds; ++r) {
        const int blk = (r << 3) + (lane >> 3);
        const bool whole = ((r + 1) << 9) <= L;
        u32x4 w[R];
        if (AHEAD) {
#pragma unroll
            for (int i = 0; i < R; ++i) w[i] = next[i];
            if (r + 1 < rounds) fetch(((r + 1) << 9) + (lane << 3), ((r + 2) << 9) <= L, next);
        } else {
            fetch((r << 9) + (lane << 3), whole, w);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            uint64_t z;
            int16_t h;
            encode_pass(w[i], L, blk, whole, &z, &h);
            if ((lane & 7) == 0 && blk < NB) put(i, blk, z, h);
        }
    }
}

// Entries [v0, v0 + 8) of a LUT row in global memory, those past the row 0
// (vec16: the row's 16-byte groups are aligned and whole).
__device__ __forceinline__ u32x4 load_lut8(const uint16_t* row, int v0, int L, bool whole,
                                           bool vec16) {
    if (vec16) return whole || v0 < L ? *(const u32x4*)(row + v0) : u32x4{0u, 0u, 0u, 0u};
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = v0 + 2 * i < L ? row[v0 + 2 * i] : 0u;
        const uint32_t b = v0 + 2 * i + 1 < L ? row[v0 + 2 * i + 1] : 0u;
        w[i] = a | (b << 16);
    }
    return w;
}

// The doubles v0 .. v0 + 7.
__device__ __forceinline__ void levels8(int v0, double (&x)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (double)(v0 + k);
}

// Writes the first n of the 8 entries w of a LUT row to dst: one 16-byte store
// when they are whole and aligned (non-temporal if nt), else 16-bit stores.
__device__ __forceinline__ void store_lut8(uint16_t* dst, const u32x4 w, int n, bool vec16,
                                           bool nt) {
    if (vec16 && n >= 8) {
        if (nt) __builtin_nontemporal_store(w, (u32x4*)dst);
        else *(u32x4*)dst = w;
    } else {
        for (int k = 0; k < min(n, 8); ++k) dst[k] = (uint16_t)(w[k >> 1] >> ((k & 1) * 16));
    }
}

// Blocks of a dense strip the form cannot hold, summed over the workgroup
// from each thread's count, without static LDS (a strip may fill the LDS): if
// any wave has one, the strip's first plane and header words are lent to a
// flag and the sum, and put back. Call after every thread has staged; every
// thread returns the same value.
__device__ __forceinline__ uint32_t dense_bad_blocks(int count, uint64_t* planes, int16_t* heads) {
    __syncthreads();
    const int16_t h0 = heads[0];
    const uint64_t z0 = planes[0];
    __syncthreads();
    if (threadIdx.x == 0) {
        heads[0] = 0;
        planes[0] = 0;
    }
    __syncthreads();
    if (__any(count)) {
        if ((threadIdx.x & 63) == 0) heads[0] = 1;
        if (count) atomicAdd((unsigned int*)planes, (unsigned int)count);
    }
    __syncthreads();
    const uint32_t n = heads[0] ? *(const unsigned int*)planes : 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        heads[0] = h0;
        planes[0] = z0;
    }
    __syncthreads();
    return n;
}

enum TileMode { kRaw = 0, kGlobal = 1, kPacked = 2, kDense = 3 };

// Workgroup-wide OR of `flag` for a packed strip, without static LDS (a
// static word would push two 80 KiB tiles over a CU's 160 KiB). The word is
// bit 31 of the first plane word: a block has 31 steps, so staging leaves
// bit 31 clear and the gather masks never reach it. Call after every thread
// has staged (planes[0] is always written: detector 0, block 0); every
// thread returns the same value.
__device__ __forceinline__ int packed_any(int flag, u32x2* planes) {
    __syncthreads();
    if (__any(flag) && (threadIdx.x & 63) == 0)
        atomicOr((unsigned int*)planes, 0x80000000u);
    __syncthreads();
    return (int)(*(const unsigned int*)planes >> 31);
}

// One correction tile: band b, detectors [d0, d0 + weff), lines [n0, n1).
// Lanes own VEC adjacent detectors of one line; q consecutive threads cover
// a line of the strip and the workgroup walks floor(blockDim.x / q) lines at
// a time. q = W / VEC (`dense` false: a wave covers whole line segments when
// q divides 64, lanes past a narrower strip idle) or ceil(weff / VEC) (`dense`
// true: no idle lanes inside a wave). If VEC does not divide weff, the last
// lane of a line takes the strip's last VEC detectors, some of which the lane
// before it takes too; both write the same values. Requirements (checked on
// the host): W = 2^logW >= weff >= VEC, image pointers aligned to 2 bytes, W /
// VEC <= blockDim.x, and the LDS size of the mode for W detectors. dn and out
// may be the same buffer (in place) if VEC | weff (every pixel is read and
// then written by the same lane) or if q divides 64 (`dense` false: a line's
// lanes are in one wave, which has loaded a line whole before it stores any of
// it), so they are deliberately not __restrict__.
template <int VEC, int UNROLL, int NT, int MODE>
__device__ __forceinline__ void apply_tile(const uint16_t* dn, const uint16_t* __restrict__ lut,
                                           uint16_t* out, int64_t N, int D, int L, int logW,
                                           int b, int d0, int weff, int64_t n0, int64_t n1,
                                           void* smem, bool lut_vec, bool dense,
                                           const uint64_t* pre_planes = nullptr,
                                           const int16_t* pre_heads = nullptr, int ci = 0,
                                           int ck = 1, int nst = 0) {
    constexpr int LOGVEC = log_vec<VEC>();
    const int W = 1 << logW;
    const int tid = threadIdx.x;
    const int nt = blockDim.x;
    const uint32_t top = (uint32_t)(L - 1);
    const size_t Lz = (size_t)L;
    const uint16_t* strip_lut = lut + ((size_t)b * (size_t)D + (size_t)d0) * Lz;
    const int logq = logW - LOGVEC;  // LDS positions per VEC slot = W / VEC
    // Lanes per strip line, and the strip's LDS positions: position (k, ln), at
    // p = (k << logq) + ln, holds detector pos_detector(k, ln), the k-th pixel
    // of lane ln.
    const int lanes = (weff + VEC - 1) >> LOGVEC;
    const int q = dense ? lanes : (1 << logq);
    auto pos_detector = [&](int k, int ln) { return min(ln << LOGVEC, weff - VEC) + k; };
    const int row = tid / q;         // this thread's line within a pass
    const int lane = tid - row * q;
    // Lines per pass, from the nst streaming threads (0: all of them).
    // Wave-uniform (the compiler cannot prove it through the division and
    // would otherwise wrap every buffer access in a waterfall loop).
    const int rpp = __builtin_amdgcn_readfirstlane((nst ? nst : nt) / q);
    // Threads past the last whole line, or past the strip, only stage.
    const bool streams = row < rpp && lane < lanes;
    const int j = pos_detector(0, lane);
    // The tile's image bytes as buffer resources: line n0, detector d0 is at
    // byte 0; the range ends after the tile's last pixel.
    const size_t tile0 = ((size_t)b * (size_t)N + (size_t)n0) * (size_t)D + (size_t)d0;
    const uint32_t span = (uint32_t)((((size_t)(n1 - n0) - 1) * (size_t)D + (size_t)weff) * 2);
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(dn + tile0, span);
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(out + tile0, span);
    // Passes of rpp x UNROLL lines over [n0, n1); the tile takes passes ci,
    // ci + ck, ci + 2 ck, ... (ck = 1: all of them).
    const uint32_t line_stride = (uint32_t)rpp * (uint32_t)D * 2u;
    const uint32_t pass_bytes = UNROLL * line_stride;
    const uint32_t pass_adv = pass_bytes * (uint32_t)ck;
    const uint32_t vo = (uint32_t)(((size_t)row * (size_t)D + (size_t)j) * 2) +
                        (uint32_t)ci * pass_bytes;
    const int all_passes =
        (int)((n1 - n0 + (int64_t)rpp * UNROLL - 1) / ((int64_t)rpp * UNROLL));
    const int passes = ci < all_passes ? (all_passes - ci + ck - 1) / ck : 0;

    if constexpr (MODE == kRaw) {
        uint16_t* tile = (uint16_t*)smem;
        // Stage: lanes run along detectors (j fastest) so that one wave's
        // 16-bit LDS writes land in consecutive addresses.
        if (lut_vec) {
            // Rounds of SU items per thread, loads first (latency overlap).
            constexpr int SU = 8;
            const int items = (L >> 3) << logW;
            for (int it0 = tid; it0 < items; it0 += nt * SU) {
                u32x4 qv[SU];
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int it = it0 + s * nt;
                    const int jj = it & (W - 1);
                    qv[s] = u32x4{0u, 0u, 0u, 0u};
                    if (it < items && jj < weff) {
                        qv[s] = *(const u32x4*)(strip_lut + (size_t)jj * Lz + (it >> logW) * 8);
                    }
                }
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int it = it0 + s * nt;
                    const int jj = it & (W - 1);
                    if (it < items && jj < weff) {
                        const u32x4 q = qv[s];
                        uint16_t* dst = tile + (((it >> logW) * 8) << logW) + jj;
                        dst[0] = (uint16_t)(q.x & 0xffffu);
                        dst[1 << logW] = (uint16_t)(q.x >> 16);
                        dst[2 << logW] = (uint16_t)(q.y & 0xffffu);
                        dst[3 << logW] = (uint16_t)(q.y >> 16);
                        dst[4 << logW] = (uint16_t)(q.z & 0xffffu);
                        dst[5 << logW] = (uint16_t)(q.z >> 16);
                        dst[6 << logW] = (uint16_t)(q.w & 0xffffu);
                        dst[7 << logW] = (uint16_t)(q.w >> 16);
                    }
                }
            }
        } else {
            const int items = L << logW;
            for (int it = tid; it < items; it += nt) {
                const int jj = it & (W - 1);
                const int v = it >> logW;
                if (jj < weff) tile[(v << logW) + jj] = strip_lut[(size_t)jj * Lz + v];
            }
        }
        __syncthreads();
        if (streams) {
            stream_lines<VEC, UNROLL, NT>(
                rin, rout, vo, line_stride, passes,
                [&](int k, uint32_t d) { return g_raw(tile, d, top, logW, j + k); }, pass_adv);
        }
        __syncthreads();  // the tile may be restaged next
    } else if constexpr (MODE == kGlobal) {
        if (streams) {
            const uint16_t* lrow = strip_lut + (size_t)j * Lz;
            stream_lines<VEC, UNROLL, NT>(
                rin, rout, vo, line_stride, passes,
                [&](int k, uint32_t d) { return g_glb(lrow + (size_t)k * Lz, d, top); }, pass_adv);
        }
    } else if constexpr (MODE == kDense) {
        const int NB = (L + 63) >> 6;
        const uint32_t hb = (uint32_t)NB << (logW + 3);  // header array, bytes from LDS start
        uint64_t* planes = (uint64_t*)smem;
        int16_t* heads = (int16_t*)((unsigned char*)smem + hb);
        int bad = 0;
        if (pre_planes) {
            // Stage the blocks k_dense_encode wrote ([band][block][detector]):
            // consecutive threads read consecutive detectors of one block.
            const int wpos = lanes << LOGVEC;
            const int items = NB * wpos;
            const size_t row0 = (size_t)b * (size_t)NB * (size_t)D + (size_t)d0;
            for (int it = tid; it < items; it += nt) {
                const int blk = it / wpos;
                const int i = it - blk * wpos;
                const int k = i & (VEC - 1), ln = i >> LOGVEC;
                const size_t g = row0 + (size_t)blk * (size_t)D + (size_t)pos_detector(k, ln);
                const int16_t hd = pre_heads[g];
                const int p = (k << logq) + ln;
                bad += (int)(hd == kDenseBad);
                planes[(blk << logW) + p] = pre_planes[g];
                heads[(blk << logW) + p] = hd;
            }
        }
        // Stage: a wave encodes kRows rows of the strip at a time (the loads of
        // a pass of all of them in flight together).
        if (!pre_planes) {
            constexpr int kRows = 4;
            const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = nt >> 6;
            for (int j0 = wv * kRows; j0 < weff; j0 += nwv * kRows) {
                encode_rows<kRows, true>(
                    L,
                    [&](int v0, bool whole, u32x4 (&w)[kRows]) {
#pragma unroll
                        for (int i = 0; i < kRows; ++i)
                            w[i] = load_lut8(strip_lut + (size_t)min(j0 + i, weff - 1) * Lz, v0, L,
                                             whole, lut_vec);
                    },
                    [&](int i, int blk, uint64_t z, int16_t h) {
                        const int jj = j0 + i;
                        if (jj >= weff) return;
                        bad += (int)(h == kDenseBad);
                        // Its position among the whole lanes, and in the last.
                        const int k = jj - (weff - VEC);
                        if ((jj >> LOGVEC) < lanes - 1) {
                            const int p = ((jj & (VEC - 1)) << logq) + (jj >> LOGVEC);
                            planes[(blk << logW) + p] = z;
                            heads[(blk << logW) + p] = h;
                        }
                        if (k >= 0) {
                            const int p = (k << logq) + lanes - 1;
                            planes[(blk << logW) + p] = z;
                            heads[(blk << logW) + p] = h;
                        }
                    });
            }
        }
        const uint32_t nbad = dense_bad_blocks(bad, planes, heads);
        if (nbad == 0) {
            if (streams)
                stream_lines<VEC, UNROLL, NT>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        const uint32_t p = (uint32_t)((k << logq) + lane);
                        return g_dense(d, top, logW, p * 8u, hb + p * 2u);
                    }, pass_adv);
        } else {
            // Some blocks of the strip are not held in dense form (one or two
            // per million of a calibration LUT, so every second or third
            // large 12-bit scene has a tile with one, which then must not be
            // the last to finish). Their levels read the global LUT row. The
            // threads that only staged stream too: thread group g of ng takes
            // every ng-th of the tile's passes, while the offsets of its
            // prefetch stay within the 32-bit range.
            const int per = nst ? nst : nt;
            const int ng0 = nt / per;
            const bool fits = ((uint64_t)passes + 3u * (uint64_t)ng0 + (uint64_t)ck) *
                                  (uint64_t)pass_adv < ((uint64_t)1 << 31);
            const int ng = __builtin_amdgcn_readfirstlane(fits ? ng0 : 1);
            // Whole waves: per is a multiple of 64.
            const int grp = __builtin_amdgcn_readfirstlane(tid / per);
            const int gtid = tid - grp * per;
            const int grow = gtid / q;
            const int glane = gtid - grow * q;
            const int gj = pos_detector(0, glane);
            const uint32_t gvo = (uint32_t)(((size_t)grow * (size_t)D + (size_t)gj) * 2) +
                                 (uint32_t)ci * pass_bytes + (uint32_t)grp * pass_adv;
            const uint32_t gadv = (uint32_t)ng * pass_adv;
            const int gpasses = grp < passes ? (passes - grp + ng - 1) / ng : 0;
            const uint16_t* lrow = strip_lut + (size_t)gj * Lz;
            if (grp >= ng || grow >= rpp || glane >= lanes || gpasses == 0) {
                // nothing to stream
            } else if (nbad <= (uint32_t)NB) {
                // Few: decode every pixel and keep the smallest header the
                // lane read in each line; a lane that met such a block then
                // takes those pixels from the LUT row. One branch per
                // register set, so that the LDS reads of a set stay in flight
                // together; nbad <= NB bounds how often it is taken (about
                // one pixel in weff).
                typedef typename Px<VEC>::T T;
                stream_sets<VEC, UNROLL, NT>(
                    rin, gvo, line_stride, gpasses, gadv,
                    [&](const T (&w)[UNROLL], uint32_t so) {
                        int hmin[UNROLL], hset = 0;
                        T r[UNROLL];
#pragma unroll
                        for (int u = 0; u < UNROLL; ++u) {
                            hmin[u] = 0;
                            r[u] = map_px<VEC>(w[u], [&](int k, uint32_t d) {
                                const uint32_t p = (uint32_t)((k << logq) + glane);
                                return g_dense_min(d, top, logW, p * 8u, hb + p * 2u, hmin[u]);
                            });
                            hset = min(hset, hmin[u]);
                        }
                        if (hset == (int)kDenseBad) {
#pragma unroll
                            for (int u = 0; u < UNROLL; ++u)
                                if (hmin[u] == (int)kDenseBad)
                                    r[u] = map_px2<VEC>(w[u], r[u], [&](int k, uint32_t d,
                                                                        uint32_t e) {
                                        const uint32_t v = d < top ? d : top;
                                        const uint32_t p = (uint32_t)((k << logq) + glane);
                                        const int h = *(lds_i16*)(uintptr_t)(
                                            ((v >> 6) << (logW + 1)) + hb + p * 2u);
                                        const uint32_t g = lrow[(size_t)k * Lz + v];
                                        return h == (int)kDenseBad ? g : e;
                                    });
                        }
#pragma unroll
                        for (int u = 0; u < UNROLL; ++u)
                            Buf<VEC, NT>::st(rout, gvo, so + u * line_stride, r[u]);
                    });
            } else {
                // Many: check every header before decoding.
                stream_lines<VEC, UNROLL, NT>(
                    rin, rout, gvo, line_stride, gpasses, [&](int k, uint32_t d) {
                        const uint32_t p = (uint32_t)((k << logq) + glane);
                        return g_dense_checked(d, top, logW, p * 8u, hb + p * 2u,
                                               lrow + (size_t)k * Lz);
                    }, gadv);
            }
        }
        __syncthreads();  // the tile may be restaged next
    } else {
        const int NB = (L + 31) >> 5;
        u32x2* planes = (u32x2*)smem;
        uint16_t* bases = (uint16_t*)(planes + (size_t)NB * W);
        int bad = 0;
        if (lut_vec && (L & 31) == 0 && logW >= 4) {
            // Stage, coalesced and bank-conflict free: a wave packs 16
            // consecutive LDS positions of one level block. Lane 4g+q loads
            // the q-th 16-byte quarter (8 entries) of the block's row for
            // position p0+g; the steps are formed two per word (see
            // encode_pass), the four quarters' bits are merged by DPP moves
            // and lane 4g writes the block's words.
            const int wl = tid & 63, wv = tid >> 6, nwv = nt >> 6;
            const int g = wl >> 2, q = wl & 3;
            const int logpg = logW - 4;
            const int units = NB << logpg;
            // Rounds of SU units per wave: all SU loads are issued before the
            // first unit is packed, so staging is not one load latency per unit.
            constexpr int SU = 8;
            for (int u0 = wv; u0 < units; u0 += nwv * SU) {
                u32x4 qv[SU];
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int u = u0 + s * nwv;
                    const int p = ((u & ((1 << logpg) - 1)) << 4) + g;
                    const int ln = p & ((1 << logq) - 1);
                    const int jj = pos_detector(p >> logq, ln);
                    qv[s] = u32x4{0u, 0u, 0u, 0u};
                    if (u < units && ln < lanes) {
                        qv[s] = *(const u32x4*)(strip_lut + (size_t)jj * Lz +
                                                (size_t)(u >> logpg) * 32 + q * 8);
                    }
                }
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int u = u0 + s * nwv;
                    if (u >= units) break;  // uniform across the wave
                    const int blk = u >> logpg;
                    const int p = ((u & ((1 << logpg) - 1)) << 4) + g;
                    const bool valid = (p & ((1 << logq) - 1)) < lanes;
                    const u32x4 w = qv[s];
                    const uint32_t nx = (uint32_t)dpp_move<kDppRowShl1>((int)w.x);
                    const uint32_t d0 = pk_sub(__builtin_amdgcn_alignbit(w.y, w.x, 16), w.x);
                    const uint32_t d1 = pk_sub(__builtin_amdgcn_alignbit(w.z, w.y, 16), w.y);
                    const uint32_t d2 = pk_sub(__builtin_amdgcn_alignbit(w.w, w.z, 16), w.z);
                    // Block step 31 (lane q = 3) does not exist.
                    const uint32_t d3 = pk_sub(__builtin_amdgcn_alignbit(nx, w.w, 16), w.w) &
                                        (q == 3 ? 0xFFFFu : 0xFFFFFFFFu);
                    // A step above 3 or negative; 16-bit steps of 0 .. 3 that
                    // wrapped around leave the lane's last entry below its
                    // first, or the next lane's first below its last.
                    const bool over = ((d0 | d1 | d2 | d3) & 0xFFFCFFFCu) != 0 ||
                                      (w.w >> 16) < (w.x & 0xffffu) ||
                                      (q < 3 && (nx & 0xffffu) < (w.w >> 16));
                    bad |= (int)(valid && over);
                    uint32_t lo = quad_plane(d0, d1, d2, d3, 0, q);
                    uint32_t hi = quad_plane(d0, d1, d2, d3, 1, q);
                    if (valid && q == 0) {
                        u32x2 pl;
                        pl.x = lo;
                        pl.y = hi;
                        planes[blk * W + p] = pl;
                        bases[blk * W + p] = (uint16_t)w.x;
                    }
                }
            }
        } else {
            // Stage, general shapes: item = (detector jj, block), blocks fastest.
            const int items = (lanes << LOGVEC) * NB;
            for (int it = tid; it < items; it += nt) {
                const int i = it / NB;
                const int blk = it - i * NB;
                const int jj = pos_detector(i & (VEC - 1), i >> LOGVEC);
                const uint16_t* src = strip_lut + (size_t)jj * Lz + (size_t)blk * 32;
                const int cnt = min(32, L - blk * 32);
                uint32_t e[32];
                if (lut_vec && cnt == 32) {
    #pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const u32x4 q = *(const u32x4*)(src + q4 * 8);
                        e[q4 * 8 + 0] = q.x & 0xffffu;
                        e[q4 * 8 + 1] = q.x >> 16;
                        e[q4 * 8 + 2] = q.y & 0xffffu;
                        e[q4 * 8 + 3] = q.y >> 16;
                        e[q4 * 8 + 4] = q.z & 0xffffu;
                        e[q4 * 8 + 5] = q.z >> 16;
                        e[q4 * 8 + 6] = q.w & 0xffffu;
                        e[q4 * 8 + 7] = q.w >> 16;
                    }
                } else {
    #pragma unroll
                    for (int i = 0; i < 32; ++i) e[i] = i < cnt ? src[i] : 0u;
                }
                uint32_t lo = 0, hi = 0;
    #pragma unroll
                for (int i = 0; i < 31; ++i) {
                    if (i + 1 < cnt) {
                        const uint32_t step = e[i + 1] - e[i];  // wraps when negative
                        bad |= step > 3u;
                        lo |= (step & 1u) << i;
                        hi |= ((step >> 1) & 1u) << i;
                    }
                }
                const int p = ((i & (VEC - 1)) << logq) + (i >> LOGVEC);
                u32x2 pl;
                pl.x = lo;
                pl.y = hi;
                planes[blk * W + p] = pl;
                bases[blk * W + p] = (uint16_t)e[0];
            }
        }
        bad = packed_any(bad, planes);
        if (streams) {
            if (!bad) {
                stream_lines<VEC, UNROLL, NT>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        return g_packed(planes, bases, d, top, logW, (k << logq) + lane);
                    }, pass_adv);
            } else {
                const uint16_t* lrow = strip_lut + (size_t)j * Lz;
                stream_lines<VEC, UNROLL, NT>(
                    rin, rout, vo, line_stride, passes,
                    [&](int k, uint32_t d) { return g_glb(lrow + (size_t)k * Lz, d, top); }, pass_adv);
            }
        }
        __syncthreads();  // the tile may be restaged next
    }
}


// ---- fused LUT build + correction (batched requests) ------------------------------------

// Computes the LUT rows of band b, detectors [d0, d0 + weff) from their
// calibration coefficients straight into the LDS tile (raw, packed or dense
// layout, as the correction tile reads them) and, if `write_lut`, also into
// the global LUT. Returns nonzero (the same on every thread) when a packed row
// has a step outside 0..3, the LDS tile is then unusable, or the number of
// blocks the dense form cannot hold.
template <int VEC, int MODE>
__device__ __forceinline__ uint32_t build_strip(const double* __restrict__ coeffs, uint16_t* lut,
                                                int D, int L, int logW, int b, int d0, int weff,
                                                bool write_lut, bool lut_vec, void* smem) {
    constexpr int LOGVEC = log_vec<VEC>();
    const int W = 1 << logW;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int logq = logW - LOGVEC;
    const uint32_t top2 = (uint32_t)(L - 1) * 0x00010001u;
    const size_t row0 = (size_t)b * (size_t)D + (size_t)d0;
    // Coefficients of row j (the last row past the strip), loaded a row ahead.
    struct Row {
        double a[4];
    };
    auto load_row = [&](int j) {
        const double* a = coeffs + (row0 + (size_t)min(j, weff - 1)) * 4;
        return Row{{a[0], a[1], a[2], a[3]}};
    };
    // The LDS positions of row j: among the whole lanes, and in the last lane
    // of a line, which takes the strip's last VEC detectors (see apply_tile).
    const int lanes = (weff + VEC - 1) >> LOGVEC;
    auto at_positions = [&](int j, auto put) {
        const int k = j - (weff - VEC);
        if ((j >> LOGVEC) < lanes - 1) put(((j & (VEC - 1)) << logq) + (j >> LOGVEC));
        if (k >= 0) put((k << logq) + lanes - 1);
    };
    if constexpr (MODE == kRaw) {
        // Item = (detector j fastest, 8-level chunk): consecutive lanes write
        // consecutive LDS entries.
        uint16_t* tile = (uint16_t*)smem;
        const int chunks = (L + 7) >> 3;
        const int items = chunks << logW;
        for (int it = tid; it < items; it += nt) {
            const int j = it & (W - 1);
            const int c = it >> logW;
            if (j >= weff) continue;
            const double* a = coeffs + (row0 + (size_t)j) * 4;
            const double a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3];
            const int v0 = c * 8;
            const int n = min(8, L - v0);
            double x[8];
            levels8(v0, x);
            const u32x4 w = lut_eight(a0, a1, a2, a3, x, top2);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < n) tile[((v0 + k) << logW) + j] = (uint16_t)(w[k >> 1] >> ((k & 1) * 16));
            if (write_lut) store_lut8(lut + (row0 + (size_t)j) * (size_t)L + v0, w, n, lut_vec, true);
        }
        __syncthreads();
        return 0;
    } else if constexpr (MODE == kDense) {
        // A wave evaluates and encodes one row at a time, 8 blocks of 64
        // levels per pass.
        const int NB = (L + 63) >> 6;
        uint64_t* planes = (uint64_t*)smem;
        int16_t* heads = (int16_t*)((unsigned char*)smem + ((size_t)NB << (logW + 3)));
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = nt >> 6;
        int bad = 0;
        Row next = load_row(wv);
        for (int j = wv; j < weff; j += nwv) {
            const Row r = next;
            next = load_row(j + nwv);
            uint16_t* dst = lut + (row0 + (size_t)j) * (size_t)L;
            encode_rows<1, false>(
                L,
                [&](int v0, bool, u32x4 (&w)[1]) {
                    double x[8];
                    levels8(v0, x);
                    w[0] = lut_eight(r.a[0], r.a[1], r.a[2], r.a[3], x, top2);
                    if (write_lut && v0 < L) store_lut8(dst + v0, w[0], L - v0, lut_vec, true);
                },
                [&](int, int blk, uint64_t z, int16_t h) {
                    bad += (int)(h == kDenseBad);
                    at_positions(j, [&](int p) {
                        planes[(blk << logW) + p] = z;
                        heads[(blk << logW) + p] = h;
                    });
                });
        }
        return dense_bad_blocks(bad, planes, heads);
    } else {
        // A wave evaluates one detector row at a time, 16 blocks of 32 levels
        // per pass: lane 4g + q computes levels 32 (16 r + g) + 8q .. + 7, so
        // the wave's global LUT stores cover 1 KiB of the row contiguously.
        // The steps are formed two per word (see encode_pass) and the four
        // lanes of a block merge their bits by DPP moves.
        const int NB = (L + 31) >> 5;
        u32x2* planes = (u32x2*)smem;
        uint16_t* bases = (uint16_t*)(planes + (size_t)NB * W);
        const int lane = tid & 63;
        const int g = lane >> 2, q = lane & 3;
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int nwv = nt >> 6;
        const int rounds = (NB + 15) >> 4;
        uint32_t wrong = 0;
        Row next = load_row(wv);
        for (int j = wv; j < weff; j += nwv) {
            const Row cur = next;
            next = load_row(j + nwv);
            uint16_t* dst = lut + (row0 + (size_t)j) * (size_t)L;
            for (int r = 0; r < rounds; ++r) {
                const int blk = (r << 4) + g;
                const int v0 = (blk << 5) + (q << 3);
                double x[8];
                levels8(v0, x);
                const u32x4 w = lut_eight(cur.a[0], cur.a[1], cur.a[2], cur.a[3], x, top2);
                if (write_lut && v0 < L) store_lut8(dst + v0, w, L - v0, lut_vec, true);
                // Step i of a block (bit i of the planes) is entry i+1 minus
                // entry i; a step that leaves the block or the row is 0.
                const uint32_t nx = (uint32_t)dpp_move<kDppRowShl1>((int)w.x);
                uint32_t d[4] = {pk_sub(__builtin_amdgcn_alignbit(w.y, w.x, 16), w.x),
                                 pk_sub(__builtin_amdgcn_alignbit(w.z, w.y, 16), w.y),
                                 pk_sub(__builtin_amdgcn_alignbit(w.w, w.z, 16), w.z),
                                 pk_sub(__builtin_amdgcn_alignbit(nx, w.w, 16), w.w)};
                if (((r + 1) << 9) <= L) {
                    d[3] &= q == 3 ? 0xFFFFu : 0xFFFFFFFFu;
                } else {
                    const int v = min(32, L - (blk << 5)) - 1 - (q << 3);  // valid steps
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        d[i] &= v >= 2 * i + 2 ? 0xFFFFFFFFu : (v == 2 * i + 1 ? 0xFFFFu : 0u);
                }
                wrong |= d[0] | d[1] | d[2] | d[3];  // a step above 3 or negative
                // (16-bit steps of 0 .. 3 that wrapped around leave a lower
                // entry after a higher one; only levels above 65533 can.)
                if (L > 65533 && v0 + 8 <= L)
                    wrong |= ((w.w >> 16) < (w.x & 0xffffu) ||
                              (q < 3 && v0 + 8 < L && (nx & 0xffffu) < (w.w >> 16))) ? 4u : 0u;
                const uint32_t lo = quad_plane(d[0], d[1], d[2], d[3], 0, q);
                const uint32_t hi = quad_plane(d[0], d[1], d[2], d[3], 1, q);
                if (q == 0 && blk < NB)
                    at_positions(j, [&](int p) {
                        planes[blk * W + p] = u32x2{lo, hi};
                        bases[blk * W + p] = (uint16_t)w.x;
                    });
            }
        }
        return (uint32_t)packed_any((wrong & 0xFFFCFFFCu) != 0 ? 1 : 0, planes);
    }
}

// Writes the strip's LUT rows to global memory (second pass of a packed
// strip that cannot be packed and whose tile did not write them already).
__device__ __forceinline__ void write_strip(const double* __restrict__ coeffs, uint16_t* lut, int D,
                                            int L, int b, int d0, int weff, bool lut_vec) {
    const uint32_t top2 = (uint32_t)(L - 1) * 0x00010001u;
    const size_t row0 = (size_t)b * (size_t)D + (size_t)d0;
    const int chunks = (L + 7) >> 3;
    const int items = chunks * weff;
    for (int it = threadIdx.x; it < items; it += blockDim.x) {
        const int j = it / chunks;
        const int v0 = (it - j * chunks) * 8;
        const int n = min(8, L - v0);
        const double* a = coeffs + (row0 + (size_t)j) * 4;
        double x[8];
        levels8(v0, x);
        store_lut8(lut + (row0 + (size_t)j) * (size_t)L + v0,
                   lut_eight(a[0], a[1], a[2], a[3], x, top2), n, lut_vec, true);
    }
}

// Global LUT gather that reads through the L2 (sc0), for rows this
// workgroup has just written.
__device__ __forceinline__ uint32_t g_glb_l2(__amdgpu_buffer_rsrc_t r, uint32_t row_off,
                                             uint32_t dnv, uint32_t top) {
    const uint32_t v = dnv < top ? dnv : top;
    return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(row_off + v * 2u), 0, 1);
}

// One fused tile of a batched request: build the strip's LUT in LDS from the
// coefficients with every thread (writing it to the global LUT too when
// write_lut), then correct lines [n0, n1) as apply_tile does, with the first
// nst threads: as many bytes in flight as the plain tiles keep.
template <int VEC, int UNROLL, int MODE>
__device__ __forceinline__ void fused_tile(const double* __restrict__ coeffs, const uint16_t* dn,
                                           uint16_t* lut, uint16_t* out, int64_t N, int D, int L,
                                           int logW, int b, int d0, int weff, int64_t n0,
                                           int64_t n1, bool write_lut, void* smem, bool lut_vec,
                                           int nst) {
    constexpr int LOGVEC = log_vec<VEC>();
    const uint32_t bad = build_strip<VEC, MODE>(coeffs, lut, D, L, logW, b, d0, weff, write_lut,
                                                lut_vec, smem);
    if (n1 > n0) {
        const int tid = threadIdx.x;
        const int logq = logW - LOGVEC;
        const int lane = tid & ((1 << logq) - 1);
        const int lanes = (weff + VEC - 1) >> LOGVEC;
        const int rpp = nst >> logq;
        const int j = min(lane << LOGVEC, weff - VEC);
        const bool streams = tid < nst && lane < lanes;
        const uint32_t top = (uint32_t)(L - 1);
        const size_t tile0 = ((size_t)b * (size_t)N + (size_t)n0) * (size_t)D + (size_t)d0;
        const uint32_t span = (uint32_t)((((size_t)(n1 - n0) - 1) * (size_t)D + (size_t)weff) * 2);
        const __amdgpu_buffer_rsrc_t rin = make_rsrc(dn + tile0, span);
        const __amdgpu_buffer_rsrc_t rout = make_rsrc(out + tile0, span);
        const uint32_t vo = (uint32_t)(((size_t)(tid >> logq) * (size_t)D + (size_t)j) * 2);
        const uint32_t line_stride = (uint32_t)rpp * (uint32_t)D * 2u;
        const int passes = (int)((n1 - n0 + (int64_t)rpp * UNROLL - 1) / ((int64_t)rpp * UNROLL));
        if (MODE != kRaw && bad) {
            // Some levels read the LUT rows in memory: they have to be there.
            if (!write_lut) write_strip(coeffs, lut, D, L, b, d0, weff, lut_vec);
            __threadfence();
            __syncthreads();
        }
        const __amdgpu_buffer_rsrc_t rl = make_rsrc(
            lut + ((size_t)b * (size_t)D + (size_t)d0) * (size_t)L, (uint32_t)((size_t)weff * L * 2));
        if (!streams) {
            // nothing to stream
        } else if constexpr (MODE == kRaw) {
            const uint16_t* tile = (const uint16_t*)smem;
            stream_lines<VEC, UNROLL, 0>(
                rin, rout, vo, line_stride, passes,
                [&](int k, uint32_t d) { return g_raw(tile, d, top, logW, j + k); });
        } else if constexpr (MODE == kDense) {
            const uint32_t hb = (uint32_t)((L + 63) >> 6) << (logW + 3);
            if (!bad) {
                stream_lines<VEC, UNROLL, 0>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        const uint32_t p = (uint32_t)((k << logq) + lane);
                        return g_dense(d, top, logW, p * 8u, hb + p * 2u);
                    });
            } else {
                stream_lines<VEC, UNROLL, 0>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        const uint32_t p = (uint32_t)((k << logq) + lane);
                        const uint32_t v = d < top ? d : top;
                        int h = 0;
                        const uint32_t e = g_dense_min(d, top, logW, p * 8u, hb + p * 2u, h);
                        return h == (int)kDenseBad
                                   ? g_glb_l2(rl, (uint32_t)((j + k) * L * 2), v, top)
                                   : e;
                    });
            }
        } else {
            const int NB = (L + 31) >> 5;
            const u32x2* planes = (const u32x2*)smem;
            const uint16_t* bases = (const uint16_t*)(planes + (size_t)NB * (1 << logW));
            if (!bad) {
                stream_lines<VEC, UNROLL, 0>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        return g_packed(planes, bases, d, top, logW, (k << logq) + lane);
                    });
            } else {
                stream_lines<VEC, UNROLL, 0>(
                    rin, rout, vo, line_stride, passes, [&](int k, uint32_t d) {
                        return g_glb_l2(rl, (uint32_t)((j + k) * L * 2), d, top);
                    });
            }
        }
    }
    __syncthreads();  // the tile may be rebuilt next
}

}  // namespace rc
