// Which pairs of 64 j-particles and 64 i-particles are inside the cutoff of
// the table force, found on the matrix cores.
//
// A pair at or beyond the cutoff clamps to the table's last node (Sec. 3.4.2);
// where that node's entries are zero the pair adds exactly zero, so only the
// others need the table.  For short-range forces these are few (one list entry
// in eighty of a TreePM cell list), and forming |d|^2 for every pair is then
// most of the work.  |r_j|^2 + |r_i|^2 - 2 r_j . r_i is a contraction: with
// the coordinates relative to a centre c of the i-particles, and each
// number split into two bf16 parts (h + m, 16 bits), it is the product of a
// j-row and an i-column of 16 terms, 32 x 32 pairs per
// v_mfma_f32_32x32x16_bf16:
//   j: xh xh xm xm yh yh ym ym | zh zh zm zm nh nm 1 1
//   i: Xh Xm Xh Xm Yh Ym Yh Ym | Zh Zm Zh Zm 1 1 Nh Nm
// with X = -2x and n, N = |r|^2.  The sign of D = n + N + X.x - T then marks the
// candidates, and each of these is evaluated as before in FP32 on the unscaled
// positions: the filter decides nothing that reaches a result.
//
// No pair inside the cutoff may be missed.  With S = |r_i|^2 + |r_j|^2 (about
// c), the parts dropped by the splits change D by at most 2^-15 S (products)
// + 2^-16 S (norms), 16 FP32 additions by 2^-18 S, and the FP32 differences
// to c by 2^-21 S; both norms are scaled by 1 - 2^-14, which takes 2^-14 S off
// D.  T is r2max, the least |d|^2 that clamps, raised by 2^-13 of itself for
// its own part of these errors.  What the raised T and norms let through
// besides is found out by the FP32 evaluation.
//
// Particles that are not ordinary() (infinite, NaN, huge) and, when the last
// node is not zero or the cutoff not filter_cut(), all i-particles get a norm that makes every pair of theirs
// a candidate; rows past a list's end and unused columns one that makes none.
#pragma once

#include <hip/hip_runtime.h>

#include "rows.h"
#include "table_pairs.h"

namespace pgh {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr float kFilterNorm = 1.0f - 0x1p-14f;
constexpr float kFilterCut = 1.0f + 0x1p-13f;
constexpr float kAlways = -1.0e36f, kNever = 1.0e37f;  // beside norms of at most 1.2e31

// Whether the products can tell distances from the cutoff: far above the
// smallest numbers, which they may flush, and no larger than the norms.  False
// for the r2max of tables without an ordinary cutoff, which need not be a number
// (a table of one node) nor above zero (|d|^2 in units of a tiny cutoff overflows).
__device__ __forceinline__ bool filter_cut(float r2max)
{
    return r2max > 1.0e-30f && r2max < 1.0e30f;
}

// The two operands of 64 particles, one per lane: t[0] of particles 0 .. 31,
// t[1] of 32 .. 63 (lanes < 32 hold the first eight terms of particle lane mod
// 32, the others the last eight).
struct FilterOps {
    u32x4 t[2];
};

__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    bf16x2 v;
    v.x = (__bf16)a;
    v.y = (__bf16)b;
    return __builtin_bit_cast(unsigned, v);
}

// The number's two bf16 parts as floats.
__device__ __forceinline__ void split_bf16(float a, float &h, float &m)
{
    h = (float)(__bf16)a;
    m = a - h;  // exact; rounded to bf16 when packed
}

// The lanes' first and second halves of terms exchanged into the operands.
__device__ __forceinline__ FilterOps filter_ops(const unsigned *k0, const unsigned *k1)
{
    FilterOps o;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const u32x2 r = __builtin_amdgcn_permlane32_swap(k0[w], k1[w], false, false);
        o.t[0][w] = r.x;
        o.t[1][w] = r.y;
    }
    return o;
}

// j-rows: positions relative to the centre and norm.
__device__ __forceinline__ FilterOps filter_rows(float x, float y, float z, float n)
{
    float xh, xm, yh, ym, zh, zm, nh, nm;
    split_bf16(x, xh, xm);
    split_bf16(y, yh, ym);
    split_bf16(z, zh, zm);
    split_bf16(n, nh, nm);
    const unsigned k0[4] = {pack_bf16(xh, xh), pack_bf16(xm, xm), pack_bf16(yh, yh),
                            pack_bf16(ym, ym)};
    const unsigned k1[4] = {pack_bf16(zh, zh), pack_bf16(zm, zm), pack_bf16(nh, nm), 0x3f803f80u};
    return filter_ops(k0, k1);
}

// i-columns: the same with X = -2x; the norm less T.
__device__ __forceinline__ FilterOps filter_cols(float x, float y, float z, float n)
{
    float xh, xm, yh, ym, zh, zm, nh, nm;
    split_bf16(-2.0f * x, xh, xm);
    split_bf16(-2.0f * y, yh, ym);
    split_bf16(-2.0f * z, zh, zm);
    split_bf16(n, nh, nm);
    const unsigned x2 = pack_bf16(xh, xm), y2 = pack_bf16(yh, ym), z2 = pack_bf16(zh, zm);
    const unsigned k0[4] = {x2, x2, y2, y2};
    const unsigned k1[4] = {z2, z2, 0x3f803f80u, pack_bf16(nh, nm)};
    return filter_ops(k0, k1);
}

// A lane's value of particle l mod 32 and of particle 32 + l mod 32.
__device__ __forceinline__ void both_halves(float v, float *o)
{
    const u32x2 r =
        __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    o[0] = __uint_as_float(r.x);
    o[1] = __uint_as_float(r.y);
}

// The least and the greatest of a wave's 64 values (all lanes active, none a
// NaN), in every lane: over each row of 16 by rotation (8, 4, 2, 1), then
// across the four rows.
template <class Op>
__device__ __forceinline__ float wave_fold(float v, Op op)
{
    v = op(v, dpp_f32<0x128>(v));
    v = op(v, dpp_f32<0x124>(v));
    v = op(v, dpp_f32<0x122>(v));
    v = op(v, dpp_f32<0x121>(v));
    const int u = (int)__float_as_uint(v);
    auto row = [&](int l) { return __uint_as_float((unsigned)__builtin_amdgcn_readlane(u, l)); };
    return op(op(row(0), row(16)), op(row(32), row(48)));
}

__device__ __forceinline__ float wave_min(float v)
{
    return wave_fold(v, [](float a, float b) { return __builtin_fminf(a, b); });
}

__device__ __forceinline__ float wave_max(float v)
{
    return wave_fold(v, [](float a, float b) { return __builtin_fmaxf(a, b); });
}

// The set bits of a ballot in lanes below this one.
__device__ __forceinline__ int lanes_below(unsigned long long who)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(who >> 32),
                                          __builtin_amdgcn_mbcnt_lo((unsigned)who, 0u));
}

// The candidates of 64 rows for the column lane mod 32 of one operand: bit
// 31 - p of lane (column, half h) is row filter_row(p, h).
__device__ __forceinline__ unsigned filter_mask(const FilterOps &rows, const u32x4 cols)
{
    unsigned m = 0;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const f32x16 zero = {};
        const f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, rows.t[t]), __builtin_bit_cast(bf16x8, cols), zero, 0, 0, 0);
        // the sign bits, shifted in one by one
#pragma unroll
        for (int r = 0; r < 16; ++r)
            m = __builtin_amdgcn_alignbit(m, __float_as_uint(d[r]), 31u);
        // one product's 16 registers at a time (the waves of a SIMD cover each
        // other's products, and more waves fit): the word is formed here
        asm volatile("" : "+v"(m));
        __builtin_amdgcn_sched_barrier(0);
    }
    return m;
}

// Rows are kept in LDS in the order of the mask's bits: half h's bit 31 - p in
// slot 32 h + p, which holds row 32 (p / 16) + 8 ((p / 4) mod 4) + 4 h + p mod 4
// (element r = p mod 16 of the matrix result).  The slot of row j:
__device__ __forceinline__ int filter_slot(int j)
{
    return ((j & 4) << 3) | ((j & 0x38) >> 1) | (j & 3);
}

// A lane's row for filter_rows: the record v relative to (cx, cy, cz), or a
// norm that makes it a candidate always or never.
__device__ __forceinline__ FilterOps filter_rows_of(const float4 v, bool valid, float cx, float cy,
                                                    float cz)
{
    const bool ok = valid && ordinary(v.x, v.y, v.z, v.w);
    const float x = ok ? v.x - cx : 0.f, y = ok ? v.y - cy : 0.f, z = ok ? v.z - cz : 0.f;
    const float n = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x)) * kFilterNorm;
    return filter_rows(x, y, z, ok ? n : valid ? kAlways : kNever);
}

// A lane's column: position, whether it is in use, and whether pairs beyond
// the cutoff may be left out at all (the last node is zero); cut = r2max.
__device__ __forceinline__ FilterOps filter_cols_of(float px, float py, float pz, bool valid,
                                                    bool last_zero, float cx, float cy, float cz,
                                                    float cut)
{
    const bool ok = valid && last_zero && ordinary(px, py, pz, 0.f);
    const float x = ok ? px - cx : 0.f, y = ok ? py - cy : 0.f, z = ok ? pz - cz : 0.f;
    const float n = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x)) * kFilterNorm;
    return filter_cols(x, y, z, ok ? n - cut * kFilterCut : valid ? kAlways : kNever);
}

}  // namespace pgh
