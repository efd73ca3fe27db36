// The "rows" mapping of the all-pairs launches (newton.hip, lut.hip): a
// workgroup holds a few i-particles as wave-uniform values, its lanes take the
// j-particles, and the lanes' sums meet at the end.  And what other kernels too do
// across the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

namespace pgh {

// Sums over the lanes of a wave, two or four values at a time: v_permlane32_swap
// exchanges the upper half of a with the lower half of b, so one add leaves
// a's sum over lane pairs (l, l + 32) in the lower half and b's in the upper;
// v_permlane16_swap does the same with rows of 16.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float fold_halves(float a, float b)
{
    const u32x2 r =
        __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}

__device__ __forceinline__ float fold_rows(float a, float b)
{
    const u32x2 r =
        __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __uint_as_float(
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}

// LDS operations of one wave complete in order; this keeps the compiler
// from moving reads of a wave's tile above the writes of its other lanes.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The sum over each row of 16 lanes, in all of them (row_ror 8, 4, 2, 1).
__device__ __forceinline__ float row_sum(float v)
{
    v += dpp_f32<0x128>(v);
    v += dpp_f32<0x124>(v);
    v += dpp_f32<0x122>(v);
    v += dpp_f32<0x121>(v);
    return v;
}

// The shape of a rows launch: i-particles and threads per workgroup, and the
// j-shares it asks for.
struct RowsShape {
    int ti, nt, shares;
};

inline RowsShape rows_shape(int ni, int nj)
{
    RowsShape r;
    // More i-particles per workgroup save j-record loads and end-of-loop
    // sums, fewer give the workgroups that fill 256 CUs eight deep.  us of
    // force at TI = 2, 4, 8: N = 4096 7.9, 8.0, 8.5; 6000 16.2, 15.2, 15.5;
    // 8192 28.1, 24.7, 24.8; 11000 -, 42.8, 45.1; 16384 -, 89.0, 85.1; 65536
    // -, 1355, 1266.  Few i-particles over a long list are bound by reading it
    // from the L2 (1000 x 60000: TI = 2, 4 24.3, 23.6; 300 x 262144, shares
    // alike: 38.6, 36.0), else by latency (256 x 4096: TI = 1, 2, 4 3.0, 3.2, 4.0).
    // Lists of more than the 4 MiB of an L2 take the most, and shares below.
    const bool beyond_l2 = nj >= 1 << 18 && ni >= 2000;
    if (ni >= 12000 || beyond_l2)
        r.ti = 8;
    else if (ni >= 4500 || (ni >= 500 && nj >= 32768) || (ni >= 200 && nj >= 65536))
        r.ti = 4;
    else
        r.ti = ni >= 200 ? 2 : 1;
    const long groups = ((long)ni + r.ti - 1) / r.ti;
    // sixteen waves per workgroup where there are few workgroups and at least
    // four records per lane (300 x 16384, four and sixteen waves: 6.4, 5.2 us)
    r.nt = r.ti <= 4 && groups < 1024 && nj >= 4096 ? 1024 : 256;
    // and shares of at least 8192 records where even these leave the chip idle
    // (64 x 60000, one and eight shares: 9.6, 6.7 us, the second launch included)
    const long waves = groups * (r.nt / 64);
    r.shares = 1;
    if (waves < (beyond_l2 ? 4096 : 2048))
        r.shares = (int)std::max(1L, std::min(((beyond_l2 ? 8192 : 4096) + waves - 1) / waves,
                                              (long)nj / 8192));
    return r;
}

}  // namespace pgh
