// All-pairs central force of arbitrary shape from the bit-binned look-up
// table on gfx950: Eq. (arbitrary_force) of Sec. 3 with the force procedure
// of Sec. 3.4.2.
//
// Per pair (unscaled FP32 positions; the paper pre-scales positions by
// sqrt(s_max-2)/rcut instead, which rounds every absolute coordinate once
// more and loses digits for close pairs, so the scale is applied to |d|^2):
//   d = r_j - r_i                                       3 sub
//   s = min(c |d|^2 + 2, s_max), c = (s_max-2)/rcut^2    mul, 2 fma, fma, min
//   k = bits(s)[23-F .. 23+E)  (low E exponent bits and high F fraction bits,
//       one v_bfe_u32), byte address 8k                  2 int
//   s_k = bits(s) with the low 23-F bits cleared         1 int
//   (G0, G1) = T[k], one ds_read_b64 from the LDS copy of the table
//   g = G0 + G1 (s - s_k)                                sub, fma
//   a += (m g) d                                         mul, 3 fma
// The table (2^(E+F) (G0, G1) pairs, at most 128 KiB) is copied into LDS once
// per workgroup; j-particles stream through LDS tiles exactly as in the
// Newton kernel.  Pairs beyond the cutoff clamp to s_max, whose node is the
// last one, where G0 = G1 = 0, so they add exactly zero.
#include <algorithm>

#include "table_pairs.h"
#include "pgh_internal.h"
#include "rows.h"

namespace pgh {
namespace {

// PHI: also the potential from the second table (a.ptable, a.phi); the LDS
// table then holds (G0, G1, P0, P1) per node.  NT threads per workgroup.
template <int KI, int JT, int U, bool HT, bool PHI, int NT = 256>
__global__ void __launch_bounds__(NT) k_table_allpairs(TableArgs a)
{
    static_assert(JT % NT == 0, "tile must be a multiple of the workgroup");
    constexpr int PER = JT / NT;
    extern __shared__ float4 dyn4[];
    float2 *stab = (float2 *)dyn4;  // (G0, G1) per node
    float4 *stab4 = dyn4;           // (G0, G1, P0, P1) per node, with PHI
    __shared__ float4 tile[2][JT];

    const int tid = threadIdx.x;
    const int ibase = blockIdx.x * (NT * KI) + tid;
    const int K = 1 << (a.E + a.F);
    const unsigned shift = 23u - (unsigned)a.F;
    const unsigned nbits = (unsigned)(a.E + a.F);
    const unsigned hmask = ~((1u << shift) - 1u);
    const float c = a.c, smax = a.smax;

    if (PHI)
        tables_to_lds<HT>(stab4, a.table, a.ptable, K, shift);
    else
        table_to_lds<HT>(stab, a.table, K, shift);

    float px[KI], py[KI], pz[KI];
    float tx[KI], ty[KI], tz[KI], tp[KI];
#pragma unroll
    for (int k = 0; k < KI; ++k) {
        int i = ibase + k * NT;
        i = i < a.ni ? i : a.ni - 1;
        px[k] = a.xi[i];
        py[k] = a.yi[i];
        pz[k] = a.zi[i];
        tx[k] = ty[k] = tz[k] = tp[k] = 0.f;
    }

    // this workgroup's share of the j-particles (blockIdx.y splits them)
    const int jbase = blockIdx.y * a.jchunk;
    const int nj = max(0, min(a.jchunk, a.nj - jbase));
    const float4 *__restrict__ jm = a.jmem + jbase;
    const int ntiles = (nj + JT - 1) / JT;
    float4 pre[PER];
    auto load_tile = [&](int t) {
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int j = t * JT + r * NT + tid;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < nj) v = jm[j];
            pre[r] = v;
        }
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int r = 0; r < PER; ++r) tile[buf][r * NT + tid] = pre[r];
    };

    load_tile(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): see the Newton kernel
    store_tile(0);
    __syncthreads();

    for (int t = 0; t < ntiles; ++t) {
        const int cur = t & 1;
        set_tile_prio(ntiles - t, ntiles);
        if (t + 1 < ntiles) load_tile(t + 1);
        const int cnt = min(JT, nj - t * JT);
        float sx[KI], sy[KI], sz[KI], sp[KI];
#pragma unroll
        for (int k = 0; k < KI; ++k) sx[k] = sy[k] = sz[k] = sp[k] = 0.f;
        auto pair = [&](const float4 p) {
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                if (PHI)
                    table_pair_pot<HT>(p, px[k], py[k], pz[k], stab4, c, smax, shift, nbits, hmask,
                                       sx[k], sy[k], sz[k], sp[k]);
                else
                    table_pair<HT>(p, px[k], py[k], pz[k], stab, c, smax, shift, nbits, hmask,
                                   sx[k], sy[k], sz[k]);
            }
        };
        if (cnt == JT) {
#pragma unroll U
            for (int jj = 0; jj < JT; ++jj) pair(tile[cur][jj]);
        } else {
#pragma unroll 2
            for (int jj = 0; jj < cnt; ++jj) pair(tile[cur][jj]);
        }
#pragma unroll
        for (int k = 0; k < KI; ++k) {
            tx[k] += sx[k];
            ty[k] += sy[k];
            tz[k] += sz[k];
            tp[k] += sp[k];
        }
        if (t + 1 < ntiles) store_tile(cur ^ 1);
        __syncthreads();
    }

    float *ox = a.ax, *oy = a.ay, *oz = a.az, *op = a.phi;
    if (gridDim.y > 1) {
        ox = a.part + (size_t)blockIdx.y * 4 * a.ni;
        oy = ox + a.ni;
        oz = oy + a.ni;
        op = oz + a.ni;
    }
#pragma unroll
    for (int k = 0; k < KI; ++k) {
        const int i = ibase + k * NT;
        if (i < a.ni) {
            ox[i] = tx[k];
            oy[i] = ty[k];
            oz[i] = tz[k];
            if (PHI) op[i] = tp[k];
        }
    }
}

// The rows mapping of the table force (see k_newton_rows): TI i-particles per
// workgroup in SGPRs, j-particles over the lanes, and the pairs beyond the
// cutoff left after |d|^2.  A pair with |d|^2 >= a.r2max clamps to the last
// node, and where that node's entries are zero its terms are exact zeros: the
// table gather, the interpolation and the sums (10 of 17 instructions and the
// LDS access) run only where some lane of the wave has a pair inside the
// cutoff, tested for four i-particles at once.
//
// The pairs that would add something else than zero are never left out: with
// a last node other than zero, or a position or mass for which 0 x d or m x 0
// is not zero (infinite, NaN, or so large that |d|^2 could overflow), every
// pair takes the whole path.
//
// Bound by the FP32 issue of |d|^2 and the test where few pairs are inside
// the cutoff, and by the launch for small sets: N = 4096 in a box of 21 cutoffs
// 28.8 -> 12.7 us a call with 2^10 nodes, in 5 cutoffs 29.3 -> 13.4, in 1.7
// cutoffs 28.9 -> 14.2.
template <int TI, int NT, bool PHI>
__global__ void __launch_bounds__(NT) k_table_rows(TableArgs a)
{
    constexpr int C = PHI ? 4 : 3;
    constexpr int V = 4 * TI;
    constexpr int W = NT / 64;
    constexpr int Q = TI < 4 ? TI : 4;  // i-particles per test
    extern __shared__ float4 dyn4[];
    __shared__ float red[W][V];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int K = 1 << (a.E + a.F);

    // the first records are in flight while the table is copied
    const int jbase = blockIdx.y * a.jchunk;
    const int nj = min(a.jchunk, a.nj - jbase);
    const float4 *__restrict__ jm = a.jmem + jbase;
    const int full = nj / NT;
    auto load = [&](int t) { return jm[min(t * NT + tid, nj - 1)]; };
    float4 p0 = load(0), p1 = load(1);
    if (PHI)
        tables_to_lds<false>(dyn4, a.table, a.ptable, K, 0u);
    else
        table_to_lds<false>((float2 *)dyn4, a.table, K, 0u);
    const TableConsts kc = table_consts(a.c, a.smax, a.E, a.F, PHI ? 4 : 3);
    const char *tab = (const char *)dyn4;
    __syncthreads();
    bool last_zero;
    if (PHI) {
        const float4 e = dyn4[K - 1];
        last_zero = e.x == 0.f && e.y == 0.f && e.z == 0.f && e.w == 0.f;
    } else {
        const float2 e = ((const float2 *)dyn4)[K - 1];
        last_zero = e.x == 0.f && e.y == 0.f;
    }
    const unsigned r2max = __float_as_uint(a.r2max);

    const int groups = (a.ni + TI - 1) / TI;
    for (int g = blockIdx.x; g < groups; g += gridDim.x) {
        const int i0 = g * TI;
        float px[TI], py[TI], pz[TI], s[TI][C];
        bool whole = !last_zero;  // uniform: no pair may be left out
#pragma unroll
        for (int k = 0; k < TI; ++k) {
            const int i = min(i0 + k, a.ni - 1);
            px[k] = uniform(a.xi[i]);
            py[k] = uniform(a.yi[i]);
            pz[k] = uniform(a.zi[i]);
            whole = whole || !ordinary(px[k], py[k], pz[k], 0.f);
#pragma unroll
            for (int c = 0; c < C; ++c) s[k][c] = 0.f;
        }
        whole = __builtin_amdgcn_readfirstlane(whole);
        auto pairs = [&](const float4 p) {
            const bool all = whole || __any(!ordinary(p.x, p.y, p.z, p.w));
#pragma unroll
            for (int k0 = 0; k0 < TI; k0 += Q) {
                float dx[Q], dy[Q], dz[Q], r2[Q];
#pragma unroll
                for (int k = 0; k < Q; ++k) {
                    dx[k] = p.x - px[k0 + k];
                    dy[k] = p.y - py[k0 + k];
                    dz[k] = p.z - pz[k0 + k];
                    r2[k] = dx[k] * dx[k];
                    r2[k] = __builtin_fmaf(dy[k], dy[k], r2[k]);
                    r2[k] = __builtin_fmaf(dz[k], dz[k], r2[k]);
                }
                // (of non-negative numbers the bits compare as they do)
                unsigned least = __float_as_uint(r2[0]);
#pragma unroll
                for (int k = 1; k < Q; ++k) least = min(least, __float_as_uint(r2[k]));
                if (!(all | __any(least < r2max))) continue;
                // the whole path for NI of them from k1 on, gathers together
                auto tail = [&](auto k1, auto n) {
                    constexpr int K1 = decltype(k1)::value, NI = decltype(n)::value;
                    TableGather<NI, PHI> q;
#pragma unroll
                    for (int k = 0; k < NI; ++k) {
                        const unsigned u = min(
                            __float_as_uint(__builtin_fmaf(r2[K1 + k], kc.c, 2.0f)), kc.smax_bits);
                        q.t[k] = *(const typename TableGather<NI, PHI>::Entry *)(
                            tab + ((u >> kc.sh) & kc.am));
                        q.ds[k] = __uint_as_float(u) - __uint_as_float(u & kc.hm);
                    }
#pragma unroll
                    for (int k = 0; k < NI; ++k) {
                        float *o = s[k0 + K1 + k];
                        const float mg = p.w * __builtin_fmaf(q.t[k].y, q.ds[k], q.t[k].x);
                        o[0] = __builtin_fmaf(mg, dx[K1 + k], o[0]);
                        o[1] = __builtin_fmaf(mg, dy[K1 + k], o[1]);
                        o[2] = __builtin_fmaf(mg, dz[K1 + k], o[2]);
                        if constexpr (PHI)
                            o[3] = __builtin_fmaf(
                                p.w, __builtin_fmaf(q.t[k].w, q.ds[k], q.t[k].z), o[3]);
                    }
                };
                using std::integral_constant;
                // one by one where a single i-particle has pairs inside
                int hits = 0;
#pragma unroll
                for (int k = 0; k < Q; ++k) hits += __any(__float_as_uint(r2[k]) < r2max) ? 1 : 0;
                if (all || Q == 1 || 2 * hits > Q) {
                    tail(integral_constant<int, 0>{}, integral_constant<int, Q>{});
                    continue;
                }
                if (__any(__float_as_uint(r2[0]) < r2max))
                    tail(integral_constant<int, 0>{}, integral_constant<int, 1>{});
                if constexpr (Q > 1)
                    if (__any(__float_as_uint(r2[1]) < r2max))
                        tail(integral_constant<int, 1>{}, integral_constant<int, 1>{});
                if constexpr (Q > 2) {
                    if (__any(__float_as_uint(r2[2]) < r2max))
                        tail(integral_constant<int, 2>{}, integral_constant<int, 1>{});
                    if (__any(__float_as_uint(r2[3]) < r2max))
                        tail(integral_constant<int, 3>{}, integral_constant<int, 1>{});
                }
            }
        };

        int t = 0;
        for (; t + 2 <= full; t += 2) {
            pairs(p0);
            p0 = load(t + 2);
            __builtin_amdgcn_sched_barrier(0);
            pairs(p1);
            p1 = load(t + 3);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (t < full) {
            pairs(p0);
            p0 = p1;
            ++t;
        }
        if (t * NT < nj) {
            // a zero-mass record far away adds exactly zero
            if (t * NT + tid >= nj) p0 = make_float4(1.0e10f, 1.0e10f, 1.0e10f, 0.f);
            pairs(p0);
        }
        if (g + (int)gridDim.x < groups) p0 = load(0), p1 = load(1);

#pragma unroll
        for (int k = 0; k < TI; ++k) {
            const float v = row_sum(fold_rows(fold_halves(s[k][0], s[k][1]),
                                              fold_halves(s[k][2], PHI ? s[k][C - 1] : 0.f)));
            const int row = lane >> 4, c = ((row & 1) << 1) | (row >> 1);
            if ((lane & 15) == 0) red[wave][4 * k + c] = v;
        }
        __syncthreads();
        if (tid < V) {
            float r = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) r += red[w][tid];
            const int c = tid & 3, i = i0 + (tid >> 2);
            if (i < a.ni && c < C) {
                if (gridDim.y > 1)
                    a.part[((size_t)blockIdx.y * 4 + c) * a.ni + i] = r;
                else
                    (c == 0 ? a.ax : c == 1 ? a.ay : c == 2 ? a.az : a.phi)[i] = r;
            }
        }
        if (g + (int)gridDim.x < groups) __syncthreads();
    }
}

using TableKernel = void (*)(TableArgs);

// Tables of more than 32 KiB in LDS (2^13 nodes and more, or 2^12 with the
// potential) leave room for one or two workgroups per CU, so they run
// workgroups of 12 waves (three per SIMD) over 768-record j-tiles: 128 KiB
// of table and 24 KiB of tiles fit the 160 KiB of a CU.  With four-wave
// workgroups such a table left one or two waves per SIMD, too few to hide
// the LDS latency of the table reads or to pair FP32 issue.
constexpr int kWideNT = 768;
constexpr size_t kWideTableBytes = 32768;
// the j-split target of wide launches: three rounds of one workgroup on each
// of 256 CUs
constexpr int kWideTargetWaves = 3 * (kWideNT / 64) * 256;

// The rows kernel copies tables of more than 16 KiB into workgroups of 16
// waves (two or one to a CU), which take several groups of i-particles each.
constexpr size_t kRowsTableBytes = 16384;

// ki = 0: the rows kernel, whose shape follows from the sizes (rows_shape).
struct TableVariant {
    const char *name;
    int ki, jt;
    TableKernel fn, fn_phi;      // force only; force and potential
    TableKernel wide, wide_phi;  // the same with kWideNT threads and tiles
};

#define PGH_TABLE_VARIANT(name, KI, JT, U, HT)                                                   \
    {name,                                                                                     \
     KI,                                                                                       \
     JT,                                                                                       \
     k_table_allpairs<KI, JT, U, HT, false>,                                                   \
     k_table_allpairs<KI, JT, U, HT, true>,                                                    \
     k_table_allpairs<KI, kWideNT, U, HT, false, kWideNT>,                                     \
     k_table_allpairs<KI, kWideNT, U, HT, true, kWideNT>}
const TableVariant kTableVariants[] = {
    PGH_TABLE_VARIANT("ki=1 jt=256 u=4", 1, 256, 4, false),
    PGH_TABLE_VARIANT("ki=2 jt=256 u=4", 2, 256, 4, false),
    PGH_TABLE_VARIANT("ki=4 jt=256 u=2", 4, 256, 2, false),
    PGH_TABLE_VARIANT("ki=1 jt=256 u=4 htab", 1, 256, 4, true),
    PGH_TABLE_VARIANT("ki=2 jt=256 u=4 htab", 2, 256, 4, true),
    {"rows", 0, 64, nullptr, nullptr, nullptr, nullptr},
};
#undef PGH_TABLE_VARIANT
constexpr int kRowsVariant = 5;
constexpr int kNumTableVariants = sizeof(kTableVariants) / sizeof(kTableVariants[0]);

bool is_phi(const TableArgs &a) { return a.phi && a.ptable; }

size_t table_lds_bytes(const TableArgs &a)
{
    return (is_phi(a) ? sizeof(float4) : sizeof(float2)) << (a.E + a.F);
}

}  // namespace

int table_allpairs_variants() { return kNumTableVariants; }

const char *table_allpairs_variant_name(int v)
{
    return (v >= 0 && v < kNumTableVariants) ? kTableVariants[v].name : nullptr;
}

int table_allpairs_default(int ni, int nj, int num_cu)
{
    // The rows kernel for small sets, whose time is launches and idle CUs with
    // a workgroup per 256 i-particles (N = 1000: 12.5 against 58 us, most of it
    // the host's; 4096 13 to 14 against 29 whatever the pairs inside).
    if ((double)ni * nj <= 3.0e7) return kRowsVariant;
    const long waves_ki2 = (long)(ni + 127) / 128;
    return waves_ki2 >= 4L * num_cu ? 1 : 0;
}

int table_allpairs_split(const TableArgs &a, int variant, size_t part_cap)
{
    const TableVariant &v = kTableVariants[variant];
    if (v.ki == 0)
        return (int)std::max(1L, std::min((long)rows_shape(a.ni, a.nj).shares,
                                          (long)(part_cap / (4 * (size_t)std::max(a.ni, 1)))));
    if (table_lds_bytes(a) > kWideTableBytes)
        return split_count(a.ni, a.nj, v.ki, kWideNT, kWideTargetWaves, part_cap);
    return split_count(a.ni, a.nj, v.ki, v.jt, kSplitTargetWaves, part_cap);
}

namespace {

template <int NT>
TableKernel rows_kernel(int ti, bool phi)
{
    switch (ti) {
        case 1: return phi ? k_table_rows<1, NT, true> : k_table_rows<1, NT, false>;
        case 2: return phi ? k_table_rows<2, NT, true> : k_table_rows<2, NT, false>;
        case 4: return phi ? k_table_rows<4, NT, true> : k_table_rows<4, NT, false>;
        default: return phi ? k_table_rows<8, NT, true> : k_table_rows<8, NT, false>;
    }
}

hipError_t launch_table_rows(TableArgs a, int S, int num_cu, hipStream_t s)
{
    const bool phi = is_phi(a);
    const size_t lds = table_lds_bytes(a);
    RowsShape r = rows_shape(a.ni, a.nj);
    long blocks = ((long)a.ni + r.ti - 1) / r.ti;
    if (lds > kRowsTableBytes) {
        r.nt = 1024;
        // as many workgroups as are resident at once, each several groups
        blocks = std::min(blocks, std::max(1L, (lds <= 65536 ? 2L : 1L) * num_cu / S));
    }
    a.jchunk = (int)(((long)a.nj + (long)S * 64 - 1) / ((long)S * 64) * 64);
    S = std::max(1, (a.nj + a.jchunk - 1) / a.jchunk);
    const TableKernel kern = r.nt == 1024 ? rows_kernel<1024>(r.ti, phi) : rows_kernel<256>(r.ti, phi);
    hipError_t e = allow_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks, S), dim3(r.nt), lds, s, a);
    e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    return launch_combine_split(a.ni, S, a.part, a.ax, a.ay, a.az, phi ? a.phi : nullptr, s);
}

}  // namespace

hipError_t launch_table_allpairs(const TableArgs &a0, int variant, int S, int num_cu,
                                 hipStream_t s)
{
    if (a0.ni <= 0) return hipSuccess;
    const TableVariant &v = kTableVariants[variant];
    TableArgs a = a0;
    const bool phi = is_phi(a);
    const size_t lds = table_lds_bytes(a);
    const bool wide = lds > kWideTableBytes;
    const int nt = wide ? kWideNT : 256, jt = wide ? kWideNT : v.jt;
    S = std::max(1, S);
    if (v.ki == 0) return launch_table_rows(a, S, num_cu, s);
    a.jchunk = (int)(((long)a.nj + (long)S * jt - 1) / ((long)S * jt) * jt);
    S = std::max(1, (a.nj + a.jchunk - 1) / a.jchunk);
    const int per_block = nt * v.ki;
    const dim3 grid((a.ni + per_block - 1) / per_block, S);
    const auto kern = wide ? (phi ? v.wide_phi : v.wide) : (phi ? v.fn_phi : v.fn);
    hipError_t e = allow_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(nt), lds, s, a);
    e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    return launch_combine_split(a.ni, S, a.part, a0.ax, a0.ay, a0.az, phi ? a0.phi : nullptr, s);
}

namespace {

// Gradient with respect to the node values when the slopes are derived from
// them, G1_k = (G0_{k+1} - G0_k) / (s_{k+1} - s_k) for k < K-1 (the table
// definition of Sec. 3.4.1), given the gradients with respect to G0 and G1
// as independent entries (interleaved like the table):
//   dL/dG0_k (total) = dL/dG0_k + dL/dG1_{k-1} / ds_{k-1} - dL/dG1_k / ds_k,
// each term present where its index exists (G1_{K-1} is the constant 0).
__global__ void __launch_bounds__(256) k_table_grad_chain(int K, unsigned shift,
                                                          const float *__restrict__ g,
                                                          float *__restrict__ out)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    // node s_k: the FP32 bits of 2.0 stepped by k units of the F-th fraction bit
    auto node = [&](int q) { return __uint_as_float(0x40000000u + ((unsigned)q << shift)); };
    float v = g[2 * k];
    if (k >= 1) v += g[2 * (k - 1) + 1] / (node(k) - node(k - 1));
    if (k + 1 < K) v -= g[2 * k + 1] / (node(k + 1) - node(k));
    out[k] = v;
}

}  // namespace

hipError_t launch_table_grad_chain(int E, int F, const float *g, float *out, hipStream_t s)
{
    const int K = 1 << (E + F);
    hipLaunchKernelGGL(k_table_grad_chain, dim3((K + 255) / 256), dim3(256), 0, s, K,
                       23u - (unsigned)F, g, out);
    return hipGetLastError();
}

}  // namespace pgh
