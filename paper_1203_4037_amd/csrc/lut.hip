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
#include "table_filter.h"

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
    if (a.dense && *a.dense == 0) return;  // k_table_near computes this call

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
// A step whose tests all found pairs of most of their i-particles inside is
// followed by this many evaluated whole without a test.
constexpr int kWholeSteps = 7;
// k_table_near: a lane's sums are added to its totals before a step that finds this many
// terms in them; a step with at most kLightHits candidates in every lane counts for as
// many, any other for all its 32 rows.
constexpr int kFreshTerms = 512, kLightHits = 4;

// One j-record of the lane against Q uniform i-particles; s[k]: their sums.
template <int Q, bool PHI>
__device__ __forceinline__ void whole_pairs(const float4 p, const float *px, const float *py,
                                            const float *pz, const char *tab, const TableConsts &kc,
                                            float (*s)[PHI ? 4 : 3])
{
    TableGather<Q, PHI> q;
    table_head<Q, false, PHI>(p, px, py, pz, tab, kc, q);
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const float mg = p.w * __builtin_fmaf(q.t[k].y, q.ds[k], q.t[k].x);
        s[k][0] = __builtin_fmaf(mg, q.dx[k], s[k][0]);
        s[k][1] = __builtin_fmaf(mg, q.dy[k], s[k][1]);
        s[k][2] = __builtin_fmaf(mg, q.dz[k], s[k][2]);
        if constexpr (PHI)
            s[k][3] = __builtin_fmaf(p.w, __builtin_fmaf(q.t[k].w, q.ds[k], q.t[k].z), s[k][3]);
    }
}

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
        int blind = 0;  // steps still to be evaluated whole without a test
        auto pairs = [&](const float4 p) {
            if (blind > 0) {
                --blind;
#pragma unroll
                for (int k0 = 0; k0 < TI; k0 += Q)
                    whole_pairs<Q, PHI>(p, px + k0, py + k0, pz + k0, tab, kc, s + k0);
                return;
            }
            const bool all = whole || __any(!ordinary(p.x, p.y, p.z, p.w));
            int most = 0;  // tests that found pairs of most of their i-particles
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
                    ++most;
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
            if (most == TI / Q) blind = kWholeSteps;
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
            // the other lanes hold the last record, which without its mass adds
            // zero (a record far away would take the last node, not a number
            // perhaps, where no pair does)
            if (t * NT + tid >= nj) p0.w = 0.f;
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

// Whether most pairs are to be evaluated: more than a quarter of 8 spread
// i-particles' pairs with 4096 spread j-particles inside the cutoff, or a last
// node that is not zero.  It chooses the kernel, never what is computed.
template <bool PHI>
__global__ void __launch_bounds__(1024) k_table_density(TableArgs a, int *dense)
{
    __shared__ int count;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    int n = 0;
    float4 p[4], q[8];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        p[k] = a.jmem[(long long)(4 * threadIdx.x + k) * a.nj / 4096];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int i = (int)((2 * k + 1) * (long long)a.ni / 16);
        q[k] = make_float4(a.xi[i], a.yi[i], a.zi[i], 0.f);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
        for (int l = 0; l < 4; ++l) {
            const float dx = p[l].x - q[k].x, dy = p[l].y - q[k].y, dz = p[l].z - q[k].z;
            n += dx * dx + dy * dy + dz * dz < a.r2max ? 1 : 0;
        }
    for (int m = 32; m; m >>= 1) n += __shfl_xor(n, m);
    if ((threadIdx.x & 63) == 0) atomicAdd(&count, n);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int K = 1 << (a.E + a.F);
        const float2 e = a.table[K - 1];
        bool zero = e.x == 0.f && e.y == 0.f;
        if (PHI) zero = zero && a.ptable[K - 1].x == 0.f && a.ptable[K - 1].y == 0.f;
        *dense = count > 8 * 4096 / 4 || !zero ? 1 : 0;
    }
}

// The all-pairs table force with the pairs beyond the cutoff found on the
// matrix cores (table_filter.h) and left out, for sets that are not small: the
// workgroup's W waves hold the same chunk of NC columns of 32 i-particles (lane
// l holds l mod 32 of each) and take a share of the j-particles each, 64
// records at a time, two steps ahead; records farther than the cutoff from the
// box around the chunk are dropped (which helps sets in cell or curve order),
// the others go to the wave's LDS tile and, as bf16 terms, into the products,
// 2 NC of them.  Each lane then evaluates its own candidates in FP32.  A step
// most of whose pairs are inside is evaluated whole, and the next kWholeSteps
// after it without a test.  The waves' sums meet in LDS at the end.
//
// Per 64 records and column 78 VALU instructions (counted; 32 of them signs, 17 its
// share of the records' terms) and two products, against 64 x 17 / 2 before: bound by
// the issue of these, one every 4.4 cycles of a SIMD, the matrix cores busy a fifth
// of the time.  N = 65536 (T16, phi off) in a box of 21 cutoffs 1121 -> 280 us, of 5
// cutoffs 1138 -> 478, with most pairs inside 1216 -> 1390 (auto_kernel leaves that to
// k_table_allpairs); N = 16384 81 -> 28 us.
template <int NC, int W, bool PHI>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_table_near(TableArgs a)
{
    constexpr int NI = 32 * NC;  // i-particles per chunk
    constexpr int C = PHI ? 4 : 3;
    extern __shared__ float4 dyn4[];
    if (a.dense && *a.dense != 0) return;  // k_table_allpairs computes this call
    const int K = 1 << (a.E + a.F);
    // after the table (one (G0, G1) takes a float4 all the same) each wave's
    // tile of 64 records, then each wave's sums of the chunk
    float4 *const tiles = dyn4 + (PHI ? K : (K + 1) / 2), *const sums = tiles + 64 * W;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float4 *const tile = tiles + 64 * wave, *const total = sums + wave * NI;

    // the wave's share of the j-particles, a multiple of 64 records
    const int per = ((a.nj + 64 * W - 1) / (64 * W)) * 64;
    const int jbase = min(wave * per, a.nj);
    const int nj = min(per, a.nj - jbase);
    const float4 *__restrict__ jm = a.jmem + jbase;
    auto load = [&](int base) { return jm[max(0, min(base + lane, nj - 1))]; };

    if (PHI)
        tables_to_lds<false>(dyn4, a.table, a.ptable, K, 0u);
    else
        table_to_lds<false>((float2 *)dyn4, a.table, K, 0u);
    const char *tab = (const char *)dyn4;
    const unsigned kshift = 23u - (unsigned)a.F;
    const TableConsts kc{a.c, __float_as_uint(a.smax), kshift - (PHI ? 4 : 3),
                         (unsigned)(K - 1) << (PHI ? 4 : 3), ~((1u << kshift) - 1u)};
    __syncthreads();
    bool last_zero = filter_cut(a.r2max);
    if (PHI) {
        const float4 e = dyn4[K - 1];
        last_zero = last_zero && e.x == 0.f && e.y == 0.f && e.z == 0.f && e.w == 0.f;
    } else {
        const float2 e = ((const float2 *)dyn4)[K - 1];
        last_zero = last_zero && e.x == 0.f && e.y == 0.f;
    }

    const int groups = (a.ni + NI - 1) / NI;
    for (int g = blockIdx.x; g < groups; g += gridDim.x) {
        const int i0 = g * NI, n_i = min(NI, a.ni - i0);
        float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0;
        if (nj > 0) p0 = load(0), p1 = load(64);
        // the chunk, 64 i-particles at a time (past its end its first)
        float ix[NC / 2], iy[NC / 2], iz[NC / 2];
        bool odd = false;
        float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int q = 0; q < NC / 2; ++q) {
            const int k = 64 * q + lane, i = i0 + (k < n_i ? k : 0);
            ix[q] = a.xi[i];
            iy[q] = a.yi[i];
            iz[q] = a.zi[i];
            odd = odd || !ordinary(ix[q], iy[q], iz[q], 0.f);
            lo[0] = __builtin_fminf(lo[0], ix[q]), hi[0] = __builtin_fmaxf(hi[0], ix[q]);
            lo[1] = __builtin_fminf(lo[1], iy[q]), hi[1] = __builtin_fmaxf(hi[1], iy[q]);
            lo[2] = __builtin_fminf(lo[2], iz[q]), hi[2] = __builtin_fmaxf(hi[2], iz[q]);
        }
        const bool whole = !last_zero || __any(odd);
        float bl[3], bh[3], ce[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            bl[c] = uniform(whole ? -INFINITY : wave_min(lo[c]));
            bh[c] = uniform(whole ? INFINITY : wave_max(hi[c]));
            ce[c] = uniform(whole ? 0.f : 0.5f * (bl[c] + bh[c]));
        }
        u32x4 cols[NC];
        float px[NC], py[NC], pz[NC];
        float tx[NC], ty[NC], tz[NC], tp[NC];
#pragma unroll
        for (int q = 0; q < NC / 2; ++q) {
            const FilterOps o = filter_cols_of(ix[q], iy[q], iz[q], 64 * q + lane < n_i, last_zero,
                                               ce[0], ce[1], ce[2], a.r2max);
            cols[2 * q] = o.t[0];
            cols[2 * q + 1] = o.t[1];
            both_halves(ix[q], px + 2 * q);
            both_halves(iy[q], py + 2 * q);
            both_halves(iz[q], pz + 2 * q);
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) tx[q] = ty[q] = tz[q] = tp[q] = 0.f;
        // A column's sums of both halves' rows go to its words in LDS before they
        // have many terms, so that FP32 rounding grows with kFreshTerms and the
        // number of these sums, not with the wave's share of the list (10^6
        // neighbours of one mass: 1.6e-4 in one running sum).
#pragma unroll
        for (int q = 0; q < NC / 2; ++q) total[64 * q + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        auto to_total = [&] {
#pragma unroll
            for (int q = 0; q < NC; q += 2) {
                // lane l: column q for l < 32, q + 1 for the others
                auto both = [&](float *v) {
                    const float a = v[q] + __shfl_xor(v[q], 32);
                    const float b = v[q + 1] + __shfl_xor(v[q + 1], 32);
                    v[q] = v[q + 1] = 0.f;
                    return lane < 32 ? a : b;
                };
                float4 t = total[32 * q + lane];
                t.x += both(tx), t.y += both(ty), t.z += both(tz);
                if (PHI) t.w += both(tp);
                total[32 * q + lane] = t;
            }
        };

        int fresh = 0;  // terms in a sum at most
        int blind = 0;  // steps still to be evaluated whole without a test
        for (int base = 0; base < nj; base += 64) {
            const float4 v = p0;
            p0 = p1;
            p1 = load(base + 128);
            const float ex = __builtin_fmaxf(__builtin_fmaxf(bl[0] - v.x, v.x - bh[0]), 0.f);
            const float ey = __builtin_fmaxf(__builtin_fmaxf(bl[1] - v.y, v.y - bh[1]), 0.f);
            const float ez = __builtin_fmaxf(__builtin_fmaxf(bl[2] - v.z, v.z - bh[2]), 0.f);
            const float r2 = __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex));
            const bool valid = base + lane < nj;
            // (each step is monotone: no pair with the chunk has a smaller |d|^2)
            const bool keep = valid && (whole || r2 < a.r2max || !ordinary(v.x, v.y, v.z, v.w));
            if (!__any(keep)) continue;
            if (fresh >= kFreshTerms) {
                to_total();
                fresh = 0;
            }
            wave_sync();  // the previous step's reads are done
            // (dropped, or past the end and so the last record again: without
            // its mass, so that the whole path adds zero for it)
            tile[filter_slot(lane)] = make_float4(v.x, v.y, v.z, keep ? v.w : 0.f);
            wave_sync();
            const float4 *mine = tile + (lane & 32);
            bool direct = blind > 0;
            unsigned m[NC];
            if (!direct) {
                const FilterOps rows = filter_rows_of(v, keep, ce[0], ce[1], ce[2]);
                int hits = 0;
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    m[q] = filter_mask(rows, cols[q]);
                    hits += __popc(m[q]);
                }
                direct = __any(hits > 12 * NC);
                if (direct) blind = kWholeSteps + 1;
                else fresh += __any(hits > kLightHits) ? 32 : kLightHits;
            }
            if (direct) {
                --blind;
                fresh += 32;
                const TableConsts kd = table_consts(a.c, a.smax, a.E, a.F, PHI ? 4 : 3);
#pragma unroll (NC == 2 ? 4 : 2)
                for (int p = 0; p < 32; ++p)
                    table_pairs_v<NC, false, PHI>(mine[p], px, py, pz, tab, kd, tx, ty, tz, tp);
                continue;
            }
            auto near = [&](unsigned w, auto q_c) {
                constexpr int q = decltype(q_c)::value;
                while (w) {
                    const int p = __builtin_clz(w);
                    w ^= 0x80000000u >> p;
                    table_pairs_v<1, false, PHI>(mine[p], px + q, py + q, pz + q, tab, kc, tx + q,
                                                 ty + q, tz + q, tp + q);
                }
            };
            near(m[0], std::integral_constant<int, 0>{});
            near(m[1], std::integral_constant<int, 1>{});
            if constexpr (NC > 2) {
                near(m[2], std::integral_constant<int, 2>{});
                near(m[3], std::integral_constant<int, 3>{});
            }
        }

        to_total();
        __syncthreads();  // then the waves' shares in order
        for (int k = tid; k < C * n_i; k += 64 * W) {
            const int c = k / n_i, i = k - c * n_i;
            float r = 0.f;
            for (int w = 0; w < W; ++w) r += ((const float *)(sums + w * NI + i))[c];
            (c == 0 ? a.ax : c == 1 ? a.ay : c == 2 ? a.az : a.phi)[i0 + i] = r;
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
    {"near", 0, 64, nullptr, nullptr, nullptr, nullptr},
};
#undef PGH_TABLE_VARIANT
constexpr int kRowsVariant = 5, kNearVariant = 6;
constexpr int kNumTableVariants = sizeof(kTableVariants) / sizeof(kTableVariants[0]);

bool is_phi(const TableArgs &a) { return a.phi && a.ptable; }

size_t table_lds_bytes(const TableArgs &a)
{
    return (is_phi(a) ? sizeof(float4) : sizeof(float2)) << (a.E + a.F);
}

// The built-in choice, made per launch (kAutoVariant, not a selectable
// variant).  Times: T16, k_table_allpairs against the kernel taken, first in a
// box of 21 cutoffs, then with every pair inside:
//   * the rows kernel up to 10^8 pairs, where k_table_allpairs' workgroup per 256
//     i-particles leaves CUs idle (N = 5500: 42 -> 15 us, 42 -> 18; 8192: 29.6 ->
//     24.9, 30.0 -> 29.0; 5000 x 20000 54 -> 34, 55 -> 44), and for few
//     i-particles;
//   * k_table_near above, for at least 8192 x 4096 (N = 10240 50 -> 21, 50 -> 63;
//     16384 88 -> 28, 94 -> 98); from as many i-particles on as give each CU more
//     than one chunk, or 4 x 10^8 pairs, every pair inside would cost it far more
//     than the 8 us of k_table_density and the launches that return at once
//     (N = 20000 144 -> 59, 155 -> 237), and k_table_density picks k_table_near
//     or k_table_allpairs on the device (20000 144 -> 68, 155 -> 152; 32768 300
//     -> 88, 325 -> 331; 65536 1097 -> 292, 1196 -> 1203);
//   * k_table_allpairs otherwise (3000 x 60000: 67 us, both others 63 and 78).
constexpr int kAutoVariant = kNumTableVariants;

enum class AutoKernel { rows, near, allpairs };

AutoKernel auto_kernel(int ni, int nj)
{
    if (nj < 256 && ni >= 16384) return AutoKernel::allpairs;
    if ((double)ni * nj <= 1.0e8 || ni < 1024) return AutoKernel::rows;
    return ni >= 8192 && nj >= 4096 ? AutoKernel::near : AutoKernel::allpairs;
}

bool auto_decides(int ni, int nj, int num_cu)
{
    return ni > 64 * num_cu || (double)ni * nj >= 4.0e8;
}

// k_table_allpairs' variant: two i-particles per lane once these fill the CUs
int allpairs_variant(int ni, int num_cu)
{
    return ((long)ni + 127) / 128 >= 4L * num_cu ? 1 : 0;
}

int rows_split(const TableArgs &a, size_t part_cap)
{
    return (int)std::max(1L, std::min((long)rows_shape(a.ni, a.nj).shares,
                                      (long)(part_cap / (4 * (size_t)std::max(a.ni, 1)))));
}

}  // namespace

int table_allpairs_variants() { return kNumTableVariants; }

const char *table_allpairs_variant_name(int v)
{
    return (v >= 0 && v < kNumTableVariants) ? kTableVariants[v].name : nullptr;
}

int table_allpairs_default() { return kAutoVariant; }

int table_allpairs_split(const TableArgs &a, int variant, int num_cu, size_t part_cap)
{
    if (variant == kAutoVariant) {
        const AutoKernel k = auto_kernel(a.ni, a.nj);
        if (k == AutoKernel::rows) return rows_split(a, part_cap);
        if (k == AutoKernel::near && !auto_decides(a.ni, a.nj, num_cu)) return 1;
        variant = allpairs_variant(a.ni, num_cu);
    }
    if (variant == kNearVariant) return 1;
    if (variant == kRowsVariant) return rows_split(a, part_cap);
    const TableVariant &v = kTableVariants[variant];
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

template <int W>
TableKernel near_kernel(int nc, bool phi)
{
    if (nc == 4) return phi ? k_table_near<4, W, true> : k_table_near<4, W, false>;
    return phi ? k_table_near<2, W, true> : k_table_near<2, W, false>;
}

hipError_t launch_table_near(const TableArgs &a, int num_cu, hipStream_t s)
{
    const bool phi = is_phi(a);
    // four columns share a record's terms; two give small sets more waves, and
    // are what LDS has room for beside the largest tables
    const size_t table = std::max(sizeof(float4), table_lds_bytes(a));
    const int nc = a.ni >= 32768 && table <= 65536 ? 4 : 2;
    // eight waves and two workgroups to a CU, or sixteen where a large table
    // (or few chunks) leaves room for one
    const int groups = (a.ni + 32 * nc - 1) / (32 * nc);
    const int w = table > 32768 || groups <= num_cu ? 16 : 8;
    const size_t lds = table + (size_t)w * (64 + 32 * nc) * sizeof(float4);
    const TableKernel kern = w == 16 ? near_kernel<16>(nc, phi) : near_kernel<8>(nc, phi);
    hipError_t e = allow_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    // a large table is copied once per CU
    const int blocks = table > 16384 ? std::min(groups, num_cu * (w == 16 ? 1 : 2)) : groups;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * w), lds, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_table_allpairs(const TableArgs &a0, int variant, int S, int num_cu,
                                 hipStream_t s)
{
    if (a0.ni <= 0) return hipSuccess;
    TableArgs a = a0;
    const bool phi = is_phi(a);
    S = std::max(1, S);
    int *const dense = a.dense;
    a.dense = nullptr;
    if (variant == kAutoVariant) {
        const AutoKernel k = auto_kernel(a.ni, a.nj);
        variant = k == AutoKernel::rows   ? kRowsVariant
                  : k == AutoKernel::near ? kNearVariant
                                          : allpairs_variant(a.ni, num_cu);
        if (k == AutoKernel::near && auto_decides(a.ni, a.nj, num_cu)) {
            a.dense = dense;
            hipLaunchKernelGGL(phi ? k_table_density<true> : k_table_density<false>, dim3(1),
                               dim3(1024), 0, s, a, dense);
            hipError_t e = hipGetLastError();
            if (e == hipSuccess) e = launch_table_near(a, num_cu, s);
            if (e != hipSuccess) return e;
            variant = allpairs_variant(a.ni, num_cu);
        }
    }
    if (variant == kNearVariant) return launch_table_near(a, num_cu, s);
    if (variant == kRowsVariant) return launch_table_rows(a, S, num_cu, s);
    const TableVariant &v = kTableVariants[variant];
    const size_t lds = table_lds_bytes(a);
    const bool wide = lds > kWideTableBytes;
    const int nt = wide ? kWideNT : 256, jt = wide ? kWideNT : v.jt;
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
    return launch_combine_split(a.ni, S, a.part, a0.ax, a0.ay, a0.az, phi ? a0.phi : nullptr, s,
                                a.dense);
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
