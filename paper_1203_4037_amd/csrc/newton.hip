// All-pairs Newton force and potential on gfx950: Eq. (newton_force) of
// Sec. 3 with the loop of Sec. 3.3 (difference, softened square distance,
// inverse square root, m/r into the potential, m/r^3 times the difference
// into the acceleration).
//
// Mapping.  A workgroup of 256 lanes (four wave64) owns 256*KI i-particles,
// KI per lane, held in VGPRs for the whole launch.  The j-particles stream
// through LDS in tiles of JT (x, y, z, m) records: every lane loads JT/256
// records with one coalesced 16-byte load each, the tile is written to LDS,
// and the inner loop reads record jj with one ds_read_b128 at a lane-uniform
// address, which the LDS broadcasts to all 64 lanes without bank conflicts.
// Tiles are double-buffered: the global loads for tile t+1 are in flight
// while tile t is consumed, and one barrier per tile separates the phases.
//
// Arithmetic per pair (KI independent chains per lane):
//   3 sub, 3 fma (|d|^2 + eps^2), v_rsq_f32, then either
//   refine=0: m*y, y*y, (m y)*(y y)                       3 mul
//   refine=1: one Newton-Raphson step folded into the products:
//             y2 = y*y, t = q*y2 - 3, u = y*t (= -2 rho), mr = (-m/2)*u
//             (= m rho), u2 = u*u, mr3 = mr*u2 (= 4 m rho^3); the 4 is
//             removed by an exact scale of the sums at the end   6 ops
//   phi -= m rho (1 op), a += mr3 * d (3 fma).
// The mass in LDS is pre-scaled by -1/2 when refining, so the step costs
// three VALU ops per pair, not four.  The "rcp" variants take rho^2 = 1/q
// from v_rcp_f32 instead of squaring (mr3 = m rho * rcp(q)): the
// transcendental unit issues beside the VALU, so this trades one VALU op
// per pair for a second transcendental.
//
// The "rows" kernel turns the mapping round: a workgroup holds TI i-particles
// as wave-uniform values, its lanes take j-particles (k_newton_rows below).
//
// Accuracy.  Sums over a tile are formed in fresh registers and added to
// the running totals once per tile, so FP32 rounding grows with
// JT + nj/JT rather than nj.  In the rows kernel a lane's sum has the
// nj / (NT S) terms of its own records (S shares), and the NT lanes' sums meet in
// a tree: 4096 + 10 steps for 10^6 j-particles.
#include <algorithm>

#include "newton_pair.h"
#include "pgh_internal.h"
#include "rows.h"

namespace pgh {

__global__ void __launch_bounds__(256) k_pack_j(int n, const float *__restrict__ x,
                                                const float *__restrict__ y,
                                                const float *__restrict__ z,
                                                const float *__restrict__ m,
                                                float4 *__restrict__ dst)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = make_float4(x[i], y[i], z[i], m[i]);
}

hipError_t launch_pack_j(int n, const float *x, const float *y, const float *z, const float *m,
                         float4 *dst, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_j, dim3((n + 255) / 256), dim3(256), 0, s, n, x, y, z, m, dst);
    return hipGetLastError();
}

// Adds the S partial sums [S][4][n] of a j-split launch in split order
// (ax..az and phi each optional): blockIdx.y is the component, and eight
// shares' loads are in flight at once, so S shares cost S / 8 memory
// latencies (one thread per particle with its four loads a share waited for in
// turn took 16.6 us for 27 shares of 20011 particles).
__global__ void __launch_bounds__(256) k_combine_split(int n, int S, const float *__restrict__ part,
                                                       float *ax, float *ay, float *az, float *phi,
                                                       const int *dense, const int *same)
{
    if (dense && *dense == 0) return;
    if (same && same_set(same)) return;
    const int c = blockIdx.y;
    float *const out = c == 0 ? ax : c == 1 ? ay : c == 2 ? az : phi;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n || !out) return;
    const float *p = part + (size_t)c * n + i;
    const size_t step = (size_t)4 * n;
    float sum = 0.f;
    int s = 0;
    for (; s + 8 <= S; s += 8) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = p[(size_t)(s + k) * step];
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += v[k];
    }
    for (; s < S; ++s) sum += p[(size_t)s * step];
    out[i] = sum;
}

hipError_t launch_combine_split(int n, int S, const float *part, float *ax, float *ay, float *az,
                                float *phi, hipStream_t s, const int *dense,
                                const int *same)
{
    if (n <= 0 || S <= 1) return hipSuccess;
    hipLaunchKernelGGL(k_combine_split, dim3((n + 255) / 256, phi ? 4 : 3), dim3(256), 0, s, n, S,
                       part, ax, ay, az, phi, dense, same);
    return hipGetLastError();
}

int split_count(int ni, int nj, int ki, int jt, int target_waves, size_t part_cap)
{
    const long waves = ((long)ni + 64L * ki - 1) / (64L * ki);
    long S = (target_waves + waves - 1) / waves;
    // at least two tiles per share, or one of 64 records (small i-sets,
    // whose waves come from the split alone)
    S = std::min(S, std::max(1L, (long)nj / (jt > 64 ? 2L * jt : (long)jt)));
    if (ni > 0) S = std::min(S, (long)(part_cap / (4 * (size_t)ni)));
    return (int)std::max(1L, S);
}

__global__ void __launch_bounds__(256) k_fill_zero(int n, float *a, float *b, float *c, float *d)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        if (a) a[i] = 0.f;
        if (b) b[i] = 0.f;
        if (c) c[i] = 0.f;
        if (d) d[i] = 0.f;
    }
}

hipError_t launch_fill_zero(int n, float *a, float *b, float *c, float *d, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_zero, dim3((n + 255) / 256), dim3(256), 0, s, n, a, b, c, d);
    return hipGetLastError();
}

namespace {

template <int KI, int JT, int U, bool RCP, bool REFINE, bool GUARD, bool PHI>
__global__ void __launch_bounds__(256) k_newton_allpairs(NewtonArgs a)
{
    if (a.same && same_set(a.same)) return;
    static_assert(JT % 256 == 0 || JT == 64, "a tile is 64 records or whole workgroup rounds");
    constexpr int PER = JT >= 256 ? JT / 256 : 1;  // records each thread loads per tile
    __shared__ float4 tile[2][JT];

    const int tid = threadIdx.x;
    const int ibase = blockIdx.x * (256 * KI) + tid;
    const float mscale = REFINE ? -0.5f : 1.0f;

    float px[KI], py[KI], pz[KI], pe[KI];
    float tx[KI], ty[KI], tz[KI], tp[KI];
#pragma unroll
    for (int k = 0; k < KI; ++k) {
        int i = ibase + k * 256;
        i = i < a.ni ? i : a.ni - 1;
        px[k] = a.xi[i];
        py[k] = a.yi[i];
        pz[k] = a.zi[i];
        pe[k] = a.eps2i ? a.eps2i[i] : a.eps2_all;
        tx[k] = ty[k] = tz[k] = tp[k] = 0.f;
    }

    // this workgroup's share of the j-particles (blockIdx.y splits them)
    const int jbase = blockIdx.y * a.jchunk;
    const int nj = max(0, min(a.jchunk, a.nj - jbase));
    const float4 *__restrict__ jm = a.jmem + jbase;
    const int ntiles = (nj + JT - 1) / JT;
    float4 pre[PER];

    // (a 64-record tile is loaded by the first wave of the workgroup)
    auto load_tile = [&](int t) {
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int j = t * JT + r * 256 + tid;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((JT >= 256 || tid < JT) && j < nj) v = jm[j];
            pre[r] = v;  // not touched until stored, so the load stays in flight
        }
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            float4 v = pre[r];
            v.w *= mscale;
            if (JT >= 256 || tid < JT) tile[buf][r * 256 + tid] = v;
        }
    };

    load_tile(0);
    // Every global load so far (i-particles, first tile) must land before the
    // tile loop; waiting here, on a path every thread takes, keeps the
    // compiler from waiting on them (and on the next tile's prefetch queued
    // behind them) inside the inner loop.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
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

        if (cnt == JT) {
#pragma unroll U
            for (int jj = 0; jj < JT; ++jj) {
                const float4 p = tile[cur][jj];
#pragma unroll
                for (int k = 0; k < KI; ++k)
                    newton_pair<REFINE, GUARD, PHI, RCP>(p, px[k], py[k], pz[k], pe[k], sx[k], sy[k],
                                                    sz[k], sp[k]);
            }
        } else {
#pragma unroll 2
            for (int jj = 0; jj < cnt; ++jj) {
                const float4 p = tile[cur][jj];
#pragma unroll
                for (int k = 0; k < KI; ++k)
                    newton_pair<REFINE, GUARD, PHI, RCP>(p, px[k], py[k], pz[k], pe[k], sx[k], sy[k],
                                                    sz[k], sp[k]);
            }
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

    const float ascale = (REFINE && !RCP) ? 0.25f : 1.0f;
    // one j-share: write the outputs; several: partial sums for k_combine_split
    float *ox = a.ax, *oy = a.ay, *oz = a.az, *op = a.phi;
    if (gridDim.y > 1) {
        ox = a.part + (size_t)blockIdx.y * 4 * a.ni;
        oy = ox + a.ni;
        oz = oy + a.ni;
        op = oz + a.ni;
    }
#pragma unroll
    for (int k = 0; k < KI; ++k) {
        const int i = ibase + k * 256;
        if (i < a.ni) {
            ox[i] = tx[k] * ascale;
            oy[i] = ty[k] * ascale;
            oz[i] = tz[k] * ascale;
            if (PHI) op[i] = tp[k];
        }
    }
}

// The "rows" kernel: TI i-particles per workgroup, the same for all its lanes
// (held in SGPRs), and the j-particles dealt over its NT lanes: each lane
// loads its own j-record straight from global memory (coalesced, two records
// ahead) and uses it for TI pairs.  No LDS traffic, no barrier and no partial
// sums in memory: the lanes' sums meet once, at the end.
//
// Bound by FP32 issue like k_newton_allpairs (the SGPR operand of the three
// subtractions costs nothing measurable beside VGPR copies).  The point of
// the mapping is that ni / TI workgroups fill the chip where ni / 256
// cannot: the other kernel then takes its waves from the j-split, whose
// partial sums cost a second launch and memory traffic, and whose shares of
// whole 256-record tiles leave the last round of workgroups partly idle.
// Measured, whole call (pack, force, combine) before and after:
// N = 1024 14.9 -> 5 us of kernels, 256 x 4096 25.4 -> 5.5 us, 4096 22.2 -> 8
// us of force, 20011 174 -> 128 us, 65536 1.29 -> 1.27 ms, 131072 5.34 ->
// 5.07 ms.  The record two steps ahead matters: with the load of the next
// record waited for at once, N = 65536 took 1.63 ms.
template <int TI, int NT, bool REFINE, bool GUARD, bool PHI>
__global__ void __launch_bounds__(NT) k_newton_rows(NewtonArgs a)
{
    if (a.same && same_set(a.same)) return;
    constexpr int V = 4 * TI;   // sums per workgroup
    constexpr int W = NT / 64;
    __shared__ float red[W][V];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * TI;
    const float mscale = REFINE ? -0.5f : 1.0f;

    float px[TI], py[TI], pz[TI], pe[TI], s[TI][4];
#pragma unroll
    for (int k = 0; k < TI; ++k) {
        const int i = min(i0 + k, a.ni - 1);
        px[k] = a.xi[i];
        py[k] = a.yi[i];
        pz[k] = a.zi[i];
        pe[k] = a.eps2i ? a.eps2i[i] : a.eps2_all;
        s[k][0] = s[k][1] = s[k][2] = s[k][3] = 0.f;
    }
    auto pairs = [&](float4 p) {
        p.w *= mscale;
#pragma unroll
        for (int k = 0; k < TI; ++k)
            newton_pair<REFINE, GUARD, PHI, false>(p, px[k], py[k], pz[k], pe[k], s[k][0], s[k][1],
                                                   s[k][2], s[k][3]);
    };

    // this workgroup's share of the j-particles (blockIdx.y splits them; no
    // share is empty)
    const int jbase = blockIdx.y * a.jchunk;
    const int nj = min(a.jchunk, a.nj - jbase);
    const float4 *__restrict__ jm = a.jmem + jbase;
    const int full = nj / NT;  // steps in which every lane has a record
    // unconditional loads (past the end the last record, not used), so that
    // no branch makes the compiler wait for one before the next is issued
    auto load = [&](int t) { return jm[min(t * NT + tid, nj - 1)]; };
    float4 p0 = load(0), p1 = load(1);
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
        // exactly zero where its own pairs are finite (a record put far away
        // would not: its |d|^2 may overflow where no pair's does)
        if (t * NT + tid >= nj) p0.w = 0.f;
        pairs(p0);
    }

#pragma unroll
    for (int k = 0; k < TI; ++k) {
        // rows 0 .. 3 of the wave now hold the sums x, z, y, phi
        const float v =
            row_sum(fold_rows(fold_halves(s[k][0], s[k][1]), fold_halves(s[k][2], s[k][3])));
        const int row = lane >> 4, c = ((row & 1) << 1) | (row >> 1);
        if ((lane & 15) == 0) red[wave][4 * k + c] = v;
    }
    __syncthreads();
    if (tid < V) {
        float r = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) r += red[w][tid];
        const int c = tid & 3, i = i0 + (tid >> 2);
        if (REFINE && c < 3) r *= 0.25f;
        if (i < a.ni) {
            if (gridDim.y > 1)
                a.part[((size_t)blockIdx.y * 4 + c) * a.ni + i] = r;
            else if (c < 3 || PHI)
                (c == 0 ? a.ax : c == 1 ? a.ay : c == 2 ? a.az : a.phi)[i] = r;
        }
    }
}

using NewtonKernel = void (*)(NewtonArgs);

template <int KI, int JT, int U, bool RCP>
struct NewtonSet {
    static NewtonKernel get(bool refine, bool guard, bool phi)
    {
        const int sel = (refine ? 4 : 0) | (guard ? 2 : 0) | (phi ? 1 : 0);
        switch (sel) {
            case 0: return k_newton_allpairs<KI, JT, U, RCP, false, false, false>;
            case 1: return k_newton_allpairs<KI, JT, U, RCP, false, false, true>;
            case 2: return k_newton_allpairs<KI, JT, U, RCP, false, true, false>;
            case 3: return k_newton_allpairs<KI, JT, U, RCP, false, true, true>;
            case 4: return k_newton_allpairs<KI, JT, U, RCP, true, false, false>;
            case 5: return k_newton_allpairs<KI, JT, U, RCP, true, false, true>;
            case 6: return k_newton_allpairs<KI, JT, U, RCP, true, true, false>;
            default: return k_newton_allpairs<KI, JT, U, RCP, true, true, true>;
        }
    }
};

template <int TI, int NT>
NewtonKernel rows_kernel_t(bool refine, bool guard, bool phi)
{
    const int sel = (refine ? 4 : 0) | (guard ? 2 : 0) | (phi ? 1 : 0);
    switch (sel) {
        case 0: return k_newton_rows<TI, NT, false, false, false>;
        case 1: return k_newton_rows<TI, NT, false, false, true>;
        case 2: return k_newton_rows<TI, NT, false, true, false>;
        case 3: return k_newton_rows<TI, NT, false, true, true>;
        case 4: return k_newton_rows<TI, NT, true, false, false>;
        case 5: return k_newton_rows<TI, NT, true, false, true>;
        case 6: return k_newton_rows<TI, NT, true, true, false>;
        default: return k_newton_rows<TI, NT, true, true, true>;
    }
}

NewtonKernel rows_kernel(const RowsShape &r, bool refine, bool guard, bool phi)
{
    if (r.nt == 1024)
        return (r.ti == 1   ? &rows_kernel_t<1, 1024>
                : r.ti == 2 ? &rows_kernel_t<2, 1024>
                            : &rows_kernel_t<4, 1024>)(refine, guard, phi);
    return (r.ti == 1   ? &rows_kernel_t<1, 256>
            : r.ti == 2 ? &rows_kernel_t<2, 256>
            : r.ti == 4 ? &rows_kernel_t<4, 256>
                        : &rows_kernel_t<8, 256>)(refine, guard, phi);
}

// ki = 0: the rows kernel, whose shape follows from the sizes (rows_shape).
struct NewtonVariant {
    const char *name;
    int ki, jt;
    NewtonKernel (*get)(bool, bool, bool);
};

const NewtonVariant kNewtonVariants[] = {
    {"ki=1 jt=256 u=8", 1, 256, &NewtonSet<1, 256, 8, false>::get},
    {"ki=1 jt=64 u=8", 1, 64, &NewtonSet<1, 64, 8, false>::get},
    {"ki=2 jt=256 u=4", 2, 256, &NewtonSet<2, 256, 4, false>::get},
    {"ki=4 jt=256 u=2", 4, 256, &NewtonSet<4, 256, 2, false>::get},
    {"ki=2 jt=512 u=8", 2, 512, &NewtonSet<2, 512, 8, false>::get},
    {"ki=1 jt=256 u=8 rcp", 1, 256, &NewtonSet<1, 256, 8, true>::get},
    {"ki=2 jt=256 u=4 rcp", 2, 256, &NewtonSet<2, 256, 4, true>::get},
    {"ki=4 jt=256 u=2 rcp", 4, 256, &NewtonSet<4, 256, 2, true>::get},
    {"rows", 0, 64, nullptr},
    // each pair once (newton_mutual.hip) where the i-particles are the
    // j-particles, else the rows kernel
    {"mutual", 0, 64, nullptr},
};
constexpr int kRowsVariant = 8, kMutualVariant = 9;
constexpr int kNumNewtonVariants = sizeof(kNewtonVariants) / sizeof(kNewtonVariants[0]);

}  // namespace

int newton_allpairs_variants() { return kNumNewtonVariants; }

const char *newton_allpairs_variant_name(int v)
{
    return (v >= 0 && v < kNumNewtonVariants) ? kNewtonVariants[v].name : nullptr;
}

int newton_allpairs_default(int ni, int nj, int num_cu)
{
    // Lists too short to give each lane of a workgroup a record: one
    // i-particle per lane (100000 x 100: the rows kernel 20 us, this 17 us).
    if (nj < 256 && ni >= 16384) return 0;
    // From 196608 i-particles up, four per lane over LDS tiles, when the
    // workgroups of its j-split spread evenly over the CUs (N = 262144: 19.1
    // against 19.9 ms with rows, 230000 15.1 against 15.4, 10^6 292 against
    // 308), which loses more than that otherwise (8 or 9 workgroups a CU at N =
    // 300000: 28.3 against 26.1 ms; 400000: 50.5 against 47.1).  Below, rows
    // (131072: 5.02 against 5.08 ms, 65536: 1.27 against 1.29 with one per
    // lane, and more the smaller the set).  pgh_autotune confirms or replaces
    // the choice for a given workload.
    if (ni < 3 << 16) return kRowsVariant;
    const long groups = ((ni + 1023L) / 1024) * newton_allpairs_split(ni, nj, 3, (size_t)64 << 20);
    const long per_cu = (groups + num_cu - 1) / num_cu;
    return 20 * groups >= 19 * per_cu * num_cu ? 3 : kRowsVariant;
}

int newton_allpairs_rows() { return kRowsVariant; }
int newton_allpairs_mutual() { return kMutualVariant; }

int newton_allpairs_split(int ni, int nj, int variant, size_t part_cap)
{
    const NewtonVariant &v = kNewtonVariants[variant];
    if (v.ki == 0)
        return (int)std::max(1L, std::min((long)rows_shape(ni, nj).shares,
                                          (long)(part_cap / (4 * (size_t)std::max(ni, 1)))));
    return split_count(ni, nj, v.ki, v.jt, kSplitTargetWaves, part_cap);
}

hipError_t launch_newton_allpairs(const NewtonArgs &a0, int variant, bool refine, bool guard,
                                  int S, hipStream_t s)
{
    if (a0.ni <= 0) return hipSuccess;
    const NewtonVariant &v = kNewtonVariants[variant];
    NewtonArgs a = a0;
    S = std::max(1, S);
    a.jchunk = (int)(((long)a.nj + (long)S * v.jt - 1) / ((long)S * v.jt) * v.jt);
    S = std::max(1, (a.nj + a.jchunk - 1) / a.jchunk);
    if (v.ki == 0) {
        const RowsShape r = rows_shape(a.ni, a.nj);
        hipLaunchKernelGGL(rows_kernel(r, refine, guard, a.phi != nullptr),
                           dim3((a.ni + r.ti - 1) / r.ti, S), dim3(r.nt), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || S == 1) return e;
        return launch_combine_split(a.ni, S, a.part, a0.ax, a0.ay, a0.az, a0.phi, s, nullptr,
                                    a.same);
    }
    const int per_block = 256 * v.ki;
    const dim3 grid((a.ni + per_block - 1) / per_block, S);
    hipLaunchKernelGGL(v.get(refine, guard, a.phi != nullptr), grid, dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    return launch_combine_split(a.ni, S, a.part, a0.ax, a0.ay, a0.az, a0.phi, s, nullptr,
                                    a.same);
}

}  // namespace pgh
