// The all-pairs Newton force of a set on itself, each pair evaluated once for
// both of its particles: the difference, the softened square distance and the
// inverse square root serve k and l alike, 17 FP32 operations and one root per
// two terms of the sum instead of 2 x 13 and two.
//
// Mapping.  The particles are cut into blocks of B = 64 x 12 x 4.  A workgroup of
// four waves takes the l-particles of one block, twelve per lane with their sums
// in registers, and a chunk of k-particles from the same block or a later one,
// wave-uniform values (SGPRs) like the i-particles of the rows kernel.  For each
// k every lane sums its twelve terms; these meet across the lanes by permlane swaps
// and DPP adds, once per k and wave, and across the waves in LDS, once per 32 k.
// A chunk of the block itself is evaluated for the l-particles only, which then
// meet every particle of their block, themselves included.
//
// The l-sums of a chunk go to lsum[block][chunk][4][B], the k-sums of a block to
// ksum[block][4][n], and k_mutual_combine adds a particle's sums in order.  A
// strip of blocks at a time where all would not fit the scratch memory.
//
// Bound by FP32 issue: 21.4 VALU instructions per pair with the potential (counted
// at N = 262144, where k_newton_allpairs issues 28.4 for the pair's two terms), one
// every 3.3 cycles of a SIMD with the three waves that 53 KB of LDS leave room for
// (3.1 there, with eight); 3 of them are the meetings of the lanes, which is what
// twelve particles per lane are for (with eight 16.6 ms at N = 262144, with four
// 19.1, with sixteen, too few waves, 17.2).  No branch inside the k-loop: past one the compiler moves
// the l-sums of four k, and spills their factors (113 ms).  Whole call, each
// pair twice (rows, ki = 4) and here: N = 262144 19.0 -> 15.7 ms, 131072 5.0 ->
// 4.0, 65536 1.27 -> 1.07, 40000 0.49 -> 0.46.
//
// Whether the i-particles are the j-particles is found by comparing every
// coordinate on the device (k_same_set): these kernels return at once where they
// differ, the kernel launched after them where they do not.
#include <algorithm>

#include "newton_pair.h"
#include "pgh_internal.h"
#include "rows.h"
#include "split.h"

namespace pgh {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// memory that no kernel of the launch writes: read by scalar loads where the
// address is wave-uniform
typedef const __attribute__((address_space(4))) f32x4 *ConstRecords;

constexpr float kFarAway = 1.0e10f;
constexpr int kLanes = 12;  // l-particles per lane
constexpr int kWaves = 4;   // waves per workgroup
constexpr int kBwdLanes = 8;  // l-particles per lane of the adjoint

__global__ void __launch_bounds__(1024) k_same_set(int n, const unsigned *__restrict__ x,
                                                   const unsigned *__restrict__ y,
                                                   const unsigned *__restrict__ z,
                                                   const uint4 *__restrict__ jmem, int *same)
{
    __shared__ int differ;
    if (threadIdx.x == 0) differ = 0;
    __syncthreads();
    bool d = false;
    for (int i = blockIdx.x * 1024 + threadIdx.x; i < n; i += gridDim.x * 1024) {
        const uint4 p = jmem[i];
        d |= p.x != x[i] || p.y != y[i] || p.z != z[i];
    }
    if (d) differ = 1;
    __syncthreads();
    if (threadIdx.x == 0) same[blockIdx.x] = !differ;
}

struct MutualArgs {
    int n;
    const float4 *jmem;
    float eps2;
    int block0;  // the strip's first block
    int chunk;   // k-particles per chunk, a divisor of the block, so that none
                 // holds particles of two blocks, and a multiple of FRESH
    int chunks;  // chunks of the strip's first block
    float *lsum, *ksum;
    const int *same;
};

// rho, or -2 rho with the Newton-Raphson step (the masses then carry -1/2)
template <bool REFINE, bool GUARD>
__device__ __forceinline__ float mutual_rho(float q)
{
    float y = __builtin_amdgcn_rsqf(q);
    if (GUARD) y = q > 0.f ? y : 0.f;
    if (REFINE) y *= __builtin_fmaf(q, y * y, -3.0f);
    return y;
}

template <bool REFINE, bool GUARD, bool PHI>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3)))
k_newton_mutual(MutualArgs a)
{
    if (a.same && !same_set(a.same)) return;
    constexpr int KL = kLanes, W = kWaves;
    constexpr int B = 64 * KL * W;
    constexpr int G = 32;      // k-particles between two meetings of the waves
    constexpr int FRESH = 64;  // terms of an l-sum before it is added to its total
    constexpr int C = PHI ? 4 : 3;
    __shared__ float red[2][W][4 * G];
    __shared__ float total[KL * 4][64 * W];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int block = a.block0 + blockIdx.y;
    const int k0 = block * B + blockIdx.x * a.chunk;
    if (k0 >= a.n) return;
    const int k1 = min(k0 + a.chunk, a.n);
    const float mscale = REFINE ? -0.5f : 1.0f, ascale = REFINE ? 0.25f : 1.0f;

    const int l0 = block * B + wave * 64 * KL + lane;
    float lx[KL], ly[KL], lz[KL], lm[KL], s[KL][4];
#pragma unroll
    for (int r = 0; r < KL; ++r) {
        const int l = l0 + 64 * r;
        float4 p = a.jmem[min(l, a.n - 1)];
        if (l >= a.n) p = make_float4(kFarAway, kFarAway, kFarAway, 0.f);
        lx[r] = p.x, ly[r] = p.y, lz[r] = p.z, lm[r] = p.w * mscale;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            s[r][c] = 0.f;
            if (c < C) total[4 * r + c][tid] = 0.f;
        }
    }
    auto to_totals = [&] {  // each lane's own words
#pragma unroll
        for (int r = 0; r < KL; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                total[4 * r + c][tid] += s[r][c];
                s[r][c] = 0.f;
            }
    };
    const ConstRecords rec = (ConstRecords)(unsigned long long)a.jmem;
    // past the end the last record again, its mass taken for zero
    auto load = [&](int k) { return rec[min(k, a.n - 1)]; };
    auto mass = [&](const f32x4 &p, int k) { return k < a.n ? p.w : 0.f; };
    constexpr int T = 4;  // records loaded ahead
    f32x4 next[T];
#pragma unroll
    for (int t = 0; t < T; ++t) next[t] = load(k0 + t);

    if (k0 < (block + 1) * B) {
        // of the block itself
        for (int g = k0; g < k1; g += FRESH) {
#pragma unroll 1
            for (int k = g; k < min(g + FRESH, k1); k += T) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const f32x4 p = next[t];
                    next[t] = load(k + T + t);
                    const float4 c = make_float4(p.x, p.y, p.z, mass(p, k + t) * mscale);
#pragma unroll
                    for (int r = 0; r < KL; ++r)
                        newton_pair<REFINE, GUARD, PHI, false>(c, lx[r], ly[r], lz[r], a.eps2,
                                                               s[r][0], s[r][1], s[r][2], s[r][3]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            to_totals();
        }
    } else {
        const int row = lane >> 4, of_row = ((row & 1) << 1) | (row >> 1);
        int buf = 0;
        for (int g = k0; g < k1; g += G, buf ^= 1) {
#pragma unroll 1
            for (int kk = 0; kk < G; kk += T) {
                float f[T][4];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const f32x4 p = next[t];
                    next[t] = load(g + kk + T + t);
                    const float km = mass(p, g + kk + t) * mscale;
                    float fx = 0.f, fy = 0.f, fz = 0.f, fp = 0.f;
#pragma unroll
                    for (int r = 0; r < KL; ++r) {
                        const float dx = p.x - lx[r], dy = p.y - ly[r], dz = p.z - lz[r];
                        float q = __builtin_fmaf(dx, dx, a.eps2);
                        q = __builtin_fmaf(dy, dy, q);
                        q = __builtin_fmaf(dz, dz, q);
                        const float rho = mutual_rho<REFINE, GUARD>(q), rho2 = rho * rho;
                        // (m rho) rho^2: rho^3 alone leaves the range of
                        // FP32 for coordinates that m rho^3 doesn't
                        const float kr = km * rho, lr = lm[r] * rho;
                        const float wk = kr * rho2, wl = lr * rho2;
                        s[r][0] = __builtin_fmaf(wk, dx, s[r][0]);
                        s[r][1] = __builtin_fmaf(wk, dy, s[r][1]);
                        s[r][2] = __builtin_fmaf(wk, dz, s[r][2]);
                        fx = __builtin_fmaf(wl, dx, fx);
                        fy = __builtin_fmaf(wl, dy, fy);
                        fz = __builtin_fmaf(wl, dz, fz);
                        if (PHI) {
                            s[r][3] -= kr;
                            fp -= lr;
                        }
                    }
                    f[t][0] = fx, f[t][1] = fy, f[t][2] = fz, f[t][3] = fp;
                }
                // each component's sums of the four k meet in the rows of the
                // wave: row 0 holds k 0, row 1 k 2, row 2 k 1, row 3 k 3
                float mine = 0.f;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float v = row_sum(fold_rows(fold_halves(f[0][c], f[1][c]),
                                                      fold_halves(f[2][c], f[3][c])));
                    mine = (lane & 3) == c ? v : mine;
                }
                // (by every lane: a branch here would let the compiler move
                // the l-sums of all T steps past it, their factors kept)
                red[buf][wave][G * (lane & 3) + kk + of_row] = mine;
            }
            // two buffers in turn: one barrier a group is enough
            __syncthreads();
            if (tid < 4 * G) {
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < W; ++w) v += red[buf][w][tid];
                const int c = tid / G, k = g + tid % G;
                if (c < 3) v *= -ascale;
                if (k < k1 && c < C) a.ksum[((size_t)blockIdx.y * 4 + c) * a.n + k] = v;
            }
            if ((g - k0) % FRESH == FRESH - G) to_totals();
        }
        to_totals();
    }
    float *out = a.lsum + ((size_t)blockIdx.y * a.chunks + blockIdx.x) * 4 * B;
#pragma unroll
    for (int r = 0; r < KL; ++r) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            out[(size_t)c * B + (wave * KL + r) * 64 + lane] =
                total[4 * r + c][tid] * (c < 3 ? ascale : 1.f);
    }
}

// Component blockIdx.y of 256 particles: the k-sums of the strip's earlier
// blocks, then the l-sums of its own chunks, eight in flight.
__global__ void __launch_bounds__(256) k_mutual_combine(MutualArgs a, int block, int blocks,
                                                        float *ax, float *ay, float *az, float *phi)
{
    if (a.same && !same_set(a.same)) return;
    const int c = blockIdx.y;
    const int i = a.block0 * block + blockIdx.x * 256 + threadIdx.x;
    if (i >= a.n) return;
    float *o = c == 0 ? ax : c == 1 ? ay : c == 2 ? az : phi;
    float sum = a.block0 > 0 ? o[i] : 0.f;
    const int b = i / block - a.block0;  // of the strip
    auto add = [&](const float *p, size_t stride, int count) {
        for (int q0 = 0; q0 < count; q0 += 64) {
            float t = 0.f;  // fresh, as FP32 rounding grows with the terms of a sum
            for (int q = q0; q < min(q0 + 64, count); q += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(q + u, count - 1) * stride];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = q + u < count ? v[u] : 0.f;
                t += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            }
            sum += t;
        }
    };
    add(a.ksum + (size_t)c * a.n + i, (size_t)4 * a.n, min(b, blocks));
    if (b < blocks) {
        const int mine = (a.n - (a.block0 + b) * block + a.chunk - 1) / a.chunk;
        add(a.lsum + ((size_t)b * a.chunks * 4 + c) * block + i % block, (size_t)4 * block, mine);
    }
    o[i] = sum;
}

// The adjoint of the force of a set on itself (adjoint.hip), each pair once: for
// k, with d = r_l - r_k and e = m_l (w_k . d) - m_k (w_l . d),
//   A += rho^3 w_l,  B += m_l rho^3,  C += rho^5 e d,  G += rho^3 (w_l . d),
// and for l the same with k and l exchanged and -d, where e is the same.  34
// operations and one root against 2 x 26 and two.  The mapping is
// k_newton_mutual's, with eight l-particles per lane: 15 registers each.
// Bound by FP32 issue: 39.6 VALU instructions per pair counted at N = 65536, two
// thirds of them multiply-adds of three registers, one every 3.7 cycles of a
// SIMD at three waves: N = 65536 2402 -> 2052 us, 131072 9481 -> 8084, 50000 1485
// -> 1222.
template <bool REFINE>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3)))
k_newton_mutual_bwd(MutualArgs a)
{
    constexpr int KL = kBwdLanes, W = kWaves, B = 64 * KL * W, G = 32, T = 2;
    __shared__ float red[2][W][4 * G];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int block = a.block0 + blockIdx.y;
    const int k0 = block * B + blockIdx.x * a.chunk;
    if (k0 >= a.n) return;
    const int k1 = min(k0 + a.chunk, a.n);
    const int l0 = block * B + wave * 64 * KL + lane;
    float lx[KL], ly[KL], lz[KL], lm[KL], lu[KL], lv[KL], lw[KL], s[KL][8];
#pragma unroll
    for (int r = 0; r < KL; ++r) {
        const int l = l0 + 64 * r, at = min(l, a.n - 1);
        float4 p = a.jmem[2 * (size_t)at], w = a.jmem[2 * (size_t)at + 1];
        if (l >= a.n) {
            p = make_float4(kFarAway, kFarAway, kFarAway, 0.f);
            w = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        lx[r] = p.x, ly[r] = p.y, lz[r] = p.z, lm[r] = p.w;
        lu[r] = w.x, lv[r] = w.y, lw[r] = w.z;
#pragma unroll
        for (int c = 0; c < 8; ++c) s[r][c] = 0.f;
    }
    const ConstRecords rec = (ConstRecords)(unsigned long long)a.jmem;
    struct Record {
        f32x4 p, w;
    };
    // past the end the last record again, its mass and weight taken for zero
    auto load = [&](int k) {
        const size_t at = 2 * (size_t)min(k, a.n - 1);
        return Record{rec[at], rec[at + 1]};
    };
    auto keep = [&](float v, int k) { return k < a.n ? v : 0.f; };
    Record next[T];
#pragma unroll
    for (int t = 0; t < T; ++t) next[t] = load(k0 + t);

    // the pair's terms of l (and the factors of those of k)
    auto pair = [&](const Record &q, float km, float ku, float kv, float kw, int r, float dx,
                    float dy, float dz, float r1, float &r3, float &wld, float &f) {
        const float r2 = r1 * r1;
        r3 = r2 * r1;
        wld = lu[r] * dx;
        wld = __builtin_fmaf(lv[r], dy, wld);
        wld = __builtin_fmaf(lw[r], dz, wld);
        float wkd = ku * dx;
        wkd = __builtin_fmaf(kv, dy, wkd);
        wkd = __builtin_fmaf(kw, dz, wkd);
        f = r3 * r2 * __builtin_fmaf(lm[r], wkd, -km * wld);
        s[r][0] = __builtin_fmaf(r3, ku, s[r][0]);
        s[r][1] = __builtin_fmaf(r3, kv, s[r][1]);
        s[r][2] = __builtin_fmaf(r3, kw, s[r][2]);
        s[r][3] = __builtin_fmaf(km, r3, s[r][3]);
        s[r][4] = __builtin_fmaf(-f, dx, s[r][4]);
        s[r][5] = __builtin_fmaf(-f, dy, s[r][5]);
        s[r][6] = __builtin_fmaf(-f, dz, s[r][6]);
        s[r][7] = __builtin_fmaf(-r3, wkd, s[r][7]);
    };
    auto root = [&](float dx, float dy, float dz) {
        float q = __builtin_fmaf(dx, dx, a.eps2);
        q = __builtin_fmaf(dy, dy, q);
        q = __builtin_fmaf(dz, dz, q);
        const float y = __builtin_amdgcn_rsqf(q);
        return REFINE ? y * __builtin_fmaf(-0.5f * q, y * y, 1.5f) : y;
    };

    if (k0 < (block + 1) * B) {
        // of the block itself, for l only; l's own term is identically zero, but
        // would enter A and B as +-m w / eps^3 and cancel only to rounding, and
        // the last particle's copies past the end, zero mass and weight or not,
        // as 0 / eps^5, which leaves the range of FP32 for small softenings
#pragma unroll 1
        for (int k = k0; k < k1; k += T) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const Record q = next[t];
                next[t] = load(k + T + t);
                const float km = keep(q.p.w, k + t), ku = keep(q.w.x, k + t),
                            kv = keep(q.w.y, k + t), kw = keep(q.w.z, k + t);
#pragma unroll
                for (int r = 0; r < KL; ++r) {
                    const float dx = lx[r] - q.p.x, dy = ly[r] - q.p.y, dz = lz[r] - q.p.z;
                    float r1 = root(dx, dy, dz), r3, wld, f;
                    r1 = l0 + 64 * r == min(k + t, a.n - 1) ? 0.f : r1;
                    pair(q, km, ku, kv, kw, r, dx, dy, dz, r1, r3, wld, f);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
        const int row = lane >> 4, comp = ((row & 1) << 1) | (row >> 1);
        int buf = 0;
        for (int g = k0; g < k1; g += G, buf ^= 1) {
#pragma unroll 1
            for (int kk = 0; kk < G; kk += T) {
                float mine = 0.f;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const Record q = next[t];
                    const int k = g + kk + t;
                    next[t] = load(k + T);
                    const float km = keep(q.p.w, k), ku = keep(q.w.x, k), kv = keep(q.w.y, k),
                                kw = keep(q.w.z, k);
                    float A[3] = {0.f, 0.f, 0.f}, Bk = 0.f, C[3] = {0.f, 0.f, 0.f}, Gk = 0.f;
#pragma unroll
                    for (int r = 0; r < KL; ++r) {
                        const float dx = lx[r] - q.p.x, dy = ly[r] - q.p.y, dz = lz[r] - q.p.z;
                        float r3, wld, f;
                        pair(q, km, ku, kv, kw, r, dx, dy, dz, root(dx, dy, dz), r3, wld, f);
                        A[0] = __builtin_fmaf(r3, lu[r], A[0]);
                        A[1] = __builtin_fmaf(r3, lv[r], A[1]);
                        A[2] = __builtin_fmaf(r3, lw[r], A[2]);
                        Bk = __builtin_fmaf(lm[r], r3, Bk);
                        C[0] = __builtin_fmaf(f, dx, C[0]);
                        C[1] = __builtin_fmaf(f, dy, C[1]);
                        C[2] = __builtin_fmaf(f, dz, C[2]);
                        Gk = __builtin_fmaf(r3, wld, Gk);
                    }
                    const float gx = km * A[0] - ku * Bk + 3.f * C[0];
                    const float gy = km * A[1] - kv * Bk + 3.f * C[1];
                    const float gz = km * A[2] - kw * Bk + 3.f * C[2];
                    // rows 0 .. 3 of the wave now hold the sums x, z, y, m
                    const float v = row_sum(fold_rows(fold_halves(gx, gy), fold_halves(gz, -Gk)));
                    mine = (lane & 1) == t ? v : mine;
                }
                red[buf][wave][G * comp + kk + (lane & 1)] = mine;
            }
            __syncthreads();  // two buffers in turn
            if (tid < 4 * G) {
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < W; ++w) v += red[buf][w][tid];
                const int c = tid / G, k = g + tid % G;
                if (k < k1) a.ksum[((size_t)blockIdx.y * 4 + c) * a.n + k] = v;
            }
        }
    }
    float *out = a.lsum + ((size_t)blockIdx.y * a.chunks + blockIdx.x) * 4 * B + l0 - block * B;
#pragma unroll
    for (int r = 0; r < KL; ++r) {
        out[64 * r] = lm[r] * s[r][0] - lu[r] * s[r][3] + 3.f * s[r][4];
        out[B + 64 * r] = lm[r] * s[r][1] - lv[r] * s[r][3] + 3.f * s[r][5];
        out[2 * B + 64 * r] = lm[r] * s[r][2] - lw[r] * s[r][3] + 3.f * s[r][6];
        out[3 * B + 64 * r] = -s[r][7];
    }
}

using MutualKernel = void (*)(MutualArgs);

MutualKernel mutual_kernel(bool refine, bool guard, bool phi)
{
    const int sel = (refine ? 4 : 0) | (guard ? 2 : 0) | (phi ? 1 : 0);
    switch (sel) {
        case 0: return k_newton_mutual<false, false, false>;
        case 1: return k_newton_mutual<false, false, true>;
        case 2: return k_newton_mutual<false, true, false>;
        case 3: return k_newton_mutual<false, true, true>;
        case 4: return k_newton_mutual<true, false, false>;
        case 5: return k_newton_mutual<true, false, true>;
        case 6: return k_newton_mutual<true, true, false>;
        default: return k_newton_mutual<true, true, true>;
    }
}

}  // namespace

MutualShape mutual_shape(int n, size_t part_cap, bool adjoint)
{
    MutualShape m{};
    m.block = 64 * kWaves * (adjoint ? kBwdLanes : kLanes);
    m.blocks = (n + m.block - 1) / m.block;
    // Short chunks balance the workgroups over the CUs, long ones write fewer
    // sums.  us with chunks of 192, 384 and 768: N = 50000 651, 734, 901; 65536
    // 1067, 1136, 1255; 131072 4127, 3975, 4084; 262144 16205, 15975, 15668.
    m.chunk = n < 100000 ? 192 : n < 230000 ? 384 : 768;
    // the adjoint: 50000 1222 us with 128, 1308 with 256; 65536 2052, 2115;
    // 131072 8070, 8084 and twice the memory
    if (adjoint) m.chunk = n < 100000 ? 128 : 256;
    const size_t per_block = (size_t)4 * n + ((size_t)n + m.chunk) / m.chunk * 4 * m.block;
    m.strip = (int)std::min<size_t>(m.blocks, part_cap / per_block);
    m.floats = per_block * m.strip;
    return m;
}

hipError_t launch_same_set(int n, const float *x, const float *y, const float *z,
                           const float4 *jmem, int *same, hipStream_t s)
{
    hipLaunchKernelGGL(k_same_set, dim3(kSameWords), dim3(1024), 0, s, n, (const unsigned *)x,
                       (const unsigned *)y, (const unsigned *)z, (const uint4 *)jmem, same);
    return hipGetLastError();
}

namespace {

hipError_t launch_strips(MutualKernel kern, const MutualShape &m, MutualArgs a, float *ox,
                         float *oy, float *oz, float *o4, hipStream_t s)
{
    for (a.block0 = 0; a.block0 < m.blocks; a.block0 += m.strip) {
        const int blocks = std::min(m.strip, m.blocks - a.block0);
        const int first = a.block0 * m.block;
        a.chunks = (a.n - first + m.chunk - 1) / m.chunk;
        a.lsum = a.ksum + (size_t)4 * a.n * blocks;
        hipLaunchKernelGGL(kern, dim3(a.chunks, blocks), dim3(64 * kWaves), 0, s, a);
        hipLaunchKernelGGL(k_mutual_combine, dim3((a.n - first + 255) / 256, o4 ? 4 : 3),
                           dim3(256), 0, s, a, m.block, blocks, ox, oy, oz, o4);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_newton_mutual(const MutualShape &m, int n, const float4 *jmem, float eps2,
                                bool refine, bool guard, float *ax, float *ay, float *az,
                                float *phi, float *part, const int *same, hipStream_t s)
{
    return launch_strips(mutual_kernel(refine, guard, phi != nullptr), m,
                         MutualArgs{n, jmem, eps2, 0, m.chunk, 0, nullptr, part, same}, ax, ay, az,
                         phi, s);
}

hipError_t launch_newton_mutual_bwd(const MutualShape &m, int n, const float4 *rec, float eps2,
                                    bool refine, float *gx, float *gy, float *gz, float *gm,
                                    float *part, hipStream_t s)
{
    return launch_strips(refine ? k_newton_mutual_bwd<true> : k_newton_mutual_bwd<false>, m,
                         MutualArgs{n, rec, eps2, 0, m.chunk, 0, nullptr, part, nullptr}, gx, gy,
                         gz, gm, s);
}

}  // namespace pgh
