// Barnes-Hut tree on gfx950 that produces the (i-group, j-list) interaction
// lists of the tree code of Sec. 5 (Barnes' shared lists for groups of
// i-particles; opening parameter theta; monopole moments, or quadrupole
// moments carried by pseudo-particles after Kawai & Makino) for the batched
// force kernels.
//
// Definitions (the FP64 oracle the tests compare against implements the same
// definitions in code of its own):
//   frame   lo = componentwise minimum of the positions, extent = the largest
//           axis range, scale = 2^21 / extent, all FP32;
//   keys    per axis min(floor((x - lo) * scale), 2^21 - 1) (FP32 subtract and
//           multiply, no contraction), 3-bit digits x|y|z from the top;
//   order   sort by (key, original index) -- a stable radix sort of the keys;
//   octree  a node of level L holds the particles sharing its first 3L key
//           bits; it splits into its non-empty octants when it holds more than
//           n_leaf particles and L < 21; nodes numbered breadth first, each
//           level in key order; node size extent / 2^L;
//   moments FP64 mass, centre of mass (plain mean when the mass is zero) and
//           second moment about it;
//   pseudo  monopole: (com, M); quadrupole: three particles of mass M/3 at
//           com + a cos(2 pi k/3) e1 + b sin(2 pi k/3) e2 from the principal
//           axes of S (a^2 = 2 (l1 - l3)/M, b^2 = 2 (l2 - l3)/M): the node's
//           mass, zero dipole and the traceless part of S;
//   groups  nodes holding at most n_crit particles (or leaves) whose parent
//           holds more, in key order;
//   walk    breadth first from the root per group; g and its ancestors are
//           opened; another node is accepted when (l/theta)^2 < d^2, d the
//           distance from its com to the group's bounding box, and adds its
//           pseudo-particles; an opened leaf adds its particles.
//
// The build keeps the sizes of the levels in a device table and waits
// for the stream once, at its end (the walk waits after its counting pass);
// neither is meant for graph capture.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>

#include "pgh_internal.h"

namespace pgh {
namespace {

constexpr unsigned long long kMask21 = (1ull << 21) - 1;

__device__ inline unsigned ord_of(float f)
{
    const unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

float float_of_ord(unsigned o)
{
    const unsigned u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
    float f;
    std::memcpy(&f, &u, sizeof f);
    return f;
}

__global__ void k_init_words(unsigned *w)
{
    const int i = threadIdx.x;
    if (i < 16) w[i] = (i < 3) ? 0xffffffffu : 0u;  // min ords, max ords, counters
}

// Componentwise min / max of the positions into w[0..2] / w[3..5] as ordered
// integers (atomics on the order-preserving image of the float).
__global__ void __launch_bounds__(256) k_frame(int n, const float *__restrict__ x,
                                               const float *__restrict__ y,
                                               const float *__restrict__ z, unsigned *w)
{
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float v[3] = {x[i], y[i], z[i]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], v[a]);
            hi[a] = fmaxf(hi[a], v[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
        for (int o = 32; o > 0; o >>= 1) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
        }
    // the workgroup's four waves, then one atomic per workgroup and value
    // (one per wave would queue thousands on the same six words)
    __shared__ float part[4][6];
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int a = 0; a < 3; ++a) part[wv][a] = lo[a], part[wv][3 + a] = hi[a];
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        float v = part[0][a];
        for (int k = 1; k < 4; ++k) v = a < 3 ? fminf(v, part[k][a]) : fmaxf(v, part[k][a]);
        if (a < 3)
            atomicMin(&w[a], ord_of(v));
        else
            atomicMax(&w[a], ord_of(v));
    }
}

// 21-bit integer -> bits at positions 0, 3, 6, ... (shift-and-mask spreading)
__device__ inline unsigned long long spread3(unsigned long long v)
{
    v &= kMask21;
    v = (v | (v << 32)) & 0x001F00000000FFFFull;
    v = (v | (v << 16)) & 0x001F0000FF0000FFull;
    v = (v | (v << 8)) & 0x100F00F00F00F00Full;
    v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

__device__ inline unsigned long long cell_of(float v, float lo, float scale)
{
    const float t = __fmul_rn(__fsub_rn(v, lo), scale);
    const float f = fminf(fmaxf(floorf(t), 0.f), 2097151.f);
    return (unsigned long long)f;
}

// Keys in input order, with the particles packed (x, y, z, m) in input order
// for the gather (one 16-byte load per particle instead of four 4-byte ones).
__global__ void __launch_bounds__(256) k_keys(int n, const float *__restrict__ x,
                                              const float *__restrict__ y,
                                              const float *__restrict__ z,
                                              const float *__restrict__ m, float lox, float loy,
                                              float loz, float scale,
                                              unsigned long long *__restrict__ key,
                                              int *__restrict__ iota, float4 *__restrict__ xin)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float px = x[i], py = y[i], pz = z[i];
    const unsigned long long kx = cell_of(px, lox, scale), ky = cell_of(py, loy, scale),
                             kz = cell_of(pz, loz, scale);
    key[i] = (spread3(kx) << 2) | (spread3(ky) << 1) | spread3(kz);
    iota[i] = i;
    xin[i] = make_float4(px, py, pz, m[i]);
}

// The particles in key order, and each particle's rank (inv[perm[r]] = r).
__global__ void __launch_bounds__(256) k_gather(int n, const int *__restrict__ perm,
                                                const float4 *__restrict__ xin, float *xs,
                                                float *ys, float *zs, float *ms, float4 *xm,
                                                int *__restrict__ inv)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const int i = perm[r];
    inv[i] = r;
    const float4 v = xin[i];
    xs[r] = v.x;
    ys[r] = v.y;
    zs[r] = v.z;
    ms[r] = v.w;
    xm[r] = v;
}

// Level table of the octree build: level L holds nodes [lvl[L], lvl[L + 1]),
// in rank order.  All sizes stay on the device: the host launches the whole
// build without waiting.
constexpr int kLvl = kTreeMaxLevel + 3;
constexpr int kLevels = kTreeMaxLevel + 1;
// What the host reads after a wait, written by kernels into pinned memory (a
// copy to ordinary host memory costs a launch and a wait of its own each).
struct TreeHostPage {
    unsigned word[16];
    int lvl[kLvl];
    int n_groups;
    long long entries;
};
__global__ void __launch_bounds__(64) k_report(const unsigned *w, const int *lvl,
                                               const int *n_groups, TreeHostPage *page)
{
    const int i = threadIdx.x;
    if (i < 16) page->word[i] = w[i];
    if (lvl && i < kLvl) page->lvl[i] = lvl[i];
    if (n_groups && i == 0) page->n_groups = *n_groups;
}

// word indices in TreeState::word
constexpr int kWordLeaves = 6, kWordOverflow = 9, kWordMaxLevel = 10;

// The octree of the sorted keys, all levels at once.  With d(r) the leading
// octal digits that key r shares with key r - 1 (-1 for r = 0), the cells that
// begin at rank r are those of the levels above d(r); such a cell is a node if
// its parent holds more than n_leaf particles.  So each rank knows from a few
// neighbouring keys the levels (consecutive ones) of the nodes that begin at
// it, as a mask, and a node's place in its level is the number of nodes of the
// level that begin at earlier ranks:
//   k_node_mask   the masks, and per chunk of 256 ranks and level their counts;
//   k_node_scan   the counts' offsets within each level;
//   k_node_write  the level table and the nodes' first rank, level, parent and
//                 first child (the children of a node are consecutive: they
//                 begin at its ranks);
//   k_node_ends   the nodes' particle counts and numbers of children.
// Four launches, bound by their latency and two passes over the keys; the same
// nodes in the same order level by level took three launches for each of the 22
// levels, 482 us of a tree of 2^20 particles; these four take 45.
constexpr int kNodeChunk = 256;  // ranks of a wave in k_node_mask and k_node_write

// leading octal digits that two keys share (kTreeMaxLevel: the same key)
__device__ inline int common_digits(unsigned long long a, unsigned long long b)
{
    const unsigned long long x = a ^ b;
    return x ? (__clzll((long long)x) - 1) / 3 : kTreeMaxLevel;
}

// the cell of a key at level L
__device__ inline unsigned long long cell_at(unsigned long long k, int L)
{
    return k >> (3 * (kTreeMaxLevel - L));
}

// First r in (lo, hi] beyond the cell at level L of rank lo (hi: none before).
__device__ inline int cell_end(const unsigned long long *key, int lo, int hi, int L)
{
    const unsigned long long c = cell_at(key[lo], L);
    int step = 8;  // most cells are small: doubling steps, then the search
    while (step < hi - lo && cell_at(key[lo + step], L) == c) {
        lo += step;
        step = min(2 * step, 1 << 29);
    }
    hi = lo + min(step, hi - lo);
    ++lo;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (cell_at(key[mid], L) == c)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__global__ void __launch_bounds__(256) k_node_mask(int n, int n_leaf,
                                                   const unsigned long long *__restrict__ key,
                                                   unsigned *__restrict__ mask, int chunks,
                                                   int *__restrict__ sums)
{
    const int lane = threadIdx.x & 63;
    const int chunk = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6);
    if (chunk >= chunks) return;
    int sum = 0;  // lane L: the chunk's nodes of level L, the lane after: its leaves
#pragma unroll 1
    for (int k = 0; k < kNodeChunk / 64; ++k) {
        const long long rl = (long long)chunk * kNodeChunk + 64 * k + lane;
        const int r = (int)min(rl, (long long)n - 1);
        const unsigned long long me = key[r];
        const int d = r == 0 ? -1 : common_digits(key[r - 1], me);
        // levels <= e of the cells that begin here are split
        const int e = n_leaf < n - r ? common_digits(me, key[r + n_leaf]) : -1;
        bool node = d < kTreeMaxLevel;
        if (node && d >= 0 && e < d) {
            // is the parent's cell, of level d, longer than n_leaf?  Its first
            // rank, if within n_leaf before r, and its length from there
            const unsigned long long c = cell_at(me, d);
            int lo = r > n_leaf ? r - n_leaf : 0, hi = r - 1;
            while (lo < hi) {
                const int mid = lo + ((hi - lo) >> 1);
                if (cell_at(key[mid], d) == c)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            node = n_leaf < n - lo && cell_at(key[lo + n_leaf], d) == c;
        }
        const int first = d + 1, last = max(first, min(e, kTreeMaxLevel - 1) + 1);
        unsigned m = node ? (2u << last) - (1u << first) : 0u;
        if (rl >= n) m = 0u;
        if (rl < n) mask[r] = m;
        for (int L = 0; L < kLevels; ++L) {
            const int c = __popcll(__ballot((m >> L) & 1));
            sum += lane == L ? c : 0;
        }
        // of the nodes that begin at a rank the deepest is a leaf
        const int c = __popcll(__ballot(m != 0));
        sum += lane == kLevels ? c : 0;
    }
    if (lane <= kLevels) sums[(size_t)lane * chunks + chunk] = sum;
}

// Inclusive prefix sum over the 64 lanes of a wave (all lanes active) by DPP
// lane moves: the sums of up to four lanes inside each row of 16 (row shifts
// by 1, 2 and 3 of the value), then of eight and of the whole row (row shifts
// by 4 and 8 of the partial sums into the upper banks), then across rows (lane
// 15 of row 0 and 2 broadcast into rows 1 and 3, lane 31 into rows 2 and 3).
__device__ inline int wave_incl_scan(int x)
{
    int v = x + __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);          // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xF, 0xF, true);          // row_shr:3
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xE, false);         // row_shr:4, banks 1-3
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xC, false);         // row_shr:8, banks 2-3
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);         // row_bcast:15, rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);         // row_bcast:31, rows 2, 3
    return v;
}

// Inclusive scan over a workgroup of 256 (wave scans, then the wave totals);
// *total receives the workgroup's sum.  Every thread of the workgroup calls it.
__device__ inline int block_incl_scan(int v, int *sh, int *total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    v = wave_incl_scan(v);
    if (lane == 63) sh[wv] = v;
    __syncthreads();
    int add = 0;
    for (int k = 0; k < wv; ++k) add += sh[k];
    *total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return v + add;
}

// Workgroup L: the exclusive offsets of the chunks' counts of level L, in
// place, and the level's size in total[L] (the last workgroup: of the leaves).
__global__ void __launch_bounds__(256) k_node_scan(int chunks, int *sums, int *total)
{
    __shared__ int sh[4];
    int *v = sums + (size_t)blockIdx.x * chunks;
    int run = 0;
    for (int c0 = 0; c0 < chunks; c0 += 1024) {
        const int c = c0 + 4 * (int)threadIdx.x;
        int x[4], sum = 0, tot = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = c + k < chunks ? v[c + k] : 0;
            sum += x[k];
        }
        int at = run + block_incl_scan(sum, sh, &tot) - sum;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (c + k < chunks) v[c + k] = at;
            at += x[k];
        }
        run += tot;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = run;
}

// More nodes than the arrays hold set the overflow word instead: every later
// kernel of the build returns at once, and the host builds again with more room.
__global__ void __launch_bounds__(256) k_node_write(int n, const unsigned *__restrict__ mask,
                                                    int chunks, const int *__restrict__ sums,
                                                    const int *__restrict__ total, int cap,
                                                    int *__restrict__ begin,
                                                    int *__restrict__ level,
                                                    int *__restrict__ first_child,
                                                    int *__restrict__ n_child,
                                                    int *__restrict__ parent, int *lvl, unsigned *w)
{
    const int lane = threadIdx.x & 63;
    const int chunk = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6);
    int off[kLevels + 1];
    long long all = 0;
    int widest = 0;
#pragma unroll
    for (int L = 0; L < kLevels; ++L) {
        const int c = total[L];
        off[L] = (int)all;
        all = min(all + c, (long long)INT_MAX);
        if (L) widest = max(widest, c);
    }
    off[kLevels] = (int)all;
    const bool over = all > cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
        for (int L = 0; L <= kLevels; ++L) lvl[L] = off[L];
        lvl[kLevels + 1] = off[kLevels];
        if (over) w[kWordOverflow] = 1u;
        w[kWordMaxLevel] = (unsigned)widest;
        w[kWordLeaves] = (unsigned)total[kLevels];
    }
    if (over || chunk >= chunks) return;
    // lane L: the nodes of level L before this step
    int run = lane < kLevels ? sums[(size_t)lane * chunks + chunk] : 0;
    const unsigned long long before = (1ull << lane) - 1;
    unsigned ms[kNodeChunk / 64];
#pragma unroll
    for (int k = 0; k < kNodeChunk / 64; ++k) {
        const long long rl = (long long)chunk * kNodeChunk + 64 * k + lane;
        ms[k] = rl < n ? mask[rl] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kNodeChunk / 64; ++k) {
        const long long rl = (long long)chunk * kNodeChunk + 64 * k + lane;
        const unsigned m = ms[k];
        int node = -1;  // this rank's node of level L - 1, where it has one
        int last = -1;  // the last node of level L - 1 that begins at or before r
#pragma unroll
        for (int L = 0; L < kLevels; ++L) {
            const unsigned long long b = __ballot((m >> L) & 1);
            const int at0 = off[L] + __builtin_amdgcn_readlane(run, L);
            if (b == 0) {
                node = -1;
                last = at0 - 1;
                continue;
            }
            const int at = at0 + __popcll(b & before);
            run += lane == L ? __popcll(b) : 0;
            const bool has = (m >> L) & 1;
            if (has) {
                if (node >= 0) first_child[node] = at;
                begin[at] = (int)rl;
                level[at] = L;
                parent[at] = last;
                if (!((m >> L) & 2)) {  // no node begins here a level below: a leaf
                    first_child[at] = -1;
                    n_child[at] = 0;
                }
            }
            node = has ? at : -1;
            last = has ? at : at - 1;
        }
    }
}

// A node ends where its next sibling begins, the last one with its cell; the
// last one also knows the number of its parent's children.
__global__ void __launch_bounds__(256) k_node_ends(int n, const unsigned long long *__restrict__ key,
                                                   const int *__restrict__ lvl,
                                                   const unsigned *__restrict__ w,
                                                   const int *__restrict__ begin,
                                                   const int *__restrict__ level,
                                                   const int *__restrict__ first_child,
                                                   const int *__restrict__ parent,
                                                   int *__restrict__ count,
                                                   int *__restrict__ n_child)
{
    if (w[kWordOverflow]) return;
    const int nodes = lvl[kLevels];
    for (int j = blockIdx.x * 256 + threadIdx.x; j < nodes; j += gridDim.x * 256) {
        const int b = begin[j], p = parent[j];
        if (j + 1 < nodes && parent[j + 1] == p) {
            count[j] = begin[j + 1] - b;
        } else {
            count[j] = cell_end(key, b, n, level[j]) - b;
            if (p >= 0) n_child[p] = j + 1 - first_child[p];
        }
    }
}

// v from another lane of the same 8-lane group by a DPP lane pattern (a
// VALU move, no LDS round trip): both 32-bit halves.
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over the 8 lanes of a node's lane group, the same in every lane: the
// lane pairs i ^ 1 and i ^ 2 inside each quad (quad_perm [1,0,3,2] and
// [2,3,0,1]), then the two quads (the half-row mirror, i <-> 7 - i).
__device__ inline double group_sum(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    return v;
}

// Moments of the nodes of one level, in FP64: a leaf from its particles, an
// internal node from its children (parallel-axis theorem).  Eight lanes take
// a node, each a share of its particles or children; the centre is the
// mass-weighted mean (the particle-count-weighted mean when the mass is zero).
__global__ void __launch_bounds__(256) k_moments(int L, const int *__restrict__ lvl,
                                                 const unsigned *__restrict__ w,
                                                 const int *__restrict__ begin,
                                                 const int *__restrict__ count,
                                                 const int *__restrict__ first_child,
                                                 const int *__restrict__ n_child,
                                                 const float4 *__restrict__ xm, NodeMoments *mom)
{
    if (w[kWordOverflow]) return;
    const int off = lvl[L], n_level = lvl[L + 1] - off;
    const int g = (int)threadIdx.x >> 3, j = (int)threadIdx.x & 7;
    for (int i0 = (int)blockIdx.x * 32; i0 < n_level; i0 += (int)gridDim.x * 32) {
        const int i = i0 + g;
        const bool valid = i < n_level;
        const int node = off + (valid ? i : 0);
        const int nch = valid ? n_child[node] : 0;
        // this lane's items: particles [k0, k1) of a leaf, or children
        const int k0 = nch ? first_child[node] : begin[node];
        const int k1 = valid ? k0 + (nch ? nch : count[node]) : k0;
        auto item = [&](int k, double *m, double *x, double *y, double *z, double *cnt) {
            if (nch) {
                const NodeMoments &q = mom[k];
                *m = q.m, *x = q.cx, *y = q.cy, *z = q.cz, *cnt = count[k];
            } else {
                const float4 p = xm[k];
                *m = p.w, *x = p.x, *y = p.y, *z = p.z, *cnt = 1.0;
            }
        };
        double M = 0, sx = 0, sy = 0, sz = 0, np = 0, px = 0, py = 0, pz = 0;
        for (int k = k0 + j; k < k1; k += 8) {
            double m, x, y, z, cnt;
            item(k, &m, &x, &y, &z, &cnt);
            M += m;
            sx += m * x, sy += m * y, sz += m * z;
            np += cnt;
            px += cnt * x, py += cnt * y, pz += cnt * z;
        }
        M = group_sum(M);
        sx = group_sum(sx), sy = group_sum(sy), sz = group_sum(sz);
        np = group_sum(np);
        px = group_sum(px), py = group_sum(py), pz = group_sum(pz);
        if (M != 0.0)
            sx /= M, sy /= M, sz /= M;
        else if (np != 0.0)
            sx = px / np, sy = py / np, sz = pz / np;
        double a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0, a5 = 0;
        for (int k = k0 + j; k < k1; k += 8) {
            double m, x, y, z, cnt;
            item(k, &m, &x, &y, &z, &cnt);
            if (nch) {
                const NodeMoments &q = mom[k];
                a0 += q.sxx, a1 += q.syy, a2 += q.szz, a3 += q.sxy, a4 += q.sxz, a5 += q.syz;
            }
            const double dx = x - sx, dy = y - sy, dz = z - sz;
            a0 += m * dx * dx, a1 += m * dy * dy, a2 += m * dz * dz;
            a3 += m * dx * dy, a4 += m * dx * dz, a5 += m * dy * dz;
        }
        a0 = group_sum(a0), a1 = group_sum(a1), a2 = group_sum(a2);
        a3 = group_sum(a3), a4 = group_sum(a4), a5 = group_sum(a5);
        // the group stores the 10 doubles side by side: lane j field j, lanes 0
        // and 1 also fields 8 and 9
        if (valid) {
            static_assert(sizeof(NodeMoments) == 10 * sizeof(double), "NodeMoments layout");
            double *dst = reinterpret_cast<double *>(mom + node);
            const double v = j == 0 ? M : j == 1 ? sx : j == 2 ? sy : j == 3 ? sz
                           : j == 4 ? a0 : j == 5 ? a1 : j == 6 ? a2 : a3;
            dst[j] = v;
            if (j < 2) dst[8 + j] = j == 0 ? a4 : a5;
        }
    }
}

// Symmetric 3x3 eigen-decomposition by cyclic Jacobi rotations (the symmetric
// Schur rotation of Golub & Van Loan, Sec. 8.5): eigenvalues in descending
// order in w, eigenvectors as the columns of V.
__device__ void jacobi3(const NodeMoments &q, double w[3], double V[3][3])
{
    double A[3][3] = {{q.sxx, q.sxy, q.sxz}, {q.sxy, q.syy, q.syz}, {q.sxz, q.syz, q.szz}};
    double Q[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
    for (int sweep = 0; sweep < 32; ++sweep) {
        const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
        const double dia = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
        // converged when the off-diagonal elements are at FP64 rounding of the
        // diagonal (rotations leave residues of that size, so a tighter
        // bound only runs sweeps that change nothing)
        if (off == 0.0 || off <= 1e-30 * dia) break;
        for (int p = 0; p < 2; ++p)
            for (int r = p + 1; r < 3; ++r) {
                const double apr = A[p][r];
                if (apr == 0.0) continue;
                const double tau = (A[r][r] - A[p][p]) / (2.0 * apr);
                const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                const double c = 1.0 / sqrt(1.0 + t * t), s = t * c;
                for (int k = 0; k < 3; ++k) {
                    const double u = A[k][p], v = A[k][r];
                    A[k][p] = c * u - s * v;
                    A[k][r] = s * u + c * v;
                }
                for (int k = 0; k < 3; ++k) {
                    const double u = A[p][k], v = A[r][k];
                    A[p][k] = c * u - s * v;
                    A[r][k] = s * u + c * v;
                }
                for (int k = 0; k < 3; ++k) {
                    const double u = Q[k][p], v = Q[k][r];
                    Q[k][p] = c * u - s * v;
                    Q[k][r] = s * u + c * v;
                }
            }
    }
    int o[3] = {0, 1, 2};
    if (A[o[1]][o[1]] > A[o[0]][o[0]]) { const int t = o[0]; o[0] = o[1]; o[1] = t; }
    if (A[o[2]][o[2]] > A[o[1]][o[1]]) { const int t = o[1]; o[1] = o[2]; o[2] = t; }
    if (A[o[1]][o[1]] > A[o[0]][o[0]]) { const int t = o[0]; o[0] = o[1]; o[1] = t; }
    for (int c = 0; c < 3; ++c) {
        w[c] = A[o[c]][o[c]];
        for (int r = 0; r < 3; ++r) V[r][c] = Q[r][o[c]];
    }
}

__global__ void __launch_bounds__(256) k_pseudo(const int *__restrict__ lvl,
                                                const unsigned *__restrict__ w,
                                                const NodeMoments *__restrict__ mom, int quad,
                                                float4 *__restrict__ pp, float4 *__restrict__ com)
{
    if (w[kWordOverflow]) return;
    const int n_nodes = lvl[kTreeMaxLevel + 1];
    for (int t = blockIdx.x * 256 + threadIdx.x; t < n_nodes; t += gridDim.x * 256) {
    const NodeMoments q = mom[t];
    com[t] = make_float4((float)q.cx, (float)q.cy, (float)q.cz, 0.f);
    if (!quad) {
        pp[t] = make_float4((float)q.cx, (float)q.cy, (float)q.cz, (float)q.m);
        continue;
    }
    double w[3], V[3][3];
    jacobi3(q, w, V);
    double a2 = 0.0, b2 = 0.0;
    if (q.m > 0.0) {
        a2 = 2.0 * (w[0] - w[2]) / q.m;
        b2 = 2.0 * (w[1] - w[2]) / q.m;
    }
    const double a = sqrt(fmax(a2, 0.0)), b = sqrt(fmax(b2, 0.0));
    const double h = 0.86602540378443864676;  // sin(2 pi / 3)
    const double cs[3] = {1.0, -0.5, -0.5}, sn[3] = {0.0, h, -h};
    for (int k = 0; k < 3; ++k) {
        const double u = a * cs[k], v = b * sn[k];
        pp[3 * t + k] = make_float4((float)(q.cx + u * V[0][0] + v * V[0][1]),
                                    (float)(q.cy + u * V[1][0] + v * V[1][1]),
                                    (float)(q.cz + u * V[2][0] + v * V[2][1]), (float)(q.m / 3.0));
    }
    }
}

// Walk record of a node: (begin, count, first child, n_child | level << 16).
__global__ void __launch_bounds__(256) k_pack_nodes(const int *__restrict__ lvl,
                                                    const unsigned *__restrict__ w,
                                                    const int *__restrict__ begin,
                                                    const int *__restrict__ count,
                                                    const int *__restrict__ first_child,
                                                    const int *__restrict__ n_child,
                                                    const int *__restrict__ level,
                                                    int4 *__restrict__ rec)
{
    if (w[kWordOverflow]) return;
    const int n_nodes = lvl[kTreeMaxLevel + 1];
    for (int t = blockIdx.x * 256 + threadIdx.x; t < n_nodes; t += gridDim.x * 256)
        rec[t] = make_int4(begin[t], count[t], first_child[t], n_child[t] | (level[t] << 16));
}

__global__ void __launch_bounds__(256) k_fill_int(int n, int *a, int v)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = v;
}

__global__ void __launch_bounds__(256) k_group_mark(const int *__restrict__ lvl,
                                                    const unsigned *__restrict__ w,
                                                    const int *__restrict__ begin,
                                                    const int *__restrict__ count,
                                                    const int *__restrict__ n_child,
                                                    const int *__restrict__ parent, int n_crit,
                                                    int *__restrict__ mark)
{
    if (w[kWordOverflow]) return;
    const int n_nodes = lvl[kTreeMaxLevel + 1];
    for (int t = blockIdx.x * 256 + threadIdx.x; t < n_nodes; t += gridDim.x * 256) {
        const bool small = count[t] <= n_crit || n_child[t] == 0;
        const int p = parent[t];
        const bool top = p < 0 || count[p] > n_crit;
        if (small && top) mark[begin[t]] = t;
    }
}

struct NonNegative {
    __host__ __device__ bool operator()(const int &v) const { return v >= 0; }
};

// One wave per group: bounding box of its particles and the i-side of its item.
__global__ void __launch_bounds__(256) k_group_info(const int *__restrict__ n_groups_dev,
                                                    const int *__restrict__ groups,
                                                    const int *__restrict__ begin,
                                                    const int *__restrict__ count,
                                                    const float *__restrict__ xs,
                                                    const float *__restrict__ ys,
                                                    const float *__restrict__ zs, float4 *glo,
                                                    float4 *ghi, pgh_item *items)
{
    const int n_groups = *n_groups_dev;
    const int lane = threadIdx.x & 63;
    for (int g = blockIdx.x * 4 + (threadIdx.x >> 6); g < n_groups; g += gridDim.x * 4) {
    const int t = groups[g];
    const int b = begin[t], c = count[t];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int k = b + lane; k < b + c; k += 64) {
        const float v[3] = {xs[k], ys[k], zs[k]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], v[a]);
            hi[a] = fmaxf(hi[a], v[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
        for (int o = 32; o > 0; o >>= 1) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
        }
    if (lane == 0) {
        glo[g] = make_float4(lo[0], lo[1], lo[2], 0.f);
        ghi[g] = make_float4(hi[0], hi[1], hi[2], 0.f);
        items[g].i_off = b;
        items[g].n_i = c;
    }
    }
}

struct WalkArgs {
    int n_groups;
    const int *groups;
    const float4 *glo, *ghi;
    const int4 *node;  // walk records (k_pack_nodes)
    const float4 *com, *pp;
    int npp;
    float rc2[kTreeMaxLevel + 1];  // (l_L / theta)^2 per level
    const float4 *xm;  // particles (x, y, z, m) in key order
    long long *glen;        // pass 1 output: list length per group
    const long long *goff;  // pass 2 input: list offset per group
    float4 *xmj;  // the lists: (x, y, z, m) per entry
    int *src;               // pass 2, optional
    unsigned *overflow;
    unsigned *max_frontier; // pass 1: the largest frontier met
};


constexpr int kWalkWaves = 4;  // waves of a workgroup, walking one group together
constexpr int kMapSeg = 256;  // entries per wave of a segment of the write pass's map

// Breadth-first walk, a workgroup of W = kWalkWaves waves per group.  Its 64 W lanes test as
// many frontier nodes at a time; prefix sums over the workgroup place each
// lane's contributions in the list and its opened children in the next
// frontier (double-buffered in LDS).  Pass 1 (WRITE = false) only counts; pass
// 2 writes the entries at the offsets of the scanned counts, in the same
// order: the contributions of the nodes tested together form one contiguous
// block of the list, which the lanes write entry by entry (coalesced), each
// finding its entry's node through a map.
//
// Bound by the latency of its steps, some 20 levels deep with a few hundred
// nodes each, so four waves share a group: 3739 groups of a tree of 2^20
// particles 63 us to count and 106 to write, against 107 and 214 with a wave
// per group; not slower with 53342 groups of at most 64 either.
template <bool WRITE, int FCAP>
__global__ void __launch_bounds__(64 * kWalkWaves) k_walk(WalkArgs a)
{
    constexpr int W = kWalkWaves;
    __shared__ int fr[2][FCAP];
    __shared__ int2 tot[2][W];
    // write pass: each lane's first entry and source code, and the lane that
    // owns each entry of a segment of kMapSeg W entries
    __shared__ int s_start[WRITE ? 64 * W : 1], s_src[WRITE ? 64 * W : 1];
    __shared__ unsigned char s_map[WRITE ? kMapSeg * W : 1];
    __shared__ float rc2[kTreeMaxLevel + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid <= kTreeMaxLevel) rc2[tid] = a.rc2[tid];
    if (!WRITE && blockIdx.x == 0 && tid == 0) a.glen[a.n_groups] = 0;  // for the scan's total
    int maxf = 0;  // largest frontier of this workgroup (one atomic at the end)
    int step = 0;
    for (int g = blockIdx.x; g < a.n_groups; g += gridDim.x) {
        const int gn = a.groups[g];
        const float4 lo = a.glo[g], hi = a.ghi[g];
        const int4 grec = a.node[gn];
        const int gb = grec.x, glev = grec.w >> 16;
        const long long out = WRITE ? a.goff[g] : 0;
        long long len = 0;
        int cur = 0, ncur = 1;
        bool over = false;
        if (tid == 0) fr[0][0] = 0;
        __syncthreads();
        while (ncur > 0) {
            int nnext = 0;
            for (int c0 = 0; c0 < ncur; c0 += 64 * W, step ^= 1) {
                const int idx = c0 + tid;
                int emit = 0, push = 0, code = 0, fc = 0;
                if (idx < ncur) {
                    const int t = fr[cur][idx];
                    const int4 r = a.node[t];
                    const float4 cm = a.com[t];
                    const int b = r.x, c = r.y, nch = r.w & 0xffff, L = r.w >> 16;
                    fc = r.z;
                    const bool anc = L <= glev && b <= gb && gb < b + c;
                    const float ex = fmaxf(fmaxf(lo.x - cm.x, cm.x - hi.x), 0.f);
                    const float ey = fmaxf(fmaxf(lo.y - cm.y, cm.y - hi.y), 0.f);
                    const float ez = fmaxf(fmaxf(lo.z - cm.z, cm.z - hi.z), 0.f);
                    const bool acc = !anc && rc2[L] < ex * ex + ey * ey + ez * ez;
                    if (acc) {
                        emit = a.npp;
                        code = t * a.npp;  // first pseudo-particle
                    } else if (nch == 0) {
                        emit = c;
                        code = -1 - b;     // first particle
                    } else {
                        push = nch;
                    }
                }
                int e_inc = wave_incl_scan(emit);
                int p_inc = wave_incl_scan(push);
                // two buffers in turn: one barrier a step is enough
                if (lane == 63) tot[step][w] = make_int2(e_inc, p_inc);
                __syncthreads();
                int e_tot = 0, p_tot = 0, e_before = 0, p_before = 0;
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    const int2 v = tot[step][k];
                    if (k < w) e_before += v.x, p_before += v.y;
                    e_tot += v.x;
                    p_tot += v.y;
                }
                e_inc += e_before;
                p_inc += p_before;
                if (nnext + p_tot > FCAP) {
                    over = true;
                    break;
                }
                for (int k = 0; k < push; ++k) fr[cur ^ 1][nnext + p_inc - push + k] = fc + k;
                if (WRITE && e_tot > 0) {
                    const int r0 = e_inc - emit;  // this lane's first entry
                    s_start[tid] = r0;
                    s_src[tid] = code;
                    const long long base = out + len;
                    // segment by segment: every lane marks its entries in the
                    // map, then the entries are written, each lane finding its
                    // entry's source through the map
                    for (int seg = 0; seg < e_tot; seg += kMapSeg * W) {
                        const int m0 = max(r0, seg), m1 = min(e_inc, seg + kMapSeg * W);
                        for (int e = m0; e < m1; ++e) s_map[e - seg] = (unsigned char)tid;
                        __syncthreads();
                        const int seg_end = min(e_tot, seg + kMapSeg * W);
                        for (int e = seg + tid; e < seg_end; e += 64 * W) {
                            const int l = s_map[e - seg];
                            const int k = e - s_start[l];
                            const int cd = s_src[l];
                            a.xmj[base + e] = cd >= 0 ? a.pp[cd + k] : a.xm[-1 - cd + k];
                            if (a.src) a.src[base + e] = cd >= 0 ? -(1 + cd + k) : -1 - cd + k;
                        }
                        __syncthreads();
                    }
                }
                len += e_tot;
                nnext += p_tot;
            }
            if (over) break;
            maxf = max(maxf, nnext);
            __syncthreads();
            cur ^= 1;
            ncur = nnext;
        }
        if (over) {
            if (tid == 0) atomicOr(a.overflow, 1u);
            len = 0;
        }
        if (!WRITE && tid == 0) a.glen[g] = len;
        __syncthreads();
    }
    if (!WRITE && tid == 0 && maxf > 0) atomicMax(a.max_frontier, (unsigned)maxf);
}

template <bool WRITE, int FCAP>
void launch_walk(const WalkArgs &a, int num_cu, hipStream_t s)
{
    // resident workgroups: FCAP's two buffers of LDS each
    const int per_cu = FCAP > kWalkFrontier / 2 ? 4 : 8;
    hipLaunchKernelGGL((k_walk<WRITE, FCAP>), dim3(std::min(a.n_groups, per_cu * num_cu)),
                       dim3(64 * kWalkWaves), 0, s, a);
}

// The walked groups' items, on the device and in pinned host memory, with the
// status words and the number of entries.
__global__ void __launch_bounds__(256) k_items_j(int n_groups, const long long *__restrict__ goff,
                                                 const long long *__restrict__ glen,
                                                 const unsigned *__restrict__ w, pgh_item *items,
                                                 pgh_item *host_items, TreeHostPage *page)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g < 16) page->word[g] = w[g];
    if (g == 0) page->entries = goff[n_groups];
    if (g >= n_groups) return;
    pgh_item it = items[g];
    it.j_off = (int)goff[g];
    it.n_j = (int)glen[g];
    items[g] = it;
    host_items[g] = it;
}

int blocks_of(long long n, int per) { return (int)std::max(1LL, (n + per - 1) / per); }

template <class T>
bool grow(T **p, long long *cap_now, long long cap_new)
{
    T *q = nullptr;
    if (hipMalloc((void **)&q, sizeof(T) * (size_t)std::max(1LL, cap_new)) != hipSuccess)
        return false;
    (void)hipFree(*p);
    *p = q;
    *cap_now = cap_new;
    return true;
}

#define TREE_HIP(call)                                                    \
    do {                                                                  \
        hipError_t e_ = (call);                                           \
        if (e_ != hipSuccess) {                                           \
            err = std::string(#call) + ": " + hipGetErrorString(e_);      \
            return PGH_EHIP;                                              \
        }                                                                 \
    } while (0)

#define TREE_ALLOC(ok)                                                    \
    do {                                                                  \
        if (!(ok)) {                                                      \
            err = "tree: device allocation failed";                       \
            return PGH_ENOMEM;                                            \
        }                                                                 \
    } while (0)

size_t temp_bytes_for(int n, int ngroups)
{
    size_t a = 0, b = 0, c = 0, d = 0;
    (void)hipcub::DeviceRadixSort::SortPairs(nullptr, a, (unsigned long long *)nullptr,
                                             (unsigned long long *)nullptr, (int *)nullptr,
                                             (int *)nullptr, n, 0, 63);
    (void)hipcub::DeviceScan::ExclusiveSum(nullptr, b, (int *)nullptr, (int *)nullptr, n + 1);
    (void)hipcub::DeviceSelect::If(nullptr, c, (int *)nullptr, (int *)nullptr, (int *)nullptr, n,
                                   NonNegative());
    (void)hipcub::DeviceScan::ExclusiveSum(nullptr, d, (long long *)nullptr,
                                           (long long *)nullptr, ngroups + 1);
    return std::max(std::max(a, b), std::max(c, d));
}

int ensure_tmp(TreeState &t, int n, std::string &err)
{
    const size_t want = temp_bytes_for(n, n);
    if (want <= t.tmp_bytes) return PGH_OK;
    (void)hipFree(t.tmp);
    t.tmp = nullptr;
    t.tmp_bytes = 0;
    TREE_ALLOC(hipMalloc(&t.tmp, want) == hipSuccess);
    t.tmp_bytes = want;
    return PGH_OK;
}

}  // namespace

void tree_release(TreeState &t)
{
    void *ps[] = {t.key, t.key_in, t.perm, t.iota, t.xs, t.ys, t.zs, t.ms, t.mark, t.xin, t.inv, t.res,
                  t.begin, t.count, t.level, t.first_child, t.n_child, t.parent, t.nc, t.mom, t.com, t.pp, t.groups, t.glo, t.ghi, t.glen, t.goff,
                  t.items, t.xmj, t.src, t.tmp, t.word, t.count_out, t.lvl,
                  t.xm, t.nrec};
    for (void *p : ps) (void)hipFree(p);
    (void)hipHostFree(t.page);
    (void)hipHostFree(t.host_items);
    t = TreeState();
}

int tree_build(TreeState &t, int n, const float *x, const float *y, const float *z,
               const float *m, int n_leaf, int n_crit, int quad, int num_cu, hipStream_t s,
               std::string &err)
{
    t.built = t.walked = 0;
    t.n = n;
    t.n_leaf = n_leaf;
    t.n_crit = n_crit;
    t.quad = quad ? 1 : 0;
    t.n_nodes = t.n_leaves = t.depth = t.n_groups = t.max_level_nodes = 0;
    t.n_entries = t.interactions = 0;
    std::fill(t.level_off, t.level_off + kTreeMaxLevel + 2, 0);
    std::fill(t.frame, t.frame + 5, 0.f);
    TREE_ALLOC(t.word || hipMalloc((void **)&t.word, 16 * sizeof(unsigned)) == hipSuccess);
    TREE_ALLOC(t.count_out || hipMalloc((void **)&t.count_out, sizeof(int)) == hipSuccess);
    TREE_ALLOC(t.lvl || hipMalloc((void **)&t.lvl, kLvl * sizeof(int)) == hipSuccess);
    TREE_ALLOC(t.page || hipHostMalloc(&t.page, sizeof(TreeHostPage)) == hipSuccess);
    if (n == 0) {
        t.built = 1;
        return PGH_OK;
    }
    if (n > t.n_cap) {
        const long long cap = std::max(n, 1024);
        long long dummy = 0;
        bool ok = grow(&t.key, &dummy, cap) && grow(&t.key_in, &dummy, cap) &&
                  grow(&t.perm, &dummy, cap) && grow(&t.iota, &dummy, cap) &&
                  grow(&t.xs, &dummy, cap) && grow(&t.ys, &dummy, cap) &&
                  grow(&t.zs, &dummy, cap) && grow(&t.ms, &dummy, cap) &&
                  grow(&t.mark, &dummy, cap) && grow(&t.xm, &dummy, cap) &&
                  grow(&t.xin, &dummy, cap) && grow(&t.inv, &dummy, cap) &&
                  grow(&t.res, &dummy, cap);
        if (!ok) {
            t.n_cap = 0;
            err = "tree: device allocation failed";
            return PGH_ENOMEM;
        }
        t.n_cap = (int)cap;
        int st = ensure_tmp(t, (int)cap, err);
        if (st) return st;
    }
    // 1. frame
    hipLaunchKernelGGL(k_init_words, dim3(1), dim3(64), 0, s, t.word);
    hipLaunchKernelGGL(k_frame, dim3(std::min(blocks_of(n, 256), num_cu)), dim3(256), 0, s, n,
                       x, y, z, t.word);
    TREE_HIP(hipGetLastError());
    TreeHostPage *page = static_cast<TreeHostPage *>(t.page);
    hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, s, t.word, (const int *)nullptr,
                       (const int *)nullptr, page);
    TREE_HIP(hipGetLastError());
    TREE_HIP(hipStreamSynchronize(s));
    const unsigned *wv = page->word;
    float lo[3], hi[3], ext = 0.f;
    for (int a = 0; a < 3; ++a) {
        lo[a] = float_of_ord(wv[a]);
        hi[a] = float_of_ord(wv[3 + a]);
        const float e = hi[a] - lo[a];
        if (e > ext) ext = e;
    }
    if (!std::isfinite(ext)) {
        err = "tree: positions must be finite";
        return PGH_ERANGE;
    }
    const float scale = ext > 0.f ? 2097152.0f / ext : 0.f;
    t.frame[0] = lo[0], t.frame[1] = lo[1], t.frame[2] = lo[2], t.frame[3] = ext;
    t.frame[4] = scale;
    // 2. keys, sort, gather
    hipLaunchKernelGGL(k_keys, dim3(blocks_of(n, 256)), dim3(256), 0, s, n, x, y, z, m, lo[0],
                       lo[1], lo[2], scale, t.key_in, t.iota, t.xin);
    TREE_HIP(hipGetLastError());
    size_t tb = t.tmp_bytes;
    TREE_HIP(hipcub::DeviceRadixSort::SortPairs(t.tmp, tb, t.key_in, t.key, t.iota, t.perm, n, 0,
                                                63, s));
    hipLaunchKernelGGL(k_gather, dim3(blocks_of(n, 256)), dim3(256), 0, s, n, t.perm, t.xin,
                       t.xs, t.ys, t.zs, t.ms, t.xm, t.inv);
    TREE_HIP(hipGetLastError());
    // 3-5. octree, moments, pseudo-particles and groups, launched with no
    // wait: the level sizes stay in a device table (lvl).  The node arrays
    // start at 2n (a tree needs about n / 2 with leaves of 8); a build that
    // outgrows them sets the overflow word, returns from every later kernel,
    // and runs again with twice the room.
    if (t.group_cap < n) {
        const long long cap = std::max(n, 1024);
        long long dummy = 0;
        TREE_ALLOC(grow(&t.groups, &dummy, cap) && grow(&t.glo, &dummy, cap) &&
                   grow(&t.ghi, &dummy, cap) && grow(&t.glen, &dummy, cap + 1) &&
                   grow(&t.goff, &dummy, cap + 1) && grow(&t.items, &dummy, cap));
        t.group_cap = (int)cap;
    }
    // the ranks' masks, the chunks' counts per level, the levels' sizes
    const long long chunks = blocks_of(n, kNodeChunk);
    const long long nc_need = n + (kLevels + 1) * (chunks + 1);
    if (t.nc_cap < nc_need) {
        long long dummy = 0;
        const long long cap = std::max(n, 1024);
        const long long words = cap + (kLevels + 1) * (blocks_of(cap, kNodeChunk) + 1LL);
        TREE_ALLOC(grow(&t.nc, &dummy, words));
        t.nc_cap = words;
    }
    long long want = std::max<long long>(2LL * n + 64, 4096);
    for (;;) {
        if (want > INT_MAX) {
            err = "tree: too many nodes";
            return PGH_ERANGE;
        }
        if (t.node_cap < want) {
            const long long cap = want;
            long long dummy = 0;
            TREE_ALLOC(grow(&t.begin, &dummy, cap) && grow(&t.count, &dummy, cap) &&
                       grow(&t.level, &dummy, cap) && grow(&t.first_child, &dummy, cap) &&
                       grow(&t.n_child, &dummy, cap) && grow(&t.parent, &dummy, cap) &&
                       grow(&t.mom, &dummy, cap) && grow(&t.com, &dummy, cap) &&
                       grow(&t.pp, &dummy, 3 * cap) && grow(&t.nrec, &dummy, cap));
            t.node_cap = (int)cap;
        }
        const int cap = t.node_cap;
        hipLaunchKernelGGL(k_init_words, dim3(1), dim3(64), 0, s, t.word);
        // level L has at most min(n, 8^L) nodes
        auto level_bound = [&](int L) {
            long long b = 1;
            for (int k = 0; k < L && b < n; ++k) b *= 8;
            return (int)std::min<long long>(b, n);
        };
        const int gnodes = std::min(blocks_of(cap, 256), 16 * num_cu);
        unsigned *mask = (unsigned *)t.nc;
        int *sums = t.nc + n, *total = sums + (kLevels + 1) * chunks;
        const dim3 by_chunk(blocks_of(chunks, 4));
        hipLaunchKernelGGL(k_node_mask, by_chunk, dim3(256), 0, s, n, n_leaf, t.key, mask,
                           (int)chunks, sums);
        hipLaunchKernelGGL(k_node_scan, dim3(kLevels + 1), dim3(256), 0, s, (int)chunks, sums, total);
        hipLaunchKernelGGL(k_node_write, by_chunk, dim3(256), 0, s, n, mask, (int)chunks, sums,
                           total, cap, t.begin, t.level, t.first_child, t.n_child, t.parent, t.lvl,
                           t.word);
        hipLaunchKernelGGL(k_node_ends, dim3(gnodes), dim3(256), 0, s, n, t.key, t.lvl, t.word,
                           t.begin, t.level, t.first_child, t.parent, t.count, t.n_child);
        TREE_HIP(hipGetLastError());
        for (int L = kTreeMaxLevel; L >= 0; --L) {
            const int grid = std::min(blocks_of(level_bound(L), 32), 16 * num_cu);
            hipLaunchKernelGGL(k_moments, dim3(grid), dim3(256), 0, s, L, t.lvl, t.word, t.begin,
                               t.count, t.first_child, t.n_child, t.xm, t.mom);
        }
        hipLaunchKernelGGL(k_pseudo, dim3(gnodes), dim3(256), 0, s, t.lvl, t.word, t.mom, t.quad,
                           t.pp, t.com);
        hipLaunchKernelGGL(k_pack_nodes, dim3(gnodes), dim3(256), 0, s, t.lvl, t.word, t.begin,
                           t.count, t.first_child, t.n_child, t.level, t.nrec);
        hipLaunchKernelGGL(k_fill_int, dim3(blocks_of(n, 256)), dim3(256), 0, s, n, t.mark, -1);
        hipLaunchKernelGGL(k_group_mark, dim3(gnodes), dim3(256), 0, s, t.lvl, t.word, t.begin,
                           t.count, t.n_child, t.parent, n_crit, t.mark);
        TREE_HIP(hipGetLastError());
        tb = t.tmp_bytes;
        TREE_HIP(hipcub::DeviceSelect::If(t.tmp, tb, t.mark, t.groups, t.count_out, n,
                                          NonNegative(), s));
        hipLaunchKernelGGL(k_group_info, dim3(std::min(blocks_of(n, 4), 16 * num_cu)), dim3(256), 0,
                           s, t.count_out, t.groups, t.begin, t.count, t.xs, t.ys, t.zs, t.glo,
                           t.ghi, t.items);
        TREE_HIP(hipGetLastError());
        // the one wait of the build: sizes and flags
        hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, s, t.word, t.lvl, t.count_out, page);
        TREE_HIP(hipGetLastError());
        TREE_HIP(hipStreamSynchronize(s));
        const int *lv = page->lvl;
        const unsigned *wv2 = page->word;
        t.n_groups = page->n_groups;
        if (wv2[kWordOverflow]) {
            want = 2LL * cap;
            continue;
        }
        t.n_nodes = lv[kTreeMaxLevel + 1];
        t.depth = 0;
        for (int L = 0; L <= kTreeMaxLevel; ++L) {
            t.level_off[L] = lv[L];
            if (lv[L + 1] > lv[L]) t.depth = L;
        }
        t.level_off[kTreeMaxLevel + 1] = lv[kTreeMaxLevel + 1];
        t.n_leaves = (int)wv2[kWordLeaves];
        t.max_level_nodes = std::max(1, (int)wv2[kWordMaxLevel]);
        break;
    }
    t.built = 1;
    return PGH_OK;
}

int tree_walk(TreeState &t, float theta, int record_src, int num_cu, hipStream_t s,
              std::string &err)
{
    t.walked = 0;
    t.max_frontier = 0;
    t.theta = theta;
    t.record_src = record_src ? 1 : 0;
    t.n_entries = t.interactions = 0;
    if (t.n_groups == 0) {
        t.walked = 1;
        return PGH_OK;
    }
    // (l_L / theta)^2 per level, rounded once from double
    WalkArgs a{};
    for (int L = 0; L <= kTreeMaxLevel; ++L) {
        const double l = std::ldexp((double)t.frame[3], -L);
        a.rc2[L] = theta > 0.f ? (float)((l / theta) * (l / theta)) : INFINITY;
    }
    hipLaunchKernelGGL(k_init_words, dim3(1), dim3(64), 0, s, t.word);
    a.n_groups = t.n_groups;
    a.groups = t.groups;
    a.glo = t.glo;
    a.ghi = t.ghi;
    a.node = t.nrec;
    a.com = t.com;
    a.pp = t.pp;
    a.npp = t.quad ? 3 : 1;
    a.xm = t.xm;
    a.glen = t.glen;
    a.goff = t.goff;
    a.overflow = t.word + 7;
    a.max_frontier = t.word + 8;
    // Pass 1 counts the lists; their scan, the items and the status words
    // come back to the host in one wait.  It runs with the small frontier
    // (LDS for 2 walking waves per SIMD); if a group's frontier outgrew it,
    // it runs again with the large one (1 per SIMD).
    TreeHostPage *page = static_cast<TreeHostPage *>(t.page);
    bool large = false;
    unsigned over = 0, maxf = 0;
    long long total = 0;
    if (t.n_groups > t.host_items_cap) {
        const int cap = t.n_groups + std::min(t.n_groups / 4, INT_MAX - t.n_groups);
        (void)hipHostFree(t.host_items);
        t.host_items = nullptr;
        t.host_items_cap = 0;
        TREE_ALLOC(hipHostMalloc((void **)&t.host_items, sizeof(pgh_item) * (size_t)cap) ==
                   hipSuccess);
        t.host_items_cap = cap;
    }
    for (;;) {
        if (large)
            launch_walk<false, kWalkFrontier>(a, num_cu, s);
        else
            launch_walk<false, kWalkFrontier / 2>(a, num_cu, s);
        TREE_HIP(hipGetLastError());
        size_t tb = t.tmp_bytes;
        TREE_HIP(hipcub::DeviceScan::ExclusiveSum(t.tmp, tb, t.glen, t.goff, t.n_groups + 1, s));
        hipLaunchKernelGGL(k_items_j, dim3(blocks_of(t.n_groups, 256)), dim3(256), 0, s,
                           t.n_groups, t.goff, t.glen, t.word, t.items, t.host_items, page);
        TREE_HIP(hipGetLastError());
        TREE_HIP(hipStreamSynchronize(s));
        over = page->word[7];
        maxf = page->word[8];
        total = page->entries;
        if (!over || large) break;
        large = true;
        hipLaunchKernelGGL(k_init_words, dim3(1), dim3(64), 0, s, t.word);
    }
    if (over) {
        err = "tree walk: a frontier exceeded " + std::to_string(kWalkFrontier) +
              " nodes (theta too small for this tree)";
        return PGH_ERANGE;
    }
    t.max_frontier = (int)maxf;
    if (total > INT_MAX) {
        err = "tree walk: the lists exceed 2^31 - 1 entries";
        return PGH_ERANGE;
    }
    if (total > t.entry_cap) {
        const long long cap = total + total / 4 + 1024;
        long long c1 = 0;
        TREE_ALLOC(grow(&t.xmj, &c1, cap));
        t.entry_cap = cap;
    }
    if (record_src && total > t.src_cap) {
        const long long cap = total + total / 4 + 1024;
        TREE_ALLOC(grow(&t.src, &t.src_cap, cap));
    }
    // The writing pass runs while the caller plans the batched launch from
    // the items (the plan's upload is ordered after it on the stream).
    a.xmj = t.xmj;
    a.src = record_src ? t.src : nullptr;
    if (large)
        launch_walk<true, kWalkFrontier>(a, num_cu, s);
    else
        launch_walk<true, kWalkFrontier / 2>(a, num_cu, s);
    TREE_HIP(hipGetLastError());
    long long inter = 0;
    for (int g = 0; g < t.n_groups; ++g)
        inter += (long long)t.host_items[g].n_i * t.host_items[g].n_j;
    t.n_entries = total;
    t.interactions = inter;
    t.walked = 1;
    return PGH_OK;
}

// The tree force in the input order: particle i's packed result (ax, ay, az,
// phi) sits at its rank inv[i]; a coalesced write of each output array from
// one 16-byte gather.
__global__ void __launch_bounds__(256) k_tree_out(int n, const int *__restrict__ inv,
                                                  const float4 *__restrict__ res, float *ax,
                                                  float *ay, float *az, float *phi)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float4 v = res[inv[i]];
    ax[i] = v.x;
    ay[i] = v.y;
    az[i] = v.z;
    if (phi) phi[i] = v.w;
}

hipError_t launch_tree_outputs(const TreeState &t, float *ax, float *ay, float *az, float *phi,
                               hipStream_t s)
{
    if (t.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tree_out, dim3(blocks_of(t.n, 256)), dim3(256), 0, s, t.n, t.inv, t.res,
                       ax, ay, az, phi);
    return hipGetLastError();
}

// One component (0..3: x, y, z, m) of the packed list entries.
__global__ void __launch_bounds__(256) k_list_component(long long n, const float4 *__restrict__ xmj,
                                                        int comp, float *__restrict__ out)
{
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const float4 v = xmj[e];
    out[e] = comp == 0 ? v.x : comp == 1 ? v.y : comp == 2 ? v.z : v.w;
}

hipError_t launch_list_component(const TreeState &t, int comp, float *out, hipStream_t s)
{
    if (t.n_entries <= 0) return hipSuccess;
    const long long blocks = (t.n_entries + 255) / 256;
    hipLaunchKernelGGL(k_list_component, dim3((unsigned)blocks), dim3(256), 0, s, t.n_entries,
                       t.xmj, comp, out);
    return hipGetLastError();
}

}  // namespace pgh
