// Table force over interaction lists in one persistent launch: the force
// procedure of Sec. 3.4.2 on the (i-group, j-list) items of a tree or TreePM
// code (Sec. 5.1), over the same plans as the batched Newton kernel
// (batch.hip: wave tasks of at most 64 i-particles, pairs of partly filled
// chunks sharing a wave, long lists cut into parts, longest-first sublists).
//
// What differs from the Newton kernel:
//   * KI i-particles per lane (1 or 2).  Each lane reads one j-record from
//     LDS per step and uses it for KI pairs: the j-record broadcast and the
//     table gather share the CU's LDS bandwidth, and with one i-particle per
//     lane the LDS, not the VALU, would bound the pair rate.  A chunk of n
//     i-particles with js lanes per i-particle (chunk_js) runs P = KI js
//     phases of R = 64 / P lanes; lane (phase p, row r) holds the chunk's
//     slots r + k R (k < KI) and takes the list's entries p, p + P, ...  A
//     paired task runs P = KI phases; its first chunk holds rows
//     [0, ceil(n_1 / KI)), the second the rows after them (the planner pairs
//     two chunks only when both fit in that many rows).
//   * The j-tile of a task without a second list is 64 TW records (TW
//     records per lane per tile), so short steps (P = 8) still get long
//     tiles.
//   * Each wave sets its issue priority from the work it has left
//     (set_wave_prio), so the waves of a SIMD finish together instead of in
//     the order they arrived.
//   * The pair arithmetic (table_pair_v) keeps every uniform operand in a
//     VGPR and finds the bin's byte offset with a shift and a mask; the
//     table sits in static LDS (2^TB entries at most), so its base folds
//     into the LDS read's offset field.
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "batch_queue.h"
#include "table_filter.h"
#include "table_pairs.h"

namespace pgh {
namespace {

// plans of at most this many tasks per wave run in the static order
constexpr int kStaticRounds = 4;
// k_batch_table_near evaluates a block of 64 records whole when some lane has
// more candidates than kDirectHits among its 2 x 32 pairs, or kDirectHits1 among
// its 32 of a single column (which break even at a quarter of the pairs inside: 4096
// lists of 32 x 1500 97 us with 12 of 32, 76 with 18), and after one with more than
// kMostHits the next kWholeBlocks without looking (64 x 1500 with every pair inside 182
// -> 158 us, with hardly any 17.3 -> 17.5; with moments or a potential, where it gained
// less than it cost the others, every block is looked at),
constexpr int kDirectHits = 24, kDirectHits1 = 18;
constexpr int kMostHits = 36, kMostHits1 = 22, kWholeBlocks = 7;
// and adds the sums of so many list entries, half of them in a lane, to the outputs.
constexpr int kSegment = 2048;

// The lanes of one task: lane (phase, row) holds slots q + k stride
// (k < KI) of its chunk (i-particles i0 + slot, the chunk's partial-sum
// lanes from lane0), and takes the list's entries phase, phase + P, ...
template <int KI>
struct TaskLanes {
    bool paired, second;
    int plog, P, R, phase, q, stride, nl, i0, lane0;
    int T, nj, ntiles;  // records per tile and list, entries, tiles
    bool act[KI];
    float px[KI], py[KI], pz[KI];
};

// KI i-particles per lane, TW j-records per lane per tile (unpaired tasks),
// 2^TB table entries at most, HT the (H, G1) form, PHI the potential table,
// WPB waves per workgroup (one table copy per workgroup), MOM also the i-side
// moments of the adjoint (table_tail_mom; the paper's form, no potential).
template <int KI, int TW, int TB, bool HT, bool PHI, int WPB, bool MOM = false>
// eight waves per SIMD whatever the workgroup size (64 VGPRs at most)
__global__ void __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_batch_table(BatchArgs a)
{
    static_assert(!MOM || (!HT && !PHI), "moments take the paper's form, no potential");
    constexpr int M = MOM ? 7 : 1;
    using Entry = std::conditional_t<PHI, float4, float2>;
    constexpr int kEntryLog = PHI ? 4 : 3;
    __shared__ Entry stab[1 << TB];
    __shared__ float4 jt[WPB][128];  // a wave's j-tile

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    // Task order: static (few tasks per wave: no atomics, and the next
    // task's fields load while the current task runs) or the sublists.
    const bool stat = a.static_order != 0;
    const TaskStream ts = task_stream(a, WPB);
    const unsigned G = gridDim.x * WPB;
    const unsigned gw = __builtin_amdgcn_readfirstlane(blockIdx.x * WPB + wave);
    const Task *const tbase = stat ? a.tasks : ts.tasks;
    const unsigned n_t = stat ? (unsigned)a.n_tasks : ts.n_tasks;
    unsigned round = 0;
    unsigned t = stat ? static_task(a, 0, gw, G) : first_task(a, WPB, wave);
    const unsigned rounds_g = stat ? static_rounds(n_t, gw, G) : 0u;  // the wave's static tasks
    float4 *tile = jt[wave];

    // j-records of tile tl of a task, TW per lane (a paired task: one of each
    // list); entries past a list's end are zero-mass records far away
    float4 pre[2];
    auto record = [&](int j_off, int n, int j) {
        float4 v = make_float4(kFar, kFar, kFar, 0.f);
        if (j < n) {
            const int jj = j_off + j;
            v = make_float4(a.xj[jj], a.yj[jj], a.zj[jj], a.mj[jj]);
        }
        return v;
    };
    auto load = [&](const Task &tk, const TaskLanes<KI> &L, int tl) {
        if (L.paired) {
            pre[0] = record(tk.j_off, tk.n_j, tl * 64 + lane);
            pre[1] = record(tk.j_off2, tk.n_j2, tl * 64 + lane);
        } else {
#pragma unroll
            for (int w = 0; w < TW; ++w) pre[w] = record(tk.j_off, tk.n_j, tl * L.T + w * 64 + lane);
        }
    };
    auto store = [&](const TaskLanes<KI> &L) {
        tile[lane] = pre[0];
        if (L.paired || TW == 2) tile[64 + lane] = pre[1];
    };
    // lane -> (phase, row) -> (list, slots); issues the task's i-particle
    // loads and the loads of its first tile
    auto begin = [&](const Task &tk) {
        TaskLanes<KI> L;
        L.paired = tk.n_i2 > 0;
        L.plog = (KI == 2 ? 1 : 0) + (L.paired ? 0 : (tk.n_i <= 16 ? 2 : (tk.n_i <= 32 ? 1 : 0)));
        L.P = 1 << L.plog;
        L.R = 64 >> L.plog;
        L.phase = lane >> (6 - L.plog);
        const int row = lane & (L.R - 1);
        L.stride = L.R, L.q = row, L.nl = tk.n_i, L.i0 = tk.i_off, L.lane0 = 0;
        L.second = false;
        if (L.paired) {
            const int ra = (tk.n_i + KI - 1) / KI, rb = (tk.n_i2 + KI - 1) / KI;
            L.second = row >= ra;
            L.stride = L.second ? rb : ra;
            L.q = L.second ? row - ra : row;
            L.nl = L.second ? tk.n_i2 : tk.n_i;
            L.i0 = L.second ? tk.i_off2 : tk.i_off;
            L.lane0 = L.second ? tk.n_i : 0;
        }
#pragma unroll
        for (int k = 0; k < KI; ++k) {
            const int slot = L.q + k * L.stride;
            L.act[k] = L.q < L.stride && slot < L.nl;
            const int i = L.i0 + (L.act[k] ? slot : 0);
            L.px[k] = a.xi[i];
            L.py[k] = a.yi[i];
            L.pz[k] = a.zi[i];
        }
        L.T = L.paired ? 64 : 64 * TW;
        L.nj = L.paired ? max(tk.n_j, tk.n_j2) : tk.n_j;
        L.ntiles = (L.nj + L.T - 1) / L.T;
        load(tk, L, 0);
        return L;
    };

    // The first task's fields, i-particles and first tile are loaded before
    // the table copy, whose latency they share.
    Task tk{};
    TaskLanes<KI> L{};
    if (t < n_t) {
        tk = tbase[t];
        L = begin(tk);
    }
    {
        const int K = 1 << (a.E + a.F);
        const unsigned shift = 23u - (unsigned)a.F;
        if (PHI)
            tables_to_lds<HT>((float4 *)stab, a.table, a.ptable, K, shift);
        else
            table_to_lds<HT>((float2 *)stab, a.table, K, shift);
    }
    const TableConsts kc = table_consts(a.c, a.smax, a.E, a.F, kEntryLog);
    const char *tab = (const char *)stab;
    __syncthreads();  // the only workgroup barrier: waves are independent after it
    if (a.prio_quarter) __builtin_amdgcn_s_setprio(3);

    while (t < n_t) {
        const unsigned tn = stat ? 0u : pop_task(ts, lane);
        // vmcnt(0): the i-particle and first-tile loads (and the ticket's
        // atomic).  Waiting here keeps the compiler from placing a full wait
        // inside the pair loop, where it would also wait for the prefetch of
        // the next tile.
        __builtin_amdgcn_s_waitcnt(0x0F70);
        const unsigned t_next =
            stat ? static_task(a, ++round, gw, G) : __builtin_amdgcn_readfirstlane(tn);
        int fld = 0;
        if (t_next < n_t && lane < 12) fld = ((const int *)(tbase + t_next))[lane];

        float tx[KI], ty[KI], tz[KI], tp[KI];
#pragma unroll
        for (int k = 0; k < KI; ++k) tx[k] = ty[k] = tz[k] = tp[k] = 0.f;
        float tm[M][KI];
#pragma unroll
        for (int c = 0; c < M * KI; ++c) tm[c / KI][c % KI] = 0.f;
        const float4 *src = tile + (L.second ? 64 : 0) + L.phase;
        // the wave's static tasks after this one (round is this task's + 1)
        const unsigned more = stat ? rounds_g - round : 0u;
        for (int tl = 0; tl < L.ntiles; ++tl) {
            // pair-slots left: the task's remaining records times the i-slots
            // each serves (64 over the lanes per i-particle), and the later
            // tasks at the mean size
            set_wave_prio(((unsigned long long)(L.nj - tl * L.T) << (6 - (L.plog - (KI == 2 ? 1 : 0)))) +
                              (unsigned long long)more * a.prio_task,
                          a.prio_quarter);
            wave_sync();  // the previous tile's reads are done
            store(L);
            wave_sync();
            if (tl + 1 < L.ntiles) load(tk, L, tl + 1);
            const int cnt = min(L.T, L.nj - tl * L.T);
            auto step = [&](const float4 p) {
                if constexpr (MOM)
                    table_pairs_mom<KI>(p, L.px, L.py, L.pz, tab, kc, tx, ty, tz, tm);
                else
                    table_pairs_v<KI, HT, PHI>(p, L.px, L.py, L.pz, tab, kc, tx, ty, tz, tp);
            };
            if (cnt == L.T) {
                // a full tile: T / P records per lane with a compile-time
                // stride, so the LDS reads take immediate offsets
                auto full = [&](auto stride_c, auto trips_c) {
                    constexpr int S = decltype(stride_c)::value;
                    constexpr int N = decltype(trips_c)::value;
#pragma unroll 2
                    for (int it = 0; it < N; ++it) step(src[it * S]);
                };
                using std::integral_constant;
                if (L.paired) {
                    full(integral_constant<int, KI>{}, integral_constant<int, 64 / KI>{});
                } else if (L.plog == (KI == 2 ? 1 : 0)) {
                    full(integral_constant<int, KI>{}, integral_constant<int, 64 * TW / KI>{});
                } else if (L.plog == (KI == 2 ? 2 : 1)) {
                    full(integral_constant<int, 2 * KI>{}, integral_constant<int, 32 * TW / KI>{});
                } else {
                    full(integral_constant<int, 4 * KI>{}, integral_constant<int, 16 * TW / KI>{});
                }
            } else {
                const int trips = (cnt + L.P - 1) >> L.plog;
#pragma unroll 2
                for (int it = 0; it < trips; ++it) step(src[it * L.P]);
            }
        }

        // add the phases of each row (lanes row, row + R, ...)
#pragma unroll
        for (int k = 0; k < KI; ++k) {
            for (int d = L.R; d < 64; d <<= 1) {
                tx[k] += __shfl_xor(tx[k], d);
                ty[k] += __shfl_xor(ty[k], d);
                tz[k] += __shfl_xor(tz[k], d);
                if (PHI) tp[k] += __shfl_xor(tp[k], d);
                if constexpr (MOM)
#pragma unroll
                    for (int c = 0; c < 7; ++c) tm[c][k] += __shfl_xor(tm[c][k], d);
            }
        }
        if (L.phase == 0) {
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                if (!L.act[k]) continue;
                const int slot = L.q + k * L.stride;
                if (tk.n_parts <= 1) {
                    const int i = L.i0 + slot;
                    a.ax[i] = tx[k];
                    a.ay[i] = ty[k];
                    a.az[i] = tz[k];
                    if (PHI) a.phi[i] = tp[k];
                    if constexpr (MOM)
#pragma unroll
                        for (int c = 0; c < 7; ++c) a.mom[(size_t)c * a.ni_total + i] = tm[c][k];
                } else {
                    // partial sums of one part of a split j-list; k_combine
                    // adds the parts of the chunk in order after this launch
                    const size_t at = (size_t)(tk.slot + tk.part) * 64 + L.lane0 + slot;
                    a.partial[at] = make_float4(tx[k], ty[k], tz[k], tp[k]);
                    if constexpr (MOM) {
                        a.mpartial[2 * at] = make_float4(tm[0][k], tm[1][k], tm[2][k], tm[3][k]);
                        a.mpartial[2 * at + 1] = make_float4(tm[4][k], tm[5][k], tm[6][k], 0.f);
                    }
                }
            }
        }
        t = t_next;
        if (t < n_t) {
            tk = task_of_fields(fld);
            L = begin(tk);
        }
    }
}

// The same force with the pairs beyond the cutoff left out (table_filter.h).
// A wave takes its task's list SB x 64 records at a time, the next ones in
// flight meanwhile (a record a lane a step ahead left it waiting for memory
// three quarters of the time):
//   * records farther than the cutoff from the box around the chunk's
//     i-particles are dropped, the others packed into the wave's LDS tile;
//   * 64 kept records at a time, the matrix cores form |d|^2 - cutoff^2 with
//     two columns of 32 i-particles (lane l holds l mod 32 and 32 + l mod 32);
//     the signs give each lane a word of candidates per column, half of the
//     rows in lanes < 32, half in the others;
//   * each lane evaluates its own candidates one after another, in FP32 as
//     k_batch_table does, reading each record by its own index.  Where the
//     pairs inside the cutoff are not few (kDirectHits) the 64 records are
//     evaluated whole, and where they are the most the next ones too.
// A paired task is its two chunks in turn.
//
// Per 64 x 64 pairs about 45 vector instructions for the operands, 64 for the
// signs (one to two issue slots each) and four products, and 26 a round of
// candidates, against 64 x 17 before; what is left is the launch, the first
// loads' latency and the rounds (a VALU instruction per SIMD every 10 cycles of
// 4096 lists of 4^3 cells, every 8 of 512 of 8^3, counted).  Measured, per call in
// graphs of twenty, with k_batch_table (KI = 2, TW = 2) and now: 4096 lists of 4^3
// cells 31.3 -> 17.5 us, 512 lists of 8^3 cells 95.5 -> 21.6, with the potential 95 ->
// 24.0; other shapes and densities at table_batch_few.
//
// MOM: also the i-side moments of the adjoint (table_tail_mom).
template <int TB, bool PHI, int WPB, int SB, bool MOM>
__global__ void __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(MOM || WPB > 4 ? 4 : 5, 8)))
k_batch_table_near(BatchArgs a)
{
    static_assert(!MOM || !PHI, "moments come without a potential");
    constexpr bool kLook = MOM || PHI;  // before every block (kMostHits)
    using Entry = std::conditional_t<PHI, float4, float2>;
    __shared__ Entry stab[1 << TB];
    __shared__ float4 jt[WPB][64 * SB];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const bool stat = a.static_order != 0;
    const TaskStream ts = task_stream(a, WPB);
    const unsigned G = gridDim.x * WPB;
    const unsigned gw = __builtin_amdgcn_readfirstlane(blockIdx.x * WPB + wave);
    const Task *const tbase = stat ? a.tasks : ts.tasks;
    const unsigned n_t = stat ? (unsigned)a.n_tasks : ts.n_tasks;
    unsigned round = 0;
    unsigned t = stat ? static_task(a, 0, gw, G) : first_task(a, WPB, wave);
    float4 *tile = jt[wave];

    // an element of a uniform array at a lane's 32-bit offset; the offset is
    // opaque, so that no address of 64 bits per lane and array is kept
    // through the loops
    auto at = [](const float *p, unsigned k) {
        unsigned o = 4u * k;
        asm volatile("" : "+v"(o));
        return *(const float *)((const char *)p + o);
    };
    auto put = [](float *p, unsigned k, float v) {
        unsigned o = 4u * k;
        asm volatile("" : "+v"(o));
        *(float *)((char *)p + o) = v;
    };
    // a chunk's i-particles (slot = lane; past the end the first) and the
    // list's next SB records of this lane (past the end the last)
    float ix, iy, iz;
    float4 pre[SB];
    auto load = [&](int j_off, int n_j, int base) {
#pragma unroll
        for (int s = 0; s < SB; ++s) {
            if (base + 64 * s >= n_j) break;
            const int j = min(base + 64 * s + lane, n_j - 1);
            pre[s] = make_float4(at(a.xj + j_off, j), at(a.yj + j_off, j), at(a.zj + j_off, j),
                                 at(a.mj + j_off, j));
        }
    };
    auto begin = [&](int i_off, int n_i, int j_off, int n_j) {
        const int i = lane < n_i ? lane : 0;
        ix = at(a.xi + i_off, i);
        iy = at(a.yi + i_off, i);
        iz = at(a.zi + i_off, i);
        load(j_off, n_j, 0);
    };

    Task tk{};
    if (t < n_t) {
        tk = tbase[t];
        begin(tk.i_off, tk.n_i, tk.j_off, tk.n_j);
    }
    const int K = 1 << (a.E + a.F);
    if (PHI)
        tables_to_lds<false>((float4 *)stab, a.table, a.ptable, K, 0u);
    else
        table_to_lds<false>((float2 *)stab, a.table, K, 0u);
    // (in SGPRs: the candidates are few and registers are not)
    const unsigned kshift = 23u - (unsigned)a.F;
    const TableConsts kc{a.c, __float_as_uint(a.smax), kshift - (PHI ? 4 : 3),
                         (unsigned)(K - 1) << (PHI ? 4 : 3), ~((1u << kshift) - 1u)};
    const char *tab = (const char *)stab;
    __syncthreads();  // the only workgroup barrier: waves are independent after it
    // whether pairs beyond the cutoff add exactly zero and can be found
    const Entry last = stab[K - 1];
    bool last_zero = last.x == 0.f && last.y == 0.f && filter_cut(a.r2max);
    if constexpr (PHI) last_zero = last_zero && last.z == 0.f && last.w == 0.f;

    while (t < n_t) {
        const unsigned tn = stat ? 0u : pop_task(ts, lane);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), as in k_batch_table
        const unsigned t_next =
            stat ? static_task(a, ++round, gw, G) : __builtin_amdgcn_readfirstlane(tn);
        int fld = 0;
        if (t_next < n_t && lane < 12) fld = ((const int *)(tbase + t_next))[lane];

        const int parts = tk.n_i2 > 0 ? 2 : 1;
        // A list is taken kSegment entries at a time, each of which adds its sums to
        // the outputs, so that FP32 rounding grows with kSegment / 2 and the number
        // of segments, not with the list (400000 neighbours of one mass: 2.0e-3 in
        // one running sum).
        bool again = false;  // of a list begun before
        for (int sub = 0; sub < parts;) {
            const int i_off = sub ? tk.i_off2 : tk.i_off, n_i = sub ? tk.n_i2 : tk.n_i;
            const int j_off = sub ? tk.j_off2 : tk.j_off, n_all = sub ? tk.n_j2 : tk.n_j;
            const int n_j = min(n_all, kSegment);
            if (sub || again) begin(i_off, n_i, j_off, n_j);

            // the box around the chunk (lanes past its end hold its first
            // i-particle), or all space when nothing may be left out
            const bool whole = !last_zero || __any(!ordinary(ix, iy, iz, 0.f));
            const float xl = uniform(whole ? -INFINITY : wave_min(ix)),
                        xh = uniform(whole ? INFINITY : wave_max(ix)),
                        yl = uniform(whole ? -INFINITY : wave_min(iy)),
                        yh = uniform(whole ? INFINITY : wave_max(iy)),
                        zl = uniform(whole ? -INFINITY : wave_min(iz)),
                        zh = uniform(whole ? INFINITY : wave_max(iz));
            const float cx = uniform(whole ? 0.f : 0.5f * (xl + xh)),
                        cy = uniform(whole ? 0.f : 0.5f * (yl + yh)),
                        cz = uniform(whole ? 0.f : 0.5f * (zl + zh));
            const float cut = uniform(whole ? INFINITY : a.r2max);
            const FilterOps cols =
                filter_cols_of(ix, iy, iz, lane < n_i, last_zero, cx, cy, cz, a.r2max);
            float px[2], py[2], pz[2];  // of both columns
            both_halves(ix, px), both_halves(iy, py), both_halves(iz, pz);
            float tx[2] = {0.f, 0.f}, ty[2] = {0.f, 0.f}, tz[2] = {0.f, 0.f}, tp[2] = {0.f, 0.f};
            float tm[MOM ? 7 : 1][2];
#pragma unroll
            for (int c = 0; c < (MOM ? 7 : 1); ++c) tm[c][0] = tm[c][1] = 0.f;
            int blind = 0;  // blocks still to be evaluated whole without a test
            for (int base = 0; base < n_j; base += 64 * SB) {
                wave_sync();  // the previous tile's reads are done
                int kept = 0;
#pragma unroll
                for (int s = 0; s < SB; ++s) {
                    if (base + 64 * s >= n_j) break;
                    // the distance to the box, formed as a pair's |d|^2 is:
                    // each step is monotone, so no pair with the box's
                    // i-particles has a smaller one
                    const float4 v = pre[s];
                    const float ex = __builtin_fmaxf(__builtin_fmaxf(xl - v.x, v.x - xh), 0.f);
                    const float ey = __builtin_fmaxf(__builtin_fmaxf(yl - v.y, v.y - yh), 0.f);
                    const float ez = __builtin_fmaxf(__builtin_fmaxf(zl - v.z, v.z - zh), 0.f);
                    const float r2 =
                        __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex));
                    const bool keep = base + 64 * s + lane < n_j &&
                                      (r2 < cut || !ordinary(v.x, v.y, v.z, v.w));
                    const unsigned long long who = __ballot(keep);
                    if (keep) {
                        const int k = kept + lanes_below(who);
                        tile[(k & ~63) | filter_slot(k & 63)] = v;
                    }
                    kept += __popcll(who);
                }
                wave_sync();
                if (base + 64 * SB < n_j) load(j_off, n_j, base + 64 * SB);

                for (int k0 = 0; k0 < kept; k0 += 64) {
                    const float4 *rows64 = tile + k0;
                    const bool valid = k0 + lane < kept;
                    const float4 *mine = rows64 + (lane & 32);  // this half's rows
                    unsigned m0 = 0, m1 = 0;
                    if (kLook || blind == 0) {
                        const FilterOps rows =
                            filter_rows_of(rows64[filter_slot(lane)], valid, cx, cy, cz);
                        m0 = filter_mask(rows, cols.t[0]);
                        if (n_i > 32) m1 = filter_mask(rows, cols.t[1]);
                        const int hits = __popc(m0) + __popc(m1);
                        const bool most = !kLook && __any(hits > (n_i > 32 ? kMostHits : kMostHits1));
                        if (__any(hits > (n_i > 32 ? kDirectHits : kDirectHits1)))
                            blind = most ? kWholeBlocks + 1 : 1;
                    }
                    if (blind > 0) {
                        --blind;
                        // rows past the last kept one are made far away, massless
                        if (!valid)
                            tile[k0 + filter_slot(lane)] = make_float4(kFar, kFar, kFar, 0.f);
                        wave_sync();
                        const TableConsts kd = table_consts(a.c, a.smax, a.E, a.F, PHI ? 4 : 3);
                        auto pairs = [&](const float4 r, auto n) {
                            constexpr int N = decltype(n)::value;
                            if constexpr (MOM) {
                                float sm[7][N];
#pragma unroll
                                for (int c = 0; c < 7 * N; ++c) sm[c / N][c % N] = tm[c / N][c % N];
                                table_pairs_mom<N>(r, px, py, pz, tab, kd, tx, ty, tz, sm);
#pragma unroll
                                for (int c = 0; c < 7 * N; ++c) tm[c / N][c % N] = sm[c / N][c % N];
                            } else {
                                table_pairs_v<N, false, PHI>(r, px, py, pz, tab, kd, tx, ty, tz, tp);
                            }
                        };
                        if (n_i > 32) {
#pragma unroll MOM ? 1 : 2
                            for (int p = 0; p < 32; ++p)
                                pairs(mine[p], std::integral_constant<int, 2>{});
                        } else {
#pragma unroll 2
                            for (int p = 0; p < 32; ++p)
                                pairs(mine[p], std::integral_constant<int, 1>{});
                        }
                        continue;
                    }
                    auto near = [&](unsigned m, auto q_c) {
                        constexpr int q = decltype(q_c)::value;
                        while (m) {
                            const int p = __builtin_clz(m);
                            m ^= 0x80000000u >> p;
                            const float4 r = mine[p];
                            TableGather<1, PHI> g;
                            table_head<1, false, PHI>(r, px + q, py + q, pz + q, tab, kc, g);
                            if constexpr (MOM) {
                                float sm[7][1];
#pragma unroll
                                for (int c = 0; c < 7; ++c) sm[c][0] = tm[c][q];
                                table_tail_mom<1>(r.w, g, tx + q, ty + q, tz + q, sm);
#pragma unroll
                                for (int c = 0; c < 7; ++c) tm[c][q] = sm[c][0];
                            } else {
                                table_tail<1, PHI>(r.w, g, tx + q, ty + q, tz + q, tp + q);
                            }
                        }
                    };
                    near(m0, std::integral_constant<int, 0>{});
                    near(m1, std::integral_constant<int, 1>{});
                }
            }

            // the two halves' rows; lane l then keeps slot l
            auto slots = [&](const float *v) {
                const float s0 = v[0] + __shfl_xor(v[0], 32), s1 = v[1] + __shfl_xor(v[1], 32);
                return lane < 32 ? s0 : s1;
            };
            const float ox = slots(tx), oy = slots(ty), oz = slots(tz);
            const float op = PHI ? slots(tp) : 0.f;
            float om[MOM ? 7 : 1];
#pragma unroll
            for (int c = 0; c < (MOM ? 7 : 1); ++c) om[c] = MOM ? slots(tm[c]) : 0.f;
            if (lane < n_i) {
                auto out = [&](float *p, float v) {
                    p += i_off;
                    put(p, lane, again ? at(p, lane) + v : v);
                };
                if (tk.n_parts <= 1) {
                    out(a.ax, ox);
                    out(a.ay, oy);
                    out(a.az, oz);
                    if (PHI) out(a.phi, op);
                    if constexpr (MOM) {
#pragma unroll
                        for (int c = 0; c < 7; ++c) out(a.mom + (size_t)c * a.ni_total, om[c]);
                    }
                } else {
                    // partial sums of one part of a split j-list (k_combine)
                    const size_t q = (size_t)(tk.slot + tk.part) * 64 + (sub ? tk.n_i : 0) + lane;
                    auto add = [&](float4 *p, float4 v) {
                        if (again) v.x += p->x, v.y += p->y, v.z += p->z, v.w += p->w;
                        *p = v;
                    };
                    add(a.partial + q, make_float4(ox, oy, oz, op));
                    if constexpr (MOM) {
                        add(a.mpartial + 2 * q, make_float4(om[0], om[1], om[2], om[3]));
                        add(a.mpartial + 2 * q + 1, make_float4(om[4], om[5], om[6], 0.f));
                    }
                }
            }
            again = n_all > kSegment;
            if (!again)
                ++sub;
            else if (sub)
                tk.j_off2 += kSegment, tk.n_j2 -= kSegment;
            else
                tk.j_off += kSegment, tk.n_j -= kSegment;
        }
        t = t_next;
        if (t < n_t) {
            tk = task_of_fields(fld);
            begin(tk.i_off, tk.n_i, tk.j_off, tk.n_j);
        }
    }
}

using TableKernel = void (*)(BatchArgs);

// A kernel of a variant for a table of 2^tb nodes, and its waves per
// workgroup.  The table's LDS bounds the workgroups per CU, so larger tables
// take wider workgroups whatever the variant's own width: up to 2^10 nodes
// the variant's; beyond 16 waves, two workgroups per CU up to 2^12 (32 KiB; one
// with the potential, 64 KiB), one beside the largest tables (128 KiB at 2^14,
// or at 2^13 with the potential), where 16 j-tiles of 2 KiB fill the 160 KiB of a
// CU.  With its own two waves per workgroup a variant would leave SIMDs idle
// there.
constexpr int kWideWaves = 16;

struct TableKernelPick {
    TableKernel k;
    int wpb;
};

template <int KI, int TW, bool HT, int WPB>
TableKernelPick pick(int tb, bool phi)
{
    if (tb <= 10)
        return {phi ? k_batch_table<KI, TW, 10, HT, true, WPB>
                    : k_batch_table<KI, TW, 10, HT, false, WPB>, WPB};
    if (tb <= 12)
        return {phi ? k_batch_table<KI, TW, 12, HT, true, kWideWaves>
                    : k_batch_table<KI, TW, 12, HT, false, kWideWaves>, kWideWaves};
    return {phi ? k_batch_table<KI, TW, 13, HT, true, kWideWaves>
                : k_batch_table<KI, TW, 14, HT, false, kWideWaves>, kWideWaves};
}

// The variant that finds the pairs inside the cutoff first: two columns of
// i-particles per lane, as many records per lane and tile (SB) as registers and,
// beside the largest tables, LDS leave room for, four waves (16 beside tables of
// more than 2^10 nodes).
TableKernelPick pick_near(int tb, bool phi)
{
    if (tb <= 10)
        return {phi ? k_batch_table_near<10, true, 4, 2, false>
                    : k_batch_table_near<10, false, 4, 4, false>, 4};
    if (tb <= 12)
        return {phi ? k_batch_table_near<12, true, kWideWaves, 2, false>
                    : k_batch_table_near<12, false, kWideWaves, 2, false>, kWideWaves};
    return {phi ? k_batch_table_near<13, true, kWideWaves, 2, false>
                : k_batch_table_near<14, false, kWideWaves, 2, false>, kWideWaves};
}

struct TableBatchVariant {
    const char *name;
    int wpb;  // waves per workgroup (tables of at most 2^10 nodes)
    TableKernelPick (*pick)(int tb, bool phi);
};

// The tile shapes the autotuner chooses among: i-particles per lane (KI),
// j-records per lane per tile (TW), waves per workgroup, the table form, and "near", which evaluates the pairs inside
// the cutoff only.  The "htab" variants keep the (H, G1)
// form in LDS (two instructions fewer per pair): the same interpolant with
// one more FP32 rounding per node, of H_k = G0_k - G1_k s_k, which is
// relative to G1_k s_k rather than to g; near rcut, where g goes to zero,
// that rounding can be a large part of the little force there, so these
// variants are parity-checked against the oracle's (H, G1) table and, for the
// method's accuracy, against the analytic force.
const TableBatchVariant kTableBatchVariants[] = {
    {"ki=1 tw=1 wg=4", 4, pick<1, 1, false, 4>},
    {"ki=2 tw=1 wg=4", 4, pick<2, 1, false, 4>},
    {"ki=2 tw=2 wg=4", 4, pick<2, 2, false, 4>},
    {"ki=1 tw=1 wg=16", 16, pick<1, 1, false, 16>},
    {"ki=2 tw=2 wg=16", 16, pick<2, 2, false, 16>},
    {"near", 4, pick_near},
    {"ki=2 tw=1 wg=4 htab", 4, pick<2, 1, true, 4>},
    {"ki=2 tw=2 wg=4 htab", 4, pick<2, 2, true, 4>},
    {"ki=2 tw=2 wg=2 htab", 2, pick<2, 2, true, 2>},
};
constexpr int kPaperVariant = 2, kNearVariant = 5;
constexpr int kNumTableBatchVariants = sizeof(kTableBatchVariants) / sizeof(kTableBatchVariants[0]);

int resident_blocks(TableKernel k, int wpb)
{
    static std::mutex mu;
    static std::map<const void *, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find((const void *)k);
    if (it != cache.end()) return it->second;
    int n = 0;
    hipFuncAttributes f{};
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, 64 * wpb, 0) != hipSuccess || n < 1)
        n = 1;
    // LDS is given out in steps of 1280 bytes, which that count may not know: a
    // workgroup too many per CU runs after all others (moments of 20000 lists of 8 x
    // 300, 12288 bytes of LDS: 13 workgroups 84 us, 12 60 us)
    if (hipFuncGetAttributes(&f, (const void *)k) == hipSuccess && f.sharedSizeBytes > 0)
        n = std::max(1, std::min(n, 163840 / (((int)f.sharedSizeBytes + 1279) / 1280 * 1280)));
    cache[(const void *)k] = n;
    return n;
}

}  // namespace

int table_batch_variants() { return kNumTableBatchVariants; }

const char *table_batch_variant_name(int v)
{
    return (v >= 0 && v < kNumTableBatchVariants) ? kTableBatchVariants[v].name : nullptr;
}

// The near kernel pays per list entry and column of 32 i-particles, whatever the
// chunk holds and wherever most pairs are; k_batch_table gives a chunk of at most
// 16 four times the lanes.  us a call of 4096 lists of n_i x 1500 with 1, 10, 25 and
// 100% of the pairs inside, k_batch_table (much alike for all) and near: n_i = 16 41:
// 35, 56, 74, 95; 32 75: 38, 58, 77, 94; 64 140: 49, 86, 146, 158; 200 400: 149, 269,
// 401, 510.  So lists of few i-particles, as of single cells, take the former: up to
// 1.2 times the time with hardly any pair inside, never 2.3 times with many.
// Which pairs are inside isn't known before the call: lists of more i-particles pay
// 1.1 to 1.3 times the former's time where half of the pairs or more are (or a table
// whose last node is not zero makes every pair count; with fewer tasks than SIMDs more:
// 300 lists of 64 x 400 24 us, 13 the former), against a half to a third of it with one
// in a hundred (there 10); the tuner (pgh_autotune_plan) times both.
bool table_batch_few(long long n_rows, long long n_chunks) { return n_rows <= 16 * n_chunks; }

int table_batch_default(bool few) { return few ? kPaperVariant : kNearVariant; }

bool table_batch_near(int v) { return v == kNearVariant; }

// The pair-slot figures of set_wave_prio: a quarter of the plan's
// interactions per wave of the launch, and its mean task.
static void set_prio_args(BatchArgs &a)
{
    const unsigned long long inter = a.interactions > 0 ? (unsigned long long)a.interactions : 0ull;
    a.prio_quarter = inter / (4ull * (unsigned long long)std::max(1, a.n_waves));
    a.prio_task = inter / (unsigned long long)std::max(1, a.n_tasks);
}

hipError_t launch_table_batch_moments(const BatchArgs &a0, bool few, int num_cu, hipStream_t s)
{
    if (a0.n_tasks <= 0) return hipSuccess;
    const int tb = a0.E + a0.F;
    // (k_batch_table here with one i-particle per lane, as the seven moments
    // take registers, and for small tables two waves per workgroup, six per SIMD)
    const int wpb = tb <= 10 ? few ? 2 : 4 : kWideWaves;
    const TableKernel k =
        few ? tb <= 10   ? k_batch_table<1, 2, 10, false, false, 2, true>
              : tb <= 12 ? k_batch_table<1, 2, 12, false, false, kWideWaves, true>
                         : k_batch_table<1, 2, 13, false, false, kWideWaves, true>
        : tb <= 10 ? k_batch_table_near<10, false, 4, 4, true>
        : tb <= 12 ? k_batch_table_near<12, false, kWideWaves, 2, true>
                   : k_batch_table_near<13, false, kWideWaves, 2, true>;
    BatchArgs a = a0;
    a.phi = nullptr;
    a.ptable = nullptr;
    const int cap = num_cu * resident_blocks(k, wpb);
    const int blocks = std::max(a.nq, std::min(cap, (a.n_tasks + wpb - 1) / wpb));
    a.n_waves = blocks * wpb;
    a.static_order = (long long)a.n_tasks <= kStaticRounds * (long long)a.n_waves ? 1 : 0;
    set_prio_args(a);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(64 * wpb), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.n_chunks == 0) return e;
    return launch_combine(a, false, s);
}

hipError_t launch_table_batch(const BatchArgs &a0, int variant, int num_cu, hipStream_t s)
{
    if (a0.n_tasks <= 0) return hipSuccess;
    if (variant < 0 || variant >= kNumTableBatchVariants) variant = kNearVariant;
    const bool phi = a0.phi && a0.ptable;
    const TableKernelPick pk = kTableBatchVariants[variant].pick(a0.E + a0.F, phi);
    const TableKernel k = pk.k;
    const int wpb = pk.wpb;
    BatchArgs a = a0;
    // one resident wave of workgroups, or fewer when there are fewer tasks
    // than waves; at least one workgroup per task sublist
    const int cap = num_cu * resident_blocks(k, wpb);
    const int blocks = std::max(a.nq, std::min(cap, (a.n_tasks + wpb - 1) / wpb));
    a.n_waves = blocks * wpb;
    a.static_order = (long long)a.n_tasks <= kStaticRounds * (long long)a.n_waves ? 1 : 0;
    set_prio_args(a);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(64 * wpb), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.n_chunks == 0) return e;
    return launch_combine(a, phi, s);
}

}  // namespace pgh
