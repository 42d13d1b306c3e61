// Core and shell lists (Sec. 2.3): C(i) = {j != i : r_ij <= r_core} and
// S(i) = {j : r_core < r_ij <= r_shell}, same-molecule pairs removed, in the
// canonical order "stencil cell offset (dz, dy, dx) lexicographic, then the
// atoms of each cell in cell order (by fixed-point x coordinate, then id)".
// One traversal of the shell stencil yields both lists: the 27 core cells are
// visited in their own lexicographic order inside it. Membership is exact:
// it is that of the uint64 squared separation in quanta of L / 2^32 against
// the integer thresholds. Dense cells take the block form (k_list_blocks.hip),
// dilute ones the lane-per-atom form below.
//
// Layout: fixed-capacity rows (row k of atom k in cell order), entries are
// cell-sorted atom indices. Counts beyond the capacity are still counted, so
// the host can grow the rows and rebuild.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "irbe_device.hpp"
#include "irbe_internal.hpp"

namespace irbe {

constexpr int kListWave = 64;
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Integer bounds on an approximate squared separation d2: d2 < *_in proves
// membership of the ball, d2 > *_out proves the opposite. PackedBounds for
// the packed 16-bit coordinates.
template <typename T>
struct Bounds {
    T core_in, core_out, shell_in, shell_out, lo_in, lo_out;
};
using PackedBounds = Bounds<uint32_t>;

__device__ __forceinline__ int wrap(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

// Squared separation of two packed positions (x | y << 16, z) minus t: exact in
// the 16-bit units (differences modulo 2^16), saturated to 32 bits.
__device__ __forceinline__ int d2_minus(uint32_t cxy, uint32_t cz, uint32_t axy, uint32_t az, int t)
{
    const s16x2 dxy = __builtin_bit_cast(s16x2, cxy) - __builtin_bit_cast(s16x2, axy);
    const int dz = (short)(cz - az);
    return __builtin_amdgcn_sdot2(dxy, dxy, dz * dz - t, true);
}

// bits shifted up by one with the sign of v below.
__device__ __forceinline__ uint32_t shift_sign(uint32_t bits, int v)
{
    return __builtin_amdgcn_alignbit(bits, (uint32_t)v, 31);
}

// Lanes with p set (a wave-uniform mask).
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// The list lengths of atom k: the stored lengths never exceed the row
// capacities, so that every reader stays inside its rows; a longer list sets
// its bit in the error word (the rows then hold its first entries only) and its
// true length still reaches maxcnt, from which the host grows the rows.
template <int MODE>
__device__ __forceinline__ void store_counts(int k, int cc, int cs, int cap_core, int cap_shell,
                                             int32_t* __restrict__ ncore, int32_t* __restrict__ nshell,
                                             uint32_t* __restrict__ err)
{
    if (MODE != kListsFull) {
        ncore[k] = min(cc, cap_core);
        if (cc > cap_core) atomicOr(err, ERR_CORE_CAP);
    } else {
        ncore[k] = cc;
    }
    if (MODE != kListsCoreOnly) {
        nshell[k] = min(cs, cap_shell);
        if (cs > cap_shell) atomicOr(err, ERR_SHELL_CAP);
    }
}

// ---------------------------------------------------------------------------
// Lane-per-atom form, for dilute systems (a few atoms per cell, e.g. the
// primitive-model electrolytes) with cells narrower than the box
// (2R + 1 <= n_c). The same lists in the same order as the block form, whose
// blocks of 32 atoms are far longer than the list radius there; here one wavefront
// takes a run of up to 64 consecutive atoms of one cell row, one atom per lane (the
// row's atoms in equal runs: groups of a fixed number of cells overflowed 64 atoms
// one time in four, for a second pass of a few).
// For every stencil row (dz, dy) the union of the atoms' x ranges is staged in
// LDS. The first atom and atom count of every row's union (two index
// ranges at most) are loaded once per run into a table held in registers,
// so that a row's cell starts and the records of its first tile are loaded in
// one memory round trip, issued before the pruning of the rows that follow.
// Each lane computes its own cell range in the union (row pruning, in cell edges
// and FP32 with a margin) and the lanes then walk their ranges in lockstep, lane a
// testing its k-th candidate at step k and shifting the sign of squared separation
// minus bound into bit masks: no branch per candidate. Candidates between two
// bounds take the exact test on full positions read from memory; then each lane
// appends its bits, four at a time, to a stage in LDS, from which full segments go
// to its list row. What bounds it: the vector instructions (260 per atom, 70 % of
// the issue slots) and the latency of the 48 rows' serial chain; segments of 16 bytes
// were written twice to memory (1.35 GB against 0.73), as the open lines of all
// wavefronts exceed the L2. 10^6 ions, 1.28 per cell, 136 + 5 members: 880 -> 705 us,
// with a skin 1,060 -> 730 us.
// ---------------------------------------------------------------------------
constexpr int kLaneTile = 128;           // staged candidates per pass of a row
constexpr int kLanePass = 24;            // candidates per pass of a row's bits
constexpr int kSeg = 16;                 // entries per stored segment (64 bytes)
constexpr int kAppend = 4;               // entries appended between two looks for full segments
constexpr int kStage = kSeg + 3;         // a lane's staged entries (an odd stride: conflict-free lanes)
// Margin of the row pruning in cell edges, far above the rounding of its FP32
// arithmetic (below 1e-5 for offsets of up to 11 cells): it never drops a member.
constexpr float kPruneMargin = 1e-4f;

// A stencil row of the lane-per-atom kernel as loaded: its union's two segments
// (first atom and atoms of A; first atom of B; atoms of both), this lane's raw
// cell start in the union and the records of its first tile.
struct RowLoad {
    int jA, nA, jB, total;
    int cst;
    u32x4 rec[kLaneTile / kListWave];
};

// (six wavefronts per SIMD, what the stage leaves of LDS: the register bounds of seven and eight spill)
template <int MODE>
__global__ __launch_bounds__(kListWave, 6) void k_build_lists_lanes(
    int n_c, int lo, int hi, int G, int parts, int seg, PackedBounds tb, uint64_t t_core, uint64_t t_lo, uint64_t t_shell, float r2_cells, bool excl,
    const uint4* __restrict__ spos, const u32x4* __restrict__ spk, const int32_t* __restrict__ cell_start,
    int cap_core, int cap_shell, int32_t* __restrict__ core, int32_t* __restrict__ ncore,
    int32_t* __restrict__ shell, int32_t* __restrict__ nshell, int32_t* __restrict__ maxcnt,
    uint32_t* __restrict__ err)
{
    __shared__ uint2 trec[kLaneTile + kLanePass];     // packed x | y, packed z
    __shared__ uint32_t tid[kLaneTile + kLanePass];   // exclusion id
    __shared__ int32_t stage[kListWave * kStage];
    __shared__ int32_t tcs[64];                    // union positions of the row's cells (segment A, then B)
    const int lane = threadIdx.x;
    // bounds relative to the first impossible squared separation of the list that is
    // appended (the core list or the shell or full list)
    constexpr bool kTwoLists = MODE == kListsSplit || MODE == kListsSplitSkin;
    const int t_out = (int)(MODE == kListsCoreOnly ? tb.core_out : tb.shell_out) + 1;
    const int t_width = t_out - (int)(MODE == kListsCoreOnly ? tb.core_in : tb.shell_in);
    const int c_off = t_out - ((int)tb.core_out + 1), c_width = (int)tb.core_out + 1 - (int)tb.core_in;
    const int l_off = t_out - ((int)tb.lo_out + 1), l_width = (int)tb.lo_out + 1 - (int)tb.lo_in;
    const int span = hi - lo + 1;
    const int g = (int)xcd_block(blockIdx.x, gridDim.x);
    const int rowid = g / parts;
    const int cz = rowid / n_c, cy = rowid % n_c;
    const int home = (cz * n_c + cy) * n_c;
    const int r0 = cell_start[home], r1 = cell_start[home + n_c];
    int32_t* const mine_st = stage + lane * kStage;
    const int nrows = span * span;  // at most 2 * kListWave (checked at the launch)
    // the row's atoms in equal runs of at most 64 (seg = 0), this wavefront taking run part,
    // part + parts, ..., or those of seg consecutive cells per wavefront
    const int runs = (r1 - r0 + kListWave - 1) / kListWave;
    const int run = runs > 0 ? (r1 - r0 + runs - 1) / runs : 0;
    auto part_start = [&](int q) { return seg > 0 ? cell_start[home + min(q * seg, n_c)] : min(r0 + q * run, r1); };
    // (the last parts are often empty: they rotate with the row, because consecutive workgroups
    // go to the shader engines in turn, and four parts in a fixed order left one of them idle)
    int part = (g - rowid * parts + rowid) % parts;
    auto cell_of = [&](uint32_t x) __attribute__((always_inline)) {
        return (int)(((uint64_t)x * (uint32_t)n_c) >> 32);
    };
    int maxc = 0, maxs = 0;
    for (int s = part_start(part), e = part_start(part + 1); s < e;) {
        // the atoms from s on, one per lane, whose cells' union fits (all of the run but in sparse rows)
        const int x0 = cell_of(spos[s].x);
        const int a1 = min(min(e, s + kListWave), cell_start[home + min(x0 + G, n_c)]);
        const int span_u = cell_of(spos[a1 - 1].x) - x0 + span;  // cells of the union x range
        const int xu0 = wrap(x0 + lo, n_c);                      // first cell of the union
        const int lenA = min(span_u, n_c - xu0);                 // cells before the wrap
        // every stencil row's union: first atom and atom count of segment A (cells
        // xu0 .. xu0 + lenA - 1) and of segment B (cells 0 .. lenB - 1, past the wrap),
        // row ri = (dz, dy) = (lo + ri / span, lo + ri % span) in lane ri % 64 of
        // rtab[ri / 64], loaded once for the run
        const int lenB = span_u - lenA;
        int4 rtab[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ri = h * kListWave + lane;
            rtab[h] = make_int4(0, 0, 0, 0);
            if (ri < nrows) {
                const int row = (wrap(cz + lo + ri / span, n_c) * n_c + wrap(cy + lo + ri % span, n_c)) * n_c;
                const int ja = cell_start[row + xu0], jb = cell_start[row];
                rtab[h] = make_int4(ja, cell_start[row + xu0 + lenA] - ja, jb, lenB > 0 ? cell_start[row + lenB] - jb : 0);
            }
        }
        // a row's union from the table, this lane's cell start in it and the records of
        // its first tile, issued together (one memory round trip)
        auto row_load = [&](int ri, int dz, int dy) __attribute__((always_inline)) {
            RowLoad d;
            const int h = ri >> 6, rl = ri & (kListWave - 1);
            d.jA = __builtin_amdgcn_readlane(h ? rtab[1].x : rtab[0].x, rl);
            d.nA = __builtin_amdgcn_readlane(h ? rtab[1].y : rtab[0].y, rl);
            d.jB = __builtin_amdgcn_readlane(h ? rtab[1].z : rtab[0].z, rl);
            d.total = d.nA + __builtin_amdgcn_readlane(h ? rtab[1].w : rtab[0].w, rl);
            const int row = (wrap(cz + dz, n_c) * n_c + wrap(cy + dy, n_c)) * n_c;
            // (every lane loads, from an index inside the arrays, so that no load sits
            // in a branch and the waits for these registers can be counted exactly;
            // lanes past the union or the tile do not use theirs)
            const int lc = min(lane, span_u);
            d.cst = cell_start[lc < lenA ? row + xu0 + lc : row + lc - lenA];
            const int cnt0 = min(kLaneTile, d.total);
#pragma unroll
            for (int q = 0; q < kLaneTile / kListWave; ++q) {
                const int t = q * kListWave + lane;
                d.rec[q] = spk[t < cnt0 ? (t < d.nA ? d.jA + t : d.jB + (t - d.nA)) : s];
            }
            return d;
        };
        const int k = s + lane;
        const bool act = k < a1;
        const uint4 si = act ? spos[k] : make_uint4(0, 0, 0, 0);
        const int ti = act ? cell_of(si.x) - x0 : 0;  // lane's home cell from x0 on
        const u32x4 pk = act ? spk[k] : u32x4{0, 0, 0, 0};  // packed x | y, z, exclusion id
        const uint32_t axy = pk.x, az = pk.y, amol = pk.z;
        int32_t* const crow = core + (int64_t)k * cap_core;
        int32_t* const srow = shell + (int64_t)k * cap_shell;
        int cc = 0, cs = 0;  // list lengths so far (cs: without the staged entries)
        int wait = 0;        // staged entries (fewer than kSeg between the appends)
        // the atom in its home cell, in cell edges (x with the margin of either side)
        const float fx_lo = (float)(si.x * (uint32_t)n_c) * 0x1p-32f - kPruneMargin, fx_hi = fx_lo + 2.0f * kPruneMargin;
        const float fy = (float)(si.y * (uint32_t)n_c) * 0x1p-32f, fz = (float)(si.z * (uint32_t)n_c) * 0x1p-32f;
        const int t0 = ti - lo;
        // distance from the slab of cells at offset d
        auto gap = [](float f, int d) __attribute__((always_inline)) {
            const float t = (float)d - f;
            return fmaxf(fmaxf(t, -1.0f - t), 0.0f);
        };
        auto slab = [&](int dz) __attribute__((always_inline)) {
            const float g = gap(fz, dz);
            return act ? r2_cells - g * g : -1.0f;
        };
        // the stencil rows in lexicographic order: row ri = (dz, dy), the squared radius left
        // in slab dz, and the lane's range in the row, cells [u_lo, u_hi] of the union
        struct Row {
            int ri, dz, dy;
            float left;
            int u_lo, u_hi;
            bool need;
        };
        // moves on to the first row that some lane needs (ri = nrows: none)
        auto seek = [&](Row& w) __attribute__((always_inline)) {
            for (; w.ri < nrows; ++w.ri) {
                if (w.dy > hi) {
                    w.dy = lo;
                    ++w.dz;
                    w.left = slab(w.dz);
                }
                const int dy = w.dy++;
                if (MODE == kListsCoreOnly && (w.dz < -1 || w.dz > 1 || dy < -1 || dy > 1)) continue;
                const float g = gap(fy, dy);
                const float rem = w.left - g * g;
                w.need = rem >= 0.0f;
                if (ballot(w.need) != 0) {
                    const float ext = __builtin_amdgcn_sqrtf(rem);
                    w.u_lo = t0 + max((int)floorf(fx_lo - ext), lo);
                    w.u_hi = t0 + min((int)floorf(fx_hi + ext), hi);
                    return;
                }
            }
        };
        Row next{0, lo, lo, slab(lo), 0, 0, false};
        seek(next);
        while (next.ri < nrows) {
            // the row's loads are in flight while the next needed row is found
            const int dz = next.dz, dy = next.dy - 1, u_lo = next.u_lo, u_hi = next.u_hi;
            const bool need = next.need;
            const RowLoad cur = row_load(next.ri, dz, dy);
            ++next.ri;
            seek(next);
            const bool core_row = MODE != kListsFull && dz >= -1 && dz <= 1 && dy >= -1 && dy <= 1;
            const int jA = cur.jA, nA = cur.nA, jB = cur.jB, total = cur.total;
            // (LDS accesses of the one wavefront of the workgroup take effect in
            // order: the previous row's reads precede these writes)
            if (lane <= span_u) tcs[lane] = cur.cst - (lane < lenA ? jA : jB - nA);
#pragma unroll
            for (int h = 0; h < kLaneTile / kListWave; ++h) {
                // (past the union: values that no lane's range covers)
                trec[h * kListWave + lane] = make_uint2(cur.rec[h].x, cur.rec[h].y);
                if (excl) tid[h * kListWave + lane] = cur.rec[h].z;
            }
            asm volatile("" ::: "memory");
            const int p_lo = need ? tcs[u_lo] : 0;
            const int p_hi = need ? tcs[u_hi + 1] : 0;
            for (int base = 0; base < total; base += kLaneTile) {
                const int cnt = min(kLaneTile, total - base);
                if (base > 0) {
                    // a row longer than one tile (crowded cells): its later tiles
                    __syncthreads();
                    for (int t = lane; t < cnt; t += kListWave) {
                        const int p = base + t;
                        const int j = p < nA ? jA + p : jB + (p - nA);
                        const u32x4 r = spk[j];
                        trec[t] = make_uint2(r.x, r.y);
                        tid[t] = r.z;
                    }
                    __syncthreads();
                }
                // this tile's part of the range, in tile positions
                const int s0 = need ? max(p_lo, base) - base : 0;
                const int len = need ? max(min(p_hi, base + cnt) - base - s0, 0) : 0;
                for (int c0 = 0; ballot(len > c0) != 0; c0 += kLanePass) {
                    // this pass's candidates in bits: the sign of the squared separation minus
                    // each bound is shifted in
                    const int mine = min(max(len - c0, 0), kLanePass);
                    const int sp = mine > 0 ? s0 + c0 : 0;  // (reads end before tile position kLaneTile + kLanePass)
                    int done = 0;
                    uint32_t in_p = 0, in_d = 0, co_p = 0, co_d = 0, lo_p = 0, lo_d = 0;
                    auto candidates = [&](auto with_core, auto with_excl) __attribute__((always_inline)) {
                        do {
                            uint2 r[4];
                            uint32_t id[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                r[u] = trec[sp + done + u];
                                if constexpr (decltype(with_excl)::value) id[u] = tid[sp + done + u];
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                // squared separation - t_out, saturating
                                int d = d2_minus(r[u].x, r[u].y, axy, az, t_out);
                                if constexpr (decltype(with_excl)::value) d = id[u] != amol ? d : INT32_MAX;
                                in_p = shift_sign(in_p, d);
                                in_d = shift_sign(in_d, d + t_width);
                                if constexpr (decltype(with_core)::value) {
                                    const int c = __builtin_elementwise_add_sat(d, c_off);
                                    co_p = shift_sign(co_p, c);
                                    co_d = shift_sign(co_d, c + c_width);
                                    if (MODE == kListsSplitSkin) {
                                        const int l = __builtin_elementwise_add_sat(d, l_off);
                                        lo_p = shift_sign(lo_p, l);
                                        lo_d = shift_sign(lo_d, l + l_width);
                                    }
                                }
                            }
                            done += 4;
                        } while (done < kLanePass && ballot(mine > done) != 0);
                    };
                    using yes = std::true_type;
                    using no = std::false_type;
                    if (excl) {
                        if (kTwoLists && core_row) candidates(yes{}, yes{});
                        else candidates(no{}, yes{});
                    } else {
                        if (kTwoLists && core_row) candidates(yes{}, no{});
                        else candidates(no{}, no{});
                    }
                    // the first candidate to the lowest bit
                    uint32_t valid = (1u << mine) - 1u;
                    if (!excl && dz == 0 && dy == 0) {
                        // without excluded pairs only the atom itself is no candidate
                        const int self = (k >= jA && k < jA + nA ? k - jA : k - jB + nA) - base - sp;
                        if (self >= 0 && self < mine) valid &= ~(1u << self);
                    }
                    const int down = 32 - done;
                    in_p = (__builtin_bitreverse32(in_p) >> down) & valid;
                    in_d = (__builtin_bitreverse32(in_d) >> down) & in_p;
                    co_p = (__builtin_bitreverse32(co_p) >> down) & valid;
                    co_d = (__builtin_bitreverse32(co_d) >> down) & co_p;
                    lo_p = (__builtin_bitreverse32(lo_p) >> down) & valid;
                    lo_d = (__builtin_bitreverse32(lo_d) >> down) & lo_p;
                    // certain members, and the candidates between two bounds (cells two or more
                    // apart are farther than the core radius: the other rows have no core bound)
                    uint32_t in_list = MODE == kListsSplitSkin ? in_d & ~lo_p : in_d & ~co_p;
                    uint32_t in_core = co_d;
                    uint32_t amb = (in_p & ~in_d) | (co_p & ~co_d) | (lo_p & ~lo_d);
                    // sorted index of candidate p: p + jdA before the segments' border, p + jdB from it on
                    const int border = nA - base - sp, jdA = jA + base + sp, jdB = jB + base + sp - nA;
                    while (ballot(amb != 0) != 0) {
                        if (amb != 0) {
                            // between the bounds: the exact test on full positions decides
                            const int p = __builtin_ctz(amb);
                            const uint32_t bit = amb & -amb;
                            amb ^= bit;
                            const uint4 sj = spos[p + (p < border ? jdA : jdB)];
                            const int32_t dx = (int32_t)(sj.x - si.x);
                            const int32_t dy2 = (int32_t)(sj.y - si.y);
                            const int32_t dz2 = (int32_t)(sj.z - si.z);
                            const uint64_t d2x = (uint64_t)((int64_t)dx * dx) + (uint64_t)((int64_t)dy2 * dy2) +
                                                 (uint64_t)((int64_t)dz2 * dz2);
                            const bool c = d2x <= t_core;
                            const bool l = MODE == kListsCoreOnly ? c
                                           : d2x <= t_shell && (MODE == kListsFull ||
                                                                (MODE == kListsSplitSkin ? d2x > t_lo : !c));
                            in_list = l ? in_list | bit : in_list & ~bit;
                            if (kTwoLists) in_core = c && core_row ? in_core | bit : in_core & ~bit;
                        }
                    }
                    uint32_t to_core = MODE == kListsCoreOnly ? in_list : in_core;
                    while (MODE != kListsFull && ballot(to_core != 0) != 0) {
                        if (to_core != 0) {
                            const int p = __builtin_ctz(to_core);
                            to_core &= to_core - 1u;
                            if (cc < cap_core) crow[cc] = p + (p < border ? jdA : jdB);
                            ++cc;
                        }
                    }
                    int left = MODE != kListsCoreOnly ? __popc(in_list) : 0;
                    while (MODE != kListsCoreOnly && ballot(left > 0) != 0) {
                        int32_t* const at = mine_st + wait;
#pragma unroll
                        for (int u = 0; u < kAppend; ++u) {
                            // (a lane with none left fills unused places)
                            const int p = __builtin_ctz(in_list | 0x80000000u);
                            at[u] = p + (p < border ? jdA : jdB);
                            in_list &= in_list - 1u;
                        }
                        const int more = min(max(left, 0), kAppend);
                        left -= kAppend;
                        wait += more;
                        // a lane with a full segment stores it and keeps the rest
                        if (wait >= kSeg) {
                            if (cs + kSeg <= cap_shell) {
#pragma unroll
                                for (int e = 0; e < kSeg; e += 4)
                                    *(int4*)(srow + cs + e) = make_int4(mine_st[e], mine_st[e + 1], mine_st[e + 2],
                                                                        mine_st[e + 3]);
                            }
#pragma unroll
                            for (int e = 0; e < kAppend - 1; ++e) mine_st[e] = mine_st[kSeg + e];
                            cs += kSeg;
                            wait -= kSeg;
                        }
                    }
                }
            }
        }
        if (MODE != kListsCoreOnly) {
            // the last, partial segment
            for (int e = 0; e < wait; ++e)
                if (cs + e < cap_shell) srow[cs + e] = mine_st[e];
            cs += wait;
        }
        if (act) {
            store_counts<MODE>(k, cc, cs, cap_core, cap_shell, ncore, nshell, err);
            maxc = max(maxc, cc);
            maxs = max(maxs, cs);
        }
        s = a1;
        if (s == e) {
            part += parts;
            s = part_start(part);
            e = part_start(part + 1);
        }
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        maxc = max(maxc, __shfl_xor(maxc, off, 64));
        maxs = max(maxs, __shfl_xor(maxs, off, 64));
    }
    if (lane == 0) {
        atomicMax(&maxcnt[0], maxc);
        atomicMax(&maxcnt[1], maxs);
    }
}

// Stencil sampling: |K(i)|, the number of atoms in the shell stencil's cells
// around atom i's cell (span^2 rows of span cells, each row at most two index
// ranges of the cell-sorted atoms), written as the shell count of every atom
// of the cell together with the cell itself (the build-time cell, which the
// batch decode uses even after the atoms have moved); one thread per cell, and
// the largest count raises maxcnt[1].
__global__ __launch_bounds__(kBlock) void k_stencil_counts(int n_c, int lo, int span,
                                                           const int32_t* __restrict__ cell_start,
                                                           int32_t* __restrict__ nshell, int32_t* __restrict__ scell,
                                                           int32_t* __restrict__ maxcnt, uint32_t* __restrict__ err)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t cells = (int64_t)n_c * n_c * n_c;
    int m = 0;
    if (c < cells) {
        const int cx = (int)(c % n_c), cy = (int)((c / n_c) % n_c), cz = (int)(c / ((int64_t)n_c * n_c));
        const int x0 = wrap(cx + lo, n_c);
        const int la = min(span, n_c - x0);  // cells before the wrap
        for (int dz = 0; dz < span; ++dz) {
            const int z = wrap(cz + lo + dz, n_c);
            for (int dy = 0; dy < span; ++dy) {
                const int row = (z * n_c + wrap(cy + lo + dy, n_c)) * n_c;
                m += cell_start[row + x0 + la] - cell_start[row + x0];
                if (span > la) m += cell_start[row + span - la] - cell_start[row];
            }
        }
        // the batch ranks are 16-bit: a larger stencil is an error (and its count is clamped)
        if (m > 65535) atomicOr(err, ERR_SHELL_CAP);
        for (int k = cell_start[c]; k < cell_start[c + 1]; ++k) {
            nshell[k] = min(m, 65535);
            scell[k] = (int32_t)c;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&maxcnt[1], m);
}

// Packed records of the sorted atoms: x | y << 16 and z, each fixed-point
// coordinate in units of 2^sh quanta taken modulo 2^16 (the separations within a
// stencil stay below 2^15 units, so their 16-bit differences are exact), the
// exclusion id (molecule, or -2 - k for an atom without one) and the sorted
// index k.
__global__ __launch_bounds__(kBlock) void k_pack_sorted(int64_t n, int sh, const uint4* __restrict__ spos,
                                                       const int32_t* __restrict__ smol, u32x4* __restrict__ spk)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint4 s = spos[k];
    const int32_t m = smol[k];
    spk[k] = u32x4{((s.x >> sh) & 0xffffu) | ((s.y >> sh) << 16), (s.z >> sh) & 0xffffu,
                   (uint32_t)(m >= 0 ? m : -2 - (int32_t)k), (uint32_t)k};
}

namespace {

// Shift s and bounds of the packed candidate test. Every separation a lane tests
// (an atom and a candidate of its own stencil, which does not wrap the box) lies
// within R + 1 cell edges (+ rounding) per axis; s is the smallest shift that fits
// that in 16 signed bits with two units to spare, so the 16-bit differences of
// the packed global coordinates are exact modulo 2^16, and each packed component
// is off by less than delta = 1 unit (s = 16, where none fits: the top 16 bits,
// delta = 3). With e = sum of component errors: D <= d2 + 2 delta sqrt(3 d2) +
// 3 delta^2 and D >= d2 - 2 delta sqrt(3 d2) for the exact squared separation D
// in the same units; the bounds follow, with one unit of margin for rounding.
struct PackedGeometry {
    int sh = 16;
    PackedBounds tb{};
};

PackedGeometry packed_geometry(const Geometry& g)
{
    PackedGeometry p;
    const double E = 4294967296.0 / (double)g.n_c;
    double delta = 3.0;
    const double M = (g.reach + 1.0) * E + 4.0;
    for (int s = 0; s <= 15; ++s) {
        if (M <= std::ldexp(1.0, 15 + s) - std::ldexp(1.0, s + 1)) {
            p.sh = s;
            delta = 1.0;
            break;
        }
    }
    // bounds in units of 2^s quanta (component errors below delta units), as doubles
    auto inner = [](uint64_t t, int s, double delta) -> double {
        const double T = (double)t / std::ldexp(1.0, 2 * s);
        const double v = std::floor(T - 2.0 * delta * std::sqrt(3.0 * T) - 3.0 * delta * delta - 1.0);
        return v > 0.0 ? v : 0.0;
    };
    auto outer = [](uint64_t t, int s, double delta) -> double {
        const double T = (double)t / std::ldexp(1.0, 2 * s);
        const double r = delta * std::sqrt(3.0) + std::sqrt(3.0 * delta * delta + T);
        double o = std::ceil(r * r) + 2.0;
        while ((o + 1.0) - 2.0 * delta * std::sqrt(3.0 * (o + 1.0)) <= T + 1.0) o += 1.0;
        return o;
    };
    auto u32 = [](double v) { return v < 4294967295.0 ? (uint32_t)v : 4294967295u; };
    p.tb.core_in = u32(inner(g.tl_core, p.sh, delta));
    p.tb.core_out = u32(outer(g.tl_core, p.sh, delta));
    p.tb.shell_in = u32(inner(g.tl_shell, p.sh, delta));
    p.tb.shell_out = u32(outer(g.tl_shell, p.sh, delta));
    p.tb.lo_in = u32(inner(g.tl_lo, p.sh, delta));
    p.tb.lo_out = u32(outer(g.tl_lo, p.sh, delta));
    return p;
}

// The stencil of the list build: with stencil sampling the core lists alone,
// over the core stencil and with rows pruned by the core radius.
Geometry list_geometry(const irbe_ctx* h)
{
    Geometry g = h->geo;
    if (h->stencil) {
        g.reach = 1;
        g.lo = -1;
        g.hi = 1;
    }
    return g;
}

}  // namespace

bool lists_by_lanes(const irbe_ctx* h)
{
    const Geometry g = list_geometry(h);
    const int span = g.hi - g.lo + 1;
    const double per_cell = (double)h->cfg.n_atoms / (double)g.n_cells;
    return 2 * g.reach + 1 <= g.n_c && per_cell < kLaneMaxPerCell && span * span <= 2 * kListWave;
}

static hipError_t launch_list_lanes(irbe_ctx* h)
{
    const Geometry g = list_geometry(h);
    const int n_c = g.n_c;
    // cells of a wavefront's run: the union x range of their stencils within one period
    // of the box and its cell starts within 64 LDS words
    const int G = std::max(1, std::min(n_c - 2 * g.reach, 64 - (g.hi - g.lo + 1)));
    // wavefronts per cell row: its runs of 64 atoms, with two standard deviations of a
    // random system's rows (fuller rows: their wavefronts take further runs)
    const double per_row = (double)h->cfg.n_atoms / ((double)n_c * n_c);
    int parts = (int)std::ceil((per_row + 2.0 * std::sqrt(per_row)) / kListWave);
    // where those runs are longer than G cells (small or very dilute boxes), a wavefront takes
    // its run in pieces, one after another; a chip that the rows leave idle (up to 2,048 of
    // them, two wavefronts per SIMD) does better with a wavefront per segment of at most
    // G cells (and 48 atoms, as segments differ in them). Build of all lists, runs against
    // segments: 1.3 ions per cell, 600 ions (49 rows) 451 and 93 us, 10^5 (1,849 rows) 306
    // and 215, 1.6 10^5 (2,500 rows) 322 and 324; 0.2 per cell, 12,000 (1,521 rows) 138 and
    // 135, 30,000 (2,809 rows) 165 and 202
    int seg = 0;
    if (n_c * n_c <= 2 * 1024 && n_c > 0.8 * G * std::ceil(per_row / kListWave)) {
        parts = std::max((n_c + G - 1) / G, (int)std::ceil(per_row / 48.0));
        seg = (n_c + parts - 1) / parts;
        parts = (n_c + seg - 1) / seg;
    }
    const int64_t groups = (int64_t)n_c * n_c * parts;
    // the packed records as for one cell per group: only a lane's own candidates
    // (within the stencil of its cell) are tested, so 16-bit differences of the
    // global coordinates are exact
    const PackedGeometry pl = packed_geometry(g);
    // the outermost list's radius in cell edges, with the margin of the row pruning
    const double r_cells = std::sqrt((double)(h->stencil ? g.tl_core : g.tl_shell)) * n_c / 4294967296.0 + kPruneMargin;
    const float r2_cells = (float)(r_cells * r_cells);
    k_pack_sorted<<<(unsigned)blocks_for(h->cfg.n_atoms, kBlock), kBlock, 0, h->stream>>>(
        h->cfg.n_atoms, pl.sh, h->spos, h->smol, (u32x4*)h->spk);
#define IRBE_LANES_ARGS                                                                                            \
    n_c, g.lo, g.hi, G, parts, seg, pl.tb, g.tl_core, g.tl_lo, g.tl_shell, r2_cells, h->n_excl > 0, h->spos, (const u32x4*)h->spk, h->cell_start, \
        h->cap_core, h->cap_shell, h->core, h->ncore, h->shell, h->nshell, h->maxcnt, h->err
    if (h->full_list)
        k_build_lists_lanes<kListsFull><<<(unsigned)groups, kListWave, 0, h->stream>>>(IRBE_LANES_ARGS);
    else if (h->stencil)
        k_build_lists_lanes<kListsCoreOnly><<<(unsigned)groups, kListWave, 0, h->stream>>>(IRBE_LANES_ARGS);
    else if (g.skin)
        k_build_lists_lanes<kListsSplitSkin><<<(unsigned)groups, kListWave, 0, h->stream>>>(IRBE_LANES_ARGS);
    else
        k_build_lists_lanes<kListsSplit><<<(unsigned)groups, kListWave, 0, h->stream>>>(IRBE_LANES_ARGS);
#undef IRBE_LANES_ARGS
    return hipGetLastError();
}

hipError_t launch_build_lists(irbe_ctx* h)
{
    const hipError_t e = lists_by_lanes(h) ? launch_list_lanes(h) : launch_list_blocks(h);
    if (e != hipSuccess || !h->stencil) return e;
    // stencil sampling: |K(i)| (the atoms of the shell stencil's cells) as the shell count
    const Geometry& gs = h->geo;
    const int64_t cells = gs.n_cells;
    k_stencil_counts<<<(unsigned)blocks_for(cells, kBlock), kBlock, 0, h->stream>>>(
        gs.n_c, gs.lo, gs.hi - gs.lo + 1, h->cell_start, h->nshell, h->scell, h->maxcnt, h->err);
    return hipGetLastError();
}

}  // namespace irbe
