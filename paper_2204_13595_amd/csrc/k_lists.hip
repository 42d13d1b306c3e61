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

// Squared separation of two packed positions (x | y << 16, z): exact in the
// 16-bit units (differences modulo 2^16); the sum of the three squares stays
// below 2^32.
__device__ __forceinline__ uint32_t d2_packed(uint32_t cxy, uint32_t cz, uint32_t axy, uint32_t az)
{
    const s16x2 dxy = __builtin_bit_cast(s16x2, cxy) - __builtin_bit_cast(s16x2, axy);
    const int dz = (short)(cz - az);
    return (uint32_t)__builtin_amdgcn_sdot2(dxy, dxy, dz * dz, false);
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
// takes up to 64 atoms of consecutive cells of one cell row, one atom per lane.
// For every stencil row (dz, dy) the union of the atoms' x ranges is staged in
// LDS as above. The first atom and atom count of every row's union (two index
// ranges at most) are loaded once per group into a table held in registers,
// so that a row's cell starts and the records of its first tile are loaded in
// one memory round trip, issued before the pruning of the rows that follow.
// Each lane computes its own cell range in the union (row pruning) and
// the lanes then walk their ranges in lockstep, lane a testing its k-th
// candidate at step k. A lane appends its shell members (or full-list
// members) to a ring of 8 entries in LDS and every 4 steps the lanes whose
// ring holds 4 unwritten entries store them as one aligned 16-byte segment of
// their list row (at most 3 + 4 entries wait in the ring); core members are
// stored directly. Candidates between the
// packed bounds take the exact test on full positions read from memory (the
// LDS footprint, about 4.4 KB, leaves room for the wavefronts that hide the
// per-row latencies).
// ---------------------------------------------------------------------------
constexpr int kLaneTile = 128;           // staged candidates per pass of a row
constexpr int kRing = 8;                 // ring entries per lane
constexpr int kSeg = 4;                  // entries per stored segment (16 bytes)
constexpr int kRingStride = kRing + 1;   // words per lane's ring (odd: conflict-free lanes)
constexpr double kLaneGroupAtoms = 60.0; // atoms per group the launch aims at (at most 64 per pass)

// A stencil row of the lane-per-atom kernel as loaded: its union's two segments
// (first atom and atoms of A; first atom of B; atoms of both), this lane's raw
// cell start in the union and the records of its first tile.
struct RowLoad {
    int jA, nA, jB, total;
    int cst;
    u32x4 rec[kLaneTile / kListWave];
};

// (eight wavefronts per SIMD requested: the register bound of 64 gains the skin lists 8%, the others are the same)
template <int MODE>
__global__ __launch_bounds__(kListWave, 8) void k_build_lists_lanes(
    int n_c, int lo, int hi, int G, PackedBounds tb, uint64_t t_core, uint64_t t_lo, uint64_t t_shell, float tfs_hi,
    const uint4* __restrict__ spos, const u32x4* __restrict__ spk, const int32_t* __restrict__ cell_start,
    const uint32_t* __restrict__ bound_g,
    int cap_core, int cap_shell, int32_t* __restrict__ core, int32_t* __restrict__ ncore,
    int32_t* __restrict__ shell, int32_t* __restrict__ nshell, int32_t* __restrict__ maxcnt,
    uint32_t* __restrict__ err)
{
    __shared__ u32x4 trec[kLaneTile + 1];          // packed x | y, packed z, exclusion id, sorted index
    __shared__ int32_t ring[kListWave * kRingStride];
    __shared__ int32_t tcs[64];                    // union positions of the row's cells (segment A, then B)
    const uint32_t* bound = bound_g;
    const int lane = threadIdx.x;
    const int span = hi - lo + 1;
    const int groups_per_row = (n_c + G - 1) / G;
    const int g = (int)xcd_block(blockIdx.x, gridDim.x);
    const int rowid = g / groups_per_row;
    const int cz = rowid / n_c, cy = rowid % n_c;
    const int x0 = (g % groups_per_row) * G;
    const int gr = min(G, n_c - x0);
    const int home = (cz * n_c + cy) * n_c;
    const int a0 = cell_start[home + x0], a1 = cell_start[home + x0 + gr];
    const int span_u = gr - 1 + span;           // cells of the union x range
    const int xu0 = wrap(x0 + lo, n_c);         // first cell of the union
    const int lenA = min(span_u, n_c - xu0);    // cells before the wrap
    int32_t* const myring = ring + lane * kRingStride;
    // every stencil row's union: first atom and atom count of segment A (cells
    // xu0 .. xu0 + lenA - 1) and of segment B (cells 0 .. lenB - 1, past the wrap),
    // row ri = (dz, dy) = (lo + ri / span, lo + ri % span) in lane ri % 64 of
    // rtab[ri / 64], loaded once for the group
    const int nrows = span * span;  // at most 2 * kListWave (checked at the launch)
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
    // first and last coordinates of the stencil's z and y cell slabs, lane l for the
    // offset lo + l (span <= 11 here), read back with readlane
    const int ls = min(lane, span - 1);
    const int zs = wrap(cz + lo + ls, n_c), ys = wrap(cy + lo + ls, n_c);
    const uint32_t zlo = bound[zs], zhi = bound[zs + 1] - 1u, ylo = bound[ys], yhi = bound[ys + 1] - 1u;
    // distance from coordinate s to the slab at offset d (the first coordinate of a slab above, the last of one below)
    auto gap = [](uint32_t s, int d, uint32_t lo_t, uint32_t hi_t, int idx) __attribute__((always_inline)) {
        if (d > 0) return (uint32_t)__builtin_amdgcn_readlane((int)lo_t, idx) - s;
        if (d < 0) return s - (uint32_t)__builtin_amdgcn_readlane((int)hi_t, idx);
        return 0u;
    };
    // the row after (dz, dy) in the stencil's lexicographic order
    auto step_row = [&](int& dz, int& dy) __attribute__((always_inline)) {
        if (++dy > hi) {
            dy = lo;
            ++dz;
        }
    };
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
            d.rec[q] = spk[t < cnt0 ? (t < d.nA ? d.jA + t : d.jB + (t - d.nA)) : a0];
        }
        return d;
    };
    int maxc = 0, maxs = 0;
    for (int chunk = a0; chunk < a1; chunk += kListWave) {
        const int k = chunk + lane;
        const bool act = k < a1;
        const uint4 si = act ? spos[k] : make_uint4(0, 0, 0, 0);
        const int cx = (int)(((uint64_t)si.x * (uint32_t)n_c) >> 32);
        const int ti = act ? wrap(cx - x0, n_c) : 0;  // lane's home cell in [0, gr)
        const u32x4 pk = act ? spk[k] : u32x4{0, 0, 0, 0};  // packed x | y, z, exclusion id
        const uint32_t axy = pk.x, az = pk.y, amol = pk.z;
        int32_t* const crow = core + (int64_t)k * cap_core;
        int32_t* const srow = shell + (int64_t)k * cap_shell;
        int cc = 0, cs = 0;  // list lengths so far
        int fs = 0;          // shell entries already stored (a multiple of kSeg)
        // the lane's range in row ri = (dz, dy): cells [u_lo, u_hi] of the union, pruned by
        // the row gap; the first row at or after ri that some lane needs (nrows: none),
        // with (dz, dy) advanced to it
        auto next_row = [&](int ri, int& dz, int& dy, int& u_lo, int& u_hi, bool& need)
                            __attribute__((always_inline)) -> int {
            for (; ri < nrows; ++ri, step_row(dz, dy)) {
                if (MODE == kListsCoreOnly && (dz < -1 || dz > 1 || dy < -1 || dy > 1)) continue;
                u_lo = ti;
                u_hi = ti + span - 1;
                need = act;
                if (act) {
                    const float gz = (float)gap(si.z, dz, zlo, zhi, dz - lo);
                    const float gy = (float)gap(si.y, dy, ylo, yhi, dy - lo);
                    const float rem = tfs_hi - gy * gy - gz * gz;
                    if (rem < 0.0f) {
                        need = false;
                    } else {
                        const uint32_t ext = (uint32_t)(__builtin_amdgcn_sqrtf(rem) * 1.000002f) + 2u;
                        const int cl = (int)(((uint64_t)(uint32_t)(si.x - ext) * (uint32_t)n_c) >> 32);
                        const int ch = (int)(((uint64_t)(uint32_t)(si.x + ext) * (uint32_t)n_c) >> 32);
                        int ol = cl - cx, oh = ch - cx;
                        if (ol > n_c / 2) ol -= n_c;
                        if (ol < -n_c / 2) ol += n_c;
                        if (oh > n_c / 2) oh -= n_c;
                        if (oh < -n_c / 2) oh += n_c;
                        u_lo = ti + (max(ol, lo) - lo);
                        u_hi = ti + (min(oh, hi) - lo);
                    }
                }
                if (ballot(need) != 0) return ri;
            }
            return nrows;
        };
        int u_lo = 0, u_hi = 0;
        bool need = false;
        int dz = lo, dy = lo;
        int rc = next_row(0, dz, dy, u_lo, u_hi, need);
        while (rc < nrows) {
            // the row's loads are in flight while the next needed row is found
            const RowLoad cur = row_load(rc, dz, dy);
            int u_lo_n = 0, u_hi_n = 0;
            bool need_n = false;
            int dz_n = dz, dy_n = dy;
            step_row(dz_n, dy_n);
            const int rn = next_row(rc + 1, dz_n, dy_n, u_lo_n, u_hi_n, need_n);
            const bool core_row = MODE != kListsFull && dz >= -1 && dz <= 1 && dy >= -1 && dy <= 1;
            const int jA = cur.jA, nA = cur.nA, jB = cur.jB, total = cur.total;
            // (LDS accesses of the one wavefront of the workgroup take effect in
            // order: the previous row's reads precede these writes)
            if (lane <= span_u) tcs[lane] = cur.cst - (lane < lenA ? jA : jB - nA);
#pragma unroll
            for (int h = 0; h < kLaneTile / kListWave; ++h)
                if (h * kListWave + lane < min(kLaneTile, total)) trec[h * kListWave + lane] = cur.rec[h];
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
                        trec[t] = spk[j];
                    }
                    __syncthreads();
                }
                // this tile's part of the range, in tile positions
                const int s0 = need ? max(p_lo, base) - base : 0;
                const int len = need ? max(min(p_hi, base + cnt) - base - s0, 0) : 0;
                int steps = len;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) steps = max(steps, __shfl_xor(steps, off, 64));
                steps = __builtin_amdgcn_readfirstlane(steps);  // (every lane holds the maximum)
                for (int st = 0; st < steps; ++st) {
                    const bool k_in = st < len;
                    const int tp = k_in ? s0 + st : kLaneTile;
                    const u32x4 r = trec[tp];
                    const uint32_t d2 = d2_packed(r.x, r.y, axy, az);
                    const bool keep = k_in && r.z != amol;
                    bool in_core = false, in_shell = false, amb;
                    if (MODE == kListsCoreOnly) {
                        in_core = keep && d2 < tb.core_in;
                        amb = keep && !in_core && d2 <= tb.core_out;
                    } else if (MODE == kListsSplitSkin) {
                        const bool c_in = d2 < tb.core_in, c_out = d2 > tb.core_out;
                        const bool l_in = d2 < tb.lo_in, l_out = d2 > tb.lo_out;
                        const bool s_in = d2 < tb.shell_in, s_out = d2 > tb.shell_out;
                        in_core = keep && c_in;
                        in_shell = keep && l_out && s_in;
                        amb = keep && !((c_in || c_out) && (l_in || (l_out && s_in) || s_out));
                    } else if (MODE == kListsSplit) {
                        const bool c_in = d2 < tb.core_in, c_out = d2 > tb.core_out;
                        const bool s_in = d2 < tb.shell_in, s_out = d2 > tb.shell_out;
                        in_core = keep && c_in;
                        in_shell = keep && c_out && s_in;
                        amb = keep && !c_in && !in_shell && !s_out;
                    } else {
                        in_shell = keep && d2 < tb.shell_in;
                        amb = keep && !in_shell && d2 <= tb.shell_out;
                    }
                    if (amb) {
                        // between the bounds: the exact test on full positions decides
                        const uint4 sj = spos[(int)r.w];
                        const int32_t dx = (int32_t)(sj.x - si.x);
                        const int32_t dy2 = (int32_t)(sj.y - si.y);
                        const int32_t dz2 = (int32_t)(sj.z - si.z);
                        const uint64_t d2x = (uint64_t)((int64_t)dx * dx) + (uint64_t)((int64_t)dy2 * dy2) +
                                             (uint64_t)((int64_t)dz2 * dz2);
                        in_core = MODE != kListsFull && d2x <= t_core;
                        in_shell = MODE != kListsCoreOnly &&
                                   (MODE == kListsSplitSkin ? d2x > t_lo : !in_core) && d2x <= t_shell;
                    }
                    if (MODE != kListsCoreOnly && in_shell) {
                        myring[cs & (kRing - 1)] = (int32_t)r.w;
                        ++cs;
                    }
                    if (MODE != kListsFull && core_row && in_core) {
                        if (cc < cap_core) crow[cc] = (int32_t)r.w;
                        ++cc;
                    }
                    if (MODE != kListsCoreOnly && (st & (kSeg - 1)) == kSeg - 1) {
                        // lanes with a full segment store it (at most one per kSeg steps)
                        if (cs - fs >= kSeg) {
                            const int o = fs & (kRing - 1);
                            if (fs + kSeg <= cap_shell)
                                *(int4*)(srow + fs) = make_int4(myring[o], myring[o + 1], myring[o + 2], myring[o + 3]);
                            fs += kSeg;
                        }
                    }
                }
                if (MODE != kListsCoreOnly) {
                    // at most one full segment waits after the last step
                    if (cs - fs >= kSeg) {
                        const int o = fs & (kRing - 1);
                        if (fs + kSeg <= cap_shell)
                            *(int4*)(srow + fs) = make_int4(myring[o], myring[o + 1], myring[o + 2], myring[o + 3]);
                        fs += kSeg;
                    }
                }
            }
            rc = rn;
            dz = dz_n;
            dy = dy_n;
            u_lo = u_lo_n;
            u_hi = u_hi_n;
            need = need_n;
        }
        if (MODE != kListsCoreOnly) {
            // the last, partial segment
            for (int e = fs; e < cs; ++e)
                if (e < cap_shell) srow[e] = myring[e & (kRing - 1)];
        }
        if (act) {
            store_counts<MODE>(k, cc, cs, cap_core, cap_shell, ncore, nshell, err);
            maxc = max(maxc, cc);
            maxs = max(maxs, cs);
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
    // cells per wavefront: groups of about kLaneGroupAtoms atoms, the union x range of
    // the group's stencils within one period of the box and its cell starts within
    // 64 LDS words, and the groups of a cell row balanced (a short last group leaves
    // its wavefront mostly idle)
    const double per_cell = (double)h->cfg.n_atoms / (double)g.n_cells;
    const int g_want = (int)std::lround(std::min(64.0, std::max(1.0, kLaneGroupAtoms / std::max(per_cell, 0.75))));
    const int g_cap = std::min(std::max(1, std::min(g_want, n_c - 2 * g.reach)), 64 - (g.hi - g.lo + 1));
    const int groups_per_row = (n_c + g_cap - 1) / g_cap;
    const int G = (n_c + groups_per_row - 1) / groups_per_row;
    const int64_t groups = (int64_t)n_c * n_c * ((n_c + G - 1) / G);
    // the packed records as for one cell per group: only a lane's own candidates
    // (within the stencil of its cell) are tested, so 16-bit differences of the
    // global coordinates are exact
    const PackedGeometry pl = packed_geometry(g);
    // FP32 threshold of the outermost list with a relative margin of 2e-6, far
    // above the FP32 rounding of the row gaps: the row pruning never drops a member.
    const float tf_hi = (float)(h->stencil ? g.tl_core : g.tl_shell) * 1.000002f;
    k_pack_sorted<<<(unsigned)blocks_for(h->cfg.n_atoms, kBlock), kBlock, 0, h->stream>>>(
        h->cfg.n_atoms, pl.sh, h->spos, h->smol, (u32x4*)h->spk);
#define IRBE_LANES_ARGS                                                                                            \
    n_c, g.lo, g.hi, G, pl.tb, g.tl_core, g.tl_lo, g.tl_shell, tf_hi, h->spos, (const u32x4*)h->spk, h->cell_start, \
        h->cell_bound, h->cap_core, h->cap_shell, h->core, h->ncore, h->shell, h->nshell, h->maxcnt, h->err
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
