// Core and shell lists on the matrix cores (Sec. 2.3): the same lists, in the
// same canonical order and by the same exact membership, as the lane-per-atom
// form of k_lists.hip builds for dilute cells.
//
// A workgroup takes a block of up to 32 consecutive atoms of one cell row (a
// run along x, since the atoms of a row are sorted by x). Per stencil row
// (dz, dy) the candidates are the atoms of an x window around the block, at
// most two index ranges (the second after the periodic wrap), found by binary
// search at the window's exact ends. The ranges, each padded to whole half words of
// 16 candidates, form one sequence of words in canonical order; a bit of a word
// is one candidate, and the block's result is one mask per (word, atom).
//
// Distances. With coordinates relative to the block's centre, in units in which
// the list radius is 64, the test value d = |a - c|^2 - T is one 16-term dot
// product of half-precision pairs: every coordinate is split into a high and a
// low part (22 bits together) and the four products of the parts are kept, the
// norms |c|^2 and |a|^2 - T (also split) are multiplied by a constant. One
// 32x32x16 MFMA gives d for 32 candidates and 32 atoms; two of them fill a word
// per lane: the operand lanes are permuted so that a lane's 2 x 16 results are
// the 32 candidates of one word of its atom. A sign bit costs one v_alignbit
// (shift the word, insert the sign) and half a v_min3 (smallest |d|). Only where
// some |d| is within the error bound of the split products does the wave take
// the exact 64-bit test on the fixed-point positions for those candidates, so
// membership never depends on the floating-point values. Stencils that wrap the
// box (2R + 1 > n_c; boxes of a few thousand atoms) take the same form with the
// distances from minimum-image differences on the vector units.
//
// A wave converts 64 candidates at a time; its chunks whose candidates can come
// within r_core of the block get a second pair of MFMAs for C(i) (same operands,
// another constant), a third with a skin. Same-molecule pairs and the atom
// itself are then cleared from the masks by position (molecules of hundreds of
// atoms: by comparing ids, chunk by chunk), and the masks are written out as
// lists, chunk by chunk: a member's place is a bit count.
//
// What bounds it: vector issue (395 instructions per atom at 3.1 M atoms of
// water, of which the 60 chunks of a block take about 100 each). Split lists of
// that box: 2.75 ms (6.03 ms with the candidate tests on the vector units and
// 16-bit list entries stored per member); of 98,304 atoms 0.14 ms (0.43 ms), of
// 2,703 atoms 0.05 ms (0.39 ms), where a wavefront per cell group left the
// chip idle.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "irbe_device.hpp"
#include "irbe_internal.hpp"

namespace irbe {

// Threads per block of atoms: four wavefronts, and eight where the stencil wraps
// the box, as those are the smallest systems, of fewer blocks than the chip has
// compute units (2,703 atoms: 128 blocks, 54 us with four).
constexpr int mask_threads(bool narrow) { return narrow ? 256 : 512; }
constexpr int kMaskWords = 128;  // words per tile (two per lane when the masks are read back by atom)
constexpr int kMaskRows = 128;  // stencil rows per pass (two index ranges each)
constexpr float kMaskUnit = 64.0f;  // the list radius in the units of the half-precision coordinates
constexpr float kMaskNorm = 64.0f;  // the norms are carried divided by this

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ int wrap_c(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

__device__ __forceinline__ uint64_t ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ uint64_t dist2_fixed(uint4 a, uint4 b)
{
    const int32_t dx = (int32_t)(b.x - a.x);
    const int32_t dy = (int32_t)(b.y - a.y);
    const int32_t dz = (int32_t)(b.z - a.z);
    return (uint64_t)((int64_t)dx * dx) + (uint64_t)((int64_t)dy * dy) + (uint64_t)((int64_t)dz * dz);
}

// v split into its leading 11 significant bits and the rest, as a half pair.
__device__ __forceinline__ uint32_t split_half(float v)
{
    const float hi = __uint_as_float(__float_as_uint(v) & 0xffffe000u);
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(hi, v - hi));
}

__device__ __forceinline__ uint32_t twice_half(float v)
{
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(v, v));
}

// Sum over the lanes below within the half-wave, inclusive (data-parallel
// primitives: shifts within rows of 16, then the row total broadcast).
__device__ __forceinline__ int half_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    return x;
}

__device__ __forceinline__ int wave_scan(int x)
{
    x = half_scan(x);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

}  // namespace

// Smallest (MIN) or largest value of the half-wave's lanes (valid in lane 31 / 63).
template <bool MIN>
__device__ __forceinline__ uint32_t half_extreme(uint32_t x)
{
    auto f = [](uint32_t a, uint32_t b) { return MIN ? min(a, b) : max(a, b); };
    // (a lane without a source sees its own value)
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x111, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x112, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x114, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x118, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x142, 0xa, 0xf, false));
    return x;
}

// One range of candidates: sorted indices base .. base + len - 1 in the half
// words half .. half + (len + 15) / 16 - 1 of the block's sequence.
struct MaskSeg {
    int base, len, half;
};

// IDS: same-molecule pairs leave the masks by the molecule ids of the candidates (and of
// the atom itself, by its index) instead of by position, chunk by chunk.
template <int MODE, bool NARROW, bool MASK, bool IDS>
__global__ __launch_bounds__(mask_threads(NARROW), NARROW ? 4 : 2) void k_list_blocks(ListBlockArgs p)
{
    constexpr int kMaskBlock = mask_threads(NARROW);
    constexpr int kMaskWaves = kMaskBlock / 64;
    constexpr bool kTwo = MODE == kListsSplit || MODE == kListsSplitSkin;  // C(i) beside S(i)
    __shared__ uint32_t ms[kMaskWords][33];              // masks of the outer list (S(i), the full list, or C(i) alone)
    __shared__ uint32_t mc[kTwo ? kMaskWords : 1][33];   // masks of C(i)
    __shared__ MaskSeg seg[2 * kMaskRows];
    __shared__ int2 wt[2 * kMaskWords];                  // a half word's first candidate and number of candidates
    __shared__ uint4 cpos[NARROW ? 1 : kMaskWaves][NARROW ? 1 : 64];
    __shared__ int wsum[kMaskWaves];
    __shared__ int cnt_s[32], cnt_c[32];                 // list lengths so far
    __shared__ int cflag[kMaskWords / 2];                // chunks that hold core candidates
    __shared__ int fw[kMaskWords];                       // their words
    __shared__ uint16_t xpre[kMaskWaves][64];            // members before each of one atom's flagged words
    __shared__ __align__(16) int32_t cid[IDS ? kMaskWaves : 1][IDS ? 64 : 1];  // ids of a chunk's candidates, in bit order
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = (int)xcd_block(blockIdx.x, gridDim.x);
    const int k0 = p.blk_start[slot] - 1;
    if (k0 < 0) return;  // an unused slot (uniform)
    const int n_c = p.n_c, lo = p.lo, span = p.span, nrows = span * span;
    const uint32_t* __restrict__ bound = p.bound;
    // the block: atoms k0 .. k0 + na - 1 of cells of one segment of row (cz, cy)
    const uint4 s0 = p.spos[k0];
    auto cell_of = [&](uint32_t s) { return (int)(((uint64_t)s * (uint32_t)n_c) >> 32); };
    const int cx = cell_of(s0.x), cy = cell_of(s0.y), cz = cell_of(s0.z);
    const int home = (cz * n_c + cy) * n_c;
    const int send = p.cell_start[home + min((cx / p.G + 1) * p.G, n_c)];
    const int na = min(32, send - k0);
    const int al = min(lane & 31, na - 1);  // this lane's atom (the last one again past the end)
    const uint4 si = p.spos[k0 + al];
    const uint32_t xlo = s0.x;
    const uint32_t xext = (uint32_t)__builtin_amdgcn_readlane((int)si.x, 31) - xlo;  // x extent of the block
    // the excluded partner this thread clears in the first round (its loads go out early)
    const int xa = tid & 31, xe = tid >> 5;
    const int2 xr = IDS ? make_int2(0, 0) : p.sxr[k0 + min(xa, na - 1)];
    auto partner = [&](int e) {
        // entry e of the atom itself and its excluded partners, whose sorted indices are
        // written for the pair kernels on the way
        if (xa >= na || e > xr.y) return -1;
        if (e == 0) return k0 + xa;
        const int j = p.rank[p.xidx[xr.x + e - 1]];
        p.sxidx[xr.x + e - 1] = j;
        return j;
    };
    const int xj = IDS ? -1 : partner(xe);
    uint4 xs = p.spos[max(xj, 0)];
    // an atom's id (without a molecule, its own), and the ids of the block's atoms by their low 6 bits
    auto id_of = [&](int k) {
        const int m = p.smol[k];
        return m >= 0 ? m : -2 - k;
    };
    const int my_id = IDS ? id_of(k0 + al) : 0;
    uint64_t ids = 0;
    if constexpr (IDS) {
        ids = 1ull << (my_id & 63);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) ids |= __shfl_xor((unsigned long long)ids, off, 64);
    }
    // centre and half extents of the block's bounding box
    const uint32_t bx = xlo + xext / 2;
    const uint32_t yb = bound[cy], zb = bound[cz];
    const uint32_t ylo = (uint32_t)__builtin_amdgcn_readlane((int)half_extreme<true>(si.y - yb), 31) + yb;
    const uint32_t yhi = (uint32_t)__builtin_amdgcn_readlane((int)half_extreme<false>(si.y - yb), 31) + yb;
    const uint32_t zlo = (uint32_t)__builtin_amdgcn_readlane((int)half_extreme<true>(si.z - zb), 31) + zb;
    const uint32_t zhi = (uint32_t)__builtin_amdgcn_readlane((int)half_extreme<false>(si.z - zb), 31) + zb;
    const uint32_t by = ylo + (yhi - ylo) / 2, bz = zlo + (zhi - zlo) / 2;
    const float us = p.unit;  // units per quantum
    const float hx = (float)(xext / 2 + 1) * us;
    const float hy = (float)((yhi - ylo) / 2 + 1) * us, hz = (float)((zhi - zlo) / 2 + 1) * us;
    auto rel = [&](uint32_t a, uint32_t b) { return (float)(int32_t)(a - b) * us; };
    const float ax = rel(si.x, bx), ay = rel(si.y, by), az = rel(si.z, bz);
    // the atoms' operand: lanes 0..31 hold the first 8 terms of atom (lane & 31), lanes 32..63 the other 8
    const bool upper = lane >= 32;
    u32x4 bf;
    float an = 0.0f;
    float band = p.band_valu;
    if constexpr (NARROW) {
        const float a1 = upper ? az : ax;
        const float a1h = __uint_as_float(__float_as_uint(a1) & 0xffffe000u);
        const float ayh = __uint_as_float(__float_as_uint(ay) & 0xffffe000u);
        an = (ax * ax + ay * ay + az * az);
        bf[0] = twice_half(-2.0f * a1h);
        bf[1] = twice_half(-2.0f * (a1 - a1h));
        bf[2] = upper ? twice_half(kMaskNorm) : twice_half(-2.0f * ayh);
        bf[3] = upper ? 0u : twice_half(-2.0f * (ay - ayh));
        // error bound of d for pairs near the threshold: |c| <= |a| + r there, so every
        // term is below S = (2 |a| + r)^2; the splits, the norms' splits and the FP32
        // accumulation of 16 terms are each within 2 S 2^-20, together below S 2^-17
        const float S = 2.0f * __builtin_amdgcn_sqrtf(hx * hx + hy * hy + hz * hz) + kMaskUnit + 1.0f;
        band = S * S * 7.62939453125e-6f;
    }
    if (tid < 32) {
        cnt_s[tid] = 0;
        cnt_c[tid] = 0;
    }
    int wbase = 0;   // words of the row passes before this one
    bool long_row = false;
    for (int rb = 0; rb < nrows; rb += kMaskRows) {
        // ---- candidate ranges of the stencil rows: thread 2 r + q, range q of row rb + r
        int sb = 0, sl = 0;
        {
            const int r = rb + (tid >> 1);
            if (r < nrows && tid < 2 * kMaskRows) {
                // (r / span: r and span are small enough for the FP32 quotient)
                const int rz = (int)(((float)r + 0.5f) * p.inv_span);
                const int dz = lo + rz, dy = lo + r - rz * span;
                const int z = wrap_c(cz + dz, n_c), y = wrap_c(cy + dy, n_c);
                const int row = (z * n_c + y) * n_c;
                const int rs = p.cell_start[row], re = p.cell_start[row + n_c];
                if constexpr (NARROW) {
                    const uint32_t gz = dz > 0 ? bound[z] - zhi : (dz < 0 ? zlo - (bound[z + 1] - 1u) : 0u);
                    const uint32_t gy = dy > 0 ? bound[y] - yhi : (dy < 0 ? ylo - (bound[y + 1] - 1u) : 0u);
                    const float rem = p.tf_hi - (float)gy * (float)gy - (float)gz * (float)gz;
                    if (rem >= 0.0f && re > rs) {
                        // (the window stays within one period: the segment rule bounds xext + 2 r by
                        // it, so the clamp takes only the rounding margin)
                        const uint32_t ext = min((uint32_t)(__builtin_amdgcn_sqrtf(rem) * 1.000002f) + 2u,
                                                 (0xffffffffu - xext) / 2u);
                        const uint32_t x0 = xlo - ext, x1 = xlo + xext + ext;
                        // range 0's thread finds the first atom at or after x0 in its cell, range 1's the
                        // first one after x1
                        const bool q = tid & 1;
                        const int c = row + cell_of(q ? x1 : x0);
                        int a = p.cell_start[c], b = p.cell_start[c + 1];
                        while (a < b) {
                            const int m = (a + b) >> 1;
                            const uint32_t x = p.spos[m].x;
                            if (q ? x <= x1 : x < x0) a = m + 1;
                            else b = m;
                        }
                        const int o = __shfl_xor(a, 1, 64);
                        if (x1 >= x0) {
                            sb = a;
                            sl = q ? 0 : o - a;
                        } else {
                            sb = q ? rs : a;
                            sl = q ? a - rs : re - a;
                        }
                    }
                } else {
                    // the whole row, from the first cell of the block's stencil (one cell per block)
                    const int m = p.cell_start[row + wrap_c(cx + lo, n_c)];
                    sb = (tid & 1) ? rs : m;
                    sl = (tid & 1) ? m - rs : re - m;
                }
            }
        }
        if (MASK) long_row |= sl + __shfl_xor(sl, 1, 64) > p.max_row;
        // ---- first half word of every range
        const int wn = (sl + 15) >> 4;
        const int inc = wave_scan(wn);
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int w0 = 2 * wbase, total = 0;
#pragma unroll
        for (int w = 0; w < kMaskWaves; ++w) {
            if (w < wave) w0 += wsum[w];
            total += wsum[w];
        }
        w0 += inc - wn;
        if (tid < 2 * kMaskRows) seg[tid] = MaskSeg{sb, sl, w0};
        const int wend = wbase + ((total + 1) >> 1);
        for (int t0 = wbase; t0 < wend; t0 += kMaskWords) {
            const int tw = min(kMaskWords, wend - t0);  // words of this tile
            for (int w = max(w0, 2 * t0); w < min(w0 + wn, 2 * (t0 + kMaskWords)); ++w) {
                const int o = (w - w0) << 4;
                wt[w - 2 * t0] = make_int2(sb + o, min(16, sl - o));
            }
            // (the half words past the last range, up to a whole chunk)
            for (int w = 2 * wbase + total - 2 * t0 + tid; w < 4 * ((tw + 1) >> 1); w += kMaskBlock)
                wt[w] = make_int2(k0, 0);
            __syncthreads();
            // ---- masks, 64 candidates (two words) per wave and pass
            const int nch = (tw + 1) >> 1;
            // the candidate this lane converts: operand row i of tile t holds bit 16 t + r of
            // word h, the bits that end up in the lanes of half h (identity without the MFMA)
            const int ci = lane & 31;
            const int cw = NARROW ? 2 * ((ci >> 2) & 1) + (lane >> 5) : lane >> 4;  // half word of the chunk's four
            const int cb = NARROW ? ((ci >> 3) << 2) + (ci & 3) : lane & 15;
            int id_n = 0;  // (its id)
            auto load_c = [&](int c, bool& ok) {
                const int2 w = wt[4 * min(c, nch - 1) + cw];
                ok = cb < w.y;
                if constexpr (IDS) id_n = id_of(ok ? w.x + cb : k0);
                return p.spos[ok ? w.x + cb : k0];
            };
            bool ok_n = false;
            uint4 sn = make_uint4(0, 0, 0, 0);
            if (wave < nch) sn = load_c(wave, ok_n);
            int members = 0;  // of this lane's atom in this wave's words
            for (int c = wave; c < nch; c += kMaskWaves) {
                const uint4 sc = sn;
                const bool ok = ok_n;
                const int id = id_n;
                sn = load_c(c + kMaskWaves, ok_n);  // the next chunk's candidates are in flight
                const float x = rel(sc.x, bx), y = rel(sc.y, by), z = rel(sc.z, bz);
                u32x4 f0, f1;
                if constexpr (NARROW) {
                    const uint32_t px = split_half(x), py = split_half(y), pz = split_half(z);
                    // (a missing candidate is far from every atom)
                    const uint32_t pn = split_half(ok ? (x * x + y * y + z * z) * (1.0f / kMaskNorm) : 30000.0f);
                    const uint32_t pc = twice_half(kMaskNorm);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(px, pz, false, false);
                    const auto s2 = __builtin_amdgcn_permlane32_swap(py, pn, false, false);
                    const auto s3 = __builtin_amdgcn_permlane32_swap(py, pc, false, false);
                    f0 = u32x4{s1[0], s1[0], s2[0], s3[0]};
                    f1 = u32x4{s1[1], s1[1], s2[1], s3[1]};
                } else {
                    cpos[wave][lane] = make_uint4(sc.x, sc.y, sc.z, ok ? 1u : 0u);
                    __builtin_amdgcn_wave_barrier();
                }
                const int myw = 2 * c + (lane >> 5);  // this lane's word
                // the lane's word of the ball D^2 <= t
                auto ball = [&](uint64_t t, float tu) __attribute__((always_inline)) -> uint32_t {
                    uint32_t word = 0;
                    float mn = 3.0e38f;
                    uint32_t amb = 0;
                    if constexpr (NARROW) {
                        u32x4 b = bf;
                        if (upper) b[3] = split_half((an - tu) * (1.0f / kMaskNorm));
                        f32x16 d0{}, d1{};
                        d0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, f0),
                                                                    __builtin_bit_cast(half8, b), d0, 0, 0, 0);
                        d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, f1),
                                                                    __builtin_bit_cast(half8, b), d1, 0, 0, 0);
#pragma unroll
                        for (int r = 15; r >= 0; --r)
                            word = __builtin_amdgcn_alignbit(word, __float_as_uint(d1[r]), 31);
#pragma unroll
                        for (int r = 15; r >= 0; --r)
                            word = __builtin_amdgcn_alignbit(word, __float_as_uint(d0[r]), 31);
#pragma unroll
                        for (int r = 0; r < 16; r += 2) {
                            mn = fminf(fminf(fabsf(d1[r]), fabsf(d1[r + 1])), mn);
                            mn = fminf(fminf(fabsf(d0[r]), fabsf(d0[r + 1])), mn);
                        }
                        if (__builtin_expect(ballot64(mn <= band) != 0, 0)) {
#pragma unroll
                            for (int r = 15; r >= 0; --r)
                                amb = __builtin_amdgcn_alignbit(amb, __float_as_uint(fabsf(d1[r]) - band), 31);
#pragma unroll
                            for (int r = 15; r >= 0; --r)
                                amb = __builtin_amdgcn_alignbit(amb, __float_as_uint(fabsf(d0[r]) - band), 31);
                        }
                    } else {
                        // minimum-image differences in FP32 (relative error of d2 below 2^-21)
#pragma unroll 8
                        for (int b = 31; b >= 0; --b) {
                            const uint4 q = cpos[wave][(lane & 32) + b];
                            const float dx = rel(q.x, si.x), dy = rel(q.y, si.y), dz = rel(q.z, si.z);
                            float d = dx * dx + dy * dy + dz * dz - tu;
                            d = q.w ? d : 3.0e38f;
                            word = __builtin_amdgcn_alignbit(word, __float_as_uint(d), 31);
                            amb = __builtin_amdgcn_alignbit(amb, __float_as_uint(fabsf(d) - band), 31);
                        }
                    }
                    // the exact test for the candidates the bound leaves open
                    while (amb) {
                        const int bit = __builtin_ctz(amb);
                        amb &= amb - 1;
                        const int2 w = wt[2 * myw + (bit >> 4)];
                        const int o = bit & 15;
                        const bool in = o < w.y && dist2_fixed(si, p.spos[o < w.y ? w.x + o : k0]) <= t;
                        word = (word & ~(1u << bit)) | ((in ? 1u : 0u) << bit);
                    }
                    return word;
                };
                // candidates with an id of the block (few chunks where molecules are small): the
                // lane's word of those with its atom's id
                uint32_t same = 0;
                if constexpr (IDS) {
                    if (ballot64(ok && ((ids >> (id & 63)) & 1ull)) != 0) {
                        cid[wave][16 * cw + cb] = ok ? id : -1;
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int b = 28; b >= 0; b -= 4) {
                            const int4 q = *(const int4*)&cid[wave][(lane & 32) + b];
                            same = (same << 4) | (q.w == my_id ? 8u : 0u) | (q.z == my_id ? 4u : 0u) |
                                   (q.y == my_id ? 2u : 0u) | (q.x == my_id ? 1u : 0u);
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                uint32_t wo = ball(p.t_out, p.tu_out) & ~same;
                if constexpr (kTwo) {
                    // candidates of this chunk near enough for C(i) (r_in: its radius, with a margin)
                    uint64_t near = ballot64(ok);
                    if (NARROW)
                        near &= ballot64(fabsf(x) <= hx + p.r_in) & ballot64(fabsf(y) <= hy + p.r_in) &
                                ballot64(fabsf(z) <= hz + p.r_in);
                    const bool any = near != 0;
                    if (lane == 0) cflag[c] = any ? 1 : 0;
                    if (any) {
                        const uint32_t wi = ball(p.t_in, p.tu_in) & ~same;
                        wo &= MODE == kListsSplitSkin ? ~ball(p.t_lo, p.tu_lo) : ~wi;
                        mc[myw][lane & 31] = wi;
                    }
                }
                ms[myw][lane & 31] = wo;
                if (MASK) members += __popc(wo);
            }
            if (MASK) atomicAdd(&cnt_s[lane & 31], members);
            __syncthreads();
            // ---- the atom itself and its excluded partners leave the masks
            for (int e = xe; !IDS && e <= 4096; e += kMaskBlock / 32) {
                // (threads of one round: 8 partners of every atom; usually one round)
                if (ballot64(e <= xr.y) == 0) break;
                int j = xj;
                uint4 sj = xs;
                if (e != xe) {
                    j = partner(e);
                    sj = p.spos[max(j, 0)];
                }
                if (e <= xr.y && j >= 0) {
                    int dz = cell_of(sj.z) - cz, dy = cell_of(sj.y) - cy;
                    dz += dz < lo ? n_c : (dz >= lo + span ? -n_c : 0);
                    dy += dy < lo ? n_c : (dy >= lo + span ? -n_c : 0);
                    const int r = (dz - lo) * span + dy - lo - rb;
                    if (dz >= lo && dz < lo + span && dy >= lo && dy < lo + span && r >= 0 && r < kMaskRows) {
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const MaskSeg g = seg[2 * r + q];
                            const int o = j - g.base;
                            const int hw = g.half + (o >> 4) - 2 * t0;
                            const int w = hw >> 1, bit = ((hw & 1) << 4) + (o & 15);
                            if (o >= 0 && o < g.len && w >= 0 && w < tw) {
                                const uint32_t old = atomicAnd(&ms[w][xa], ~(1u << bit));
                                if (MASK && ((old >> bit) & 1u)) atomicAdd(&cnt_s[xa], -1);
                                if (kTwo && cflag[w >> 1]) atomicAnd(&mc[w][xa], ~(1u << bit));
                            }
                        }
                    }
                }
            }
            __syncthreads();
            // ---- the lists, in candidate order: wave w writes atoms 8 w .. 8 w + 7
            const int aw = wave * (32 / kMaskWaves);
            if constexpr (MASK) {
                // the masks as they are, each atom's row contiguous; the last words of a
                // row padded with zeros to a multiple of four
                const int tz = t0 + kMaskWords < wend ? kMaskWords : (tw + 3) & ~3;
#pragma unroll
                for (int q = 0; q < kMaskWords; q += 64) {
                    const int w = q + lane;
                    if (w >= tz || t0 + w >= p.cap_words) continue;
                    uint32_t* const row = p.mask + (int64_t)(k0 + aw) * p.cap_words + t0;
#pragma unroll 2
                    for (int a = 0; a < 32 / kMaskWaves; ++a)
                        if (aw + a < na) row[a * p.cap_words + w] = w < tw ? ms[w][aw + a] : 0u;
                    if (wave == 0) {
                        const int2 v = make_int2(w < tw ? wt[2 * w].x : k0, w < tw ? wt[2 * w + 1].x : k0);
                        *(int2*)&p.words[2 * ((int64_t)slot * p.cap_words + t0 + w)] = v;
                    }
                }
            } else if constexpr (MODE != kListsCoreOnly) {
                constexpr int NA = 32 / kMaskWaves;
                uint32_t wd[NA], we[NA];
                int cs[NA];
                const int cap = p.cap_shell;
                int32_t* const rows = p.shell + (int64_t)(k0 + aw) * cap;
#pragma unroll
                for (int a = 0; a < NA; ++a) {
                    wd[a] = lane < tw ? ms[lane][aw + a] : 0u;
                    we[a] = lane + 64 < tw ? ms[lane + 64][aw + a] : 0u;
                    cs[a] = __builtin_amdgcn_readfirstlane(cnt_s[aw + a]);
                }
                const int nat = min(NA, na - aw);  // atoms of this wave
                for (int c = 0; c < nch; ++c) {
                    if (c == 32) {
#pragma unroll
                        for (int a = 0; a < NA; ++a) wd[a] = we[a];
                    }
                    const int c2 = 2 * (c & 31);
                    const int j = wt[4 * c + (lane >> 4)].x + (lane & 15);
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
                        if (a >= nat) continue;
                        const uint32_t m0 = (uint32_t)__builtin_amdgcn_readlane((int)wd[a], c2);
                        const uint32_t m1 = (uint32_t)__builtin_amdgcn_readlane((int)wd[a], c2 + 1);
                        const uint64_t m = ((uint64_t)m1 << 32) | m0;
                        if (m == 0) continue;
                        const int pos = (int)__builtin_amdgcn_mbcnt_hi(m1, __builtin_amdgcn_mbcnt_lo(m0, (uint32_t)cs[a]));
                        cs[a] += __popcll(m);
                        // (entries past the row's capacity are counted, not stored)
                        if (cs[a] <= cap) {
                            if (__builtin_amdgcn_inverse_ballot_w64(m)) rows[a * cap + pos] = j;
                        } else if (__builtin_amdgcn_inverse_ballot_w64(m) && pos < cap) {
                            rows[a * cap + pos] = j;
                        }
                    }
                }
                if (lane == 0)
#pragma unroll
                    for (int a = 0; a < NA; ++a)
                        if (a < nat) cnt_s[aw + a] = cs[a];
            }
            if constexpr (MODE != kListsFull) {
                // C(i), a few members per word: a lane per word (of the flagged chunks) counts, then
                // a lane per member finds its word (binary search over the members before each)
                // and its bit (by halving the word), so that a row is stored in order
                const uint64_t fl = ballot64(lane < nch && (!kTwo || cflag[lane] != 0));
                const int nf = 2 * __popcll(fl);
                if (wave == 0 && ((fl >> lane) & 1ull)) {
                    const int o = 2 * (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fl >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fl, 0u));
                    fw[o] = 2 * lane;
                    fw[o + 1] = 2 * lane + 1;
                }
                __syncthreads();
                const auto& mm = *(kTwo ? &mc : (const uint32_t(*)[kTwo ? kMaskWords : 1][33])&ms);
                for (int f0 = 0; f0 < nf; f0 += 64) {
                    const int w = f0 + lane < nf ? fw[f0 + lane] : tw;
                    for (int a = aw; a < min(aw + 32 / kMaskWaves, na); ++a) {
                        const uint32_t m = w < tw ? mm[w][a] : 0u;
                        const int n1 = __popc(m);
                        const int inc = wave_scan(n1);
                        xpre[wave][lane] = (uint16_t)(inc - n1);
                        const int cc = __builtin_amdgcn_readfirstlane(cnt_c[a]);
                        const int total_c = __builtin_amdgcn_readlane(inc, 63);
                        __builtin_amdgcn_wave_barrier();
                        int32_t* const crow = p.core + (int64_t)(k0 + a) * p.cap_core + cc;
                        for (int r = lane; r < total_c; r += 64) {
                            int i = 0;
#pragma unroll
                            for (int st = 32; st >= 1; st >>= 1) i += xpre[wave][i + st] <= (uint32_t)r ? st : 0;
                            const int wi = fw[f0 + i];
                            const int b = nth_set_bit(mm[wi][a], (uint32_t)r - xpre[wave][i]);
                            // (entries past the row's capacity are counted, not stored)
                            if (cc + r < p.cap_core) crow[r] = wt[2 * wi + (b >> 4)].x + (b & 15);
                        }
                        __builtin_amdgcn_wave_barrier();
                        if (lane == 0) cnt_c[a] = cc + total_c;
                    }
                }
            }
            __syncthreads();
        }
        wbase = wend;
        __syncthreads();
    }
    if (MASK) {
        // reported to the host: a block with more words than a row holds (its masks are
        // cut off there), and a crowded stencil row (its masks are whole: the handle only
        // changes to 32-bit entries with the next build)
        if (ballot64(long_row) != 0 && lane == 0) atomicOr(p.err, ERR_SHELL_ROW);
        if (tid == 0) {
            p.nw[slot] = min(wbase, p.cap_words);
            if (wbase > p.cap_words) atomicOr(p.err, ERR_SHELL_CAP);
            if (wbase > __hip_atomic_load(&p.maxcnt[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&p.maxcnt[2], wbase);
        }
        if (tid < na) p.slot_of[k0 + tid] = slot;
    }
    // ---- lengths: the stored ones never exceed the row capacities; a longer list sets its
    // bit in the error word and its true length reaches maxcnt
    if (wave == 0) {
        int maxc = 0, maxs = 0;
        if (lane < na) {
            const int k = k0 + lane;
            const int s = cnt_s[lane];
            const int c = cnt_c[lane];
            if (MODE != kListsFull) {
                p.ncore[k] = min(c, p.cap_core);
                if (c > p.cap_core) atomicOr(p.err, ERR_CORE_CAP);
                maxc = c;
            } else {
                p.ncore[k] = 0;
            }
            if (MODE != kListsCoreOnly) {
                p.nshell[k] = min(s, p.cap_shell);
                if (s > p.cap_shell) atomicOr(p.err, ERR_SHELL_CAP);
                maxs = s;
            }
        }
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) {
            maxc = max(maxc, __shfl_xor(maxc, off, 64));
            maxs = max(maxs, __shfl_xor(maxs, off, 64));
        }
        if (lane == 0) {
            // (one atomic only where the running maximum grows)
            if (maxc > __hip_atomic_load(&p.maxcnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&p.maxcnt[0], maxc);
            if (maxs > __hip_atomic_load(&p.maxcnt[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&p.maxcnt[1], maxs);
        }
    }
}

ListBlockShape list_block_shape(const Geometry& geo, bool core_only)
{
    ListBlockShape s;
    s.reach = core_only ? 1 : geo.reach;
    const int n_c = geo.n_c;
    s.narrow = 2 * s.reach + 1 <= n_c;
    s.lo = core_only ? -1 : geo.lo;
    s.span = core_only ? 3 : geo.hi - geo.lo + 1;
    // cells per segment: one where the stencil wraps the box (the candidates' order
    // starts at the atom's own cell there); else as many as keep a block's window
    // within one period, and a block no longer than about 12 list radii (the
    // range of the half-precision coordinates), in balanced segments
    int cap = 1;
    if (s.narrow) cap = std::max(1, std::min(n_c - 2 * s.reach, 12 * s.reach));
    s.gpr = (n_c + cap - 1) / cap;
    s.G = (n_c + s.gpr - 1) / s.gpr;
    s.gpr = (n_c + s.G - 1) / s.G;
    return s;
}

int64_t list_block_slots(const Geometry& geo, bool core_only, int64_t n)
{
    const ListBlockShape s = list_block_shape(geo, core_only);
    return n / 32 + (int64_t)geo.n_c * geo.n_c * s.gpr + 1;
}

bool exclusions_by_id(const irbe_ctx* h) { return h->max_excl > kPartnersMost; }

// Rows of more than kMaskTableWords words: the pair kernel takes a table of them per atom,
// and a word and its bases per draw from memory, where indices take one cache line per
// draw. Indices are better while their lists stay in the last-level cache (256 MiB), with
// few draws, with long core lists (the table's LDS and registers cost wavefronts) and in
// FP64 (fewer wavefronts still). The line lies where the distinct lines of 32 indices that
// the draws read pass 0.11 per word and 0.05 per core entry. Forces, indices against
// masks, 400,000 atoms of 100 per nm^3 (r_core, r_shell; draws): 0.6, 1.8; 30: 447 and
// 471 us, 50: 588 and 493, 100: 861 and 649; 0.7, 2.0; 30: 524 and 587, 100: 1,003 and
// 789; 1.0, 1.6; 100: 978 and 1,057; 1.0, 2.0; 100: 1,180 and 1,112; 0.9, 1.6; 100, at
// 45,000 atoms (255 MB): 137 and 145, at 65,000: 199 and 162; FP64, 98,304 atoms, 0.7,
// 2.0; 100: 375 and 424. The build writes masks two to three times faster, but lists are
// also kept. Lists whose indices would take more than 32 GiB, a ninth of the card, are masks in any case.
bool long_masks(const irbe_ctx* h, double words)
{
    if (1.2 * words > kMaskMaxWords) return false;
    const Geometry& g = h->geo;
    const double n = (double)h->cfg.n_atoms;
    auto members = [&](uint64_t t) {  // expected atoms within sqrt(t) quanta
        const double r = std::sqrt((double)t) / 4294967296.0;
        return 4.0 / 3.0 * 3.14159265358979323846 * r * r * r * n;
    };
    const double core = members(g.tl_core), list = members(g.tl_shell) - members(g.tl_lo);
    if (1.3 * 4.0 * list * n > 32.0 * 1073741824.0) return true;
    if (h->fp64 || 4.0 * list * n <= 256.0 * 1048576.0) return false;
    const double lines = std::max(1.0, list / 32.0);
    const double read = lines * (1.0 - std::pow(1.0 - 1.0 / lines, (double)h->cfg.p_shell));
    return read > 0.11 * words + 0.05 * core;
}

int mask_words_wanted(const irbe_ctx* h)
{
    const Geometry& g = h->geo;
    if (h->full_list || h->stencil || lists_by_lanes(h)) return 0;
    const double per_cell = (double)h->cfg.n_atoms / (double)g.n_cells;
    if (per_cell < kLaneMaxPerCell) return 0;
    const ListBlockShape s = list_block_shape(g, false);
    if (s.span * s.span > kMaskRows) return 0;
    // expected words of a block: per stencil row within reach its window's atoms
    // and, for the padding of its one or two ranges, half a word
    const double E = 1.0 / g.n_c;  // in units of the box
    const double r = std::sqrt((double)g.tl_shell) / 4294967296.0;
    const double per_row = (double)h->cfg.n_atoms / ((double)g.n_c * (double)g.n_c);  // atoms per cell row
    const double len = std::min(32.0 / per_row, s.G * E);
    double words = 0.0;
    for (int dz = s.lo; dz < s.lo + s.span; ++dz)
        for (int dy = s.lo; dy < s.lo + s.span; ++dy) {
            const double gz = std::max(0, std::abs(dz) - 1) * E, gy = std::max(0, std::abs(dy) - 1) * E;
            const double rem = r * r - gz * gz - gy * gy;
            if (s.narrow && rem <= 0.0) continue;
            const double w = s.narrow ? std::min(1.0, len + 2.0 * std::sqrt(rem)) : 1.0;
            words += w * per_row / 32.0 + 0.5;
        }
    // a margin of 1.6 for the blocks of thin cell rows (a build that needs more grows
    // the rows); rows are long where a fifth more than the mean would not fit short ones
    const bool is_long = 1.2 * words > kMaskTableWords;
    if (is_long && !long_masks(h, words)) return 0;
    const int most = is_long ? kMaskMaxWords : kMaskTableWords;
    return std::min(most, ((int)std::ceil(1.6 * words) + 8 + 3) / 4 * 4);
}

// Candidates of a stencil row up to which a handle keeps its shell lists as masks:
// 1,024, and for stencils of at most 32 rows 65,536 over their rows (rounded up to
// a power of two), so that row and place in it fit 16 bits. The masks need no such
// bound; it is the crowding up to which the compact storage is promised, and beyond
// which a few blocks' long mask rows would size the rows of all atoms.
static int mask_row_most(int rows)
{
    int bits = 0;
    while ((1 << bits) < rows) ++bits;
    return std::max(1024, 65536 >> bits);
}

hipError_t launch_list_blocks(irbe_ctx* h)
{
    const Geometry& g = h->geo;
    const ListBlockShape s = list_block_shape(g, h->stencil);
    const int64_t n = h->cfg.n_atoms;
    const int64_t slots = list_block_slots(g, h->stencil, n);
    ListBlockArgs p{};
    p.n_c = g.n_c;
    p.lo = s.lo;
    p.span = s.span;
    p.G = s.G;
    p.cap_core = h->cap_core;
    p.cap_shell = h->cap_shell;
    p.t_out = h->stencil ? g.tl_core : g.tl_shell;
    p.t_in = g.tl_core;
    p.t_lo = g.tl_lo;
    const double r_out = std::sqrt((double)p.t_out);
    const double unit = kMaskUnit / r_out;
    p.unit = (float)unit;
    p.inv_span = 1.0f / (float)s.span;
    p.max_row = mask_row_most(s.span * s.span);
    auto tu = [unit](uint64_t t) { return (float)((double)t * unit * unit); };
    p.tu_out = tu(p.t_out);
    p.tu_in = tu(p.t_in);
    p.tu_lo = tu(p.t_lo);
    p.r_in = (float)(std::sqrt((double)p.t_in) * unit * 1.00001 + 0.01);
    // FP32 threshold of the row gaps with a relative margin of 2e-6, far above their rounding
    p.tf_hi = (float)p.t_out * 1.000002f;
    p.band_valu = p.tu_out * 1.9073486328125e-6f;  // 4 x 2^-21
    p.spos = h->spos;
    p.cell_start = h->cell_start;
    p.bound = h->cell_bound;
    p.blk_start = h->blk_start;
    p.sxr = h->sxr;
    p.sxidx = h->sxidx;
    p.xidx = h->xidx;
    p.rank = h->rank;
    p.smol = h->smol;
    p.core = h->core;
    p.ncore = h->ncore;
    p.shell = h->shell;
    p.nshell = h->nshell;
    p.maxcnt = h->maxcnt;
    p.err = h->err;
    p.mask = (uint32_t*)h->shell;
    p.words = h->blk_words;
    p.nw = h->blk_nw;
    p.slot_of = h->slot_of;
    p.cap_words = h->cap_words;
    using std::false_type;
    using std::true_type;
    auto run = [&](auto mode, auto mask) {
        constexpr int M = decltype(mode)::value;
        constexpr bool K = decltype(mask)::value;
        auto go = [&](auto narrow, auto ids) {
            constexpr bool N = decltype(narrow)::value;
            k_list_blocks<M, N, K, decltype(ids)::value><<<(unsigned)slots, mask_threads(N), 0, h->stream>>>(p);
        };
        if (s.narrow && exclusions_by_id(h)) go(true_type{}, true_type{});
        else if (s.narrow) go(true_type{}, false_type{});
        else if (exclusions_by_id(h)) go(false_type{}, true_type{});
        else go(false_type{}, false_type{});
    };
    if (h->full_list) run(std::integral_constant<int, kListsFull>{}, false_type{});
    else if (h->stencil) run(std::integral_constant<int, kListsCoreOnly>{}, false_type{});
    else if (g.skin && h->masks) run(std::integral_constant<int, kListsSplitSkin>{}, true_type{});
    else if (g.skin) run(std::integral_constant<int, kListsSplitSkin>{}, false_type{});
    else if (h->masks) run(std::integral_constant<int, kListsSplit>{}, true_type{});
    else run(std::integral_constant<int, kListsSplit>{}, false_type{});
    return hipGetLastError();
}

}  // namespace irbe
