// Binning (Sec. 2.3: cells of edge >= r_core): fixed-point quantization of the
// positions, cell histogram, exclusive scan, scatter, in-cell ordering by
// (x coordinate, atom id), and the gather of a cell-sorted structure-of-arrays
// copy of the system.
#include <algorithm>
#include <type_traits>

#include "irbe_device.hpp"
#include "irbe_internal.hpp"

namespace irbe {

int64_t blocks_for(int64_t n, int block) { return (n + block - 1) / block; }

__global__ void k_fill_i32(int32_t* __restrict__ p, int32_t v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u32x4(uint4* __restrict__ p, int64_t n4)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n4) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void k_fill_u8(uint8_t* __restrict__ p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_fill_i32(hipStream_t s, int32_t* p, int32_t v, int64_t n)
{
    if (n <= 0) return hipSuccess;
    k_fill_i32<<<(unsigned)blocks_for(n, kBlock), kBlock, 0, s>>>(p, v, n);
    return hipGetLastError();
}

// Zero a device buffer with kernels (no memset nodes, so the calls stay safe
// inside captured graphs).
hipError_t launch_fill_bytes0(hipStream_t s, void* p, size_t bytes)
{
    if (bytes == 0) return hipSuccess;
    const int64_t n4 = (int64_t)(bytes / 16);
    if (n4 > 0 && ((uintptr_t)p % 16) == 0) {
        k_fill_u32x4<<<(unsigned)blocks_for(n4, kBlock), kBlock, 0, s>>>((uint4*)p, n4);
        const size_t rest = bytes - (size_t)n4 * 16;
        if (rest) k_fill_u8<<<1, kBlock, 0, s>>>((uint8_t*)p + n4 * 16, (int64_t)rest);
    } else {
        k_fill_u8<<<(unsigned)blocks_for((int64_t)bytes, kBlock), kBlock, 0, s>>>((uint8_t*)p, (int64_t)bytes);
    }
    return hipGetLastError();
}

// s = rint(frac(x / L) * 2^32) mod 2^32, computed as rint((u - floor(u)) * 2^32)
// with u = x * (1/L). Contraction is off so the FP64 rounding is exactly that
// of the separate multiply and subtract.
__device__ __forceinline__ uint32_t quantize1(double x, double inv_l, bool& bad)
{
#pragma clang fp contract(off)
    if (!isfinite(x)) {
        bad = true;
        return 0u;
    }
    const double u = x * inv_l;
    const double f = u - floor(u);
    const double t = rint(f * 4294967296.0);
    return (uint32_t)((uint64_t)t & 0xffffffffull);
}

__device__ __forceinline__ uint32_t cell_coord(uint32_t s, int n_c) { return (uint32_t)(((uint64_t)s * (uint32_t)n_c) >> 32); }

template <typename real>
__global__ __launch_bounds__(kBlock) void k_quantize_hist(int64_t n, const real* __restrict__ pos, double inv_l,
                                                          int n_c, uint4* __restrict__ sq,
                                                          int32_t* __restrict__ cell_count,
                                                          int32_t* __restrict__ slot, uint32_t* err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool bad = false;
    const uint32_t sx = quantize1((double)pos[3 * i + 0], inv_l, bad);
    const uint32_t sy = quantize1((double)pos[3 * i + 1], inv_l, bad);
    const uint32_t sz = quantize1((double)pos[3 * i + 2], inv_l, bad);
    const uint32_t cell = (cell_coord(sz, n_c) * (uint32_t)n_c + cell_coord(sy, n_c)) * (uint32_t)n_c + cell_coord(sx, n_c);
    sq[i] = make_uint4(sx, sy, sz, cell);
    // the atom's place among its cell's atoms (any order: each cell is sorted later).
    // Consecutive lanes in one cell (a molecule's atoms, neighbouring molecules of an
    // ordered input) form a run whose first lane takes the run's places with one
    // atomic; the active lanes of a wavefront are a prefix of it.
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t prev = (uint32_t)__shfl_up((int)cell, 1, 64);
    const bool head = lane == 0 || prev != cell;
    const uint64_t heads = __builtin_amdgcn_ballot_w64(head);
    const uint64_t active = __builtin_amdgcn_ballot_w64(true);
    const uint64_t upto = (2ull << lane) - 1ull;  // lanes 0 .. lane (all ones for lane 63)
    const int first = 63 - __builtin_clzll(heads & upto);
    int base = 0;
    if (head) {
        const uint64_t later = heads & ~upto;
        const int end = later ? __builtin_ctzll(later) : 64 - __builtin_clzll(active);
        base = atomicAdd(&cell_count[cell], end - lane);
    }
    slot[i] = __shfl(base, first, 64) + (lane - first);
    if (bad) atomicOr(err, ERR_NONFINITE);
}

// Exclusive scan, 1024 elements per block; the block total goes to sums[b].
constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void k_scan_block(const int32_t* __restrict__ in, int32_t* __restrict__ out,
                                                           int32_t* __restrict__ sums, int64_t n)
{
    __shared__ int32_t wave_tot[kScanBlock / 64];
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t v = i < n ? in[i] : 0;
    int32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    if (wave == 0) {
        int32_t t = lane < kScanBlock / 64 ? wave_tot[lane] : 0;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(t, off, 64);
            if (lane >= off) t += y;
        }
        if (lane < kScanBlock / 64) wave_tot[lane] = t;
    }
    __syncthreads();
    const int32_t base = wave > 0 ? wave_tot[wave - 1] : 0;
    if (i < n) out[i] = base + x - v;
    if (threadIdx.x == kScanBlock - 1) sums[blockIdx.x] = base + x;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_add(int32_t* __restrict__ out, const int32_t* __restrict__ sums, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    if (i < n && blockIdx.x > 0) out[i] += sums[blockIdx.x];
}

// The last step of the scan: the block offsets, and the total behind the last element.
__global__ __launch_bounds__(kScanBlock) void k_scan_finish(const int32_t* __restrict__ in, int32_t* __restrict__ out,
                                                            const int32_t* __restrict__ sums, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    if (i >= n) return;
    const int32_t v = out[i] + (blockIdx.x > 0 ? sums[blockIdx.x] : 0);
    out[i] = v;
    if (i == n - 1) out[n] = v + in[i];
}

// The whole scan in one workgroup, for at most kScanSmall elements: each thread
// its own run of ITEMS (a multiple of 4) in registers.
constexpr int64_t kScanSmall = 16 * kScanBlock;

template <int ITEMS>
__global__ __launch_bounds__(kScanBlock) void k_scan_small(const int32_t* __restrict__ in, int32_t* __restrict__ out, int n)
{
    __shared__ int32_t wave_tot[kScanBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = (int)threadIdx.x * ITEMS;
    int32_t v[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; q += 4) {
        int4 x = make_int4(0, 0, 0, 0);
        if (i0 + q + 3 < n) {
            x = *(const int4*)(in + i0 + q);
        } else {
            if (i0 + q < n) x.x = in[i0 + q];
            if (i0 + q + 1 < n) x.y = in[i0 + q + 1];
            if (i0 + q + 2 < n) x.z = in[i0 + q + 2];
        }
        v[q] = x.x;
        v[q + 1] = x.y;
        v[q + 2] = x.z;
        v[q + 3] = x.w;
    }
    int32_t sum = 0;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) sum += v[q];
    int32_t x = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    int32_t base = x - sum;
    for (int w = 0; w < wave; ++w) base += wave_tot[w];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int i = i0 + q;
        if (i < n) out[i] = base;
        base += v[q];
        if (i == n - 1) out[n] = base;
    }
}

// Exclusive scan of in[0..n) into out[0..n]; out[n] = total. levels holds the
// per-level block-sum buffers sized at handle creation.
static hipError_t scan_exclusive(irbe_ctx* h, const int32_t* in, int32_t* out, int64_t n)
{
    if (n <= kScanSmall) {
        if (n <= 4 * kScanBlock) k_scan_small<4><<<1, kScanBlock, 0, h->stream>>>(in, out, (int)n);
        else k_scan_small<16><<<1, kScanBlock, 0, h->stream>>>(in, out, (int)n);
        return hipGetLastError();
    }
    const int64_t nb = blocks_for(n, kScanBlock);
    int32_t* sums = h->scan_levels[0];
    k_scan_block<<<(unsigned)nb, kScanBlock, 0, h->stream>>>(in, out, sums, n);
    // scan the block totals level by level
    std::vector<int64_t> lens{nb};
    int level = 0;
    while (lens.back() > 1) {
        const int64_t m = lens.back();
        const int64_t mb = blocks_for(m, kScanBlock);
        int32_t* cur = h->scan_levels[level];
        int32_t* nxt = h->scan_levels[level + 1];
        k_scan_block<<<(unsigned)mb, kScanBlock, 0, h->stream>>>(cur, cur, nxt, m);
        lens.push_back(mb);
        ++level;
    }
    for (int lv = level - 1; lv >= 0; --lv) {
        const int64_t m = lens[lv];
        k_scan_add<<<(unsigned)blocks_for(m, kScanBlock), kScanBlock, 0, h->stream>>>(h->scan_levels[lv],
                                                                                      h->scan_levels[lv + 1], m);
    }
    k_scan_finish<<<(unsigned)nb, kScanBlock, 0, h->stream>>>(in, out, h->scan_levels[0], n);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_scatter(int64_t n, const uint4* __restrict__ sq,
                                                    const int32_t* __restrict__ cell_start,
                                                    const int32_t* __restrict__ slot, int32_t* __restrict__ perm)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    perm[cell_start[sq[i].w] + slot[i]] = (int32_t)i;
}

// The FP32 pair kernels' record of an atom: the fixed-point coordinates and the
// charge rounded to 19 mantissa bits (to nearest, ties away from zero), whose
// freed 4 low bits carry the type (n_types <= 16).
__device__ __forceinline__ uint4 pos_charge_record(uint4 s, float q, int32_t type)
{
    const uint32_t b = (__float_as_uint(q) + 8u) & ~15u;
    return make_uint4(s.x, s.y, s.z, b | ((uint32_t)type & 15u));
}

// Order each cell's atoms by (fixed-point x coordinate, atom id); sorting by x
// lets the list build trim its candidate ranges. Slot t of the cell-grouped
// order `in` holds an atom; its place in the cell is the number of the cell's
// atoms with a smaller key (keys are distinct, as the ids are): one thread per
// atom over the cell's few tens of atoms, whose loads the threads of one cell
// share. The thread then writes the atom's sorted records there (and, where it
// opens a block of the list build, the block).
template <typename real>
__global__ __launch_bounds__(kBlock) void k_cell_order(int64_t n, const int32_t* __restrict__ cell_start,
                                                       const uint4* __restrict__ sq, const int32_t* __restrict__ in,
                                                       int32_t* __restrict__ perm, const int32_t* __restrict__ type,
                                                       const real* __restrict__ q, const int32_t* __restrict__ mol,
                                                       const int32_t* __restrict__ xoff, uint4* __restrict__ spos,
                                                       real* __restrict__ sqr, uint4* __restrict__ spq,
                                                       int32_t* __restrict__ smol, int2* __restrict__ sxr,
                                                       int32_t* __restrict__ rank, int n_c, int32_t* __restrict__ brow,
                                                       int G, int gpr, int32_t* __restrict__ blk_start)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int32_t i = in[t];
    const uint4 s = sq[i];
    const int32_t b = cell_start[s.w], e = cell_start[s.w + 1];
    int32_t r = 0;
    for (int32_t u = b; u < e; u += 4) {
        // (four at a time, for their dependent loads: 0.119 -> 0.100 ms at 3.1M atoms)
        int32_t o[4];
        uint32_t xo[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = in[min(u + v, e - 1)];
#pragma unroll
        for (int v = 0; v < 4; ++v) xo[v] = sq[o[v]].x;
#pragma unroll
        for (int v = 0; v < 4; ++v) r += (u + v < e && (xo[v] < s.x || (xo[v] == s.x && o[v] < i))) ? 1 : 0;
    }
    const int32_t k = b + r;
    perm[k] = i;
    // the cell's row (z, y) and x (s.w is the cell id)
    const uint32_t row = s.w / (uint32_t)n_c;
    if (brow) brow[k] = (int32_t)(((row / (uint32_t)n_c) << 16) | (row % (uint32_t)n_c));
    spos[k] = make_uint4(s.x, s.y, s.z, (uint32_t)type[i]);
    sqr[k] = q[i];
    if (std::is_same<real, float>::value) spq[k] = pos_charge_record(s, (float)q[i], type[i]);
    smol[k] = mol[i];
    sxr[k] = make_int2(xoff[i], xoff[i + 1] - xoff[i]);
    rank[i] = k;
    if (gpr > 0) {
        // blocks of 32 atoms of a segment (G consecutive cells of a cell row, at most the cells
        // that keep a block's window within one period): those of the segment whose first atom
        // is f take the slots floor(f / 32) + segment + 0, 1, ..., which are disjoint for any
        // atom counts (at most n / 32 + segments slots, the unused ones stay 0)
        const uint32_t g = (s.w - row * (uint32_t)n_c) / (uint32_t)G;
        const int32_t f = cell_start[row * (uint32_t)n_c + g * (uint32_t)G];
        const int32_t o = k - f;
        if ((o & 31) == 0) blk_start[(f >> 5) + (int32_t)(row * (uint32_t)gpr + g) + (o >> 5)] = k + 1;
    }
}

// Excluded partners as sorted indices (same layout as the caller-order table).
__global__ __launch_bounds__(kBlock) void k_excl_sorted(int64_t n_excl, const int32_t* __restrict__ xidx,
                                                        const int32_t* __restrict__ rank, int32_t* __restrict__ sxidx)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n_excl) sxidx[e] = rank[xidx[e]];
}

hipError_t launch_bin(irbe_ctx* h, const void* pos)
{
    const int64_t n = h->cfg.n_atoms;
    const unsigned nb = (unsigned)blocks_for(n, kBlock);
    // the list maxima, the cell counts and the block slots lie in one array
    const bool blocks = !lists_by_lanes(h);
    const int64_t slots = blocks ? list_block_slots(h->geo, h->stencil, n) : 0;
    hipError_t e = launch_fill_i32(h->stream, h->maxcnt, 0, (h->cell_count - h->maxcnt) + h->geo.n_cells + slots);
    if (e != hipSuccess) return e;
    if (h->fp64)
        k_quantize_hist<double><<<nb, kBlock, 0, h->stream>>>(n, (const double*)pos, h->geo.inv_l, h->geo.n_c, h->sq,
                                                              h->cell_count, h->smol, h->err);
    else
        k_quantize_hist<float><<<nb, kBlock, 0, h->stream>>>(n, (const float*)pos, h->geo.inv_l, h->geo.n_c, h->sq,
                                                             h->cell_count, h->smol, h->err);
    e = scan_exclusive(h, h->cell_count, h->cell_start, h->geo.n_cells);
    if (e != hipSuccess) return e;
    // the atoms grouped by cell into nshell, each at the place its histogram atomic
    // returned (held in smol), then each cell ordered; nshell and smol are free until
    // the list build and k_cell_order rewrite them
    k_scatter<<<nb, kBlock, 0, h->stream>>>(n, h->sq, h->cell_start, h->smol, h->nshell);
    const ListBlockShape s = list_block_shape(h->geo, h->stencil);
    const int gpr = blocks ? s.gpr : 0;
    if (h->fp64)
        k_cell_order<double><<<nb, kBlock, 0, h->stream>>>(n, h->cell_start, h->sq, h->nshell, h->perm, h->type_orig,
                                                           (const double*)h->q_orig, h->mol_orig, h->xoff, h->spos,
                                                           (double*)h->sq_r, nullptr, h->smol, h->sxr, h->rank,
                                                           h->geo.n_c, h->brow, s.G, gpr, h->blk_start);
    else
        k_cell_order<float><<<nb, kBlock, 0, h->stream>>>(n, h->cell_start, h->sq, h->nshell, h->perm, h->type_orig,
                                                          (const float*)h->q_orig, h->mol_orig, h->xoff, h->spos,
                                                          (float*)h->sq_r, h->spq, h->smol, h->sxr, h->rank,
                                                          h->geo.n_c, h->brow, s.G, gpr, h->blk_start);
    // (the block form of the list build writes the excluded partners' sorted indices itself where they are few)
    if ((!blocks || exclusions_by_id(h)) && h->n_excl > 0)
        k_excl_sorted<<<(unsigned)blocks_for(h->n_excl, kBlock), kBlock, 0, h->stream>>>(h->n_excl, h->xidx, h->rank,
                                                                                        h->sxidx);
    return hipGetLastError();
}

// The k-vector draw: one thread per sample l draws m_l and its FP64 constants
// kcoef[4l..4l+3] = (kx, ky, kz, c_l) with c_l = ke (S/p) 4 pi / (V k^2)
// (Eqs. (2.6)-(2.8)): per axis by inverse CDF on 64-bit Philox words, the triple
// (0,0,0) redrawn.
struct KDraw {
    int P, M;
    uint64_t seed, step;
    const uint64_t* U;
    double two_pi_l, coef0;
    int4* kvec;
    double* kcoef;
};

__device__ void k_draw_sample(const KDraw& d, int l)
{
    WordStream st(d.seed, d.step, (uint32_t)l, kTagKspace);
    int m[3];
    do {
        for (int a = 0; a < 3; ++a) {
            const uint64_t hi = st.next();
            const uint64_t lo = st.next();
            const uint64_t u = (hi << 32) | lo;
            // least t in [0, 2M] with u < U[t] (U is non-decreasing, U[2M] = max)
            int a0 = 0, b0 = 2 * d.M;
            while (a0 < b0) {
                const int mid = (a0 + b0) >> 1;
                if (u < d.U[mid]) b0 = mid;
                else a0 = mid + 1;
            }
            m[a] = a0 - d.M;
        }
    } while (m[0] == 0 && m[1] == 0 && m[2] == 0);
    d.kvec[l] = make_int4(m[0], m[1], m[2], 0);
    const double kx = d.two_pi_l * m[0], ky = d.two_pi_l * m[1], kz = d.two_pi_l * m[2];
    const double k2 = kx * kx + ky * ky + kz * kz;
    d.kcoef[4 * l + 0] = kx;
    d.kcoef[4 * l + 1] = ky;
    d.kcoef[4 * l + 2] = kz;
    d.kcoef[4 * l + 3] = d.coef0 / k2;
}

// Re-quantize positions for a force evaluation on the lists of the last build:
// the sorted order (perm) is kept, positions and charges are refreshed. The first
// kd_blocks blocks draw the k-vectors instead (a chain of table look-ups that one
// launch hides behind the atoms).
template <typename real>
__global__ __launch_bounds__(kBlock) void k_requantize(int64_t n, const real* __restrict__ pos, double inv_l,
                                                       const int32_t* __restrict__ rank,
                                                       const int32_t* __restrict__ type, const real* __restrict__ q,
                                                       uint4* __restrict__ sq, uint4* __restrict__ spos,
                                                       real* __restrict__ sqr, uint4* __restrict__ spq, uint32_t* err,
                                                       int kd_blocks, KDraw kd)
{
    if ((int)blockIdx.x < kd_blocks) {
        const int l = (int)(blockIdx.x * kBlock + threadIdx.x);
        if (l < kd.P) k_draw_sample(kd, l);
        return;
    }
    const int64_t i = (int64_t)(blockIdx.x - kd_blocks) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool bad = false;
    const uint32_t sx = quantize1((double)pos[3 * i + 0], inv_l, bad);
    const uint32_t sy = quantize1((double)pos[3 * i + 1], inv_l, bad);
    const uint32_t sz = quantize1((double)pos[3 * i + 2], inv_l, bad);
    const int32_t k = rank[i];
    sq[i] = make_uint4(sx, sy, sz, sq[i].w);
    // (FP32: the pair kernels read the one record; spos and sqr stay those of the build: scattered
    // writes of 16 instead of 36 bytes per atom, 0.089 -> 0.051 ms at 3.1M atoms)
    if constexpr (std::is_same<real, float>::value) {
        spq[k] = pos_charge_record(make_uint4(sx, sy, sz, 0u), q[i], type[i]);
    } else {
        spos[k] = make_uint4(sx, sy, sz, (uint32_t)type[i]);
        sqr[k] = q[i];
    }
    if (bad) atomicOr(err, ERR_NONFINITE);
}

hipError_t launch_requantize(irbe_ctx* h, const void* pos, uint64_t step)
{
    const int64_t n = h->cfg.n_atoms;
    const int P = h->cfg.p_kspace;
    const double L = h->cfg.box_length;
    const double V = L * L * L;
    const double pi = 3.14159265358979323846;
    const KDraw kd{P, h->kM, h->cfg.seed, step, h->ktab, 2.0 * pi / L,
                   h->cfg.coulomb_k * (h->kS / (double)P) * 4.0 * pi / V, h->kvec, h->kcoef};
    const int kdb = (int)blocks_for(P, kBlock);
    const unsigned nb = (unsigned)(blocks_for(n, kBlock) + kdb);
    if (h->fp64)
        k_requantize<double><<<nb, kBlock, 0, h->stream>>>(n, (const double*)pos, h->geo.inv_l, h->rank, h->type_orig,
                                                           (const double*)h->q_orig, h->sq, h->spos,
                                                           (double*)h->sq_r, nullptr, h->err, kdb, kd);
    else
        k_requantize<float><<<nb, kBlock, 0, h->stream>>>(n, (const float*)pos, h->geo.inv_l, h->rank, h->type_orig,
                                                          (const float*)h->q_orig, h->sq, h->spos, (float*)h->sq_r,
                                                          h->spq, h->err, kdb, kd);
    return hipGetLastError();
}

// Sum of q^2 (FP64) for the self energy.
template <typename real>
__global__ __launch_bounds__(kBlock) void k_sum_q2_part(int64_t n, const real* __restrict__ q, double* __restrict__ part)
{
    __shared__ double lds[kBlock / 64];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (i < n) {
        const double x = (double)q[i];
        v = x * x;
    }
    double vals[1] = {v};
    double out;
    block_sum_vec<1, kBlock>(vals, lds, threadIdx.x, out);
    if (threadIdx.x == 0) part[blockIdx.x] = out;
}

__global__ __launch_bounds__(kReduceBlock) void k_sum_part(int64_t nb, const double* __restrict__ part, double* __restrict__ out)
{
    __shared__ double lds[kReduceBlock / 64];
    double v = 0.0;
    for (int64_t b = threadIdx.x; b < nb; b += kReduceBlock) v += part[b];
    double vals[1] = {v};
    double o;
    block_sum_vec<1, kReduceBlock>(vals, lds, threadIdx.x, o);
    if (threadIdx.x == 0) out[0] = o;
}

hipError_t launch_sum_q2(irbe_ctx* h)
{
    const int64_t n = h->cfg.n_atoms;
    const int64_t nb = blocks_for(n, kBlock);
    if (h->fp64)
        k_sum_q2_part<double><<<(unsigned)nb, kBlock, 0, h->stream>>>(n, (const double*)h->q_orig, h->q2part);
    else
        k_sum_q2_part<float><<<(unsigned)nb, kBlock, 0, h->stream>>>(n, (const float*)h->q_orig, h->q2part);
    k_sum_part<<<1, kReduceBlock, 0, h->stream>>>(nb, h->q2part, h->sumq2);
    return hipGetLastError();
}

// The LJ tables as kernel arguments (at most 1 KiB).
template <typename real>
struct LjArg {
    LJ<real> tab[kLjArgTypes * kLjArgTypes];
    real raw[2 * kLjArgTypes * kLjArgTypes];
};

template <typename real>
__global__ __launch_bounds__(64) void k_store_lj(LjArg<real> a, int nt2, LJ<real>* __restrict__ tab,
                                                 real* __restrict__ raw)
{
    const int t = threadIdx.x;
    if (t < nt2) tab[t] = a.tab[t];
    if (t < 2 * nt2) raw[t] = a.raw[t];
}

template <typename real>
hipError_t launch_store_lj(irbe_ctx* h, const LJ<real>* tab, const real* raw)
{
    const int nt2 = h->cfg.n_types * h->cfg.n_types;
    if (h->cfg.n_types > kLjArgTypes) return hipErrorInvalidValue;
    LjArg<real> a{};
    std::copy(tab, tab + nt2, a.tab);
    std::copy(raw, raw + 2 * nt2, a.raw);
    k_store_lj<real><<<1, 64, 0, h->stream>>>(a, nt2, (LJ<real>*)h->lj, (real*)h->lj_raw);
    return hipGetLastError();
}

template hipError_t launch_store_lj<float>(irbe_ctx*, const LJ<float>*, const float*);
template hipError_t launch_store_lj<double>(irbe_ctx*, const LJ<double>*, const double*);

}  // namespace irbe
