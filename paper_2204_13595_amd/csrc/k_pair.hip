// Short-range part of the force (Sec. 2.3) and its adjoint.
//
// Forward, per atom i (cell order), Eqs. (2.10)-(2.12):
//   F_i = sum_{j in C(i)} f_ij + w_i sum_{j in B(i)} f_ij + F_i^excl
// with B(i) a batch of p_shell ranks of S(i) drawn without replacement by
// Floyd's algorithm from the Philox word stream of (seed, step, caller id of
// i), w_i = N_S / p_shell (all members and w_i = 1 when N_S <= p_shell). The
// per-block FP64 sums of the uncorrected short-range force give F^corr.
// Full-list mode: one list of every pair within r_shell, weight 1.
// Stencil sampling (STENCIL): the ranks are drawn from K(i), the atoms of the
// shell stencil's cells (N_S replaced by |K(i)|), turned into atom indices by
// k_stencil_decode, and a drawn atom contributes only when it lies in the
// shell annulus T_c < D^2 <= T_s at the current positions (i itself and i's
// molecule come out of the decode as -1).
// Lists built with a skin (skin): every list entry is tested at the current
// positions, core entries counting only at D^2 <= T_c, shell entries only at
// T_c < D^2 <= T_s and full-list entries only at D^2 <= T_s.
#include <algorithm>
#include <type_traits>

#include "irbe_device.hpp"
#include "irbe_internal.hpp"

namespace irbe {

template <typename real>
struct PairParams {
    real quantum;   // L / 2^32
    real q2;        // quantum^2
    real beta;
    real kbeta;     // 0.45 beta
    real gexp;      // -beta^2 log2(e)
    real cgauss;    // 2 beta / sqrt(pi)
    real ke;
};

template <typename real>
static PairParams<real> pair_params(const irbe_ctx* h)
{
    PairParams<real> pp;
    const double beta = h->cfg.ewald_beta;
    pp.quantum = (real)h->geo.quantum;
    pp.q2 = (real)(h->geo.quantum * h->geo.quantum);
    pp.beta = (real)beta;
    pp.kbeta = (real)(0.45 * beta);
    pp.gexp = (real)(-beta * beta * 1.4426950408889634);
    pp.cgauss = (real)(2.0 * beta / 1.7724538509055160273);
    pp.ke = (real)h->cfg.coulomb_k;
    return pp;
}

// Position (type in .w) and charge of sorted atom j. FP32 evaluations read one
// 16-byte record: the fixed-point coordinates and, in the fourth word, the
// charge rounded to 19 mantissa bits (relative change below 2^-20) with the
// atom's type in the 4 bits this frees, so that a pair costs one gather
// instead of two; FP64 evaluations read the position and the exact charge.
template <typename real>
struct Atoms {
    const uint4* __restrict__ spos;
    const real* __restrict__ sqr;
    const uint4* __restrict__ spq;
    __device__ __forceinline__ void get(int64_t j, uint4& p, real& q) const
    {
        if constexpr (std::is_same<real, float>::value) {
            const uint4 r = spq[j];
            p = make_uint4(r.x, r.y, r.z, r.w & 15u);
            q = __uint_as_float(r.w & ~15u);
        } else {
            p = spos[j];
            q = sqr[j];
        }
    }
};

// Exact squared separation in quanta (minimum image through 32-bit wrap-around).
__device__ __forceinline__ uint64_t dist2_q(uint4 a, uint4 b)
{
    const int32_t dx = (int32_t)(b.x - a.x);
    const int32_t dy = (int32_t)(b.y - a.y);
    const int32_t dz = (int32_t)(b.z - a.z);
    return (uint64_t)((int64_t)dx * dx) + (uint64_t)((int64_t)dy * dy) + (uint64_t)((int64_t)dz * dz);
}

// The shell-membership test on exact squared separations in quanta
// (T_c < D^2 <= T_s), used by stencil sampling and by lists built with a skin.
__device__ __forceinline__ bool in_annulus(uint4 a, uint4 b, uint64_t t_lo, uint64_t t_hi)
{
    const uint64_t d2 = dist2_q(a, b);
    return d2 > t_lo && d2 <= t_hi;
}

// The pair terms come in two forms. Full lists and lists kept with a skin (forces
// only) and the gradients take the fused one: separations in quanta scaled once
// per atom, erfc through exp(x^2) erfc(x), so that one exponential serves both
// terms of Eq. (2.10) (errors no larger).
// Lists rebuilt every step, and every energy, keep the plain form: the MD state
// integrated from those forces, and the FP64 energies, virials and LJ gradients
// summed from the FP32 terms, resolve a change of their last bits, and runs are
// to be reproduced bit for bit.
// The fused form's products with separations in quanta (up to 2^31) would overflow FP32
// where the force itself is 10^30 and less (atoms within 0.002 nm of each other), so its
// charges and LJ coefficients are scaled by 2^-32, which rounds nothing, and the sums
// by the box length instead of the quantum: the same bits wherever both are finite.
constexpr double kFusedScale = 2.3283064365386963e-10;  // 2^-32
constexpr bool fused_form(bool full, bool ev, bool skin) { return !ev && (full || skin); }

// Separation in quanta (minimum image).
template <typename real>
__device__ __forceinline__ void separation_q(uint4 a, uint4 b, real& dx, real& dy, real& dz)
{
    dx = (real)(int32_t)(b.x - a.x);
    dy = (real)(int32_t)(b.y - a.y);
    dz = (real)(int32_t)(b.z - a.z);
}

template <typename real>
__device__ __forceinline__ void separation(uint4 a, uint4 b, real quantum, real& dx, real& dy, real& dz)
{
    dx = (real)(int32_t)(b.x - a.x) * quantum;
    dy = (real)(int32_t)(b.y - a.y) * quantum;
    dz = (real)(int32_t)(b.z - a.z) * quantum;
}

// The radial parts of a pair: 1/r, 1/r^2, exp(-(beta r)^2) and
// g = erfc(beta r)/r + cgauss exp(-(beta r)^2) (and erfc(beta r) for energies).
template <typename real>
struct Radial {
    real rinv, rinv2, ex, ec, g;
};

template <typename real>
__device__ __forceinline__ Radial<real> radial(real r2, const PairParams<real>& pp)
{
    using M = Math<real>;
    Radial<real> o;
    o.rinv = M::rsqrt_(r2);
    const real r = r2 * o.rinv;
    const real br = pp.beta * r;
    o.ex = M::gauss_(br, pp.gexp * r2);
    o.rinv2 = o.rinv * o.rinv;
    if constexpr (std::is_same<real, float>::value) {
        const float e1 = M::erfcx_(pp.kbeta, r);
        o.ec = o.ex * e1;
        o.g = o.ex * fmaf(e1, o.rinv, pp.cgauss);
    } else {
        o.ec = erfc(br);
        o.g = o.ec * o.rinv + pp.cgauss * o.ex;
    }
    return o;
}

// phi of f_ij = phi r_ij (Eq. (2.10)), fused form.
template <typename real>
__device__ __forceinline__ real pair_phi_fused(real r2, real qq, const LJ<real>& lj, const PairParams<real>& pp)
{
    const Radial<real> o = radial(r2, pp);
    const real r6 = o.rinv2 * o.rinv2 * o.rinv2;
    const real ljf = r2 < lj.rc2 ? r6 * (lj.a12 * r6 - lj.b6) : (real)0;
    return -o.rinv2 * (qq * o.g + ljf);
}

// phi of f_ij = phi r_ij (Eq. (2.10)) and, when EV, the pair energies.
template <typename real, bool EV>
__device__ __forceinline__ real pair_phi(real r2, real qq, const LJ<real>& lj, const PairParams<real>& pp, real& uc,
                                         real& ul)
{
    using M = Math<real>;
    const real rinv = M::rsqrt_(r2);
    const real r = r2 * rinv;
    const real br = pp.beta * r;
    const real ex = M::exp_(-br * br);
    const real ec = M::erfc_ex(br, ex);
    const real rinv2 = rinv * rinv;
    const real r6 = rinv2 * rinv2 * rinv2;
    const bool lj_on = r2 < lj.rc2;
    real phi = -qq * rinv2 * (ec * rinv + pp.cgauss * ex);
    phi -= lj_on ? r6 * rinv2 * (lj.a12 * r6 - lj.b6) : (real)0;
    if (EV) {
        uc = qq * ec * rinv;
        ul = lj_on ? r6 * (lj.c12 * r6 - lj.c6) - lj.esh : (real)0;
    }
    return phi;
}

// Force, energy and virial sums of one list (core or shell batch). Fused form:
// forces over the box length.
template <typename real>
struct PairSum {
    real fx = 0, fy = 0, fz = 0;
    real uc = 0, ul = 0;
    real v[6] = {0, 0, 0, 0, 0, 0};
};

template <typename real, bool EV, bool FUSED>
__device__ __forceinline__ void add_pair(PairSum<real>& a, uint4 si, real qi, uint4 sj, real qj, const LJ<real>& lje,
                                         const PairParams<real>& pp)
{
    real dx, dy, dz;
    if constexpr (FUSED) {
        separation_q(si, sj, dx, dy, dz);
        const real r2 = (dx * dx + dy * dy + dz * dz) * pp.q2;
        const real phi = pair_phi_fused<real>(r2, qi * qj, lje, pp);
        a.fx += phi * dx;
        a.fy += phi * dy;
        a.fz += phi * dz;
    } else {
        separation(si, sj, pp.quantum, dx, dy, dz);
        // (written out, so that every kernel rounds the terms alike)
        const real r2 = fma(dz, dz, fma(dx, dx, dy * dy));
        real uc, ul;
        const real phi = pair_phi<real, EV>(r2, qi * qj, lje, pp, uc, ul);
        a.fx += phi * dx;
        a.fy += phi * dy;
        a.fz += phi * dz;
        if (EV) {
            a.uc += uc;
            a.ul += ul;
            a.v[0] += phi * dx * dx; a.v[1] += phi * dy * dy; a.v[2] += phi * dz * dz;
            a.v[3] += phi * dx * dy; a.v[4] += phi * dx * dz; a.v[5] += phi * dy * dz;
        }
    }
}

// One Floyd step: draw r in [0, t], insert r or (if taken) t into the bitmap
// (word w of this thread's bitmap at bits[w * stride]). The words of r and of
// t are read together (one memory round trip per step); either one is then
// updated. Every element inserted before this step is below t, so t's own bit
// is clear.
__device__ __forceinline__ int floyd_step(WordStream& st, uint32_t* bits, int stride, int t)
{
    const int r = (int)st.below((uint32_t)t + 1u);
    const uint32_t wr = bits[(r >> 5) * stride];
    const uint32_t wt = bits[(t >> 5) * stride];
    const bool taken = (wr >> (r & 31)) & 1u;
    const int v = taken ? t : r;
    bits[(v >> 5) * stride] = (taken ? wt : wr) | (1u << (v & 31));
    return v;
}

// Floyd's algorithm for atom k (sorted index) when N_S > p~: p~ ranks of
// [0, N_S) without replacement, from the word stream of its caller id.
__device__ __forceinline__ void floyd_row(int64_t k, int ns, const int32_t* __restrict__ perm, int p_shell,
                                          int p_stride, uint64_t seed, uint64_t step, uint32_t* bits, int stride,
                                          uint16_t* __restrict__ ranks)
{
    const int words = (ns + 31) >> 5;
    for (int t = 0; t < words; ++t) bits[t * stride] = 0u;
    WordStream st(seed, step, (uint32_t)perm[k], kTagShell);
    uint16_t* out = ranks + k * (int64_t)p_stride;
    const int t0 = ns - p_shell;
    int c = 0;
    for (; c + 4 <= p_shell; c += 4) {
        const uint32_t v0 = (uint32_t)floyd_step(st, bits, stride, t0 + c);
        const uint32_t v1 = (uint32_t)floyd_step(st, bits, stride, t0 + c + 1);
        const uint32_t v2 = (uint32_t)floyd_step(st, bits, stride, t0 + c + 2);
        const uint32_t v3 = (uint32_t)floyd_step(st, bits, stride, t0 + c + 3);
        *(uint2*)(out + c) = make_uint2(v0 | (v1 << 16), v2 | (v3 << 16));
    }
    for (; c < p_shell; ++c) out[c] = (uint16_t)floyd_step(st, bits, stride, t0 + c);
}

// The same ranks, four steps at a time, for bitmaps in LDS. The four words of
// one Philox block serve steps c .. c+3. Unless a lane's multiply-shift needs
// its rejection test (low product word below the bound: about one draw in
// 10^7), the four draws r are then known before any bitmap access, and their
// membership tests go to LDS together as test-and-set operations, which return
// each word as it was before their own bit was set: r is taken when its bit was
// already set, or when it equals the t of an earlier step of the four that was
// taken (that t is inserted only after the four). A free r is inserted by its
// own test-and-set. From the first block in which some lane of the wavefront
// needs the rejection test, and for the steps after the last full block, the
// one-step form continues with the same word stream.
__device__ __forceinline__ void floyd_row_lds(int64_t k, int ns, const int32_t* __restrict__ perm, int p_shell,
                                              int p_stride, uint64_t seed, uint64_t step, uint32_t* bits, int stride,
                                              uint16_t* __restrict__ ranks)
{
    const int words = (ns + 31) >> 5;
    for (int t = 0; t < words; ++t) bits[t * stride] = 0u;
    WordStream st(seed, step, (uint32_t)perm[k], kTagShell);
    uint16_t* out = ranks + k * (int64_t)p_stride;
    const int t0 = ns - p_shell;
    int c = 0;
    for (; c + 4 <= p_shell; c += 4) {
        const Words4 b = philox10(st.c0, st.block, st.c2, st.c3, st.k0, st.k1);
        const uint32_t w[4] = {b.x, b.y, b.z, b.w};
        uint32_t r[4];
        bool hard = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bound = (uint32_t)(t0 + c + j) + 1u;
            const uint64_t m = (uint64_t)w[j] * bound;
            hard |= (uint32_t)m < bound;
            r[j] = (uint32_t)(m >> 32);
        }
        if (__builtin_amdgcn_ballot_w64(hard) != 0) break;  // this block again, one step at a time
        ++st.block;
        uint32_t old[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            old[j] = __hip_atomic_fetch_or(&bits[(r[j] >> 5) * stride], 1u << (r[j] & 31), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WAVEFRONT);
        uint32_t v[4];
        bool taken[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t t = (uint32_t)(t0 + c + j);
            bool tk = (old[j] >> (r[j] & 31)) & 1u;
#pragma unroll
            for (int i = 0; i < j; ++i) tk |= taken[i] && r[j] == t - (uint32_t)(j - i);
            taken[j] = tk;
            v[j] = tk ? t : r[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t t = (uint32_t)(t0 + c + j);
            __hip_atomic_fetch_or(&bits[(t >> 5) * stride], taken[j] ? 1u << (t & 31) : 0u, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        *(uint2*)(out + c) = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
    }
    for (; c < p_shell; ++c) out[c] = (uint16_t)floyd_step(st, bits, stride, t0 + c);
}

// ---------------------------------------------------------------------------
// Forward, cooperative form: the shell batch ranks are drawn first (one thread
// per atom, Floyd's algorithm into a row of 16-bit ranks), then one wavefront
// evaluates one atom at a time with its lanes spread over the atom's core
// list, its batch and its excluded pairs. Each atom's list rows are then read
// by one wavefront at one time (coalesced for the core and full lists, one
// short burst of lines for the sampled shell ranks) instead of entry by entry
// over the whole kernel.
// ---------------------------------------------------------------------------
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_draw_batches(int64_t n, const int32_t* __restrict__ perm,
                                                        const int32_t* __restrict__ nshell, int p_shell, int p_stride,
                                                        uint64_t seed, uint64_t step, uint16_t* __restrict__ ranks)
{
    extern __shared__ uint32_t bitmap[];
    const int64_t k = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (k >= n) return;
    const int ns = nshell[k];
    if (ns <= p_shell) return;
    floyd_row_lds(k, ns, perm, p_shell, p_stride, seed, step, bitmap + threadIdx.x, BLOCK, ranks);
}

// The same for systems that leave the chip idle at one thread per atom: half a
// wavefront per atom, lane l drawing steps 4 l .. 4 l + 3 from block l of the atom's
// words (at most 128 steps). Floyd's rule without the order of the steps: the draw r
// of step c is taken when an earlier step drew r too, or when r = t0 + c' is the t of
// an earlier step c' whose draw was taken. The first comes from the smallest step of
// each value (LDS minimum), the second by repetition until nothing changes. A half
// that meets the rejection test of the multiply-shift takes the one-step form.
// What bounds the other form there is one thread's chain of 25 blocks and bitmap round
// trips, about 14 us for 100 draws however few the atoms. One thread against half a
// wavefront, 100 draws: 14.3 and 4.8 us at 2,703 atoms, 14.9 and 7.8 at 12,288, but 29.6
// and 33.3 at 98,304, where this form's idle lanes (25 of 32 draw) cost more than the
// chain. The fewer the draws, the shorter the chain and the more lanes idle: draw and
// pairs with 10 draws, 24,000 ions: 14.0 and 16.7 us; 24,000 atoms of water, 20 draws:
// 26.5 and 29.2, 50: 31.1 and 30.7; 8,000 atoms, 10: 14.8 and 14.8. The line is that of
// equal times, about 500 (draws - 4) atoms; up to 8,192 atoms few draws take either alike.
constexpr int kHalfDrawBlock = 256;
constexpr int kHalfDrawMost = 128;         // steps
constexpr int64_t kHalfDrawAtoms = 32768;

static bool half_draw(int64_t n, int p_shell)
{
    return p_shell <= kHalfDrawMost &&
           n < std::min<int64_t>(kHalfDrawAtoms, std::max<int64_t>(8192, 500 * (int64_t)(p_shell - 4)));
}

__global__ __launch_bounds__(kHalfDrawBlock) void k_draw_batches_half(int64_t n, const int32_t* __restrict__ perm,
                                                                      const int32_t* __restrict__ nshell, int p_shell,
                                                                      int p_stride, uint64_t seed, uint64_t step,
                                                                      int table, uint16_t* __restrict__ ranks)
{
    extern __shared__ uint32_t bitmap[];
    const int half = (int)threadIdx.x >> 5, l = (int)threadIdx.x & 31;
    const int64_t k = (int64_t)blockIdx.x * (kHalfDrawBlock / 32) + half;
    if (k >= n) return;
    const int ns = nshell[k];
    if (ns <= p_shell) return;
    uint32_t* const first = bitmap + half * table;  // [ns] smallest step that drew the value
    const int t0 = ns - p_shell;
    const Words4 w = philox10((uint32_t)perm[k], (uint32_t)l, (uint32_t)step,
                              ((uint32_t)(step >> 32) << 1) | kTagShell, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint32_t words[4] = {w.x, w.y, w.z, w.w};
    int r[4];
    bool in[4], taken[4], reject = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = 4 * l + u;
        in[u] = c < p_shell;
        const uint32_t bound = (uint32_t)(t0 + c) + 1u;
        const uint64_t m = (uint64_t)words[u] * bound;
        r[u] = in[u] ? (int)(m >> 32) : 0;
        if (in[u] && (uint32_t)m < bound && (uint32_t)m < (0u - bound) % bound) reject = true;
    }
    // (the lanes of a half run together: the LDS operations below take effect in program order)
    const uint64_t half_mask = 0xffffffffull << (threadIdx.x & 32);
    if ((__builtin_amdgcn_ballot_w64(reject) & half_mask) != 0) {
        if (l == 0) floyd_row(k, ns, perm, p_shell, p_stride, seed, step, first, 1, ranks);
        return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (in[u]) first[r[u]] = 0xffffffffu;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (in[u]) atomicMin(&first[r[u]], (uint32_t)(4 * l + u));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int u = 0; u < 4; ++u) taken[u] = in[u] && first[r[u]] != (uint32_t)(4 * l + u);
    for (;;) {
        // the taken steps of this half, one word per step of a lane
        uint32_t word[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) word[u] = (uint32_t)(__builtin_amdgcn_ballot_w64(taken[u]) >> (threadIdx.x & 32));
        bool more = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = r[u] - t0;  // the step whose t the draw is
            if (!in[u] || taken[u] || c < 0 || c >= 4 * l + u) continue;
            const uint32_t wc = (c & 2) ? ((c & 1) ? word[3] : word[2]) : ((c & 1) ? word[1] : word[0]);
            if ((wc >> (c >> 2)) & 1u) taken[u] = more = true;
        }
        if ((__builtin_amdgcn_ballot_w64(more) & half_mask) == 0) break;
    }
    if (4 * l < p_shell) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = (uint32_t)(taken[u] ? t0 + 4 * l + u : r[u]);
        *(uint2*)(ranks + k * (int64_t)p_stride + 4 * l) = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
    }
}

// The same with the bitmaps in device memory, for lists too long for LDS: a
// grid of `threads` threads takes the atoms in turn, thread t's bitmap word w
// at bits[w * threads + t].
__global__ __launch_bounds__(256) void k_draw_batches_global(int64_t n, const int32_t* __restrict__ perm,
                                                             const int32_t* __restrict__ nshell, int p_shell,
                                                             int p_stride, uint64_t seed, uint64_t step,
                                                             uint32_t* __restrict__ bits, int threads,
                                                             uint16_t* __restrict__ ranks)
{
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    if (t >= threads) return;
    for (int64_t k = t; k < n; k += threads) {
        const int ns = nshell[k];
        if (ns > p_shell) floyd_row(k, ns, perm, p_shell, p_stride, seed, step, bits + t, threads, ranks);
    }
}

// Stencil sampling: K(i), the atoms of the shell stencil's cells around atom
// i's cell at the build, runs over the stencil rows (dz, dy) in order, each row
// being the cells cx + lo .. cx + lo + span - 1 (cyclic), i.e. at most two
// index ranges of the cell-sorted atoms. A wavefront keeps the rows of one cell
// in LDS (one row per lane, prefix sums by wave scan) and turns a rank of K(i)
// into an atom with a binary search over the rows' first ranks.
constexpr int kDecodeRows = 128;  // stencil rows (span^2) supported

template <int ROWS>
struct StencilRows {
    int32_t pre[ROWS];  // first rank of each row
    int32_t a[ROWS];    // first atom of the row's first range
    int32_t la[ROWS];   // length of the first range
    int32_t b[ROWS];    // first atom of the second range (after the wrap)
};

struct StencilArgs {
    const int32_t* cell_start;
    const int32_t* scell;  // cell of each sorted atom at the build
    const int32_t* smol;   // molecule of each sorted atom
    int n_c, lo, span;
};

__device__ __forceinline__ int wrap_cell(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

// The rows of build cell `cell` into T (every lane of the wavefront takes part).
template <int ROWS>
__device__ void stencil_rows_build(StencilRows<ROWS>& T, int cell, const StencilArgs& sa, int lane)
{
    const int n_c = sa.n_c, span = sa.span, nrows = span * span;
    const int cx = cell % n_c, cy = (cell / n_c) % n_c, cz = cell / (n_c * n_c);
    const int x0 = wrap_cell(cx + sa.lo, n_c);
    const int la_c = min(span, n_c - x0);  // cells before the wrap
    int base = 0;
    for (int t0 = 0; t0 < nrows; t0 += 64) {
        const int t = t0 + lane;
        int len = 0, va = 0, vla = 0, vb = 0;
        if (t < nrows) {
            const int z = wrap_cell(cz + t / span + sa.lo, n_c);
            const int y = wrap_cell(cy + t % span + sa.lo, n_c);
            const int row = (z * n_c + y) * n_c;
            va = sa.cell_start[row + x0];
            vla = sa.cell_start[row + x0 + la_c] - va;
            vb = sa.cell_start[row];
            len = vla + (span > la_c ? sa.cell_start[row + span - la_c] - vb : 0);
        }
        int incl = len;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        if (t < nrows) {
            T.pre[t] = base + incl - len;
            T.a[t] = va;
            T.la[t] = vla;
            T.b[t] = vb;
        }
        base += __shfl(incl, 63, 64);
    }
}

// Atom (sorted index) of rank r of K(i) for a cell whose rows are in T: the row
// is the last one whose first rank is <= r.
template <int ROWS>
__device__ __forceinline__ int stencil_rows_atom(const StencilRows<ROWS>& T, int nrows, int r)
{
    int lo_k = 0, hi_k = nrows - 1;
    while (lo_k < hi_k) {
        const int mid = (lo_k + hi_k + 1) >> 1;
        if (T.pre[mid] <= r) lo_k = mid;
        else hi_k = mid - 1;
    }
    const int o = r - T.pre[lo_k];
    const int la = T.la[lo_k];
    return o < la ? T.a[lo_k] + o : T.b[lo_k] + (o - la);
}

// Shell lists as masks: a wavefront finds a member of an atom's row by its rank, the
// word by binary search over the members before each, the bit by halving the word.
// Rows of up to kMaskTableWords words (SHORT) lie in LDS whole, with the words' first
// candidates (those of the atom's block). Longer ones (LONG) keep only the members before
// each word there, in 16 bits; a search's word and bases then come from memory, in one
// round trip of two loads.
enum { kIndices = 0, kMasksShort = 1, kMasksLong = 2 };

template <int ENC>
struct MaskTable {};

template <>
struct MaskTable<kMasksShort> {
    uint32_t pre[kMaskTableWords];   // members before word w
    uint32_t word[kMaskTableWords];
    int32_t base[2 * kMaskTableWords];  // sorted index of the first candidate of half q of word w at 2 w + q
};

template <>
struct MaskTable<kMasksLong> {
    uint16_t pre[kMaskMaxWords];  // members before word w
};

// The words of an atom's row that a lane loads ahead of the table: four of every 256.
template <int ENC>
struct MaskWords {
    uint4 v[ENC == kMasksLong ? 2 : 1];
};

// This lane's four words of words q .. q + 255 of atom a's row (nw words).
__device__ __forceinline__ uint4 mask_load(const ShellMasks& sm, int64_t a, int nw, int q, int lane)
{
    return q + 4 * lane < nw ? *(const uint4*)(sm.mask + a * (int64_t)sm.cap + q + 4 * lane) : make_uint4(0u, 0u, 0u, 0u);
}

template <int ENC>
__device__ __forceinline__ MaskWords<ENC> mask_ahead(const ShellMasks& sm, int64_t a, int nw, int lane)
{
    MaskWords<ENC> m;
    m.v[0] = mask_load(sm, a, nw, 0, lane);
    if constexpr (ENC == kMasksLong) m.v[1] = mask_load(sm, a, nw, 256, lane);
    return m;
}

// The first candidates of the words of block `slot`.
__device__ __forceinline__ void mask_bases(MaskTable<kMasksShort>& T, const ShellMasks& sm, int slot, int nw, int lane)
{
    const int32_t* const b = sm.words + 2 * (int64_t)slot * sm.cap;
#pragma unroll
    for (int q = 0; q < 2 * kMaskTableWords; q += 256)
        if (q + 4 * lane < 2 * nw) *(int4*)&T.base[q + 4 * lane] = *(const int4*)(b + q + 4 * lane);
    __builtin_amdgcn_wave_barrier();
}

// The members before each of this lane's four words (among the 256 of the lanes); c[3]: in all four.
__device__ __forceinline__ uint32_t mask_scan(uint4 m, uint32_t (&c)[4])
{
    c[0] = __popc(m.x);
    c[1] = c[0] + __popc(m.y);
    c[2] = c[1] + __popc(m.z);
    c[3] = c[2] + __popc(m.w);
    int x = (int)c[3];
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return (uint32_t)x - c[3];
}

// The lanes' words and the members before each into the table (the wavefront's
// own: its later reads follow these writes in order).
__device__ __forceinline__ void mask_rows(MaskTable<kMasksShort>& T, const ShellMasks&, int64_t, int,
                                          const MaskWords<kMasksShort>& mk, int lane)
{
    uint32_t c[4];
    const uint32_t p = mask_scan(mk.v[0], c);
    *(uint4*)&T.pre[4 * lane] = make_uint4(p, p + c[0], p + c[1], p + c[2]);
    *(uint4*)&T.word[4 * lane] = mk.v[0];
    __builtin_amdgcn_wave_barrier();
}

// (the words past the first 512 are loaded here)
__device__ __forceinline__ void mask_rows(MaskTable<kMasksLong>& T, const ShellMasks& sm, int64_t a, int nw,
                                          const MaskWords<kMasksLong>& mk, int lane)
{
    uint32_t before = 0;
    for (int q = 0; q < nw; q += 256) {
        const uint4 m = q == 0 ? mk.v[0] : (q == 256 ? mk.v[1] : mask_load(sm, a, nw, q, lane));
        uint32_t c[4];
        const uint32_t p = before + mask_scan(m, c);
        *(uint2*)&T.pre[q + 4 * lane] = make_uint2((p & 0xffffu) | ((p + c[0]) << 16), ((p + c[1]) & 0xffffu) | ((p + c[2]) << 16));
        before = bcast(p + c[3], 63);
    }
    __builtin_amdgcn_wave_barrier();
}

// Sorted index of member r (below the list's length) of a row of nw words
// (clamped to the last atom: the rows of a build that reported too few words
// per row still read in bounds).
__device__ __forceinline__ int mask_member(const MaskTable<kMasksShort>& T, const ShellMasks&, int64_t, int, int nw, int r,
                                           int last)
{
    int w = 0;
    if (nw > 128 && T.pre[128] <= (uint32_t)r) w = 128;
#pragma unroll
    for (int s = 64; s >= 1; s >>= 1) w += T.pre[w + s] <= (uint32_t)r ? s : 0;
    const int b = nth_set_bit(T.word[w], (uint32_t)r - T.pre[w]);
    return (int)min((uint32_t)(T.base[2 * w + (b >> 4)] + (b & 15)), (uint32_t)last);
}

// (a, slot: the atom and its block, whose rows in memory hold the word and its bases)
__device__ __forceinline__ int mask_member(const MaskTable<kMasksLong>& T, const ShellMasks& sm, int64_t a, int slot, int nw,
                                           int r, int last)
{
    int w = 0;
    for (int s = 1 << (31 - __builtin_clz(nw | 1)); s >= 1; s >>= 1)
        w += w + s < nw && (uint32_t)T.pre[w + s] <= (uint32_t)r ? s : 0;
    const uint32_t m = sm.mask[a * (int64_t)sm.cap + w];
    const int2 base = *(const int2*)&sm.words[2 * ((int64_t)slot * sm.cap + w)];
    const int b = nth_set_bit(m, (uint32_t)r - T.pre[w]);
    return (int)min((uint32_t)((b >> 4 ? base.y : base.x) + (b & 15)), (uint32_t)last);
}

// A drawn atom j of atom a (sorted indices) counts as a shell pair: not a
// itself, not of a's molecule, and in the shell annulus.
__device__ __forceinline__ bool stencil_member(int64_t a, int j, int mi, int mj, uint4 si, uint4 sj, uint64_t t_core,
                                               uint64_t t_shell)
{
    return j >= 0 && j != (int)a && !(mi >= 0 && mj == mi) && in_annulus(si, sj, t_core, t_shell);
}

// Read-back of the decoded batch (the atoms at the drawn ranks, -1 for i itself
// and i's molecule): one wavefront per apw consecutive atoms.
constexpr int kDecodeBlock = 256;

__global__ __launch_bounds__(kDecodeBlock) void k_stencil_decode(int64_t n, int apw, StencilArgs sa,
                                                                 const int32_t* __restrict__ nshell, int p_shell,
                                                                 int p_stride, const uint16_t* __restrict__ ranks,
                                                                 int32_t* __restrict__ batch_j)
{
    __shared__ StencilRows<kDecodeRows> rows[kDecodeBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t a0 = ((int64_t)blockIdx.x * (kDecodeBlock / 64) + wave) * apw;
    const int64_t a1 = min(n, a0 + apw);
    const int nrows = sa.span * sa.span;
    int cur = -1;
    for (int64_t a = a0; a < a1; ++a) {
        const int cell = sa.scell[a];
        if (cell != cur) {
            stencil_rows_build(rows[wave], cell, sa, lane);
            cur = cell;
        }
        const int m = nshell[a];
        const bool sample = m > p_shell;
        const int cnt = sample ? p_shell : m;
        const int mi = sa.smol[a];
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        int32_t* out = batch_j + a * (int64_t)p_stride;
        // the lane's first two slots with their loads issued together
        const int q0 = lane < cnt ? (sample ? (int)rrow[lane] : lane) : -1;
        const int q1 = lane + 64 < cnt ? (sample ? (int)rrow[lane + 64] : lane + 64) : -1;
        int j0 = q0 >= 0 ? stencil_rows_atom(rows[wave], nrows, q0) : -1;
        int j1 = q1 >= 0 ? stencil_rows_atom(rows[wave], nrows, q1) : -1;
        const int m0 = sa.smol[max(j0, 0)], m1 = sa.smol[max(j1, 0)];
        if (j0 == (int)a || (mi >= 0 && m0 == mi)) j0 = -1;
        if (j1 == (int)a || (mi >= 0 && m1 == mi)) j1 = -1;
        if (q0 >= 0) out[lane] = j0;
        if (q1 >= 0) out[lane + 64] = j1;
        for (int c = lane + 128; c < cnt; c += 64) {
            int j = stencil_rows_atom(rows[wave], nrows, sample ? (int)rrow[c] : c);
            if (j == (int)a || (mi >= 0 && sa.smol[j] == mi)) j = -1;
            out[c] = j;
        }
    }
}

// Shell lists as masks: the drawn atoms of the current batch (the list members
// at the drawn ranks) into batch_j, for the adjoint when no forward at this
// step wrote them. One wavefront per apw consecutive atoms.
template <int ENC>
__global__ __launch_bounds__(kDecodeBlock) void k_list_decode(int64_t n, int apw, ShellMasks sm,
                                                              const int32_t* __restrict__ nshell, int p_shell,
                                                              int p_stride, const uint16_t* __restrict__ ranks,
                                                              int32_t* __restrict__ batch_j)
{
    __shared__ __align__(16) MaskTable<ENC> tab[kDecodeBlock / 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t a0 = ((int64_t)blockIdx.x * (kDecodeBlock / 64) + wave) * apw;
    const int64_t a1 = min(n, a0 + apw);
    MaskTable<ENC>& T = tab[wave];
    int cur = -1, nw = 0;
    for (int64_t a = a0; a < a1; ++a) {
        const int slot = sm.slot_of[a];
        if (slot != cur) {
            nw = sm.nw[slot];
            if constexpr (ENC == kMasksShort) mask_bases(T, sm, slot, nw, lane);
            cur = slot;
        }
        const int m = nshell[a];
        const bool sample = m > p_shell;
        const int cnt = sample ? p_shell : m;
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        mask_rows(T, sm, a, nw, mask_ahead<ENC>(sm, a, nw, lane), lane);
        for (int c = lane; c < cnt; c += 64)
            batch_j[a * (int64_t)p_stride + c] =
                mask_member(T, sm, a, slot, nw, sample ? (int)rrow[c] : c, (int)n - 1);
    }
}

constexpr int kCoopBlock = 256;

// A core pair (ex = false, accumulated into pc) or an excluded pair (ex = true,
// into px) with one code path: the excluded-pair correction -erf(br)/r equals
// the real-space term erfc(br)/r minus the bare 1/r, so its force factor is the
// Coulomb part of phi plus qq / r^3, without LJ. Forces only. (Fused form: both
// into pc.)
template <typename real, bool FUSED>
__device__ __forceinline__ void add_pair_or_excl(PairSum<real>& pc, PairSum<real>& px, uint4 si, real qi, uint4 sj,
                                                 real qj, const LJ<real>& lj, const PairParams<real>& pp, bool ex)
{
    real dx, dy, dz;
    const real qq = qi * qj;
    if constexpr (FUSED) {
        separation_q(si, sj, dx, dy, dz);
        const real r2 = (dx * dx + dy * dy + dz * dz) * pp.q2;
        const Radial<real> o = radial(r2, pp);
        const real r6 = o.rinv2 * o.rinv2 * o.rinv2;
        const real ljf = r2 < lj.rc2 ? r6 * (lj.a12 * r6 - lj.b6) : (real)0;
        const real phi = -o.rinv2 * (qq * o.g + (ex ? -qq * o.rinv : ljf));
        pc.fx += phi * dx;
        pc.fy += phi * dy;
        pc.fz += phi * dz;
    } else {
        using M = Math<real>;
        separation(si, sj, pp.quantum, dx, dy, dz);
        const real r2 = dx * dx + dy * dy + dz * dz;
        const real rinv = M::rsqrt_(r2);
        const real r = r2 * rinv;
        const real br = pp.beta * r;
        const real e = M::exp_(-br * br);
        const real ec = M::erfc_ex(br, e);
        const real rinv2 = rinv * rinv;
        const real r6 = rinv2 * rinv2 * rinv2;
        const real coul = -qq * rinv2 * (ec * rinv + pp.cgauss * e);
        const real ljf = r2 < lj.rc2 ? r6 * rinv2 * (lj.a12 * r6 - lj.b6) : (real)0;
        const real phi = ex ? coul + qq * rinv2 * rinv : coul - ljf;
        const real fx = phi * dx, fy = phi * dy, fz = phi * dz;
        pc.fx += ex ? (real)0 : fx;
        pc.fy += ex ? (real)0 : fy;
        pc.fz += ex ? (real)0 : fz;
        px.fx += ex ? fx : (real)0;
        px.fy += ex ? fy : (real)0;
        px.fz += ex ? fz : (real)0;
    }
}

// Excluded-pair correction f = psi r_ij of one pair, accumulated into px.
template <typename real, bool EV>
__device__ __forceinline__ void add_excl(PairSum<real>& px, uint4 si, real qi, uint4 sj, real qj,
                                         const PairParams<real>& pp)
{
    using M = Math<real>;
    real dx, dy, dz;
    separation(si, sj, pp.quantum, dx, dy, dz);
    const real r2 = dx * dx + dy * dy + dz * dz;
    const real qq = qi * qj;
    const real rinv = M::rsqrt_(r2);
    const real r = r2 * rinv;
    const real br = pp.beta * r;
    const real ex = M::exp_(-br * br);
    const real ef = M::erf_(br);
    const real rinv2 = rinv * rinv;
    const real psi = -qq * rinv2 * (pp.cgauss * ex - ef * rinv);
    px.fx += psi * dx;
    px.fy += psi * dy;
    px.fz += psi * dz;
    if (EV) {
        px.uc += -qq * ef * rinv;
        px.v[0] += psi * dx * dx; px.v[1] += psi * dy * dy; px.v[2] += psi * dz * dz;
        px.v[3] += psi * dx * dy; px.v[4] += psi * dx * dz; px.v[5] += psi * dy * dz;
    }
}

// Excluded partners of an atom up to which they share the passes of its full list; more
// come 64 for each of the wavefront's atoms in turn, which mostly share them, as their
// records are read from L2 for every atom otherwise. Forces, in the passes against in
// turn, molecules of 400: 96,000 atoms 312 and 278 us, 12,000 atoms 46 and 49; of
// 1,000: 584 and 470, 66 and 65; of 4,000: 2,068 and 1,622, 194 and 161.
constexpr int kExclFolded = 512;

template <typename real, bool FULL, bool EV, bool STENCIL, bool SKIN, int ENC>
__global__ __launch_bounds__(kCoopBlock, ENC && !EV && sizeof(real) == 4 ? 5 : 1) void k_pair_coop(
    int64_t n, int apw, PairParams<real> pp, const uint4* __restrict__ spos, const real* __restrict__ sqr,
    const uint4* __restrict__ spq, const int2* __restrict__ sxr, const int32_t* __restrict__ sxidx,
    const int32_t* __restrict__ core, const int32_t* __restrict__ ncore, int cap_core,
    const int32_t* __restrict__ shell, const int32_t* __restrict__ nshell, int cap_shell,
    const LJ<real>* __restrict__ lj_g, int n_types, int p_shell, int p_stride, const uint16_t* __restrict__ ranks,
    StencilArgs sa, uint64_t t_core, uint64_t t_shell, real* __restrict__ fsr, double* __restrict__ part,
    int32_t* __restrict__ bj_out, ShellMasks sm)
{
    __shared__ LJ<real> lj[256];
    __shared__ double red[kPairPartials * (kCoopBlock / 64)];
    __shared__ real excl_f[FULL && !EV ? kCoopBlock / 64 : 1][4][3];  // full lists: excluded pairs of large molecules
    __shared__ StencilRows<STENCIL ? kDecodeRows : 1> srows[kCoopBlock / 64];  // stencil rows of one cell per wave
    __shared__ __align__(16) unsigned char mtab[ENC ? (kCoopBlock / 64) * sizeof(MaskTable<ENC>) : 16];  // masks: one atom's row per wave
    constexpr bool kPass = FULL && !EV;
    constexpr bool kFused = fused_form(FULL, EV, SKIN);  // (ke and quantum come scaled)
    const int nt2 = n_types * n_types;
    for (int t = threadIdx.x; t < nt2; t += kCoopBlock) {
        LJ<real> e = lj_g[t];
        if (kFused) {
            e.a12 *= (real)kFusedScale;
            e.b6 *= (real)kFusedScale;
        }
        lj[t] = e;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    // the wavefront's index as a wave-uniform value, so that its atoms' indices and
    // row addresses are scalar
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t gw = blk * (kCoopBlock / 64) + wave;
    const int64_t a0 = gw * apw;
    const int64_t a1 = min(n, a0 + apw);
    // lanes 0, 16 and 32 keep the force sums' components (wave_sum4)
    const int f_comp = (lane & 15) == 0 && lane < 48 ? lane >> 4 : -1;
    double fc_sum = 0.0;
    PairSum<real> ev;  // per-lane energy/virial totals (forces unused)
    const Atoms<real> at{spos, sqr, spq};
    // per-atom headers of the wavefront's atoms, one atom per lane, read once
    const int64_t ah = min(a0 + min(lane, apw - 1), n - 1);
    uint4 h_s;
    real h_q;
    at.get(ah, h_s, h_q);
    const int h_nc = FULL ? 0 : ncore[ah];
    const int h_ns = nshell[ah];
    const int2 h_x = sxr[ah];
    const int h_mol = STENCIL ? sa.smol[ah] : 0;
    const int h_slot = ENC ? sm.slot_of[ah] : 0;
    const int h_nw = ENC ? sm.nw[h_slot] : 0;
    MaskTable<ENC>& T = reinterpret_cast<MaskTable<ENC>*>(mtab)[ENC ? wave : 0];
    // shell weight N_S / p~ (1 when every member is taken), one division per lane
    const real h_w = (!FULL && h_ns > p_shell) ? (real)((double)h_ns / (double)p_shell) : (real)1;
    const int nrows = sa.span * sa.span;
    int tcell = -1;  // the cell whose stencil rows sit in srows[wave]
    int tslot = -1;  // the block whose words' bases sit in T
    // first-level indices of one atom's first pass: the lane's first core entry,
    // its two batch ranks (or shell positions) and its first excluded partner
    // Without energies the excluded partners follow the core entries in one slot
    // (entries nc .. nc + nx - 1 of the combined list); with energies they keep
    // their own slot.
    constexpr bool kFold = !EV;
    auto first_level = [&](int64_t a, int t, int& jc, int& r0, int& r1, int& jx, MaskWords<ENC>& mk) {
        if (ENC) mk = mask_ahead<ENC>(sm, a, bcast(h_nw, t), lane);
        const int nc = bcast(h_nc, t);
        const int ns = bcast(h_ns, t);
        const int2 xr = make_int2(bcast(h_x.x, t), bcast(h_x.y, t));
        const bool sample = !FULL && ns > p_shell;
        const int cnt = sample ? p_shell : ns;
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        if (kFold)
            jc = lane < nc ? core[a * (int64_t)cap_core + lane]
                           : (lane < nc + xr.y ? sxidx[xr.x + lane - nc] : -1);
        else
            jc = lane < nc ? core[a * (int64_t)cap_core + lane] : -1;
        r0 = lane < cnt ? (sample ? (int)rrow[lane] : lane) : -1;
        r1 = lane + 64 < cnt ? (sample ? (int)rrow[lane + 64] : lane + 64) : -1;
        if (STENCIL) {
            // ranks of K(i) -> atoms, through the rows of the atom's build cell
            const int cell = sa.scell[a];
            if (cell != tcell) {
                stencil_rows_build(srows[wave], cell, sa, lane);
                tcell = cell;
            }
            if (r0 >= 0) r0 = stencil_rows_atom(srows[wave], nrows, r0);
            if (r1 >= 0) r1 = stencil_rows_atom(srows[wave], nrows, r1);
        }
        jx = (!kFold && lane < xr.y) ? sxidx[xr.x + lane] : -1;
    };
    // atom a's mask row (its lanes' words mk) into the wavefront's table
    auto mask_table = [&](int64_t a, int t, const MaskWords<ENC>& mk) {
        if constexpr (ENC == kMasksShort) {
            const int slot = bcast(h_slot, t);
            if (slot != tslot) {
                mask_bases(T, sm, slot, bcast(h_nw, t), lane);
                tslot = slot;
            }
        }
        if constexpr (ENC != kIndices) mask_rows(T, sm, a, bcast(h_nw, t), mk, lane);
    };
    // the shell member at position q of atom a's list as a mask in the table
    auto masked = [&](int64_t a, int t, int q) -> int {
        if constexpr (ENC != kIndices) return mask_member(T, sm, a, bcast(h_slot, t), bcast(h_nw, t), q, (int)n - 1);
        return -1;
    };
    // second level of an atom's first pass: the shell members at its two ranks (the
    // atoms themselves with stencil sampling)
    auto second_level = [&](int64_t a, int t, int r0, int r1, const MaskWords<ENC>& mk, int& e0, int& e1) {
        if (STENCIL) {
            e0 = r0;
            e1 = r1;
        } else if (ENC) {
            mask_table(a, t, mk);
            e0 = r0 >= 0 ? masked(a, t, r0) : -1;
            e1 = r1 >= 0 ? masked(a, t, r1) : -1;
        } else {
            const int32_t* s1 = shell + a * (int64_t)cap_shell;
            e0 = r0 >= 0 ? s1[r0] : -1;
            e1 = r1 >= 0 ? s1[r1] : -1;
        }
    };
    // a pipeline over the wavefront's atoms: while atom a's pairs are evaluated,
    // the shell entries of atom a + 1 and the first level of atom a + 2 are loaded
    // (issued after atom a's gathers, so that waiting for those does not wait for
    // them: the vector memory counter is in order)
    // Full list without energies: the list and the excluded partners (those of large
    // molecules before it, kExclFolded) as one sequence
    // of 64-entry passes, the indices of the pass after next and the atoms of the next
    // one in flight while a pass is evaluated. Bound by vector issue (13 passes of a
    // water atom's 728 entries at about 60 slots): 3,145,728 atoms 4.4 ms, 4.92 ms as
    // a loop of dependent loads with the excluded pairs in a pass of their own.
    if constexpr (kPass) {
        static_assert(kAtomsPerWaveList <= 4, "sums of excluded pairs per atom");
        auto folded = [&](int t) { const int nx = bcast(h_x.y, t); return nx <= kExclFolded ? nx : 0; };
        const bool large = __builtin_amdgcn_ballot_w64(h_x.y > kExclFolded) != 0;
        if (large) {
            PairSum<real> e[4];
            for (int c0 = 0, more = 1; more; c0 += 64) {
                more = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int nx = a0 + t < a1 ? bcast(h_x.y, t) : 0;
                    if (nx <= kExclFolded || c0 >= nx) continue;
                    more |= c0 + 64 < nx;
                    if (c0 + lane < nx) {
                        const uint4 si = make_uint4(bcast(h_s.x, t), bcast(h_s.y, t), bcast(h_s.z, t), bcast(h_s.w, t));
                        uint4 sj;
                        real q;
                        at.get(sxidx[bcast(h_x.x, t) + c0 + lane], sj, q);
                        add_pair_or_excl<real, kFused>(e[t], e[t], si, bcast(h_q, t) * pp.ke, sj, q, lj[0], pp, true);
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const real f = wave_sum4(e[t].fx, e[t].fy, e[t].fz, e[t].fz);
                if (f_comp >= 0) excl_f[wave][t][f_comp] = f;
            }
        }
        auto entry = [&](int64_t a, int t, int pass) -> int {
            const int ns = bcast(h_ns, t), nx = folded(t);
            const int e = pass * 64 + lane;
            const int32_t* const srow = shell + a * (int64_t)cap_shell;
            if (pass * 64 + 64 <= ns) return srow[e];  // (uniform: a pass of list entries only)
            return e < ns ? srow[e] : (e < ns + nx ? sxidx[bcast(h_x.x, t) + e - ns] : -1);
        };
        int n_j0 = -1, n_j1 = -1;  // the next atom's first two passes
        if (a0 < a1) {
            n_j0 = entry(a0, 0, 0);
            n_j1 = entry(a0, 0, 1);
        }
        for (int64_t a = a0; a < a1; ++a) {
            const int t = (int)(a - a0);
            const uint4 si = make_uint4(bcast(h_s.x, t), bcast(h_s.y, t), bcast(h_s.z, t), bcast(h_s.w, t));
            const real qi = bcast(h_q, t) * pp.ke;
            const LJ<real>* const lrow = lj + (int)si.w * n_types;
            const int ns = bcast(h_ns, t);
            const int passes = (ns + folded(t) + 63) >> 6;
            int j = n_j0, jn = n_j1;
            uint4 pj;
            real qj;
            at.get(max(j, 0), pj, qj);
            if (a + 1 < a1) {
                n_j0 = entry(a + 1, t + 1, 0);
                n_j1 = entry(a + 1, t + 1, 1);
            }
            PairSum<real> pc, px;  // (px unused)
            for (int p = 0; p < passes; ++p) {
                const uint4 sj = pj;
                const real q = qj;
                const bool in = j >= 0;
                j = jn;
                at.get(max(j, 0), pj, qj);
                jn = p + 2 < passes ? entry(a, t, p + 2) : -1;
                const bool ex = p * 64 + lane >= ns;
                if (in && (ex || !SKIN || dist2_q(si, sj) <= t_shell))
                    add_pair_or_excl<real, kFused>(pc, px, si, qi, sj, q, lrow[sj.w], pp, ex);
            }
            real f = wave_sum4(pc.fx, pc.fy, pc.fz, pc.fz);
            if (large && f_comp >= 0) f += excl_f[wave][t][f_comp];
            f *= pp.quantum;
            if (f_comp >= 0) {
                fsr[3 * a + f_comp] = f;
                fc_sum += (double)f;
            }
        }
    }
    int n_jc = -1, n_e0 = -1, n_e1 = -1, n_jx = -1;  // atom a: first level and shell entries
    int m_jc = -1, m_r0 = -1, m_r1 = -1, m_jx = -1;  // atom a + 1: first level
    MaskWords<ENC> m_mk{};                           // ... and its mask words
    if (!kPass && a0 < a1) {
        int r0, r1;
        first_level(a0, 0, n_jc, r0, r1, n_jx, m_mk);
        second_level(a0, 0, r0, r1, m_mk, n_e0, n_e1);
        if (a0 + 1 < a1) first_level(a0 + 1, 1, m_jc, m_r0, m_r1, m_jx, m_mk);
    }
    for (int64_t a = a0; !kPass && a < a1; ++a) {
        const int t = (int)(a - a0);
        const int jc = n_jc, e0 = n_e0, e1 = n_e1, jx = n_jx;
        const uint4 si = make_uint4(bcast(h_s.x, t), bcast(h_s.y, t), bcast(h_s.z, t),
                                    bcast(h_s.w, t));
        const real qi = bcast(h_q, t) * pp.ke;
        // LJ coefficients of the pair types
        const int li = (int)si.w * n_types;
        auto ljof = [&](uint4 sj) -> LJ<real> { return lj[li + (int)sj.w]; };
        const int nc = bcast(h_nc, t);
        const int ns = bcast(h_ns, t);
        const int2 xr = make_int2(bcast(h_x.x, t), bcast(h_x.y, t));
        const int32_t* crow = core + a * (int64_t)cap_core;
        const int32_t* srow = shell + a * (int64_t)cap_shell;
        // shell member at position q of the atom's list (masks: the atom's row in T)
        auto member = [&](int q) -> int { return ENC ? masked(a, t, q) : srow[q]; };
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        const bool sample = !FULL && ns > p_shell;
        const int cnt = sample ? p_shell : ns;
        const real w = bcast(h_w, t);
        PairSum<real> pc, ps, px;
        const int js0 = e0, js1 = e1;
        const int mi = STENCIL ? bcast(h_mol, t) : 0;
        const int mj0 = STENCIL ? sa.smol[max(js0, 0)] : 0;
        const int mj1 = STENCIL ? sa.smol[max(js1, 0)] : 0;
        if (!FULL && bj_out) {
            // the batch atoms, for the backward expected at this step (with stencil
            // sampling -1 for i itself and i's molecule, as k_stencil_decode writes)
            auto bj = [&](int j, int mj) { return STENCIL && (j == (int)a || (mi >= 0 && mj == mi)) ? -1 : j; };
            int32_t* o = bj_out + a * (int64_t)p_stride;
            if (lane < cnt) o[lane] = bj(js0, mj0);
            if (lane + 64 < cnt) o[lane + 64] = bj(js1, mj1);
        }
        // (unused slots load atom 0, so that every position is one 16-byte load)
        uint4 pjc, pj0, pj1, pjx;
        real qjc, qj0, qj1, qjx;
        at.get(max(jc, 0), pjc, qjc);
        at.get(max(js0, 0), pj0, qj0);
        at.get(max(js1, 0), pj1, qj1);
        if (kFold) {
            pjx = pjc;
            qjx = qjc;
        } else {
            at.get(max(jx, 0), pjx, qjx);
        }
        if (a + 1 < a1) {
            n_jc = m_jc;
            n_jx = m_jx;
            second_level(a + 1, t + 1, m_r0, m_r1, m_mk, n_e0, n_e1);
            if (a + 2 < a1) first_level(a + 2, t + 2, m_jc, m_r0, m_r1, m_jx, m_mk);
        }
        // skin: a core entry counts inside r_core, a list shell entry inside the annulus
        // (the whole ball in full-list mode), at these positions
        auto core_ok = [&](uint4 sj) { return !SKIN || dist2_q(si, sj) <= t_core; };
        auto shell_ok = [&](uint4 sj) {
            if (!SKIN) return true;
            const uint64_t d2 = dist2_q(si, sj);
            return d2 <= t_shell && (FULL || d2 > t_core);
        };
        if (kFold) {
            if (jc >= 0 && (lane >= nc || core_ok(pjc))) add_pair_or_excl<real, kFused>(pc, px, si, qi, pjc, qjc, ljof(pjc), pp, lane >= nc);
        } else {
            if (jc >= 0 && core_ok(pjc)) add_pair<real, EV, kFused>(pc, si, qi, pjc, qjc, ljof(pjc), pp);
            if (jx >= 0) add_excl<real, EV>(px, si, qi, pjx, qjx, pp);
        }
        if (STENCIL ? stencil_member(a, js0, mi, mj0, si, pj0, t_core, t_shell) : (js0 >= 0 && shell_ok(pj0)))
            add_pair<real, EV, kFused>(ps, si, qi, pj0, qj0, ljof(pj0), pp);
        if (STENCIL ? stencil_member(a, js1, mi, mj1, si, pj1, t_core, t_shell) : (js1 >= 0 && shell_ok(pj1)))
            add_pair<real, EV, kFused>(ps, si, qi, pj1, qj1, ljof(pj1), pp);
        // the rest (long lists and large batches)
        if (kFold) {
            for (int c = lane + 64; c < nc + xr.y; c += 64) {
                const int j = c < nc ? crow[c] : sxidx[xr.x + c - nc];
                uint4 sj;
                real qj;
                at.get(j, sj, qj);
                if (c >= nc || core_ok(sj)) add_pair_or_excl<real, kFused>(pc, px, si, qi, sj, qj, ljof(sj), pp, c >= nc);
            }
        } else {
            for (int c = lane + 64; c < nc; c += 64) {
                const int j = crow[c];
                uint4 sj;
                real qj;
                at.get(j, sj, qj);
                if (core_ok(sj)) add_pair<real, EV, kFused>(pc, si, qi, sj, qj, ljof(sj), pp);
            }
            for (int c = lane + 64; c < xr.y; c += 64) {
                uint4 sj;
                real qj;
                at.get(sxidx[xr.x + c], sj, qj);
                add_excl<real, EV>(px, si, qi, sj, qj, pp);
            }
        }
        if (STENCIL && cnt > 128) {
            // the next atom's first pass may have put another cell's rows in place
            const int cell = sa.scell[a];
            if (cell != tcell) {
                stencil_rows_build(srows[wave], cell, sa, lane);
                tcell = cell;
            }
        }
        // (the table holds the next atom's row by now)
        if (ENC && cnt > 128) mask_table(a, t, mask_ahead<ENC>(sm, a, bcast(h_nw, t), lane));
        for (int c = lane + 128; c < cnt; c += 64) {
            if (STENCIL) {
                const int j = stencil_rows_atom(srows[wave], nrows, sample ? (int)rrow[c] : c);
                const int mj = sa.smol[j];
                if (bj_out) bj_out[a * (int64_t)p_stride + c] = (j == (int)a || (mi >= 0 && mj == mi)) ? -1 : j;
                uint4 sj;
                real qj;
                at.get(j, sj, qj);
                if (stencil_member(a, j, mi, mj, si, sj, t_core, t_shell))
                    add_pair<real, EV, kFused>(ps, si, qi, sj, qj, ljof(sj), pp);
            } else {
                const int j = member(sample ? (int)rrow[c] : c);
                if (!FULL && bj_out) bj_out[a * (int64_t)p_stride + c] = j;
                uint4 sj;
                real qj;
                at.get(j, sj, qj);
                if (shell_ok(sj)) add_pair<real, EV, kFused>(ps, si, qi, sj, qj, ljof(sj), pp);
            }
        }
        // one set of sums: the excluded-pair forces cancel pairwise, so the momentum
        // correction may sum them with the rest
        const real fu = kFused ? pp.quantum : (real)1;
        const real tz = pc.fz + w * ps.fz + px.fz;
        const real f = fu * wave_sum4(pc.fx + w * ps.fx + px.fx, pc.fy + w * ps.fy + px.fy, tz, tz);
        if (f_comp >= 0) {
            fsr[3 * a + f_comp] = f;
            fc_sum += (double)f;
        }
        if (EV) {
            ev.uc += pc.uc + w * ps.uc;
            ev.ul += pc.ul + w * ps.ul;
            ev.fx += px.uc;  // excluded-pair energy
#pragma unroll
            for (int c = 0; c < 6; ++c) ev.v[c] += pc.v[c] + w * ps.v[c] + px.v[c];
        }
    }
    // per-block sums: the force sums sit in one lane per component and wavefront; with
    // energies nine more values, summed over the lanes
    constexpr int NW = kCoopBlock / 64;
    if (f_comp >= 0) red[f_comp * NW + wave] = fc_sum;
    if (EV) {
        double vals[9];
        vals[0] = 0.5 * (double)ev.uc;
        vals[1] = 0.5 * (double)ev.ul;
        vals[2] = 0.5 * (double)ev.fx;
        for (int c = 0; c < 6; ++c) vals[3 + c] = -0.5 * (double)ev.v[c];
#pragma unroll
        for (int c = 0; c < 9; ++c) {
            const double t = wave_sum(vals[c]);
            if (lane == 0) red[(3 + c) * NW + wave] = t;
        }
    }
    __syncthreads();
    if (threadIdx.x < (EV ? 12 : 3)) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += red[threadIdx.x * NW + w];
        part[blk * (int64_t)kPairPartials + threadIdx.x] = t;
    }
}

// Entries of a lane's first pass in k_pair_thread (a multiple of 4).
constexpr int kThreadFirst = 12;

// Sparse lists (every atom's core list and batch within a few dozen entries, as
// in the dilute electrolytes): two lanes per atom, the even one walking its core
// list and excluded partners, the odd one its batch, so that no wavefront idles on
// an atom with a handful of pairs. Same sums and partials as k_pair_coop (split
// lists; the two lanes' sums are the ones that kernel adds at the end). The loads
// bound it: ten or so dependent gathers per atom over three levels (ranks, shell
// entries, positions), one cache line and address each; the lane pair keeps half
// the registers of one thread per atom and so twice the gathers in flight, and
// indices come four to a load. 10^6 ions, 10 of 136 drawn: 239 -> 217 us
// (218 -> 193 us on kept lists); 14 L2 requests of 700 cycles per atom are what is left.
template <typename real, bool EV>
__global__ __launch_bounds__(kCoopBlock) void k_pair_thread(
    int64_t n, PairParams<real> pp, const uint4* __restrict__ spos, const real* __restrict__ sqr,
    const uint4* __restrict__ spq, const int2* __restrict__ sxr, const int32_t* __restrict__ sxidx,
    const int32_t* __restrict__ core, const int32_t* __restrict__ ncore, int cap_core,
    const int32_t* __restrict__ shell, const int32_t* __restrict__ nshell, int cap_shell,
    const LJ<real>* __restrict__ lj_g, int n_types, int p_shell, int p_stride, const uint16_t* __restrict__ ranks,
    uint64_t t_core, uint64_t t_shell, bool skin, real* __restrict__ fsr, double* __restrict__ part,
    int32_t* __restrict__ bj_out)
{
    __shared__ LJ<real> lj[256];
    __shared__ double red[kPairPartials * (kCoopBlock / 64)];
    const int nt2 = n_types * n_types;
    for (int t = threadIdx.x; t < nt2; t += kCoopBlock) lj[t] = lj_g[t];
    __syncthreads();
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t a = blk * (kCoopBlock / 2) + (threadIdx.x >> 1);
    const bool batch = threadIdx.x & 1;
    constexpr int NV = EV ? 12 : 3;
    double vals[NV];
    for (int c = 0; c < NV; ++c) vals[c] = 0.0;
    const Atoms<real> at{spos, sqr, spq};
    if (a < n) {
        uint4 si;
        real qi;
        at.get(a, si, qi);
        qi *= pp.ke;
        // LJ coefficients of the pair types
        const int li = (int)si.w * n_types;
        auto ljof = [&](uint4 sj) -> LJ<real> { return lj[li + (int)sj.w]; };
        const int ns = nshell[a];
        const bool sample = ns > p_shell;
        const int cnt = batch ? min(ns, p_shell) : ncore[a];
        const int32_t* crow = core + a * (int64_t)cap_core;
        const int32_t* srow = shell + a * (int64_t)cap_shell;
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        // entries c0 .. c0 + 3 of this lane's list (-1 past its end; the rows and their
        // capacities are multiples of four entries)
        auto ranks4 = [&](int c0) -> int4 {
            if (!sample) return make_int4(c0, c0 + 1, c0 + 2, c0 + 3);
            const uint2 r = *(const uint2*)(rrow + c0);
            return make_int4((int)(r.x & 0xffffu), (int)(r.x >> 16), (int)(r.y & 0xffffu), (int)(r.y >> 16));
        };
        auto first4 = [&](int c0) -> int4 {
            if (c0 >= cnt) return make_int4(-1, -1, -1, -1);
            return batch ? ranks4(c0) : *(const int4*)(crow + c0);
        };
        auto entries4 = [&](int c0, int4 r, int* j) {
            j[0] = c0 < cnt ? (batch ? srow[r.x] : r.x) : -1;
            j[1] = c0 + 1 < cnt ? (batch ? srow[r.y] : r.y) : -1;
            j[2] = c0 + 2 < cnt ? (batch ? srow[r.z] : r.z) : -1;
            j[3] = c0 + 3 < cnt ? (batch ? srow[r.w] : r.w) : -1;
        };
        // the batch atoms, for the backward expected at this step
        auto keep4 = [&](int c0, const int* j) {
            if (bj_out && batch && c0 < cnt)
                *(int4*)(bj_out + a * (int64_t)p_stride + c0) = make_int4(j[0], j[1], j[2], j[3]);
        };
        PairSum<real> p, px;
        auto pair = [&](int j, uint4 sj, real qj) {
            if (j < 0) return;
            if (skin) {
                const uint64_t d2 = dist2_q(si, sj);
                if (batch ? d2 <= t_core || d2 > t_shell : d2 > t_core) return;
            }
            add_pair<real, EV, false>(p, si, qi, sj, qj, ljof(sj), pp);
        };
        // the first pass, each level's loads issued together
        int4 r[kThreadFirst / 4];
        int j[kThreadFirst];
#pragma unroll
        for (int u = 0; u < kThreadFirst; u += 4) r[u / 4] = first4(u);
#pragma unroll
        for (int u = 0; u < kThreadFirst; u += 4) entries4(u, r[u / 4], j + u);
        uint4 sj[kThreadFirst];
        real qj[kThreadFirst];
#pragma unroll
        for (int u = 0; u < kThreadFirst; ++u) at.get(max(j[u], 0), sj[u], qj[u]);
#pragma unroll
        for (int u = 0; u < kThreadFirst; u += 4) keep4(u, j + u);
#pragma unroll
        for (int u = 0; u < kThreadFirst; ++u) pair(j[u], sj[u], qj[u]);
        // the rest four entries at a time
        for (int c0 = kThreadFirst; c0 < cnt; c0 += 4) {
            int jt[4];
            uint4 st[4];
            real qt[4];
            entries4(c0, first4(c0), jt);
#pragma unroll
            for (int u = 0; u < 4; ++u) at.get(max(jt[u], 0), st[u], qt[u]);
            keep4(c0, jt);
#pragma unroll
            for (int u = 0; u < 4; ++u) pair(jt[u], st[u], qt[u]);
        }
        if (!batch) {
            const int2 xr = sxr[a];
            for (int c = 0; c < xr.y; ++c) {
                uint4 sx;
                real qx;
                at.get(sxidx[xr.x + c], sx, qx);
                add_excl<real, EV>(px, si, qi, sx, qx, pp);
            }
        }
        // the batch lane's sums to the even lane
        PairSum<real> ps;
        ps.fx = __shfl_xor(p.fx, 1, 64);
        ps.fy = __shfl_xor(p.fy, 1, 64);
        ps.fz = __shfl_xor(p.fz, 1, 64);
        if (EV) {
            ps.uc = __shfl_xor(p.uc, 1, 64);
            ps.ul = __shfl_xor(p.ul, 1, 64);
            for (int c = 0; c < 6; ++c) ps.v[c] = __shfl_xor(p.v[c], 1, 64);
        }
        if (!batch) {
            const real w = sample ? (real)((double)ns / (double)p_shell) : (real)1;
            const real fx = p.fx + w * ps.fx + px.fx;
            const real fy = p.fy + w * ps.fy + px.fy;
            const real fz = p.fz + w * ps.fz + px.fz;
            fsr[3 * a + 0] = fx;
            fsr[3 * a + 1] = fy;
            fsr[3 * a + 2] = fz;
            vals[0] = (double)fx;
            vals[1] = (double)fy;
            vals[2] = (double)fz;
            if (EV) {
                vals[3] = 0.5 * (double)(p.uc + w * ps.uc);
                vals[4] = 0.5 * (double)(p.ul + w * ps.ul);
                vals[5] = 0.5 * (double)px.uc;
                for (int c = 0; c < 6; ++c) vals[6 + c] = -0.5 * (double)(p.v[c] + w * ps.v[c] + px.v[c]);
            }
        }
    }
    double out;
    block_sum_vec<NV, kCoopBlock>(vals, red, threadIdx.x, out);
    if (threadIdx.x < NV) part[blk * (int64_t)kPairPartials + threadIdx.x] = out;
}

static StencilArgs stencil_args(const irbe_ctx* h)
{
    StencilArgs sa;
    sa.cell_start = h->cell_start;
    sa.scell = h->scell;
    sa.smol = h->smol;
    sa.n_c = h->geo.n_c;
    sa.lo = h->geo.lo;
    sa.span = h->geo.hi - h->geo.lo + 1;
    return sa;
}

// Stencil sampling: the drawn atoms of the current batch into h->batch_j (for
// read-back; the pair kernels decode the ranks themselves).
hipError_t launch_stencil_decode(irbe_ctx* h)
{
    if (!h->stencil) return hipErrorInvalidValue;
    const StencilArgs sa = stencil_args(h);
    if (sa.span * sa.span > kDecodeRows) return hipErrorInvalidValue;
    const int64_t n = h->cfg.n_atoms;
    const hipError_t e = ensure_batch_atoms(h);
    if (e != hipSuccess) return e;
    const int apw = 16;
    const int64_t waves = blocks_for(n, apw);
    k_stencil_decode<<<(unsigned)blocks_for(waves, kDecodeBlock / 64), kDecodeBlock, 0, h->stream>>>(
        n, apw, sa, h->nshell, h->cfg.p_shell, h->p_stride, h->ranks, h->batch_j);
    return hipGetLastError();
}

// Shell lists as masks: the drawn atoms of the current ranks into h->batch_j.
static hipError_t launch_list_decode(irbe_ctx* h)
{
    if (!h->masks) return hipErrorInvalidValue;
    const int64_t n = h->cfg.n_atoms;
    const hipError_t e = ensure_batch_atoms(h);
    if (e != hipSuccess) return e;
    const int apw = 16;
    const int64_t waves = blocks_for(n, apw);
    auto run = [&](auto enc) {
        k_list_decode<decltype(enc)::value><<<(unsigned)blocks_for(waves, kDecodeBlock / 64), kDecodeBlock, 0, h->stream>>>(
            n, apw, h->shell_masks(), h->nshell, h->cfg.p_shell, h->p_stride, h->ranks, h->batch_j);
    };
    if (h->cap_words > kMaskTableWords) run(std::integral_constant<int, kMasksLong>{});
    else run(std::integral_constant<int, kMasksShort>{});
    return hipGetLastError();
}

// Threads per block of the batch draw and the LDS its bitmaps take (one bitmap
// of the longest list per thread); more than 64 KiB means device memory.
static int draw_block(const irbe_ctx* h, size_t* lds)
{
    const int words = (h->shell_bound() + 31) / 32;
    int block = 256;
    while (block > 64 && (size_t)words * block * 4 > 32 * 1024) block /= 2;
    if (block == 64 && (size_t)words * block * 4 > 64 * 1024) block = 32;
    *lds = (size_t)words * block * 4;
    return block;
}

bool draw_bitmaps_in_lds(const irbe_ctx* h)
{
    size_t lds = 0;
    draw_block(h, &lds);
    return lds <= 64 * 1024;
}

// Batch ranks of every atom for `step` (kept until the lists or the step change).
static hipError_t launch_draw(irbe_ctx* h, uint64_t step)
{
    if (h->full_list || (h->ranks_valid && h->ranks_step == step)) return hipSuccess;
    const int64_t n = h->cfg.n_atoms;
    const int words = (h->shell_bound() + 31) / 32;
    size_t lds = 0;
    const int block = draw_block(h, &lds);
    const unsigned nb = (unsigned)blocks_for(n, block);
    const size_t half_lds = (size_t)(kHalfDrawBlock / 32) * h->shell_bound() * 4;
    if (half_draw(n, h->cfg.p_shell) && half_lds <= 64 * 1024) {
        k_draw_batches_half<<<(unsigned)blocks_for(n, kHalfDrawBlock / 32), kHalfDrawBlock, half_lds, h->stream>>>(
            n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride, h->cfg.seed, step, h->shell_bound(), h->ranks);
    } else if (lds > 64 * 1024) {
        // bitmaps in device memory: as many threads as fit 1 GiB of bitmaps
        const int64_t threads = std::max<int64_t>(256, std::min<int64_t>(n, ((int64_t)1 << 28) / words) / 256 * 256);
        hipError_t e = ensure_draw_bits(h, (size_t)threads * (size_t)words);
        if (e != hipSuccess) return e;
        k_draw_batches_global<<<(unsigned)(threads / 256), 256, 0, h->stream>>>(
            n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride, h->cfg.seed, step, h->draw_bits, (int)threads,
            h->ranks);
    } else if (block == 256)
        k_draw_batches<256><<<nb, 256, lds, h->stream>>>(n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride,
                                                         h->cfg.seed, step, h->ranks);
    else if (block == 128)
        k_draw_batches<128><<<nb, 128, lds, h->stream>>>(n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride,
                                                         h->cfg.seed, step, h->ranks);
    else if (block == 64)
        k_draw_batches<64><<<nb, 64, lds, h->stream>>>(n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride,
                                                       h->cfg.seed, step, h->ranks);
    else
        k_draw_batches<32><<<nb, 32, lds, h->stream>>>(n, h->perm, h->nshell, h->cfg.p_shell, h->p_stride,
                                                       h->cfg.seed, step, h->ranks);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        h->ranks_valid = true;
        h->ranks_step = step;
        h->batch_j_valid = h->batch_j_fwd = false;
    }
    return e;
}

// Atoms per wavefront of a small system's forces: halved (down to 2, which the per-block
// sums are sized for) while fewer than kWavesWanted wavefronts, four per SIMD, would run.
// 2,703 atoms: 29 -> 10 us with 2 instead of 8; 1,536 atoms, full lists and energies in
// FP64: 40 -> 23 us; 12,288 atoms: 26 -> 17 us.
constexpr int64_t kWavesWanted = 4096;

static int spread_atoms(int64_t n, int apw)
{
    while (apw > 2 && blocks_for(n, apw) < kWavesWanted) apw = std::max(2, apw / 2);
    return apw;
}

template <typename real, bool FULL, bool EV, bool STENCIL, bool SKIN, int ENC = kIndices>
static hipError_t launch_coop_t(irbe_ctx* h, uint64_t step)
{
    const int64_t n = h->cfg.n_atoms;
    PairParams<real> pp = pair_params<real>(h);
    if (fused_form(FULL, EV, SKIN)) {
        pp.ke *= (real)kFusedScale;
        pp.quantum *= (real)(1.0 / kFusedScale);
    }
    hipError_t e = launch_draw(h, step);
    if (e != hipSuccess) return e;
    // stencil sampling keeps one cell's stencil rows for consecutive atoms: longer
    // runs of atoms per wavefront pay there, shorter ones with list-drawn batches
    // (the FP32 energies add up over a wavefront's atoms in FP32: their runs stay as they are)
    int apw = STENCIL ? kAtomsPerWaveStencil : (FULL ? kAtomsPerWaveList : kAtomsPerWaveSplit);
    if (!EV || sizeof(real) == 8) apw = spread_atoms(n, apw);
    const int64_t waves = blocks_for(n, apw);
    const unsigned nb = (unsigned)blocks_for(waves, kCoopBlock / 64);
    if ((int64_t)nb > h->part_blocks) return hipErrorInvalidValue;
    // the batch atoms for the backward, when one followed the last forward (into a
    // buffer that backward allocated: a forward allocates nothing here)
    int32_t* bj_out = (!FULL && h->keep_batch) ? h->batch_j : nullptr;
    k_pair_coop<real, FULL, EV, STENCIL, SKIN, ENC><<<nb, kCoopBlock, 0, h->stream>>>(
        n, apw, pp, h->spos, (const real*)h->sq_r, h->spq, h->sxr, h->sxidx, h->core, h->ncore, h->cap_core,
        h->shell, h->nshell, h->cap_shell, (const LJ<real>*)h->lj, h->cfg.n_types, h->cfg.p_shell, h->p_stride,
        h->ranks, stencil_args(h), h->geo.t_core, h->geo.t_shell, (real*)h->fsr, h->pair_part, bj_out, h->shell_masks());
    h->pair_nb = nb;
    if (bj_out) h->batch_j_valid = h->batch_j_fwd = true;
    return hipGetLastError();
}

template <typename real, bool EV>
static hipError_t launch_thread_t(irbe_ctx* h, uint64_t step)
{
    const int64_t n = h->cfg.n_atoms;
    const PairParams<real> pp = pair_params<real>(h);
    hipError_t e = launch_draw(h, step);
    if (e != hipSuccess) return e;
    const unsigned nb = (unsigned)blocks_for(n, kCoopBlock / 2);
    if ((int64_t)nb > h->part_blocks) return hipErrorInvalidValue;
    // the batch atoms for the backward, as in launch_coop_t
    int32_t* bj_out = h->keep_batch ? h->batch_j : nullptr;
    k_pair_thread<real, EV><<<nb, kCoopBlock, 0, h->stream>>>(
        n, pp, h->spos, (const real*)h->sq_r, h->spq, h->sxr, h->sxidx, h->core, h->ncore, h->cap_core, h->shell, h->nshell,
        h->cap_shell, (const LJ<real>*)h->lj, h->cfg.n_types, h->cfg.p_shell, h->p_stride, h->ranks, h->geo.t_core,
        h->geo.t_shell, h->geo.skin, (real*)h->fsr, h->pair_part, bj_out);
    h->pair_nb = nb;
    if (bj_out) h->batch_j_valid = h->batch_j_fwd = true;
    return hipGetLastError();
}

// The cooperative kernel for the list mode, energies and skin.
template <typename real, bool SKIN>
static hipError_t launch_coop_s(irbe_ctx* h, uint64_t step, bool ev)
{
    if (h->full_list)
        return ev ? launch_coop_t<real, true, true, false, SKIN>(h, step)
                  : launch_coop_t<real, true, false, false, SKIN>(h, step);
    if (h->stencil)
        return ev ? launch_coop_t<real, false, true, true, SKIN>(h, step)
                  : launch_coop_t<real, false, false, true, SKIN>(h, step);
    if (h->masks && h->cap_words > kMaskTableWords)
        return ev ? launch_coop_t<real, false, true, false, SKIN, kMasksLong>(h, step)
                  : launch_coop_t<real, false, false, false, SKIN, kMasksLong>(h, step);
    if (h->masks)
        return ev ? launch_coop_t<real, false, true, false, SKIN, kMasksShort>(h, step)
                  : launch_coop_t<real, false, false, false, SKIN, kMasksShort>(h, step);
    return ev ? launch_coop_t<real, false, true, false, SKIN>(h, step)
              : launch_coop_t<real, false, false, false, SKIN>(h, step);
}

// Split lists whose longest core list plus batch stays within this many entries
// take the thread-per-atom kernel (32-bit shell entries only: the cooperative
// kernel reads the masks).
constexpr int kSparsePairs = 32;

template <typename real>
static hipError_t launch_coop_r(irbe_ctx* h, uint64_t step, bool ev)
{
    if (!h->full_list && !h->stencil && !h->masks &&
        h->max_core + std::min(h->max_shell, h->cfg.p_shell) <= kSparsePairs)
        return ev ? launch_thread_t<real, true>(h, step) : launch_thread_t<real, false>(h, step);
    return h->geo.skin ? launch_coop_s<real, true>(h, step, ev) : launch_coop_s<real, false>(h, step, ev);
}

// Reduce the per-block partials in a fixed order, in two stages: stage 1 sums
// contiguous ranges of blocks into kReduceSlices slices, stage 2 sums the
// slices: ev_pair[0..11] = totals, fcorr = (sum of the uncorrected short-range
// force) / N when rbl.
constexpr int kReduceSlices = 256;
// blocks up to which the second stage sums the partials itself: four per thread,
// one launch of about 5 us in place of two
constexpr int64_t kReduceDirect = 4 * kReduceBlock;

template <int NV>
__global__ __launch_bounds__(kReduceBlock) void k_pair_reduce1(int64_t nb, const double* __restrict__ part,
                                                               double* __restrict__ slices)
{
    __shared__ double lds[NV * (kReduceBlock / 64)];
    const int64_t per = (nb + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = blockIdx.x * per, b1 = min(nb, b0 + per);
    double vals[NV];
    for (int c = 0; c < NV; ++c) vals[c] = 0.0;
    for (int64_t b = b0 + threadIdx.x; b < b1; b += kReduceBlock)
        for (int c = 0; c < NV; ++c) vals[c] += part[b * kPairPartials + c];
    double out;
    block_sum_vec<NV, kReduceBlock>(vals, lds, threadIdx.x, out);
    if (threadIdx.x < NV) slices[blockIdx.x * 12 + threadIdx.x] = out;
}

template <int NV>
__global__ __launch_bounds__(kReduceBlock) void k_pair_reduce2(int n_slices, int stride,
                                                               const double* __restrict__ slices, int64_t n, int rbl,
                                                               double* __restrict__ ev_pair,
                                                               double* __restrict__ fcorr)
{
    __shared__ double lds[NV * (kReduceBlock / 64)];
    double vals[NV];
    for (int c = 0; c < NV; ++c) vals[c] = 0.0;
    for (int b = threadIdx.x; b < n_slices; b += kReduceBlock)
        for (int c = 0; c < NV; ++c) vals[c] += slices[b * stride + c];
    double out;
    block_sum_vec<NV, kReduceBlock>(vals, lds, threadIdx.x, out);
    if (threadIdx.x < NV) ev_pair[threadIdx.x] = out;
    if (threadIdx.x < 3) fcorr[threadIdx.x] = rbl ? out / (double)n : 0.0;
}

hipError_t launch_pair_reduce(irbe_ctx* h, bool ev)
{
    // (without energies the blocks write the three force sums only; few blocks are summed
    // in one launch, as slices of one block each)
    auto run = [&](auto nv) {
        constexpr int NV = decltype(nv)::value;
        if (h->pair_nb <= kReduceDirect) {
            k_pair_reduce2<NV><<<1, kReduceBlock, 0, h->stream>>>((int)h->pair_nb, kPairPartials, h->pair_part,
                                                                  h->cfg.n_atoms, h->full_list ? 0 : 1, h->ev_pair,
                                                                  h->fcorr);
            return;
        }
        k_pair_reduce1<NV><<<kReduceSlices, kReduceBlock, 0, h->stream>>>(h->pair_nb, h->pair_part, h->pair_slices);
        k_pair_reduce2<NV><<<1, kReduceBlock, 0, h->stream>>>(kReduceSlices, 12, h->pair_slices, h->cfg.n_atoms,
                                                              h->full_list ? 0 : 1, h->ev_pair, h->fcorr);
    };
    if (ev) run(std::integral_constant<int, 12>{});
    else run(std::integral_constant<int, 3>{});
    return hipGetLastError();
}

hipError_t launch_pair_forces(irbe_ctx* h, uint64_t step, bool ev)
{
    const hipError_t e = h->fp64 ? launch_coop_r<double>(h, step, ev) : launch_coop_r<float>(h, step, ev);
    // each forward renews the prediction: a backward after it sets keep_batch again
    h->keep_batch = false;
    h->fwd_pending = true;
    return e;
}

// ---------------------------------------------------------------------------
// Adjoint of the short-range force (vector-Jacobian product with G = dL/dF at
// fixed lists and batches). With f_ij = phi(r) r_ij, J = phi I + (phi'/r) r r^T
// is symmetric and even in r_ij, so for the symmetric sets (C(i), the full list,
// the excluded pairs) the gradient is gathered per atom:
//   dL/dr_i += sum_j J (G'_j - G'_i),  dL/dq_i += sum_j (ke q_j a(r)) r_ij.(G'_j - G'_i)
// where a(r) is the Coulomb factor of phi / (-ke q_i q_j). The sampled shell
// terms are one-sided: dL/dr_i -= w J G'_i and dL/dr_j += w J G'_i, and likewise
// for the charges. G' = G - mean(G) for the pair terms when the momentum
// correction is applied; excluded pairs use G. LJ table gradients are
// accumulated per (t_i, t_j) entry in FP64.
//
// The scatter onto j is a transpose. Device-scope atomics on this chip are
// executed at the memory side, one transaction per lane, so instead each block
// (a run of consecutive cell-ordered atoms, which lie in one or two cell rows)
// stages its records (j, w J G'_i, charge term) in LDS, counts them per
// (source row, destination row) key, reserves one contiguous range per key in
// the destination row's bucket with a single atomic, and writes the records
// there. A second kernel reduces each row's bucket in LDS and adds the row's
// gradients with plain stores. LDS floating-point atomics are several times
// slower than integer ones here, so the row sums are accumulated in 64-bit
// fixed point, scaled by a power of two chosen from the row's largest record
// (bounded above by the largest component any contributing block staged)
// and record count so that no sum can overflow (integer sums are also
// independent of the order). Records that do not fit (a third source row in
// one block, a full bucket, an atom beyond the LDS row window) fall back to
// device atomics, so the result never depends on the capacities.
// ---------------------------------------------------------------------------
template <typename real>
struct PairGrad {
    real phi, dphi_r;   // phi and phi'(r)/r
    real a_coul;        // erfc/r^3 + 2b e^{-b^2 r^2}/(sqrt(pi) r^2): phi_coul = -qq a_coul
    real c_lj;          // 48 s^12/r^14 - 24 s^6/r^8: phi_lj = -eps c_lj
    real dc_dsig;       // d c_lj / d sigma
};

// LJ constants of one type pair for the adjoint (sigma powers folded in).
template <typename real>
struct LJGrad {
    real a48, b24;    // 48 s^12, 24 s^6:   c_lj = (a48 r^-6 - b24) r^-8
    real a672, b192;  // 672 s^12, 192 s^6: d c_lj / dr = (b192 - a672 r^-6) r^-9
    real as, bs;      // 576 s^11, 144 s^5: d c_lj / d sigma = (as r^-6 - bs) r^-8
    real eps, rc2;    // the LJ term acts at r^2 < rc2
};

template <typename real>
__device__ __forceinline__ LJGrad<real> lj_grad_entry(real sig, real eps, real lj_cut)
{
    const real s2 = sig * sig;
    const real s6 = s2 * s2 * s2;
    const real s12 = s6 * s6;
    LJGrad<real> L;
    L.a48 = (real)48 * s12;
    L.b24 = (real)24 * s6;
    L.a672 = (real)672 * s12;
    L.b192 = (real)192 * s6;
    L.as = sig != (real)0 ? (real)576 * s12 / sig : (real)0;
    L.bs = sig != (real)0 ? (real)144 * s6 / sig : (real)0;
    L.eps = eps;
    L.rc2 = lj_cut > (real)0 ? lj_cut * sig * lj_cut * sig : Math<real>::max_();
    return L;
}

// xp: an excluded pair, whose correction -erf(br)/r is the real-space term
// erfc(br)/r minus the bare 1/r: the Coulomb factor gains -1/r^3, phi gains
// qq/r^3, phi'/r gains -3 qq/r^5, and there is no LJ term.
template <typename real>
__device__ __forceinline__ PairGrad<real> pair_grad(real r2, real qq, const LJGrad<real>& L, const PairParams<real>& pp,
                                                    bool xp = false)
{
    // with A = erfc/r^3, B = cgauss e^{-b^2 r^2}/r^2 and a = A + B (- 1/r^3): phi = -qq a and
    // phi'/r = qq (3 a / r^2 + 2 b^2 B) for the Coulomb part
    const Radial<real> o = radial(r2, pp);
    const real rinv2 = o.rinv2;
    const real B = pp.cgauss * o.ex * rinv2;
    const real a = (xp ? o.g - o.rinv : o.g) * rinv2;
    const real r6 = rinv2 * rinv2 * rinv2;
    const real r8 = r6 * rinv2;
    const real on = (xp || !(r2 < L.rc2)) ? (real)0 : r8;
    const real C = on * (L.a48 * r6 - L.b24);
    const real dC = on * rinv2 * (L.b192 - L.a672 * r6);
    PairGrad<real> g;
    g.a_coul = a;
    g.phi = -qq * a - L.eps * C;
    g.dphi_r = qq * ((real)3 * rinv2 * a + (real)2 * pp.beta * pp.beta * B) - L.eps * dC;
    g.c_lj = C;
    g.dc_dsig = on * (L.as * r6 - L.bs);
    return g;
}

template <typename real>
__device__ __forceinline__ void load3(const real* p, int64_t k, real& x, real& y, real& z)
{
    x = p[3 * k];
    y = p[3 * k + 1];
    z = p[3 * k + 2];
}

// Geometry of the shell-adjoint buckets. Row R = cz n_c + cy holds the atoms of
// cells [R n_c, (R + 1) n_c); its bucket starts at
// floor(cell_start[R n_c] p9 / 8) + kBucketSlack R records (9/8 of the expected
// p_eff records per atom, plus slack).
struct BucketArgs {
    int n_c, lo, span;            // shell stencil offsets lo .. lo + span - 1 per axis
    int64_t p9;                   // 9 * p_eff
    const int32_t* cell_start;
    unsigned long long* cursor;   // [n_c^2] records reserved per destination row
    unsigned long long* rowmax;   // [n_c^2] bits of the largest |record component| (as a non-negative double)
    void* rec_c;                  // real[4 * total]
    uint16_t* rec_j;              // [total]
    unsigned long long* n_atomic; // records that took device atomics instead of a bucket
    const int32_t* brow;          // cell (z, y) at the build of each sorted atom (z << 16 | y), used for the keys
                                  // when positions may have moved since (lists with a skin); null: from positions
};

__device__ __forceinline__ int64_t bucket_start(const BucketArgs& bk, int row)
{
    const int64_t a = bk.cell_start[(int64_t)row * bk.n_c];
    return ((a * bk.p9) >> 3) + (int64_t)kBucketSlack * row;
}

__device__ __forceinline__ int cell_row(uint4 s, int n_c)
{
    const int cz = (int)(((uint64_t)s.z * (uint32_t)n_c) >> 32);
    const int cy = (int)(((uint64_t)s.y * (uint32_t)n_c) >> 32);
    return cz * n_c + cy;
}

// Cell coordinates (z, y) of sorted atom k for the bucket keys: those of its
// cell at the list build when the positions may have moved since, else those
// of its position.
__device__ __forceinline__ void key_cell(const BucketArgs& bk, int64_t k, uint4 s, int& z, int& y)
{
    if (bk.brow) {
        const int b = bk.brow[k];
        z = b >> 16;
        y = b & 0xffff;
    } else {
        z = (int)(((uint64_t)s.z * (uint32_t)bk.n_c) >> 32);
        y = (int)(((uint64_t)s.y * (uint32_t)bk.n_c) >> 32);
    }
}

// Offset d = c_j - c_i of a stencil cell mapped into [lo, lo + span).
__device__ __forceinline__ int stencil_offset(int cj, int ci, int lo, int span, int n_c)
{
    int d = cj - ci;
    if (d < lo) d += n_c;
    if (d >= lo + span) d -= n_c;
    return d;
}

template <typename real>
__device__ __forceinline__ void scatter_atomic(real* gscat, real* gqscat, int64_t j, real x, real y, real z, real q)
{
    atomicAdd(&gscat[3 * j + 0], x);
    atomicAdd(&gscat[3 * j + 1], y);
    atomicAdd(&gscat[3 * j + 2], z);
    atomicAdd(&gqscat[j], q);
}

// One wavefront per atom (cell order), lanes over the atom's lists. BK: the
// shell scatter goes through the LDS-staged buckets (dynamic LDS: rec_cap
// records of 4 reals + j + key, then 7 ints per key).
// STENCIL: the batch of stencil sampling, decoded (drawn atoms, -1: none); BATCH:
// the list-drawn batch as the forward wrote it (batch_j), in place of the ranks
// and the shell rows.
template <typename real, bool FULL, bool WANT_LJ, bool BK, bool STENCIL, bool SKIN, bool BATCH>
__global__ __launch_bounds__(kCoopBlock) void k_pair_adjoint(
    int64_t n, int apw, PairParams<real> pp, const uint4* __restrict__ spos, const real* __restrict__ sqr,
    const uint4* __restrict__ spq, const int2* __restrict__ sxr, const int32_t* __restrict__ sxidx, const int32_t* __restrict__ core,
    const int32_t* __restrict__ ncore, int cap_core, const int32_t* __restrict__ shell,
    const int32_t* __restrict__ nshell, int cap_shell, const real* __restrict__ ljraw_g, int n_types, int p_shell,
    int p_stride, const uint16_t* __restrict__ ranks, const int32_t* __restrict__ batch_j, uint64_t t_core,
    uint64_t t_shell, real lj_cut, const real* __restrict__ gs, const double* __restrict__ gmean_d,
    real* __restrict__ gself, real* __restrict__ gscat, real* __restrict__ gqself, real* __restrict__ gqscat,
    double* __restrict__ ljpart, BucketArgs bk, int rec_cap)
{
    constexpr int NLJ = 2 * kMaxTypesGrad * kMaxTypesGrad;
    constexpr int NW = kCoopBlock / 64;
    __shared__ LJGrad<real> ljg[256];
    __shared__ int lj_row[16];  // 1 when some sigma of type t's row is nonzero (else no LJ term or gradient)
    __shared__ double ljacc[NW][NLJ];
    __shared__ int nrec;
    __shared__ double bmaxw[NW];
    extern __shared__ __align__(16) unsigned char bk_lds[];
    real* rc = (real*)bk_lds;                              // [rec_cap][4]
    int32_t* rj = (int32_t*)(rc + 4 * (size_t)rec_cap);    // [rec_cap] sorted index of j
    uint16_t* rk = (uint16_t*)(rj + rec_cap);              // [rec_cap] key
    const int span2 = bk.span * bk.span;
    const int nkeys = 2 * span2;
    int32_t* kcnt = (int32_t*)(rk + ((rec_cap + 1) & ~1));  // [nkeys] records per key
    int32_t* kcur = kcnt + nkeys;                           // [nkeys] write cursor
    int32_t* kbase = kcur + nkeys;                          // [nkeys] reserved offset in the bucket
    int32_t* kdst = kbase + nkeys;                          // [nkeys] destination row
    int32_t* kfirst = kdst + nkeys;                         // [nkeys] first atom of the row
    int32_t* kcap = kfirst + nkeys;                         // [nkeys] bucket capacity
    int32_t* kcount = kcap + nkeys;                         // [nkeys] atoms of the row in the LDS window
    const int nt2 = n_types * n_types;
    for (int t = threadIdx.x; t < nt2; t += kCoopBlock) ljg[t] = lj_grad_entry(ljraw_g[t], ljraw_g[nt2 + t], lj_cut);
    if (threadIdx.x < n_types) {
        int any = 0;
        for (int u = 0; u < n_types; ++u) any |= ljraw_g[threadIdx.x * n_types + u] != (real)0;
        lj_row[threadIdx.x] = any;
    }
    // the wavefront's index as a wave-uniform value (scalar atom indices and row addresses)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (WANT_LJ)
        for (int t = lane; t < NLJ; t += 64) ljacc[wave][t] = 0.0;
    if (BK) {
        for (int t = threadIdx.x; t < nkeys; t += kCoopBlock) kcnt[t] = 0;
        if (threadIdx.x == 0) nrec = 0;
    }
    __syncthreads();
    const real mx = FULL ? (real)0 : (real)gmean_d[0];
    const real my = FULL ? (real)0 : (real)gmean_d[1];
    const real mz = FULL ? (real)0 : (real)gmean_d[2];
    const real ke = pp.ke;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t gw = blk * NW + wave;
    const int64_t a0 = gw * apw;
    const int64_t a1 = min(n, a0 + apw);
    // cell row of the block's first atom: the block's atoms lie in rows row0, row0 + 1, ...
    int row0 = 0;
    if (BK) {
        const int64_t f = min(blk * NW * apw, n - 1);
        int z, y;
        if constexpr (std::is_same<real, float>::value) key_cell(bk, f, spq[f], z, y);
        else key_cell(bk, f, spos[f], z, y);
        row0 = z * bk.n_c + y;
    }
    real lane_max = 0;  // largest |component| of the records this lane staged
    const Atoms<real> at{spos, sqr, spq};
    // per-atom headers of the wavefront's atoms, one atom per lane, read once
    const int64_t ah = min(a0 + min(lane, apw - 1), n - 1);
    uint4 h_s;
    real h_q;
    at.get(ah, h_s, h_q);
    const real h_gx = gs[3 * ah], h_gy = gs[3 * ah + 1], h_gz = gs[3 * ah + 2];
    const int h_nsym = FULL ? nshell[ah] : ncore[ah];
    const int h_ns = FULL ? 0 : nshell[ah];
    const int2 h_x = sxr[ah];
    // shell weight N_S / p~ (1 when every member is taken), one division per lane
    const real h_w = h_ns > p_shell ? (real)((double)h_ns / (double)p_shell) : (real)1;
    // first-level indices of one atom's first pass: the lane's first symmetric-list entry
    // or excluded partner and its two batch ranks (or shell positions)
    auto first_level = [&](int64_t a, int t, int& jc, int& r0, int& r1) {
        const int nsym = bcast(h_nsym, t);
        const int ns = bcast(h_ns, t);
        const int2 xr = make_int2(bcast(h_x.x, t), bcast(h_x.y, t));
        const bool sample = ns > p_shell;
        const int cnt = sample ? p_shell : ns;
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;
        const int32_t* srow_sym = FULL ? shell + a * (int64_t)cap_shell : core + a * (int64_t)cap_core;
        // the excluded partners follow the symmetric list (entries nsym .. nsym + nx - 1)
        jc = lane < nsym ? srow_sym[lane] : (lane < nsym + xr.y ? sxidx[xr.x + lane - nsym] : -1);
        if (STENCIL || BATCH) {
            // the decoded batch (atoms; with stencil sampling -1 for i itself and i's
            // molecule) in place of ranks
            const int32_t* brow = batch_j + a * (int64_t)p_stride;
            r0 = lane < cnt ? brow[lane] : -1;
            r1 = lane + 64 < cnt ? brow[lane + 64] : -1;
        } else {
            r0 = lane < cnt ? (sample ? (int)rrow[lane] : lane) : -1;
            r1 = lane + 64 < cnt ? (sample ? (int)rrow[lane + 64] : lane + 64) : -1;
        }
    };
    int n_jc = -1, n_r0 = -1, n_r1 = -1;
    if (a0 < a1) first_level(a0, 0, n_jc, n_r0, n_r1);
    for (int64_t a = a0; a < a1; ++a) {
        const int t_a = (int)(a - a0);
        const int jc = n_jc, r0 = n_r0, r1 = n_r1;
        // the next atom's first-level loads go out before this atom's dependent ones
        if (a + 1 < a1) first_level(a + 1, t_a + 1, n_jc, n_r0, n_r1);
        const uint4 si = make_uint4(bcast(h_s.x, t_a), bcast(h_s.y, t_a), bcast(h_s.z, t_a),
                                    bcast(h_s.w, t_a));
        const int ti = (int)si.w;
        const int li = __mul24(ti, n_types);  // the atom's row of the LJ table
        int zi = 0, yi = 0;  // the atom's cell for the bucket keys
        if (BK) key_cell(bk, a, si, zi, yi);
        // with every sigma of its row zero, the atom has no LJ term and no LJ gradient
        const bool lj_i = WANT_LJ && lj_row[ti];
        const real qi = ke * bcast(h_q, t_a);
        const real gx = bcast(h_gx, t_a), gy = bcast(h_gy, t_a), gz = bcast(h_gz, t_a);
        const real pgx = gx - mx, pgy = gy - my, pgz = gz - mz;  // G'_i
        const int nsym = bcast(h_nsym, t_a);
        const int ns = bcast(h_ns, t_a);
        const int2 xr = make_int2(bcast(h_x.x, t_a), bcast(h_x.y, t_a));
        real rx = 0, ry = 0, rz = 0, rq = 0;
        real acc_sig[kMaxTypesGrad], acc_eps[kMaxTypesGrad];
#pragma unroll
        for (int t = 0; t < kMaxTypesGrad; ++t) acc_sig[t] = acc_eps[t] = 0;
        const int32_t* srow_sym = FULL ? shell + a * (int64_t)cap_shell : core + a * (int64_t)cap_core;
        const int32_t* srow = shell + a * (int64_t)cap_shell;
        const bool sample = ns > p_shell;
        const int cnt = sample ? p_shell : ns;
        const real w = bcast(h_w, t_a);
        const uint16_t* rrow = ranks + a * (int64_t)p_stride;

        // symmetric sets (core pairs, or the whole list in full-list mode, and the
        // excluded pairs, xp): gathered. G'_j - G'_i = G_j - G_i, so the same
        // difference serves both.
        auto sym_pair = [&](uint4 sj, real qj, real gjx, real gjy, real gjz, bool xp) {
            real dx, dy, dz;
            separation(si, sj, pp.quantum, dx, dy, dz);
            const real r2 = dx * dx + dy * dy + dz * dz;
            const LJGrad<real>& L = ljg[li + (int)sj.w];
            const PairGrad<real> g = pair_grad(r2, qi * qj, L, pp, xp);
            const real ex_ = gjx - gx, ey_ = gjy - gy, ez_ = gjz - gz;
            const real gd = dx * ex_ + dy * ey_ + dz * ez_;
            const real dg = g.dphi_r * gd;
            rx += g.phi * ex_ + dg * dx;
            ry += g.phi * ey_ + dg * dy;
            rz += g.phi * ez_ + dg * dz;
            rq += qj * g.a_coul * gd;
            if (lj_i) {
                const real gdi = dx * pgx + dy * pgy + dz * pgz;
                const int tj = (int)sj.w;
#pragma unroll
                for (int t = 0; t < kMaxTypesGrad; ++t)
                    if (t == tj) {
                        acc_sig[t] += -L.eps * g.dc_dsig * gdi;
                        acc_eps[t] += -g.c_lj * gdi;
                    }
            }
        };
        // sampled shell pairs, one-sided: gathered for i, scattered for j
        auto shell_pair = [&](int j, uint4 sj, real qj) {
            real dx, dy, dz;
            separation(si, sj, pp.quantum, dx, dy, dz);
            const real r2 = dx * dx + dy * dy + dz * dz;
            const LJGrad<real>& L = ljg[li + (int)sj.w];
            const PairGrad<real> g = pair_grad(r2, qi * qj, L, pp);
            const real gdi = dx * pgx + dy * pgy + dz * pgz;
            const real wphi = w * g.phi, dg = w * g.dphi_r * gdi;
            const real jx_ = wphi * pgx + dg * dx;
            const real jy_ = wphi * pgy + dg * dy;
            const real jz_ = wphi * pgz + dg * dz;
            rx -= jx_;
            ry -= jy_;
            rz -= jz_;
            const real wag = w * g.a_coul * gdi;
            rq -= qj * wag;
            const real jq_ = -qi * wag;
            bool staged = false;
            if (BK) {
                // key: (source row - row0, row offset of j), on the cells of the build
                // when positions may have moved since
                const int nc_ = bk.n_c;
                const int src = zi * nc_ + yi - row0;  // wave-uniform
                int zj, yj;
                key_cell(bk, j, sj, zj, yj);
                const int kz = stencil_offset(zj, zi, bk.lo, bk.span, nc_) - bk.lo;
                const int ky = stencil_offset(yj, yi, bk.lo, bk.span, nc_) - bk.lo;
                if (src >= 0 && src < 2 && kz >= 0 && kz < bk.span && ky >= 0 && ky < bk.span) {
                    const int key = src * span2 + kz * bk.span + ky;
                    const uint64_t m = __ballot(1);
                    const int leader = __ffsll((unsigned long long)m) - 1;
                    int base = 0;
                    if (lane == leader) base = atomicAdd(&nrec, __popcll(m));
                    base = __shfl(base, leader, 64);
                    const int slot = base + __popcll(m & ((1ull << lane) - 1ull));
                    if (slot < rec_cap) {
                        rc[4 * slot + 0] = jx_;
                        rc[4 * slot + 1] = jy_;
                        rc[4 * slot + 2] = jz_;
                        rc[4 * slot + 3] = jq_;
                        rj[slot] = j;
                        rk[slot] = (uint16_t)key;
                        atomicAdd(&kcnt[key], 1);
                        lane_max = fmax(lane_max, fmax(fmax(fabs(jx_), fabs(jy_)), fmax(fabs(jz_), fabs(jq_))));
                        staged = true;
                    }
                }
            }
            if (!staged) {
                scatter_atomic(gscat, gqscat, (int64_t)j, jx_, jy_, jz_, jq_);
                if (BK) atomicAdd(bk.n_atomic, 1ull);
            }
            if (lj_i) {
                const int tj = (int)sj.w;
#pragma unroll
                for (int t = 0; t < kMaxTypesGrad; ++t)
                    if (t == tj) {
                        acc_sig[t] += w * (-L.eps * g.dc_dsig * gdi);
                        acc_eps[t] += w * (-g.c_lj * gdi);
                    }
            }
        };
        // first pass, every load of the dependent levels issued together (unused
        // slots load atom 0)
        const int js0 = (STENCIL || BATCH) ? r0 : ((!FULL && r0 >= 0) ? srow[r0] : -1);
        const int js1 = (STENCIL || BATCH) ? r1 : ((!FULL && r1 >= 0) ? srow[r1] : -1);
        const int ic = max(jc, 0), i0 = max(js0, 0), i1 = max(js1, 0);
        uint4 pjc, pj0, pj1;
        real qjc, qj0, qj1;
        at.get(ic, pjc, qjc);
        const real gcx = gs[3 * (int64_t)ic], gcy = gs[3 * (int64_t)ic + 1], gcz = gs[3 * (int64_t)ic + 2];
        at.get(i0, pj0, qj0);
        at.get(i1, pj1, qj1);
        // skin: a symmetric-list entry counts inside r_core (r_shell for the full
        // list), a list shell entry inside the annulus, at these positions
        const uint64_t t_sym = FULL ? t_shell : t_core;
        auto sym_ok = [&](uint4 sj) { return !SKIN || dist2_q(si, sj) <= t_sym; };
        constexpr bool shell_test = STENCIL || SKIN;
        if (jc >= 0 && (lane >= nsym || sym_ok(pjc))) sym_pair(pjc, qjc, gcx, gcy, gcz, lane >= nsym);
        if (js0 >= 0 && (!shell_test || in_annulus(si, pj0, t_core, t_shell))) shell_pair(js0, pj0, qj0);
        if (js1 >= 0 && (!shell_test || in_annulus(si, pj1, t_core, t_shell))) shell_pair(js1, pj1, qj1);
        // the rest (long lists and large batches)
        for (int c = lane + 64; c < nsym + xr.y; c += 64) {
            const int j = c < nsym ? srow_sym[c] : sxidx[xr.x + c - nsym];
            uint4 sj;
            real qj;
            at.get(j, sj, qj);
            if (c >= nsym || sym_ok(sj))
                sym_pair(sj, qj, gs[3 * (int64_t)j], gs[3 * (int64_t)j + 1], gs[3 * (int64_t)j + 2], c >= nsym);
        }
        if (!FULL)
            for (int c = lane + 128; c < cnt; c += 64) {
                if (STENCIL || BATCH) {
                    const int j = batch_j[a * (int64_t)p_stride + c];
                    if (j < 0) continue;
                    uint4 sj;
                    real qj;
                    at.get(j, sj, qj);
                    if (!shell_test || in_annulus(si, sj, t_core, t_shell)) shell_pair(j, sj, qj);
                } else {
                    const int j = srow[sample ? (int)rrow[c] : c];
                    uint4 sj;
                    real qj;
                    at.get(j, sj, qj);
                    if (!SKIN || in_annulus(si, sj, t_core, t_shell)) shell_pair(j, sj, qj);
                }
            }
        const real r = wave_sum4(rx, ry, rz, rq);
        if ((lane & 15) == 0) {
            if (lane < 48) gself[3 * a + (lane >> 4)] = r;
            else gqself[a] = ke * r;
        }
        if (lj_i && ti < kMaxTypesGrad) {
            static_assert(kMaxTypesGrad == 4, "one row of lanes per partner type");
            const real s_sig = wave_sum4(acc_sig[0], acc_sig[1], acc_sig[2], acc_sig[3]);
            const real s_eps = wave_sum4(acc_eps[0], acc_eps[1], acc_eps[2], acc_eps[3]);
            if ((lane & 15) == 0) {
                const int t = ti * kMaxTypesGrad + (lane >> 4);
                ljacc[wave][t] += (double)s_sig;
                ljacc[wave][kMaxTypesGrad * kMaxTypesGrad + t] += (double)s_eps;
            }
        }
    }
    if (WANT_LJ) {
        __syncthreads();
        if (threadIdx.x < NLJ) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += ljacc[w][threadIdx.x];
            ljpart[blk * (int64_t)NLJ + threadIdx.x] = t;
        }
    }
    if (BK) {
        // reserve one range per key in its destination row's bucket, and raise the
        // row's bound on |record| to this block's largest staged component
        double wmax = (double)lane_max;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) wmax = fmax(wmax, __shfl_xor(wmax, off, 64));
        if (lane == 0) bmaxw[wave] = wmax;
        __syncthreads();
        double bmax = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) bmax = fmax(bmax, bmaxw[w]);
        for (int t = threadIdx.x; t < nkeys; t += kCoopBlock) {
            const int c = kcnt[t];
            kcur[t] = 0;
            if (c == 0) continue;
            const int src = row0 + t / span2;
            const int rem = t % span2;
            const int dz = rem / bk.span + bk.lo, dy = rem % bk.span + bk.lo;
            int z = src / bk.n_c + dz, y = src % bk.n_c + dy;
            z = z < 0 ? z + bk.n_c : (z >= bk.n_c ? z - bk.n_c : z);
            y = y < 0 ? y + bk.n_c : (y >= bk.n_c ? y - bk.n_c : y);
            const int dst = z * bk.n_c + y;
            const int64_t b0 = bucket_start(bk, dst);
            const int64_t cap = bucket_start(bk, dst + 1) - b0;
            kdst[t] = dst;
            kfirst[t] = bk.cell_start[(int64_t)dst * bk.n_c];
            kcount[t] = min(bk.cell_start[(int64_t)(dst + 1) * bk.n_c] - kfirst[t], kBucketRowLds);
            kcap[t] = (int32_t)min(cap, (int64_t)INT32_MAX);
            const unsigned long long old = atomicAdd(&bk.cursor[dst], (unsigned long long)c);
            kbase[t] = (int32_t)min(old, (unsigned long long)INT32_MAX);
            atomicMax(&bk.rowmax[dst], (unsigned long long)__double_as_longlong(bmax));
        }
        __syncthreads();
        const int nr = min(nrec, rec_cap);
        real* out_c = (real*)bk.rec_c;
        for (int s = threadIdx.x; s < nr; s += kCoopBlock) {
            const int key = rk[s];
            const int64_t pos = (int64_t)kbase[key] + atomicAdd(&kcur[key], 1);
            const int j = rj[s];
            const int jrel = j - kfirst[key];
            const int dst = kdst[key];
            if (pos < kcap[key]) {
                const int64_t at = bucket_start(bk, dst) + pos;
                if (jrel >= 0 && jrel < kcount[key]) {
                    out_c[4 * at + 0] = rc[4 * s + 0];
                    out_c[4 * at + 1] = rc[4 * s + 1];
                    out_c[4 * at + 2] = rc[4 * s + 2];
                    out_c[4 * at + 3] = rc[4 * s + 3];
                    bk.rec_j[at] = (uint16_t)jrel;
                    continue;
                }
                bk.rec_j[at] = (uint16_t)0xffffu;  // reserved slot left empty
            }
            scatter_atomic(gscat, gqscat, (int64_t)j, rc[4 * s + 0], rc[4 * s + 1], rc[4 * s + 2], rc[4 * s + 3]);
            atomicAdd(bk.n_atomic, 1ull);
        }
    }
}

template <typename real>
struct Rec4;
template <>
struct Rec4<float> {
    using type = float4;
};
template <>
struct Rec4<double> {
    using type = double4;
};

// Reduce one destination row's bucket: 64-bit fixed-point LDS sums over its
// records, then added to the row's scatter gradients (the atomics of the
// fallback paths already in place). One block per row. With m a bound on the
// row's largest |record component| and nr its record count, values are scaled
// by 2^sh with m nr 2^sh < 2^62, so no partial sum overflows.
template <typename real>
__global__ __launch_bounds__(512) void k_bucket_reduce(BucketArgs bk, real* __restrict__ gscat,
                                                       real* __restrict__ gqscat)
{
    __shared__ long long acc[4 * kBucketRowLds];  // component-major: acc[d * kBucketRowLds + j]
    const int row = (int)xcd_block(blockIdx.x, gridDim.x);
    const int first = bk.cell_start[(int64_t)row * bk.n_c];
    const int count = bk.cell_start[(int64_t)(row + 1) * bk.n_c] - first;
    const int nl = min(count, kBucketRowLds);
    const int64_t b0 = bucket_start(bk, row);
    const int64_t cap = bucket_start(bk, row + 1) - b0;
    const int64_t nr = (int64_t)min(bk.cursor[row], (unsigned long long)cap);
    const double mx = __longlong_as_double((long long)bk.rowmax[row]);
    if (nr == 0 || !(mx > 0.0)) return;  // block-uniform: no records or all zero
    int e;
    frexp(mx * (double)nr, &e);  // mx nr < 2^e
    const int sh = 62 - e;
    for (int t = threadIdx.x; t < nl; t += 512)
        for (int d = 0; d < 4; ++d) acc[d * kBucketRowLds + t] = 0;
    __syncthreads();
    using V4 = typename Rec4<real>::type;
    const V4* rcg = (const V4*)bk.rec_c + b0;
    const uint16_t* rjg = bk.rec_j + b0;
    // kU records per thread per pass, all loads issued before the LDS updates
    // (indices past the end are clamped to the last record and then ignored)
    constexpr int kU = 4;
    for (int64_t s0 = 0; s0 < nr; s0 += 512 * kU) {
        int jr[kU];
        V4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t s = s0 + u * 512 + threadIdx.x;
            const int64_t sc = min(s, nr - 1);
            jr[u] = rjg[sc];
            v[u] = rcg[sc];
            if (s >= nr) jr[u] = nl;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (jr[u] >= nl) continue;
            atomicAdd((unsigned long long*)&acc[0 * kBucketRowLds + jr[u]],
                      (unsigned long long)__double2ll_rn(ldexp((double)v[u].x, sh)));
            atomicAdd((unsigned long long*)&acc[1 * kBucketRowLds + jr[u]],
                      (unsigned long long)__double2ll_rn(ldexp((double)v[u].y, sh)));
            atomicAdd((unsigned long long*)&acc[2 * kBucketRowLds + jr[u]],
                      (unsigned long long)__double2ll_rn(ldexp((double)v[u].z, sh)));
            atomicAdd((unsigned long long*)&acc[3 * kBucketRowLds + jr[u]],
                      (unsigned long long)__double2ll_rn(ldexp((double)v[u].w, sh)));
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nl; k += 512) {
        const int64_t j = first + k;
        gscat[3 * j + 0] += (real)ldexp((double)acc[0 * kBucketRowLds + k], -sh);
        gscat[3 * j + 1] += (real)ldexp((double)acc[1 * kBucketRowLds + k], -sh);
        gscat[3 * j + 2] += (real)ldexp((double)acc[2 * kBucketRowLds + k], -sh);
        gqscat[j] += (real)ldexp((double)acc[3 * kBucketRowLds + k], -sh);
    }
}

template <typename real, bool FULL, bool WANT_LJ, bool BK, bool STENCIL, bool BATCH = false>
static hipError_t launch_adj_t(irbe_ctx* h, uint64_t step, int apw, const BucketArgs& bk, int rec_cap, size_t lds)
{
    const int64_t n = h->cfg.n_atoms;
    const PairParams<real> pp = pair_params<real>(h);
    hipError_t e = launch_draw(h, step);
    if (e != hipSuccess) return e;
    if (STENCIL && !h->batch_j_valid) {
        // the adjoint reads the batch decoded once (its blocks hold too few atoms
        // for the per-wavefront decode of the forward kernel to pay)
        e = launch_stencil_decode(h);
        if (e != hipSuccess) return e;
        h->batch_j_valid = true;
    }
    const int64_t waves = blocks_for(n, apw);
    const unsigned nb = (unsigned)blocks_for(waves, kCoopBlock / 64);
    if ((int64_t)nb > h->part_blocks) return hipErrorInvalidValue;
    h->adj_nb = nb;
#define IRBE_ADJ_ARGS                                                                                         \
    n, apw, pp, h->spos, (const real*)h->sq_r, h->spq, h->sxr, h->sxidx, h->core, h->ncore, h->cap_core, h->shell, \
        h->nshell, h->cap_shell, (const real*)h->lj_raw, h->cfg.n_types, h->cfg.p_shell, h->p_stride, h->ranks,  \
        h->batch_j, h->geo.t_core, h->geo.t_shell, (real)h->cfg.lj_cut, (const real*)h->gs, h->gmean,             \
        (real*)h->gself, (real*)h->gscat, (real*)h->gqself, (real*)h->gqscat, h->ljpart, bk, rec_cap
    if (h->geo.skin)
        k_pair_adjoint<real, FULL, WANT_LJ, BK, STENCIL, true, BATCH><<<nb, kCoopBlock, lds, h->stream>>>(IRBE_ADJ_ARGS);
    else
        k_pair_adjoint<real, FULL, WANT_LJ, BK, STENCIL, false, BATCH><<<nb, kCoopBlock, lds, h->stream>>>(IRBE_ADJ_ARGS);
    h->adj_used_batch = BATCH;
#undef IRBE_ADJ_ARGS
    e = hipGetLastError();
    if (e != hipSuccess || !BK) return e;
    const unsigned rows = (unsigned)((int64_t)bk.n_c * bk.n_c);
    k_bucket_reduce<real><<<rows, 512, 0, h->stream>>>(bk, (real*)h->gscat, (real*)h->gqscat);
    return hipGetLastError();
}

template <typename real, bool BK>
static hipError_t launch_adj_r(irbe_ctx* h, uint64_t step, bool want_lj, int apw, const BucketArgs& bk, int rec_cap,
                               size_t lds)
{
    if (h->full_list)
        return want_lj ? launch_adj_t<real, true, true, false, false>(h, step, apw, bk, 0, 0)
                       : launch_adj_t<real, true, false, false, false>(h, step, apw, bk, 0, 0);
    if (h->stencil) {
        // (the batch atoms the forward wrote when it was asked to, else decoded)
        const bool from_fwd = h->ranks_valid && h->ranks_step == step && h->batch_j_valid && h->batch_j_fwd;
        const hipError_t e = want_lj ? launch_adj_t<real, false, true, BK, true>(h, step, apw, bk, rec_cap, lds)
                                     : launch_adj_t<real, false, false, BK, true>(h, step, apw, bk, rec_cap, lds);
        h->adj_used_batch = from_fwd;
        return e;
    }
    // the batch atoms the forward wrote, when they are those of this step's ranks
    // (launch_draw keeps them unless it draws again); with shell lists as masks
    // the atoms at the ranks decoded once otherwise
    hipError_t e = launch_draw(h, step);
    if (e != hipSuccess) return e;
    const bool from_fwd = h->batch_j_valid && h->batch_j_fwd;
    if (h->masks && !h->batch_j_valid) {
        e = launch_list_decode(h);
        if (e != hipSuccess) return e;
        h->batch_j_valid = true;
        h->batch_j_fwd = false;
    }
    if (h->batch_j_valid) {
        e = want_lj ? launch_adj_t<real, false, true, BK, false, true>(h, step, apw, bk, rec_cap, lds)
                    : launch_adj_t<real, false, false, BK, false, true>(h, step, apw, bk, rec_cap, lds);
        h->adj_used_batch = from_fwd;
        return e;
    }
    return want_lj ? launch_adj_t<real, false, true, BK, false>(h, step, apw, bk, rec_cap, lds)
                   : launch_adj_t<real, false, false, BK, false>(h, step, apw, bk, rec_cap, lds);
}

hipError_t launch_pair_adjoint(irbe_ctx* h, uint64_t step, bool want_q, bool want_lj)
{
    (void)want_q;
    const int64_t n = h->cfg.n_atoms;
    // the scatter sums, the buckets' cursors and the atomics counter lie in one array
    const int64_t rows = (int64_t)h->geo.n_c * h->geo.n_c;
    hipError_t e = launch_fill_bytes0(h->stream, h->gscat, 4 * (size_t)n * h->real_size + (2 * (size_t)rows + 1) * 8);
    if (e != hipSuccess) return e;
    // bucketed transpose of the shell scatter when a block of >= 8 atoms' records
    // fits the LDS staging area and the keys fit their table
    BucketArgs bk{};
    bk.n_c = h->geo.n_c;
    bk.lo = h->geo.lo;
    bk.span = h->geo.hi - h->geo.lo + 1;
    int p_eff = std::max(1, std::min(h->cfg.p_shell, std::max(h->shell_bound(), 1)));
    if (h->stencil) {
        // records only for the drawn atoms inside the shell: p~ times the shell's
        // share of the stencil volume, with a margin (the rest take the atomics)
        const double L = h->cfg.box_length, edge = L / h->geo.n_c;
        const double span = (double)(h->geo.hi - h->geo.lo + 1) * edge;
        const double rs = h->cfg.r_shell, rc = h->cfg.r_core;
        const double frac = std::min(1.0, 4.0 / 3.0 * 3.14159265358979323846 * (rs * rs * rs - rc * rc * rc) / (span * span * span));
        p_eff = std::max(1, std::min(p_eff, (int)std::ceil(1.3 * frac * h->cfg.p_shell)));
    }
    // records staged per block: room for the shell terms of every atom of the block
    // (kCoopBlock / 64 wavefronts of apw atoms, p_eff records each); apw fills a
    // budget that keeps five blocks on a CU, but is at least 2 (the bucketed
    // path's minimum) while the records fit the LDS limit (p~ <= 256 in FP32,
    // 128 in FP64; beyond, the shell terms take device atomics)
    const int waves_pb = kCoopBlock / 64;
    const int rec_budget = h->fp64 ? kBucketRecD : kBucketRecF;
    const int rec_max = h->fp64 ? kBucketRecMaxD : kBucketRecMaxF;
    int apw = std::min(kAtomsPerWave, std::max(2, rec_budget / (waves_pb * p_eff)));
    // a block's atoms within two cell rows, the source rows its keys cover: at most
    // 0.9 of a row's mean population per block (dilute small boxes), else the rest
    // of its shell records would take the atomic fallback
    const double row_atoms = (double)n / ((double)bk.n_c * (double)bk.n_c);
    apw = std::min(apw, std::max(2, (int)(0.9 * row_atoms / waves_pb)));
    if (waves_pb * apw * p_eff > rec_max) apw = rec_max / (waves_pb * p_eff);
    const int rec_cap = waves_pb * std::max(apw, 1) * p_eff;
    const int nkeys = 2 * bk.span * bk.span;
    const bool use_bk = !h->full_list && apw >= 2 && nkeys <= kBucketMaxKeys;
    size_t lds = 0;
    if (use_bk) {
        bk.p9 = 9 * (int64_t)p_eff;
        const int64_t total = ((int64_t)n * bk.p9 >> 3) + (int64_t)kBucketSlack * (rows + 1);
        e = ensure_buckets(h, total);
        if (e != hipSuccess) return e;
        bk.n_atomic = h->adj_atomics;
        bk.brow = h->geo.skin ? h->brow : nullptr;
        bk.cell_start = h->cell_start;
        bk.cursor = h->bk_cursor;
        bk.rowmax = h->bk_cursor + rows;
        bk.rec_c = h->bk_c;
        bk.rec_j = h->bk_j;
        lds = (size_t)rec_cap * (4 * h->real_size + 4) + (size_t)((rec_cap + 1) & ~1) * 2 + (size_t)nkeys * 7 * 4;
    }
    h->adj_all_atomic = !use_bk;
    if (h->fp64)
        return use_bk ? launch_adj_r<double, true>(h, step, want_lj, apw, bk, rec_cap, lds)
                      : launch_adj_r<double, false>(h, step, want_lj, kAtomsPerWave, bk, 0, 0);
    return use_bk ? launch_adj_r<float, true>(h, step, want_lj, apw, bk, rec_cap, lds)
                  : launch_adj_r<float, false>(h, step, want_lj, kAtomsPerWave, bk, 0, 0);
}

}  // namespace irbe
