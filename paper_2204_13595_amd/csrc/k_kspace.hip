// Long-range part: random batch Ewald (Sec. 2.2).
//   k-draw:  p vectors m_l from P_k = exp(-k^2/(4 alpha))/S, k = 2 pi m / L
//            (Eqs. (2.6)-(2.8)), per axis by inverse CDF on 64-bit Philox
//            words, the triple (0,0,0) redrawn;
//   rho:     rho_l = sum_j q_j e^{i k_l . r_j} (Eq. (2.4)) with the exact integer
//            phase (m_l . s_j) mod 2^32, FP64 accumulation, fixed-order
//            two-stage reduction;
//   force:   F_i^long,* = -ke q_i sum_l (S/p) 4 pi k_l/(V k_l^2) Im(e^{-i k_l.r_i} rho_l)
//            (Eq. (2.9)), added to the corrected short-range force and written
//            in the caller's atom order.
// Plus the adjoint (A_l = sum_m q_m (G_m . k_l) e^{i theta_ml}) and the
// energy/virial finalisation.
#include <algorithm>
#include <type_traits>

#include "irbe_device.hpp"
#include "irbe_internal.hpp"

namespace irbe {

// k-vectors per block row of the structure-factor kernels (measured optima at 3.1M
// atoms and p = 100: 8 forward and 16 in the adjoint, whose row also carries A).
constexpr int rho_chunk(bool adj) { return adj ? 16 : 8; }

// Atoms per thread: 16 in FP32 and 8 in FP64 (the optima at 3.1M atoms) while that
// gives kRhoMinBlocks blocks, else a quarter, else one, so that small systems
// still spread over the chip (2,703 atoms, p = 200: 25 blocks of 128 sines and
// cosines per thread and k-vector row took 14 us).
constexpr int64_t kRhoMinBlocks = 256;
constexpr int rho_most(bool fp64) { return fp64 ? 8 : 16; }

int rho_atoms(const irbe_ctx* h, bool adj)
{
    const int most = rho_most(h->fp64);
    if (h->rho_wide) return most;
    const int64_t rows = blocks_for(h->cfg.p_kspace, rho_chunk(adj));
    for (int a = most; a > 1; a /= 4)
        if (blocks_for(h->cfg.n_atoms, (int64_t)kBlock * a) * rows >= kRhoMinBlocks) return a;
    return 1;
}

// Blocks of partial sums: the larger count of the two shapes.
int64_t rho_blocks(const irbe_ctx* h)
{
    return blocks_for(h->cfg.n_atoms, (int64_t)kBlock * std::min(rho_atoms(h, false), rho_atoms(h, true)));
}

// Partial structure factors: block (b, c) sums atoms [b*kBlock*A, ...) for the
// k-vectors of chunk c. part layout: [(l * nb + b) * NV + v], NV = 2 (rho) or
// 4 (rho and A).
template <typename real, bool ADJ, int A>
__global__ __launch_bounds__(kBlock) void k_rho_partial(int64_t n, int P, const uint4* __restrict__ sq,
                                                        const real* __restrict__ q, const int4* __restrict__ kvec,
                                                        const double* __restrict__ kcoef, const real* __restrict__ G,
                                                        double* __restrict__ part)
{
    constexpr int RC = rho_chunk(ADJ);
    constexpr int NV = ADJ ? 4 : 2;
    __shared__ double lds[NV * RC * (kBlock / 64)];
    const int64_t nb = gridDim.x;
    const int l0 = blockIdx.y * RC;
    uint32_t sx[A], sy[A], sz[A];
    real qa[A], gx[A], gy[A], gz[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int64_t i = (int64_t)blockIdx.x * kBlock * A + (int64_t)a * kBlock + threadIdx.x;
        if (i < n) {
            const uint4 s = sq[i];
            sx[a] = s.x; sy[a] = s.y; sz[a] = s.z;
            qa[a] = q[i];
            if (ADJ) {
                gx[a] = G[3 * i]; gy[a] = G[3 * i + 1]; gz[a] = G[3 * i + 2];
            }
        } else {
            sx[a] = sy[a] = sz[a] = 0u;
            qa[a] = 0;
            gx[a] = gy[a] = gz[a] = 0;
        }
    }
    double acc[NV * RC];
#pragma unroll
    for (int c = 0; c < RC; ++c) {
        const int l = l0 + c;
        double re = 0.0, im = 0.0, are = 0.0, aim = 0.0;
        if (l < P) {
            const int4 m = kvec[l];
            real kx = 0, ky = 0, kz = 0;
            if (ADJ) {
                kx = (real)kcoef[4 * l]; ky = (real)kcoef[4 * l + 1]; kz = (real)kcoef[4 * l + 2];
            }
#pragma unroll
            for (int a = 0; a < A; ++a) {
                real sn, cs;
                Math<real>::sincos_rev(phase_rev<real>(m.x, m.y, m.z, sx[a], sy[a], sz[a]), &sn, &cs);
                re += (double)(qa[a] * cs);
                im += (double)(qa[a] * sn);
                if (ADJ) {
                    const real g = qa[a] * (gx[a] * kx + gy[a] * ky + gz[a] * kz);
                    are += (double)(g * cs);
                    aim += (double)(g * sn);
                }
            }
        }
        acc[NV * c + 0] = re;
        acc[NV * c + 1] = im;
        if (ADJ) {
            acc[NV * c + 2] = are;
            acc[NV * c + 3] = aim;
        }
    }
    double out;
    block_sum_vec<NV * RC, kBlock>(acc, lds, threadIdx.x, out);
    if (threadIdx.x < NV * RC) {
        const int c = threadIdx.x / NV, v = threadIdx.x % NV;
        const int l = l0 + c;
        if (l < P) part[((int64_t)l * nb + blockIdx.x) * NV + v] = out;
    }
}

// rho_l (and A_l) = fixed-order sums of the partials; then the per-k constants
// of the force (KForce) or adjoint (KAdj) kernels.
template <typename real, bool ADJ>
__global__ __launch_bounds__(kReduceBlock) void k_rho_final(int64_t nb, const double* __restrict__ part,
                                                            const double* __restrict__ kcoef, double* __restrict__ rho,
                                                            double* __restrict__ Avec, void* __restrict__ kconst)
{
    constexpr int NV = ADJ ? 4 : 2;
    __shared__ double lds[NV * (kReduceBlock / 64)];
    const int l = blockIdx.x;
    double vals[NV];
    for (int v = 0; v < NV; ++v) vals[v] = 0.0;
    for (int64_t b = threadIdx.x; b < nb; b += kReduceBlock)
        for (int v = 0; v < NV; ++v) vals[v] += part[((int64_t)l * nb + b) * NV + v];
    double out;
    block_sum_vec<NV, kReduceBlock>(vals, lds, threadIdx.x, out);
    __shared__ double tot[4];
    if (threadIdx.x < NV) tot[threadIdx.x] = out;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double c = kcoef[4 * l + 3];
        rho[2 * l] = tot[0];
        rho[2 * l + 1] = tot[1];
        if (!ADJ) {
            KForce<real> kf;
            kf.kx = (real)kcoef[4 * l];
            kf.ky = (real)kcoef[4 * l + 1];
            kf.kz = (real)kcoef[4 * l + 2];
            kf.a = (real)(c * tot[1]);
            kf.b = (real)(c * tot[0]);
            kf.pad0 = kf.pad1 = kf.pad2 = 0;
            ((KForce<real>*)kconst)[l] = kf;
        } else {
            Avec[2 * l] = tot[2];
            Avec[2 * l + 1] = tot[3];
            KAdj<real> ka;
            ka.kx = (real)kcoef[4 * l];
            ka.ky = (real)kcoef[4 * l + 1];
            ka.kz = (real)kcoef[4 * l + 2];
            ka.ar = (real)(c * tot[2]);
            ka.ai = (real)(c * tot[3]);
            ka.rr = (real)(c * tot[0]);
            ka.ri = (real)(c * tot[1]);
            ka.pad = 0;
            ((KAdj<real>*)kconst)[l] = ka;
        }
    }
}

template <typename real, bool ADJ, int A>
static hipError_t launch_rho_a(irbe_ctx* h, const void* grad)
{
    const int64_t n = h->cfg.n_atoms;
    const int P = h->cfg.p_kspace;
    const int64_t nb = blocks_for(n, kBlock * A);
    const dim3 grid((unsigned)nb, (unsigned)((P + rho_chunk(ADJ) - 1) / rho_chunk(ADJ)));
    k_rho_partial<real, ADJ, A><<<grid, kBlock, 0, h->stream>>>(n, P, h->sq, (const real*)h->q_orig, h->kvec, h->kcoef,
                                                                 (const real*)grad, h->rho_part);
    k_rho_final<real, ADJ><<<P, kReduceBlock, 0, h->stream>>>(nb, h->rho_part, h->kcoef, h->rho, h->Avec,
                                                               ADJ ? h->kadj : h->kforce);
    return hipGetLastError();
}

template <typename real, bool ADJ>
static hipError_t launch_rho_t(irbe_ctx* h, const void* grad)
{
    constexpr int most = rho_most(sizeof(real) == 8);
    const int a = rho_atoms(h, ADJ);
    if (a == most) return launch_rho_a<real, ADJ, most>(h, grad);
    if (a == most / 4) return launch_rho_a<real, ADJ, most / 4>(h, grad);
    return launch_rho_a<real, ADJ, 1>(h, grad);
}

hipError_t launch_rho(irbe_ctx* h, const void* grad, bool with_adjoint)
{
    if (with_adjoint) return h->fp64 ? launch_rho_t<double, true>(h, grad) : launch_rho_t<float, true>(h, grad);
    return h->fp64 ? launch_rho_t<double, false>(h, nullptr) : launch_rho_t<float, false>(h, nullptr);
}

// Per atom (caller order): F_i = F_i^sr - F^corr + F_i^long,* with
// F_i^long,* = -q_i sum_l k_l (cos th a_l - sin th b_l), a_l = ke c_l Im rho_l,
// b_l = ke c_l Re rho_l, so that Im(e^{-i th} rho) = cos th Im rho - sin th Re rho.
template <typename real>
__global__ __launch_bounds__(kBlock) void k_kspace_forces(int64_t n, int P, const uint4* __restrict__ sq,
                                                          const real* __restrict__ q, const int32_t* __restrict__ rank,
                                                          const real* __restrict__ fsr, const int4* __restrict__ kvec,
                                                          const KForce<real>* __restrict__ kf,
                                                          const double* __restrict__ fcorr, real* __restrict__ force)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint4 s = sq[i];
    real fx = 0, fy = 0, fz = 0;
    for (int l = 0; l < P; ++l) {
        const int4 m = kvec[l];
        const KForce<real> c = kf[l];
        real sn, cs;
        Math<real>::sincos_rev(phase_rev<real>(m.x, m.y, m.z, s.x, s.y, s.z), &sn, &cs);
        const real g = cs * c.a - sn * c.b;
        fx += g * c.kx;
        fy += g * c.ky;
        fz += g * c.kz;
    }
    const real qi = q[i];
    const int64_t k = rank[i];
    force[3 * i + 0] = fsr[3 * k + 0] - (real)fcorr[0] - qi * fx;
    force[3 * i + 1] = fsr[3 * k + 1] - (real)fcorr[1] - qi * fy;
    force[3 * i + 2] = fsr[3 * k + 2] - (real)fcorr[2] - qi * fz;
}

// k-vectors whose constants a block of the lanes-per-atom kernels stages in LDS.
constexpr int kKspaceTile = 128;

// Value of lane J of the group of LPA lanes (4 or 16) that this lane belongs to.
template <int LPA, int J>
__device__ __forceinline__ int group_bcast(int v)
{
    // quad_perm (J, J, J, J) or row_newbcast:J
    constexpr int ctrl = LPA == 4 ? J * 0x55 : 0x150 + J;
    return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, true);
}
template <int LPA, int J>
__device__ __forceinline__ float group_bcast(float v)
{
    return __int_as_float(group_bcast<LPA, J>(__float_as_int(v)));
}
template <int LPA, int J>
__device__ __forceinline__ double group_bcast(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = group_bcast<LPA, J>((int)(b & 0xffffffffll)), hi = group_bcast<LPA, J>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The same with LPA lanes per atom, for systems that leave the chip idle at one
// thread per atom: the lanes evaluate the sines and cosines of LPA k-vectors at
// once and then all add the LPA terms in the k-vectors' order (the additions of
// the form above, bit for bit).
template <typename real, int LPA>
__global__ __launch_bounds__(kBlock) void k_kspace_forces_lanes(
    int64_t n, int P, const uint4* __restrict__ sq, const real* __restrict__ q, const int32_t* __restrict__ rank,
    const real* __restrict__ fsr, const int4* __restrict__ kvec, const KForce<real>* __restrict__ kf,
    const double* __restrict__ fcorr, real* __restrict__ force)
{
    __shared__ int4 km[kKspaceTile];
    __shared__ KForce<real> kc[kKspaceTile];
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = min(t / LPA, n - 1);
    const int ln = (int)(threadIdx.x % LPA);
    const uint4 s = sq[i];
    real fx = 0, fy = 0, fz = 0;
    for (int l0 = 0; l0 < P; l0 += kKspaceTile) {
        const int cnt = min(kKspaceTile, P - l0);
        __syncthreads();
        for (int l = threadIdx.x; l < kKspaceTile; l += kBlock) {
            // (terms past the last k-vector are exact zeros)
            km[l] = l < cnt ? kvec[l0 + l] : make_int4(0, 0, 0, 0);
            kc[l] = l < cnt ? kf[l0 + l] : KForce<real>{};
        }
        __syncthreads();
        for (int l = 0; l < cnt; l += LPA) {
            real sn, cs;
            const int4 m = km[l + ln];
            Math<real>::sincos_rev(phase_rev<real>(m.x, m.y, m.z, s.x, s.y, s.z), &sn, &cs);
            const real g = cs * kc[l + ln].a - sn * kc[l + ln].b;
            auto add = [&](auto j) {
                constexpr int J = decltype(j)::value;
                const real gj = group_bcast<LPA, J>(g);
                fx += gj * kc[l + J].kx;
                fy += gj * kc[l + J].ky;
                fz += gj * kc[l + J].kz;
            };
            add(std::integral_constant<int, 0>{});
            add(std::integral_constant<int, 1>{});
            add(std::integral_constant<int, 2>{});
            add(std::integral_constant<int, 3>{});
            if constexpr (LPA == 16) {
                add(std::integral_constant<int, 4>{});
                add(std::integral_constant<int, 5>{});
                add(std::integral_constant<int, 6>{});
                add(std::integral_constant<int, 7>{});
                add(std::integral_constant<int, 8>{});
                add(std::integral_constant<int, 9>{});
                add(std::integral_constant<int, 10>{});
                add(std::integral_constant<int, 11>{});
                add(std::integral_constant<int, 12>{});
                add(std::integral_constant<int, 13>{});
                add(std::integral_constant<int, 14>{});
                add(std::integral_constant<int, 15>{});
            }
        }
    }
    if (ln != 0 || t / LPA >= n) return;
    const real qi = q[i];
    const int64_t k = rank[i];
    force[3 * i + 0] = fsr[3 * k + 0] - (real)fcorr[0] - qi * fx;
    force[3 * i + 1] = fsr[3 * k + 1] - (real)fcorr[1] - qi * fy;
    force[3 * i + 2] = fsr[3 * k + 2] - (real)fcorr[2] - qi * fz;
}

// Lanes per atom of the k-space kernels: one while that gives the chip its waves
// (131,072 atoms: two waves on each of 1,024 SIMDs), four below, sixteen for the
// smallest systems. One against several lanes, forces, p = 200: 45 -> 28 us at
// 98,304 atoms (4), 43 -> 7.1 us at 2,703 atoms (16); FP64, p = 100, 98,304 atoms:
// 48 -> 27 us. The several lanes repeat the additions, so a full chip loses by them: p = 100,
// 1, 4 and 16 lanes, 2,700 atoms 26.8, 7.3, 7.1 us; 8,000: 26.9, 7.4, 9.1; 16,384: 26.6, 7.6,
// 13.0; 131,072: 25.0, 21.6, 65.9; 262,144: 26.5, 37.5, 125 (equal times of 4 and 16 at about
// 4,000 atoms, of 1 and 4 at about 180,000, for any p from 50 to 600).
static int kspace_lanes(const irbe_ctx* h)
{
    const int64_t n = h->cfg.n_atoms;
    return n >= 131072 ? 1 : (n >= 16384 ? 4 : 16);
}

template <typename real>
static hipError_t launch_kspace_forces_t(irbe_ctx* h, void* force)
{
    const int64_t n = h->cfg.n_atoms;
    const int lpa = kspace_lanes(h);
    const unsigned nb = (unsigned)blocks_for(n * lpa, kBlock);
#define IRBE_KSPACE_ARGS                                                                                             \
    n, h->cfg.p_kspace, h->sq, (const real*)h->q_orig, h->rank, (const real*)h->fsr, h->kvec,                        \
        (const KForce<real>*)h->kforce, h->fcorr, (real*)force
    if (lpa == 1) k_kspace_forces<real><<<nb, kBlock, 0, h->stream>>>(IRBE_KSPACE_ARGS);
    else if (lpa == 4) k_kspace_forces_lanes<real, 4><<<nb, kBlock, 0, h->stream>>>(IRBE_KSPACE_ARGS);
    else k_kspace_forces_lanes<real, 16><<<nb, kBlock, 0, h->stream>>>(IRBE_KSPACE_ARGS);
#undef IRBE_KSPACE_ARGS
    return hipGetLastError();
}

hipError_t launch_kspace_forces(irbe_ctx* h, void* force)
{
    return h->fp64 ? launch_kspace_forces_t<double>(h, force) : launch_kspace_forces_t<float>(h, force);
}

// ev[0..10] = U_coul, U_lj, U_long, U_self, U_excl, W_xx, W_yy, W_zz, W_xy, W_xz, W_yz.
// U_long* = sum_l (c_l / 2) |rho_l|^2 (c_l carries ke (S/p) 4 pi/(V k^2)); its
// virial U_l (delta_ab - 2 k_a k_b (1/k^2 + 1/(4 alpha))).
__global__ __launch_bounds__(kReduceBlock) void k_energy_finalize(int P, const double* __restrict__ kcoef,
                                                                  const double* __restrict__ rho,
                                                                  const double* __restrict__ ev_pair,
                                                                  const double* __restrict__ sumq2, double self_coef,
                                                                  double inv_4alpha, double* __restrict__ ev)
{
    __shared__ double lds[7 * (kReduceBlock / 64)];
    double vals[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int l = threadIdx.x; l < P; l += kReduceBlock) {
        const double kx = kcoef[4 * l], ky = kcoef[4 * l + 1], kz = kcoef[4 * l + 2], c = kcoef[4 * l + 3];
        const double k2 = kx * kx + ky * ky + kz * kz;
        const double u = 0.5 * c * (rho[2 * l] * rho[2 * l] + rho[2 * l + 1] * rho[2 * l + 1]);
        const double g = 2.0 * (1.0 / k2 + inv_4alpha);
        vals[0] += u;
        vals[1] += u * (1.0 - g * kx * kx);
        vals[2] += u * (1.0 - g * ky * ky);
        vals[3] += u * (1.0 - g * kz * kz);
        vals[4] += -u * g * kx * ky;
        vals[5] += -u * g * kx * kz;
        vals[6] += -u * g * ky * kz;
    }
    double out;
    block_sum_vec<7, kReduceBlock>(vals, lds, threadIdx.x, out);
    __shared__ double tot[7];
    if (threadIdx.x < 7) tot[threadIdx.x] = out;
    __syncthreads();
    if (threadIdx.x == 0) {
        ev[0] = ev_pair[3];
        ev[1] = ev_pair[4];
        ev[2] = tot[0];
        ev[3] = self_coef * sumq2[0];
        ev[4] = ev_pair[5];
        for (int c = 0; c < 6; ++c) ev[5 + c] = ev_pair[6 + c] + tot[1 + c];
    }
}

hipError_t launch_energy_finalize(irbe_ctx* h, double* ev)
{
    const double beta = h->cfg.ewald_beta;
    const double self_coef = -h->cfg.coulomb_k * beta / 1.7724538509055160273;
    k_energy_finalize<<<1, kReduceBlock, 0, h->stream>>>(h->cfg.p_kspace, h->kcoef, h->rho, h->ev_pair, h->sumq2,
                                                         self_coef, 1.0 / (4.0 * beta * beta), ev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Backward.
// ---------------------------------------------------------------------------

// dL/dF into cell order, and per-block FP64 sums for mean(G).
template <typename real>
__global__ __launch_bounds__(kBlock) void k_gather_grad(int64_t n, const int32_t* __restrict__ perm,
                                                        const real* __restrict__ G, real* __restrict__ gs,
                                                        double* __restrict__ part)
{
    __shared__ double lds[3 * (kBlock / 64)];
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double vals[3] = {0, 0, 0};
    if (k < n) {
        const int64_t i = perm[k];
        const real gx = G[3 * i], gy = G[3 * i + 1], gz = G[3 * i + 2];
        gs[3 * k] = gx;
        gs[3 * k + 1] = gy;
        gs[3 * k + 2] = gz;
        vals[0] = (double)gx;
        vals[1] = (double)gy;
        vals[2] = (double)gz;
    }
    double out;
    block_sum_vec<3, kBlock>(vals, lds, threadIdx.x, out);
    if (threadIdx.x < 3) part[blockIdx.x * 3 + threadIdx.x] = out;
}

__global__ __launch_bounds__(kReduceBlock) void k_mean3(int64_t nb, const double* __restrict__ part, int64_t n,
                                                        double* __restrict__ mean)
{
    __shared__ double lds[3 * (kReduceBlock / 64)];
    double vals[3] = {0, 0, 0};
    for (int64_t b = threadIdx.x; b < nb; b += kReduceBlock)
        for (int c = 0; c < 3; ++c) vals[c] += part[b * 3 + c];
    double out;
    block_sum_vec<3, kReduceBlock>(vals, lds, threadIdx.x, out);
    if (threadIdx.x < 3) mean[threadIdx.x] = out / (double)n;
}

hipError_t launch_gather_grad(irbe_ctx* h, const void* grad)
{
    const int64_t n = h->cfg.n_atoms;
    const int64_t nb = blocks_for(n, kBlock);
    if (h->fp64)
        k_gather_grad<double><<<(unsigned)nb, kBlock, 0, h->stream>>>(n, h->perm, (const double*)grad, (double*)h->gs,
                                                                      h->gpart);
    else
        k_gather_grad<float><<<(unsigned)nb, kBlock, 0, h->stream>>>(n, h->perm, (const float*)grad, (float*)h->gs,
                                                                     h->gpart);
    k_mean3<<<1, kReduceBlock, 0, h->stream>>>(nb, h->gpart, n, h->gmean);
    return hipGetLastError();
}

// Per atom (caller order): the k-space adjoint plus the short-range parts.
//   dL/dr_n = -ke q_n sum_l c_l k_l [Re(e^{i th} conj A_l) - g_nl Re(e^{-i th} rho_l)]
//   dL/dq_n = -ke sum_l c_l [Im(e^{i th} conj A_l) + g_nl Im(e^{-i th} rho_l)]
// LPA lanes per atom (1, 4 or 16) take every LPA-th k-vector; their sums are then
// added in the group.
template <typename real, int LPA>
__global__ __launch_bounds__(kBlock) void k_kspace_adjoint(int64_t n, int P, const uint4* __restrict__ sq,
                                                           const real* __restrict__ q, const real* __restrict__ G,
                                                           const int32_t* __restrict__ rank,
                                                           const int4* __restrict__ kvec,
                                                           const KAdj<real>* __restrict__ ka,
                                                           const real* __restrict__ gself,
                                                           const real* __restrict__ gscat,
                                                           const real* __restrict__ gqself,
                                                           const real* __restrict__ gqscat, real* __restrict__ gpos,
                                                           real* __restrict__ gq)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (LPA == 1 && t >= n) return;
    const int64_t i = LPA == 1 ? t : min(t / LPA, n - 1);
    const int ln = LPA == 1 ? 0 : (int)(threadIdx.x % LPA);
    const uint4 s = sq[i];
    const real gx = G[3 * i], gy = G[3 * i + 1], gz = G[3 * i + 2];
    real px = 0, py = 0, pz = 0, pq = 0;
#pragma unroll LPA > 1 ? 4 : 1
    for (int l = ln; l < P; l += LPA) {
        const int4 m = kvec[l];
        const KAdj<real> c = ka[l];
        real sn, cs;
        Math<real>::sincos_rev(phase_rev<real>(m.x, m.y, m.z, s.x, s.y, s.z), &sn, &cs);
        const real g = gx * c.kx + gy * c.ky + gz * c.kz;
        const real eA_re = cs * c.ar + sn * c.ai;
        const real eA_im = sn * c.ar - cs * c.ai;
        const real er_re = cs * c.rr + sn * c.ri;
        const real er_im = cs * c.ri - sn * c.rr;
        const real tt = eA_re - g * er_re;
        px += tt * c.kx;
        py += tt * c.ky;
        pz += tt * c.kz;
        pq += eA_im + g * er_im;
    }
    auto group_sum = [](real v) {
        if (LPA == 16) {
            v = butterfly_add<8>(v);
            v = butterfly_add<4>(v);
        }
        if (LPA >= 4) {
            v = butterfly_add<2>(v);
            v = butterfly_add<1>(v);
        }
        return v;
    };
    px = group_sum(px);
    py = group_sum(py);
    pz = group_sum(pz);
    pq = group_sum(pq);
    if (LPA > 1 && (ln != 0 || t / LPA >= n)) return;
    const real qi = q[i];
    const int64_t k = rank[i];
    gpos[3 * i + 0] = gself[3 * k + 0] + gscat[3 * k + 0] - qi * px;
    gpos[3 * i + 1] = gself[3 * k + 1] + gscat[3 * k + 1] - qi * py;
    gpos[3 * i + 2] = gself[3 * k + 2] + gscat[3 * k + 2] - qi * pz;
    if (gq) gq[i] = gqself[k] + gqscat[k] - pq;
}

// LJ table gradients: fixed-order two-stage sum of the per-block partials
// (slices of contiguous blocks, then the slices).
constexpr int kLjSlices = 256;
constexpr int64_t kLjDirect = 2 * kReduceBlock;

__global__ __launch_bounds__(kReduceBlock) void k_lj_reduce1(int64_t nb, const double* __restrict__ part,
                                                             double* __restrict__ slices)
{
    constexpr int NLJ = 2 * kMaxTypesGrad * kMaxTypesGrad;
    __shared__ double lds[NLJ * (kReduceBlock / 64)];
    const int64_t per = (nb + kLjSlices - 1) / kLjSlices;
    const int64_t b0 = blockIdx.x * per, b1 = min(nb, b0 + per);
    double vals[NLJ];
    for (int v = 0; v < NLJ; ++v) vals[v] = 0.0;
    for (int64_t b = b0 + threadIdx.x; b < b1; b += kReduceBlock)
        for (int v = 0; v < NLJ; ++v) vals[v] += part[b * NLJ + v];
    double o;
    block_sum_vec<NLJ, kReduceBlock>(vals, lds, threadIdx.x, o);
    if (threadIdx.x < NLJ) slices[blockIdx.x * NLJ + threadIdx.x] = o;
}

__global__ __launch_bounds__(kReduceBlock) void k_lj_reduce2(int n_slices, const double* __restrict__ slices,
                                                             int n_types, double* __restrict__ out)
{
    constexpr int NLJ = 2 * kMaxTypesGrad * kMaxTypesGrad;
    __shared__ double lds[NLJ * (kReduceBlock / 64)];
    double vals[NLJ];
    for (int v = 0; v < NLJ; ++v) vals[v] = 0.0;
    for (int b = threadIdx.x; b < n_slices; b += kReduceBlock)
        for (int v = 0; v < NLJ; ++v) vals[v] += slices[b * NLJ + v];
    double o;
    block_sum_vec<NLJ, kReduceBlock>(vals, lds, threadIdx.x, o);
    if (threadIdx.x < NLJ) {
        const int half = kMaxTypesGrad * kMaxTypesGrad;
        const int which = threadIdx.x / half;  // 0 sigma, 1 eps
        const int e = threadIdx.x % half;
        const int a = e / kMaxTypesGrad, t = e % kMaxTypesGrad;
        if (a < n_types && t < n_types) out[which * n_types * n_types + a * n_types + t] = o;
    }
}

template <typename real>
static hipError_t launch_kspace_adjoint_t(irbe_ctx* h, const void* grad, void* grad_pos, void* grad_q)
{
    const int64_t n = h->cfg.n_atoms;
    const int lpa = kspace_lanes(h);
    const unsigned nb = (unsigned)blocks_for(n * lpa, kBlock);
#define IRBE_KADJ_ARGS                                                                                              \
    n, h->cfg.p_kspace, h->sq, (const real*)h->q_orig, (const real*)grad, h->rank, h->kvec,                          \
        (const KAdj<real>*)h->kadj, (const real*)h->gself, (const real*)h->gscat, (const real*)h->gqself,            \
        (const real*)h->gqscat, (real*)grad_pos, (real*)grad_q
    if (lpa == 1) k_kspace_adjoint<real, 1><<<nb, kBlock, 0, h->stream>>>(IRBE_KADJ_ARGS);
    else if (lpa == 4) k_kspace_adjoint<real, 4><<<nb, kBlock, 0, h->stream>>>(IRBE_KADJ_ARGS);
    else k_kspace_adjoint<real, 16><<<nb, kBlock, 0, h->stream>>>(IRBE_KADJ_ARGS);
#undef IRBE_KADJ_ARGS
    return hipGetLastError();
}

hipError_t launch_kspace_adjoint(irbe_ctx* h, const void* grad, void* grad_pos, void* grad_q, double* grad_lj)
{
    const hipError_t e = h->fp64 ? launch_kspace_adjoint_t<double>(h, grad, grad_pos, grad_q)
                                 : launch_kspace_adjoint_t<float>(h, grad, grad_pos, grad_q);
    if (e != hipSuccess || !grad_lj) return e;
    if (h->adj_nb <= kLjDirect) {
        // few blocks: summed in one launch, as slices of one block each
        k_lj_reduce2<<<1, kReduceBlock, 0, h->stream>>>((int)h->adj_nb, h->ljpart, h->cfg.n_types, grad_lj);
        return hipGetLastError();
    }
    k_lj_reduce1<<<kLjSlices, kReduceBlock, 0, h->stream>>>(h->adj_nb, h->ljpart, h->lj_slices);
    k_lj_reduce2<<<1, kReduceBlock, 0, h->stream>>>(kLjSlices, h->lj_slices, h->cfg.n_types, grad_lj);
    return hipGetLastError();
}

}  // namespace irbe
