// Device kernels of liblf for gfx950 (CDNA4): initialisation, the FP64
// scale-factor update, reductions, energies and field export.  The fused
// kick-drift sweep lives in lf_sweep.hip.
//
// Equation references: Sainio, "CUDAEASY", arXiv:0911.5692, Sec. II.B.
#include "lf_internal.h"
#include "lf_scale.h"

#include <math.h>

namespace lf {

// ---------------------------------------------------------------- helpers

// Sum NV per-thread doubles over the block in a fixed order (wave butterfly,
// then waves in index order) and store the NV totals at out.  Deterministic.
template <int NV>
__device__ inline void block_sum_store(double (&v)[NV], double *out)
{
    __shared__ double sm[NV][16];
    const int t = threadIdx.x + threadIdx.y * blockDim.x;
    const int nthreads = blockDim.x * blockDim.y;
    const int lane = t & 63, wave = t >> 6, nw = (nthreads + 63) >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        v[i] = wave_sum(v[i]);
    }
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) sm[i][wave] = v[i];
    }
    __syncthreads();
    if (t < NV) {
        double s = 0.0;
        for (int w = 0; w < nw; ++w) s += sm[t][w];
        out[t] = s;
    }
}

// Stage 2 of every reduction: one block of kStage2Threads sums nblk rows of
// nv partials in a fixed order.  Result in `tot` (valid in thread 0 after the
// call; all threads see it through shared memory).
template <int NV>
__device__ inline void stage2_sum(const double *part, int nblk, double (&tot)[NV])
{
    __shared__ double res[NV];
    double acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.0;
    for (int j = threadIdx.x; j < nblk; j += blockDim.x) {
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] += part[(size_t)j * NV + i];
    }
    block_sum_store<NV>(acc, res);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) tot[i] = res[i];
}

// ---------------------------------------------------------------- init

// Moments of an input state (element type Tin), FP64 per site:
//  0,1: sum f_i   2,3: sum u_i   4,5: sum u_i^2
//  6,7: raw gradient sum of f_i (grad_raw<ST>: no 1/dx^2, no stencil weight)
//  8: sum f1^beta   9: sum f1^2 f2^2
template <typename Tin, int ST>
__global__ void __launch_bounds__(256) k_input_moments(const Tin *__restrict__ f1, const Tin *__restrict__ f2,
                                                       const Tin *__restrict__ u1, const Tin *__restrict__ u2,
                                                       int N, int beta, double *part)
{
    const int64_t N3 = (int64_t)N * N * N;
    double acc[kNMom];
#pragma unroll
    for (int i = 0; i < kNMom; ++i) acc[i] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (int64_t)gridDim.x * blockDim.x) {
        const Wrap w(i, N);
        const double a = (double)f1[i], b = (double)f2[i];
        const double p = (double)u1[i], q = (double)u2[i];
        acc[0] += a; acc[1] += b; acc[2] += p; acc[3] += q;
        acc[4] += p * p; acc[5] += q * q;
        acc[6] += grad_raw<ST>([&](int dx, int dy, int dz) { return (double)f1[w(dx, dy, dz)]; }, a);
        acc[7] += grad_raw<ST>([&](int dx, int dy, int dz) { return (double)f2[w(dx, dy, dz)]; }, b);
        acc[8] += ipow_d(a, beta);
        acc[9] += a * a * b * b;
    }
    block_sum_store<kNMom>(acc, part + (size_t)blockIdx.x * kNMom);
}

// Background, scale factor and (physical = 1) the Friedmann a'_0 of the
// initial state (Sec. II.B: conversion to program units, desynchronisation).
__global__ void __launch_bounds__(kStage2Threads) k_init_scalars(const double *part, int nblk,
                                                                 const DevParams *__restrict__ P,
                                                                 DevScalars *S, int physical,
                                                                 double a0, double ad0)
{
    double m[kNMom];
    stage2_sum<kNMom>(part, nblk, m);
    if (threadIdx.x >= 64) return;  // one wave, every lane alike; lane 0 writes
    const double N3 = P->N3, r = P->r, s = P->s;
    const double mf1 = m[0] / N3, mf2 = m[1] / N3, mu1 = m[2] / N3, mu2 = m[3] / N3;
    double conv = 0.0;
    unsigned int bad = 0;
    for (int i = 0; i < kNMom; ++i) bad |= !isfinite(m[i]);
    if (physical) {
        // a'^2 = (kappa^2/3) a^(2-2r) rho_pr with physical velocities u
        const double rho = (0.5 * (m[4] + m[5])
                            + 0.5 * pow(a0, -2.0 * s - 2.0) * P->gw * (m[6] + m[7]) / (P->dx * P->dx)
                            + P->c1 * pow(a0, P->p1) * m[8] / (double)P->beta
                            + 0.5 * P->G * pow(a0, P->p2) * m[9]) / N3;
        const double q = (P->kappa2 / 3.0) * pow(a0, 2.0 - 2.0 * r) * rho;
        bad |= !(q >= 0.0);
        ad0 = sqrt(q);
        conv = r * ad0 / a0;
    }
    const double vb1 = mu1 + conv * mf1, vb2 = mu2 + conv * mf2;
    const double h = 0.5 * P->dt;
    const double pw = scale_power(threadIdx.x, P, a0 + h * ad0);
    if (threadIdx.x < kNPow) S->pw[threadIdx.x] = pw;
    if (threadIdx.x != 0) return;
    S->mean_f[0] = mf1; S->mean_f[1] = mf2;
    S->mean_u[0] = mu1; S->mean_u[1] = mu2;
    S->conv = conv;
    S->ad0 = ad0;
    S->bg_f[0] = mf1 + h * vb1;
    S->bg_f[1] = mf2 + h * vb2;
    S->bg_v[0] = vb1;
    S->bg_v[1] = vb2;
    S->a_half = a0 + h * ad0;
    S->ad = ad0;
    S->step = 0;
    S->status = bad;
}

// Deviations from the background at tau = 0, desynchronised by dt/2:
//   e = (u - u_bar) + conv (f - f_bar),  d = (f - f_bar) + dt/2 e.
template <typename T, typename Tin>
__global__ void __launch_bounds__(256) k_init_fields(const Tin *__restrict__ f1, const Tin *__restrict__ f2,
                                                     const Tin *__restrict__ u1, const Tin *__restrict__ u2,
                                                     T *d1, T *d2, T *e1, T *e2, int N,
                                                     const DevParams *__restrict__ P,
                                                     const DevScalars *__restrict__ S)
{
    const int64_t N3 = (int64_t)N * N * N;
    const double h = 0.5 * P->dt, conv = S->conv;
    const double mf1 = S->mean_f[0], mf2 = S->mean_f[1], mu1 = S->mean_u[0], mu2 = S->mean_u[1];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double a = (double)f1[i] - mf1, b = (double)f2[i] - mf2;
        const double p = ((double)u1[i] - mu1) + conv * a;
        const double q = ((double)u2[i] - mu2) + conv * b;
        d1[i] = (T)(a + h * p);
        d2[i] = (T)(b + h * q);
        e1[i] = (T)p;
        e2[i] = (T)q;
    }
}

// ---------------------------------------------------------------- reductions

// Sums over the stored fields that the next scale-factor update needs
// (eq. scale): the raw gradient sums of f_i (grad_raw<ST>), sum f1^beta and
// sum f1^2 f2^2 with f = f_bar + d evaluated in FP64.
template <typename T, int ST>
__global__ void __launch_bounds__(256) k_reduce(const T *__restrict__ d1, const T *__restrict__ d2, int N,
                                                const double *__restrict__ bg_f, int beta, double *part)
{
    const int64_t N3 = (int64_t)N * N * N;
    const double g1 = bg_f[0], g2 = bg_f[1];
    double acc[kNPart] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (int64_t)gridDim.x * blockDim.x) {
        const Wrap w(i, N);
        const double a = (double)d1[i], b = (double)d2[i];
        acc[0] += grad_raw<ST>([&](int dx, int dy, int dz) { return (double)d1[w(dx, dy, dz)]; }, a);
        acc[1] += grad_raw<ST>([&](int dx, int dy, int dz) { return (double)d2[w(dx, dy, dz)]; }, b);
        const double x1 = g1 + a, x2 = g2 + b;
        acc[2] += ipow_d(x1, beta);
        acc[3] += x1 * x1 * x2 * x2;
    }
    block_sum_store<kNPart>(acc, part + (size_t)blockIdx.x * kNPart);
}

__global__ void __launch_bounds__(kStage2Threads) k_sum_partials4(const double *part, int nblk, double *out)
{
    double t[kNPart];
    stage2_sum<kNPart>(part, nblk, t);
    if (threadIdx.x < kNPart) out[threadIdx.x] = t[threadIdx.x];
}

// Install checkpointed totals as the pending partials: row 0 holds the
// totals, the other rows zero, so the fixed-order stage 2 returns them
// bitwise.
__global__ void k_set_pending(double *part, int nblk, const double *tot)
{
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < nblk * kNPart;
         j += gridDim.x * blockDim.x)
        part[j] = (j < kNPart) ? tot[j] : 0.0;
}

// ---------------------------------------------------------------- a-update

// One step of the scale factor and the homogeneous mode, and the coefficients
// of the fused kick-drift (lf_scale.h), by one block.  The sweeps of a lone
// lattice do this in their own blocks (CoefsOfStep in lf_sweep_common.h); this
// is for launch shapes with many partial rows, the plain sweep and ensembles.
__device__ void aupdate_block(const double *part, int nblk, const DevParams *__restrict__ P, const DevScalars *S,
                              DevScalars *So, CoefPair *C, DevScalars *tape)
{
    double t[kNPart];
    stage2_sum<kNPart>(part, nblk, t);
    if (threadIdx.x >= 64) return;
    const int beta = P->beta;
    ScaleStep o;
    scale_step(t, ScaleIn(P, S), beta, o);
    if (threadIdx.x == 0) scale_commit(t, o, P, S, So, C, tape, beta);
    scale_commit_powers(o.an, P, So);
}

__global__ void __launch_bounds__(kStage2Threads) k_aupdate(const double *part, int nblk,
                                                            const DevParams *__restrict__ P,
                                                            const DevScalars *S, DevScalars *So, CoefPair *C,
                                                            DevScalars *tape)
{
    aupdate_block(part, nblk, P, S, So, C, tape);
}

__global__ void __launch_bounds__(64) k_set_powers(const DevParams *__restrict__ P, DevScalars *S)
{
    const double pw = scale_power(threadIdx.x, P, S->a_half);
    if (threadIdx.x < kNPow) S->pw[threadIdx.x] = pw;
}

// Ensemble: block r updates realization r.
__global__ void __launch_bounds__(kStage2Threads) k_aupdate_ens(const EnsEntry *tab, int *queue, int parity)
{
    // the sweep that follows takes its work items from these counters (one
    // per XCD, 32 ints apart)
    if (blockIdx.x == 0 && threadIdx.x < 8)
        __hip_atomic_store(queue + 32 * threadIdx.x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const EnsEntry &e = tab[blockIdx.x];
    aupdate_block(e.part[parity], e.rows, e.P, e.S[parity], e.S[parity ^ 1], e.Cw, nullptr);
}

// ---------------------------------------------------------------- energies

// Both diagnostics below need, per site at the synchronised time k, the
// synchronised deviations s_i = d_i(k+1/2) - (dt/2) e_i(k) at the site and at
// its forward neighbours (+x, +y, +z for the 7-point gradient; the 13 forward
// bonds of the 27-point Dirichlet form, which reach x-1..x+1, y-1..y+1 and
// z..z+1), and the velocity deviation e_i(k) at the site.
//
// k_diag_march: a block owns a 64 x 4 KI column tile and marches z over a
// chunk; each thread holds KI sites of a column (rows ly, ly + 4, ...): two
// for the 7-point stencil (energies 14% and rho/p 4% faster at 512^3 than
// one), one for the 27-point stencil, whose wider ring and 13 bonds per site
// made two (and four) slower.
// The s values of planes z and z+1 sit in LDS with a one-cell ring (three
// buffers, one barrier per plane); plane z+2 is loaded into registers while
// plane z is evaluated.  Each array element is read from HBM about once,
// plus the ring (mostly L2 hits) and one plane per chunk, instead of once per
// neighbour.  The grid walks a static list of (tile, chunk) items, so any N
// fits a fixed number of partial rows; per-site arithmetic is FP64 and the
// block sums are deterministic.
constexpr int kDiagX = 64, kDiagLW = kDiagX + 2;  // tile width; LDS row with its ring
template <int ST>
constexpr int diag_ki() { return ST == 27 ? 1 : 2; }
template <int ST>
constexpr int diag_y() { return 4 * diag_ki<ST>(); }  // tile rows

// ring cells a plane needs beyond the tile: 7 points, the +x column and the
// +y row; 27 points, the whole ring
template <int ST>
constexpr int diag_ring() { return ST == 27 ? 2 * kDiagLW + 2 * diag_y<ST>() : kDiagX + diag_y<ST>(); }
static_assert(diag_ring<7>() <= 256 && diag_ring<27>() <= 256, "the ring fits one cell per thread");

template <int ST>
__device__ inline void diag_ring_cell(int c, int &lx, int &ly)
{
    constexpr int DY = diag_y<ST>();
    if (ST == 27) {
        if (c < kDiagLW) { lx = c - 1; ly = -1; }
        else if (c < 2 * kDiagLW) { lx = c - kDiagLW - 1; ly = DY; }
        else if (c < 2 * kDiagLW + DY) { lx = -1; ly = c - 2 * kDiagLW; }
        else { lx = kDiagX; ly = c - 2 * kDiagLW - DY; }
    } else {
        if (c < DY) { lx = kDiagX; ly = c; }
        else { lx = c - DY; ly = DY; }
    }
}

// MODE 0: the energy sums of k_energy_final (kNEn per block row):
//  0,1: sum (v_i - r (a'/a) f_i)^2   2,3: raw gradient sums of f_i
//  4: sum f1^beta   5: sum f1^2 f2^2
// MODE 1: energy density and pressure per site (eq. rho-pres in program
// units): rho = sum_i K_i + G_i + V_pr, p = sum_i K_i - G_i/3 - V_pr,
// K_i = (v_i - r (a'/a) f_i)^2/2, G_i = a^(-2s-2) grad2(f_i)/2 with grad2 the
// stencil's gradient energy density; rho, p may be NULL.  Sums: rho, p.
// bid, nb: this block's index among the nb that share the items.
template <typename T, int ST, int MODE, typename To>
__device__ __forceinline__ void diag_march(const T *__restrict__ d1, const T *__restrict__ d2,
                                           const T *__restrict__ e1, const T *__restrict__ e2, int N, int zchunk,
                                           int ntx, int nty, int nitems, const DevParams *__restrict__ P,
                                           const DevScalars *__restrict__ S, To *__restrict__ rho,
                                           To *__restrict__ pr, double *__restrict__ part, const int bid,
                                           const int nb)
{
    constexpr int NV = MODE == 0 ? kNEn : 2;
    constexpr int NR = diag_ring<ST>();
    constexpr int KI = diag_ki<ST>(), DY = diag_y<ST>();
    constexpr int PL = kDiagLW * (DY + 2);
    __shared__ double sv[3][2][PL];  // [buffer][field][plane with ring]

    const double h = 0.5 * P->dt, r = P->r, sx = P->s;
    const double ak = S->a_half - h * S->ad, hub = S->ad / ak;
    const double gs1 = S->bg_f[0] - h * S->bg_v[0], gs2 = S->bg_f[1] - h * S->bg_v[1];
    const double vb1 = S->bg_v[0], vb2 = S->bg_v[1];
    const double gfac = 0.5 * pow(ak, -2.0 * sx - 2.0) * P->gw / (P->dx * P->dx);
    const double cv1 = P->c1 * pow(ak, P->p1) / (double)P->beta, cv2 = 0.5 * P->G * pow(ak, P->p2);
    const int beta = P->beta;
    const int64_t NN = (int64_t)N * N;

    const int t = threadIdx.x, lx = t & 63, ly0 = t >> 6;
    int slot[KI];
#pragma unroll
    for (int k = 0; k < KI; ++k) slot[k] = (ly0 + 4 * k + 1) * kDiagLW + lx + 1;
    const bool hasr = t < NR;
    int rx = 0, ry = 0;
    if (hasr) diag_ring_cell<ST>(t, rx, ry);
    const int rslot = (ry + 1) * kDiagLW + rx + 1;
    auto wrap = [N](int v) { return ((v % N) + N) % N; };
    auto plane = [&](const T *a, int z) { return a + (int64_t)(z >= N ? z - N : z) * NN; };

    double acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.0;

    for (int base = 0; base + bid < nitems; base += nb) {
        // energies: XCD-contiguous tiles share their ring rows in L2 (3% faster
        // at 512^3); rho/p, which also streams two output arrays, runs 7%
        // faster in the plain order
        const int item = MODE == 0 ? xcd_item(base, nitems, bid, nb) : base + bid;
        const int tx = item % ntx, rest = item / ntx, ty = rest % nty, tz = rest / nty;
        const int x0 = tx * kDiagX, y0 = ty * DY, z0 = tz * zchunk;
        const int z1 = min(z0 + zchunk, N);
        // in-plane offsets, wrapped (inactive lanes hold the periodic images
        // their active neighbours need)
        bool act[KI];
        int off[KI];
#pragma unroll
        for (int k = 0; k < KI; ++k) {
            act[k] = (x0 + lx < N) && (y0 + ly0 + 4 * k < N);
            off[k] = wrap(y0 + ly0 + 4 * k) * N + wrap(x0 + lx);
        }
        const int roff = wrap(y0 + ry) * N + wrap(x0 + rx);

        // registers of the plane in flight: the thread's sites and ring cell, 4 arrays
        T rd1[KI], rd2[KI], re1[KI], re2[KI], hd1 = 0, hd2 = 0, he1 = 0, he2 = 0;
        auto load = [&](int z) {
            const T *a1 = plane(d1, z), *a2 = plane(d2, z), *b1 = plane(e1, z), *b2 = plane(e2, z);
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                rd1[k] = a1[off[k]]; rd2[k] = a2[off[k]]; re1[k] = b1[off[k]]; re2[k] = b2[off[k]];
            }
            if (hasr) { hd1 = a1[roff]; hd2 = a2[roff]; he1 = b1[roff]; he2 = b2[roff]; }
        };
        auto stage = [&](int b) {
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                sv[b][0][slot[k]] = (double)rd1[k] - h * (double)re1[k];
                sv[b][1][slot[k]] = (double)rd2[k] - h * (double)re2[k];
            }
            if (hasr) {
                sv[b][0][rslot] = (double)hd1 - h * (double)he1;
                sv[b][1][rslot] = (double)hd2 - h * (double)he2;
            }
        };
        // own velocity deviations of planes z and z+1
        double ec1[KI], ec2[KI], en1[KI], en2[KI];
        load(z0);
        stage(0);
#pragma unroll
        for (int k = 0; k < KI; ++k) { ec1[k] = (double)re1[k]; ec2[k] = (double)re2[k]; }
        load(z0 + 1);
        stage(1);
#pragma unroll
        for (int k = 0; k < KI; ++k) { en1[k] = (double)re1[k]; en2[k] = (double)re2[k]; }
        if (z0 + 1 < z1) load(z0 + 2);
        __syncthreads();

        int b0 = 0;
        for (int z = z0; z < z1; ++z) {
            const int b1 = b0 == 2 ? 0 : b0 + 1, b2 = b1 == 2 ? 0 : b1 + 1;
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                if (!act[k]) continue;
                const int sl = slot[k];
                const double *p1 = sv[b0][0], *q1 = sv[b1][0], *p2 = sv[b0][1], *q2 = sv[b1][1];
                auto sy1 = [&](int dx, int dy, int dz) { return (dz ? q1 : p1)[sl + dy * kDiagLW + dx]; };
                auto sy2 = [&](int dx, int dy, int dz) { return (dz ? q2 : p2)[sl + dy * kDiagLW + dx]; };
                const double s1 = p1[sl], s2 = p2[sl];
                const double x1 = gs1 + s1, x2 = gs2 + s2;
                const double u1 = (vb1 + ec1[k]) - r * hub * x1;
                const double u2 = (vb2 + ec2[k]) - r * hub * x2;
                if (MODE == 0) {
                    acc[0] += u1 * u1;
                    acc[1] += u2 * u2;
                    acc[2] += grad_raw<ST>(sy1, s1);
                    acc[3] += grad_raw<ST>(sy2, s2);
                    acc[4] += ipow_d(x1, beta);
                    acc[5] += x1 * x1 * x2 * x2;
                } else {
                    double g = grad_raw<ST>(sy1, s1);
                    g += grad_raw<ST>(sy2, s2);
                    const double K = 0.5 * (u1 * u1 + u2 * u2), Gs = gfac * g;
                    const double V = cv1 * ipow_d(x1, beta) + cv2 * x1 * x1 * x2 * x2;
                    const double rr = K + Gs + V, pp = K - Gs / 3.0 - V;
                    const int64_t i = (int64_t)z * NN + off[k];
                    // streamed once: non-temporal
                    if (rho) __builtin_nontemporal_store((To)rr, rho + i);
                    if (pr) __builtin_nontemporal_store((To)pp, pr + i);
                    acc[0] += rr;
                    acc[1] += pp;
                }
            }
            if (z + 1 < z1) {
                // plane z+2 into the buffer last read for plane z-1
                stage(b2);
#pragma unroll
                for (int k = 0; k < KI; ++k) {
                    ec1[k] = en1[k]; ec2[k] = en2[k];
                    en1[k] = (double)re1[k]; en2[k] = (double)re2[k];
                }
                if (z + 2 < z1) load(z + 3);
            }
            __syncthreads();
            b0 = b1;
        }
    }
    block_sum_store<NV>(acc, part + (size_t)bid * NV);
}

template <typename T, int ST, int MODE, typename To>
__global__ void __launch_bounds__(256) k_diag_march(const T *__restrict__ d1, const T *__restrict__ d2,
                                                    const T *__restrict__ e1, const T *__restrict__ e2, int N,
                                                    int zchunk, int ntx, int nty, int nitems,
                                                    const DevParams *__restrict__ P,
                                                    const DevScalars *__restrict__ S, To *__restrict__ rho,
                                                    To *__restrict__ pr, double *__restrict__ part)
{
    diag_march<T, ST, MODE, To>(d1, d2, e1, e2, N, zchunk, ntx, nty, nitems, P, S, rho, pr, part, blockIdx.x,
                                gridDim.x);
}

// The energies of every realization of an ensemble, block row y one of them:
// one launch and one for the final sums instead of two and a blocking copy
// per realization (15 of 64^3 to 160^3: 0.9 ms a call before).  Blocks and rows
// are those of a lone lattice's energies, so the bits are too.
template <typename T, int ST>
__global__ void __launch_bounds__(256) k_diag_ens(const EnsEntry *__restrict__ tab, const int parity)
{
    const EnsEntry &e = tab[blockIdx.y];
    if ((int)blockIdx.x >= e.dgrid) return;
    const T *const *b = (const T *const *)e.buf[parity];
    diag_march<T, ST, 0, float>(b[0], b[1], b[2], b[3], e.N, e.dchunk, e.dntx, e.dnty, e.ditems, e.P, e.S[parity],
                                nullptr, nullptr, e.enp, blockIdx.x, e.dgrid);
}

// out: step, a, a', a'/a, K1, K2, G1, G2, P, rho, R, status (as double)
__device__ inline void energy_final(const double *part, int nblk, const DevParams *__restrict__ P,
                                    const DevScalars *__restrict__ S, double *out)
{
    double t[kNEn];
    stage2_sum<kNEn>(part, nblk, t);
    if (threadIdx.x != 0) return;
    const double N3 = P->N3, h = 0.5 * P->dt, s = P->s, r = P->r;
    const double ak = S->a_half - h * S->ad, ad = S->ad;
    const double K1 = 0.5 * t[0] / N3, K2 = 0.5 * t[1] / N3;
    const double gf = 0.5 * pow(ak, -2.0 * s - 2.0) * P->gw / (P->dx * P->dx * N3);
    const double G1 = gf * t[2], G2 = gf * t[3];
    const double Pv = (P->c1 * pow(ak, P->p1) * t[4] / (double)P->beta + 0.5 * P->G * pow(ak, P->p2) * t[5]) / N3;
    const double rho = K1 + K2 + G1 + G2 + Pv;
    const double R = (P->kappa2 / 3.0) * pow(ak, 2.0 - 2.0 * r) * rho / (ad * ad) - 1.0;
    unsigned int bad = S->status;
    for (int i = 0; i < kNEn; ++i) bad |= !isfinite(t[i]);
    out[0] = (double)S->step; out[1] = ak; out[2] = ad; out[3] = ad / ak;
    out[4] = K1; out[5] = K2; out[6] = G1; out[7] = G2; out[8] = Pv; out[9] = rho;
    out[10] = (P->kappa2 > 0.0) ? R : 0.0;
    out[11] = (double)bad;
}

__global__ void __launch_bounds__(kStage2Threads) k_energy_final(const double *part, int nblk,
                                                                 const DevParams *__restrict__ P,
                                                                 const DevScalars *__restrict__ S,
                                                                 double *out)
{
    energy_final(part, nblk, P, S, out);
}

__global__ void __launch_bounds__(kStage2Threads) k_energy_final_ens(const EnsEntry *__restrict__ tab, int parity,
                                                                     double *out)
{
    const EnsEntry &e = tab[blockIdx.x];
    energy_final(e.enp, e.dgrid, e.P, e.S[parity], out + (size_t)blockIdx.x * kEnOut);
}

// ---------------------------------------------------------------- rho and p

__global__ void __launch_bounds__(kStage2Threads) k_rho_p_final(const double *part, int nblk,
                                                                const DevParams *__restrict__ P, double *out)
{
    double t[2];
    stage2_sum<2>(part, nblk, t);
    if (threadIdx.x != 0) return;
    out[0] = t[0] / P->N3;
    out[1] = t[1] / P->N3;
    out[2] = out[1] / out[0];
}

// ---------------------------------------------------------------- export

// A block takes kFlat x 256 sites in address order, all of its loads in flight
// at once, and streams the results (non-temporal): FP32 to FP32 at 512^3 785
// us a call against 925 for a grid-stride loop of plain stores (835 with one
// site a thread, 855 with four), at 256^3 104 against 154.  WANT: the outputs
// that are written, bit j for f1, f2, v1, v2; a kernel each, so that arrays no
// output needs are not read and the loads stay unconditional (with conditional
// ones all four outputs took 926 us instead of 723).
constexpr int kFlat = 2;

template <typename T, typename To, int WANT>
__global__ void __launch_bounds__(256) k_get_fields(const T *__restrict__ d1, const T *__restrict__ d2,
                                                    const T *__restrict__ e1, const T *__restrict__ e2,
                                                    To *f1, To *f2, To *v1, To *v2, const int64_t start,
                                                    const int64_t N3, const DevParams *__restrict__ P,
                                                    const DevScalars *__restrict__ S, int sync)
{
    constexpr bool F1 = WANT & 1, F2 = WANT & 2, V1 = WANT & 4, V2 = WANT & 8;
    const double h = sync ? 0.5 * P->dt : 0.0;
    const double g1 = S->bg_f[0] - h * S->bg_v[0], g2 = S->bg_f[1] - h * S->bg_v[1];
    const double vb1 = S->bg_v[0], vb2 = S->bg_v[1];
    const int64_t i0 = start + (int64_t)blockIdx.x * (256 * kFlat) + threadIdx.x;
    T v[kFlat][4];
#pragma unroll
    for (int k = 0; k < kFlat; ++k) {
        const int64_t i = i0 + 256 * k < N3 ? i0 + 256 * k : N3 - 1;
        if constexpr (F1) v[k][0] = d1[i];
        if constexpr (F2) v[k][1] = d2[i];
        if constexpr (F1 || V1) v[k][2] = e1[i];
        if constexpr (F2 || V2) v[k][3] = e2[i];
    }
#pragma unroll
    for (int k = 0; k < kFlat; ++k) {
        const int64_t i = i0 + 256 * k;
        if (i >= N3) break;
        if constexpr (F1) __builtin_nontemporal_store((To)(g1 + ((double)v[k][0] - h * (double)v[k][2])), f1 + i);
        if constexpr (F2) __builtin_nontemporal_store((To)(g2 + ((double)v[k][1] - h * (double)v[k][3])), f2 + i);
        if constexpr (V1) __builtin_nontemporal_store((To)(vb1 + (double)v[k][2]), v1 + i);
        if constexpr (V2) __builtin_nontemporal_store((To)(vb2 + (double)v[k][3]), v2 + i);
    }
}

// Synchronised deviation from the background of one field, FP64:
// d(k) = d(k+1/2) - h e(k) (h = dt/2) for a field, e(k) for a velocity.
template <typename T>
__global__ void __launch_bounds__(256) k_sync_deviation(const T *__restrict__ d, const T *__restrict__ e,
                                                        double *out, int64_t N3, double h, int velocity)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = velocity ? (double)e[i] : (double)d[i] - h * (double)e[i];
}

static int grid_for(int64_t n, int per_block, int cap)
{
    int64_t g = (n + per_block - 1) / per_block;
    return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

// ---------------------------------------------------------------- synthetic state

// A deterministic small-amplitude state for timing runs (autotuner): hash
// noise of amplitude 1e-4 around f_bar = (1, 0), v_bar = (0, 0), a = 1, a' = 1/2.
__device__ inline double hash01(uint64_t x)
{
    x ^= x >> 33; x *= 0xff51afd7ed558ccdULL; x ^= x >> 33; x *= 0xc4ceb9fe1a85ec53ULL; x ^= x >> 33;
    return (double)(x >> 11) * (1.0 / 9007199254740992.0) - 0.5;
}

template <typename T>
__global__ void __launch_bounds__(256) k_fill_synthetic(T *d1, T *d2, T *e1, T *e2, int N, DevScalars *S)
{
    const int64_t N3 = (int64_t)N * N * N;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (int64_t)gridDim.x * blockDim.x) {
        d1[i] = (T)(2e-4 * hash01(4 * i));
        d2[i] = (T)(2e-4 * hash01(4 * i + 1));
        e1[i] = (T)(2e-4 * hash01(4 * i + 2));
        e2[i] = (T)(2e-4 * hash01(4 * i + 3));
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        S->a_half = 1.0; S->ad = 0.5;
        S->bg_f[0] = 1.0; S->bg_f[1] = 0.0; S->bg_v[0] = 0.0; S->bg_v[1] = 0.0;
        S->step = 0; S->status = 0;
    }
}

// ---------------------------------------------------------------- launchers

void launch_fill_synthetic(int dtype, void *const s4[4], int N, DevScalars *S, hipStream_t st)
{
    const int64_t N3 = (int64_t)N * N * N;
    const int g = grid_for(N3, 256, 65536);
    if (dtype == 0)
        hipLaunchKernelGGL(k_fill_synthetic<float>, dim3(g), dim3(256), 0, st, (float *)s4[0], (float *)s4[1],
                           (float *)s4[2], (float *)s4[3], N, S);
    else
        hipLaunchKernelGGL(k_fill_synthetic<double>, dim3(g), dim3(256), 0, st, (double *)s4[0], (double *)s4[1],
                           (double *)s4[2], (double *)s4[3], N, S);
}


template <typename Tin, int ST>
static void input_moments_t(const void *f1, const void *f2, const void *v1, const void *v2, int N,
                            int beta, double *part, int nblk, hipStream_t st)
{
    hipLaunchKernelGGL((k_input_moments<Tin, ST>), dim3(nblk), dim3(256), 0, st, (const Tin *)f1,
                       (const Tin *)f2, (const Tin *)v1, (const Tin *)v2, N, beta, part);
}

void launch_input_moments(int stencil, int in_dtype, const void *f1, const void *f2, const void *v1,
                          const void *v2, int N, int beta, double *part, int nblk, hipStream_t st)
{
    if (stencil == 27) {
        if (in_dtype == 0) input_moments_t<float, 27>(f1, f2, v1, v2, N, beta, part, nblk, st);
        else input_moments_t<double, 27>(f1, f2, v1, v2, N, beta, part, nblk, st);
    } else {
        if (in_dtype == 0) input_moments_t<float, 7>(f1, f2, v1, v2, N, beta, part, nblk, st);
        else input_moments_t<double, 7>(f1, f2, v1, v2, N, beta, part, nblk, st);
    }
}

void launch_init_scalars(const double *part, int nblk, const DevParams *P, DevScalars *S,
                         int physical, double a0, double ad0, hipStream_t st)
{
    hipLaunchKernelGGL(k_init_scalars, dim3(1), dim3(kStage2Threads), 0, st, part, nblk, P, S,
                       physical, a0, ad0);
}

template <typename T, typename Tin>
static void init_fields_t(const void *f1, const void *f2, const void *v1, const void *v2, void *d1,
                          void *d2, void *e1, void *e2, int N, const DevParams *P,
                          const DevScalars *S, hipStream_t st)
{
    const int64_t N3 = (int64_t)N * N * N;
    hipLaunchKernelGGL((k_init_fields<T, Tin>), dim3(grid_for(N3, 256, 65536)), dim3(256), 0, st,
                       (const Tin *)f1, (const Tin *)f2, (const Tin *)v1, (const Tin *)v2, (T *)d1,
                       (T *)d2, (T *)e1, (T *)e2, N, P, S);
}

void launch_init_fields(int dtype, int in_dtype, const void *f1, const void *f2, const void *v1,
                        const void *v2, void *d1, void *d2, void *e1, void *e2, int N,
                        const DevParams *P, const DevScalars *S, hipStream_t st)
{
    if (dtype == 0 && in_dtype == 0) init_fields_t<float, float>(f1, f2, v1, v2, d1, d2, e1, e2, N, P, S, st);
    else if (dtype == 0) init_fields_t<float, double>(f1, f2, v1, v2, d1, d2, e1, e2, N, P, S, st);
    else if (in_dtype == 0) init_fields_t<double, float>(f1, f2, v1, v2, d1, d2, e1, e2, N, P, S, st);
    else init_fields_t<double, double>(f1, f2, v1, v2, d1, d2, e1, e2, N, P, S, st);
}

template <typename T, int ST>
static void reduce_t(const void *d1, const void *d2, int N, const double *bg_f, int beta, double *part,
                     int nblk, hipStream_t st)
{
    hipLaunchKernelGGL((k_reduce<T, ST>), dim3(nblk), dim3(256), 0, st, (const T *)d1, (const T *)d2, N,
                       bg_f, beta, part);
}

void launch_reduce(int stencil, int dtype, const void *d1, const void *d2, int N, const double *bg_f,
                   int beta, double *part, int nblk, hipStream_t st)
{
    if (stencil == 27) {
        if (dtype == 0) reduce_t<float, 27>(d1, d2, N, bg_f, beta, part, nblk, st);
        else reduce_t<double, 27>(d1, d2, N, bg_f, beta, part, nblk, st);
    } else {
        if (dtype == 0) reduce_t<float, 7>(d1, d2, N, bg_f, beta, part, nblk, st);
        else reduce_t<double, 7>(d1, d2, N, bg_f, beta, part, nblk, st);
    }
}

void launch_aupdate(const double *part, int nblk, const DevParams *P, const DevScalars *S, DevScalars *So,
                    CoefPair *C, hipStream_t st, DevScalars *tape)
{
    hipLaunchKernelGGL(k_aupdate, dim3(1), dim3(kStage2Threads), 0, st, part, nblk, P, S, So, C, tape);
}

void launch_set_powers(const DevParams *P, DevScalars *S, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_powers, dim3(1), dim3(64), 0, st, P, S);
}

void launch_aupdate_ens(const EnsEntry *tab, int R, int *queue, int parity, hipStream_t st)
{
    hipLaunchKernelGGL(k_aupdate_ens, dim3(R), dim3(kStage2Threads), 0, st, tab, queue, parity);
}

// Launch shape of k_diag_march for an N^3 lattice: tiles of 64 x DY, z-chunks
// chosen so that the items fill about `rows` blocks; grid = min(items, rows).
struct DiagShape {
    int ntx, nty, zchunk, items, grid;
};

static DiagShape diag_shape(int N, int rows, int DY)
{
    DiagShape d;
    d.ntx = (N + kDiagX - 1) / kDiagX;
    d.nty = (N + DY - 1) / DY;
    const int tiles = d.ntx * d.nty;
    int nz = rows / tiles;
    nz = nz < 1 ? 1 : (nz > N ? N : nz);
    d.zchunk = (N + nz - 1) / nz;
    nz = (N + d.zchunk - 1) / d.zchunk;
    d.items = tiles * nz;
    d.grid = d.items < rows ? d.items : rows;
    return d;
}

template <typename T, int ST, int MODE, typename To>
static int diag_t(const void *const s4[4], int N, const DevParams *P, const DevScalars *S, To *rho, To *pr,
                  double *part, int rows, hipStream_t st)
{
    const DiagShape d = diag_shape(N, rows, diag_y<ST>());
    hipLaunchKernelGGL((k_diag_march<T, ST, MODE, To>), dim3(d.grid), dim3(256), 0, st, (const T *)s4[0],
                       (const T *)s4[1], (const T *)s4[2], (const T *)s4[3], N, d.zchunk, d.ntx, d.nty, d.items,
                       P, S, rho, pr, part);
    return d.grid;
}

void launch_energy(int stencil, int dtype, const void *const s4[4], int N, const DevParams *P,
                   const DevScalars *S, double *part, int nblk, double *out_dev, hipStream_t st)
{
    int g;
    if (stencil == 27) {
        if (dtype == 0) g = diag_t<float, 27, 0, float>(s4, N, P, S, nullptr, nullptr, part, nblk, st);
        else g = diag_t<double, 27, 0, float>(s4, N, P, S, nullptr, nullptr, part, nblk, st);
    } else {
        if (dtype == 0) g = diag_t<float, 7, 0, float>(s4, N, P, S, nullptr, nullptr, part, nblk, st);
        else g = diag_t<double, 7, 0, float>(s4, N, P, S, nullptr, nullptr, part, nblk, st);
    }
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(kStage2Threads), 0, st, part, g, P, S, out_dev);
}

void ens_diag_shape(int stencil, int rows, EnsEntry *e)
{
    const DiagShape d = diag_shape(e->N, rows, stencil == 27 ? diag_y<27>() : diag_y<7>());
    e->dchunk = d.zchunk;
    e->dntx = d.ntx;
    e->dnty = d.nty;
    e->ditems = d.items;
    e->dgrid = d.grid;
}

void launch_energy_ens(int stencil, int dtype, const EnsEntry *tab, int R, int gmax, int parity, double *out_dev,
                       hipStream_t st)
{
    const dim3 grid(gmax, R), block(256);
    if (stencil == 27) {
        if (dtype == 0) hipLaunchKernelGGL((k_diag_ens<float, 27>), grid, block, 0, st, tab, parity);
        else hipLaunchKernelGGL((k_diag_ens<double, 27>), grid, block, 0, st, tab, parity);
    } else {
        if (dtype == 0) hipLaunchKernelGGL((k_diag_ens<float, 7>), grid, block, 0, st, tab, parity);
        else hipLaunchKernelGGL((k_diag_ens<double, 7>), grid, block, 0, st, tab, parity);
    }
    hipLaunchKernelGGL(k_energy_final_ens, dim3(R), dim3(kStage2Threads), 0, st, tab, parity, out_dev);
}

// A launch holds less than 2^32 threads, which one of all sites would exceed at
// 2048^3: above 512^3 the sites are dealt to several.
constexpr int64_t kFlatLaunch = (int64_t)1 << 27;

template <typename T, typename To, int WANT = 15>
static void get_fields_t(const void *const s4[4], void *const o[4], int N, const DevParams *P,
                         const DevScalars *S, int sync, hipStream_t st)
{
    if constexpr (WANT > 0) {
        const int want = (o[0] ? 1 : 0) | (o[1] ? 2 : 0) | (o[2] ? 4 : 0) | (o[3] ? 8 : 0);
        if (want != WANT) {
            get_fields_t<T, To, WANT - 1>(s4, o, N, P, S, sync, st);
            return;
        }
        const int64_t N3 = (int64_t)N * N * N;
        for (int64_t start = 0; start < N3; start += kFlatLaunch) {
            const int64_t n = N3 - start < kFlatLaunch ? N3 - start : kFlatLaunch;
            hipLaunchKernelGGL((k_get_fields<T, To, WANT>), dim3((unsigned)((n + 256 * kFlat - 1) / (256 * kFlat))),
                               dim3(256), 0, st, (const T *)s4[0], (const T *)s4[1], (const T *)s4[2],
                               (const T *)s4[3], (To *)o[0], (To *)o[1], (To *)o[2], (To *)o[3], start, N3, P, S,
                               sync);
        }
    }
}

void launch_get_fields(int dtype, int out_dtype, const void *const s4[4], void *const out[4], int N,
                       const DevParams *P, const DevScalars *S, int synchronized, hipStream_t st)
{
    if (dtype == 0 && out_dtype == 0) get_fields_t<float, float>(s4, out, N, P, S, synchronized, st);
    else if (dtype == 0) get_fields_t<float, double>(s4, out, N, P, S, synchronized, st);
    else if (out_dtype == 0) get_fields_t<double, float>(s4, out, N, P, S, synchronized, st);
    else get_fields_t<double, double>(s4, out, N, P, S, synchronized, st);
}

template <int ST>
static int rho_p_s(int dtype, int out_dtype, const void *const s4[4], void *rho, void *pr, int N,
                   const DevParams *P, const DevScalars *S, double *part, int nblk, hipStream_t st)
{
    if (dtype == 0 && out_dtype == 0)
        return diag_t<float, ST, 1, float>(s4, N, P, S, (float *)rho, (float *)pr, part, nblk, st);
    if (dtype == 0) return diag_t<float, ST, 1, double>(s4, N, P, S, (double *)rho, (double *)pr, part, nblk, st);
    if (out_dtype == 0)
        return diag_t<double, ST, 1, float>(s4, N, P, S, (float *)rho, (float *)pr, part, nblk, st);
    return diag_t<double, ST, 1, double>(s4, N, P, S, (double *)rho, (double *)pr, part, nblk, st);
}

void launch_rho_p(int stencil, int dtype, int out_dtype, const void *const s4[4], void *rho, void *pr, int N,
                  const DevParams *P, const DevScalars *S, double *part, int nblk, double *out_dev,
                  hipStream_t st)
{
    const int g = stencil == 27 ? rho_p_s<27>(dtype, out_dtype, s4, rho, pr, N, P, S, part, nblk, st)
                                : rho_p_s<7>(dtype, out_dtype, s4, rho, pr, N, P, S, part, nblk, st);
    hipLaunchKernelGGL(k_rho_p_final, dim3(1), dim3(kStage2Threads), 0, st, part, g, P, out_dev);
}

// ---------------------------------------------------------------- bandwidth reference

// The benchmark's bandwidth reference: one element per lane over a grid that
// covers the arrays once, blocks in address order, non-temporal stores (the
// fastest order for this byte mix on gfx950: 6.2 TB/s at 512^3 against 5.0
// for a grid-stride loop with 16-byte lanes).
__global__ void __launch_bounds__(256) k_stream_copy(const float *__restrict__ a0, const float *__restrict__ a1,
                                                     const float *__restrict__ a2, const float *__restrict__ a3,
                                                     float *__restrict__ b0, float *__restrict__ b1,
                                                     float *__restrict__ b2, float *__restrict__ b3, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float x0 = a0[i], x1 = a1[i], x2 = a2[i], x3 = a3[i];
    __builtin_nontemporal_store(x0, b0 + i);
    __builtin_nontemporal_store(x1, b1 + i);
    __builtin_nontemporal_store(x2, b2 + i);
    __builtin_nontemporal_store(x3, b3 + i);
}

void launch_stream_copy(const float *const a[4], float *const b[4], int64_t n, hipStream_t st)
{
    if (n < 1) return;
    const int64_t blocks = (n + 255) / 256;  // n <= 2048^3: at most 2^25 blocks
    hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)blocks), dim3(256), 0, st, a[0], a[1], a[2], a[3], b[0], b[1],
                       b[2], b[3], n);
}

void launch_sync_deviation(int dtype, const void *d, const void *e, double *out, int N, double h, int velocity,
                           hipStream_t st)
{
    const int64_t N3 = (int64_t)N * N * N;
    if (dtype == 0)
        hipLaunchKernelGGL(k_sync_deviation<float>, dim3(grid_for(N3, 256, 65536)), dim3(256), 0, st,
                           (const float *)d, (const float *)e, out, N3, h, velocity);
    else
        hipLaunchKernelGGL(k_sync_deviation<double>, dim3(grid_for(N3, 256, 65536)), dim3(256), 0, st,
                           (const double *)d, (const double *)e, out, N3, h, velocity);
}

void launch_sum_partials(const double *part, int nblk, int nv, double *out, hipStream_t st)
{
    (void)nv;
    hipLaunchKernelGGL(k_sum_partials4, dim3(1), dim3(kStage2Threads), 0, st, part, nblk, out);
}

void launch_set_pending(double *part, int nblk, const double *totals, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_pending, dim3(grid_for((int64_t)nblk * kNPart, 256, 1024)), dim3(256), 0,
                       st, part, nblk, totals);
}

}  // namespace lf
