// The scale-factor update of one leapfrog step in FP64 (Sainio,
// arXiv:0911.5692, eq. scale, eq. scalar-evo, eq. evo), shared by the
// scale-factor kernels (lf_kernels.hip) and by the sweeps that form it in
// their own blocks (lf_sweep_common.h).  Every multiply and add rounds by
// itself (contraction is off), so that all of its inlined copies give the
// same bits: every block of a sweep, a lone lattice and an ensemble member
// then agree on the scale factor and on the coefficients.
#pragma once
#include "lf_internal.h"

#include <math.h>

namespace lf {

// Uniform values from vector into scalar registers.
__device__ inline float uniform(float x)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ inline double uniform(double x)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                            __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// The sum over a wave, in every lane: lanes 32 apart are added first, then 16,
// 8, 4, 2 and 1.  The partners are reached by lane swaps and DPP moves in the
// vector unit.  With 2 x 6 permutes through the LDS for each of the sums at the
// start and at the end of every block of a sweep (the same bits), a step took
// 1.0 us more at 32^3 FP64 (7.8 -> 6.8), 1.4 at 128^3 FP32 (7 points, 23.0 ->
// 21.6) and 1.2 at 100^3 FP32 (27 points).
template <int CTRL>
__device__ inline double dpp_move(double x)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}
__device__ inline double wave_sum(double x)
{
    int hi = __double2hiint(x), lo = __double2loint(x);
    auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    x = __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    hi = __double2hiint(x), lo = __double2loint(x);
    h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    x = __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    x += dpp_move<0x128>(x);  // row_ror:8, 4: by now equal in lanes 16, 8 apart
    x += dpp_move<0x124>(x);
    x += dpp_move<0x4e>(x);  // quad_perm [2, 3, 0, 1], [1, 0, 3, 2]
    x += dpp_move<0xb1>(x);
    return x;
}

// The parameters and the scalars a step starts from do not change while a
// kernel that updates the scale factor runs: read through the constant
// address space they come in scalar loads and stay in scalar registers.
template <typename T>
using InConst = const __attribute__((address_space(4))) T;
template <typename T>
__device__ inline InConst<T> *in_const(const T *p)
{
    return (InConst<T> *)p;
}

// What the update needs besides the sums.
struct ScaleIn {
    double N3, dx, dt, r, s, c1, G, gw, kappa2;
    double a, w, g1, g2, v1, v2, pw[kNPow];
    __device__ inline ScaleIn(const DevParams *Pg, const DevScalars *Sg)
    {
        InConst<DevParams> *P = in_const(Pg);
        InConst<DevScalars> *S = in_const(Sg);
        N3 = P->N3; dx = P->dx; dt = P->dt; r = P->r; s = P->s; c1 = P->c1; G = P->G; gw = P->gw;
        kappa2 = P->kappa2;
        a = S->a_half; w = S->ad;
        g1 = S->bg_f[0]; g2 = S->bg_f[1]; v1 = S->bg_v[0]; v2 = S->bg_v[1];
#pragma unroll
        for (int j = 0; j < kNPow; ++j) pw[j] = S->pw[j];
    }
    // The values are there from here on: without it the compiler moves the
    // loads down to their first use, behind the sums, where their latency is
    // not hidden by that of the rows.
    __device__ inline void arrived() const
    {
        asm volatile("" ::"s"(N3), "s"(dx), "s"(dt), "s"(r), "s"(s), "s"(c1), "s"(G), "s"(gw), "s"(kappa2));
        asm volatile("" ::"s"(a), "s"(w), "s"(g1), "s"(g2), "s"(v1), "s"(v2));
        asm volatile("" ::"s"(pw[0]), "s"(pw[1]), "s"(pw[2]), "s"(pw[3]), "s"(pw[4]));
    }
};

__device__ inline double ipow_d(double x, int n)
{
    double r = 1.0;
    for (int i = 0; i < n; ++i) r *= x;
    return r;
}

__device__ inline double binom_d(int n, int k)
{
    double r = 1.0;
    for (int i = 1; i <= k; ++i) r = r * (double)(n - k + i) / (double)i;
    return r;
}

// The powers of a that a step starting at a = a_{k+1/2} needs (DevScalars::pw):
// a^p1, a^p2, a^(-2s-2r-1), a^(2s+2), a^(-2s-2).  They depend on a alone, so
// whoever sets a_half sets them too, and the next step finds them ready
// instead of evaluating pow between its sums and its kick.
__device__ inline double scale_power(int j, const DevParams *Pg, double a)
{
    InConst<DevParams> *P = in_const(Pg);
    const double r = P->r, s = P->s;
    const double ex = j == 0 ? P->p1 : j == 1 ? P->p2 : j == 2 ? -2.0 * s - 2.0 * r - 1.0
                    : j == 3 ? 2.0 * s + 2.0 : -2.0 * s - 2.0;
    return pow(a, ex);
}

// What one update yields: the kick's coefficients at k+1/2 and the scalars
// of the next state.
struct ScaleStep {
    double Cl, Cf, C2, ch;  // ch: dt c1 a^p1 (see scale_h)
    double an, u, g1n, g2n, vb1, vb2;
    unsigned int bad;
};

// h[j-1] of the kick, j = 1..beta-1: ch C(beta-1, j) g1^(beta-1-j).
__device__ inline double scale_h(double ch, int beta, int j, double g1)
{
    return ch * binom_d(beta - 1, j) * ipow_d(g1, beta - 1 - j);
}

// State on entry (in): a_{k+1/2}, a'_k, background f_bar(k+1/2), v_bar(k), the
// powers of a; t: the sums over f(k+1/2).
//   F_a = kappa^2 a^(-2s-2r-1) [Sg/3 + a^(2s+2) SV]
//   a'_{k+1} solves a'_{k+1} = a'_k + dt[(-s-2)((a'_k + a'_{k+1})/2)^2/a + F_a]
//     (time-centred; the root that tends to a'_k + dt F_a as the quadratic
//      coefficient vanishes, written in the cancellation-free form)
//   a'_{k+1/2} = (a'_k + a'_{k+1})/2, a''_{k+1/2} = (a'_{k+1} - a'_k)/dt,
//   a_{k+3/2} = a_{k+1/2} + dt a'_{k+1}.
__device__ inline void scale_step(const double (&t)[kNPart], const ScaleIn &in, const int beta, ScaleStep &o)
{
#pragma clang fp contract(off)
    const double N3 = in.N3, dx = in.dx, dt = in.dt, r = in.r, s = in.s, c1 = in.c1, G = in.G, a = in.a, w = in.w;
    const double ap1 = in.pw[0], ap2 = in.pw[1], aF = in.pw[2], aV = in.pw[3], alpha = in.pw[4];
    const double Sg = in.gw * (t[0] + t[1]) / (dx * dx * N3);
    const double SV = (c1 * ap1 * t[2] / (double)beta + 0.5 * G * ap2 * t[3]) / N3;
    const double Fa = in.kappa2 * aF * (Sg / 3.0 + aV * SV);
    const double c = (-s - 2.0) * dt / (4.0 * a);
    const double disc = 1.0 - 8.0 * c * w - 4.0 * c * dt * Fa;
    const double u = 2.0 * (c * w * w + w + dt * Fa) / ((1.0 - 2.0 * c * w) + sqrt(disc));
    const double adh = 0.5 * (w + u), add = (u - w) / dt;
    const double bc = r * (s - r + 2.0) * (adh / a) * (adh / a) + r * add / a;
    o.an = a + dt * u;
    o.u = u;

    // homogeneous mode: same kick and drift with zero Laplacian
    const double g1 = in.g1, g2 = in.g2;
    const double dV1 = c1 * ap1 * ipow_d(g1, beta - 1) + G * ap2 * g1 * g2 * g2;
    const double dV2 = G * ap2 * g1 * g1 * g2;
    o.vb1 = in.v1 + dt * (bc * g1 - dV1);
    o.vb2 = in.v2 + dt * (bc * g2 - dV2);
    o.g1n = g1 + dt * o.vb1;
    o.g2n = g2 + dt * o.vb2;

    // coefficients at k+1/2
    o.ch = dt * c1 * ap1;
    o.Cl = dt * alpha * in.gw / (dx * dx);
    o.Cf = dt * bc;
    o.C2 = dt * G * ap2;

    unsigned int bad = 0;
#pragma unroll
    for (int i = 0; i < kNPart; ++i) bad |= !isfinite(t[i]);
    o.bad = bad | !(disc >= 0.0) | !isfinite(u);
}

// Writes the update's results but the powers: So, the coefficient block C and,
// if tape is not NULL, a copy of the scalars the step started from.  One
// thread.
__device__ inline void scale_commit(const double (&t)[kNPart], const ScaleStep &o, const DevParams *Pg,
                                    const DevScalars *Sg, DevScalars *So, CoefPair *__restrict__ C, DevScalars *tape,
                                    const int beta)
{
    InConst<DevParams> *P = in_const(Pg);
    InConst<DevScalars> *S = in_const(Sg);
    if (tape) *tape = *Sg;
    const double dt = P->dt, g1 = S->bg_f[0], g2 = S->bg_f[1];
    Coef<double> &cd = C->d;
    Coef<float> &cf = C->f;
    cd.Cl = o.Cl; cd.Cf = o.Cf; cd.dt = dt; cd.C2 = o.C2; cd.g1 = g1; cd.g2 = g2;
    cd.two_g1 = 2.0 * g1; cd.two_g2 = 2.0 * g2; cd.g1sq = g1 * g1; cd.nh = beta - 1;
    cf.Cl = (float)o.Cl; cf.Cf = (float)o.Cf; cf.dt = (float)dt; cf.C2 = (float)o.C2;
    cf.g1 = (float)g1; cf.g2 = (float)g2; cf.two_g1 = (float)(2.0 * g1);
    cf.two_g2 = (float)(2.0 * g2); cf.g1sq = (float)(g1 * g1); cf.nh = beta - 1;
    for (int j = 0; j < kMaxBeta; ++j) {
        const double hj = j < beta - 1 ? scale_h(o.ch, beta, j + 1, g1) : 0.0;
        cd.h[j] = hj;
        cf.h[j] = (float)hj;
    }
    C->g1n = o.g1n;
    C->g2n = o.g2n;
    So->status = S->status | o.bad;
#pragma unroll
    for (int i = 0; i < kNPart; ++i) So->pend[i] = t[i];
    So->a_half = o.an;
    So->ad = o.u;
    So->bg_f[0] = o.g1n; So->bg_f[1] = o.g2n;
    So->bg_v[0] = o.vb1; So->bg_v[1] = o.vb2;
    So->step = S->step + 1;
}

// The powers of the state the update leaves, one per lane of a wave.
__device__ inline void scale_commit_powers(double an, const DevParams *P, DevScalars *So)
{
    const int l = threadIdx.x & 63;
    const double pw = scale_power(l, P, an);
    if (l < kNPow) So->pw[l] = pw;
}

}  // namespace lf
