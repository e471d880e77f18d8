// Per-site arithmetic shared by the LDS sweeps of liblf (7-point in
// lf_sweep.hip, 27-point in lf_sweep27.hip): the uniform kick coefficients,
// the force with the potential difference expanded around the FP64
// background, and the XCD-aware block order.
#pragma once
#include "lf_internal.h"
#include "lf_scale.h"

namespace lf {

template <typename T>
__device__ inline const Coef<T> &coef_of(const CoefPair *C);
template <>
__device__ inline const Coef<float> &coef_of<float>(const CoefPair *C) { return C->f; }
template <>
__device__ inline const Coef<double> &coef_of<double>(const CoefPair *C) { return C->d; }

// Uniform per-step coefficients, read once per block (scalar loads).
template <typename T, int NH>
struct Coefs {
    T Cl, Cf, dt, C2, g1, g2, two_g1, two_g2, g1sq;
    T h[NH];
    template <typename C>
    __device__ inline void load(const C &c)
    {
        Cl = c.Cl; Cf = c.Cf; dt = c.dt; C2 = c.C2; g1 = c.g1; g2 = c.g2;
        two_g1 = c.two_g1; two_g2 = c.two_g2; g1sq = c.g1sq;
#pragma unroll
        for (int j = 0; j < NH; ++j) h[j] = c.h[j];
    }
    // Every value, and x and y, into scalar registers.  Arithmetic on
    // floating-point values is vector arithmetic, also of uniform ones, and the
    // compiler drops a lane read of what it knows to be uniform, or moves it to
    // where the value came from, and keeps the result in a vector register.  Past
    // the empty asm it does not know where they came from.
    __device__ inline void to_scalar(double &x, double &y)
    {
        asm("" : "+v"(Cl), "+v"(Cf), "+v"(dt), "+v"(C2), "+v"(g1), "+v"(g2), "+v"(two_g1), "+v"(two_g2),
                 "+v"(g1sq), "+v"(x), "+v"(y));
#pragma unroll
        for (int j = 0; j < NH; ++j) asm("" : "+v"(h[j]));
        Cl = uniform(Cl); Cf = uniform(Cf); dt = uniform(dt); C2 = uniform(C2); g1 = uniform(g1); g2 = uniform(g2);
        two_g1 = uniform(two_g1); two_g2 = uniform(two_g2); g1sq = uniform(g1sq);
#pragma unroll
        for (int j = 0; j < NH; ++j) h[j] = uniform(h[j]);
        x = uniform(x);
        y = uniform(y);
    }
    // Velocity increments of both fields at one site from the raw stencil
    // sums (s6a, s6b: the integer-weighted neighbour sum including the centre
    // term; Cl carries 1/dx^2 and the stencil weight) and the deviations
    // a = d1, b = d2.  Every multiply-add is an explicit fma, so that each
    // inlined copy rounds alike: a ring site then equals, to the bit, the site
    // that the neighbouring tile stores.  HORNER_ROUNDED: which of the two
    // products of dv1 = hor a + C2 q is rounded before they are added.
    template <bool HORNER_ROUNDED>
    __device__ inline void force(T a, T b, T s6a, T s6b, T &inc_a, T &inc_b) const
    {
#pragma clang fp contract(off)
        T hor = h[NH - 1];
#pragma unroll
        for (int j = NH - 2; j >= 0; --j) hor = fma(hor, a, h[j]);
        const T t2 = g2 + b;
        const T q = fma(g1 * b, two_g2 + b, (a * t2) * t2);
        const T dv1 = HORNER_ROUNDED ? fma(q, C2, hor * a) : fma(hor, a, C2 * q);
        const T w = fma(g1sq, b, (a * (two_g1 + a)) * t2);
        inc_a = fma(Cf, a, Cl * s6a) - dv1;
        inc_b = fma(-C2, w, fma(Cf, b, Cl * s6b));
    }
    // The same increments as the 27-point sweep rounds them (it too computes a
    // site in several copies of its loop and, redundantly, as another tile's
    // ring site).
    __device__ inline void force_fma(T a, T b, T s6a, T s6b, T &inc_a, T &inc_b) const
    {
        T hor = h[NH - 1];
#pragma unroll
        for (int j = NH - 2; j >= 0; --j) hor = fma(hor, a, h[j]);
        const T t2 = g2 + b;
        const T dv1 = fma(hor, a, C2 * fma(a * t2, t2, (g1 * b) * (two_g2 + b)));
        const T dv2 = C2 * fma(a * (two_g1 + a), t2, g1sq * b);
        inc_a = fma(Cl, s6a, fma(Cf, a, -dv1));
        inc_b = fma(Cl, s6b, fma(Cf, b, -dv2));
    }
};

// Coefs::force of the 7-point sweeps: one rounding for beta 2, 3 and 6, and for
// beta 4 and 5 one in tiles of one site a thread and the other in wider ones.
// These are the roundings that stored results were made with.
constexpr bool horner_rounded(int nh, bool wide) { return nh == 5 || (nh >= 3 && wide); }

template <typename T>
__device__ inline T six_sum(T xm, T xp, T ym, T yp, T zm, T zp, T c)
{
    return fma(T(-6), c, ((xm + xp) + (ym + yp)) + (zm + zp));
}

template <int NH>
__device__ inline double potential_pow(double x)
{
    double r = x;
#pragma unroll
    for (int j = 0; j < NH; ++j) r *= x;  // x^(NH+1) = x^beta
    return r;
}

// The step's coefficients as a scale-factor kernel left them.
struct CoefsFrom {
    const CoefPair *__restrict__ C;
    template <typename T, int NH>
    __device__ inline void get(Coefs<T, NH> &c, double &g1n, double &g2n) const
    {
        c.load(coef_of<T>(C));
        g1n = C->g1n;
        g2n = C->g2n;
    }
    __device__ inline void finish() const {}
};

// The totals of a step's partial rows, formed by a whole block of 256 threads
// and the same in every thread.  The rows are added in the order of the
// scale-factor kernel (thread, wave, block), so both give the same bits.
__device__ inline void step_totals(const StepSource &q, const ScaleIn &in, double (&tot)[kNPart])
{
    static_assert(kStage2Threads == 256, "rows are dealt to the threads as in stage 2");
    __shared__ double sm[kNPart][4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    // all of the thread's rows in flight at once
    constexpr int kRows = kFusedRows / 256;
    double row[kRows][kNPart];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int j = t + 256 * k;
#pragma unroll
        for (int i = 0; i < kNPart; ++i) row[k][i] = j < q.rows ? q.part[(size_t)j * kNPart + i] : 0.0;
    }
    in.arrived();
#pragma unroll
    for (int i = 0; i < kNPart; ++i) {
        double x = 0.0;
#pragma unroll
        for (int k = 0; k < kRows; ++k) x += row[k][i];
        x = wave_sum(x);
        if (lane == 0) sm[i][w] = x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kNPart; ++i) {
        tot[i] = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) tot[i] += sm[i][v];
    }
}

// Writes what a fused step leaves besides the arrays; first wave of a block.
__device__ inline void step_commit(const StepSource &q, const double (&tot)[kNPart], const ScaleStep &o)
{
    if (threadIdx.x == 0) scale_commit(tot, o, q.P, q.S, q.So, q.C, q.tape, in_const(q.P)->beta);
    scale_commit_powers(o.an, q.P, q.So);
}

// The extra block of a fused step (StepSource::extra).
__device__ inline void step_extra_block(const StepSource &q)
{
    const ScaleIn in(q.P, q.S);
    double tot[kNPart];
    step_totals(q, in, tot);
    if (threadIdx.x >= 64) return;
    ScaleStep o;
    scale_step(tot, in, in_const(q.P)->beta, o);
    step_commit(q, tot, o);
}

// The step's coefficients formed in this block (StepSource), or read from C
// when a scale-factor kernel ran.  A kernel of its own for this chain of
// dependent FP64 operations on one block takes 5 to 6 us between two sweeps
// in which the device does nothing else; in every block of the sweep it
// takes about 2.  Step times, two kernels against one, with wave sums by LDS
// permutes on both sides: 32^3 FP64 10.8 -> 8.8 us, 128^3 FP32 25.6 -> 23.8,
// 256^3 114.3 -> 110.9, 512^3 792 -> 789 (7 points).  The coefficients stay in
// scalar registers: in vector ones (as they were without to_scalar() and the scalar
// loads of get()) the sweeps that fill the register file spilled inside their
// loops.  FP64 32x16 tiles at 200^3 315 -> 135 us, FP32 64x16 at 256^3 177 -> 126,
// FP64 27 points at 256^3 246 -> 235, FP32 27 points at 160^3 46.2 -> 43.3.
// SCALAR: FP32 tiles of one site a thread have registers to spare and keep the
// coefficients in vector ones (27 points, 48^3 10.35 us against 10.7, 100^3 21.35
// against 21.65).  `first`: this block writes the results.
template <bool SCALAR>
struct CoefsOfStep {
    const StepSource &q;
    const bool first;
    __device__ inline CoefsOfStep(const StepSource &src, bool f) : q(src), first(f) {}
    template <typename T, int NH>
    __device__ inline void get(Coefs<T, NH> &c, double &g1n, double &g2n) const
    {
        if (!q.part) {
            // in scalar loads: from vector ones, the values of both branches
            // would live in vector registers
            InConst<CoefPair> *C = in_const(q.C);
            if constexpr (sizeof(T) == 4) c.load(C->f);
            else c.load(C->d);
            g1n = C->g1n;
            g2n = C->g2n;
            return;
        }
        const ScaleIn in(q.P, q.S);
        double tot[kNPart];
        step_totals(q, in, tot);
        ScaleStep o;
        scale_step(tot, in, NH + 1, o);
        const double g1 = in.g1, g2 = in.g2;
        c.Cl = (T)o.Cl; c.Cf = (T)o.Cf; c.dt = (T)in.dt; c.C2 = (T)o.C2; c.g1 = (T)g1; c.g2 = (T)g2;
        c.two_g1 = (T)(2.0 * g1); c.two_g2 = (T)(2.0 * g2); c.g1sq = (T)(g1 * g1);
#pragma unroll
        for (int j = 0; j < NH; ++j) c.h[j] = (T)scale_h(o.ch, NH + 1, j + 1, g1);
        g1n = o.g1n;
        g2n = o.g2n;
        if constexpr (SCALAR) c.to_scalar(g1n, g2n);
        if (first && threadIdx.x == 0) {
            StepResult &r = result();
#pragma unroll
            for (int i = 0; i < kNPart; ++i) r.t[i] = tot[i];
            r.o = o;
        }
    }
    // The results are written when the march is over: the stores and pow
    // among the first loads would set the kernel's register count.
    __device__ inline void finish() const
    {
        if (!q.part || !first || threadIdx.x >= 64) return;
        step_commit(q, result().t, result().o);
    }

private:
    struct StepResult {
        double t[kNPart];
        ScaleStep o;
    };
    __device__ static inline StepResult &result()
    {
        __shared__ StepResult r;
        return r;
    }
};

template <typename T, int TX, int TY>
using StepCoefs = CoefsOfStep<(TX * TY > 256 || sizeof(T) == 8)>;

// Where the z-planes of the four input arrays (d1, d2, e1, e2) of a z-slab
// sweep lie.  A sweep reads d on planes [z0-2, z1] and e on [z0-1, z1-1] of
// a chunk [z0, z1) of [0, nz).  Planes 0 .. nz-1 are the arrays' own; plane
// z < 0 lies at lo[i] + (z+2) N^2 and plane z >= nz at hi[i] + (z-nz) N^2,
// in the slab's halo buffers (e is never read above the slab).  Only the
// slab kernels use this; the periodic ones wrap the plane index.
template <typename T>
struct ZPlanes {
    const T *lo[4];
    const T *hi[4];
    int nz;
    __device__ inline const T *at(int i, const T *p, int z, int64_t NN) const
    {
        return z < 0 ? lo[i] + (int64_t)(z + 2) * NN
                     : (z >= nz ? hi[i] + (int64_t)(z - nz) * NN : p + (int64_t)z * NN);
    }
};

template <typename T>
inline ZPlanes<T> planes_of(const SweepIO &io)
{
    ZPlanes<T> zp;
    for (int i = 0; i < 4; ++i) {
        zp.lo[i] = (const T *)io.lo[i];
        zp.hi[i] = (const T *)io.hi[i];
    }
    zp.nz = io.nz;
    return zp;
}

// Work item loop of the persistent ensemble sweeps.  The items are split
// into one segment per XCD (items seg[x] .. seg[x+1] - 1), each holding whole z-chunks
// of some realizations, longest first; a block takes the next item of its own
// XCD's segment (hardware places block b on XCD b mod 8) from that segment's
// counter, so the tiles of one chunk run together on one L2 and find their
// neighbours' halo rows there.  When its segment is used up it takes items of
// the other segments in turn.  queue holds the counters (queue[32 x], 128
// bytes apart), reset to 0 by the batched scale-factor kernel that runs
// before every sweep, followed by seg[0..8].  Every thread of the block sees the same index; fn(i) runs for
// each item.
constexpr int kEnsXcd = 8, kEnsQueueStride = 32;

template <typename F>
__device__ inline void for_each_item(int *queue, int nitems, F &&fn)
{
    const int *seg = queue + kEnsXcd * kEnsQueueStride;  // segment bounds follow the counters
    __shared__ int s_item;
    const int home = blockIdx.x % kEnsXcd;
    int k = 0;  // thread 0: segments used up so far, own segment first
    for (;;) {
        if (threadIdx.x == 0) {
            int item = -1;
            while (k < kEnsXcd) {
                const int x = (home + k) % kEnsXcd;
                const int j = seg[x] + atomicAdd(queue + x * kEnsQueueStride, 1);
                if (j < seg[x + 1] && j < nitems) {
                    item = j;
                    break;
                }
                ++k;
            }
            s_item = item;
        }
        __syncthreads();
        const int i = s_item;
        if (i < 0) break;
        fn(i);
        __syncthreads();  // LDS (and s_item) are reused by the next item
    }
}

}  // namespace lf
