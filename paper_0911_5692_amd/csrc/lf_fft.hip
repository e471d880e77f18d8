// FFT-based parts of liblf, gfx950: the vacuum initial state and the power
// spectra of the fields.
//
// Vacuum initial state (Sainio, arXiv:0911.5692, Sec. II.B: homogeneous values
// are inputs, the random fluctuations are generated by the program through an
// FFT), for each of the four arrays j = 0..3 (f1, f2, u1, u2):
//   1. unit normal white noise per site from the counter-based generator
//      Philox4x32-10 (Salmon et al., SC'11): counter (i mod 2^32, i div 2^32,
//      j, 0), key (seed mod 2^32, seed div 2^32), two 53-bit uniforms
//      U = (hi 2^21 + lo div 2^11 + 1) 2^-53 in (0, 1] and the Box-Muller
//      normal sqrt(-2 ln U1) cos(2 pi U2);
//   2. forward transform;
//   3. mode n multiplied by sqrt(N^3 P(k) / L^3) / N^3 with
//      P = eps^2 / (2 omega_k) (fields) or eps^2 omega_k / 2 (velocities),
//      omega_k = sqrt(k^2 + m_i^2), k = 2 pi |n| / L; zero at n = 0 and for
//      |n| above the cutoff;
//   4. inverse transform, 5. the homogeneous value added.
// All FP64.  The 1/N^3 of the inverse transform is folded into the filter.
//
// Power spectrum (the FFT diagnostics the paper names as the next step,
// Sec. IV): transform of the synchronised deviation of a field from its
// homogeneous value (so the FFT's rounding scales with the fluctuation, not
// with the mean), the homogeneous value entering only the n = 0 mode
// (F_0 = N^3 bg + D_0), then the shell average
//   power[s] = (L^3/N^6) sum_{rint|n| = s} |F_n|^2 / count[s]
// over the full set of modes (the conjugate half of the real transform counted
// through weights 2).
//
// Sizes without large prime factors (spectrum_own, vacuum_own) are transformed
// here, line by line in LDS (lf_fft_line.h), so that each direction is one pass over the half
// spectrum and everything around the transform rides along:
//   spectrum: x pass (synchronised deviation formed on load), y pass, z pass
//     (shells summed from LDS; the transform is never written);
//   vacuum: x pass (noise formed on load), y pass, z pass (transform, filter,
//     inverse), inverse y pass, inverse x pass (homogeneous value added on
//     store).  Modes above the cutoff are neither stored nor read between
//     the passes (at the default cutoff N/4: half of the x modes and half of
//     the y rows).
// The passes are bound by memory: at 512^3 the half spectrum is 1.08 GB, and
// the library's transform alone reads and writes it three times besides the
// separate passes before and after it.  Two real lines go through one complex
// transform (a + i b), so odd N need nothing of their own.
// At 512^3 (FP32 fields) one spectrum takes 1.55 ms (x pass 0.52, y 0.48, z 0.50;
// 2.8 before: deviation 0.32, transform 1.83, shells 0.54), of which its bytes
// (5.4 GB) take 0.9 at the rate of a plain copy; one vacuum array 1.75 ms
// (x 0.93, y 0.22, z 0.15, y 0.22, x 0.48; 5.3 before), of which the noise's
// arithmetic takes about 0.55.  Between its loads and stores a pass is bound by
// the LDS exchanges, the twiddle loads and the FP64 arithmetic of its stages,
// about 8 us for the 128 KB that two blocks of a CU hold, which run beside the
// other block's memory phases in part.
// Other sizes go through hipFFT D2Z/Z2D with separate kernels.
#include "lf_internal.h"

#include <hipfft/hipfft.h>
#include <math.h>
#include <stdio.h>

#include <map>
#include <mutex>
#include <utility>

#include "lf.h"
#include "lf_fft_line.h"

namespace lf {

namespace {

constexpr unsigned kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr unsigned kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// Ten Philox4x32 rounds; the round key is bumped between rounds.
__device__ inline uint4 philox4x32_10(uint4 c, uint2 k)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k.x += kPhiloxW0;
            k.y += kPhiloxW1;
        }
        // one 32 x 32 -> 64 bit multiply each, not a low and a high half
        const unsigned long long p0 = (unsigned long long)kPhiloxM0 * c.x;
        const unsigned long long p1 = (unsigned long long)kPhiloxM1 * c.z;
        c = make_uint4((unsigned)(p1 >> 32) ^ c.y ^ k.x, (unsigned)p1, (unsigned)(p0 >> 32) ^ c.w ^ k.y,
                       (unsigned)p0);
    }
    return c;
}

// (m + 1) 2^-53, m the top 53 bits of the two words.
__device__ inline double uniform53(unsigned hi, unsigned lo)
{
    return fma((double)hi, 0x1p-32, (double)((lo >> 11) + 1u) * 0x1p-53);
}

// The noise in FP64 is bound by its arithmetic, so its three functions are
// written for the arguments that occur, from series and Newton steps: with the
// math library's log, sqrt and cos (which reduce arguments of any size and
// look for the special ones) a site took twice the instructions.  One array's
// noise at 512^3: 0.93 -> 0.54 ms; four vacuum arrays 8.5 -> 7.1 ms.  Against 80-bit
// arithmetic over 4 million word pairs, the ends of both uniforms among them,
// the radius is as far off as before (rms 0.47 of 2^-53) and the noise less
// (rms 2.8e-16 -> 1.0e-16), since the turn is no longer rounded.

// A constant kept in scalar registers: the multiply-add then takes it as its
// addend, where one in vector registers is first copied into the result.
__device__ inline double in_sgpr(double c)
{
    asm("" : "+s"(c));
    return c;
}

// log u for u = m 2^-53, 1 <= m <= 2^53: u = 2^e f with f in [sqrt(1/2), sqrt(2)),
// t = f - 1 (exact), s = t / (2 + t), log f = 2 atanh(s) = t - s (t - s^2 Q),
// Q = sum_k 2 s^2k / (2k + 3); since s <= 0.172 nine terms leave 1e-17.
__device__ inline double log_unit(double u)
{
    constexpr double kLn2Hi = 0x1.62e42fefa3800p-1, kLn2Lo = 0x1.ef35793c76730p-45;  // e kLn2Hi is exact
    double f = __builtin_amdgcn_frexp_mant(u);
    int ei = __builtin_amdgcn_frexp_exp(u);
    const bool low = f < 0.70710678118654752;
    f = low ? f + f : f;
    ei = low ? ei - 1 : ei;
    const double e = (double)ei, t = f - 1.0, d = 2.0 + t;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    double s = t * r;
    s = fma(fma(-d, s, t), r, s);
    const double z = s * s;
    double q = 2.0 / 19.0;
    q = fma(q, z, in_sgpr(2.0 / 17.0));
    q = fma(q, z, in_sgpr(2.0 / 15.0));
    q = fma(q, z, in_sgpr(2.0 / 13.0));
    q = fma(q, z, in_sgpr(2.0 / 11.0));
    q = fma(q, z, in_sgpr(2.0 / 9.0));
    q = fma(q, z, in_sgpr(2.0 / 7.0));
    q = fma(q, z, in_sgpr(2.0 / 5.0));
    q = fma(q, z, in_sgpr(2.0 / 3.0));
    const double eh = e * kLn2Hi, c = eh + t;
    const double cl = t - (c - eh);  // c + cl = e kLn2Hi + t
    return c - fma(s, fma(-z, q, t), -fma(e, kLn2Lo, cl));
}

// sqrt x for x = 0 or 1e-16 <= x <= 100: Newton steps from the hardware's
// estimate of 1 / sqrt(x).
__device__ inline double sqrt_plain(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return x > 0.0 ? g : 0.0;
}

// cos(2 pi u) as sin(pi y), y = 1/2 - 2 u, which is exact for the uniforms, as is
// its remainder y - rint(y) in [-1/2, 1/2]; the series of sin(pi y) / y to y^20
// leaves 1e-18.  (A rounded 2 pi u, as the argument of a cosine, is off by up to
// 6e-16.)
__device__ inline double cos_turn(double u)
{
    double y = fma(u, -2.0, 0.5);
    const double k = rint(y);
    y -= k;
    const double z = y * y;
    double p = 0x1.2877020d52cf0p-31;  // (-1)^k pi^(2k + 1) / (2k + 1)!
    p = fma(p, z, in_sgpr(-0x1.8a404211f9547p-26));
    p = fma(p, z, in_sgpr(0x1.aaec32af93359p-21));
    p = fma(p, z, in_sgpr(-0x1.6fadb9f155744p-16));
    p = fma(p, z, in_sgpr(0x1.e8f434d018d63p-12));
    p = fma(p, z, in_sgpr(-0x1.e3074fde8871fp-8));
    p = fma(p, z, in_sgpr(0x1.50783487ee782p-4));
    p = fma(p, z, in_sgpr(-0x1.32d2cce62bd86p-1));
    p = fma(p, z, in_sgpr(0x1.466bc6775aae2p+1));
    p = fma(p, z, in_sgpr(-0x1.4abbce625be53p+2));
    p = fma(p, z, in_sgpr(0x1.1a62633145c07p-53));  // pi in two parts
    const double v = fma(y, 0x1.921fb54442d18p+1, y * p);
    return (int)k & 1 ? -v : v;
}

// Unit normal noise of site i of array j.
__device__ inline double vacuum_noise(unsigned long long i, unsigned j, uint2 key)
{
    const uint4 x = philox4x32_10(make_uint4((unsigned)i, (unsigned)(i >> 32), j, 0u), key);
    const double u1 = uniform53(x.x, x.y), u2 = uniform53(x.z, x.w);
    return sqrt_plain(-2.0 * log_unit(u1)) * cos_turn(u2);
}

// What a mode of the noise is multiplied by: the spectrum, and the 1/N^3 of
// the inverse transform.
struct VacuumFilter {
    double L, m2, eps2, cutoff, norm;
    int velocity;
    __device__ inline double operator()(int nx, int ny, int nz) const
    {
        const double nn = sqrt((double)nx * nx + (double)ny * ny + (double)nz * nz);
        if (!(nn > 0.0) || nn > cutoff) return 0.0;
        const double k = 2.0 * M_PI * nn / L;
        const double omega = sqrt(k * k + m2);
        const double P = velocity ? eps2 * omega / 2.0 : eps2 / (2.0 * omega);
        return norm * sqrt(P);
    }
};

__global__ void __launch_bounds__(256) k_vacuum_noise(double *out, long long N3, unsigned long long seed, int j)
{
    const uint2 key = make_uint2((unsigned)seed, (unsigned)(seed >> 32));
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (long long)gridDim.x * blockDim.x)
        out[i] = vacuum_noise((unsigned long long)i, (unsigned)j, key);
}

// Half-spectrum layout of D2Z: N x N x (N/2 + 1), last index fastest.
__global__ void __launch_bounds__(256) k_vacuum_filter(double2 *W, int N, VacuumFilter flt)
{
    const int NH = N / 2 + 1;
    const long long tot = (long long)N * N * NH;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < tot;
         idx += (long long)gridDim.x * blockDim.x) {
        const int kx = (int)(idx % NH);
        const long long t = idx / NH;
        const int ky = (int)(t % N), kz = (int)(t / N);
        const int ny = ky <= N / 2 ? ky : ky - N, nz = kz <= N / 2 ? kz : kz - N;
        const double f = flt(kx, ny, nz);
        double2 w = W[idx];
        w.x *= f;
        w.y *= f;
        W[idx] = w;
    }
}

__global__ void __launch_bounds__(256) k_add_const(double *a, long long N3, double c)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N3;
         i += (long long)gridDim.x * blockDim.x)
        a[i] = c + a[i];
}

int grid_of(long long n)
{
    const long long g = (n + 255) / 256;
    return (int)(g > 65536 ? 65536 : g);
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Both plans with caller-provided work areas; *work = the larger need.
int make_plans(int N, hipfftHandle *fwd, hipfftHandle *inv, size_t *work, char *msg, size_t len)
{
    *fwd = *inv = 0;
    size_t wf = 0, wi = 0;
    hipfftResult r = hipfftCreate(fwd);
    if (r == HIPFFT_SUCCESS) r = hipfftSetAutoAllocation(*fwd, 0);
    if (r == HIPFFT_SUCCESS) r = hipfftMakePlan3d(*fwd, N, N, N, HIPFFT_D2Z, &wf);
    if (r == HIPFFT_SUCCESS) r = hipfftCreate(inv);
    if (r == HIPFFT_SUCCESS) r = hipfftSetAutoAllocation(*inv, 0);
    if (r == HIPFFT_SUCCESS) r = hipfftMakePlan3d(*inv, N, N, N, HIPFFT_Z2D, &wi);
    if (r != HIPFFT_SUCCESS) {
        snprintf(msg, len, "hipFFT plan creation for %d^3 failed (hipfftResult %d)", N, (int)r);
        if (*fwd) (void)hipfftDestroy(*fwd);
        if (*inv) (void)hipfftDestroy(*inv);
        *fwd = *inv = 0;
        return 1;
    }
    *work = wf > wi ? wf : wi;
    return 0;
}

// The D2Z and Z2D plans of an N^3 lattice on one device.  Making a plan costs
// tens of milliseconds (hipFFT builds and compiles its kernels), several times
// the transforms themselves, so each (device, N) pair is planned once and kept
// until the process ends.  The plans own no work area (the caller's workspace
// is bound at each use), only host state and small twiddle tables.  Binding a
// stream and a work area and enqueuing the transforms must not interleave with
// another thread's use of the same plans: callers hold the returned lock until
// their transforms are enqueued.
struct Plans {
    hipfftHandle fwd = 0, inv = 0;
    size_t work = 0;
};

std::mutex g_plan_mu;

int cached_plans(int N, Plans *out, std::unique_lock<std::mutex> *lock, char *msg, size_t len)
{
    static std::map<std::pair<int, int>, Plans> cache;
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        snprintf(msg, len, "hipGetDevice: %s", hipGetErrorString(e));
        return 1;
    }
    std::unique_lock<std::mutex> g(g_plan_mu);
    auto it = cache.find({dev, N});
    if (it == cache.end()) {
        Plans p;
        if (make_plans(N, &p.fwd, &p.inv, &p.work, msg, len)) return 1;
        it = cache.emplace(std::make_pair(dev, N), p).first;
    }
    *out = it->second;
    if (lock) *lock = std::move(g);
    return 0;
}

// ---------------------------------------------------------------- spectra

// The shell floor(sqrt(r2) + 1/2): m with m^2 - m < r2 <= m^2 + m, from an FP32
// root set right by at most one.
__device__ inline int shell_of(int r2)
{
    const int m = (int)(__builtin_amdgcn_sqrtf((float)r2) + 0.5f), mm = m * m;
    return m + (r2 - mm > m) - (r2 - mm <= -m && r2 > 0);
}

// One step of the scan below: lanes that receive a value (CTRL: the DPP
// pattern, ROWS: the rows of 16 lanes it writes) of their own shell add it.
template <int CTRL, int ROWS>
__device__ inline void run_step(int key, double &p)
{
    const int ko = __builtin_amdgcn_update_dpp(-1, key, CTRL, ROWS, 0xf, false);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(p), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(p), CTRL, ROWS, 0xf, false);
    if (ko == key) p += __hiloint2double(hi, lo);
}

// Sums the runs of equal shells over a wave's lanes (shells non-decreasing
// across the lanes, so an equal shell at an earlier lane means that the whole
// stretch between belongs to the run) and adds each run to the wave's
// histogram from its last lane: one lane per shell, in a fixed order, without
// atomics.  The lanes exchange by DPP: a scan by LDS permutes was half of the
// z pass's time.
__device__ inline void scan_runs(int key, double &p)
{
    run_step<0x111, 0xf>(key, p);  // row_shr:1, 2, 4, 8 within 16 lanes
    run_step<0x112, 0xf>(key, p);
    run_step<0x114, 0xf>(key, p);
    run_step<0x118, 0xf>(key, p);
    run_step<0x142, 0xa>(key, p);  // row_bcast:15 into rows 1 and 3
    run_step<0x143, 0xc>(key, p);  // row_bcast:31 into rows 2 and 3
}

__device__ inline void add_runs(int key, double p, int nbins, double *hist)
{
    scan_runs(key, p);
    const int kn = __builtin_amdgcn_update_dpp(-1, key, 0x130, 0xf, 0xf, false);  // wave_shl:1
    if (kn != key && key < nbins) hist[key] += p;
}

// The same with two shells a lane, k0 <= k1: half the scans (with the shells
// from FP32 roots, the z pass of 512^3 0.56 -> 0.50 ms).  A lane whose
// shells differ ends the run of k0, to which the lanes before it may belong.
// No shell is written twice: a lane's k1 only if the next lane's k0 is another.
__device__ inline void add_runs2(int k0, double q0, int k1, double q1, int nbins, double *hist)
{
    const bool same = k0 == k1;
    double p = same ? q0 + q1 : q1;
    scan_runs(k1, p);
    const int kn = __builtin_amdgcn_update_dpp(-1, k0, 0x130, 0xf, 0xf, false);  // wave_shl:1
    const int kp = __builtin_amdgcn_update_dpp(-1, k1, 0x138, 0xf, 0xf, false);  // wave_shr:1
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(p), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(p), 0x138, 0xf, 0xf, false);
    if (!same && k0 < nbins) hist[k0] += kp == k0 ? q0 + __hiloint2double(hi, lo) : q0;
    if (kn != k1 && k1 < nbins) hist[k1] += p;
}

// One block of nw = blockDim.x / 64 waves per kz plane; wave w walks the rows
// ky = w, w + nw, ... and keeps its own LDS histogram.  F0: receives D_0.
__global__ void __launch_bounds__(512) k_spectrum_bins(const double2 *__restrict__ W, int N, int nbins,
                                                       double *__restrict__ part, double *F0)
{
    extern __shared__ double hist[];  // [wave][nbins]
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, nw = blockDim.x >> 6;
    double *hp = hist + (size_t)wv * nbins;
    for (int b = t; b < nw * nbins; b += blockDim.x) hist[b] = 0.0;
    __syncthreads();
    const int NH = N / 2 + 1, kz = blockIdx.x;
    if (kz == 0 && t == 0) *F0 = W[0].x;
    const int nz = kz <= N / 2 ? kz : kz - N;
    for (int ky = wv; ky < N; ky += nw) {
        const int ny = ky <= N / 2 ? ky : ky - N;
        const int r2 = ny * ny + nz * nz;
        const double2 *row = W + ((size_t)kz * N + ky) * NH;
        for (int x0 = 0; x0 < NH; x0 += 64) {
            const int kx = x0 + lane;
            int key = 0x7fffffff;
            double p = 0.0;
            if (kx < NH) {
                key = shell_of(r2 + kx * kx);
                const double w = (kx == 0 || 2 * kx == N) ? 1.0 : 2.0;
                const double2 v = row[kx];
                p = w * (v.x * v.x + v.y * v.y);
            }
            add_runs(key, p, nbins, hp);
        }
    }
    __syncthreads();
    for (int b = t; b < nbins; b += blockDim.x) {
        double P = 0.0;
        for (int w = 0; w < nw; ++w) P += hist[(size_t)w * nbins + b];
        part[(size_t)blockIdx.x * nbins + b] = P;
    }
}

// Modes per shell, from one octant with weights (cnt cleared before): whole
// numbers, so the order of the atomics does not matter.
__global__ void __launch_bounds__(256) k_shell_count(int N, int nbins, unsigned long long *cnt)
{
    extern __shared__ unsigned int hc[];
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) hc[b] = 0;
    __syncthreads();
    const int H = N / 2 + 1, nz = blockIdx.x;
    auto weight = [N](int n) { return (n == 0 || 2 * n == N) ? 1u : 2u; };
    for (int i = threadIdx.x; i < H * H; i += blockDim.x) {
        const int ny = i / H, nx = i - ny * H;
        const int key = shell_of((long long)nz * nz + (long long)ny * ny + (long long)nx * nx);
        if (key < nbins) atomicAdd(&hc[key], weight(nx) * weight(ny) * weight(nz));
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += blockDim.x)
        if (hc[b]) atomicAdd(&cnt[b], (unsigned long long)hc[b]);
}

// Clears the counts and, with tw, fills exp(-2 pi i n/N), n < N.
__global__ void __launch_bounds__(256) k_fft_setup(double2 *tw, int N, unsigned long long *cnt, int nbins)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (tw && i < N) {
        double sn, cs;
        sincospi(2.0 * (double)i / (double)N, &sn, &cs);
        tw[i] = make_double2(cs, -sn);
    }
    if (i < nbins) cnt[i] = 0;
}

// 64 bins per block; the block's 16 waves each add every 16th partial row in
// row order, then wave 0 adds the 16 wave sums in wave order.  Shell 0 is the
// n = 0 mode alone: F_0 = N^3 bg + D_0 (real), bg the homogeneous value at
// the synchronised time.
__global__ void __launch_bounds__(1024) k_spectrum_final(const double *__restrict__ part, int nblk, int nbins,
                                                         double scale, const double *__restrict__ F0,
                                                         const unsigned long long *__restrict__ cnt,
                                                         const DevScalars *__restrict__ S, int fld, int velocity,
                                                         double h, double n3, double *out)
{
    __shared__ double sp[16][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int b = blockIdx.x * 64 + lane;
    double P = 0.0;
    if (b < nbins)
        for (int j = g; j < nblk; j += 16) P += part[(size_t)j * nbins + b];
    sp[g][lane] = P;
    __syncthreads();
    if (g != 0 || b >= nbins) return;
    P = 0.0;
    for (int w = 0; w < 16; ++w) P += sp[w][lane];
    if (b == 0) {
        const double bg = velocity ? S->bg_v[fld] : S->bg_f[fld] - h * S->bg_v[fld];
        const double f0 = n3 * bg + *F0;
        P = f0 * f0;
    }
    const double C = (double)cnt[b];
    out[b] = C > 0.0 ? P / C * scale : 0.0;
    out[nbins + b] = C;
}

// ---------------------------------------------------------------- line passes

// Waves per SIMD the passes are compiled for: two blocks of 512 threads per CU
// with the butterflies of 2, 4 and 8 points; those of 3, 5 and 7 need more
// registers.  In blocks of 1024 threads, where four waves are all there can be,
// they spill 57 to 70 of them.
constexpr int fft_waves(int nt, bool exact) { return exact || nt == 1024 ? 4 : 2; }

// Lines per block and threads of the passes over N-point lines: B 16-byte
// columns make the memory segments of the y and z passes (128 bytes and more up
// to N = 1024), and N B points of LDS let two blocks share a CU up to N = 512.
template <typename F>
void with_fft_tile(int N, F &&f)
{
    using std::integral_constant;
    auto go = [&](auto b, auto nt) {
        if (N * (int)b == kFftPts * (int)nt && (N & (N - 1)) == 0) f(b, nt, std::true_type{});
        else f(b, nt, std::false_type{});
    };
    if (N <= 128) go(integral_constant<int, 16>{}, integral_constant<int, 256>{});
    else if (N <= 256) go(integral_constant<int, 16>{}, integral_constant<int, 512>{});
    else if (N <= 512) go(integral_constant<int, 8>{}, integral_constant<int, 512>{});
    else if (N <= 1024) go(integral_constant<int, 8>{}, integral_constant<int, 1024>{});
    else go(integral_constant<int, 4>{}, integral_constant<int, 1024>{});
}

int fft_tile_b(int N) { return N <= 256 ? 16 : (N <= 1024 ? 8 : 4); }

// Half spectrum of the passes: element (kx, y, z) at (z N + y) NS + kx, kx < nk
// (the modes kept), rows padded to whole column tiles.
int fft_stride(int N, int nk)
{
    const int b = fft_tile_b(N);
    return (nk + b - 1) / b * b;
}

// Sources of the x pass.  kLoads: read from memory, four(i, v) gives the values of
// four sites from i; otherwise computed, operator()(i) gives that of site i.
template <typename T>
struct SyncSource {  // synchronised deviation of a field, or a velocity's deviation
    static constexpr bool kLoads = true;
    const T *d, *e;
    double h;
    int velocity;
    __device__ inline double value(T dv, T ev) const { return velocity ? (double)ev : (double)dv - h * (double)ev; }
    // four consecutive elements from i, a multiple of four (the arrays start
    // on 256 bytes)
    __device__ inline void four(long long i, double (&v)[4]) const
    {
        typedef T V4 __attribute__((ext_vector_type(4)));
        const V4 ev = *(const V4 *)(e + i);
        const V4 dv = velocity ? ev : *(const V4 *)(d + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = value(dv[k], ev[k]);
    }
};

struct NoiseSource {
    static constexpr bool kLoads = false;
    uint2 key;
    unsigned j;
    __device__ inline double operator()(long long i) const
    {
        return vacuum_noise((unsigned long long)i, j, key);
    }
};

// x pass: 2 B rows of the source per block, two through each complex line
// (a + i b); modes kx < nk of every row into W.
template <int B, int NT, bool EXACT, typename Src>
__global__ void __launch_bounds__(NT, fft_waves(NT, EXACT)) k_fft_x(const Src src, FftPlan pl, const double2 *__restrict__ tw,
                                                       double2 *__restrict__ W, int nk, int NS)
{
    extern __shared__ double2 s[];
    const int N = pl.N, t = threadIdx.x;
    const long long rows = (long long)N * N, r0 = (long long)blockIdx.x * 2 * B;
    double *sd = (double *)s;
    if constexpr (!Src::kLoads) {
        // bound by the arithmetic of the source: one element at a time
        const float inv = 1.0f / (float)N;
#pragma unroll 1
        for (int i = t; i < 2 * B * N; i += NT) {
            const int rl = div_by(i, inv);
            sd[2 * fft_slot<B>(i - rl * N, rl >> 1) + (rl & 1)] = r0 + rl < rows ? src(r0 * N + i) : 0.0;
        }
    } else if constexpr (EXACT) {
        // four elements a thread and row: all of a block's loads in flight
        constexpr int G = kFftPts / 2;
        const int l4 = 29 - __clz(N);  // log2(N / 4)
        double v[G][4];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = t + NT * g, rl = i >> l4, x = (i - (rl << l4)) * 4;
            src.four((r0 + rl) * N + x, v[g]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = t + NT * g, rl = i >> l4, x = (i - (rl << l4)) * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) sd[2 * fft_slot<B>(x + k, rl >> 1) + (rl & 1)] = v[g][k];
        }
    } else {
        static_assert(EXACT || !Src::kLoads, "rows of memory come in fours");
    }
    __syncthreads();
    fft_lines<B, NT, EXACT>(s, pl, tw);
    const float inv = 1.0f / (float)nk;
#pragma unroll
    for (int u = 0; u < kFftPts / 2 + 1; ++u) {  // B nk <= B (N/2 + 1) <= (4 + 1) NT
        const int i = t + NT * u, c = div_by(i, inv), k = i - c * nk;
        if (c >= B) break;
        const double2 p = s[fft_slot<B>(k, c)], q = s[fft_slot<B>(k ? N - k : 0, c)];
        const long long r = r0 + 2 * c;
        if (r < rows) W[r * NS + k] = make_double2(0.5 * (p.x + q.x), 0.5 * (p.y - q.y));
        if (r + 1 < rows) W[(r + 1) * NS + k] = make_double2(0.5 * (p.y + q.y), 0.5 * (q.x - p.x));
    }
}

// Inverse x pass: B pairs of rows of W back to real rows of out, plus c.
template <int B, int NT, bool EXACT>
__global__ void __launch_bounds__(NT, fft_waves(NT, EXACT)) k_fft_x_inv(const double2 *__restrict__ W, FftPlan pl,
                                                           const double2 *__restrict__ tw, double *__restrict__ out,
                                                           int nk, int NS, double add)
{
    extern __shared__ double2 s[];
    const int N = pl.N, t = threadIdx.x;
    const long long rows = (long long)N * N, r0 = (long long)blockIdx.x * 2 * B;
    // the modes that were not kept
    const int gap = N - 2 * nk + 1;  // n = nk .. N - nk
    for (int i = t; i < gap * B; i += NT) s[fft_slot<B>(nk + i / B, i % B)] = make_double2(0.0, 0.0);
    constexpr int U = kFftPts / 2 + 1;  // as in the x pass
    const float inv = 1.0f / (float)nk;
    double2 va[U], vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = t + NT * u, c = div_by(i, inv), k = i - c * nk;
        const long long r = r0 + 2 * c;
        va[u] = (c < B && r < rows) ? W[r * NS + k] : make_double2(0.0, 0.0);
        vb[u] = (c < B && r + 1 < rows) ? W[(r + 1) * NS + k] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = t + NT * u, c = div_by(i, inv), k = i - c * nk;
        if (c >= B) break;
        const double2 a = va[u], b = vb[u];
        // swapped parts (inverse); modes 0 and N/2 of a real row are real
        if (k == 0 || 2 * k == N) {
            s[fft_slot<B>(k, c)] = make_double2(b.x, a.x);
        } else {
            s[fft_slot<B>(k, c)] = make_double2(a.y + b.x, a.x - b.y);
            s[fft_slot<B>(N - k, c)] = make_double2(b.x - a.y, a.x + b.y);
        }
    }
    __syncthreads();
    fft_lines<B, NT, EXACT>(s, pl, tw);
    const double *sd = (const double *)s;
    if constexpr (EXACT) {
        typedef double V2 __attribute__((ext_vector_type(2)));
        const int l2 = 30 - __clz(N);  // log2(N / 2)
#pragma unroll
        for (int u = 0; u < kFftPts; ++u) {
            const int i = t + NT * u, rl = i >> l2, x = (i - (rl << l2)) * 2, part = 1 - (rl & 1);
            const V2 v = {add + sd[2 * fft_slot<B>(x, rl >> 1) + part],
                          add + sd[2 * fft_slot<B>(x + 1, rl >> 1) + part]};
            __builtin_nontemporal_store(v, (V2 *)(out + (r0 + rl) * N + x));
        }
    } else {
        const float invn = 1.0f / (float)N;
        for (int i = t; i < 2 * B * N; i += NT) {
            const int rl = div_by(i, invn);
            if (r0 + rl < rows)
                __builtin_nontemporal_store(add + sd[2 * fft_slot<B>(i - rl * N, rl >> 1) + 1 - (rl & 1)],
                                            out + r0 * N + i);
        }
    }
}

// Which columns (kx, ky) hold a mode that is kept: |n| <= cutoff for some kz.
struct Kept {
    double cutoff;
    __device__ inline bool operator()(int kx, int ny) const
    {
        return !(sqrt((double)kx * kx + (double)ny * ny) > cutoff);
    }
};

// y pass, in place: B columns of one z plane per block.  INV: the inverse;
// columns that are not kept are not stored by the forward pass and count as
// zero in the inverse one.
template <int B, int NT, bool EXACT, bool INV>
__global__ void __launch_bounds__(NT, fft_waves(NT, EXACT)) k_fft_y(double2 *__restrict__ W, FftPlan pl,
                                                       const double2 *__restrict__ tw, int nk, int NS, int ntile,
                                                       Kept kept)
{
    extern __shared__ double2 s[];
    const int N = pl.N, t = threadIdx.x;
    const int z = blockIdx.x / ntile, kx0 = (blockIdx.x - z * ntile) * B;
    double2 *p = W + (long long)z * N * NS + kx0;
    const int c = t % B;  // 256 is a multiple of B
    const bool live = kx0 + c < nk;
    auto ok = [&](int y) { return kept(kx0 + c, y <= N / 2 ? y : y - N); };
    double2 v[kFftPts];
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int y = (t + NT * u) / B;
        v[u] = (live && y < N && (!INV || ok(y))) ? p[(long long)y * NS + c] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int y = (t + NT * u) / B;
        if (y < N) s[fft_slot<B>(y, c)] = INV ? make_double2(v[u].y, v[u].x) : v[u];
    }
    __syncthreads();
    fft_lines<B, NT, EXACT>(s, pl, tw);
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int y = (t + NT * u) / B;
        if (!live || y >= N || (!INV && !ok(y))) continue;
        const double2 q = s[fft_slot<B>(y, c)];
        p[(long long)y * NS + c] = INV ? make_double2(q.y, q.x) : q;
    }
}

// z pass of the vacuum state, in place: forward transform, filter, inverse
// transform of B columns per block.  ky runs over the nky rows with
// |ny| <= nk - 1.
template <int B, int NT, bool EXACT>
__global__ void __launch_bounds__(NT, fft_waves(NT, EXACT)) k_fft_z_filter(double2 *__restrict__ W, FftPlan pl,
                                                              const double2 *__restrict__ tw, int nk, int NS,
                                                              int ntile, int nky, Kept kept, VacuumFilter flt)
{
    extern __shared__ double2 s[];
    const int N = pl.N, t = threadIdx.x;
    const int j = blockIdx.x / ntile, kx0 = (blockIdx.x - j * ntile) * B;
    const int ky = j < nk ? j : N - nky + j;
    const int ny = ky <= N / 2 ? ky : ky - N;
    const int c = t % B;
    if (!kept(kx0, ny)) return;  // the whole tile: its columns grow in |n| with kx
    const bool live = kx0 + c < nk && kept(kx0 + c, ny);
    double2 *p = W + (long long)ky * NS + kx0;
    const long long plane = (long long)N * NS;
    double2 v[kFftPts];
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int z = (t + NT * u) / B;
        v[u] = (live && z < N) ? p[z * plane + c] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int z = (t + NT * u) / B;
        if (z < N) s[fft_slot<B>(z, c)] = v[u];
    }
    __syncthreads();
    fft_lines<B, NT, EXACT>(s, pl, tw);
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int z = (t + NT * u) / B;
        if (z >= N) continue;
        const double f = flt(kx0 + c, ny, z <= N / 2 ? z : z - N);
        const double2 q = s[fft_slot<B>(z, c)];
        s[fft_slot<B>(z, c)] = make_double2(q.y * f, q.x * f);
    }
    __syncthreads();
    fft_lines<B, NT, EXACT>(s, pl, tw);
#pragma unroll
    for (int u = 0; u < kFftPts; ++u) {
        const int z = (t + NT * u) / B;
        if (!live || z >= N) continue;
        const double2 q = s[fft_slot<B>(z, c)];
        p[z * plane + c] = make_double2(q.y, q.x);
    }
}

// z pass of the spectrum: transforms B columns at a time and sums their
// shells from LDS.  The grid walks the items (ky, column tile) in a fixed
// order, so the block partials are reproducible.  The modes kz and -kz of a
// column lie on one shell and are added first; along kz the shells do not
// decrease.  nh waves sum, each into its own histogram (as many as fit in the
// LDS).
template <int B, int NT, bool EXACT>
__global__ void __launch_bounds__(NT, fft_waves(NT, EXACT)) k_fft_z_bins(const double2 *__restrict__ W, FftPlan pl,
                                                            const double2 *__restrict__ tw, int nk, int NS, int ntile,
                                                            int nbins, int nh, double *__restrict__ part, double *F0)
{
    extern __shared__ double2 s[];
    const int N = pl.N, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    double *hist = (double *)(s + (size_t)N * B);  // [wave][nbins]
    for (int b = t; b < nh * nbins; b += NT) hist[b] = 0.0;
    const int HP = (N + 1) / 2, c = t % B;  // kz of which kz and -kz both occur, and 0
    const long long plane = (long long)N * NS;
    double2 v[kFftPts];
    auto load = [&](int item) {
        const int ky = item / ntile, kx0 = (item - ky * ntile) * B;
        const double2 *p = W + (long long)ky * NS + kx0;
#pragma unroll
        for (int u = 0; u < kFftPts; ++u) {
            const int z = (t + NT * u) / B;
            v[u] = (kx0 + c < nk && z < N) ? p[z * plane + c] : make_double2(0.0, 0.0);
        }
    };
    if ((int)blockIdx.x < N * ntile) load(blockIdx.x);
    for (int item = blockIdx.x; item < N * ntile; item += gridDim.x) {
        const int ky = item / ntile, kx0 = (item - ky * ntile) * B;
#pragma unroll
        for (int u = 0; u < kFftPts; ++u) {
            const int z = (t + NT * u) / B;
            if (z < N) s[fft_slot<B>(z, c)] = v[u];
        }
        __syncthreads();
        fft_lines<B, NT, EXACT>(s, pl, tw);
        // the next item's columns on their way while this one's are summed
        if (item + (int)gridDim.x < N * ntile) load(item + gridDim.x);
        if (item == 0 && t == 0) *F0 = s[fft_slot<B>(0, 0)].x;
        if (wv < nh) {
            const int ny = ky <= N / 2 ? ky : ky - N;
            double *hp = hist + (size_t)wv * nbins;
            for (int cc = wv; cc < B && kx0 + cc < nk; cc += nh) {
                const int kx = kx0 + cc, r2 = kx * kx + ny * ny;
                const double w = (kx == 0 || 2 * kx == N) ? 1.0 : 2.0;
                auto power = [&](int kz) {
                    const double2 a = s[fft_slot<B>(kz, cc)], b = s[fft_slot<B>(kz ? N - kz : 0, cc)];
                    const double q = a.x * a.x + a.y * a.y;
                    return w * (kz ? q + (b.x * b.x + b.y * b.y) : q);
                };
                for (int z0 = 0; z0 < HP; z0 += 128) {
                    const int kz = z0 + 2 * lane;
                    int k0 = 0x7fffffff, k1 = 0x7fffffff;
                    double q0 = 0.0, q1 = 0.0;
                    if (kz < HP) {
                        // eight lanes the even one first, eight the odd one: all banks
                        const bool odd = (lane & 8) && kz + 1 < HP;
                        k0 = shell_of(r2 + kz * kz);
                        q0 = power(kz + odd);
                        if (kz + 1 < HP) {
                            k1 = shell_of(r2 + (kz + 1) * (kz + 1));
                            q1 = power(kz + !odd);
                        }
                        const double x = odd ? q1 : q0;
                        q1 = odd ? q0 : q1;
                        q0 = x;
                    }
                    add_runs2(k0, q0, k1, q1, nbins, hp);
                }
            }
            if (wv == 0 && 2 * HP == N) {  // N even: kz = N/2 of the tile's columns
                const int kx = kx0 + lane;
                int key = 0x7fffffff;
                double q = 0.0;
                if (lane < B && kx < nk) {
                    key = shell_of(kx * kx + ny * ny + HP * HP);
                    const double2 a = s[fft_slot<B>(HP, lane)];
                    q = ((kx == 0 || 2 * kx == N) ? 1.0 : 2.0) * (a.x * a.x + a.y * a.y);
                }
                add_runs(key, q, nbins, hp);
            }
        }
        __syncthreads();
    }
    __syncthreads();
    for (int b = t; b < nbins; b += NT) {
        double P = 0.0;
        for (int w = 0; w < nh; ++w) P += hist[(size_t)w * nbins + b];
        part[(size_t)blockIdx.x * nbins + b] = P;
    }
}

template <typename K>
hipError_t fft_lds(K *kernel, size_t bytes)
{
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

constexpr size_t kLdsOfCu = 160 * 1024;

// Blocks of the spectrum's z pass: two per CU.
constexpr int kBinBlocks = 512;

}  // namespace

int spectrum_bins(int N)
{
    const int h = N / 2;
    return (int)floor(sqrt(3.0 * h * h) + 0.5) + 1;
}

namespace {

// Sizes that go through the line passes; the others through hipFFT.  Both ways
// measured (spectra of four fields; the whole vacuum state; us; library -> own):
//   powers of two from 128: 128^3 667 -> 518 and 497 -> 301, 256^3 1775 -> 1140
//     and 2590 -> 1010, 512^3 11090 -> 6400 and 22150 -> 7070, 1024^3 108 -> 58 ms
//     and 222 -> 71 ms;
//   factors of 3, 5 and 7: vacuum at the default cutoff 100^3 393 -> 300, 144^3
//     640 -> 628, 210^3 1876 -> 1344, 270^3 3109 -> 3268 (the one that is slower of 47
//     from 96 to 1000), 400^3 13360 -> 6980, 600^3 46.4 -> 34.4 ms, 768^3 97 -> 50,
//     1000^3 218 -> 117.  With all modes kept even sizes with few factors are up to
//     1.7 times slower (200^3 1307 -> 1571, 270^3 3126 -> 5197, 540^3 29.2 -> 47.7 ms,
//     600^3 46.4 -> 62.0), but the library first plans for 1.6 to 2.0 s per size and
//     process, which is hundreds to thousands of such calls.  Spectra were not
//     faster: 200^3 980 -> 1138, 400^3 6965 -> 7269;
//   small: 64^3 370 -> 410 and 176 -> 196 (few blocks, as many launches).
bool spectrum_own(int N) { return N >= 128 && (N & (N - 1)) == 0; }
bool vacuum_own(int N) { return N >= 96 && fft_plan(N).stages > 0; }

}  // namespace

namespace {

// Workspace of the spectrum: [twiddles][half spectrum][FFT work area, field]
// [partial rows][counts][result, D_0]; work: hipFFT's need, 0 for the line
// passes.
struct SpectrumLayout {
    size_t tw, W, work, field, part, cnt, out, total;
    int rows;
};

SpectrumLayout spectrum_layout(int N, bool own, size_t work)
{
    SpectrumLayout L{};
    const size_t nb = spectrum_bins(N);
    L.rows = own ? kBinBlocks : N;
    size_t off = 0;
    L.tw = off; off += own ? align256((size_t)N * sizeof(double2)) : 0;
    L.W = off; off += own ? align256((size_t)N * N * fft_stride(N, N / 2 + 1) * sizeof(double2))
                          : vacuum_spectrum_bytes(N);
    L.work = off; off += align256(work);
    L.field = off; off += own ? 0 : align256((size_t)N * N * N * sizeof(double));
    L.part = off; off += align256((size_t)L.rows * nb * sizeof(double));
    L.cnt = off; off += align256(nb * sizeof(unsigned long long));
    L.out = off; off += align256((2 * nb + 1) * sizeof(double));
    L.total = off;
    return L;
}

// x, y and z pass of the spectrum.
template <typename T>
hipError_t spectrum_passes(int N, const SyncSource<T> &src, int nbins, hipStream_t st, const double2 *tw, double2 *W,
                           double *part, int *nblk, double *F0)
{
    const FftPlan pl = fft_plan(N);
    const int nk = N / 2 + 1, NS = fft_stride(N, nk);
    hipError_t e = hipSuccess;
    with_fft_tile(N, [&](auto b, auto nt, auto ex) {
        constexpr int B = decltype(b)::value, NT = decltype(nt)::value;
        constexpr bool EXACT = true;  // spectrum_own
        if constexpr (decltype(ex)::value) {
            const size_t lds = (size_t)N * B * sizeof(double2);
            const int ntile = (nk + B - 1) / B;
            int nh = 4;
            while (nh > 1 && lds + (size_t)nh * nbins * sizeof(double) > kLdsOfCu) nh >>= 1;
            const size_t lds_z = lds + (size_t)nh * nbins * sizeof(double);
            const int items = N * ntile;
            *nblk = items < kBinBlocks ? items : kBinBlocks;
            if ((e = fft_lds(k_fft_x<B, NT, EXACT, SyncSource<T>>, lds)) != hipSuccess) return;
            if ((e = fft_lds(k_fft_y<B, NT, EXACT, false>, lds)) != hipSuccess) return;
            if ((e = fft_lds(k_fft_z_bins<B, NT, EXACT>, lds_z)) != hipSuccess) return;
            const long long rows = (long long)N * N;
            hipLaunchKernelGGL((k_fft_x<B, NT, EXACT, SyncSource<T>>), dim3((unsigned)((rows + 2 * B - 1) / (2 * B))),
                               dim3(NT), lds, st, src, pl, tw, W, nk, NS);
            hipLaunchKernelGGL((k_fft_y<B, NT, EXACT, false>), dim3(N * ntile), dim3(NT), lds, st, W, pl, tw, nk, NS,
                               ntile, Kept{1e300});
            hipLaunchKernelGGL((k_fft_z_bins<B, NT, EXACT>), dim3(*nblk), dim3(NT), lds_z, st, W, pl, tw, nk, NS,
                               ntile, nbins, nh, part, F0);
            e = hipGetLastError();
        }
    });
    return e;
}

}  // namespace

size_t vacuum_spectrum_bytes(int N) { return align256((size_t)N * N * (N / 2 + 1) * sizeof(double2)); }

int spectrum_workspace_bytes(int N, size_t *bytes, char *msg, size_t len)
{
    Plans pl;
    const bool own = spectrum_own(N);
    if (!own && cached_plans(N, &pl, nullptr, msg, len)) return 1;
    *bytes = spectrum_layout(N, own, pl.work).total;
    return 0;
}

int spectrum_compute(int N, double L, int dtype, const void *d, const void *ev, const DevScalars *S, int fld,
                     int velocity, double h, int nbins, hipStream_t st, void *ws, size_t ws_bytes, double *power,
                     double *count, char *msg, size_t len)
{
    Plans pl;
    std::unique_lock<std::mutex> lock;
    const bool own = spectrum_own(N);
    if (!own && cached_plans(N, &pl, &lock, msg, len)) return 1;
    const SpectrumLayout lay = spectrum_layout(N, own, pl.work);
    if (ws_bytes < lay.total) {
        snprintf(msg, len, "spectrum workspace of %zu bytes, %zu needed", ws_bytes, lay.total);
        return 2;
    }
    char *w = (char *)ws;
    double2 *tw = (double2 *)(w + lay.tw), *W = (double2 *)(w + lay.W);
    double *part = (double *)(w + lay.part), *out = (double *)(w + lay.out), *F0 = out + 2 * (size_t)nbins;
    unsigned long long *cnt = (unsigned long long *)(w + lay.cnt);
    const int setup = (N > nbins ? N : nbins);
    hipLaunchKernelGGL(k_fft_setup, dim3((setup + 255) / 256), dim3(256), 0, st, own ? tw : nullptr, N, cnt, nbins);
    hipLaunchKernelGGL(k_shell_count, dim3(N / 2 + 1), dim3(256), (size_t)nbins * sizeof(unsigned int), st, N, nbins,
                       cnt);
    hipError_t e = hipGetLastError();
    int nblk = N, rc = 0;
    if (own) {
        if (e == hipSuccess && dtype == 0)
            e = spectrum_passes(N, SyncSource<float>{(const float *)d, (const float *)ev, h, velocity}, nbins, st, tw,
                                W, part, &nblk, F0);
        else if (e == hipSuccess)
            e = spectrum_passes(N, SyncSource<double>{(const double *)d, (const double *)ev, h, velocity}, nbins, st,
                                tw, W, part, &nblk, F0);
    } else {
        double *field = (double *)(w + lay.field);
        launch_sync_deviation(dtype, d, ev, field, N, h, velocity, st);
        hipfftResult r = hipfftSetStream(pl.fwd, st);
        if (r == HIPFFT_SUCCESS) r = hipfftSetWorkArea(pl.fwd, w + lay.work);
        if (r == HIPFFT_SUCCESS) r = hipfftExecD2Z(pl.fwd, (hipfftDoubleReal *)field, (hipfftDoubleComplex *)W);
        lock.unlock();
        if (r != HIPFFT_SUCCESS) {
            snprintf(msg, len, "hipFFT execution failed (hipfftResult %d)", (int)r);
            rc = 1;
        } else if (e == hipSuccess) {
            // 8 waves per block (two blocks per CU at 512^3) while their
            // histograms fit in 64 KB of LDS, else 4
            const int nw = (size_t)8 * 8 * nbins <= 65536 ? 8 : 4;
            const size_t lds = (size_t)nw * nbins * sizeof(double);
            e = fft_lds(k_spectrum_bins, lds);
            if (e == hipSuccess) {
                hipLaunchKernelGGL(k_spectrum_bins, dim3(N), dim3(64 * nw), lds, st, W, N, nbins, part, F0);
                e = hipGetLastError();
            }
        }
    }
    if (!rc && e == hipSuccess) {
        const double n3 = (double)N * N * N;
        hipLaunchKernelGGL(k_spectrum_final, dim3((nbins + 63) / 64), dim3(1024), 0, st, part, nblk, nbins,
                           L * L * L / (n3 * n3), F0, cnt, S, fld, velocity, h, n3, out);
        e = hipGetLastError();
    }
    if (!rc && e == hipSuccess) e = hipMemcpyAsync(power, out, nbins * sizeof(double), hipMemcpyDeviceToHost, st);
    if (!rc && e == hipSuccess)
        e = hipMemcpyAsync(count, out + nbins, nbins * sizeof(double), hipMemcpyDeviceToHost, st);
    const hipError_t es = hipStreamSynchronize(st);
    if (e == hipSuccess) e = es;
    if (!rc && e != hipSuccess) {
        snprintf(msg, len, "spectrum: %s", hipGetErrorString(e));
        rc = 1;
    }
    return rc;
}

namespace {

// Workspace of the vacuum generator: [twiddles][half spectrum], or
// [half spectrum][hipFFT's work area].
size_t vacuum_bytes(int N, bool own, size_t work)
{
    return own ? align256((size_t)N * sizeof(double2)) +
                     align256((size_t)N * N * fft_stride(N, N / 2 + 1) * sizeof(double2))
               : vacuum_spectrum_bytes(N) + align256(work);
}

// One array through the line passes.
hipError_t vacuum_passes(int N, const NoiseSource &src, const VacuumFilter &flt, double add, hipStream_t st,
                         const double2 *tw, double2 *W, double *out)
{
    const FftPlan pl = fft_plan(N);
    const int half = N / 2, kc = flt.cutoff < half ? (int)flt.cutoff : half;  // largest |n_i| kept
    const int nk = kc + 1, NS = fft_stride(N, nk), nky = 2 * kc + 1 < N ? 2 * kc + 1 : N;
    hipError_t e = hipSuccess;
    with_fft_tile(N, [&](auto b, auto nt, auto ex) {
        constexpr int B = decltype(b)::value, NT = decltype(nt)::value;
        constexpr bool EXACT = decltype(ex)::value;
        const size_t lds = (size_t)N * B * sizeof(double2);
        const int ntile = (nk + B - 1) / B;
        if ((e = fft_lds(k_fft_x<B, NT, EXACT, NoiseSource>, lds)) != hipSuccess) return;
        if ((e = fft_lds(k_fft_y<B, NT, EXACT, false>, lds)) != hipSuccess) return;
        if ((e = fft_lds(k_fft_y<B, NT, EXACT, true>, lds)) != hipSuccess) return;
        if ((e = fft_lds(k_fft_z_filter<B, NT, EXACT>, lds)) != hipSuccess) return;
        if ((e = fft_lds(k_fft_x_inv<B, NT, EXACT>, lds)) != hipSuccess) return;
        const long long rows = (long long)N * N;
        const dim3 gx((unsigned)((rows + 2 * B - 1) / (2 * B))), tb(NT);
        const Kept kept{flt.cutoff};
        hipLaunchKernelGGL((k_fft_x<B, NT, EXACT, NoiseSource>), gx, tb, lds, st, src, pl, tw, W, nk, NS);
        hipLaunchKernelGGL((k_fft_y<B, NT, EXACT, false>), dim3(N * ntile), tb, lds, st, W, pl, tw, nk, NS, ntile, kept);
        hipLaunchKernelGGL((k_fft_z_filter<B, NT, EXACT>), dim3(nky * ntile), tb, lds, st, W, pl, tw, nk, NS, ntile, nky,
                           kept, flt);
        hipLaunchKernelGGL((k_fft_y<B, NT, EXACT, true>), dim3(N * ntile), tb, lds, st, W, pl, tw, nk, NS, ntile, kept);
        hipLaunchKernelGGL((k_fft_x_inv<B, NT, EXACT>), gx, tb, lds, st, W, pl, tw, out, nk, NS, add);
        e = hipGetLastError();
    });
    return e;
}

}  // namespace

int vacuum_workspace(int N, size_t *bytes, char *msg, size_t len)
{
    Plans pl;
    const bool own = vacuum_own(N);
    if (!own && cached_plans(N, &pl, nullptr, msg, len)) return 1;
    *bytes = vacuum_bytes(N, own, pl.work);
    return 0;
}

int vacuum_generate(int N, double L, const lf_vacuum *v, hipStream_t st, void *ws, size_t ws_bytes,
                    double *const out[4], char *msg, size_t len)
{
    Plans pl;
    std::unique_lock<std::mutex> lock;
    const bool own = vacuum_own(N);
    if (!own && cached_plans(N, &pl, &lock, msg, len)) return 1;
    const size_t need = vacuum_bytes(N, own, pl.work);
    if (ws_bytes < need) {
        snprintf(msg, len, "vacuum workspace of %zu bytes, %zu needed", ws_bytes, need);
        return 2;
    }
    const long long N3 = (long long)N * N * N;
    const double n3 = (double)N * N * N;
    VacuumFilter flt{L, 0.0, v->eps2, v->cutoff > 0.0 ? v->cutoff : N / 4.0, sqrt(n3 / (L * L * L)) / n3, 0};
    hipError_t e = hipSuccess;
    hipfftResult r = HIPFFT_SUCCESS;
    double2 *W = (double2 *)((char *)ws + (own ? align256((size_t)N * sizeof(double2)) : 0));
    if (own) {
        hipLaunchKernelGGL(k_fft_setup, dim3((N + 255) / 256), dim3(256), 0, st, (double2 *)ws, N,
                           (unsigned long long *)nullptr, 0);
        e = hipGetLastError();
    } else {
        void *wk = (char *)ws + vacuum_spectrum_bytes(N);
        r = hipfftSetStream(pl.fwd, st);
        if (r == HIPFFT_SUCCESS) r = hipfftSetStream(pl.inv, st);
        if (r == HIPFFT_SUCCESS) r = hipfftSetWorkArea(pl.fwd, wk);
        if (r == HIPFFT_SUCCESS) r = hipfftSetWorkArea(pl.inv, wk);
    }
    for (int j = 0; j < 4 && r == HIPFFT_SUCCESS && e == hipSuccess; ++j) {
        const int fld = j & 1;  // f1, f2, u1, u2
        const int vel = j >> 1;
        const double add = vel ? v->u0[fld] : v->f0[fld];
        flt.m2 = v->m2[fld];
        flt.velocity = vel;
        if (own) {
            const NoiseSource src{make_uint2((unsigned)v->seed, (unsigned)(v->seed >> 32)), (unsigned)j};
            e = vacuum_passes(N, src, flt, add, st, (const double2 *)ws, W, out[j]);
            continue;
        }
        hipLaunchKernelGGL(k_vacuum_noise, dim3(grid_of(N3)), dim3(256), 0, st, out[j], N3,
                           (unsigned long long)v->seed, j);
        r = hipfftExecD2Z(pl.fwd, (hipfftDoubleReal *)out[j], (hipfftDoubleComplex *)W);
        if (r != HIPFFT_SUCCESS) break;
        hipLaunchKernelGGL(k_vacuum_filter, dim3(grid_of((long long)N * N * (N / 2 + 1))), dim3(256), 0, st, W, N,
                           flt);
        r = hipfftExecZ2D(pl.inv, (hipfftDoubleComplex *)W, (hipfftDoubleReal *)out[j]);
        if (r != HIPFFT_SUCCESS) break;
        hipLaunchKernelGGL(k_add_const, dim3(grid_of(N3)), dim3(256), 0, st, out[j], N3, add);
    }
    if (lock.owns_lock()) lock.unlock();
    int rc = 0;
    if (r != HIPFFT_SUCCESS) {
        snprintf(msg, len, "hipFFT execution failed (hipfftResult %d)", (int)r);
        rc = 1;
    }
    const hipError_t es = hipStreamSynchronize(st);
    if (e == hipSuccess) e = es;
    if (!rc && e != hipSuccess) {
        snprintf(msg, len, "vacuum generation: %s", hipGetErrorString(e));
        rc = 1;
    }
    return rc;
}

}  // namespace lf
