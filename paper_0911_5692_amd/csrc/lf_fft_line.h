// FFTs of a batch of lattice lines held in LDS, FP64, for the transforms of
// lf_fft.hip: lengths whose prime factors are at most 7.
//
// A block of NT threads holds B lines of N complex points, up to 8 per thread.
// The transform is
// the self-sorting (Stockham) decimation of N into radices 2, 3, 4, 5, 7 and
// 8: in a stage of radix R after stages of product m, butterfly j
// takes the points j + r N/R, multiplies point r by w^(k r N/(m R)) with
// k = j mod m and w = exp(-2 pi i/N), transforms them, and leaves output q at
// (j div m) m R + k + q m.  A stage's points go through registers (all of
// them are read before the first is written), so one LDS buffer holds the
// batch: at 512 points x 8 lines two blocks fit on a CU, and the loads of one
// run beside the butterflies of the other.
// Only the forward transform exists; with the parts of every point swapped
// before and after, it is the (unnormalised) inverse.
#pragma once
#include <hip/hip_runtime.h>

namespace lf {

constexpr int kFftPts = 8;  // most points per thread

struct FftPlan {
    int N, stages;
    unsigned char radix[12];
};

// Radices of N, or stages = 0 if a prime factor is too large.
inline FftPlan fft_plan(int N)
{
    FftPlan p{};
    p.N = N;
    int n = N, twos = 0;
    while (n % 2 == 0) { n /= 2; ++twos; }
    int fours = twos % 3 == 1 ? (twos >= 4 ? 2 : 0) : (twos % 3 == 2 ? 1 : 0);
    int eights = (twos - 2 * fours) / 3, two = twos - 2 * fours - 3 * eights;
    auto add = [&](int r, int times) {
        for (; times > 0; --times) p.radix[p.stages++] = (unsigned char)r;
    };
    add(8, eights);
    add(4, fours);
    add(2, two);
    for (int r : {3, 5, 7}) {
        int t = 0;
        while (n % r == 0) { n /= r; ++t; }
        if (p.stages + t > 12) return FftPlan{};
        add(r, t);
    }
    if (n != 1) return FftPlan{};
    return p;
}

// Point n of line c: the line index is permuted with n, so that a walk along
// one line (by ones or fours) spreads over the banks as one across the lines
// does.
template <int B>
__device__ inline int fft_slot(int n, int c)
{
    return n * B + (c ^ ((n ^ (n >> 3)) & (B - 1)));
}

// i div n for 0 <= i < 2^21, inv = 1.0f / n (the quotient's distance from the
// next whole number, 0.5 / n, exceeds the rounding).
__device__ inline int div_by(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

__device__ inline double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }  // -i a

__device__ inline void dft4(double2 &a, double2 &b, double2 &c, double2 &d)
{
    const double2 t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = mul_mi(csub(b, d));
    a = cadd(t0, t2);
    b = cadd(t1, t3);
    c = csub(t0, t2);
    d = csub(t1, t3);
}

// cos and sin of 2 pi k/R, k = 1 .. (R-1)/2
template <int R>
struct Roots;
template <>
struct Roots<3> {
    static constexpr double c[1] = {-0.5}, s[1] = {0.866025403784438646764};
};
template <>
struct Roots<5> {
    static constexpr double c[2] = {0.309016994374947424102, -0.809016994374947424102};
    static constexpr double s[2] = {0.951056516295153572116, 0.587785252292473129169};
};
template <>
struct Roots<7> {
    static constexpr double c[3] = {0.623489801858733530525, -0.222520933956314404289, -0.900968867902419126236};
    static constexpr double s[3] = {0.781831482468029808708, 0.974927912181823607018, 0.433883739117558120476};
};
// Forward DFT of R points in place.
template <int R>
__device__ inline void dft(double2 (&v)[R])
{
    if constexpr (R == 2) {
        const double2 t = v[0];
        v[0] = cadd(t, v[1]);
        v[1] = csub(t, v[1]);
    } else if constexpr (R == 4) {
        dft4(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        dft4(v[0], v[2], v[4], v[6]);
        dft4(v[1], v[3], v[5], v[7]);
        constexpr double q = 0.707106781186547524401;
        const double2 o0 = v[1], o1 = make_double2(q * (v[3].x + v[3].y), q * (v[3].y - v[3].x));
        const double2 o2 = mul_mi(v[5]), o3 = make_double2(q * (v[7].y - v[7].x), -q * (v[7].x + v[7].y));
        const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
        v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
        v[1] = cadd(e1, o1); v[5] = csub(e1, o1);
        v[2] = cadd(e2, o2); v[6] = csub(e2, o2);
        v[3] = cadd(e3, o3); v[7] = csub(e3, o3);
    } else {
        // odd prime: cosine and sine sums over the pairs r, R - r
        constexpr int H = (R - 1) / 2;
        double2 a[H], b[H];
        double2 x0 = v[0];
#pragma unroll
        for (int r = 0; r < H; ++r) {
            a[r] = cadd(v[r + 1], v[R - 1 - r]);
            b[r] = csub(v[r + 1], v[R - 1 - r]);
            x0 = cadd(x0, a[r]);
        }
        const double2 c0 = v[0];
        v[0] = x0;
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            double2 A = c0, S = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const int k = (q * r) % R;
                const double cc = Roots<R>::c[(k <= H ? k : R - k) - 1];
                const double ss = k <= H ? Roots<R>::s[k - 1] : -Roots<R>::s[R - k - 1];
                A.x = fma(cc, a[r - 1].x, A.x);
                A.y = fma(cc, a[r - 1].y, A.y);
                S.x = fma(ss, b[r - 1].x, S.x);
                S.y = fma(ss, b[r - 1].y, S.y);
            }
            v[q] = make_double2(A.x + S.y, A.y - S.x);
            v[R - q] = make_double2(A.x - S.y, A.y + S.x);
        }
    }
}

// One stage over the block's B lines, N B <= 8 NT points.  EXACT: N is a power
// of two and N B = 8 NT, so every thread has the same number of butterflies
// and m divides by a shift.  Otherwise threads past the last butterfly repeat
// it (the same values to the same slots): masks for every butterfly cost more
// than they save.
template <int R, int B, int NT, bool EXACT>
__device__ __forceinline__ void fft_stage(double2 *s, int N, int m, const double2 *__restrict__ tw)
{
    constexpr int K = EXACT ? kFftPts / R : (kFftPts + R - 1) / R;
    const int nb = N / R, last = nb * B - 1, step = N / (m * R), lm = 31 - __clz(m);
    const float inv_m = 1.0f / (float)m;
    double2 v[K][R];
    int out[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int i = threadIdx.x + NT * k;
        if (!EXACT) i = min(i, last);
        const int c = i % B, j = i / B;
        const int jm = EXACT ? j >> lm : div_by(j, inv_m);
        const int km = j - jm * m;
#pragma unroll
        for (int r = 0; r < R; ++r) v[k][r] = s[fft_slot<B>(j + r * nb, c)];
        if (m > 1) {
#pragma unroll
            for (int r = 1; r < R; ++r) v[k][r] = cmul(v[k][r], tw[km * r * step]);
        }
        dft<R>(v[k]);
        out[k] = jm * m * R + km;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int i = threadIdx.x + NT * k;
        if (!EXACT) i = min(i, last);
        const int c = i % B;
#pragma unroll
        for (int q = 0; q < R; ++q) s[fft_slot<B>(out[k] + q * m, c)] = v[k][q];
    }
    __syncthreads();
}

// Forward transform of the block's lines in LDS (staged, barrier passed);
// tw: exp(-2 pi i n/N), n < N.  Ends with a barrier.
template <int B, int NT, bool EXACT>
__device__ __forceinline__ void fft_lines(double2 *s, const FftPlan &pl, const double2 *__restrict__ tw)
{
    int m = 1;
    for (int i = 0; i < pl.stages; ++i) {
        const int R = pl.radix[i];
        if constexpr (EXACT) {
            if (R == 8) fft_stage<8, B, NT, true>(s, pl.N, m, tw);
            else if (R == 4) fft_stage<4, B, NT, true>(s, pl.N, m, tw);
            else fft_stage<2, B, NT, true>(s, pl.N, m, tw);
        } else {
            switch (R) {
            case 2: fft_stage<2, B, NT, false>(s, pl.N, m, tw); break;
            case 3: fft_stage<3, B, NT, false>(s, pl.N, m, tw); break;
            case 4: fft_stage<4, B, NT, false>(s, pl.N, m, tw); break;
            case 5: fft_stage<5, B, NT, false>(s, pl.N, m, tw); break;
            case 7: fft_stage<7, B, NT, false>(s, pl.N, m, tw); break;
            default: fft_stage<8, B, NT, false>(s, pl.N, m, tw); break;
            }
        }
        m *= R;
    }
}

}  // namespace lf
