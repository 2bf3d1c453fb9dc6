// Harmonic-space half of the split convolution (Sutter, Wandelt & Elsner 2012,
// Sec. 2, eq. 1): the truncated l-space kernel Khat_l, l <= lcut, applied to a
// HEALPix RING map by spherical-harmonic analysis with the pixel quadrature
// and synthesis,
//
//     a_lm = Omega sum_p x_p conj(Y_lm(p)),
//     y_p  = sum_{l <= lcut} Khat_l sum_m a_lm Y_lm(p),
//
// with Y_lm = lambda_lm(cos theta) e^{i m phi} and the orthonormal associated
// Legendre functions lambda_lm.  The paper runs this half on host cores with an
// SHT library while the GPU sums the real-space half; here both halves run on
// the GPU, in stream-ordered kernels, all in FP64.  A ring and its N-S mirror
// have the same length and the same first longitude, so every kernel works on
// pairs: with e = x_ring + x_mirror and o = x_ring - x_mirror, even l + m sees
// only e and odd l + m only o.
//
//  1. k_ring_fwd      per ring pair: the longitude sums of z = e + i o,
//                     Z(m) = sum_j z_j e^{-i m phi_j} for m = -lcut .. lcut,
//                     by FFTs of a quarter of the ring (k_sht_dft_fwd, direct
//                     sums, at low lcut and on small maps);
//  2. k_leg_fwd       per (m, chunk of ring pairs): Legendre functions by a
//                     two-degree recurrence, times E(m) and O(m), reduced over
//                     the rings into per-chunk partial sums;
//  3. k_sht_mul       the sums over chunks turned into a_lm, multiplied by
//                     Omega Khat_l, and turned into synthesis coefficients;
//  4. k_leg_bwd       per (m, ring pair): the even and odd sums over l;
//  5. k_ring_bwd      per ring pair: the pixels of both rings by inverse FFTs
//                     of a quarter of the ring (k_sht_dft_bwd otherwise).
//
// lambda_mm underflows FP64 for large m near the poles, so the recurrence
// carries a power-of-two scale: a value is stored * 2^(512 sc) with sc <= 0, and
// terms are used only once sc reaches 0 (below that they are < 2^-330 times
// the ring's other terms).  Results are deterministic: no atomics.
//
// At Nside 2048 and lcut 1500 the half takes 2.4 ms: longitude sums 0.56 + 0.45 ms
// (one Goertzel or Clenshaw sum per frequency on cap rings and radix-2 FFTs on
// belt rings took 2.06 + 2.13 ms), Legendre sums 0.87 + 0.75 ms (2.08 + 1.24 ms with
// the one-degree recurrence and a reduction through LDS).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <new>
#include <string>
#include <vector>

#include "arkcos_internal.hpp"

namespace arkcos {

// One ring as the transform kernels see it (0-based).
struct ShtRing {
    double z;       // cos theta
    double s;       // sin theta
    double log2s;   // log2 sin theta
    int n;          // pixels
    int first;      // RING index of pixel 0
    int two_o;      // 1: pixel j at phi = (j + 1/2) 2 pi / n, 0: at j 2 pi / n
    int pad;
};
static_assert(sizeof(ShtRing) == 40, "ShtRing layout");

// One ring pair of an FFT launch: northern ring, transform length k = n / 4,
// log2 of the FFT length P, and the offset of the chirp spectrum in the plan's
// table (0 for the direct transforms, P = k).
struct ShtFftRing {
    int ring;
    int k;
    int lg;
    int chirp;
};

constexpr int kShtThreads = 256;
constexpr int kShtMaxPairs = 4;     // pairs of orders per thread and pass in k_sht_dft_fwd
constexpr double kShtDirectWork = 6e7;   // pixels x orders up to which every ring is summed directly
constexpr int kShtMaxK = 4096;      // longest quarter ring the FFTs take
constexpr int kLegBlock = 4;        // recurrence steps (two degrees each) per reduction
constexpr int kLegFwdRings = 8;     // ring pairs per lane of k_leg_fwd on large maps
constexpr int kLegBwdRings = 4;     // and of k_leg_bwd
constexpr int kLegFlush = 32;       // reductions kept in LDS between sums over the waves
constexpr double kScaleUp = 0x1p128;     // rescale threshold of a scaled value
constexpr double kScaleStep = 0x1p-512;  // one scale step

// Steps of order m: step k covers the degrees m + 2k and m + 2k + 1, padded to
// whole blocks.
__host__ __device__ inline int leg_steps(int m, int L)
{
    return ((L - m) / 2 + kLegBlock) / kLegBlock * kLegBlock;
}

// Ring-pair rows of the longitude sums hold two arrays (m >= 0 and m <= 0, or
// even and odd sums) of 4 lq complex values, the orders of one class m mod 4
// contiguous: an FFT of a quarter ring yields one class, and its loads and
// stores are then consecutive.
__host__ __device__ inline int order_slot(int m, int lq) { return (m & 3) * lq + (m >> 2); }

// The order m of workgroup b (gridDim.x is a multiple of 64).  Workgroups go
// to the eight XCDs in turn; the eight orders that share the 128-byte lines of
// every ring row run on one XCD one after the other, so that its L2 serves
// (merges) their 16-byte reads (writes).
__device__ __forceinline__ int leg_order(int b)
{
    const int e = ((((b >> 3) >> 3) * 8 + (b & 7)) << 3) + ((b >> 3) & 7);
    return 32 * (e >> 5) + 4 * (e & 7) + ((e >> 3) & 3);
}
static int leg_grid(int L) { return 64 * ((4 * (L / 32 + 1) + 7) / 8); }

// Recurrence tables and coefficients are wave-uniform and read-only while a
// kernel runs: through the constant address space they are scalar loads.
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using uptr = const __attribute__((address_space(4))) T *;
#else
template <class T>
using uptr = const T *;
#endif
typedef double d2v __attribute__((ext_vector_type(2)));
typedef double d4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 add2(double2 a, double2 b)
{
    return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 sub2(double2 a, double2 b)
{
    return make_double2(a.x - b.x, a.y - b.y);
}
// Roots of unity of a ring: at(u) = e^{i pi u / n} for an integer |u| < 2^31.  The
// angle in turns, reduced exactly, is the nearest of kRoots table entries plus
// a remainder of at most half a step (pi / 64 radians), whose sine and cosine
// are short Taylor sums (truncation below 1e-16): no division and no integer
// modulo, a fifth of the instructions of sincospi.  The table stands in LDS.
constexpr int kRoots = 64;
struct RingRoots {
    const double2 *roots;
    double n2, inv;   // 2n, 1/(2n)
    __device__ __forceinline__ RingRoots(const double2 *table, int n)
        : roots(table), n2(2.0 * n), inv(1.0 / (2.0 * n)) {}
    __device__ __forceinline__ double2 at(int u) const
    {
        const double ud = (double)u;
        const double t = fma(-rint(ud * inv), n2, ud) * inv;
        const double q = rint(t * kRoots);
        const double x = fma(q, -1.0 / kRoots, t) * 6.283185307179586477;
        const double x2 = x * x;
        const double sn =
            x * fma(x2, fma(x2, fma(x2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), 1.0);
        const double cs =
            fma(x2, fma(x2, fma(x2, fma(x2, 1.0 / 40320.0, -1.0 / 720.0), 1.0 / 24.0), -0.5), 1.0);
        return cmul(roots[(int)q & (kRoots - 1)], make_double2(cs, sn));
    }
};
// The table into LDS, by threads 0 .. kRoots - 1 (a barrier follows in the caller).
__device__ __forceinline__ void load_roots(double2 *lds, const double2 *__restrict__ roots)
{
    if (threadIdx.x < kRoots) lds[threadIdx.x] = roots[threadIdx.x];
}

// ----------------------------------------------------------- ring FFTs --
// With z the n = 4k complex samples of a ring pair, the class q = 4a + c of
// its transform is a length-k transform of the folded samples
//     Z(4a + c) = sum_{j<k} e^{-2 pi i a j / k} e^{-2 pi i c j / n} sum_t (-i)^{ct} z_{j + tk},
// done in LDS: on belt rings whose k is a power of two directly, else by
// Bluestein's chirp transform, a circular convolution of length P = 2^lg >= 2k - 1
// with b(t) = e^{+pi i t^2 / k}, whose spectrum (times 1/P) is a plan table.  The
// FFT is radix 8, one butterfly of each pass per thread, decimation in frequency
// from natural to digit-reversed order, and its inverse back, so no pass
// reorders.  The first pass (radix 2 or 4 where lg is no multiple of 3) and the
// last pass of the inverse act on entries t + i P/8, i < 8, of thread t: they
// run in registers, on the samples as they are loaded and on the results as they
// are stored.  Against one Goertzel sum per frequency, O(n lcut) per ring, the cap
// rings cost O(P log P); what bounds the kernels is the latency of their loads
// and barriers (the waves wait 0.4 to 0.7 of their cycles; vector instructions take 0.25 to 0.45 of
// the SIMDs').  The forward kernels also spill registers (58 without the chirp,
// 0.24 ms against the inverse's 0.16 at k = 2048; 19 with it), and the 1024-thread ones of k > 2048,
// held to 128 registers, spill 584 and 565 (1.5 + 1.4 ms at Nside 4096).  LDS entries
// are padded by one in eight, so that the short-stride passes spread over the
// banks.
__host__ __device__ inline int fft_pad(int i) { return i + (i >> 3); }
static size_t fft_lds_bytes(int lg) { return (size_t)(fft_pad(1 << lg) + kRoots) * sizeof(double2); }

// Four-point transform in place, without twiddles; INV: the inverse.
template <bool INV>
__device__ __forceinline__ void dft4(double2 &a0, double2 &a1, double2 &a2, double2 &a3)
{
    const double2 t0 = add2(a0, a2), t1 = sub2(a0, a2), t2 = add2(a1, a3), d = sub2(a1, a3);
    const double2 t3 = INV ? make_double2(-d.y, d.x) : make_double2(d.y, -d.x);
    a0 = add2(t0, t2);
    a1 = add2(t1, t3);
    a2 = sub2(t0, t2);
    a3 = sub2(t1, t3);
}

// Eight-point transform: frequency f = s + 2r at entry 4s + r.  The inverse
// takes that order and returns the natural one.
__device__ __forceinline__ void dft8(double2 e[8])
{
    constexpr double h = 0.70710678118654752440;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double2 d = sub2(e[r], e[r + 4]);
        e[r] = add2(e[r], e[r + 4]);
        // times e^{-2 pi i r / 8}
        e[r + 4] = r == 0 ? d
                 : r == 1 ? make_double2(h * (d.x + d.y), h * (d.y - d.x))
                 : r == 2 ? make_double2(d.y, -d.x)
                          : make_double2(h * (d.y - d.x), -h * (d.x + d.y));
    }
    dft4<false>(e[0], e[1], e[2], e[3]);
    dft4<false>(e[4], e[5], e[6], e[7]);
}
__device__ __forceinline__ void idft8(double2 e[8])
{
    constexpr double h = 0.70710678118654752440;
    dft4<true>(e[0], e[1], e[2], e[3]);
    dft4<true>(e[4], e[5], e[6], e[7]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double2 b = e[r + 4];
        // times e^{+2 pi i r / 8}
        const double2 d = r == 0 ? b
                        : r == 1 ? make_double2(h * (b.x - b.y), h * (b.x + b.y))
                        : r == 2 ? make_double2(-b.y, b.x)
                                 : make_double2(-h * (b.x + b.y), h * (b.x - b.y));
        e[r + 4] = sub2(e[r], d);
        e[r] = add2(e[r], d);
    }
}

// Twiddles w^f of entry 4s + r, f = s + 2r, from w; INV: their conjugates.
template <bool INV>
__device__ __forceinline__ void twiddle8(double2 e[8], double2 w1)
{
    if (INV) w1 = conj2(w1);
    const double2 w2 = cmul(w1, w1), w3 = cmul(w1, w2), w4 = cmul(w2, w2);
    e[4] = cmul(e[4], w1);
    e[1] = cmul(e[1], w2);
    e[5] = cmul(e[5], w3);
    e[2] = cmul(e[2], w4);
    e[6] = cmul(e[6], cmul(w4, w1));
    e[3] = cmul(e[3], cmul(w4, w2));
    e[7] = cmul(e[7], cmul(w4, w3));
}

// The first forward pass, on entries t + i P/8: radix 8, 4 or 2 as lg mod 3 is
// 0, 2 or 1.  tw[t] = e^{-2 pi i t / Pm}, t < Pm/4, Pm = 2^lgm the plan's longest FFT.
__device__ __forceinline__ void fft_first(double2 e[8], const double2 *__restrict__ tw, int lg,
                                          int lgm, int t)
{
    const int s8 = (1 << lg) >> 3;
    if (lg % 3 == 0) {
        dft8(e);
        if (s8 > 1) twiddle8<false>(e, tw[t << (lgm - lg)]);
    } else if (lg % 3 == 2) {   // stride P/4: entries i, i + 2, i + 4, i + 6
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double2 w1 = tw[(t + i * s8) << (lgm - lg)];
            const double2 w2 = cmul(w1, w1), w3 = cmul(w1, w2);
            dft4<false>(e[i], e[i + 2], e[i + 4], e[i + 6]);
            e[i + 2] = cmul(e[i + 2], w1);
            e[i + 4] = cmul(e[i + 4], w2);
            e[i + 6] = cmul(e[i + 6], w3);
        }
    } else {   // stride P/2: entries i, i + 4
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // e^{-2 pi i j / P}, the second quarter of the table by -i
            double2 w = tw[(t + (i & 1) * s8) << (lgm - lg)];
            if (i >= 2) w = make_double2(w.y, -w.x);
            const double2 d = sub2(e[i], e[i + 4]);
            e[i] = add2(e[i], e[i + 4]);
            e[i + 4] = cmul(d, w);
        }
    }
}

// Its inverse: the last pass of the inverse transform.
__device__ __forceinline__ void fft_last_inverse(double2 e[8], const double2 *__restrict__ tw,
                                                 int lg, int lgm, int t)
{
    const int s8 = (1 << lg) >> 3;
    if (lg % 3 == 0) {
        if (s8 > 1) twiddle8<true>(e, tw[t << (lgm - lg)]);
        idft8(e);
    } else if (lg % 3 == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double2 w1 = conj2(tw[(t + i * s8) << (lgm - lg)]);
            const double2 w2 = cmul(w1, w1), w3 = cmul(w1, w2);
            e[i + 2] = cmul(e[i + 2], w1);
            e[i + 4] = cmul(e[i + 4], w2);
            e[i + 6] = cmul(e[i + 6], w3);
            dft4<true>(e[i], e[i + 2], e[i + 4], e[i + 6]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double2 w = tw[(t + (i & 1) * s8) << (lgm - lg)];
            if (i >= 2) w = make_double2(w.y, -w.x);
            const double2 d = cmul(e[i + 4], conj2(w));
            e[i + 4] = sub2(e[i], d);
            e[i] = add2(e[i], d);
        }
    }
}

// The transform of e (entries t + i P/8 of thread t; P = 2^lg >= 8), in LDS z.
// BLUE: the convolution with the chirp spectrum bh, back in e; else the result
// stands in z, frequency a at fft_place(a).  Every thread of the workgroup calls
// it; threads from P/8 on only meet the barriers.  z is free on entry; the
// caller puts a barrier before it reuses z.
template <bool BLUE>
__device__ __forceinline__ void ring_dft(double2 e[8], double2 *z, const double2 *__restrict__ tw,
                                         const double2 *__restrict__ bh, int lg, int lgm)
{
    const int t = (int)threadIdx.x, s8 = (1 << lg) >> 3;
    const bool on = t < s8;
    // stride of the pass after the first one
    int lh = (lg % 3 == 0 ? lg - 3 : lg / 3 * 3) - 3;
    if (on) fft_first(e, tw, lg, lgm, t);
    if (lh < 0) {   // P = 8: one thread, one pass
        if (BLUE && on) {
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = cmul(e[r], bh[r]);
            idft8(e);
        }
        if (!BLUE && on)
#pragma unroll
            for (int r = 0; r < 8; ++r) z[fft_pad(r)] = e[r];
        __syncthreads();
        return;
    }
    if (on)
#pragma unroll
        for (int i = 0; i < 8; ++i) z[fft_pad(t + i * s8)] = e[i];
    for (; lh >= 0; lh -= 3) {
        const int h = 1 << lh, j = t & (h - 1), i0 = ((t - j) << 3) + j;
        double2 w = make_double2(1.0, 0.0);
        double2 f[8];
        if (on && lh > 0) w = tw[j << (lgm - lh - 3)];   // (ahead of the barrier)
        if (BLUE && on && lh == 0)
#pragma unroll
            for (int r = 0; r < 8; ++r) f[r] = bh[8 * t + r];
        __syncthreads();
        if (on) {
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = z[fft_pad(i0 + r * h)];
            dft8(e);
            if (lh > 0) {
                twiddle8<false>(e, w);
            } else if (BLUE) {
                // the last forward butterflies, the product and the first
                // inverse ones act on the same eight entries
#pragma unroll
                for (int r = 0; r < 8; ++r) e[r] = cmul(e[r], f[r]);
                idft8(e);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) z[fft_pad(i0 + r * h)] = e[r];
        }
    }
    if (!BLUE) {
        __syncthreads();
        return;
    }
    for (lh = 3; lh + 3 <= lg - (lg % 3 == 0 ? 3 : lg % 3); lh += 3) {
        const int h = 1 << lh, j = t & (h - 1), i0 = ((t - j) << 3) + j;
        double2 w = make_double2(1.0, 0.0);
        if (on) w = tw[j << (lgm - lh - 3)];
        __syncthreads();
        if (on) {
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = z[fft_pad(i0 + r * h)];
            twiddle8<true>(e, w);
            idft8(e);
#pragma unroll
            for (int r = 0; r < 8; ++r) z[fft_pad(i0 + r * h)] = e[r];
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = z[fft_pad(t + i * s8)];
        fft_last_inverse(e, tw, lg, lgm, t);
    }
}

// Place of frequency a in the output order of ring_dft<false>.
__device__ __forceinline__ int fft_place(int a, int lg)
{
    int pos = 0;
    const int b = lg % 3;
    lg -= b;
    if (b) {
        pos = (a & ((1 << b) - 1)) << lg;
        a >>= b;
    }
    while (lg > 0) {
        lg -= 3;
        pos += (((a & 1) << 2) | ((a >> 1) & 3)) << lg;
        a >>= 3;
    }
    return pos;
}

// Chirp spectra, one workgroup per length: b(t) = e^{pi i t^2 / k} for |t| < k,
// transformed in the order of ring_dft, times 1/P.
__global__ __launch_bounds__(1024) void k_chirp(const ShtFftRing *__restrict__ list,
                                                const double2 *__restrict__ tw,
                                                const double2 *__restrict__ roots,
                                                double2 *__restrict__ chirp, int lgm)
{
    extern __shared__ double2 lds[];
    double2 *z = lds + kRoots;
    load_roots(lds, roots);
    __syncthreads();
    const ShtFftRing Q = list[blockIdx.x];
    const RingRoots W(lds, 4 * Q.k);
    const int P = 1 << Q.lg;
    double2 e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int j = (int)threadIdx.x + i * (P >> 3), t = min(j, P - j);
        // t^2 / k = 4 t^2 / n
        e[i] = t >= 0 && t < Q.k ? W.at(4 * t * t) : make_double2(0.0, 0.0);
    }
    ring_dft<false>(e, z, tw, nullptr, Q.lg, lgm);
    const double inv = 1.0 / (double)P;
    for (int i = threadIdx.x; i < P; i += 1024) {
        const double2 v = z[fft_pad(i)];
        chirp[Q.chirp + i] = make_double2(v.x * inv, v.y * inv);
    }
}

// Workgroup (ring pair of the list, map), which takes the four classes in turn
// from the pixels it holds in registers.
template <int T, bool BLUE>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(2)))
void k_ring_fwd(const ShtRing *__restrict__ rings,
                                                const ShtFftRing *__restrict__ list,
                                                const double2 *__restrict__ tw,
                                                const double2 *__restrict__ roots,
                                                const double2 *__restrict__ chirp, int lgm,
                                                const float *__restrict__ x, long long npix,
                                                double2 *__restrict__ F, int L, int lq,
                                                int nnorth)
{
    extern __shared__ double2 lds[];
    double2 *z = lds + kRoots;
    load_roots(lds, roots);
    const ShtFftRing Q = list[blockIdx.x];
    const ShtRing R = rings[Q.ring];
    const bool equator = Q.ring == nnorth - 1;
    const float *xa = x + (size_t)blockIdx.y * npix + R.first;
    const float *xb = x + (size_t)blockIdx.y * npix + rings[2 * nnorth - 2 - Q.ring].first;
    const int k = Q.k, s8 = (1 << Q.lg) >> 3, t0 = (int)threadIdx.x;
    constexpr int JN = BLUE ? 4 : 8;   // entries t + i P/8 from 4 on are padding (k <= P/2)
    float pa[JN][4], pb[JN][4];
#pragma unroll
    for (int i = 0; i < JN; ++i) {
        const int j = t0 + i * s8;
        const bool in = t0 < s8 && j < k;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            pa[i][t] = in ? xa[j + t * k] : 0.0f;
            pb[i][t] = in && !equator ? xb[j + t * k] : 0.0f;
        }
    }
    __syncthreads();   // the roots
    const RingRoots W(lds, R.n);
    double2 *row = F + ((size_t)blockIdx.y * nnorth + Q.ring) * 8 * lq;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double2 e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < JN; ++i) {
            const int j = t0 + i * s8;
            double2 s[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double p = (double)pa[i][t], q = (double)pb[i][t];
                s[t] = make_double2(p + q, equator ? 0.0 : p - q);
            }
            double2 v;
            if (c & 1) {
                const double2 d0 = sub2(s[0], s[2]), d1 = sub2(s[1], s[3]);
                v = c == 1 ? make_double2(d0.x + d1.y, d0.y - d1.x)
                           : make_double2(d0.x - d1.y, d0.y + d1.x);
            } else {
                const double2 d0 = add2(s[0], s[2]), d1 = add2(s[1], s[3]);
                v = c == 0 ? add2(d0, d1) : sub2(d0, d1);
            }
            if (BLUE || c) v = cmul(v, W.at(-(BLUE ? 4 * j * j : 0) - 2 * c * j));
            if (t0 < s8 && j < k) e[i] = v;
        }
        ring_dft<BLUE>(e, z, tw, chirp + Q.chirp, Q.lg, lgm);
        // Z(m) e^{-i m phi_0} of the orders m = q mod n, q = 4a + c, and
        // Z(-m) e^{i m phi_0} of the orders m = -q mod n; phi_0 = two_o pi / n
        if (BLUE && R.n <= L) {
            // several orders per frequency: all threads share them
            if (t0 < s8)
#pragma unroll
                for (int i = 0; i < JN; ++i) {
                    const int a = t0 + i * s8;
                    if (a < k) z[fft_pad(a)] = cmul(e[i], W.at(-4 * a * a));
                }
            __syncthreads();
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                for (int m = (side ? (4 - c) & 3 : c) + 4 * t0; m <= L; m += 4 * T) {
                    const int r = m % R.n;
                    const int a = ((side && r ? R.n - r : r) - c) >> 2;
                    row[side * 4 * lq + order_slot(m, lq)] =
                        cmul(z[fft_pad(a)], W.at((side ? m : -m) * R.two_o));
                }
            }
            __syncthreads();
            continue;
        }
#pragma unroll
        for (int i = 0; i < JN; ++i) {
            const int a = t0 + i * s8, q = 4 * a + c;
            if (t0 >= s8 || a >= k || (q > L && R.n - q > L)) continue;
            const double2 v = BLUE ? cmul(e[i], W.at(-4 * a * a)) : z[fft_pad(fft_place(a, Q.lg))];
            const double2 w = R.two_o ? W.at(q) : make_double2(1.0, 0.0);
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                // m = q + (multiple of n): e^{-i m phi_0} = +-e^{-i q phi_0}; m = n - q: -e^{-i q phi_0}
                bool neg = side && q && R.two_o;
                for (int m = side && q ? R.n - q : q; m <= L; m += R.n) {
                    const double2 y = cmul(v, conj2(w));
                    row[side * 4 * lq + order_slot(m, lq)] = neg ? make_double2(-y.x, -y.y) : y;
                    neg ^= R.two_o != 0;
                }
            }
        }
        __syncthreads();
    }
}

// The inverse: with He(m), Ho(m) the even and odd sums times e^{i m phi_0} and
// c_m = 1 (m = 0) or 2, the pixels are the real parts of sum_m c_m H(m)
// e^{2 pi i m j / n}, i.e. the inverse transform of the Hermitian spectrum
//     S(q) = sum_{m = q mod n, m > 0} H(m) + sum_{m = -q mod n, m > 0} conj H(m)
// (+ Re H(0) at q = 0), of S = S_e + i S_o for both rings at once.  One
// workgroup per (ring pair, map) takes the classes 0, 2, 1, 3 in turn and keeps
// their sums for its pixels in registers.
template <int T, bool BLUE>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(2)))
void k_ring_bwd(const ShtRing *__restrict__ rings, const ShtFftRing *__restrict__ list,
                const double2 *__restrict__ tw, const double2 *__restrict__ roots,
                const double2 *__restrict__ chirp, int lgm, const double2 *__restrict__ G,
                float *out, long long npix, int L, int lq, int nnorth, int accumulate)
{
    extern __shared__ double2 lds[];
    double2 *z = lds + kRoots;
    load_roots(lds, roots);
    const ShtFftRing Q = list[blockIdx.x];
    const ShtRing R = rings[Q.ring];
    const double2 *ge = G + ((size_t)blockIdx.y * nnorth + Q.ring) * 8 * lq;
    const double2 *go = ge + 4 * lq;
    float *oa = out + (size_t)blockIdx.y * npix + R.first;
    float *ob = out + (size_t)blockIdx.y * npix + rings[2 * nnorth - 2 - Q.ring].first;
    const bool equator = Q.ring == nnorth - 1;
    const int k = Q.k, s8 = (1 << Q.lg) >> 3, t0 = (int)threadIdx.x;
    constexpr int JN = BLUE ? 4 : 8;
    const RingRoots W(lds, R.n);
    // short rings, on which several orders fall on one frequency, give each
    // frequency 2^sl lanes and pass the spectrum through LDS
    const bool folds = R.n <= 2 * L;
    int sl = 0;
    while (sl < 6 && (R.n << sl) < L && (k << (sl + 1)) <= T) ++sl;
    const int sub = t0 & ((1 << sl) - 1);
    const bool flip = R.two_o && sl == 0;   // an odd number of ring lengths per step
    __syncthreads();   // the roots
    // u_0, then u_0 + u_2; u_0 - u_2; u_1 (u_c the class's share of quarter 0)
    double2 ya[JN], yb[JN], yc[JN];
#pragma unroll
    for (int ci = 0; ci < 4; ++ci) {
        const int c = ((ci & 1) << 1) | (ci >> 1);   // 0, 2, 1, 3
        // conj (S_e + i S_o) at q = 4a + c (the inverse transform is the conjugate
        // of the transform of the conjugate), times the chirp
        double2 e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = make_double2(0.0, 0.0);
        if (folds) {
            for (int a0 = 0; a0 < k; a0 += T >> sl) {
                const int a = a0 + (t0 >> sl);
                double2 se = make_double2(0.0, 0.0), so = se;
                if (a < k) {
                    const int q = 4 * a + c;
                    if (q == 0 && sub == 0) {
                        se.x = ge[0].x;
                        so.x = go[0].x;
                    }
                    // this lane's share of the orders +-q mod n; phi_0 n / pi = two_o, so
                    // the phase of m + n is (-1)^two_o times that of m
#pragma unroll
                    for (int side = 0; side < 2; ++side) {
                        const int m1 = (side || !q ? R.n - q : q) + sub * R.n;
                        if (m1 > L) continue;
                        double2 w = W.at(m1 * R.two_o);
                        for (int m = m1; m <= L; m += R.n << sl) {
                            const double2 he = cmul(ge[order_slot(m, lq)], w);
                            const double2 ho = cmul(go[order_slot(m, lq)], w);
                            se = add2(se, side ? conj2(he) : he);
                            so = add2(so, side ? conj2(ho) : ho);
                            if (flip) w = make_double2(-w.x, -w.y);
                        }
                    }
                }
                double2 v = make_double2(se.x - so.y, -(se.y + so.x));
                for (int d = 1; d < 1 << sl; d <<= 1) {
                    v.x += __shfl_xor(v.x, d);
                    v.y += __shfl_xor(v.y, d);
                }
                if (sub == 0 && a < k) z[fft_pad(a)] = BLUE ? cmul(v, W.at(-4 * a * a)) : v;
            }
            __syncthreads();
            if (t0 < s8)
#pragma unroll
                for (int i = 0; i < JN; ++i)
                    if (t0 + i * s8 < k) e[i] = z[fft_pad(t0 + i * s8)];
            __syncthreads();
        } else {
            // one order at most per frequency: m = q, or m = n - q (conjugate)
            double2 he[JN], ho[JN];
#pragma unroll
            for (int i = 0; i < JN; ++i) {
                const int a = t0 + i * s8, q = 4 * a + c, m = q <= L ? q : R.n - q;
                const bool in = t0 < s8 && a < k && m <= L;
                const int sm = order_slot(in ? m : 0, lq);
                he[i] = in ? ge[sm] : make_double2(0.0, 0.0);
                ho[i] = in ? go[sm] : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int i = 0; i < JN; ++i) {
                const int a = t0 + i * s8, q = 4 * a + c;
                const bool up = q <= L;
                double2 se = he[i], so = ho[i];
                if (R.two_o) {
                    const double2 w = W.at(up ? q : R.n - q);
                    se = cmul(se, w);
                    so = cmul(so, w);
                }
                if (q == 0) se.y = so.y = 0.0;
                if (!up) {
                    se = conj2(se);
                    so = conj2(so);
                }
                e[i] = make_double2(se.x - so.y, -(se.y + so.x));
                if (BLUE) e[i] = cmul(e[i], W.at(-4 * a * a));
            }
        }
        ring_dft<BLUE>(e, z, tw, chirp + Q.chirp, Q.lg, lgm);
#pragma unroll
        for (int i = 0; i < JN; ++i) {
            const int j = t0 + i * s8;
            if (t0 >= s8 || j >= k) continue;
            double2 v = BLUE ? e[i] : z[fft_pad(fft_place(j, Q.lg))];
            if (BLUE || c) v = cmul(v, W.at(-(BLUE ? 4 * j * j : 0) - 2 * c * j));
            v.y = -v.y;
            if (ci == 0) {
                ya[i] = v;
            } else if (ci == 1) {
                yb[i] = sub2(ya[i], v);
                ya[i] = add2(ya[i], v);
            } else if (ci == 2) {
                yc[i] = v;
            } else {
                // quarters t: sum over c of i^(ct) u_c
                const double2 s = add2(yc[i], v), d = sub2(yc[i], v);
                const double2 id = make_double2(-d.y, d.x);
                const double2 y[4] = {add2(ya[i], s), add2(yb[i], id), sub2(ya[i], s),
                                      sub2(yb[i], id)};
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float va = (float)(y[t].x + y[t].y), vb = (float)(y[t].x - y[t].y);
                    const int p = j + t * k;
                    oa[p] = accumulate ? oa[p] + va : va;
                    if (!equator) ob[p] = accumulate ? ob[p] + vb : vb;
                }
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------- direct ring sums --
// For rings on which the FFTs are the longer way (see ring_direct).  With the folds of
// the FFTs, real for each of e and o: a_0 = s_0 + s_1 + s_2 + s_3 and a_2 = s_0 - s_1 +
// s_2 - s_3 for the classes 0 and 2, p = s_0 - s_2 and q = s_1 - s_3 for the classes
// 1 (p - i q) and 3 (p + i q), s_t the samples of quarter t.  Goertzel on the k samples of a
// fold: s_j = x_j + 2 cos(w) s_{j-1} - s_{j-2}, and sum_j x_j e^{-i w j} =
// e^{-i w (k-1)} (s_{k-1} - e^{-i w} s_{k-2}).  Two samples per step update (s1, s2) in
// place: s2 <- c s1 + x_j - s2, s1 <- c s2 + x_{j+1} - s1.  A thread takes the orders 2p and
// 2p + 1, six real sums of length n/4 (against four of length n without the folds), for K
// values of p; waves past lcut only stage.  One launch covers p = p0 .. p0 + K kShtThreads - 1.
// FP64 issue bounds it.
template <int K>
__global__ __launch_bounds__(kShtThreads) void k_sht_dft_fwd(const ShtRing *__restrict__ rings,
                                                             const int *__restrict__ ring_list,
                                                             const double2 *__restrict__ roots,
                                                             const float *__restrict__ x,
                                                             long long npix,
                                                             double2 *__restrict__ F, int p0,
                                                             int L, int lq, int nnorth)
{
    __shared__ double2 sx[4 * kShtThreads];   // a_0, a_2, p, q of a sample, each (e, o)
    __shared__ double2 rt[kRoots];
    load_roots(rt, roots);
    const int r = ring_list[blockIdx.x];
    const ShtRing R = rings[r];
    const bool equator = r == nnorth - 1;
    const float *xa = x + (size_t)blockIdx.y * npix + R.first;
    const float *xb = x + (size_t)blockIdx.y * npix + rings[2 * nnorth - 2 - r].first;
    const int k = R.n >> 2;
    const int first = p0 + K * ((int)threadIdx.x & ~63);
    const int pl = first + ((int)threadIdx.x & 63);   // p = pl + 64 i: all of one parity
    const bool busy = __builtin_amdgcn_readfirstlane(2 * first) <= L;
    // state of the even order (e, o) and of the odd one (p e, p o, q e, q o)
    double ce[K], co[K], s1[K][6], s2[K][6];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int m = 2 * (pl + 64 * i);
        ce[i] = 2.0 * cospi(2.0 * (double)(m % R.n) / (double)R.n);
        co[i] = 2.0 * cospi(2.0 * (double)((m + 1) % R.n) / (double)R.n);
#pragma unroll
        for (int f = 0; f < 6; ++f) s1[i][f] = s2[i][f] = 0.0;
    }
    float va[4], vb[4];
    auto load = [&](int j0) {
        const int j = j0 + (int)threadIdx.x;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            va[t] = j < k ? xa[j + t * k] : 0.0f;
            vb[t] = j < k && !equator ? xb[j + t * k] : 0.0f;
        }
    };
    load(0);
    for (int j0 = 0; j0 < k; j0 += kShtThreads) {
        __syncthreads();
        {
            double e[4], o[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                e[t] = (double)va[t] + (double)vb[t];
                o[t] = equator ? 0.0 : (double)va[t] - (double)vb[t];
            }
            double2 *d = sx + 4 * threadIdx.x;
            d[0] = make_double2((e[0] + e[2]) + (e[1] + e[3]), (o[0] + o[2]) + (o[1] + o[3]));
            d[1] = make_double2((e[0] + e[2]) - (e[1] + e[3]), (o[0] + o[2]) - (o[1] + o[3]));
            d[2] = make_double2(e[0] - e[2], o[0] - o[2]);
            d[3] = make_double2(e[1] - e[3], o[1] - o[3]);
        }
        __syncthreads();
        if (j0 + kShtThreads < k) load(j0 + kShtThreads);
        if (!busy) continue;
        const int cnt = min(kShtThreads, k - j0);
        const double2 *u = sx + (pl & 1), *w = sx + 2;
        int j = 0;
        for (; j + 1 < cnt; j += 2, u += 8, w += 8) {
            const double2 ua = u[0], pa = w[0], qa = w[1], ub = u[4], pb = w[4], qb = w[5];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const double fa[6] = {ua.x, ua.y, pa.x, pa.y, qa.x, qa.y};
                const double fb[6] = {ub.x, ub.y, pb.x, pb.y, qb.x, qb.y};
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    const double c = f < 2 ? ce[i] : co[i];
                    s2[i][f] = fma(c, s1[i][f], fa[f] - s2[i][f]);
                    s1[i][f] = fma(c, s2[i][f], fb[f] - s1[i][f]);
                }
            }
        }
        if (j < cnt) {   // the last sample of an odd k
            const double2 ua = u[0], pa = w[0], qa = w[1];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const double fa[6] = {ua.x, ua.y, pa.x, pa.y, qa.x, qa.y};
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    const double v = fma(f < 2 ? ce[i] : co[i], s1[i][f], fa[f] - s2[i][f]);
                    s2[i][f] = s1[i][f];
                    s1[i][f] = v;
                }
            }
        }
    }
    if (!busy) return;
    double2 *row = F + ((size_t)blockIdx.y * nnorth + r) * 8 * lq;
    const RingRoots W(rt, R.n);
#pragma unroll
    for (int i = 0; i < K; ++i) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int m = 2 * (pl + 64 * i) + d;
            if (m > L) continue;
            double sw, cw;
            sincospi(2.0 * (double)(m % R.n) / (double)R.n, &sw, &cw);
            // s_{k-1} - e^{-i w} s_{k-2} of a real fold
            auto tail = [&](int f) {
                return make_double2(s1[i][f] - cw * s2[i][f], sw * s2[i][f]);
            };
            double2 E, O;
            if (d == 0) {
                E = tail(0);
                O = tail(1);
            } else {
                const double2 pe = tail(2), po = tail(3), qe = tail(4), qo = tail(5);
                const double g = (m & 3) == 1 ? 1.0 : -1.0;   // p -+ i q
                E = make_double2(fma(g, qe.y, pe.x), fma(-g, qe.x, pe.y));
                O = make_double2(fma(g, qo.y, po.x), fma(-g, qo.x, po.y));
            }
            const double2 ph = W.at(-m * (2 * (k - 1) + R.two_o));   // and e^{-i m phi_0}
            E = cmul(E, ph);
            O = cmul(O, ph);
            // Z(m) = E + i O, Z(-m) = conj E + i conj O
            row[order_slot(m, lq)] = make_double2(E.x - O.y, E.y + O.x);
            row[4 * lq + order_slot(m, lq)] = make_double2(E.x + O.y, -E.y + O.x);
        }
    }
}

// The inverse, y_j = Re sum_m H_m e^{i m a_j}, a_j = 2 pi j / n, H_m = c_m G_r(m) e^{i m phi_0},
// by classes: with u_c = sum_{m = c mod 4} H_m e^{i m a_j} the pixels of the four quarters are
// y_{j + tk} = Re sum_c i^{ct} u_c.  u_c is e^{i c a_j} times a sum in steps of b = 4 a_j =
// 2 pi j / k, from the real Clenshaw sums C = sum h cos, S = sum h sin of the real and imaginary
// parts (shared coefficient 2 cos b); at k - j the cosines are the same and the sines change
// sign.  So a thread obtains eight pixels from eight sums of lcut / 4 terms.  One workgroup per
// ring: of both rings of a pair (blockIdx.z) it is faster than in one workgroup, and on small maps,
// whose time is the chain of one workgroup, too.  FP64 issue bounds it elsewhere.
__host__ __device__ inline int dft_groups(int L) { return (L >> 2) + 1; }
static size_t dft_bwd_lds(int L) { return (size_t)4 * dft_groups(L) * sizeof(double2); }
__global__ __launch_bounds__(kShtThreads) void k_sht_dft_bwd(const ShtRing *__restrict__ rings,
                                                             const int *__restrict__ ring_list,
                                                             const double2 *__restrict__ roots,
                                                             const double2 *__restrict__ G,
                                                             float *__restrict__ out,
                                                             long long npix, int L, int lq,
                                                             int nnorth, int accumulate)
{
    extern __shared__ double2 H[];   // zero past lcut
    const int r = ring_list[blockIdx.x];
    const bool south = blockIdx.z != 0;
    if (south && r == nnorth - 1) return;   // the equator
    const ShtRing R = rings[r];
    const double2 *row = G + ((size_t)blockIdx.y * nnorth + r) * 8 * lq;
    const int A = dft_groups(L), k = R.n >> 2;
    __shared__ double2 rt[kRoots];
    load_roots(rt, roots);
    __syncthreads();
    const RingRoots W(rt, R.n);
    const double sign = south ? -1.0 : 1.0;
    for (int m = threadIdx.x; m < 4 * A; m += kShtThreads) {
        double2 h = make_double2(0.0, 0.0);
        if (m <= L) {
            const double2 e = row[order_slot(m, lq)], o = row[4 * lq + order_slot(m, lq)];
            const double c = m == 0 ? 1.0 : 2.0;
            h = cmul(make_double2(c * fma(sign, o.x, e.x), c * fma(sign, o.y, e.y)),
                     W.at(m * R.two_o));
        }
        H[m] = h;
    }
    __syncthreads();
    float *o = out + (size_t)blockIdx.y * npix + (south ? rings[2 * nnorth - 2 - r].first : R.first);
    for (int j = threadIdx.x; j <= k >> 1; j += kShtThreads) {
        double sb, cb;
        sincospi(2.0 * (double)j / (double)k, &sb, &cb);
        const double cc = 2.0 * cb;
        // b_a = h_a + 2 cos(b) b_{a+1} - b_{a+2} from a = A - 1 down to 1, two steps at
        // a time in place (b1 holds the newest term); an odd count starts from b_{A-1} = h_{A-1}
        double b1[4][2], b2[4][2];   // class; real and imaginary part
        const bool odd = (A & 1) == 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double2 ha = H[4 * (A - 1) + c];
            b1[c][0] = odd ? ha.x : 0.0;
            b1[c][1] = odd ? ha.y : 0.0;
            b2[c][0] = b2[c][1] = 0.0;
        }
        for (int a = odd ? A - 2 : A - 1; a > 1; a -= 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double2 ha = H[4 * a + c], hb = H[4 * a - 4 + c];
                b2[c][0] = fma(cc, b1[c][0], ha.x - b2[c][0]);
                b2[c][1] = fma(cc, b1[c][1], ha.y - b2[c][1]);
                b1[c][0] = fma(cc, b2[c][0], hb.x - b1[c][0]);
                b1[c][1] = fma(cc, b2[c][1], hb.y - b1[c][1]);
            }
        }
        // u_c at j, and at k - j, where e^{i c a} is i^c times the conjugate
        const double2 w1 = W.at(2 * j), w2 = cmul(w1, w1), w3 = cmul(w1, w2);
        double2 u[4], v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double2 h0 = H[c];
            const double Cr = fma(b1[c][0], cb, h0.x - b2[c][0]);
            const double Ci = fma(b1[c][1], cb, h0.y - b2[c][1]);
            const double Sr = sb * b1[c][0], Si = sb * b1[c][1];
            u[c] = make_double2(Cr - Si, Ci + Sr);
            v[c] = make_double2(Cr + Si, Ci - Sr);
            if (c > 0) {
                const double2 w = c == 1 ? w1 : (c == 2 ? w2 : w3);
                u[c] = cmul(u[c], w);
                v[c] = cmul(v[c], conj2(w));
            }
        }
#pragma unroll
        for (int side = 0; side < 2; ++side) {   // pixels j + tk, then k - j + tk
            const int jj = side ? k - j : j;
            if (side && (j == 0 || jj == j)) break;
            const double e = side ? v[0].x - v[2].x : u[0].x + u[2].x;
            const double f = side ? v[0].x + v[2].x : u[0].x - u[2].x;
            const double re = side ? v[3].y - v[1].y : u[1].x + u[3].x;
            const double im = side ? v[1].x + v[3].x : u[1].y - u[3].y;
            const double y[4] = {e + re, f - im, e - re, f + im};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int at = jj + t * k;
                o[at] = accumulate ? o[at] + (float)y[t] : (float)y[t];
            }
        }
    }
}

// ----------------------------------------------------------- Legendre --
// With c_l = sqrt((l^2 - m^2) / (4 l^2 - 1)), z lambda_l = c_{l+1} lambda_{l+1} +
// c_l lambda_{l-1}.  The functions p_k = lambda_{m+2k+1} / z are even in z, and
// both parities follow from them locally (Ishioka 2018):
//     lambda_{m+2k+1} = z p_k,   lambda_{m+2k} = c_{m+2k+1} p_k + c_{m+2k} p_{k-1}.
// Applying z twice gives a recurrence in steps of two degrees; scaled by
// constants nu_k, p_k = nu_k pi_k, it reads pi_{k+1} = (A_k z^2 + B_k) pi_k - pi_{k-1}.
// So two degrees of a ring pair cost two FMAs of recurrence and four of sums,
// against three and two per degree of the one-degree recurrence.
//
// lambda_mm of a ring times sqrt(2m + 3) (= p_0) in scaled form: returns the
// mantissa and sets sc.  pnorm[m] is log2 of the normalisation.
__device__ __forceinline__ double leg_start(double pnorm, int m, double log2s, int &sc)
{
    const double e = pnorm + (double)m * log2s;   // log2 p_0
    if (e >= -384.0) {
        sc = 0;
        return exp2(e);
    }
    sc = (int)floor((e + 384.0) / 512.0);          // mantissa in [2^-384, 2^128)
    return exp2(e - 512.0 * sc);
}

// Lane exchanges of the reduction below.
__device__ __forceinline__ double half_swap_add(double a, double b, bool rows16)
{
    // 32-lane (16-lane) halves: the lower lanes return the sum of a over both
    // halves, the upper ones that of b
    const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    v2u lo, hi;
    if (rows16) {
        lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
        hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false,
                                              false);
    } else {
        lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
        hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false,
                                              false);
    }
    return __longlong_as_double(((unsigned long long)hi.x << 32) | lo.x) +
           __longlong_as_double(((unsigned long long)hi.y << 32) | lo.y);
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const unsigned long long u = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xF, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
// Sums of sixteen values over the wave: lane l returns that of v[l >> 2].
// Each step halves the values a lane carries, so the reduction takes 17 adds
// instead of 96 and no LDS.
__device__ __forceinline__ double reduce16(double v[16])
{
    const int lane = (int)threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = half_swap_add(v[i], v[i + 8], false);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = half_swap_add(v[i], v[i + 4], true);
    const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        v[i] = (b3 ? v[i + 2] : v[i]) + dpp_move<0x128>(b3 ? v[i] : v[i + 2]);   // row_ror:8
    double s = (b2 ? v[1] : v[0]) + dpp_move<0x141>(b2 ? v[0] : v[1]);           // half mirror
    s += dpp_move<0x4E>(s);
    s += dpp_move<0xB1>(s);
    return s;
}

// Workgroup (order m, chunk of ring pairs, map): the sums S_k = sum pi_k E and
// T_k = sum pi_k z O over the chunk's ring pairs, with E = (Z(m) + conj Z(-m)) / 2
// and O = (Z(m) - conj Z(-m)) / 2i.  Chunks count from ring_lo[m], below which
// no ring contributes; a wave takes 64 R consecutive ring pairs, R per lane.
// What bounds it is vector issue: at Nside 2048 and lcut 1500 (0.87 ms) vector instructions take 0.69
// of the cycles at 2.4 GHz, 0.82 of those at the clock it runs at, and its FP64 work comes to 31 of
// the 72 TFLOP/s of a large matrix product.  The six FMAs per ring pair and two degrees, about
// 5.5 cycles each at nominal clock, are 0.43 ms; the reduction over the wave adds half of that at
// four ring pairs per lane, a quarter at eight; the rest is the test for scaled values, lanes beyond
// the ring range and, for a fifth of the time, waits for the coefficients.  Loading the next
// block's coefficients ahead was slower (the copies cost more than the waits).
template <int R>
__global__ __launch_bounds__(kShtThreads) __attribute__((amdgpu_waves_per_eu(R == 8 ? 2 : 4)))
void k_leg_fwd(const ShtRing *__restrict__ rings, const double2 *__restrict__ F,
               const double2 *__restrict__ ab_all, const double *__restrict__ pnorm,
               const int *__restrict__ ring_lo, const int *__restrict__ step_base,
               double *__restrict__ part_all, int L, int lq, int nnorth, int nsteps)
{
    __shared__ double ws[kShtThreads / 64][kLegFlush * 16];
    const int m = leg_order(blockIdx.x);
    if (m > L) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const int i0 = ring_lo[m] + (int)blockIdx.y * R * kShtThreads;
    if (i0 >= nnorth) return;
    const int first = i0 + 64 * R * wave;
    const bool idle = first >= nnorth;   // (wave-uniform)
    const int steps = leg_steps(m, L);
    const double2 *ab = ab_all + step_base[m];
    F += (size_t)blockIdx.z * nnorth * 8 * lq;
    double *part = part_all + 4 * (((size_t)blockIdx.y * gridDim.z + blockIdx.z) * nsteps + step_base[m]);
    double z2[R], p1[R], p0[R];
    double2 E[R], O[R];
    int sc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = first + 64 * q + lane;
        const int ii = min(i, nnorth - 1);
        const ShtRing Rg = rings[ii];
        const double2 *row = F + (size_t)ii * 8 * lq + order_slot(m, lq);
        const double2 zp = row[0], zm = row[4 * lq];
        const double w = i < nnorth ? 0.5 : 0.0, wz = w * Rg.z;
        E[q] = make_double2(w * (zp.x + zm.x), w * (zp.y - zm.y));
        O[q] = make_double2(wz * (zp.y + zm.y), wz * (zm.x - zp.x));
        z2[q] = Rg.z * Rg.z;
        p0[q] = 0.0;
        p1[q] = leg_start(pnorm[m], m, Rg.log2s, sc[q]);
    }
    int slot = 0, k0 = 0;
    for (int k = 0; k < steps; k += kLegBlock) {
        if (idle) {
            if (lane < 16) ws[wave][slot * 16 + lane] = 0.0;
        } else {
            double v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = 0.0;
            d2v c[kLegBlock];
#pragma unroll
            for (int j = 0; j < kLegBlock; ++j) c[j] = ((uptr<d2v>)ab)[k + j];
            bool scaled = false;
#pragma unroll
            for (int q = 0; q < R; ++q) scaled |= sc[q] < 0;
            if (!__any(scaled)) {
#pragma unroll
                for (int j = 0; j < kLegBlock; ++j) {
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const double p = p1[q];
                        v[4 * j] = fma(p, E[q].x, v[4 * j]);
                        v[4 * j + 1] = fma(p, E[q].y, v[4 * j + 1]);
                        v[4 * j + 2] = fma(p, O[q].x, v[4 * j + 2]);
                        v[4 * j + 3] = fma(p, O[q].y, v[4 * j + 3]);
                        p1[q] = fma(fma(c[j].x, z2[q], c[j].y), p, -p0[q]);
                        p0[q] = p;
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < kLegBlock; ++j) {
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const double p = p1[q];
                        const double u = sc[q] == 0 ? p : 0.0;
                        v[4 * j] = fma(u, E[q].x, v[4 * j]);
                        v[4 * j + 1] = fma(u, E[q].y, v[4 * j + 1]);
                        v[4 * j + 2] = fma(u, O[q].x, v[4 * j + 2]);
                        v[4 * j + 3] = fma(u, O[q].y, v[4 * j + 3]);
                        p1[q] = fma(fma(c[j].x, z2[q], c[j].y), p, -p0[q]);
                        p0[q] = p;
                    }
                }
                // a block grows a value by less than 2^100, far below the range
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    if (sc[q] < 0 && fabs(p1[q]) > kScaleUp) {
                        p1[q] *= kScaleStep;
                        p0[q] *= kScaleStep;
                        ++sc[q];
                    }
                }
            }
            const double s = reduce16(v);
            if ((lane & 3) == 0) ws[wave][slot * 16 + (lane >> 2)] = s;
        }
        if (++slot == kLegFlush || k + kLegBlock >= steps) {
            __syncthreads();
            for (int e = threadIdx.x; e < slot * 16; e += kShtThreads) {
                double t = ws[0][e];
#pragma unroll
                for (int w = 1; w < kShtThreads / 64; ++w) t += ws[w][e];
                part[(size_t)k0 * 4 + e] = t;
            }
            __syncthreads();
            k0 += slot * kLegBlock;
            slot = 0;
        }
    }
}

// From the sums S_k, T_k (over the ring chunks, in chunk order) the
// coefficients a_{m+2k} = c_{m+2k+1} nu_k S_k + c_{m+2k} nu_{k-1} S_{k-1} and
// a_{m+2k+1} = nu_k T_k, times Omega Khat_l, and from these the synthesis
// coefficients of pi_k (even: De_k = nu_k (a_{m+2k} c_{m+2k+1} + a_{m+2k+2}
// c_{m+2k+2})) and of z pi_k (odd: Do_k = nu_k a_{m+2k+1}).
__global__ __launch_bounds__(kShtThreads) void k_sht_mul(
    const double *__restrict__ part, const double *__restrict__ kscale,
    const double *__restrict__ nu, const int *__restrict__ ring_lo,
    const int *__restrict__ step_base, double4 *__restrict__ D, int L, int nnorth, int chunk,
    int nsteps)
{
    const int m = blockIdx.y, map = blockIdx.z;
    const int k = blockIdx.x * kShtThreads + threadIdx.x;
    if (k >= leg_steps(m, L)) return;
    const int base = step_base[m];
    const int nchunk = (nnorth - ring_lo[m] + chunk - 1) / chunk;
    auto sums = [&](int kk) {
        double4 t = make_double4(0.0, 0.0, 0.0, 0.0);
        if (kk < 0 || m + 2 * kk > L) return t;
        for (int c = 0; c < nchunk; ++c) {
            const double4 p = reinterpret_cast<const double4 *>(
                part)[((size_t)c * gridDim.z + map) * nsteps + base + kk];
            t.x += p.x;
            t.y += p.y;
            t.z += p.z;
            t.w += p.w;
        }
        const double v = nu[base + kk];
        t.x *= v;
        t.y *= v;
        t.z *= v;
        t.w *= v;
        return t;
    };
    auto coef = [&](int l) {   // c_l
        const double dl = l, dm = m;
        return sqrt((dl * dl - dm * dm) / (4.0 * dl * dl - 1.0));
    };
    const double4 sm = sums(k - 1), s0 = sums(k), sp = sums(k + 1);
    const int l = m + 2 * k;
    double4 d = make_double4(0.0, 0.0, 0.0, 0.0);
    if (l <= L) {
        const double ca = k > 0 ? coef(l) : 0.0, cb = coef(l + 1), cc = coef(l + 2),
                     cd = coef(l + 3), v = nu[base + k];
        const double ks0 = kscale[l];
        d.x = cb * ks0 * (cb * s0.x + ca * sm.x);
        d.y = cb * ks0 * (cb * s0.y + ca * sm.y);
        if (l + 2 <= L) {
            const double ks2 = kscale[l + 2];
            d.x = fma(cc * ks2, cd * sp.x + cc * s0.x, d.x);
            d.y = fma(cc * ks2, cd * sp.y + cc * s0.y, d.y);
        }
        d.x *= v;
        d.y *= v;
        if (l + 1 <= L) {
            d.z = v * kscale[l + 1] * s0.z;
            d.w = v * kscale[l + 1] * s0.w;
        }
    }
    D[(size_t)map * nsteps + base + k] = d;
}

// Workgroup (order m, chunk of ring pairs, map): the even and odd sums over l
// of the chunk's ring pairs, laid out as in k_leg_fwd; rings below ring_lo[m]
// get zeros.
template <int R>
__global__ __launch_bounds__(kShtThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_leg_bwd(const ShtRing *__restrict__ rings, const double4 *__restrict__ D_all,
               const double2 *__restrict__ ab_all, const double *__restrict__ pnorm,
               const int *__restrict__ ring_lo, const int *__restrict__ step_base,
               double2 *__restrict__ G, int L, int lq, int nnorth, int nsteps)
{
    const int m = leg_order(blockIdx.x);
    if (m > L) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const int lo = ring_lo[m], c0 = (int)blockIdx.y * R * kShtThreads;
    G += (size_t)blockIdx.z * nnorth * 8 * lq;
    for (int i = c0 + (int)threadIdx.x; i < min(c0 + R * kShtThreads, lo); i += kShtThreads) {
        double2 *row = G + (size_t)i * 8 * lq + order_slot(m, lq);
        row[0] = make_double2(0.0, 0.0);
        row[4 * lq] = make_double2(0.0, 0.0);
    }
    const int first = lo + c0 + 64 * R * wave;
    if (first >= nnorth) return;
    const int steps = leg_steps(m, L);
    const double2 *ab = ab_all + step_base[m];
    const double4 *D = D_all + (size_t)blockIdx.z * nsteps + step_base[m];
    double z2[R], p1[R], p0[R];
    double2 e[R], o[R];
    int sc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const ShtRing Rg = rings[min(first + 64 * q + lane, nnorth - 1)];
        z2[q] = Rg.z * Rg.z;
        p0[q] = 0.0;
        p1[q] = leg_start(pnorm[m], m, Rg.log2s, sc[q]);
        e[q] = o[q] = make_double2(0.0, 0.0);
    }
    for (int k = 0; k < steps; k += kLegBlock) {
        d2v c[kLegBlock];
        d4v d[kLegBlock];
#pragma unroll
        for (int j = 0; j < kLegBlock; ++j) {
            c[j] = ((uptr<d2v>)ab)[k + j];
            d[j] = ((uptr<d4v>)D)[k + j];
        }
        bool scaled = false;
#pragma unroll
        for (int q = 0; q < R; ++q) scaled |= sc[q] < 0;
        if (!__any(scaled)) {
#pragma unroll
            for (int j = 0; j < kLegBlock; ++j) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double p = p1[q];
                    e[q].x = fma(p, d[j].x, e[q].x);
                    e[q].y = fma(p, d[j].y, e[q].y);
                    o[q].x = fma(p, d[j].z, o[q].x);
                    o[q].y = fma(p, d[j].w, o[q].y);
                    p1[q] = fma(fma(c[j].x, z2[q], c[j].y), p, -p0[q]);
                    p0[q] = p;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < kLegBlock; ++j) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double p = p1[q];
                    const double u = sc[q] == 0 ? p : 0.0;
                    e[q].x = fma(u, d[j].x, e[q].x);
                    e[q].y = fma(u, d[j].y, e[q].y);
                    o[q].x = fma(u, d[j].z, o[q].x);
                    o[q].y = fma(u, d[j].w, o[q].y);
                    p1[q] = fma(fma(c[j].x, z2[q], c[j].y), p, -p0[q]);
                    p0[q] = p;
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if (sc[q] < 0 && fabs(p1[q]) > kScaleUp) {
                    p1[q] *= kScaleStep;
                    p0[q] *= kScaleStep;
                    ++sc[q];
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = first + 64 * q + lane;
        if (i >= nnorth) continue;
        const double z = rings[i].z;
        double2 *row = G + (size_t)i * 8 * lq + order_slot(m, lq);
        row[0] = e[q];
        row[4 * lq] = make_double2(z * o[q].x, z * o[q].y);
    }
}

// ---------------------------------------------------------------- host --
// Ring pairs of one FFT launch: those of similar FFT length, so that LDS and
// threads fit them.
struct ShtBucket {
    int first = 0, count = 0;   // entries of the plan's list
    int lg = 0;                 // log2 of the longest FFT
    int threads = 0;
    bool direct = false;
};

struct Harm {
    int nside = 0;
    int nrings = 0;
    int nnorth = 0;     // northern rings and the equator: 2 Nside
    int lcut = 0;
    int max_batch = 1;
    int nmaps = 1;      // maps of one pass over the kernels (workspace)
    int lq = 0;         // orders of one class mod 4, rounded up to whole lines
    int nchunk = 0;     // most ring chunks of k_leg_fwd
    int leg_r = 1;      // ring pairs per lane of k_leg_fwd
    int nsteps = 0;     // recurrence steps of all orders
    int device = -1;
    long long npix = 0;
    long long nalm = 0;
    double omega = 0.0;
    std::vector<double> khat;
    ShtRing *d_rings = nullptr;
    double2 *d_ab = nullptr;      // A_k, B_k of every order
    double *d_nu = nullptr;
    double *d_pnorm = nullptr;
    double *d_kscale = nullptr;
    int *d_ring_lo = nullptr;     // per m: first northern ring whose terms matter
    int *d_step_base = nullptr;   // per m: first step
    int *d_dft_rings = nullptr;   // rings of the direct sums
    ShtFftRing *d_fft_rings = nullptr;
    double2 *d_tw = nullptr;
    double2 *d_roots = nullptr;
    double2 *d_chirp = nullptr;
    std::vector<ShtBucket> buckets;
    int n_dft = 0, n_fft = 0, lgm = 0;
    double2 *d_F = nullptr;       // nmaps x nnorth rows: Z(m), Z(-m), then even, odd sums
    double *d_part = nullptr;     // nchunk x nmaps x nsteps x 4
    double4 *d_D = nullptr;       // nmaps x nsteps
    long long device_bytes = 0;
};

static void harm_free(Harm &h)
{
    if (h.device >= 0) {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(h.device);
        (void)hipDeviceSynchronize();
        for (void *p : {(void *)h.d_rings, (void *)h.d_ab, (void *)h.d_nu, (void *)h.d_pnorm,
                        (void *)h.d_kscale, (void *)h.d_ring_lo, (void *)h.d_step_base,
                        (void *)h.d_dft_rings, (void *)h.d_fft_rings, (void *)h.d_tw, (void *)h.d_roots,
                        (void *)h.d_chirp, (void *)h.d_F, (void *)h.d_part, (void *)h.d_D})
            if (p) (void)hipFree(p);
        (void)hipSetDevice(cur);
    }
    h.d_rings = nullptr;
    h.d_ab = nullptr;
    h.d_nu = nullptr;
    h.d_pnorm = nullptr;
    h.d_kscale = nullptr;
    h.d_ring_lo = nullptr;
    h.d_step_base = nullptr;
    h.d_dft_rings = nullptr;
    h.d_fft_rings = nullptr;
    h.d_tw = nullptr;
    h.d_roots = nullptr;
    h.d_chirp = nullptr;
    h.d_F = nullptr;
    h.d_part = nullptr;
    h.d_D = nullptr;
}

static int harm_alloc(void **p, size_t bytes, long long *total)
{
    if (hipMalloc(p, std::max<size_t>(bytes, 16)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ARKCOS_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    }
    *total += (long long)bytes;
    return ARKCOS_OK;
}

template <class T>
static int harm_upload(T **p, const std::vector<T> &v, long long *total)
{
    int rc = harm_alloc((void **)p, v.size() * sizeof(T), total);
    if (rc) return rc;
    if (!v.empty())
        ARKCOS_HIP_CHECK(hipMemcpy(*p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    return ARKCOS_OK;
}

static int harm_upload_kernel(Harm &h)
{
    std::vector<double> ks(h.lcut + 1);
    for (int l = 0; l <= h.lcut; ++l) ks[l] = h.omega * h.khat[l];
    ARKCOS_HIP_CHECK(hipMemcpy(h.d_kscale, ks.data(), ks.size() * sizeof(double),
                               hipMemcpyHostToDevice));
    return ARKCOS_OK;
}

// (belt rings without the chirp have at most 4096 points, 512 threads)
#define ARKCOS_RING_KERNEL(name)                                                             \
    static auto name##_kernel(const ShtBucket &B)                                            \
    {                                                                                        \
        switch (B.threads) {                                                                 \
            case 128: return B.direct ? k_##name<128, false> : k_##name<128, true>;          \
            case 256: return B.direct ? k_##name<256, false> : k_##name<256, true>;          \
            case 512: return B.direct ? k_##name<512, false> : k_##name<512, true>;          \
            default: return k_##name<1024, true>;                                            \
        }                                                                                    \
    }
ARKCOS_RING_KERNEL(ring_fwd)
ARKCOS_RING_KERNEL(ring_bwd)
#undef ARKCOS_RING_KERNEL

// Whether a ring pair of quarter length k takes the direct sums: their time grows with
// lcut, the FFTs' does not.  Measured per sample of a ring pair, both ways (Nside 512-4096, one map):
// direct 7.5 + 0.105 lcut ps; FFTs 21-26 ps on belts of k = 1024, 2048 and 4096, 54 ps on those of
// k = 512, 61 ps with the chirp transforms of k <= 2048 and 108-128 ps above (1024 threads, held to 128
// registers, of which they spill hundreds).  Nside 2048, lcut 100: 0.61 ms of direct sums for the
// whole half against 0.95 ms of FFTs; lcut 300: 1.23 against 1.03 ms; Nside 3000, lcut 100: 1.17
// against 5.69 ms.
static bool ring_direct(int k, bool belt, int lcut)
{
    if (k > kShtMaxK) return true;   // (the transform does not fit the LDS)
    if (belt) return lcut < (k >= 1024 ? 128 : 256);
    return lcut < (k > 2048 ? 1024 : 512);
}

// Ring pairs by FFT length, and those left to the direct sums.
static int harm_build_ffts(Harm &h, const std::vector<ShtRing> &rings)
{
    // Small maps take the direct sums on every ring, up to kShtDirectWork = npix (lcut + 1) of
    // a map: the FFT kernels are a long chain of short passes, whose start-up dominates there
    // (both ways at Nside 128, lcut 511: direct 29 us, FFTs 90 us; at Nside 256, lcut 255: 39 and 87 us).
    const bool use_fft = std::getenv("ARKCOS_SHT_NO_FFT") == nullptr &&
                         (double)h.npix * (h.lcut + 1) > kShtDirectWork;
    std::vector<int> dft;
    std::vector<ShtFftRing> list[5], spectra;   // (spectra: one entry per chirped length)
    long long chirp = 0;
    std::vector<long long> at((size_t)h.nside + 1, -1);   // chirp spectrum of length k
    for (int i = 0; i < h.nnorth; ++i) {
        const int k = rings[i].n / 4;
        // the belt rings without the chirp if they can; caps hold few power-of-two rings
        const bool direct = k == h.nside && k >= 8 && (k & (k - 1)) == 0;
        if (!use_fft || ring_direct(k, direct, h.lcut)) {
            dft.push_back(i);
            continue;
        }
        ShtFftRing q{};
        q.ring = i;
        q.k = k;
        q.lg = 3;
        while ((1 << q.lg) < (direct ? k : 2 * k - 1)) ++q.lg;
        if (!direct) {
            if (at[k] < 0) {
                at[k] = chirp;
                q.chirp = (int)chirp;
                chirp += 1LL << q.lg;
                spectra.push_back(q);
            }
            q.chirp = (int)at[k];
        }
        h.lgm = std::max(h.lgm, q.lg);
        // chirped, by FFT length: up to 1024, 2048, 4096, longer; then direct
        list[direct ? 4 : (q.lg <= 10 ? 0 : q.lg - 10)].push_back(q);
    }
    h.lgm = std::max(h.lgm, 5);
    std::reverse(dft.begin(), dft.end());   // longest first
    std::vector<ShtFftRing> all;
    for (int b = 0; b < 5; ++b) {
        if (list[b].empty()) continue;
        ShtBucket B;
        B.first = (int)all.size();
        B.count = (int)list[b].size();
        for (const ShtFftRing &q : list[b]) B.lg = std::max(B.lg, q.lg);
        B.direct = b == 4;
        B.threads = std::max(128, (1 << B.lg) / 8);   // a radix-8 butterfly each
        // longest first (equatorward rings), so that the last workgroups are short
        std::stable_sort(list[b].begin(), list[b].end(),
                         [](const ShtFftRing &p, const ShtFftRing &q) { return p.k > q.k; });
        all.insert(all.end(), list[b].begin(), list[b].end());
        h.buckets.push_back(B);
    }
    h.n_dft = (int)dft.size();
    h.n_fft = (int)all.size();
    const int Pm = 1 << h.lgm;
    std::vector<double2> tw(Pm / 4);
    for (int t = 0; t < Pm / 4; ++t)
        tw[t] = make_double2(std::cos(2.0 * M_PI * t / Pm), -std::sin(2.0 * M_PI * t / Pm));
    int rc;
    if ((rc = harm_upload(&h.d_dft_rings, dft, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_fft_rings, all, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_tw, tw, &h.device_bytes))) return rc;
    std::vector<double2> roots(kRoots);
    for (int t = 0; t < kRoots; ++t)
        roots[t] = make_double2(std::cos(2.0 * M_PI * t / kRoots), std::sin(2.0 * M_PI * t / kRoots));
    if ((rc = harm_upload(&h.d_roots, roots, &h.device_bytes))) return rc;
    if ((rc = harm_alloc((void **)&h.d_chirp, (size_t)chirp * sizeof(double2), &h.device_bytes)))
        return rc;
    const int lds = (int)fft_lds_bytes(h.lgm);
    ARKCOS_HIP_CHECK(hipFuncSetAttribute((const void *)k_chirp,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    for (const ShtBucket &B : h.buckets)
        for (const void *f : {(const void *)ring_fwd_kernel(B), (const void *)ring_bwd_kernel(B)})
            ARKCOS_HIP_CHECK(
                hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    if (h.n_dft > 0)
        ARKCOS_HIP_CHECK(hipFuncSetAttribute((const void *)k_sht_dft_bwd,
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)dft_bwd_lds(h.lcut)));
    if (!spectra.empty()) {
        ShtFftRing *d = nullptr;
        long long bytes = 0;
        if ((rc = harm_upload(&d, spectra, &bytes))) return rc;
        hipLaunchKernelGGL(k_chirp, dim3((unsigned)spectra.size()), dim3(1024), lds, nullptr, d,
                           h.d_tw, h.d_roots, h.d_chirp, h.lgm);
        const hipError_t e = hipGetLastError() == hipSuccess ? hipStreamSynchronize(nullptr)
                                                             : hipErrorLaunchFailure;
        (void)hipFree(d);
        ARKCOS_HIP_CHECK(e);
    }
    return ARKCOS_OK;
}

static int harm_build(Harm &h)
{
    const int L = h.lcut;
    std::vector<ShtRing> rings(h.nrings);
    for (int i = 0; i < h.nrings; ++i) {
        const HostRing g = ring_geometry(h.nside, i + 1);
        rings[i].z = g.z;
        rings[i].s = g.s;
        rings[i].log2s = std::log2(g.s);
        rings[i].n = g.n;
        rings[i].first = (int)g.first;
        rings[i].two_o = g.two_o;
        rings[i].pad = 0;
    }
    // Recurrence tables.  With l = m + 2k + 1, z^2 p_k = c_{l+1} c_{l+2} p_{k+1} +
    // (c_{l+1}^2 + c_l^2) p_k + c_l c_{l-1} p_{k-1}; nu_{k+1} = nu_{k-1} c_l c_{l-1} /
    // (c_{l+1} c_{l+2}) makes the last coefficient 1.
    std::vector<int> step_base(L + 2, 0);
    for (int m = 0; m <= L; ++m) step_base[m + 1] = step_base[m] + leg_steps(m, L);
    h.nsteps = step_base[L + 1];
    std::vector<double2> ab((size_t)h.nsteps, make_double2(0.0, 0.0));
    std::vector<double> nu((size_t)h.nsteps, 0.0), pnorm(L + 1), c2(L + 8);
    double acc = -std::log2(4.0 * M_PI);
    for (int m = 0; m <= L; ++m) {
        if (m > 0) acc += std::log2((2.0 * m + 1.0) / (2.0 * m));
        pnorm[m] = 0.5 * (acc + std::log2(2.0 * m + 3.0));
        for (int l = m; l <= L + 5; ++l)   // c_l^2
            c2[l] = ((double)l - m) * ((double)l + m) / (4.0 * l * l - 1.0);
        double v0 = 1.0, v1 = 1.0;   // nu_k, nu_{k+1}
        const int base = step_base[m];
        for (int k = 0; m + 2 * k <= L; ++k) {
            const int l = m + 2 * k + 1;
            const double g = std::sqrt(c2[l + 1] * c2[l + 2]);
            const double A = v0 / (v1 * g);
            ab[base + k] = make_double2(A, -(c2[l + 1] + c2[l]) * A);
            nu[base + k] = v0;
            // nu_{k+2} = nu_k c_{l+2} c_{l+1} / (c_{l+3} c_{l+4})
            const double next = v0 * g / std::sqrt(c2[l + 3] * c2[l + 4]);
            v0 = v1;
            v1 = next;
        }
    }
    // Per order m, the first northern ring (rings run from the pole to the
    // equator, sin theta increasing) on which some p_k exceeds 2^-394: below it
    // every term is negligible and the Legendre kernels skip the ring.  For
    // fixed l and m, |lambda_lm| grows with sin theta until the oscillatory
    // range, so the rings that matter are a suffix and a bisection finds its
    // start.
    std::vector<int> ring_lo(L + 1, 0);
    auto matters = [&](int i, int m) {
        const ShtRing &Rg = rings[i];
        const double e = pnorm[m] + m * Rg.log2s;      // log2 p_0
        if (e > -394.0) return true;
        double scale = std::floor(e);               // |pi_k| = v1 2^scale
        double v1 = std::exp2(e - scale);
        double v2 = 0.0;
        const int base = step_base[m];
        const double z2 = Rg.z * Rg.z;
        for (int k = 0; m + 2 * k <= L; ++k) {
            const double v = (ab[base + k].x * z2 + ab[base + k].y) * v1 - v2;
            v2 = v1;
            v1 = v;
            const double av = std::fabs(v1);
            if (av > 0x1p200 || (av < 0x1p-200 && v1 != 0.0)) {
                int ex = 0;
                std::frexp(v1, &ex);
                v1 = std::ldexp(v1, -ex);
                v2 = std::ldexp(v2, -ex);
                scale += ex;
            }
            // (log2 |v1| <= 200 after the rescale)
            if (scale > -594.0 && v1 != 0.0 && std::log2(std::fabs(v1)) + scale > -394.0)
                return true;
        }
        return false;
    };
    for (int m = 0; m <= L; ++m) {
        int lo = 0, hi = h.nnorth - 1;           // first index in [lo, hi] that matters
        if (!matters(hi, m)) {
            ring_lo[m] = hi;
            continue;
        }
        while (lo < hi) {
            const int mid = lo + (hi - lo) / 2;
            if (matters(mid, m)) hi = mid; else lo = mid + 1;
        }
        ring_lo[m] = lo;
    }
    h.lq = ((L >> 2) + 8) & ~7;
    // maps that pass through the kernels together: small maps fill the chip only
    // as a group, and a group's workspace (rows, partial sums and coefficients, of
    // which the last two grow as lcut^2 at any Nside) stays below 512 MB
    const size_t rows = (size_t)h.nnorth * 8 * h.lq * sizeof(double2);
    const size_t coefs = (size_t)(h.nchunk + 1) * h.nsteps * sizeof(double4);
    h.nmaps = (int)std::max<size_t>(
        1, std::min<size_t>({(size_t)h.max_batch, 64, (512u << 20) / (rows + coefs)}));
    ARKCOS_HIP_CHECK(hipGetDevice(&h.device));
    int rc;
    if ((rc = harm_upload(&h.d_rings, rings, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_ab, ab, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_nu, nu, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_pnorm, pnorm, &h.device_bytes))) return rc;
    if ((rc = harm_alloc((void **)&h.d_kscale, (L + 1) * sizeof(double), &h.device_bytes)))
        return rc;
    if ((rc = harm_upload(&h.d_ring_lo, ring_lo, &h.device_bytes))) return rc;
    if ((rc = harm_upload(&h.d_step_base, step_base, &h.device_bytes))) return rc;
    if ((rc = harm_build_ffts(h, rings))) return rc;
    if ((rc = harm_alloc((void **)&h.d_F, (size_t)h.nmaps * rows, &h.device_bytes))) return rc;
    if ((rc = harm_alloc((void **)&h.d_part,
                         (size_t)h.nchunk * h.nmaps * h.nsteps * 4 * sizeof(double),
                         &h.device_bytes)))
        return rc;
    if ((rc = harm_alloc((void **)&h.d_D, (size_t)h.nmaps * h.nsteps * sizeof(double4),
                         &h.device_bytes)))
        return rc;
    return harm_upload_kernel(h);
}

// The kernels for nb <= nmaps maps.
static int harm_launch(const Harm &h, const float *in, float *out, int nb, int accumulate,
                       hipStream_t s)
{
    const int L = h.lcut;
    for (const ShtBucket &B : h.buckets) {
        hipLaunchKernelGGL(ring_fwd_kernel(B), dim3(B.count, nb), dim3(B.threads), fft_lds_bytes(B.lg), s, h.d_rings,
                           h.d_fft_rings + B.first, h.d_tw, h.d_roots, h.d_chirp, h.lgm,
                           in, h.npix, h.d_F, L, h.lq, h.nnorth);
    }
    // pairs of orders per thread, kShtMaxPairs per launch
    for (int p0 = 0, left = L / 2 / kShtThreads + 1; h.n_dft > 0 && left > 0;
         p0 += kShtMaxPairs * kShtThreads, left -= kShtMaxPairs) {
        switch (std::min(left, kShtMaxPairs)) {
#define ARKCOS_DFT_CASE(K)                                                                   \
    case K:                                                                                  \
        hipLaunchKernelGGL(k_sht_dft_fwd<K>, dim3(h.n_dft, nb), dim3(kShtThreads), 0, s,    \
                           h.d_rings, h.d_dft_rings, h.d_roots, in, h.npix, h.d_F, p0, L, \
                           h.lq, h.nnorth);                                                       \
        break;
            ARKCOS_DFT_CASE(1) ARKCOS_DFT_CASE(2) ARKCOS_DFT_CASE(3)
            default: ARKCOS_DFT_CASE(4)
#undef ARKCOS_DFT_CASE
        }
    }
    auto lf = h.leg_r == 1 ? k_leg_fwd<1> : (h.leg_r == 2 ? k_leg_fwd<2> : k_leg_fwd<kLegFwdRings>);
    auto lb = h.leg_r == 1 ? k_leg_bwd<1> : (h.leg_r == 2 ? k_leg_bwd<2> : k_leg_bwd<kLegBwdRings>);
    const int cf = kShtThreads * h.leg_r;
    const int cb = kShtThreads * std::min(h.leg_r, kLegBwdRings);
    hipLaunchKernelGGL(lf, dim3(leg_grid(L), (h.nnorth + cf - 1) / cf, nb), dim3(kShtThreads), 0, s,
                       h.d_rings, h.d_F, h.d_ab, h.d_pnorm, h.d_ring_lo, h.d_step_base, h.d_part,
                       L, h.lq, h.nnorth, h.nsteps);
    hipLaunchKernelGGL(k_sht_mul, dim3((leg_steps(0, L) + kShtThreads - 1) / kShtThreads, L + 1, nb),
                       dim3(kShtThreads), 0, s, h.d_part, h.d_kscale, h.d_nu, h.d_ring_lo,
                       h.d_step_base, h.d_D, L, h.nnorth, cf, h.nsteps);
    hipLaunchKernelGGL(lb, dim3(leg_grid(L), (h.nnorth + cb - 1) / cb, nb), dim3(kShtThreads), 0, s,
                       h.d_rings, h.d_D, h.d_ab, h.d_pnorm, h.d_ring_lo, h.d_step_base, h.d_F, L,
                       h.lq, h.nnorth, h.nsteps);
    for (const ShtBucket &B : h.buckets) {
        hipLaunchKernelGGL(ring_bwd_kernel(B), dim3(B.count, nb), dim3(B.threads), fft_lds_bytes(B.lg), s,
                           h.d_rings, h.d_fft_rings + B.first, h.d_tw, h.d_roots, h.d_chirp,
                           h.lgm, h.d_F, out, h.npix, L, h.lq, h.nnorth, accumulate);
    }
    if (h.n_dft > 0)
        hipLaunchKernelGGL(k_sht_dft_bwd, dim3(h.n_dft, nb, 2), dim3(kShtThreads),
                           dft_bwd_lds(L), s, h.d_rings, h.d_dft_rings,
                           h.d_roots, h.d_F, out, h.npix, L, h.lq, h.nnorth, accumulate);
    ARKCOS_HIP_CHECK(hipGetLastError());
    return ARKCOS_OK;
}

static bool overlap(const float *a, const float *b, long long n)
{
    return a < b + n && b < a + n;
}

}  // namespace arkcos

using namespace arkcos;

extern "C" {

int arkcos_harm_create(int nside, int lcut, const double *khat, int max_batch,
                       arkcos_harm_t *out)
{
    clear_error();
    if (!out) return fail(ARKCOS_EINVAL, "NULL output pointer");
    *out = nullptr;
    if (nside < 1 || nside > ARKCOS_MAX_NSIDE)
        return fail(ARKCOS_EINVAL, "nside must lie in 1.." + std::to_string(ARKCOS_MAX_NSIDE));
    if (lcut < 0) return fail(ARKCOS_EINVAL, "lcut must be >= 0");
    if (lcut > ARKCOS_MAX_LCUT)
        return fail(ARKCOS_EUNSUPPORTED, "lcut above " + std::to_string(ARKCOS_MAX_LCUT));
    if (!khat) return fail(ARKCOS_EINVAL, "NULL khat");
    if (max_batch < 1) return fail(ARKCOS_EINVAL, "max_batch must be >= 1");
    Harm *h = new (std::nothrow) Harm();
    if (!h) return fail(ARKCOS_ENOMEM, "host allocation failed");
    h->nside = nside;
    h->nrings = 4 * nside - 1;
    h->nnorth = 2 * nside;
    h->lcut = lcut;
    h->max_batch = max_batch;
    h->npix = 12LL * nside * nside;
    h->omega = 4.0 * M_PI / (double)h->npix;
    h->nalm = (long long)(lcut + 1) * (lcut + 2) / 2;
    // more ring pairs per lane share the coefficients and the reduction; small
    // maps need the waves instead (at 600 ring pairs two per lane run 6 % faster
    // than four, at 4096 eight 4 % faster than four)
    h->leg_r = h->nnorth >= 1024 ? kLegFwdRings : (h->nnorth >= 512 ? 2 : 1);
    h->nchunk = (h->nnorth + kShtThreads * h->leg_r - 1) / (kShtThreads * h->leg_r);
    int rc;
    try {
        h->khat.assign(khat, khat + lcut + 1);
        rc = harm_build(*h);
    } catch (const std::bad_alloc &) {
        rc = fail(ARKCOS_ENOMEM, "host allocation failed while building the transform plan");
    }
    if (rc != ARKCOS_OK) {
        harm_free(*h);
        delete h;
        return rc;
    }
    *out = reinterpret_cast<arkcos_harm_t>(h);
    return ARKCOS_OK;
}

int arkcos_harm_destroy(arkcos_harm_t harm)
{
    clear_error();
    if (!harm) return ARKCOS_OK;
    Harm *h = reinterpret_cast<Harm *>(harm);
    harm_free(*h);
    delete h;
    return ARKCOS_OK;
}

int arkcos_harm_set_kernel(arkcos_harm_t harm, const double *khat)
{
    clear_error();
    if (!harm || !khat) return fail(ARKCOS_EINVAL, "NULL pointer");
    Harm *h = reinterpret_cast<Harm *>(harm);
    h->khat.assign(khat, khat + h->lcut + 1);
    int cur = 0;
    ARKCOS_HIP_CHECK(hipGetDevice(&cur));
    ARKCOS_HIP_CHECK(hipSetDevice(h->device));
    int rc = harm_upload_kernel(*h);
    (void)hipSetDevice(cur);
    return rc;
}

int arkcos_harm_get_info(arkcos_harm_t harm, int *nside, int *lcut, long long *nalm,
                         long long *device_bytes)
{
    clear_error();
    if (!harm) return fail(ARKCOS_EINVAL, "NULL transform plan");
    const Harm *h = reinterpret_cast<const Harm *>(harm);
    if (nside) *nside = h->nside;
    if (lcut) *lcut = h->lcut;
    if (nalm) *nalm = h->nalm;
    if (device_bytes) *device_bytes = h->device_bytes;
    return ARKCOS_OK;
}

int arkcos_harm_convolve(arkcos_harm_t harm, const float *d_in, float *d_out, int nbatch,
                         int accumulate, void *stream)
{
    clear_error();
    TraceRange tr("arkcos_harm_convolve");
    if (!harm || !d_in || !d_out) return fail(ARKCOS_EINVAL, "NULL pointer");
    const Harm *h = reinterpret_cast<const Harm *>(harm);
    if (nbatch < 1 || nbatch > h->max_batch)
        return fail(ARKCOS_EINVAL, "nbatch must lie in 1.." + std::to_string(h->max_batch));
    if (accumulate != 0 && accumulate != 1) return fail(ARKCOS_EINVAL, "accumulate must be 0 or 1");
    if (overlap(d_in, d_out, h->npix * nbatch))
        return fail(ARKCOS_EINVAL, "d_in and d_out overlap");
    for (int b = 0; b < nbatch; b += h->nmaps) {
        int rc = harm_launch(*h, d_in + (size_t)b * h->npix, d_out + (size_t)b * h->npix,
                             std::min(h->nmaps, nbatch - b), accumulate, (hipStream_t)stream);
        if (rc) return rc;
    }
    return ARKCOS_OK;
}

int arkcos_split_convolve(arkcos_plan_t plan, arkcos_harm_t harm, const float *d_in,
                          float *d_out, int nbatch, void *stream)
{
    clear_error();
    TraceRange tr("arkcos_split_convolve");
    if (!plan || !harm) return fail(ARKCOS_EINVAL, "NULL plan");
    const Plan *P = reinterpret_cast<const Plan *>(plan);
    const Harm *h = reinterpret_cast<const Harm *>(harm);
    if (P->nside != h->nside)
        return fail(ARKCOS_EINVAL, "the two halves are planned for different Nside");
    int rc = arkcos_convolve(plan, d_in, d_out, nbatch, stream);
    if (rc) return rc;
    return arkcos_harm_convolve(harm, d_in, d_out, nbatch, 1, stream);
}

}  // extern "C"
