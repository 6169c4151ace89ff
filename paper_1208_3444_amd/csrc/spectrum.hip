// Velocity power spectrum of tracer tracks: for each tracer, the periodogram
// of its velocity series over the track's rows (the power spectrum of a
// single particle's velocity that Section I names as the method's goal),
//   E(k) = (1/M) sum_c | sum_{n<M} w_c[n] exp(-2 pi i k n / M) |^2,  k <= M/2.
//
// M, the number of grid points of a run, is any integer.  From kDirectRows
// rows on the transform is Bluestein's (IEEE Trans. Audio Electroacoust. 18, 451
// (1970)): with k n = (k^2 + n^2 - (k - n)^2) / 2 it is the convolution of
// w[n] c[n], c[n] = exp(-i pi n^2 / M), with conj(c), taken by FFTs of length
// L, the power of two at or above 2 M - 1, in one workgroup's LDS (up to
// kMaxFftRows rows).  A tracer's x and y components make one complex series
// (its real and imaginary part), z another; the powers of the two real series
// add up to (|Z(k)|^2 + |Z(M - k)|^2) / 2, so they need not be separated, and
// the last product with c (modulus 1) falls away.  Series of different
// tracers never mix: a NaN stays with its tracer.
//
// The FFT works in place: decimation in frequency forward, leaving the result
// in digit-reversed order, the product with the convolution kernel's transform
// in that order, decimation in time back.  A thread holds eight points, one
// radix-8 butterfly a pass (the first pass radix 2 or 4 where L is not a power
// of 8), and the middle passes on either side of the product stay in its
// registers.  LDS words are padded by one in eight, which keeps every stride
// free of bank conflicts.  The table of roots, chirp and kernel transform is made
// by one workgroup before every call (about 6 us), so that a call captured in
// a graph holds all it needs.
//
// Fewer rows, and more than kMaxFftRows, take a direct transform: one thread
// per (tracer, k), O(M^2); a block covers 256 consecutive k of one tracer and
// stages the tracer's three velocity columns through LDS in chunks; twiddles
// from a table indexed by k n reduced modulo M exactly.  It waits on the table
// (one load per row and thread).
// Measured, direct / FFT: 512 tracers, 1001 rows 302 / 29 us, 2001 rows 1232 /
// 74 us; 64 tracers, 301 rows 20.5 / 14.1 us, 4096 rows 1394 / 125 us; below
// about 160 rows both are bound by their two launches (12-13 us).  4096 rows
// fill a CU's LDS.
// Accuracy, direct / FFT, against extended precision, 1001 rows: noise 1.3e-15 /
// 7e-16 of the mean power (rms), a decaying velocity 2e-14 / 5e-15; in bins far
// below the strongest the FFT's rounding floor is the higher one, about twice in
// amplitude (1e-15 of the series' norm).
#include "colatus_internal.h"

#include <hip/hip_runtime.h>

namespace colatus {

namespace {

constexpr int kSpecThreads = 256;
constexpr int kSpecChunk = 1024;  // rows staged per LDS pass (24 KB)

// W[j] = exp(-2 pi i j / M) as (cos, -sin), j < M.
__global__ void twiddle_kernel(double2 *__restrict__ W, int64_t M)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= M)
        return;
    double s, c;
    sincospi(2.0 * ((double)j / (double)M), &s, &c);
    W[j] = make_double2(c, -s);
}

__global__ __launch_bounds__(kSpecThreads) void spectrum_kernel(
    const double *__restrict__ track, int64_t M, int32_t T, int remove_mean,
    const double2 *__restrict__ W, int64_t K, int64_t k_blocks, double *__restrict__ out)
{
    __shared__ double wv[3][kSpecChunk];
    __shared__ double red[3][kSpecThreads];
    const int64_t t = blockIdx.x / k_blocks;
    const int64_t k = (blockIdx.x % k_blocks) * kSpecThreads + threadIdx.x;
    const int tid = threadIdx.x;
    const int64_t row = 6 * (int64_t)T;
    const double *v0 = track + 3 * (int64_t)T + t;  // v_c of tracer t at row n: v0[n row + c T]

    double mu[3] = {0.0, 0.0, 0.0};
    if (remove_mean) {
        // fixed-order block sum: strided partial per thread, then a tree
        double s[3] = {0.0, 0.0, 0.0};
        for (int64_t n = tid; n < M; n += kSpecThreads)
            for (int c = 0; c < 3; ++c)
                s[c] += v0[n * row + c * (int64_t)T];
        for (int c = 0; c < 3; ++c)
            red[c][tid] = s[c];
        __syncthreads();
        for (int h = kSpecThreads / 2; h > 0; h >>= 1) {
            if (tid < h)
                for (int c = 0; c < 3; ++c)
                    red[c][tid] += red[c][tid + h];
            __syncthreads();
        }
        for (int c = 0; c < 3; ++c)
            mu[c] = red[c][0] / (double)M;
    }

    double re[3] = {0.0, 0.0, 0.0}, im[3] = {0.0, 0.0, 0.0};
    const int64_t kk = k < K ? k : 0;  // idle lanes still stage and sync
    int64_t j = 0;                     // k n mod M
    for (int64_t n0 = 0; n0 < M; n0 += kSpecChunk) {
        const int len = (int)(M - n0 < kSpecChunk ? M - n0 : kSpecChunk);
        __syncthreads();
        for (int q = tid; q < len; q += kSpecThreads)
            for (int c = 0; c < 3; ++c)
                wv[c][q] = v0[(n0 + q) * row + c * (int64_t)T] - mu[c];
        __syncthreads();
        for (int q = 0; q < len; ++q) {
            const double2 w = W[j];
            for (int c = 0; c < 3; ++c) {
                re[c] = fma(wv[c][q], w.x, re[c]);
                im[c] = fma(wv[c][q], w.y, im[c]);
            }
            j += kk;
            if (j >= M)
                j -= M;
        }
    }
    if (k < K) {
        double e = 0.0;
        for (int c = 0; c < 3; ++c)
            e += re[c] * re[c] + im[c] * im[c];
        out[t * K + k] = e / (double)M;
    }
}

// ---------------------------------------------------------------------------
// The in-place FFT of one thread group of L / 8 threads.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b)
{
    return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 csub(double2 a, double2 b)
{
    return make_double2(a.x - b.x, a.y - b.y);
}
// a times -i (forward) or +i (back)
template <bool FWD> __device__ __forceinline__ double2 crot(double2 a)
{
    return FWD ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}

template <bool FWD> __device__ __forceinline__ void dft2(double2 &a, double2 &b)
{
    const double2 t = csub(a, b);
    a = cadd(a, b);
    b = t;
}

// y_q = sum_k x_k W_4^{k q}, in place
template <bool FWD>
__device__ __forceinline__ void dft4(double2 &x0, double2 &x1, double2 &x2, double2 &x3)
{
    const double2 a = cadd(x0, x2), b = csub(x0, x2), c = cadd(x1, x3),
                  d = crot<FWD>(csub(x1, x3));
    x0 = cadd(a, c);
    x1 = cadd(b, d);
    x2 = csub(a, c);
    x3 = csub(b, d);
}

// y_q = sum_k x_k W_8^{k q}, in place: two transforms of four, even and odd k
template <bool FWD> __device__ __forceinline__ void dft8(double2 (&x)[8])
{
    constexpr double h = 0.70710678118654752440;
    dft4<FWD>(x[0], x[2], x[4], x[6]);
    dft4<FWD>(x[1], x[3], x[5], x[7]);
    // odd part times W_8^q = (h, -+h), -+i, (-h, -+h)
    const double2 o1 = x[3], o3 = x[7];
    const double2 t1 = FWD ? make_double2(h * (o1.x + o1.y), h * (o1.y - o1.x))
                           : make_double2(h * (o1.x - o1.y), h * (o1.y + o1.x));
    const double2 t2 = crot<FWD>(x[5]);
    const double2 t3 = FWD ? make_double2(h * (o3.y - o3.x), -h * (o3.x + o3.y))
                           : make_double2(-h * (o3.x + o3.y), h * (o3.x - o3.y));
    const double2 e0 = x[0], e1 = x[2], e2 = x[4], e3 = x[6], o0 = x[1];
    x[0] = cadd(e0, o0);
    x[4] = csub(e0, o0);
    x[1] = cadd(e1, t1);
    x[5] = csub(e1, t1);
    x[2] = cadd(e2, t2);
    x[6] = csub(e2, t2);
    x[3] = cadd(e3, t3);
    x[7] = csub(e3, t3);
}

// powers w^1 .. w^7 of w (conjugated on the way back)
template <bool FWD> __device__ __forceinline__ void powers(double2 w, double2 (&p)[8])
{
    if (!FWD)
        w.y = -w.y;
    p[1] = w;
    p[2] = cmul(w, w);
    p[3] = cmul(p[2], w);
    p[4] = cmul(p[2], p[2]);
    p[5] = cmul(p[4], w);
    p[6] = cmul(p[3], p[3]);
    p[7] = cmul(p[4], p[3]);
}

__device__ __forceinline__ int padded(int i) { return i + (i >> 3); }

template <int LOG> struct Fft {
    static constexpr int L = 1 << LOG;
    static constexpr int TG = L / 8;                   // threads
    static constexpr int R0 = 1 << (LOG % 3);          // radix of the first pass (1: none)
    static constexpr int kWords = L + L / 8;           // padded length

    // forward passes but the last (stride 1), on buf; root: exp(-2 pi i j / L)
    static __device__ __forceinline__ void forward(double2 *buf, const double2 *root, int t)
    {
        if constexpr (R0 > 1) {
            constexpr int s = L / R0;
#pragma unroll
            for (int b = 0; b < 8 / R0; ++b) {
                const int j = t + b * TG;
                double2 x[4];
#pragma unroll
                for (int k = 0; k < R0; ++k)
                    x[k] = buf[padded(j + k * s)];
                const double2 w = root[j];
                if constexpr (R0 == 2) {
                    dft2<true>(x[0], x[1]);
                    x[1] = cmul(x[1], w);
                } else {
                    dft4<true>(x[0], x[1], x[2], x[3]);
                    const double2 w2 = cmul(w, w);
                    x[1] = cmul(x[1], w);
                    x[2] = cmul(x[2], w2);
                    x[3] = cmul(x[3], cmul(w2, w));
                }
#pragma unroll
                for (int k = 0; k < R0; ++k)
                    buf[padded(j + k * s)] = x[k];
            }
            __syncthreads();
        }
#pragma unroll
        for (int n = L / R0; n > 8; n /= 8) {
            const int s = n / 8, j = t % s, base = (t / s) * n + j;
            double2 x[8], p[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                x[k] = buf[padded(base + k * s)];
            powers<true>(root[j * (L / n)], p);
            dft8<true>(x);
            buf[padded(base)] = x[0];
#pragma unroll
            for (int k = 1; k < 8; ++k)
                buf[padded(base + k * s)] = cmul(x[k], p[k]);
            __syncthreads();
        }
    }

    // the inverse passes but the first (stride 1)
    static __device__ __forceinline__ void backward(double2 *buf, const double2 *root, int t)
    {
#pragma unroll
        for (int n = 64; n <= L / R0; n *= 8) {
            __syncthreads();
            const int s = n / 8, j = t % s, base = (t / s) * n + j;
            double2 x[8], p[8];
            powers<false>(root[j * (L / n)], p);
            x[0] = buf[padded(base)];
#pragma unroll
            for (int k = 1; k < 8; ++k)
                x[k] = cmul(buf[padded(base + k * s)], p[k]);
            dft8<false>(x);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                buf[padded(base + k * s)] = x[k];
        }
        if constexpr (R0 > 1) {
            __syncthreads();
            constexpr int s = L / R0;
#pragma unroll
            for (int b = 0; b < 8 / R0; ++b) {
                const int j = t + b * TG;
                double2 x[4];
                double2 w = root[j];
                w.y = -w.y;
                x[0] = buf[padded(j)];
                x[1] = cmul(buf[padded(j + s)], w);
                if constexpr (R0 == 2) {
                    dft2<false>(x[0], x[1]);
                } else {
                    const double2 w2 = cmul(w, w);
                    x[2] = cmul(buf[padded(j + 2 * s)], w2);
                    x[3] = cmul(buf[padded(j + 3 * s)], cmul(w2, w));
                    dft4<false>(x[0], x[1], x[2], x[3]);
                }
#pragma unroll
                for (int k = 0; k < R0; ++k)
                    buf[padded(j + k * s)] = x[k];
            }
        }
        __syncthreads();
    }
};

// exp(-i pi n^2 / M), n^2 reduced modulo 2 M exactly
__device__ __forceinline__ double2 chirp(int n, int M)
{
    const int r = (int)(((int64_t)n * n) % (2 * (int64_t)M));
    double s, c;
    sincospi((double)r / (double)M, &s, &c);
    return make_double2(c, -s);
}

// One workgroup: table = [roots exp(-2 pi i j / L), L][chirp, M][transform of the
// convolution kernel conj(chirp(|k|)) over L, in the forward passes' order, L].
template <int LOG>
__global__ __launch_bounds__(Fft<LOG>::TG) void spectrum_plan_kernel(int M,
                                                                     double2 *__restrict__ table)
{
    using F = Fft<LOG>;
    __shared__ double2 buf[F::kWords];
    const int t = (int)threadIdx.x;
    double2 *root = table, *ch = table + F::L, *kern = ch + M;
    for (int j = t; j < F::L; j += F::TG) {
        double s, c;
        sincospi(2.0 * j / F::L, &s, &c);
        root[j] = make_double2(c, -s);
        buf[padded(j)] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    for (int n = t; n < M; n += F::TG) {
        double2 c = chirp(n, M);
        ch[n] = c;
        c.y = -c.y;
        buf[padded(n)] = c;
        if (n > 0)
            buf[padded(F::L - n)] = c;
    }
    __syncthreads();  // the roots, too, are read back by this workgroup
    F::forward(buf, root, t);
    double2 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        x[k] = buf[padded(8 * t + k)];
    dft8<true>(x);
#pragma unroll
    for (int k = 0; k < 8; ++k)
        kern[8 * t + k] = make_double2(x[k].x / F::L, x[k].y / F::L);
}

// One workgroup per tracer; G = 2: its two complex series (x + i y, z) at the
// same time, one per group of L / 8 threads; G = 1 (long series): one after the
// other.  Blocks of neighbouring tracers, which share cache lines of the
// track, run on one XCD (blocks go to the eight XCDs in turn).
template <int LOG, int G>
__global__ __launch_bounds__(Fft<LOG>::TG *G) void spectrum_fft_kernel(
    const double *__restrict__ track, int M, int32_t T, int remove_mean,
    const double2 *__restrict__ table, double *__restrict__ out)
{
    using F = Fft<LOG>;
    __shared__ double2 buf[G][F::kWords];
    const int per = (T + 7) / 8, b = (int)blockIdx.x;
    const int tr = (b % 8) * per + b / 8;
    if (tr >= T)
        return;
    const int g = G == 2 ? (int)threadIdx.x / F::TG : 0, t = (int)threadIdx.x % F::TG;
    const double2 *root = table, *ch = table + F::L, *kern = ch + M;
    const int64_t row = 6 * (int64_t)T;
    const int K = M / 2 + 1;
    double e[4] = {0.0, 0.0, 0.0, 0.0};  // powers of k = t + TG i (K <= L / 4 + 1)
#pragma unroll 1
    for (int series = g; series < 2; series += G) {
        const double *va = track + (3 + 2 * series) * (int64_t)T + tr;  // x or z
        double a[4], c[4];
        double sa = 0.0, sc = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = t + i * F::TG;
            a[i] = n < M ? va[n * row] : 0.0;
            c[i] = n < M && series == 0 ? va[n * row + T] : 0.0;
            sa += a[i];
            sc += c[i];
        }
        double ma = 0.0, mc = 0.0;
        if (remove_mean) {
            // a tree over the group's sums, in the words the series takes next
            buf[g][t] = make_double2(sa, sc);
            __syncthreads();
            for (int h = F::TG / 2; h > 0; h >>= 1) {
                if (t < h)
                    buf[g][t] = cadd(buf[g][t], buf[g][t + h]);
                __syncthreads();
            }
            ma = buf[g][0].x / (double)M;
            mc = buf[g][0].y / (double)M;
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int n = t + i * F::TG;
            double2 z = make_double2(0.0, 0.0);
            if (i < 4 && n < M)
                z = cmul(make_double2(a[i & 3] - ma, series == 0 ? c[i & 3] - mc : 0.0), ch[n]);
            buf[g][padded(n)] = z;
        }
        __syncthreads();
        F::forward(buf[g], root, t);
        // the stride-1 passes, the product between them
        double2 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            x[k] = buf[g][padded(8 * t + k)];
        dft8<true>(x);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            x[k] = cmul(x[k], kern[8 * t + k]);
        dft8<false>(x);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            buf[g][padded(8 * t + k)] = x[k];
        F::backward(buf[g], root, t);
        if constexpr (G == 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = t + i * F::TG;
                if (k < K) {
                    const double2 p = buf[0][padded(k)], q = buf[0][padded(k > 0 ? M - k : 0)];
                    e[i] += 0.5 * ((p.x * p.x + p.y * p.y) + (q.x * q.x + q.y * q.y));
                }
            }
            __syncthreads();  // the next series overwrites the buffer
        }
    }
    if constexpr (G == 2) {
        for (int k = (int)threadIdx.x; k < K; k += 2 * F::TG) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double2 u = buf[q][padded(k)], v = buf[q][padded(k > 0 ? M - k : 0)];
                s += 0.5 * ((u.x * u.x + u.y * u.y) + (v.x * v.x + v.y * v.y));
            }
            out[(int64_t)tr * K + k] = s / (double)M;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = t + i * F::TG;
            if (k < K)
                out[(int64_t)tr * K + k] = e[i] / (double)M;
        }
    }
}

constexpr int kDirectRows = 160;
constexpr int kMaxFftRows = 4096;

template <int LOG, int G>
hipError_t launch_fft(const double *track, int M, int32_t T, int remove_mean, double2 *table,
                      double *out, hipStream_t stream)
{
    hipLaunchKernelGGL(spectrum_plan_kernel<LOG>, dim3(1), dim3(Fft<LOG>::TG), 0, stream, M,
                       table);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((spectrum_fft_kernel<LOG, G>), dim3((unsigned)((T + 7) / 8 * 8)),
                       dim3(Fft<LOG>::TG * G), 0, stream, track, M, T, remove_mean, table, out);
    return hipGetLastError();
}

bool by_fft(int64_t M) { return M >= kDirectRows && M <= kMaxFftRows; }

int fft_log(int64_t M)
{
    int lg = 9;
    while (((int64_t)1 << lg) < 2 * M - 1)
        ++lg;
    return lg;
}

}  // namespace

size_t velocity_spectrum_scratch(int64_t M)
{
    const int64_t n = by_fft(M) ? 2 * ((int64_t)1 << fft_log(M)) + M : M;
    return (size_t)n * sizeof(double2);
}

hipError_t launch_velocity_spectrum(const double *track, int64_t M, int32_t T, int remove_mean,
                                    double *scratch, double *out, hipStream_t stream)
{
    double2 *W = reinterpret_cast<double2 *>(scratch);
    if (by_fft(M)) {
        const int m = (int)M;
        switch (fft_log(M)) {
        case 9: return launch_fft<9, 2>(track, m, T, remove_mean, W, out, stream);
        case 10: return launch_fft<10, 2>(track, m, T, remove_mean, W, out, stream);
        case 11: return launch_fft<11, 2>(track, m, T, remove_mean, W, out, stream);
        case 12: return launch_fft<12, 1>(track, m, T, remove_mean, W, out, stream);
        case 13: return launch_fft<13, 1>(track, m, T, remove_mean, W, out, stream);
        default: return hipErrorInvalidValue;
        }
    }
    hipLaunchKernelGGL(twiddle_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, stream,
                       W, M);
    const int64_t K = M / 2 + 1;
    const int64_t kb = (K + kSpecThreads - 1) / kSpecThreads;
    hipLaunchKernelGGL(spectrum_kernel, dim3((unsigned)(kb * T)), dim3(kSpecThreads), 0, stream,
                       track, M, T, remove_mean, W, K, kb, out);
    return hipGetLastError();
}

}  // namespace colatus
