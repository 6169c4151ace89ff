// Transpose-Jacobian pair sum of many cotangents on the FP64 matrix
// instruction (form 3 of the adjoint, FP64 pairs, the unit cotangents of
// colatus_ftle: matrix_adjoint in api.cpp says why only those).  With M(d) = r^-3 I -
// 3 r^-5 d d^T,
//   out_k = sum_j M(d)(m_k lam_j - m_j lam_k) = m_k P_k - D_k lam_k,
//   P_k = sum_j M(d_kj) lam_j,   D_k = sum_j m_j M(d_kj),
// P is a matrix product over (source, component) shared by all cotangents, and
// D, one symmetric 3 x 3 matrix per target, is summed once for all of them.
//
// v_mfma_f64_16x16x4_f64 takes, per lane, one element of a 16 x 4 left operand:
// lane l holds the pair (target l % 16, source l / 16), computes that pair's
// M once, and feeds its six entries as the left operands of nine products
// (alpha, beta) for every group of 16 cotangents, whose right operands are
// lam_beta of four sources, read from LDS.  Per 64 pairs and group: nine
// products of 64 cycles; the pairs' 35 FP64 operations (about 150 cycles) are
// shared by up to three groups (48 cotangents, 72 accumulator registers).  The
// ordered loop spends 13 vector operations per pair and cotangent where a
// product spends 9, at the same rate (the matrix and vector FP64 units are
// one), and reads more.  Bound by the matrix products.  Measured at 20^3: 48
// cotangents 1780 us with the ordered loop, 930 us so (703 us of it products).
//
// A block of four waves takes 64 targets (16 a wave) and a slice of sources,
// staged 16 at a time.  The pair j == k is left out by its index: its terms
// cancel exactly, but m_k eps^-3 lam_k - m_k eps^-3 lam_k summed apart would not.
#include "colatus_internal.h"

#include <math.h>

namespace colatus {
namespace {

typedef double double4v __attribute__((ext_vector_type(4)));

constexpr int kStage = 16;        // sources staged at a time
constexpr int kStride = 18;       // doubles per staged row of 16: no bank conflicts
constexpr int kAdjGroups = 3;     // groups of 16 cotangents per launch

template <int G, bool MASK>
__global__ __launch_bounds__(256) void adjoint_matrix_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const double *__restrict__ lam, int n_cot, int c0, const WorkItem *__restrict__ items,
    int n_items, double *__restrict__ part)
{
    // rows: x, y, z, m, then lam of (cotangent, component)
    constexpr int kRows = 4 + 48 * G;
    __shared__ double st[kRows][kStride];
    __shared__ double sd[4][16][6];
    const int it = (int)blockIdx.x;
    if (it >= n_items)
        return;
    const WorkItem w = items[it];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kq = lane >> 4;
    const int64_t i = w.i0 + wave * 16 + col;  // this lane's target in the pairs
    const int64_t ii = i < w.i1 ? i : w.i0;
    const double xi = x[ii], yi = x[N + ii], zi = x[2 * N + ii];
    const double eps2 = w.eps2;
    const int nc = n_cot - c0 < 16 * G ? n_cot - c0 : 16 * G;

    double4v acc[3][G];
    double d[6];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int g = 0; g < G; ++g)
            acc[a][g] = (double4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
        d[q] = 0.0;

    // the next stage's words are loaded while this one is worked on: thread t
    // takes source t % 16 of the rows t / 16, t / 16 + 16, ...
    constexpr int kPer = (kRows + 15) / 16;
    const int sj = tid & 15, sr = tid >> 4;
    double v[kPer];
    auto fetch = [&](int64_t j0) {
        const int64_t j = j0 + sj;
        const bool jv = j < w.j1;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int r = sr + 16 * q;
            double t = 0.0;  // missing sources: zero mass and cotangents
            if (r < 3)
                t = x[(int64_t)r * N + (jv ? j : w.i0)];
            else if (r == 3)
                t = jv ? m[j] : 0.0;
            else if (r < kRows && (r - 4) / 3 < nc)
                t = jv ? lam[((int64_t)c0 * 3 + (r - 4)) * N + j] : 0.0;
            v[q] = t;
        }
    };
    fetch(w.j0);
    for (int64_t j0 = w.j0; j0 < w.j1; j0 += kStage) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (sr + 16 * q < kRows)
                st[sr + 16 * q][sj] = v[q];
        __syncthreads();
        if (j0 + kStage < w.j1)
            fetch(j0 + kStage);
#pragma unroll 1
        for (int k = 0; k < kStage; k += 4) {
            const int js = k + kq;
            const double dx = st[0][js] - xi, dy = st[1][js] - yi, dz = st[2][js] - zi;
            const double mj = st[3][js];
            const double s = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
            double rinv = rsqrt_refine(s, __builtin_amdgcn_rsq(s));
            // the pair of a particle with itself; a missing source
            bool out = j0 + js == i || j0 + js >= w.j1;
            if constexpr (MASK)
                out = out || !(s > 0.0);
            rinv = out ? 0.0 : rinv;
            const double r2 = rinv * rinv, r3 = r2 * rinv, t = -3.0 * (r3 * r2);
            const double tx = t * dx, ty = t * dy, tz = t * dz;
            double M[6];  // xx, xy, xz, yy, yz, zz
            M[0] = fma(tx, dx, r3);
            M[1] = tx * dy;
            M[2] = tx * dz;
            M[3] = fma(ty, dy, r3);
            M[4] = ty * dz;
            M[5] = fma(tz, dz, r3);
#pragma unroll
            for (int q = 0; q < 6; ++q)
                d[q] = fma(mj, M[q], d[q]);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const double l = st[4 + (g * 16 + col) * 3 + b][js];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        constexpr int e[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
                        acc[a][g] =
                            __builtin_amdgcn_mfma_f64_16x16x4f64(M[e[a][b]], l, acc[a][g], 0, 0, 0);
                    }
                }
            }
        }
    }
    // D of a target: the four source groups of its lanes, in a fixed butterfly
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        d[q] += __shfl_xor(d[q], 16, 64);
        d[q] += __shfl_xor(d[q], 32, 64);
        if (kq == 0)
            sd[wave][col][q] = d[q];
    }
    __syncthreads();
    // element v of a lane: target kq + 4 v of the wave, cotangent col of the group
#pragma unroll
    for (int vv = 0; vv < 4; ++vv) {
        const int tl = kq + 4 * vv;
        const int64_t k = w.i0 + wave * 16 + tl;
        if (k >= w.i1)
            continue;
        const double mk = m[k];
        const double *D = sd[wave][tl];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int c = g * 16 + col;
            if (c >= nc)
                continue;
            const double *lk = lam + ((int64_t)(c0 + c) * 3) * N + k;
            const double lx = lk[0], ly = lk[N], lz = lk[2 * N];
            double *o = part + (((int64_t)w.slice * n_cot + (c0 + c)) * 3) * N + k;
            o[0] = fma(mk, acc[0][g][vv], -fma(D[0], lx, fma(D[1], ly, D[2] * lz)));
            o[N] = fma(mk, acc[1][g][vv], -fma(D[1], lx, fma(D[3], ly, D[4] * lz)));
            o[2 * N] = fma(mk, acc[2][g][vv], -fma(D[2], lx, fma(D[4], ly, D[5] * lz)));
        }
    }
}

template <int G>
hipError_t launch_g(bool mask, const double *x, const double *m, int64_t N, const double *lam,
                    int n_cot, int c0, const WorkItem *items, int n_items, double *part,
                    hipStream_t s)
{
    if (mask)
        hipLaunchKernelGGL((adjoint_matrix_kernel<G, true>), dim3((unsigned)n_items), dim3(256), 0,
                           s, x, m, N, lam, n_cot, c0, items, n_items, part);
    else
        hipLaunchKernelGGL((adjoint_matrix_kernel<G, false>), dim3((unsigned)n_items), dim3(256),
                           0, s, x, m, N, lam, n_cot, c0, items, n_items, part);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint_matrix(bool mask_self, const double *x, const double *m, int64_t N,
                                 int n_cot, const double *lam, const WorkItem *items, int n_items,
                                 double *part, hipStream_t stream)
{
    for (int c0 = 0; c0 < n_cot; c0 += 16 * kAdjGroups) {
        const int groups = (n_cot - c0 + 15) / 16;
        const hipError_t e =
            groups >= 3   ? launch_g<3>(mask_self, x, m, N, lam, n_cot, c0, items, n_items, part,
                                        stream)
            : groups == 2 ? launch_g<2>(mask_self, x, m, N, lam, n_cot, c0, items, n_items, part,
                                        stream)
                          : launch_g<1>(mask_self, x, m, N, lam, n_cot, c0, items, n_items, part,
                                        stream);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace colatus
