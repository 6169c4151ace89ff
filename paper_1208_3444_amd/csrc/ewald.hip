// Periodic boundaries (Section II solves the motion equations in a periodic
// box): the reciprocal-space part of the Ewald sum and its constants.  The
// real-space part is the pair sweep's (pair_sweep.hip, ewald_real_kernel).
//
// With the box side L and reciprocal vectors k = 2 pi n / L, n != 0,
// |n| <= n_max:
//   S(k)   = sum_j m_j exp(i k . x_j)                       (structure factor)
//   W(k)   = (4 pi / L^3) window(k) / k^2 S(k)
//   g^K    = sum_k k Im(exp(-i k . x_i) W(k))                (field, no G)
//   psi^K  = sum_k Re(exp(-i k . x_i) W(k))                  (potential part)
// window(k) = exp(-k^2 / 4 alpha^2) for FP32 pairs (Gaussian splitting), the
// prolate window's transform for FP64 pairs (ewald_window.h).
//
// Both sums factor over a column (n_x, n_y) of k-space and its n_z = +-q:
//   exp(i k . x) = A E_q,  A = exp(2 pi i (n_x x + n_y y) / L),  E_q = exp(2 pi i q z / L).
// Half of the columns suffices (k and -k give conjugate terms), and +q and -q
// share the four real products of A = A_r + i A_i with E_q = B_c + i B_s:
//   a = 2 w sum m A_r B_c,  b = 2 w sum m A_r B_s,
//   c = 2 w sum m A_i B_c,  d = 2 w sum m A_i B_s,     w the weight of both
// (for q = 0 the single vector's weight without the 2): a matrix product over
// the particles, [A_r A_i] x [B_c B_s], four multiply-adds per (particle, +-q)
// and no phase recurrence over q.  The field needs, per particle and column,
//   V  = sum_q (a B_c + b B_s) + i (c B_c + d B_s)
//   V' = sum_q q (c B_s - d B_c) + i q (b B_c - a B_s),
// again a matrix product ([B_c B_s] x table, eight per +-q), and then
//   g_x, g_y, psi from n_x, n_y, 1 times conj(A) V,  g_z from conj(A) V'.
// Both products run on the FP64 matrix instruction (v_mfma_f64_16x16x4_f64,
// 64 cycles measured).  It shares the pipeline with the vector FMA and has its
// rate; what it saves is operands: one LDS or cache word per lane feeds 16
// multiply-adds.  (The field with the table as scalar operands of vector FMAs,
// the fewest operations, waited on scalar loads: 124 us at 32^3, |n| <= 14.)
#include "colatus_internal.h"

#include <math.h>

namespace colatus {
namespace {

typedef double double4v __attribute__((ext_vector_type(4)));

// LDS words of one particle's axis phases, in pairs (cos, sin): padded so that
// the four particles of an operand fall on other banks (counted over the
// tiles' columns: 9.3 passes of the banks per operand at 24 pairs, 11.4 at 19,
// 15.7 at 17; the field kernel takes 19 to leave room for two blocks per CU).
constexpr int kSkPairs = 24, kKfPairs = 19;

// E_n = exp(2 pi i n x / L), n <= kEwMaxN, of one coordinate, scaled by f, into
// LDS words [n][cos, sin]: one sincospi, then E_n = E_{n/2} E_{n - n/2} (at most
// four products deep).
__device__ __forceinline__ void axis_phases(double x, double inv_L, double f, double (*out)[2])
{
    double c[kEwMaxN + 1], s[kEwMaxN + 1];
    c[0] = 1.0;
    s[0] = 0.0;
    sincospi(2.0 * x * inv_L, &s[1], &c[1]);
    // a non-finite coordinate marks every phase, the constant one included
    c[0] += 0.0 * s[1];
#pragma unroll
    for (int n = 2; n <= kEwMaxN; ++n) {
        const int h = n / 2, r = n - h;
        c[n] = c[h] * c[r] - s[h] * s[r];
        s[n] = s[h] * c[r] + c[h] * s[r];
    }
#pragma unroll
    for (int n = 0; n <= kEwMaxN; ++n) {
        out[n][0] = f * c[n];
        out[n][1] = f * s[n];
    }
}

// ---------------------------------------------------------------------------
// Structure factors: rows 16 = 8 columns x {A_r, A_i}, columns 16 = 8 q x
// {B_c, B_s}, four particles deep.  A block of eight waves stages the axis
// phases of 32 particles in LDS (the mass multiplies the x phases), and each
// wave keeps NP row tiles with both q tiles (q < 8 and q >= 8) and NS row tiles
// with the first alone in accumulators.  An operand element is half of one
// complex product.  Accumulators go out as they lie, one slot per chunk; sums
// over chunks are in chunk order.  Two waves per SIMD hide each other's LDS
// reads; with one (two blocks of four waves sharing a chunk's tiles, which
// halves the slots) the kernel took 54 us instead of 39 at 32^3.  Bound by the
// matrix products (17 us) and the LDS words of their left operands.  With the
// sums over the chunks, one lane per run of k with a phase recurrence took
// 59 us at 20^3 and 116 us at 32^3 (|n| <= 14); so 31 and 50 us.
// ---------------------------------------------------------------------------
constexpr int kSkTile = 32;

template <int NP, int NS>
__global__ __launch_bounds__(512) void ewald_sk_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N, int64_t chunk,
    const EwaldSkPlan *__restrict__ plan, int n_units, double inv_L, double *__restrict__ part)
{
    // [axis][particle][n][cos, sin]; q = 15, beyond every n_max, stays zero
    __shared__ double ph[3][kSkTile][kSkPairs][2];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int gw = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kp = lane >> 4, cc = row >> 1, half = row & 1;
    constexpr int kSlots = NP + NS;
    int tile[kSlots], nx[kSlots], ny[kSlots];
    double sg[kSlots];
    double4v acc0[kSlots], acc1[NP];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        tile[s] = __builtin_amdgcn_readfirstlane(
            (int)plan->slots[gw][s < NP ? s : kEwPairs + s - NP]);
        const int c = (tile[s] >= 0 ? tile[s] : 0) * 8 + cc;  // an idle slot repeats tile 0
        const int vx = plan->cols[c].x, vy = plan->cols[c].y;
        nx[s] = vx;
        ny[s] = vy < 0 ? -vy : vy;
        // A_r = X_c Y_c - X_s Y_s, A_i = X_s Y_c + X_c Y_s; Y_s odd in n_y
        sg[s] = (half ? 1.0 : -1.0) * (vy < 0 ? -1.0 : 1.0);
        acc0[s] = (double4v){0.0, 0.0, 0.0, 0.0};
        if (s < NP)
            acc1[s] = (double4v){0.0, 0.0, 0.0, 0.0};
    }
    if (tid < 3 * kSkTile)
        ph[tid / kSkTile][tid % kSkTile][kEwQ - 1][0] =
            ph[tid / kSkTile][tid % kSkTile][kEwQ - 1][1] = 0.0;
    const int64_t j0 = (int64_t)blockIdx.x * chunk;
    const int64_t j1 = j0 + chunk < N ? j0 + chunk : N;
    for (int64_t t0 = j0; t0 < j1; t0 += kSkTile) {
        __syncthreads();
        if (tid < 3 * kSkTile) {
            const int axis = tid / kSkTile, p = tid % kSkTile;
            const int64_t j = t0 + p;
            // a missing particle has zero phases along x (mass 0)
            const bool v = j < j1;
            axis_phases(v ? x[(int64_t)axis * N + j] : 0.0, inv_L,
                        axis == 0 ? (v ? m[j] : 0.0) : 1.0, ph[axis][p]);
        }
        __syncthreads();
        const int n4 = (int)((j1 - t0 < kSkTile ? j1 - t0 : kSkTile) + 3) & ~3;
#pragma unroll 1
        for (int k = 0; k < n4; k += 4) {
            const int p = k + kp;
            const double b0 = ph[2][p][cc][half], b1 = ph[2][p][cc + 8][half];
            double a[kSlots];
#pragma unroll
            for (int s = 0; s < kSlots; ++s)
                a[s] = fma(ph[0][p][nx[s]][half], ph[1][p][ny[s]][0],
                           sg[s] * (ph[0][p][nx[s]][1 - half] * ph[1][p][ny[s]][1]));
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                acc0[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b0, acc0[s], 0, 0, 0);
                if (s < NP)
                    acc1[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b1, acc1[s], 0, 0, 0);
            }
        }
    }
    // element v * 64 + lane of a unit: row (lane / 16) + 4 v, column lane % 16
    double *out = part + (int64_t)blockIdx.x * n_units * 256 + lane;
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        if (tile[s] < 0)
            continue;
        const int u = s < NP ? 2 * tile[s] : tile[s] + plan->n_pairs;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            out[(int64_t)u * 256 + v * 64] = acc0[s][v];
            if (s < NP)
                out[(int64_t)(u + 1) * 256 + v * 64] = acc1[s][v];
        }
    }
}

// The field's table: each element of a unit summed over the chunks (four
// thread groups take every fourth chunk each, added in group order), times its
// weights, to its two places, V's and V's derivative's (EwaldDest; -1: padding).
__global__ __launch_bounds__(1024) void ewald_sk_reduce_kernel(
    const double *__restrict__ part, int n_chunks, int n_units,
    const EwaldDest *__restrict__ dest, double *__restrict__ table)
{
    __shared__ double red[4][256];
    const int e = (int)(threadIdx.x & 255), g = (int)(threadIdx.x >> 8);
    const int64_t at = (int64_t)blockIdx.x * 256 + e;
    double t = 0.0;
#pragma unroll 8
    for (int c = g; c < n_chunks; c += 4)
        t += part[(int64_t)c * n_units * 256 + at];
    red[g][e] = t;
    __syncthreads();
    if (g == 0) {
        const EwaldDest d = dest[at];
        if (d.v >= 0) {
            t = ((t + red[1][e]) + red[2][e]) + red[3][e];
            table[d.v] = d.wv * t;
            table[d.z] = d.wz * t;
        }
    }
}

// The field and potential part: rows 16 particles, columns 16 = 4 columns of
// k-space x {V_r, V_i, V'_r, V'_i}, the products over (q, {B_c, B_s}) four at a
// time.  A wave holds the z phases of two row tiles (32 particles) in
// registers and walks the column tiles of its range (blockIdx.y); a table
// operand (64 consecutive doubles) serves both.  The lane of V_r, V_i, .. of a
// column multiplies its four particles' sums by its part of conj(A), formed
// from the axis phases in LDS, and adds them to its own field sums: lanes of V
// to (g_x, g_y, psi), lanes of V' to g_z; the 16 lanes of a particle are added
// at the end by a fixed butterfly.  Ranges are of equal work (host).
// PHI: also the potential part.  Operands and columns of the next tile are
// loaded ahead: without that the loads' latency tripled the time.  At 20^3 /
// 32^3 (|n| <= 14) 25 / 59 us, against 33 / 107 us with a sincospi and a phase
// recurrence per run of k; 24 us of products at 32^3, the rest the epilogue's
// LDS words and 200 cycles of vector work per tile.
constexpr int kKfParticles = 128;

template <bool PHI>
__global__ __launch_bounds__(256) void ewald_kforce_kernel(
    const double *__restrict__ x, int64_t N, const EwaldColTile *__restrict__ tiles,
    const int32_t *__restrict__ range, const double *__restrict__ table, double inv_L,
    double *__restrict__ out)
{
    __shared__ double ph[2][kKfParticles][kKfPairs][2];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * kKfParticles;
    {
        const int axis = tid / kKfParticles, p = tid % kKfParticles;
        const int64_t i = p0 + p;
        axis_phases(i < N ? x[(int64_t)axis * N + i] : 0.0, inv_L, 1.0, ph[axis][p]);
    }
    // z phases as the left operand: row particle, depth (q, cos / sin) = 4 ks + lane / 16
    constexpr int KS = kEwQ / 2;
    double za[2][KS];
    const int kq = lane >> 4, trig = kq & 1;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
        const int64_t i = p0 + wave * 32 + rt * 16 + (lane & 15);
        double s1, c1;
        sincospi(2.0 * (i < N ? x[2 * N + i] : 0.0) * inv_L, &s1, &c1);
        const double c2 = c1 * c1 - s1 * s1, s2 = 2.0 * s1 * c1;
        const double c4 = c2 * c2 - s2 * s2, s4 = 2.0 * s2 * c2;
        const double c8 = c4 * c4 - s4 * s4, s8 = 2.0 * s4 * c4;
        // E_{2 ks + kq / 2}; ks in binary
        double c = kq >= 2 ? c1 : 1.0 + 0.0 * s1, s = kq >= 2 ? s1 : 0.0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            double ec = c, es = s;
            if (ks & 1) {
                const double t = ec * c2 - es * s2;
                es = es * c2 + ec * s2;
                ec = t;
            }
            if (ks & 2) {
                const double t = ec * c4 - es * s4;
                es = es * c4 + ec * s4;
                ec = t;
            }
            if (ks & 4) {
                const double t = ec * c8 - es * s8;
                es = es * c8 + ec * s8;
                ec = t;
            }
            za[rt][ks] = trig ? es : ec;
        }
    }
    __syncthreads();
    const int cc = (lane & 15) >> 2, type = lane & 3;
    // the multiplier of this lane's sums: -A_i for V_r and V'_r, A_r for V_i and V'_i
    // (w = A_r V_i - A_i V_r); for psi the other part, A_r V_r + A_i V_i
    const int odd = type & 1;
    double f1[2][4], f2[2][4], fp[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            f1[rt][v] = f2[rt][v] = fp[rt][v] = 0.0;
    const int t0 = range[blockIdx.y], t1 = range[blockIdx.y + 1];
    // the next tile's operands and columns are loaded while this tile is worked on
    double b[KS];
    int nxn = 0, nyn = 0, ksn = 0;
    auto fetch = [&](int t) {
        const EwaldColTile &ct = tiles[t];
        const double *w = table + (int64_t)t * (KS * 64) + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            b[ks] = w[ks * 64];
        nxn = ct.nx[cc];
        nyn = ct.ny[cc];
        ksn = ct.ks;
    };
    if (t0 < t1)
        fetch(t0);
    for (int t = t0; t < t1; ++t) {
        double bb[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            bb[ks] = b[ks];
        const int nx = nxn, vy = nyn, n_ks = ksn;
        fetch(t + 1 < t1 ? t + 1 : t);
        double4v d0 = (double4v){0.0, 0.0, 0.0, 0.0}, d1 = d0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks >= n_ks)
                break;
            d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(za[0][ks], bb[ks], d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(za[1][ks], bb[ks], d1, 0, 0, 0);
        }
        const int ny = vy < 0 ? -vy : vy;
        const double sy = vy < 0 ? -1.0 : 1.0;
        // c = A_r (odd types) or A_i (even, whose sign goes to k1, k2)
        const double sg = odd ? -sy : sy, s1 = odd ? 1.0 : -1.0;
        const double k1 = s1 * (type < 2 ? (double)nx : 1.0), k2 = type < 2 ? s1 * vy : 0.0;
        const double kp = type < 2 ? 1.0 : 0.0;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int p = wave * 32 + rt * 16 + (lane >> 4) + 4 * v;
                const double xa = ph[0][p][nx][1 - odd], xb = ph[0][p][nx][odd];
                const double yc = ph[1][p][ny][0], ys = ph[1][p][ny][1];
                const double d = rt == 0 ? d0[v] : d1[v];
                const double u = fma(xa, yc, sg * (xb * ys)) * d;
                f1[rt][v] = fma(k1, u, f1[rt][v]);
                f2[rt][v] = fma(k2, u, f2[rt][v]);
                if constexpr (PHI)
                    fp[rt][v] = fma(kp * fma(xb, yc, -sg * (xa * ys)), d, fp[rt][v]);
            }
    }
    // lanes 16 q .. 16 q + 15 share a particle: types 0, 1 hold g_x (f1), g_y (f2)
    // and psi, types 2, 3 g_z (f1); column cc in bits 2-3
    const double two_pi_L = 2.0 * 3.14159265358979323846 * inv_L;
    double *o = out + (int64_t)blockIdx.y * 4 * N;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double g1 = f1[rt][v], g2 = f2[rt][v], gp = fp[rt][v];
#pragma unroll
            for (int off = 1; off < 16; off = off == 1 ? 4 : off * 2) {
                g1 += __shfl_xor(g1, off, 64);
                g2 += __shfl_xor(g2, off, 64);
                if constexpr (PHI)
                    gp += __shfl_xor(gp, off, 64);
            }
            const int64_t i = p0 + wave * 32 + rt * 16 + (lane >> 4) + 4 * v;
            if (i < N && (lane & 15) == 0) {
                o[i] = two_pi_L * g1;
                o[N + i] = two_pi_L * g2;
                if constexpr (PHI)
                    o[3 * N + i] = gp;
            }
            if (i < N && (lane & 15) == 2)
                o[2 * N + i] = two_pi_L * g1;
        }
}

// gk[c][i] = sum over ranges (in order) of the partial fields; with pk also
// pk[i] likewise plus m_i self_c + bg_c M: self_c takes the particle's own
// smooth part away, bg_c is the removed background.  blockIdx.y: the component.
__global__ __launch_bounds__(256) void ewald_kreduce_kernel(
    const double *__restrict__ part, int n_ranges, int64_t N, const double *__restrict__ m,
    double self_c, const double *__restrict__ msum, double bg_c, double *__restrict__ gk,
    double *__restrict__ pk)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int comp = (int)blockIdx.y;
    if (i >= N)
        return;
    double t = 0.0;
#pragma unroll 8
    for (int r = 0; r < n_ranges; ++r)
        t += part[((int64_t)r * 4 + comp) * N + i];
    if (comp < 3)
        gk[comp * N + i] = t;
    else
        pk[i] = t + m[i] * self_c + bg_c * msum[0];
}

// Total mass, one block, fixed order (for the background constant).
__global__ __launch_bounds__(1024) void ewald_mass_kernel(const double *__restrict__ m, int64_t N,
                                                          double *__restrict__ out)
{
    __shared__ double sh[1024];
    double t = 0.0;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < N; i += 1024)
        t += m[i];
    sh[threadIdx.x] = t;
    __syncthreads();
    for (int off = 512; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        out[0] = sh[0];
}

}  // namespace

hipError_t launch_ewald_kspace(const EwaldArgs &A, hipStream_t stream)
{
    const double inv_L = 1.0 / A.L;
    const int64_t N = A.N;
    if (A.n_units < 1 || A.n_sk_chunks < 1 || A.n_ranges < 1 ||
        (int64_t)A.n_sk_chunks * A.sk_chunk < N)
        return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    if (A.pk && !A.mass_ready) {
        hipLaunchKernelGGL(ewald_mass_kernel, dim3(1), dim3(1024), 0, stream, A.m, N, A.msum);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    const dim3 sk_grid((unsigned)A.n_sk_chunks);
    if (A.sk_slots_p <= 3)
        hipLaunchKernelGGL((ewald_sk_kernel<3, kEwSingles>), sk_grid, dim3(512), 0, stream, A.x, A.m, N,
                           A.sk_chunk, A.sk_plan, A.n_units, inv_L, A.sk_part);
    else
        hipLaunchKernelGGL((ewald_sk_kernel<kEwPairs, kEwSingles>), sk_grid, dim3(512), 0, stream, A.x,
                           A.m, N, A.sk_chunk, A.sk_plan, A.n_units, inv_L, A.sk_part);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    hipLaunchKernelGGL(ewald_sk_reduce_kernel, dim3((unsigned)A.n_units), dim3(1024), 0, stream,
                       A.sk_part, A.n_sk_chunks, A.n_units, A.dest, A.table);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    const dim3 kf_grid((unsigned)((N + kKfParticles - 1) / kKfParticles), (unsigned)A.n_ranges);
    if (A.pk)
        hipLaunchKernelGGL(ewald_kforce_kernel<true>, kf_grid, dim3(256), 0, stream, A.x, N, A.tiles,
                           A.range, A.table, inv_L, A.kpart);
    else
        hipLaunchKernelGGL(ewald_kforce_kernel<false>, kf_grid, dim3(256), 0, stream, A.x, N, A.tiles,
                           A.range, A.table, inv_L, A.kpart);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    hipLaunchKernelGGL(ewald_kreduce_kernel, dim3((unsigned)((N + 255) / 256), A.pk ? 4 : 3),
                       dim3(256), 0, stream, A.kpart, A.n_ranges, N, A.m, A.self_c, A.msum, A.bg_c,
                       A.gk, A.pk);
    return hipGetLastError();
}

}  // namespace colatus
