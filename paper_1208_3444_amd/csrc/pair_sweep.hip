// Pair sweeps of the direct-summation (particle-particle) scheme: the O(N^2)
// hot loop of the method (Section II: the force computation dominates the
// cost; Appendix A: one GPU thread per target particle looping over every
// source).  Gfx950 design, not a translation of the paper's kernel.
//
// Symmetric loops (form 2, the default up to 2^18 particles per box): the
// pair terms of the forward sum and of its adjoint change sign when the two
// particles swap, so each unordered pair is evaluated once.  A box is cut
// into parts of 256; a work item (one wave) holds part p's targets in
// registers, four per lane, while part q's sources pass around the wave one
// lane per step (DPP rotation) carrying their reaction accumulators.  Each
// partial-sum slot (part p's pull on a particle) is written once; an O(N)
// kernel adds the slots in a fixed order, so results are deterministic.  The
// forward loop runs 2x2 blocks of part pairs in workgroups of four waves
// that add the partial sums of a shared part in LDS before writing, halving
// the slots.
//
// Ordered loops (forms 0 and 1; larger boxes, many-cotangent adjoints):
//   * a work item is (block of target particles) x (slice of sources); the
//     slices of one target block write separate partial sums;
//   * each lane keeps R targets in registers; sources are staged tile by tile
//     into LDS (one source per thread) and read back as wave-uniform
//     broadcasts, so one LDS read feeds R pair interactions;
//   * per-tile FP32 partial sums are folded into FP64 or an unevaluated FP32
//     (hi, lo) pair with TwoSum (Knuth), bounding the accumulation error.
//
// Both: FP32 pairs use coordinates relative to the centre of the target
// block's (part's) bounding box (FP64 subtract, then round to FP32), so the
// FP32 pair arithmetic keeps the relative accuracy of the separation itself;
// rsqrt is the hardware v_rsq_f32 in FP32 and v_rsq_f64 refined by one Newton
// step in FP64; no MFMA: the pair interaction is not a dense contraction.
//
// The persistent variant launches about one grid of resident workgroups and
// pulls work items from a device counter until none are left (every
// workgroup's last fetch sees the counter past the end and exits).
#include "colatus_internal.h"
#include "device_math.h"
#include "ewald_window.h"

#include <math.h>
#include <type_traits>

namespace colatus {
namespace {

enum AccMode { kDirect = 0, kTwoSum = 1, kFold64 = 2 };

template <typename T> struct V4;
template <> struct V4<float> { using type = float4; };
template <> struct V4<double> { using type = double4; };

// Centre of the bounding box of the block's valid targets, for every thread.
template <int TPB, int R>
__device__ __forceinline__ void block_centre(const double (&tx)[R], const double (&ty)[R],
                                             const double (&tz)[R], const bool (&valid)[R],
                                             double (*red)[6], double &cx, double &cy,
                                             double &cz)
{
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (valid[r]) {
            v[0] = fmin(v[0], tx[r]);
            v[1] = fmin(v[1], ty[r]);
            v[2] = fmin(v[2], tz[r]);
            v[3] = fmax(v[3], tx[r]);
            v[4] = fmax(v[4], ty[r]);
            v[5] = fmax(v[5], tz[r]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            v[q] = fmin(v[q], __shfl_xor(v[q], off, 64));
            v[q + 3] = fmax(v[q + 3], __shfl_xor(v[q + 3], off, 64));
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            red[wave][q] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 6; ++q)
        v[q] = red[0][q];
#pragma unroll
    for (int w = 1; w < TPB / 64; ++w) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            v[q] = fmin(v[q], red[w][q]);
            v[q + 3] = fmax(v[q + 3], red[w][q + 3]);
        }
    }
    cx = 0.5 * (v[0] + v[3]);
    cy = 0.5 * (v[1] + v[4]);
    cz = 0.5 * (v[2] + v[5]);
}

// Fetch the next work item index (persistent) or this block's (one-shot).
__device__ __forceinline__ int next_item(int persistent, int *counter, int *s_item, int iter)
{
    if (!persistent)
        return iter == 0 ? (int)blockIdx.x : 0x7fffffff;
    if (threadIdx.x == 0)
        *s_item = atomicAdd(counter, 1);
    __syncthreads();
    int it = *s_item;
    __syncthreads();
    return it;
}

// ---------------------------------------------------------------------------
// Forward sweep: sum_j m_j (x_j - x_k) r^-3 (and sum_j m_j r^-1 with PHI).
//
// Per pair: 3 subtractions, 3 FMAs for s = |d|^2 + eps^2, one v_rsq, then
// the weight w = m_j r^-3 and 3 FMAs into the accumulators.  The weight is
// formed either as m r^-1 (r^-1 r^-1) (FORM 0) or as (m r^-1) rcp(s)
// (FORM 1, one VALU multiply fewer, one more transcendental, which gfx950
// issues beside the VALU stream).  When every mass of the box is equal
// (EQM), m_j leaves the loop and multiplies the slice's partial sum once.
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T pad_coord();
template <> __device__ __forceinline__ float pad_coord<float>() { return 1e30f; }
template <> __device__ __forceinline__ double pad_coord<double>() { return 1e150; }

template <typename T> __device__ __forceinline__ T rcp_t(T s);
template <> __device__ __forceinline__ float rcp_t<float>(float s) { return __builtin_amdgcn_rcpf(s); }
template <> __device__ __forceinline__ double rcp_t<double>(double s) { return 1.0 / s; }

// Four sources at a time against the lane's R targets, FP32 in the phases of
// sym_chunk (the estimates of all 4 R pairs in one burst); each sum adds its
// sources in order.  One FP32 evaluation of 300 000 particles 24.1 -> 22.6 ms;
// FP64, never paired, measured 1 % slower so and keeps the compiler's order.
template <typename T, int R, bool PHI, bool MASK, bool EQM, int FORM, typename V>
__device__ __forceinline__ void sweep_tile(const V *__restrict__ tile, int nt4, const T (&xi)[R],
                                           const T (&yi)[R], const T (&zi)[R], T eps2,
                                           T (&ax)[R], T (&ay)[R], T (&az)[R], T (&ph)[R])
{
    for (int jj = 0; jj < nt4; jj += 4) {
        T dx[4][R], dy[4][R], dz[4][R], s[4][R], y[4][R], q[4][R], mj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const V pj = tile[jj + u];
            mj[u] = pj.w;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dx[u][r] = pj.x - xi[r];
                dy[u][r] = pj.y - yi[r];
                dz[u][r] = pj.z - zi[r];
                s[u][r] = fma_t(dx[u][r], dx[u][r], eps2);
                s[u][r] = fma_t(dy[u][r], dy[u][r], s[u][r]);
                s[u][r] = fma_t(dz[u][r], dz[u][r], s[u][r]);
            }
        }
        if constexpr (sizeof(T) == 4)
            burst_begin();
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                y[u][r] = rsq_raw(s[u][r]);
                if constexpr (FORM == 1)
                    q[u][r] = rcp_t<T>(s[u][r]);
            }
        if constexpr (sizeof(T) == 4)
            burst_end();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T rinv = rsqrt_from(s[u][r], y[u][r]);
                T mr = EQM ? rinv : mj[u] * rinv;
                T w3;
                if constexpr (FORM == 1)
                    w3 = mr * q[u][r];
                else
                    w3 = mr * (rinv * rinv);
                if constexpr (MASK) {
                    w3 = s[u][r] > (T)0 ? w3 : (T)0;
                    mr = s[u][r] > (T)0 ? mr : (T)0;
                }
                ax[r] = fma_t(w3, dx[u][r], ax[r]);
                ay[r] = fma_t(w3, dy[u][r], ay[r]);
                az[r] = fma_t(w3, dz[u][r], az[r]);
                if constexpr (PHI)
                    ph[r] += mr;
            }
        }
    }
}

template <typename T, int ACC, int R, int TPB, bool PHI, bool MASK, int FORM>
__global__ __launch_bounds__(TPB) void pair_sweep_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const WorkItem *__restrict__ items, int n_items, int *__restrict__ counter,
    int persistent, const double *__restrict__ box_mass, double *__restrict__ part,
    double *__restrict__ part_phi, int64_t *__restrict__ step_inc)
{
    using V = typename V4<T>::type;
    __shared__ V tile[TPB];
    __shared__ double red[TPB / 64][6];
    __shared__ int s_item;
    const int tid = threadIdx.x;
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    if (step_inc && blockIdx.x == 0 && tid == 0)
        *step_inc += 1;

    for (int iter = 0;; ++iter) {
        const int it = next_item(persistent, counter, &s_item, iter);
        if (it >= n_items)
            break;
        const WorkItem w = items[it];
        // common mass of the box, or NaN when the masses differ
        const double mbox = box_mass ? box_mass[w.box] : NAN;
        const bool eqm = !isnan(mbox);

        double tx[R], ty[R], tz[R];
        bool valid[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = w.i0 + tid + (int64_t)r * TPB;
            valid[r] = i < w.i1;
            const int64_t ii = valid[r] ? i : w.i0;
            tx[r] = X[ii];
            ty[r] = Y[ii];
            tz[r] = Z[ii];
        }
        double cx, cy, cz;
        block_centre<TPB, R>(tx, ty, tz, valid, red, cx, cy, cz);

        T xi[R], yi[R], zi[R];
        T ax[R], ay[R], az[R], ph[R];
        T hx[R], hy[R], hz[R], hp[R];      // TwoSum hi
        T lx[R], ly[R], lz[R], lp[R];      // TwoSum lo
        double bx[R], by[R], bz[R], bp[R]; // FP64 fold
#pragma unroll
        for (int r = 0; r < R; ++r) {
            xi[r] = (T)(tx[r] - cx);
            yi[r] = (T)(ty[r] - cy);
            zi[r] = (T)(tz[r] - cz);
            ax[r] = ay[r] = az[r] = ph[r] = (T)0;
            hx[r] = hy[r] = hz[r] = hp[r] = (T)0;
            lx[r] = ly[r] = lz[r] = lp[r] = (T)0;
            bx[r] = by[r] = bz[r] = bp[r] = 0.0;
        }
        const T eps2 = (T)w.eps2;

        for (int64_t jt = w.j0; jt < w.j1; jt += TPB) {
            const int64_t j = jt + tid;
            V v;
            if (j < w.j1) {
                v.x = (T)(X[j] - cx);
                v.y = (T)(Y[j] - cy);
                v.z = (T)(Z[j] - cz);
                v.w = (T)m[j];
            } else {
                // padding: so far away that the pair adds nothing (FP32: s
                // overflows to +inf and r^-1 = 0; FP64: r^-3 underflows to 0)
                v.x = v.y = v.z = pad_coord<T>();
                v.w = (T)0;
            }
            __syncthreads();
            tile[tid] = v;
            __syncthreads();
            const int nt = (int)((w.j1 - jt) < TPB ? (w.j1 - jt) : TPB);
            const int nt4 = (nt + 3) & ~3;
            if (eqm)
                sweep_tile<T, R, PHI, MASK, true, FORM>(tile, nt4, xi, yi, zi, eps2, ax, ay, az,
                                                        ph);
            else
                sweep_tile<T, R, PHI, MASK, false, FORM>(tile, nt4, xi, yi, zi, eps2, ax, ay, az,
                                                         ph);
            if constexpr (ACC == kTwoSum) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    two_sum_add(hx[r], lx[r], (float)ax[r]);
                    two_sum_add(hy[r], ly[r], (float)ay[r]);
                    two_sum_add(hz[r], lz[r], (float)az[r]);
                    if constexpr (PHI)
                        two_sum_add(hp[r], lp[r], (float)ph[r]);
                    ax[r] = ay[r] = az[r] = ph[r] = (T)0;
                }
            } else if constexpr (ACC == kFold64) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    bx[r] += (double)ax[r];
                    by[r] += (double)ay[r];
                    bz[r] += (double)az[r];
                    if constexpr (PHI)
                        bp[r] += (double)ph[r];
                    ax[r] = ay[r] = az[r] = ph[r] = (T)0;
                }
            }
        }

        const int64_t slot = (int64_t)w.slice;
        const double scale = eqm ? mbox : 1.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!valid[r])
                continue;
            const int64_t i = w.i0 + tid + (int64_t)r * TPB;
            double ox, oy, oz, op;
            if constexpr (ACC == kTwoSum) {
                ox = (double)hx[r] + (double)lx[r];
                oy = (double)hy[r] + (double)ly[r];
                oz = (double)hz[r] + (double)lz[r];
                op = (double)hp[r] + (double)lp[r];
            } else if constexpr (ACC == kFold64) {
                ox = bx[r];
                oy = by[r];
                oz = bz[r];
                op = bp[r];
            } else {
                ox = (double)ax[r];
                oy = (double)ay[r];
                oz = (double)az[r];
                op = (double)ph[r];
            }
            part[(slot * 3 + 0) * N + i] = scale * ox;
            part[(slot * 3 + 1) * N + i] = scale * oy;
            part[(slot * 3 + 2) * N + i] = scale * oz;
            if constexpr (PHI)
                part_phi[slot * N + i] = scale * op;
        }
    }
}

// ---------------------------------------------------------------------------
// Symmetric forward sweep (form 2, FP32 pairs).  The pair term of Eq. (1) is
// antisymmetric: the pull of j on k, m_j d r^-3 with d = x_j - x_k, and the
// pull of k on j, -m_k d r^-3, share d, s = |d|^2 + eps^2 and r^-3.  Each
// unordered pair is therefore evaluated once and applied to both particles.
//
// A work item is a pair of parts (p, q), p < q, of one partition of a box.
// The W waves of the workgroup hold part p's U = 64 R W targets in registers
// (R per lane).  Part q's sources pass through in chunks of 64, one per lane;
// after every step each source moves one lane on (a DPP rotation of the whole
// wave) and carries the accumulator of its reaction with it, so after 64
// steps every source has met every target of the wave and is back in its
// lane with its reaction complete.  The waves' reactions are added in a fixed
// order.  Part p's partial sum from part q goes to the item's target slot
// and part q's reaction from part p to its reaction slot (with one item per
// workgroup slots q and p; the grouped form below numbers them by
// super-part): each (slot, particle) is written once, and the O(N) kernels
// add the slots in a fixed order.  The diagonal item (p, p) evaluates the
// ordered pairs of its part with the same loop and no reaction.
//
// Per unordered pair with equal masses: 3 subtractions, 3 FMAs, one v_rsq,
// 2 multiplies, 3 + 3 FMAs; per step and lane 6 rotations shared by R pairs.
// ---------------------------------------------------------------------------
// A value known to be equal in every lane, moved to a scalar register.
__device__ __forceinline__ float uniform(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lane l receives the value lane (l - 1) mod 64 held (DPP wave_ror:1); every
// lane of the wave must be active.
__device__ __forceinline__ float wave_rotate(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x13C, 0xF, 0xF, true));
}
__device__ __forceinline__ double wave_rotate(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x13C, 0xF, 0xF, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x13C, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lane l receives the value lane (l + 1) mod 64 held (DPP wave_rol:1).
__device__ __forceinline__ float wave_rotate_back(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x134, 0xF, 0xF, true));
}
__device__ __forceinline__ double wave_rotate_back(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x134, 0xF, 0xF, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x134, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Far-away coordinate of a missing target or source of the symmetric loops.
// Forward: s overflows (FP32) or r^-3 underflows (FP64) and the pair adds 0.
// Adjoint: s must stay finite so that d.u does (r^-3 underflows to 0).
template <typename T> __device__ __forceinline__ T sym_pad();
template <> __device__ __forceinline__ float sym_pad<float>() { return 1e30f; }
template <> __device__ __forceinline__ double sym_pad<double>() { return 1e150; }
template <typename T> __device__ __forceinline__ T adj_pad();
template <> __device__ __forceinline__ float adj_pad<float>() { return 1e18f; }
template <> __device__ __forceinline__ double adj_pad<double>() { return 1e150; }

// 64 steps of one source chunk against the lane's R targets.  REACT: also
// accumulate the reaction on the travelling source (q*); EQM: the box's common
// mass leaves the loop (weights r^-3 and r^-1 only).
//
// A step is three phases: the R separations, a burst of the R reciprocal
// square roots with the rotations of everything that travels, and the
// weights with the accumulations (see burst_begin for why).  The positions
// rotate for the next step; the masses and reactions rotate just before this
// step uses them (the masses start one lane back, the reactions, zero at
// first, take one more rotation at the end), so that all rotations share the
// one burst.  A piece of a diagonal (R = 1, no reaction) takes U = 4 steps at
// a time for the same batch of four.  Measured (FP32, equal masses, one 64^3
// evaluation / 20 steps at 32^3): 13.0 / 4.66 ms with the compiler's own order,
// 10.3 / 3.63 ms so.  PHASED = false leaves the order to the compiler, for sweeps
// with too few waves to pair (sym_phased); both give the same bits.
template <typename T, int R, bool REACT, bool EQM, bool PHI, bool MASK, bool PHASED>
__device__ __forceinline__ void sym_chunk(T sx, T sy, T sz, T sm, T &qx, T &qy, T &qz, T &qp,
                                          const T (&xi)[R], const T (&yi)[R], const T (&zi)[R],
                                          const T (&mi)[R], T eps2, T (&ax)[R], T (&ay)[R],
                                          T (&az)[R], T (&ap)[R])
{
    if constexpr (!PHASED) {
#pragma unroll 2
        for (int k = 0; k < 64; ++k) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T dx = sx - xi[r];
                const T dy = sy - yi[r];
                const T dz = sz - zi[r];
                T s = fma_t(dx, dx, eps2);
                s = fma_t(dy, dy, s);
                s = fma_t(dz, dz, s);
                T rinv, w;
                if constexpr (sizeof(T) == 8 && !PHI) {
                    w = rinv3_from(s, rsq_raw(s));
                    if constexpr (MASK)
                        w = s > (T)0.0 ? w : (T)0.0;
                } else {
                    rinv = rsqrt_from(s, rsq_raw(s));
                    if constexpr (MASK)
                        rinv = s > (T)0.0 ? rinv : (T)0.0;
                    w = rinv * (rinv * rinv);
                }
                const T wt = EQM ? w : sm * w;
                ax[r] = fma_t(wt, dx, ax[r]);
                ay[r] = fma_t(wt, dy, ay[r]);
                az[r] = fma_t(wt, dz, az[r]);
                if constexpr (PHI)
                    ap[r] += EQM ? rinv : sm * rinv;
                if constexpr (REACT) {
                    const T ws = EQM ? w : mi[r] * w;
                    qx = fma_t(-ws, dx, qx);
                    qy = fma_t(-ws, dy, qy);
                    qz = fma_t(-ws, dz, qz);
                    if constexpr (PHI)
                        qp += EQM ? rinv : mi[r] * rinv;
                }
            }
            sx = wave_rotate(sx);
            sy = wave_rotate(sy);
            sz = wave_rotate(sz);
            if constexpr (!EQM)
                sm = wave_rotate(sm);
            if constexpr (REACT) {
                qx = wave_rotate(qx);
                qy = wave_rotate(qy);
                qz = wave_rotate(qz);
                if constexpr (PHI)
                    qp = wave_rotate(qp);
            }
        }
        return;
    }
    constexpr int U = R == 1 && !REACT ? 4 : 1;
    constexpr int B = U * R;
    static_assert(U == 1 || !REACT, "a reaction rotates every step");
    if constexpr (!EQM)
        sm = wave_rotate_back(sm);
#pragma unroll 1
    for (int k = 0; k < 64; k += U) {
        T dx[B], dy[B], dz[B], s[B], y[B], su[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int b = u * R + r;
                dx[b] = sx - xi[r];
                dy[b] = sy - yi[r];
                dz[b] = sz - zi[r];
                s[b] = fma_t(dx[b], dx[b], eps2);
                s[b] = fma_t(dy[b], dy[b], s[b]);
                s[b] = fma_t(dz[b], dz[b], s[b]);
            }
            if (u + 1 < U) {
                sx = wave_rotate(sx);
                sy = wave_rotate(sy);
                sz = wave_rotate(sz);
            }
        }
        burst_begin();
#pragma unroll
        for (int b = 0; b < B; ++b)
            y[b] = rsq_raw(s[b]);
        phase_mark();
        sx = wave_rotate(sx);
        sy = wave_rotate(sy);
        sz = wave_rotate(sz);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (!EQM)
                sm = wave_rotate(sm);
            su[u] = sm;
        }
        if constexpr (REACT) {
            qx = wave_rotate(qx);
            qy = wave_rotate(qy);
            qz = wave_rotate(qz);
            if constexpr (PHI)
                qp = wave_rotate(qp);
        }
        burst_end();
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int b = u * R + r;
                T rinv, w;
                if constexpr (sizeof(T) == 8 && !PHI) {
                    w = rinv3_from(s[b], y[b]);
                    if constexpr (MASK)
                        w = s[b] > (T)0.0 ? w : (T)0.0;
                } else {
                    rinv = rsqrt_from(s[b], y[b]);
                    if constexpr (MASK)
                        rinv = s[b] > (T)0.0 ? rinv : (T)0.0;
                    w = rinv * (rinv * rinv);
                }
                const T wt = EQM ? w : su[u] * w;
                ax[r] = fma_t(wt, dx[b], ax[r]);
                ay[r] = fma_t(wt, dy[b], ay[r]);
                az[r] = fma_t(wt, dz[b], az[r]);
                if constexpr (PHI)
                    ap[r] += EQM ? rinv : su[u] * rinv;
                if constexpr (REACT) {
                    // -(pull) accumulates with the opposite sign until the end:
                    // the same roundings, and no negated operand
                    const T ws = EQM ? w : mi[r] * w;
                    qx = fma_t(ws, dx[b], qx);
                    qy = fma_t(ws, dy[b], qy);
                    qz = fma_t(ws, dz[b], qz);
                    if constexpr (PHI)
                        qp += EQM ? rinv : mi[r] * rinv;
                }
            }
        }
        phase_mark();
    }
    if constexpr (REACT) {
        qx = -wave_rotate(qx);
        qy = -wave_rotate(qy);
        qz = -wave_rotate(qz);
        if constexpr (PHI)
            qp = wave_rotate(qp);
    }
}

// One work item of the symmetric sweep.  REACT: a pair of parts (p < q),
// R targets per lane, with the reaction on the sources; otherwise a piece of
// a diagonal item: one target per lane against the whole part, no reaction
// (every unordered pair inside the part is met twice, once from each side).
// FOLD: the sources of a part exceed 256 and the targets' FP32 partial sums
// are folded every 256 sources; with at most 256 every partial sum (a
// target's from one part, a source's reaction from one part) is a single
// FP32 sum of at most 256 terms, like the ordered loop's per-tile partials.
template <typename T, int ACC, int R, int W, bool FOLD, bool REACT, bool PHI, bool MASK,
          bool PHASED>
__device__ __forceinline__ void sym_item(const WorkItem &w, const double *__restrict__ X,
                                         const double *__restrict__ Y,
                                         const double *__restrict__ Z,
                                         const double *__restrict__ m, int64_t N,
                                         const double *__restrict__ box_mass,
                                         double *__restrict__ part,
                                         double *__restrict__ part_phi, double (*red)[6],
                                         T (*react)[W][PHI ? 4 : 3][64])
{
    constexpr int TPB = 64 * W;
    constexpr int NQ = PHI ? 4 : 3;
    // FP32 pairs without folding: every slot is one FP32 sum, stored as FP32
    // without the box mass (the readers apply it in FP64)
    constexpr bool F32OUT = sizeof(T) == 4 && !FOLD;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double mbox = box_mass ? box_mass[w.box] : NAN;
    const bool eqm = !isnan(mbox);

    double tx[R], ty[R], tz[R];
    bool valid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(wave * 64 * R + r * 64 + lane);
        valid[r] = i < w.i1;
        const int64_t ii = valid[r] ? i : w.i0;
        tx[r] = X[ii];
        ty[r] = Y[ii];
        tz[r] = Z[ii];
    }
    double cx, cy, cz;
    block_centre<TPB, R>(tx, ty, tz, valid, red, cx, cy, cz);
    cx = uniform(cx);
    cy = uniform(cy);
    cz = uniform(cz);

    // Missing targets sit far away with zero mass: they neither pull nor are
    // pulled (FP32 s overflows to +inf, r^-1 = 0).
    T xi[R], yi[R], zi[R], mi[R];
    T ax[R], ay[R], az[R], ap[R];
    float hx[R], hy[R], hz[R], hp[R];  // TwoSum (FP32 pairs only)
    float lx[R], ly[R], lz[R], lp[R];
    double bx[R], by[R], bz[R], bp[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(wave * 64 * R + r * 64 + lane);
        if (valid[r]) {
            xi[r] = (T)(tx[r] - cx);
            yi[r] = (T)(ty[r] - cy);
            zi[r] = (T)(tz[r] - cz);
            mi[r] = (T)m[i];
        } else {
            xi[r] = yi[r] = zi[r] = sym_pad<T>();
            mi[r] = (T)0.0;
        }
        ax[r] = ay[r] = az[r] = ap[r] = (T)0.0;
        if constexpr (FOLD) {
            hx[r] = hy[r] = hz[r] = hp[r] = (T)0.0;
            lx[r] = ly[r] = lz[r] = lp[r] = (T)0.0;
            bx[r] = by[r] = bz[r] = bp[r] = 0.0;
        }
    }
    const T eps2 = uniform((T)w.eps2);
    const double scale = eqm ? mbox : 1.0;
    const int n_chunks = (int)((w.j1 - w.j0 + 63) / 64);

    for (int c = 0; c < n_chunks; ++c) {
        const int64_t j = w.j0 + (int64_t)c * 64 + lane;
        const bool jv = j < w.j1;
        T sx = sym_pad<T>(), sy = sym_pad<T>(), sz = sym_pad<T>(), sm = (T)0.0;
        if (jv) {
            sx = (T)(X[j] - cx);
            sy = (T)(Y[j] - cy);
            sz = (T)(Z[j] - cz);
            sm = (T)m[j];
        }
        T qx = (T)0.0, qy = (T)0.0, qz = (T)0.0, qp = (T)0.0;
        if (eqm)
            sym_chunk<T, R, REACT, true, PHI, MASK, PHASED>(sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi,
                                                         mi, eps2, ax, ay, az, ap);
        else
            sym_chunk<T, R, REACT, false, PHI, MASK, PHASED>(sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi,
                                                          mi, eps2, ax, ay, az, ap);
        if constexpr (FOLD) {
            if ((c & 3) == 3 || c == n_chunks - 1) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (ACC == kTwoSum) {
                        two_sum_add(hx[r], lx[r], ax[r]);
                        two_sum_add(hy[r], ly[r], ay[r]);
                        two_sum_add(hz[r], lz[r], az[r]);
                        if constexpr (PHI)
                            two_sum_add(hp[r], lp[r], ap[r]);
                        ax[r] = ay[r] = az[r] = ap[r] = (T)0.0;
                    } else if constexpr (ACC == kFold64) {
                        bx[r] += (double)ax[r];
                        by[r] += (double)ay[r];
                        bz[r] += (double)az[r];
                        if constexpr (PHI)
                            bp[r] += (double)ap[r];
                        ax[r] = ay[r] = az[r] = ap[r] = (T)0.0;
                    }
                }
            }
        }
        if constexpr (REACT) {
            // reaction on this chunk's sources: the waves' sums in a fixed order
            double o[NQ];
            if constexpr (W == 1) {
                o[0] = (double)qx;
                o[1] = (double)qy;
                o[2] = (double)qz;
                if constexpr (PHI)
                    o[NQ - 1] = (double)qp;
            } else {
                T(*buf)[NQ][64] = react[c & 1];
                buf[wave][0][lane] = qx;
                buf[wave][1][lane] = qy;
                buf[wave][2][lane] = qz;
                if constexpr (PHI)
                    buf[wave][NQ - 1][lane] = qp;
                __syncthreads();
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    if constexpr (ACC == kTwoSum) {
                        float hi = (float)buf[0][q][lane], lo = 0.0f;
#pragma unroll
                        for (int v = 1; v < W; ++v)
                            two_sum_add(hi, lo, buf[v][q][lane]);
                        o[q] = (double)hi + (double)lo;
                    } else if constexpr (ACC == kFold64) {
                        double t = 0.0;
#pragma unroll
                        for (int v = 0; v < W; ++v)
                            t += (double)buf[v][q][lane];
                        o[q] = t;
                    } else {
                        T t = buf[0][q][lane];
#pragma unroll
                        for (int v = 1; v < W; ++v)
                            t += buf[v][q][lane];
                        o[q] = (double)t;
                    }
                }
            }
            if (wave == 0 && jv) {
                const int64_t rs = (int64_t)w.rslice;
                if constexpr (F32OUT) {
                    float *pf = reinterpret_cast<float *>(part);
                    pf[(rs * 3 + 0) * N + j] = qx;
                    pf[(rs * 3 + 1) * N + j] = qy;
                    pf[(rs * 3 + 2) * N + j] = qz;
                    if constexpr (PHI)
                        reinterpret_cast<float *>(part_phi)[rs * N + j] = qp;
                } else {
                    part[(rs * 3 + 0) * N + j] = scale * o[0];
                    part[(rs * 3 + 1) * N + j] = scale * o[1];
                    part[(rs * 3 + 2) * N + j] = scale * o[2];
                    if constexpr (PHI)
                        part_phi[rs * N + j] = scale * o[NQ - 1];
                }
            }
        }
    }

    const int64_t slot = (int64_t)w.slice;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!valid[r])
            continue;
        const int64_t i = w.i0 + (int64_t)(wave * 64 * R + r * 64 + lane);
        if constexpr (F32OUT) {
            float *pf = reinterpret_cast<float *>(part);
            pf[(slot * 3 + 0) * N + i] = ax[r];
            pf[(slot * 3 + 1) * N + i] = ay[r];
            pf[(slot * 3 + 2) * N + i] = az[r];
            if constexpr (PHI)
                reinterpret_cast<float *>(part_phi)[slot * N + i] = ap[r];
            continue;
        }
        double ox, oy, oz, op;
        if constexpr (FOLD && ACC == kTwoSum) {
            ox = (double)hx[r] + (double)lx[r];
            oy = (double)hy[r] + (double)ly[r];
            oz = (double)hz[r] + (double)lz[r];
            op = (double)hp[r] + (double)lp[r];
        } else if constexpr (FOLD && ACC == kFold64) {
            ox = bx[r];
            oy = by[r];
            oz = bz[r];
            op = bp[r];
        } else {
            ox = (double)ax[r];
            oy = (double)ay[r];
            oz = (double)az[r];
            op = (double)ap[r];
        }
        part[(slot * 3 + 0) * N + i] = scale * ox;
        part[(slot * 3 + 1) * N + i] = scale * oy;
        part[(slot * 3 + 2) * N + i] = scale * oz;
        if constexpr (PHI)
            part_phi[slot * N + i] = scale * op;
    }
}

// One wave per workgroup with four targets per lane is held to 96 VGPRs (80 with the
// plain loop) so that five (six) waves share each SIMD.
template <typename T, int ACC, int R, int W, bool PHI, bool MASK, bool PHASED>
__global__ __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 || R * W != 4 ? 1 : PHASED ? 5 : 6))) void
pair_sweep_sym_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const WorkItem *__restrict__ items, int n_items, int *__restrict__ counter,
    int persistent, const double *__restrict__ box_mass, double *__restrict__ part,
    double *__restrict__ part_phi, int64_t *__restrict__ step_inc)
{
    constexpr bool FOLD = 64 * R * W > 256;
    __shared__ double red[W][6];
    __shared__ T react[W > 1 ? 2 : 1][W][PHI ? 4 : 3][64];
    __shared__ int s_item;
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    if (step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *step_inc += 1;

    for (int iter = 0;; ++iter) {
        const int it = next_item(persistent, counter, &s_item, iter);
        if (it >= n_items)
            break;
        const WorkItem w = items[it];
        if (w.kind == 0)
            sym_item<T, ACC, R, W, FOLD, true, PHI, MASK, PHASED>(w, X, Y, Z, m, N, box_mass, part,
                                                                  part_phi, red, react);
        else
            sym_item<T, ACC, 1, W, FOLD, false, PHI, MASK, PHASED>(w, X, Y, Z, m, N, box_mass,
                                                                   part, part_phi, red, react);
    }
}

// ---------------------------------------------------------------------------
// Grouped symmetric sweep: four waves per workgroup, each on its own work
// item.  Parts pair up into super-parts {2A, 2A+1}; the group of two
// super-parts A < B is the 2x2 block of part pairs {p0, p1} x {q0, q1}
// (wave 2a + b: targets p_a, sources q_b).  The two waves with the same
// target part add their targets' partial sums (wave 2a's + wave 2a+1's), the
// two with the same source part their reactions (wave b's + wave b+2's),
// through LDS, so the block writes one slot per particle where the single
// items wrote two: a particle of a box of P parts gets ceil(P/2) + 1 slots
// instead of P (slot B for super-part B != A, slot A for the pair inside
// its super-part, the last for its diagonal; a part alone in its super-part
// puts its diagonal in slot A).  Items without a partner (tmate / rmate 0),
// and the groups of unrelated items (pairs inside super-parts, diagonal
// pieces), write their slots directly; padding items (kind -1) only take
// part in the barriers.  A combined slot is one addition (FP32 with FP32
// pairs, FP64 with FP64 pairs) of two partial sums of at most 256 terms.
// ---------------------------------------------------------------------------
constexpr int kGroupWaves = 4;

// Centre of the bounding box of one wave's valid targets, in every lane.
template <int R>
__device__ __forceinline__ void wave_centre(const double (&tx)[R], const double (&ty)[R],
                                            const double (&tz)[R], const bool (&valid)[R],
                                            double &cx, double &cy, double &cz)
{
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (valid[r]) {
            v[0] = fmin(v[0], tx[r]);
            v[1] = fmin(v[1], ty[r]);
            v[2] = fmin(v[2], tz[r]);
            v[3] = fmax(v[3], tx[r]);
            v[4] = fmax(v[4], ty[r]);
            v[5] = fmax(v[5], tz[r]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            v[q] = fmin(v[q], __shfl_xor(v[q], off, 64));
            v[q + 3] = fmax(v[q + 3], __shfl_xor(v[q + 3], off, 64));
        }
    }
    cx = uniform(0.5 * (v[0] + v[3]));
    cy = uniform(0.5 * (v[1] + v[4]));
    cz = uniform(0.5 * (v[2] + v[5]));
}

// The bounding box [lo, hi] of one wave's targets, in every lane (scalar
// registers); targets not to be counted repeat a valid one.
template <int R>
__device__ __forceinline__ void wave_box(const double (&tx)[R], const double (&ty)[R],
                                         const double (&tz)[R], double (&lo)[3], double (&hi)[3])
{
    lo[0] = hi[0] = tx[0];
    lo[1] = hi[1] = ty[0];
    lo[2] = hi[2] = tz[0];
#pragma unroll
    for (int r = 1; r < R; ++r) {
        lo[0] = fmin(lo[0], tx[r]);
        lo[1] = fmin(lo[1], ty[r]);
        lo[2] = fmin(lo[2], tz[r]);
        hi[0] = fmax(hi[0], tx[r]);
        hi[1] = fmax(hi[1], ty[r]);
        hi[2] = fmax(hi[2], tz[r]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            lo[q] = fmin(lo[q], __shfl_xor(lo[q], off, 64));
            hi[q] = fmax(hi[q], __shfl_xor(hi[q], off, 64));
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        lo[q] = uniform(lo[q]);
        hi[q] = uniform(hi[q]);
    }
}

// One slot value of particle i: FP32 sums stored as FP32 without the box
// mass; FP64 sums stored multiplied by it (scale, 1 when the masses differ).
template <typename T, bool PHI>
__device__ __forceinline__ void grp_store(double *__restrict__ part, double *__restrict__ part_phi,
                                          int64_t N, int64_t slot, int64_t i, T vx, T vy, T vz,
                                          T vp, double scale)
{
    if constexpr (sizeof(T) == 4) {
        float *pf = reinterpret_cast<float *>(part);
        pf[(slot * 3 + 0) * N + i] = vx;
        pf[(slot * 3 + 1) * N + i] = vy;
        pf[(slot * 3 + 2) * N + i] = vz;
        if constexpr (PHI)
            reinterpret_cast<float *>(part_phi)[slot * N + i] = vp;
    } else {
        part[(slot * 3 + 0) * N + i] = scale * vx;
        part[(slot * 3 + 1) * N + i] = scale * vy;
        part[(slot * 3 + 2) * N + i] = scale * vz;
        if constexpr (PHI)
            part_phi[slot * N + i] = scale * vp;
    }
}

// The pair loop of one wave's item (R targets per lane; REACT: a pair of
// parts with the reaction on the sources, else a diagonal piece).  The
// targets' partial sums are left in (ax, ay, az, ap); the reactions go to
// rst[NQ][256] (LDS, chunk c at 64 c + lane) when the item has a reaction
// partner, else straight to slot rslice.
template <typename T, int R, bool REACT, bool PHI, bool MASK, bool PHASED>
__device__ __forceinline__ void grp_item(const WorkItem &w, const double *__restrict__ X,
                                         const double *__restrict__ Y,
                                         const double *__restrict__ Z,
                                         const double *__restrict__ m, int64_t N, double mbox,
                                         double *__restrict__ part, double *__restrict__ part_phi,
                                         T (*rst)[256], T (&ax)[R], T (&ay)[R], T (&az)[R],
                                         T (&ap)[R], bool (&valid)[R])
{
    const int lane = threadIdx.x & 63;
    const bool eqm = !isnan(mbox);
    double tx[R], ty[R], tz[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        valid[r] = i < w.i1;
        const int64_t ii = valid[r] ? i : w.i0;
        tx[r] = X[ii];
        ty[r] = Y[ii];
        tz[r] = Z[ii];
    }
    double cx, cy, cz;
    wave_centre<R>(tx, ty, tz, valid, cx, cy, cz);
    T xi[R], yi[R], zi[R], mi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        if (valid[r]) {
            xi[r] = (T)(tx[r] - cx);
            yi[r] = (T)(ty[r] - cy);
            zi[r] = (T)(tz[r] - cz);
            mi[r] = (T)m[i];
        } else {
            xi[r] = yi[r] = zi[r] = sym_pad<T>();
            mi[r] = (T)0.0;
        }
        ax[r] = ay[r] = az[r] = ap[r] = (T)0.0;
    }
    const T eps2 = uniform((T)w.eps2);
    const double scale = eqm ? mbox : 1.0;
    const int n_chunks = (int)((w.j1 - w.j0 + 63) / 64);
    for (int c = 0; c < n_chunks; ++c) {
        const int64_t j = w.j0 + (int64_t)c * 64 + lane;
        const bool jv = j < w.j1;
        T sx = sym_pad<T>(), sy = sym_pad<T>(), sz = sym_pad<T>(), sm = (T)0.0;
        if (jv) {
            sx = (T)(X[j] - cx);
            sy = (T)(Y[j] - cy);
            sz = (T)(Z[j] - cz);
            sm = (T)m[j];
        }
        T qx = (T)0.0, qy = (T)0.0, qz = (T)0.0, qp = (T)0.0;
        if (eqm)
            sym_chunk<T, R, REACT, true, PHI, MASK, PHASED>(sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi,
                                                         mi, eps2, ax, ay, az, ap);
        else
            sym_chunk<T, R, REACT, false, PHI, MASK, PHASED>(sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi,
                                                          mi, eps2, ax, ay, az, ap);
        if constexpr (REACT) {
            if (rst) {
                rst[0][c * 64 + lane] = qx;
                rst[1][c * 64 + lane] = qy;
                rst[2][c * 64 + lane] = qz;
                if constexpr (PHI)
                    rst[3][c * 64 + lane] = qp;
            } else if (jv) {
                grp_store<T, PHI>(part, part_phi, N, (int64_t)w.rslice, j, qx, qy, qz, qp, scale);
            }
        }
    }
}

// FP32 pairs: five waves share each SIMD (96 VGPRs), six with the plain loop (80).
template <typename T, bool PHI, bool MASK, bool PHASED>
__global__ __launch_bounds__(64 * kGroupWaves)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : PHASED ? 5 : 6))) void
pair_sweep_sym_grp_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const WorkItem *__restrict__ items, int n_groups, int *__restrict__ counter,
    int persistent, const double *__restrict__ box_mass, double *__restrict__ part,
    double *__restrict__ part_phi, int64_t *__restrict__ step_inc)
{
    constexpr int NQ = PHI ? 4 : 3;
    // targets exported by the odd waves of a target pair; reactions of the
    // waves with a reaction partner
    __shared__ T tbuf[kGroupWaves / 2][NQ][256];
    __shared__ T rbuf[kGroupWaves][NQ][256];
    __shared__ int s_item;
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    // the wave index is uniform in the wave: the item loads to scalar registers
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *step_inc += 1;

    for (int iter = 0;; ++iter) {
        const int g = next_item(persistent, counter, &s_item, iter);
        if (g >= n_groups)
            break;
        const WorkItem w = items[(int64_t)g * kGroupWaves + wave];
        const double mbox = (w.kind >= 0 && box_mass) ? box_mass[w.box] : NAN;
        const double scale = isnan(mbox) ? 1.0 : mbox;
        T ax[4], ay[4], az[4], ap[4];
        bool valid[4] = {false, false, false, false};
        if (w.kind == 0) {
            grp_item<T, 4, true, PHI, MASK, PHASED>(w, X, Y, Z, m, N, mbox, part, part_phi,
                                                    w.rmate ? rbuf[wave] : nullptr, ax, ay, az,
                                                    ap, valid);
            if (!w.tmate) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (valid[r])
                        grp_store<T, PHI>(part, part_phi, N, (int64_t)w.slice,
                                          w.i0 + (int64_t)(r * 64 + lane), ax[r], ay[r], az[r],
                                          ap[r], scale);
            } else if (wave & 1) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    tbuf[wave >> 1][0][r * 64 + lane] = ax[r];
                    tbuf[wave >> 1][1][r * 64 + lane] = ay[r];
                    tbuf[wave >> 1][2][r * 64 + lane] = az[r];
                    if constexpr (PHI)
                        tbuf[wave >> 1][3][r * 64 + lane] = ap[r];
                }
            }
        } else if (w.kind == 1) {
            T bx[1], by[1], bz[1], bp[1];
            bool v1[1];
            grp_item<T, 1, false, PHI, MASK, PHASED>(w, X, Y, Z, m, N, mbox, part, part_phi,
                                                     nullptr, bx, by, bz, bp, v1);
            if (v1[0])
                grp_store<T, PHI>(part, part_phi, N, (int64_t)w.slice, w.i0 + lane, bx[0], by[0],
                                  bz[0], bp[0], scale);
        }
        __syncthreads();
        if (w.kind == 0 && w.tmate && !(wave & 1)) {
            // targets: this wave's (sources q0) + the odd wave's (sources q1)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (valid[r]) {
                    const int e = r * 64 + lane;
                    T vp = (T)0.0;
                    if constexpr (PHI)
                        vp = ap[r] + tbuf[wave >> 1][3][e];
                    grp_store<T, PHI>(part, part_phi, N, (int64_t)w.slice, w.i0 + e,
                                      ax[r] + tbuf[wave >> 1][0][e], ay[r] + tbuf[wave >> 1][1][e],
                                      az[r] + tbuf[wave >> 1][2][e], vp, scale);
                }
        }
        if (w.kind == 0 && w.rmate && wave < 2) {
            // reactions on sources q_b: from targets p0 (wave b) + p1 (wave b + 2)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int e = c * 64 + lane;
                const int64_t j = w.j0 + e;
                if (j < w.j1) {
                    T vp = (T)0.0;
                    if constexpr (PHI)
                        vp = rbuf[wave][3][e] + rbuf[wave + 2][3][e];
                    grp_store<T, PHI>(part, part_phi, N, (int64_t)w.rslice, j,
                                      rbuf[wave][0][e] + rbuf[wave + 2][0][e],
                                      rbuf[wave][1][e] + rbuf[wave + 2][1][e],
                                      rbuf[wave][2][e] + rbuf[wave + 2][2][e], vp, scale);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Symmetric adjoint sweep (form 2, FP32 pairs, one cotangent per launch).
// The adjoint pair term M(d)(m_k lam_j - m_j lam_k), M(d) = r^-3 I -
// 3 r^-5 d d^T, changes sign when k and j swap (M(-d) = M(d)), so each
// unordered pair is evaluated once, with the work items, slots and DPP
// rotation of the symmetric forward sweep; the travelling source carries
// its position, cotangent (and mass) and the accumulator of its reaction.
// Missing sources and targets sit at 1e18 with zero mass and cotangent: s
// stays finite in FP32 (3e36) while r^-3 underflows to 0, so d.u stays
// finite and the pair adds exactly 0.
//
// FULL chunks (every target and source lane holds a particle, so no padding
// position enters) apply r^-3 inside the accumulation instead:
// v = r^-3 (u - 3 r^-2 (d.u) d), added as fma(r^-3, ., acc) to the target
// and fma(-r^-3, ., q) to the reaction: three multiplies fewer per pair.
// There d.u is formed from the unscaled u, which against a padding position
// (|d| ~ 1e18) would overflow FP32 for |u| above ~1e20; chunks with padding
// therefore keep the scaled form.
//
// The step's phases are those of sym_chunk; the cotangent travels like the
// mass (one lane back at first, rotated just before its use).  A 24^3 mixed
// adjoint of 8 steps, one cotangent: 1559 -> 1312 us.
// ---------------------------------------------------------------------------
template <typename T, int R, bool REACT, bool EQM, bool MASK, bool FULL>
__device__ __forceinline__ void sym_adj_chunk(T sx, T sy, T sz, T sm, T slx, T sly, T slz,
                                              T &qx, T &qy, T &qz, const T (&xi)[R],
                                              const T (&yi)[R], const T (&zi)[R],
                                              const T (&mk)[R], const T (&lkx)[R],
                                              const T (&lky)[R], const T (&lkz)[R], T eps2,
                                              T (&ax)[R], T (&ay)[R], T (&az)[R])
{
    const T minus3 = sizeof(T) == 4 ? in_vgpr((T)-3.0) : (T)-3.0;
    if constexpr (!EQM)
        sm = wave_rotate_back(sm);
    slx = wave_rotate_back(slx);
    sly = wave_rotate_back(sly);
    slz = wave_rotate_back(slz);
#pragma unroll 1
    for (int k = 0; k < 64; ++k) {
        T dx[R], dy[R], dz[R], s[R], y[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            dx[r] = sx - xi[r];
            dy[r] = sy - yi[r];
            dz[r] = sz - zi[r];
            s[r] = fma_t(dx[r], dx[r], eps2);
            s[r] = fma_t(dy[r], dy[r], s[r]);
            s[r] = fma_t(dz[r], dz[r], s[r]);
        }
        burst_begin();
#pragma unroll
        for (int r = 0; r < R; ++r)
            y[r] = rsq_raw(s[r]);
        phase_mark();
        sx = wave_rotate(sx);
        sy = wave_rotate(sy);
        sz = wave_rotate(sz);
        slx = wave_rotate(slx);
        sly = wave_rotate(sly);
        slz = wave_rotate(slz);
        if constexpr (!EQM)
            sm = wave_rotate(sm);
        if constexpr (REACT) {
            qx = wave_rotate(qx);
            qy = wave_rotate(qy);
            qz = wave_rotate(qz);
        }
        burst_end();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            T rinv = rsqrt_from(s[r], y[r]);
            if constexpr (MASK)
                rinv = s[r] > (T)0.0 ? rinv : (T)0.0;
            // M(d) u = r^-3 u - 3 r^-5 (d.u) d = u' - 3 r^-2 (d.u') d with
            // u' = r^-3 u (one multiply fewer per pair than scaling t)
            const T r2 = rinv * rinv;
            const T r3 = r2 * rinv;
            const T m3r2 = minus3 * r2;
            T ux, uy, uz;
            if constexpr (EQM) {
                ux = slx - lkx[r];
                uy = sly - lky[r];
                uz = slz - lkz[r];
            } else {
                // both products rounded before the difference, so that the
                // self pair (j = k, inside a diagonal part) gives u = 0
                // exactly; a fused m_k lam_j - m_j lam_k would leave the
                // product's rounding error, which r^-3 = eps^-3 amplifies
#pragma clang fp contract(off)
                ux = mk[r] * slx - sm * lkx[r];
                uy = mk[r] * sly - sm * lky[r];
                uz = mk[r] * slz - sm * lkz[r];
            }
            // the reaction accumulates with the opposite sign until the end
            if constexpr (FULL) {
                const T du = fma_t(dx[r], ux, fma_t(dy[r], uy, dz[r] * uz));
                const T t = m3r2 * du;
                const T vx = fma_t(t, dx[r], ux);
                const T vy = fma_t(t, dy[r], uy);
                const T vz = fma_t(t, dz[r], uz);
                ax[r] = fma_t(r3, vx, ax[r]);
                ay[r] = fma_t(r3, vy, ay[r]);
                az[r] = fma_t(r3, vz, az[r]);
                if constexpr (REACT) {
                    qx = fma_t(r3, vx, qx);
                    qy = fma_t(r3, vy, qy);
                    qz = fma_t(r3, vz, qz);
                }
            } else {
                ux *= r3;
                uy *= r3;
                uz *= r3;
                const T du = fma_t(dx[r], ux, fma_t(dy[r], uy, dz[r] * uz));
                const T t = m3r2 * du;
                const T vx = fma_t(t, dx[r], ux);
                const T vy = fma_t(t, dy[r], uy);
                const T vz = fma_t(t, dz[r], uz);
                ax[r] += vx;
                ay[r] += vy;
                az[r] += vz;
                if constexpr (REACT) {
                    qx += vx;
                    qy += vy;
                    qz += vz;
                }
            }
        }
        phase_mark();
    }
    if constexpr (REACT) {
        qx = -wave_rotate(qx);
        qy = -wave_rotate(qy);
        qz = -wave_rotate(qz);
    }
}

// A slot value of the symmetric adjoint: FP32 pairs store the FP32 sum as it
// is (the readers apply the box mass), FP64 pairs the scaled FP64 value.
__device__ __forceinline__ void store_slot(double *part, int64_t k, float v, double)
{
    reinterpret_cast<float *>(part)[k] = v;
}
__device__ __forceinline__ void store_slot(double *part, int64_t k, double v, double scale)
{
    part[k] = scale * v;
}

// One work item of the symmetric adjoint sweep, cotangent c of n_cot; parts
// of at most 256 particles (one FP32 partial per slot, as in the forward).
template <typename T, int R, bool REACT, bool MASK>
__device__ __forceinline__ void sym_adj_item(const WorkItem &w, const double *__restrict__ X,
                                             const double *__restrict__ Y,
                                             const double *__restrict__ Z,
                                             const double *__restrict__ m,
                                             const double *__restrict__ lam, int n_cot, int c,
                                             int64_t N, const double *__restrict__ box_mass,
                                             double *__restrict__ part, double (*red)[6])
{
    const int lane = threadIdx.x & 63;
    const double mbox = box_mass ? box_mass[w.box] : NAN;
    const bool eqm = !isnan(mbox);
    const double *LX = lam + ((int64_t)c * 3 + 0) * N;
    const double *LY = lam + ((int64_t)c * 3 + 1) * N;
    const double *LZ = lam + ((int64_t)c * 3 + 2) * N;

    double tx[R], ty[R], tz[R];
    bool valid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        valid[r] = i < w.i1;
        const int64_t ii = valid[r] ? i : w.i0;
        tx[r] = X[ii];
        ty[r] = Y[ii];
        tz[r] = Z[ii];
    }
    double cx, cy, cz;
    block_centre<64, R>(tx, ty, tz, valid, red, cx, cy, cz);
    cx = uniform(cx);
    cy = uniform(cy);
    cz = uniform(cz);

    T xi[R], yi[R], zi[R], mk[R], lkx[R], lky[R], lkz[R];
    T ax[R], ay[R], az[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        if (valid[r]) {
            xi[r] = (T)(tx[r] - cx);
            yi[r] = (T)(ty[r] - cy);
            zi[r] = (T)(tz[r] - cz);
            mk[r] = (T)m[i];
            lkx[r] = (T)LX[i];
            lky[r] = (T)LY[i];
            lkz[r] = (T)LZ[i];
        } else {
            xi[r] = yi[r] = zi[r] = adj_pad<T>();
            mk[r] = lkx[r] = lky[r] = lkz[r] = (T)0.0;
        }
        ax[r] = ay[r] = az[r] = (T)0.0;
    }
    const T eps2 = uniform((T)w.eps2);
    const double scale = eqm ? mbox : 1.0;
    const int n_chunks = (int)((w.j1 - w.j0 + 63) / 64);
    const bool full_t = w.i1 - w.i0 == (int64_t)(64 * R);

    for (int ch = 0; ch < n_chunks; ++ch) {
        const int64_t j = w.j0 + (int64_t)ch * 64 + lane;
        const bool jv = j < w.j1;
        T sx = adj_pad<T>(), sy = adj_pad<T>(), sz = adj_pad<T>(), sm = (T)0.0;
        T slx = (T)0.0, sly = (T)0.0, slz = (T)0.0;
        if (jv) {
            sx = (T)(X[j] - cx);
            sy = (T)(Y[j] - cy);
            sz = (T)(Z[j] - cz);
            sm = (T)m[j];
            slx = (T)LX[j];
            sly = (T)LY[j];
            slz = (T)LZ[j];
        }
        T qx = (T)0.0, qy = (T)0.0, qz = (T)0.0;
        const bool full = full_t && w.j0 + (int64_t)(ch + 1) * 64 <= w.j1;
        if (eqm && full)
            sym_adj_chunk<T, R, REACT, true, MASK, true>(sx, sy, sz, sm, slx, sly, slz, qx, qy, qz,
                                                      xi, yi, zi, mk, lkx, lky, lkz, eps2, ax,
                                                      ay, az);
        else if (eqm)
            sym_adj_chunk<T, R, REACT, true, MASK, false>(sx, sy, sz, sm, slx, sly, slz, qx, qy, qz,
                                                       xi, yi, zi, mk, lkx, lky, lkz, eps2, ax,
                                                       ay, az);
        else if (full)
            sym_adj_chunk<T, R, REACT, false, MASK, true>(sx, sy, sz, sm, slx, sly, slz, qx, qy,
                                                       qz, xi, yi, zi, mk, lkx, lky, lkz, eps2,
                                                       ax, ay, az);
        else
            sym_adj_chunk<T, R, REACT, false, MASK, false>(sx, sy, sz, sm, slx, sly, slz, qx, qy,
                                                        qz, xi, yi, zi, mk, lkx, lky, lkz, eps2,
                                                        ax, ay, az);
        if constexpr (REACT) {
            if (jv) {
                const int64_t rs = (int64_t)w.rslice;
                store_slot(part, ((rs * n_cot + c) * 3 + 0) * N + j, qx, scale);
                store_slot(part, ((rs * n_cot + c) * 3 + 1) * N + j, qy, scale);
                store_slot(part, ((rs * n_cot + c) * 3 + 2) * N + j, qz, scale);
            }
        }
    }
    const int64_t slot = (int64_t)w.slice;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!valid[r])
            continue;
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        store_slot(part, ((slot * n_cot + c) * 3 + 0) * N + i, ax[r], scale);
        store_slot(part, ((slot * n_cot + c) * 3 + 1) * N + i, ay[r], scale);
        store_slot(part, ((slot * n_cot + c) * 3 + 2) * N + i, az[r], scale);
    }
}

template <typename T, int R, bool MASK>
__global__ __launch_bounds__(64) void adjoint_sweep_sym_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const double *__restrict__ lam, int n_cot, int c, const WorkItem *__restrict__ items,
    int n_items, int *__restrict__ counter, int persistent, const double *__restrict__ box_mass,
    double *__restrict__ part)
{
    __shared__ double red[1][6];
    __shared__ int s_item;
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    for (int iter = 0;; ++iter) {
        const int it = next_item(persistent, counter, &s_item, iter);
        if (it >= n_items)
            break;
        const WorkItem w = items[it];
        if (w.kind == 0)
            sym_adj_item<T, R, true, MASK>(w, X, Y, Z, m, lam, n_cot, c, N, box_mass, part, red);
        else
            sym_adj_item<T, 1, false, MASK>(w, X, Y, Z, m, lam, n_cot, c, N, box_mass, part, red);
    }
}

// ---------------------------------------------------------------------------
// Adjoint sweep: sum_j M(d)(m_k lam_j - m_j lam_k), M(d) = r^-3 I - 3 r^-5 d d^T,
// for C cotangents sharing the geometry.  lam is [n_cot][3][N]; this launch
// handles cotangents [c0, c0 + C).  part is [slices][n_cot][3][N].
// ---------------------------------------------------------------------------
// Pair loop of the adjoint sweep over one LDS tile.  With equal masses
// (EQM) the bracket m_k lam_j - m_j lam_k is m (lam_j - lam_k); the common
// m multiplies the slice's partial sum once instead.
template <typename T, int R, int C, bool MASK, bool EQM, bool PHASED, typename V>
__device__ __forceinline__ void adjoint_tile(const V *__restrict__ tile,
                                             const T *__restrict__ ltile, int nt,
                                             const T (&xi)[R], const T (&yi)[R],
                                             const T (&zi)[R], const T (&mk)[R],
                                             const T (&lk)[R][3 * C], T eps2,
                                             T (&acc)[R][3 * C])
{
    constexpr int LW = 3 * C;
    // PHASED (FP32): four pairs' estimates in one burst, else the compiler's order
    constexpr int U = PHASED ? 4 / R : 1;
    const T minus3 = PHASED ? in_vgpr((T)-3) : (T)-3;
    for (int j0 = 0; j0 < nt; j0 += U) {
        T dx[U][R], dy[U][R], dz[U][R], s[U][R], y[U][R], mj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // the tile is at least U long; sources past nt are not added
            const V pj = tile[j0 + u];
            mj[u] = pj.w;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dx[u][r] = pj.x - xi[r];
                dy[u][r] = pj.y - yi[r];
                dz[u][r] = pj.z - zi[r];
                s[u][r] = fma_t(dx[u][r], dx[u][r], eps2);
                s[u][r] = fma_t(dy[u][r], dy[u][r], s[u][r]);
                s[u][r] = fma_t(dz[u][r], dz[u][r], s[u][r]);
            }
        }
        if constexpr (PHASED)
            burst_begin();
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r)
                y[u][r] = rsq_raw(s[u][r]);
        if constexpr (PHASED)
            burst_end();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u >= nt)
                break;
            T lt[LW];
#pragma unroll
            for (int q = 0; q < LW; ++q)
                lt[q] = ltile[(j0 + u) * LW + q];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                T rinv = rsqrt_from(s[u][r], y[u][r]);
                if constexpr (MASK)
                    rinv = s[u][r] > (T)0 ? rinv : (T)0;
                const T r2 = rinv * rinv;
                const T r3 = r2 * rinv;
                const T m3r5 = minus3 * (r3 * r2);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    T ux, uy, uz;
                    if constexpr (EQM) {
                        ux = lt[3 * c + 0] - lk[r][3 * c + 0];
                        uy = lt[3 * c + 1] - lk[r][3 * c + 1];
                        uz = lt[3 * c + 2] - lk[r][3 * c + 2];
                    } else {
                        // rounded products, then the difference: u = 0 exactly
                        // for the self pair (see the symmetric loop)
#pragma clang fp contract(off)
                        ux = mk[r] * lt[3 * c + 0] - mj[u] * lk[r][3 * c + 0];
                        uy = mk[r] * lt[3 * c + 1] - mj[u] * lk[r][3 * c + 1];
                        uz = mk[r] * lt[3 * c + 2] - mj[u] * lk[r][3 * c + 2];
                    }
                    const T ex = dx[u][r], ey = dy[u][r], ez = dz[u][r];
                    const T du = fma_t(ex, ux, fma_t(ey, uy, ez * uz));
                    const T t = m3r5 * du;
                    acc[r][3 * c + 0] = fma_t(t, ex, fma_t(r3, ux, acc[r][3 * c + 0]));
                    acc[r][3 * c + 1] = fma_t(t, ey, fma_t(r3, uy, acc[r][3 * c + 1]));
                    acc[r][3 * c + 2] = fma_t(t, ez, fma_t(r3, uz, acc[r][3 * c + 2]));
                }
            }
        }
    }
}

template <typename T, int ACC, int R, int TPB, int C, bool MASK, bool PHASED>
__global__ __launch_bounds__(TPB) void adjoint_sweep_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const double *__restrict__ lam, int n_cot, int c0,
    const WorkItem *__restrict__ items, int n_items, int *__restrict__ counter,
    int persistent, const double *__restrict__ box_mass, double *__restrict__ part)
{
    using V = typename V4<T>::type;
    constexpr int LW = 3 * C;
    __shared__ V tile[TPB];
    __shared__ T ltile[TPB * LW];
    __shared__ double red[TPB / 64][6];
    __shared__ int s_item;
    const int tid = threadIdx.x;
    const double *X = x, *Y = x + N, *Z = x + 2 * N;

    for (int iter = 0;; ++iter) {
        const int it = next_item(persistent, counter, &s_item, iter);
        if (it >= n_items)
            break;
        const WorkItem w = items[it];
        const double mbox = box_mass ? box_mass[w.box] : NAN;
        const bool eqm = !isnan(mbox);

        double tx[R], ty[R], tz[R];
        bool valid[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = w.i0 + tid + (int64_t)r * TPB;
            valid[r] = i < w.i1;
            const int64_t ii = valid[r] ? i : w.i0;
            tx[r] = X[ii];
            ty[r] = Y[ii];
            tz[r] = Z[ii];
        }
        double cx, cy, cz;
        block_centre<TPB, R>(tx, ty, tz, valid, red, cx, cy, cz);

        T xi[R], yi[R], zi[R], mk[R];
        T lk[R][LW];    // lam_k
        T acc[R][LW];   // tile partial / direct sum
        double fold[R][LW];
        T hi[R][LW], lo[R][LW];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = w.i0 + tid + (int64_t)r * TPB;
            const int64_t ii = valid[r] ? i : w.i0;
            xi[r] = (T)(tx[r] - cx);
            yi[r] = (T)(ty[r] - cy);
            zi[r] = (T)(tz[r] - cz);
            mk[r] = (T)m[ii];
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    lk[r][3 * c + q] = (T)lam[((int64_t)(c0 + c) * 3 + q) * N + ii];
                    acc[r][3 * c + q] = (T)0;
                    fold[r][3 * c + q] = 0.0;
                    hi[r][3 * c + q] = (T)0;
                    lo[r][3 * c + q] = (T)0;
                }
        }
        const T eps2 = (T)w.eps2;

        for (int64_t jt = w.j0; jt < w.j1; jt += TPB) {
            const int64_t j = jt + tid;
            V v;
            T lj[LW];
            if (j < w.j1) {
                v.x = (T)(X[j] - cx);
                v.y = (T)(Y[j] - cy);
                v.z = (T)(Z[j] - cz);
                v.w = (T)m[j];
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        lj[3 * c + q] = (T)lam[((int64_t)(c0 + c) * 3 + q) * N + j];
            } else {
                v.x = v.y = v.z = v.w = (T)0;
#pragma unroll
                for (int q = 0; q < LW; ++q)
                    lj[q] = (T)0;
            }
            __syncthreads();
            tile[tid] = v;
#pragma unroll
            for (int q = 0; q < LW; ++q)
                ltile[tid * LW + q] = lj[q];
            __syncthreads();
            const int nt = (int)((w.j1 - jt) < TPB ? (w.j1 - jt) : TPB);
            if (eqm)
                adjoint_tile<T, R, C, MASK, true, PHASED>(tile, ltile, nt, xi, yi, zi, mk, lk, eps2,
                                                          acc);
            else
                adjoint_tile<T, R, C, MASK, false, PHASED>(tile, ltile, nt, xi, yi, zi, mk, lk,
                                                           eps2, acc);
            if constexpr (ACC != kDirect) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int q = 0; q < LW; ++q) {
                        if constexpr (ACC == kTwoSum)
                            two_sum_add(hi[r][q], lo[r][q], (float)acc[r][q]);
                        else
                            fold[r][q] += (double)acc[r][q];
                        acc[r][q] = (T)0;
                    }
            }
        }

        const int64_t slot = (int64_t)w.slice;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!valid[r])
                continue;
            const int64_t i = w.i0 + tid + (int64_t)r * TPB;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    double o;
                    if constexpr (ACC == kTwoSum)
                        o = (double)hi[r][3 * c + q] + (double)lo[r][3 * c + q];
                    else if constexpr (ACC == kFold64)
                        o = fold[r][3 * c + q];
                    else
                        o = (double)acc[r][3 * c + q];
                    part[((slot * n_cot + (c0 + c)) * 3 + q) * N + i] = eqm ? mbox * o : o;
                }
        }
    }
}

__global__ void zero_counter_kernel(int *counter) { *counter = 0; }

// ---------------------------------------------------------------------------
// Host-side dispatch over the template instantiations.
// ---------------------------------------------------------------------------
struct LaunchShape {
    int grid;
};

int device_cu_count()
{
    static int cached = -1;
    if (cached > 0)
        return cached;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
        n = 256;
    cached = n;
    return n;
}

template <typename K>
int persistent_grid(K kernel, int tpb, size_t dyn_lds, int n_items)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, tpb, dyn_lds) !=
            hipSuccess ||
        per_cu <= 0)
        per_cu = 1;
    long g = (long)per_cu * device_cu_count();
    return (int)(g < n_items ? g : n_items);
}

template <typename T, int ACC, int R, int TPB, bool PHI, bool MASK, int FORM>
hipError_t launch_fwd(const double *x, const double *m, int64_t N, const WorkItem *items,
                      int n_items, int *counter, bool persistent, const double *box_mass,
                      double *part, double *part_phi, int64_t *step_inc, hipStream_t stream)
{
    auto k = pair_sweep_kernel<T, ACC, R, TPB, PHI, MASK, FORM>;
    int grid = persistent ? persistent_grid(k, TPB, 0, n_items) : n_items;
    if (grid <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k, dim3(grid), dim3(TPB), 0, stream, x, m, N, items, n_items, counter,
                       persistent ? 1 : 0, box_mass, part, part_phi, step_inc);
    return hipGetLastError();
}

struct FwdArgs {
    const double *x, *m;
    int64_t N;
    const WorkItem *items;
    int n_items;
    int *counter;
    bool persistent;
    const double *box_mass;
    double *part, *part_phi;
    int64_t *step_inc;
    hipStream_t s;
};

template <typename T, int ACC, int R, int W, bool PHI, bool MASK, bool PHASED>
hipError_t launch_sym(const FwdArgs &a)
{
    auto k = pair_sweep_sym_kernel<T, ACC, R, W, PHI, MASK, PHASED>;
    int grid = a.persistent ? persistent_grid(k, 64 * W, 0, a.n_items) : a.n_items;
    if (grid <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * W), 0, a.s, a.x, a.m, a.N, a.items, a.n_items,
                       a.counter, a.persistent ? 1 : 0, a.box_mass, a.part, a.part_phi,
                       a.step_inc);
    return hipGetLastError();
}

template <typename T, int ACC, int R, int W, bool PHASED>
hipError_t dispatch_sym_flags(bool phi, bool mask, const FwdArgs &a)
{
    if (phi)
        return mask ? launch_sym<T, ACC, R, W, true, true, PHASED>(a)
                    : launch_sym<T, ACC, R, W, true, false, PHASED>(a);
    return mask ? launch_sym<T, ACC, R, W, false, true, PHASED>(a)
                : launch_sym<T, ACC, R, W, false, false, PHASED>(a);
}

// The loop of a sweep of single items, by its waves of part pairs (of all items, FP64)
// as the grouped one's (sym_phased).  Plain / phased, us, FP32 pairs: R = 4, one wave,
// 11 000 particles (903 pairs) 49.7 / 51.3; R = 8 and R = 4 with two waves, 8000 (120
// pairs) 134 / 141 and 77.6 / 83.2.  FP64 8000 (496 pairs) 59.8 / 62.6.
template <typename T, int ACC, int R, int W>
hipError_t dispatch_sym_items(const TileCfg &cfg, bool phi, bool mask, const FwdArgs &a)
{
    const int64_t waves = (sizeof(T) == 8 ? (int64_t)a.n_items : cfg.pairs) * W;
    return waves > (sizeof(T) == 8 || R * W == 4 ? 1024 : 640)
               ? dispatch_sym_flags<T, ACC, R, W, true>(phi, mask, a)
               : dispatch_sym_flags<T, ACC, R, W, false>(phi, mask, a);
}

// Whether a grouped sweep takes the phased loop (sym_chunk), which pays once most
// SIMDs hold two waves to pair.  Plain / phased, us, equal masses unless said:
// FP32: 10 000 particles (195 groups of part pairs, 1 per CU at most) 43.3 / 44.9,
// 11 500 (259) 64.1 / 47.7, 40 boxes of 300-3300 (356 groups, of them fewer
// than 256 of pairs) 44.8 / 46.1, 24 000 140 / 114.  FP64, its v_rsq alone to hide:
// 10 000 (235 groups in all) 55.9 / 58.4, 11 000 (280) 61.5 / 60.3, 32 768 350 /
// 344; with the potential 8000 61.9 / 67.6, 15 000 (501) 110 / 113, 16 000 (567)
// 117 / 116, 49 boxes of 300-3300 (533) 80.2 / 77.5.  Boxes of one part, without
// pairs: FP32 2000 boxes of 30 (500 groups) 10.8 / 10.4, 100 000 (25 000) 164 / 179
// (unequal masses 191 / 184), with the potential 8000 boxes of 200 212 / 210; FP64
// 2000 of 30 13.0 / 13.9, 8000 of 200 (8000) 328 / 320, with the potential 13.4 /
// 15.5 and 309 / 327 (100 000 of 30).
bool sym_phased(bool fp64, bool phi, int n_groups, const TileCfg &cfg)
{
    constexpr int kCUs = 256;
    if (cfg.slices == 1)
        return fp64 ? !phi && n_groups >= 4 * kCUs : phi || n_groups < 4 * kCUs;
    if (fp64)
        return n_groups > (phi ? 2 * kCUs : kCUs);
    return cfg.pairs > (int64_t)kGroupWaves * kCUs;
}

// Grouped symmetric sweep: a.items holds kGroupWaves items per group.
template <typename T, bool PHI, bool MASK, bool PHASED>
hipError_t launch_sym_grp(const FwdArgs &a, int n_groups)
{
    auto k = pair_sweep_sym_grp_kernel<T, PHI, MASK, PHASED>;
    const int tpb = 64 * kGroupWaves;
    int grid = a.persistent ? persistent_grid(k, tpb, 0, n_groups) : n_groups;
    if (grid <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k, dim3(grid), dim3(tpb), 0, a.s, a.x, a.m, a.N, a.items, n_groups,
                       a.counter, a.persistent ? 1 : 0, a.box_mass, a.part, a.part_phi,
                       a.step_inc);
    return hipGetLastError();
}

template <typename T, bool PHASED>
hipError_t dispatch_sym_grp_flags(bool phi, bool mask, const FwdArgs &a, int n_groups)
{
    if (phi)
        return mask ? launch_sym_grp<T, true, true, PHASED>(a, n_groups)
                    : launch_sym_grp<T, true, false, PHASED>(a, n_groups);
    return mask ? launch_sym_grp<T, false, true, PHASED>(a, n_groups)
                : launch_sym_grp<T, false, false, PHASED>(a, n_groups);
}

template <typename T>
hipError_t dispatch_sym_grp(const TileCfg &cfg, bool phi, bool mask, const FwdArgs &a)
{
    if (a.n_items % kGroupWaves != 0)
        return hipErrorInvalidValue;
    const int n_groups = a.n_items / kGroupWaves;
    return sym_phased(sizeof(T) == 8, phi, n_groups, cfg)
               ? dispatch_sym_grp_flags<T, true>(phi, mask, a, n_groups)
               : dispatch_sym_grp_flags<T, false>(phi, mask, a, n_groups);
}

template <typename T, int ACC>
hipError_t dispatch_sym(const TileCfg &cfg, bool phi, bool mask, const FwdArgs &a)
{
    if (cfg.group) {
        if (cfg.R != 4 || cfg.tpb != 64)
            return hipErrorInvalidValue;
        return dispatch_sym_grp<T>(cfg, phi, mask, a);
    }
    if constexpr (sizeof(T) == 4) {
        if (cfg.R == 4 && cfg.tpb == 64)
            return dispatch_sym_items<T, ACC, 4, 1>(cfg, phi, mask, a);
        if (cfg.R == 8 && cfg.tpb == 64)
            return dispatch_sym_items<T, ACC, 8, 1>(cfg, phi, mask, a);
        if (cfg.R == 4 && cfg.tpb == 128)
            return dispatch_sym_items<T, ACC, 4, 2>(cfg, phi, mask, a);
    } else {
        if (cfg.R == 4 && cfg.tpb == 64)
            return dispatch_sym_items<T, ACC, 4, 1>(cfg, phi, mask, a);
        if (cfg.R == 2 && cfg.tpb == 128)
            return dispatch_sym_items<T, ACC, 2, 2>(cfg, phi, mask, a);
    }
    return hipErrorInvalidValue;
}

template <typename T, int ACC, int R, int TPB, int FORM>
hipError_t dispatch_fwd_flags(bool phi, bool mask, const FwdArgs &a)
{
#define COLATUS_FWD_F(P, M)                                                                   \
    return launch_fwd<T, ACC, R, TPB, P, M, FORM>(a.x, a.m, a.N, a.items, a.n_items, a.counter, \
                                                  a.persistent, a.box_mass, a.part, a.part_phi, \
                                                  a.step_inc, a.s);
    if (phi) {
        if (mask) {
            COLATUS_FWD_F(true, true)
        }
        COLATUS_FWD_F(true, false)
    }
    if (mask) {
        COLATUS_FWD_F(false, true)
    }
    COLATUS_FWD_F(false, false)
#undef COLATUS_FWD_F
}

template <typename T, int ACC, int FORM>
hipError_t dispatch_fwd_shape(const TileCfg &cfg, bool phi, bool mask, const FwdArgs &a)
{
#define COLATUS_FWD(RR, TT)                                                                  \
    if (cfg.R == RR && cfg.tpb == TT)                                                        \
        return dispatch_fwd_flags<T, ACC, RR, TT, FORM>(phi, mask, a);
    COLATUS_FWD(1, 256)
    COLATUS_FWD(2, 256)
    COLATUS_FWD(4, 256)
    COLATUS_FWD(1, 128)
    COLATUS_FWD(2, 128)
    COLATUS_FWD(4, 128)
#undef COLATUS_FWD
    return hipErrorInvalidValue;
}

template <typename T, int ACC>
hipError_t dispatch_fwd_form(int form, const TileCfg &cfg, bool phi, bool mask, const FwdArgs &a)
{
    if (form == 2)
        return dispatch_sym<T, ACC>(cfg, phi, mask, a);
    if (form == 1)
        return dispatch_fwd_shape<T, ACC, 1>(cfg, phi, mask, a);
    return dispatch_fwd_shape<T, ACC, 0>(cfg, phi, mask, a);
}

// Whether the ordered adjoint sweep takes the phased loop (adjoint_tile; FP32 pairs):
// up to one block of four waves per CU it hides latency, and eight cotangents gain at
// every size unless coincident pairs are masked.  Plain / phased, us, equal masses, N = 4096 (256 blocks), 6145 (625) and
// 20 011: one cotangent 32.6 / 30.9, 39.2 / 42.0, 243 / 247; four 54.2 / 51.9, 80.0 /
// 80.8, 512 / 519; eight 78.8 / 78.8, 153 / 151, 1031 / 1019.  Unequal masses gain
// more (one cotangent 39.6 / 32.4, 44.7 / 43.9, 270 / 266), but a kernel with each
// loop for its masses runs the plain one slower (N = 4097: 31.6 -> 34.0).  Eight
// cotangents with the mask, a whole call: 11 000 particles 481 / 494, 32 768 3117 /
// 3167.  FP64 instructions are never paired, and batching them measured 1 % slower.
template <typename T, int C> bool adj_phased(bool mask, int n_items)
{
    return sizeof(T) == 4 && ((C == 8 && !mask) || n_items <= 256);
}

template <typename T, int ACC, int R, int TPB, int C, bool MASK, bool PHASED>
hipError_t launch_adj_k(const double *x, const double *m, int64_t N, const double *lam, int n_cot,
                        int c0, const WorkItem *items, int n_items, int *counter, bool persistent,
                        const double *box_mass, double *part, hipStream_t stream)
{
    auto k = adjoint_sweep_kernel<T, ACC, R, TPB, C, MASK, PHASED>;
    const int grid = persistent ? persistent_grid(k, TPB, 0, n_items) : n_items;
    hipLaunchKernelGGL(k, dim3(grid), dim3(TPB), 0, stream, x, m, N, lam, n_cot, c0, items,
                       n_items, counter, persistent ? 1 : 0, box_mass, part);
    return hipGetLastError();
}

template <typename T, int ACC, int R, int TPB, int C>
hipError_t launch_adj(bool mask, const double *x, const double *m, int64_t N, const double *lam,
                      int n_cot, int c0, const WorkItem *items, int n_items, int *counter,
                      bool persistent, const double *box_mass, double *part, hipStream_t stream)
{
    auto go = [&](auto launch) {
        return launch(x, m, N, lam, n_cot, c0, items, n_items, counter, persistent, box_mass, part,
                      stream);
    };
    if constexpr (sizeof(T) == 4)
        if (adj_phased<T, C>(mask, n_items))
            return mask ? go(launch_adj_k<T, ACC, R, TPB, C, true, true>)
                        : go(launch_adj_k<T, ACC, R, TPB, C, false, true>);
    return mask ? go(launch_adj_k<T, ACC, R, TPB, C, true, false>)
                : go(launch_adj_k<T, ACC, R, TPB, C, false, false>);
}

template <typename T, int R, bool MASK>
hipError_t launch_adj_sym(const double *x, const double *m, int64_t N, const double *lam,
                          int n_cot, const WorkItem *items, int n_items, int *counter,
                          bool persistent, const double *box_mass, double *part, hipStream_t s)
{
    auto k = adjoint_sweep_sym_kernel<T, R, MASK>;
    const int grid = persistent ? persistent_grid(k, 64, 0, n_items) : n_items;
    for (int c = 0; c < n_cot; ++c) {
        if (c > 0 && persistent)
            hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, s, counter);
        hipLaunchKernelGGL(k, dim3(grid), dim3(64), 0, s, x, m, N, lam, n_cot, c, items, n_items,
                           counter, persistent ? 1 : 0, box_mass, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <typename T, int ACC>
hipError_t dispatch_adj(const TileCfg &cfg, bool mask, const double *x, const double *m,
                        int64_t N, int n_cot, const double *lam, const WorkItem *items,
                        int n_items, int *counter, bool persistent, const double *box_mass,
                        double *part, hipStream_t s)
{
    if (cfg.form == 2) {
        if (cfg.R != 4 || cfg.tpb != 64)
            return hipErrorInvalidValue;
        return mask ? launch_adj_sym<T, 4, true>(x, m, N, lam, n_cot, items, n_items, counter,
                                                 persistent, box_mass, part, s)
                    : launch_adj_sym<T, 4, false>(x, m, N, lam, n_cot, items, n_items, counter,
                                                  persistent, box_mass, part, s);
    }
    // Cotangents in chunks of 8, then 4, then 1; the work counter is re-armed
    // before every chunk after the first.
    int c0 = 0;
    bool first = true;
    while (c0 < n_cot) {
        const int left = n_cot - c0;
        if (!first && persistent) {
            hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, s, counter);
        }
        first = false;
        hipError_t e;
        const bool r2 = cfg.R >= 2;
        if (left >= 8) {
            // eight cotangents keep 24 accumulators per target: one target per lane
            e = launch_adj<T, ACC, 1, 256, 8>(mask, x, m, N, lam, n_cot, c0, items, n_items,
                                              counter, persistent, box_mass, part, s);
            c0 += 8;
        } else if (left >= 4) {
            e = r2 ? launch_adj<T, ACC, 2, 256, 4>(mask, x, m, N, lam, n_cot, c0, items, n_items,
                                                    counter, persistent, box_mass, part, s)
                   : launch_adj<T, ACC, 1, 256, 4>(mask, x, m, N, lam, n_cot, c0, items, n_items,
                                                    counter, persistent, box_mass, part, s);
            c0 += 4;
        } else {
            e = r2 ? launch_adj<T, ACC, 2, 256, 1>(mask, x, m, N, lam, n_cot, c0, items, n_items,
                                                    counter, persistent, box_mass, part, s)
                   : launch_adj<T, ACC, 1, 256, 1>(mask, x, m, N, lam, n_cot, c0, items, n_items,
                                                    counter, persistent, box_mass, part, s);
            c0 += 1;
        }
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Periodic boundaries: the real-space part of the Ewald sum, on the work
// items of the symmetric loop (parts of 256, four targets per lane, one wave;
// each unordered pair evaluated once and applied to both particles: the
// term changes sign when the two particles swap).  Per pair, with d the
// nearest image of x_j - x_k, r = |d|:
//   w   = (r^2 + eps^2)^{-3/2} - P(r) r^{-3}
//   psi = (r^2 + eps^2)^{-1/2} - Phi(r) / r
// i.e. the Plummer pair of Eq. (1) less the smooth long-range part that the
// reciprocal-space sum carries; the other images are negligible (the short-range
// kernel ends, to the precision's resolution, at half the box).  FP32 pairs:
// Phi = erf(alpha r), P = erf(u) - (2u / sqrt(pi)) e^{-u^2}, u = alpha r.  FP64
// pairs: the prolate window (ewald_window.h), whose Phi / r and P / r^3 are
// polynomials in r^2 up to r_c = L / 2 and 1 / r and 1 / r^3 beyond.  r == 0: w = 0; a
// part's own particle has psi = (eps^2)^{-1/2} (0 at eps == 0), the value the
// open-box loop gives its self pair and the O(N) kernels remove, and its smooth
// part is the self term's; another particle at the same place has psi less the
// limit of Phi / r.
// FP64 pairs take coordinates relative to the item's first target, each
// wrapped to its nearest image before the subtraction, and wrap the pair's
// separation once more.  FP32 pairs take 32-bit fixed-point coordinates
// (below).  Masses multiply every term (missing particles have mass 0), and
// the slots hold them: readers are given no common mass.
// ---------------------------------------------------------------------------
struct EwaldReal {
    double L, invL;
    double rc2;          // r_c^2
    double tscale;       // -2 / r_c^2: t = 1 + tscale r^2
    const double *poly;  // device: P r^{-3} in powers of t (kWindowDegree + 1), then
                         // Phi r^{-1} (kWindowDegree + 2)
};

__device__ __forceinline__ double wrap_image(double d, double L)
{
    return d - L * rint(d / L);
}

// 64 steps of one source chunk (sources travel around the wave as in
// sym_chunk) against the lane's R targets, FP64.  wx, wy, wz: this axis'
// separations may exceed half the box (ewald_item) and are wrapped to the
// nearest image.  A step whose pairs all lie beyond r_c skips the polynomials,
// one whose pairs all lie within it the second square root.  The polynomials'
// constants are read from LDS at the start of every step, every lane the
// same word: kept in registers they take half the waves, and scalar loads in
// the loop wait too long (20^3 / 32^3 evaluations: 275 / 1304 us so, 258 / 1317
// kept in registers, 460 / 1577 by scalar loads).  Bound by FP64 issue; with
// the math library's erf and exp (about 180 issue slots per pair; 76 now, counted)
// a 32^3 evaluation took 2.95 ms.
template <int R, bool REACT, bool PHI>
__device__ __forceinline__ void ewald_chunk(bool wx, bool wy, bool wz, double sx, double sy,
                                            double sz, double sm, double &qx, double &qy,
                                            double &qz, double &qp,
                                            const double (&xi)[R], const double (&yi)[R],
                                            const double (&zi)[R], const double (&mi)[R],
                                            double eps2, const EwaldReal &E, const double *spoly,
                                            double (&ax)[R], double (&ay)[R], double (&az)[R],
                                            double (&ap)[R])
{
#pragma unroll 1
    for (int k = 0; k < 64; ++k) {
        double dx[R], dy[R], dz[R], r2[R], w[R], psi[R], F[R], S[R];
        bool near = false, far = false;
        constexpr int kPoly = PHI ? 2 * kWindowDegree + 3 : kWindowDegree + 1;
        double poly[kPoly];
        int at = 0;
        asm volatile("" : "+v"(at));  // read in this step, not before the loop
#pragma unroll
        for (int i = 0; i < kPoly; ++i)
            poly[i] = spoly[at + i];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            dx[r] = sx - xi[r];
            dy[r] = sy - yi[r];
            dz[r] = sz - zi[r];
        }
        if (wx)
#pragma unroll
            for (int r = 0; r < R; ++r)
                dx[r] = fma(-E.L, rint(dx[r] * E.invL), dx[r]);
        if (wy)
#pragma unroll
            for (int r = 0; r < R; ++r)
                dy[r] = fma(-E.L, rint(dy[r] * E.invL), dy[r]);
        if (wz)
#pragma unroll
            for (int r = 0; r < R; ++r)
                dz[r] = fma(-E.L, rint(dz[r] * E.invL), dz[r]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            r2[r] = fma(dx[r], dx[r], fma(dy[r], dy[r], dz[r] * dz[r]));
            near = near || r2[r] < E.rc2;
            far = far || !(r2[r] < E.rc2);
            const double s = r2[r] + eps2;
            const double y = __builtin_amdgcn_rsq(s);
            w[r] = rinv3_exact(s, y);
            if constexpr (PHI)
                psi[r] = rsqrt_exact(s, y);
            F[r] = S[r] = 0.0;
        }
        if (__any(near)) {
            double t[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                t[r] = fma(E.tscale, r2[r], 1.0);
                F[r] = poly[kWindowDegree];
                if constexpr (PHI)
                    S[r] = poly[2 * kWindowDegree + 2];
            }
#pragma unroll
            for (int i = kWindowDegree - 1; i >= 0; --i)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    F[r] = fma(F[r], t[r], poly[i]);
            if constexpr (PHI) {
#pragma unroll
                for (int i = kWindowDegree; i >= 0; --i)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        S[r] = fma(S[r], t[r], poly[kWindowDegree + 1 + i]);
            }
        }
        if (__any(far)) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double y = __builtin_amdgcn_rsq(r2[r]);
                const bool in = r2[r] < E.rc2;
                F[r] = in ? F[r] : rinv3_exact(r2[r], y);
                if constexpr (PHI)
                    S[r] = in ? S[r] : rsqrt_exact(r2[r], y);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool nz = r2[r] > 0.0;
            w[r] = nz ? w[r] - F[r] : 0.0;
            const double wt = sm * w[r];
            ax[r] = fma(wt, dx[r], ax[r]);
            ay[r] = fma(wt, dy[r], ay[r]);
            az[r] = fma(wt, dz[r], az[r]);
            if constexpr (PHI) {
                if (!(eps2 > 0.0))
                    psi[r] = nz ? psi[r] : 0.0;
                psi[r] -= S[r];
                ap[r] = fma(sm, psi[r], ap[r]);
            }
            if constexpr (REACT) {
                const double ws = mi[r] * w[r];
                qx = fma(-ws, dx[r], qx);
                qy = fma(-ws, dy[r], qy);
                qz = fma(-ws, dz[r], qz);
                if constexpr (PHI)
                    qp = fma(mi[r], psi[r], qp);
            }
        }
        sx = wave_rotate(sx);
        sy = wave_rotate(sy);
        sz = wave_rotate(sz);
        sm = wave_rotate(sm);
        if constexpr (REACT) {
            qx = wave_rotate(qx);
            qy = wave_rotate(qy);
            qz = wave_rotate(qz);
            if constexpr (PHI)
                qp = wave_rotate(qp);
        }
    }
}

// One work item of FP64 pairs (kind 0: a pair of parts with the reaction;
// kind 1: 64 targets against a part).  Slots as the symmetric loop's, FP64,
// masses included.
template <int R, bool REACT, bool PHI>
__device__ __forceinline__ void ewald_item(const WorkItem &w, const double *__restrict__ X,
                                           const double *__restrict__ Y,
                                           const double *__restrict__ Z,
                                           const double *__restrict__ m, int64_t N,
                                           double *__restrict__ part,
                                           double *__restrict__ part_phi, const EwaldReal &E,
                                           const double *spoly)
{
    const int lane = threadIdx.x & 63;
    const double L = E.L;
    // reference point: the item's first target (wave-uniform)
    const double cx = X[w.i0], cy = Y[w.i0], cz = Z[w.i0];
    double xi[R], yi[R], zi[R], mi[R];
    double ax[R], ay[R], az[R], ap[R];
    bool valid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        valid[r] = i < w.i1;
        const int64_t ii = valid[r] ? i : w.i0;
        xi[r] = wrap_image(X[ii] - cx, L);
        yi[r] = wrap_image(Y[ii] - cy, L);
        zi[r] = wrap_image(Z[ii] - cz, L);
        mi[r] = valid[r] ? m[i] : 0.0;
        ax[r] = ay[r] = az[r] = ap[r] = 0.0;
    }
    // the targets' bounding box: centre b, half extent h.  A source taken at
    // its image nearest to b is at its nearest image to every target if it lies
    // within L / 2 - h of b; a chunk whose sources all do needs no wrap on that
    // axis (about two thirds of the axes with particles in Morton order).  A NaN
    // compares false and takes the wrap.
    double lo[3], hi[3];
    wave_box<R>(xi, yi, zi, lo, hi);
    const double bx = 0.5 * (lo[0] + hi[0]), by = 0.5 * (lo[1] + hi[1]),
                 bz = 0.5 * (lo[2] + hi[2]);
    // a little inside the limit, for the roundings of b and h
    const double ex = 0.4999999 * L - 0.5 * (hi[0] - lo[0]),
                 ey = 0.4999999 * L - 0.5 * (hi[1] - lo[1]),
                 ez = 0.4999999 * L - 0.5 * (hi[2] - lo[2]);
    const double eps2 = w.eps2;
    const int n_chunks = (int)((w.j1 - w.j0 + 63) / 64);
    for (int c = 0; c < n_chunks; ++c) {
        const int64_t j = w.j0 + (int64_t)c * 64 + lane;
        const bool jv = j < w.j1;
        double sx = bx, sy = by, sz = bz, sm = 0.0;
        if (jv) {
            // as the targets first, so that a part's own particle is at r = 0
            sx = wrap_image(X[j] - cx, L);
            sx -= L * rint((sx - bx) / L);
            sy = wrap_image(Y[j] - cy, L);
            sy -= L * rint((sy - by) / L);
            sz = wrap_image(Z[j] - cz, L);
            sz -= L * rint((sz - bz) / L);
            sm = m[j];
        }
        const bool wx = !__all(fabs(sx - bx) <= ex), wy = !__all(fabs(sy - by) <= ey),
                   wz = !__all(fabs(sz - bz) <= ez);
        double qx = 0.0, qy = 0.0, qz = 0.0, qp = 0.0;
        ewald_chunk<R, REACT, PHI>(wx, wy, wz, sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi, mi,
                                   eps2, E, spoly, ax, ay, az, ap);
        if constexpr (REACT) {
            if (jv) {
                const int64_t rs = (int64_t)w.rslice;
                part[(rs * 3 + 0) * N + j] = qx;
                part[(rs * 3 + 1) * N + j] = qy;
                part[(rs * 3 + 2) * N + j] = qz;
                if constexpr (PHI)
                    part_phi[rs * N + j] = qp;
            }
        }
    }
    if constexpr (PHI && !REACT) {
        // a piece of a diagonal: its targets' own pairs took the limit of Phi / r off,
        // which is the self term's
        if (w.i0 >= w.j0 && w.i0 < w.j1) {
            double own = spoly[2 * kWindowDegree + 2];
#pragma unroll
            for (int i = kWindowDegree; i >= 0; --i)
                own += spoly[kWindowDegree + 1 + i];
#pragma unroll
            for (int r = 0; r < R; ++r)
                ap[r] = fma(mi[r], own, ap[r]);
        }
    }
    const int64_t slot = (int64_t)w.slice;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!valid[r])
            continue;
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        part[(slot * 3 + 0) * N + i] = ax[r];
        part[(slot * 3 + 1) * N + i] = ay[r];
        part[(slot * 3 + 2) * N + i] = az[r];
        if constexpr (PHI)
            part_phi[slot * N + i] = ap[r];
    }
}

// FP32 pairs on fixed-point coordinates.  Each coordinate is stored as
// round(x 2^32 / L) modulo 2^32 (FP64 arithmetic, exact for |x| below
// 2^21 L); the difference
// of two such values, read as a signed 32-bit integer, is the nearest image
// of the separation to 2^-32 L, with no wrap arithmetic, and one conversion
// gives it in FP32.  Inside the loop lengths are in units of L / 2^32; the
// stores scale the sums back (the force by (2^32 / L)^2, the potential by
// 2^32 / L).
struct EwaldFx {
    float eps2;      // eps^2 in those units
    float c_exp;     // -alpha^2 log2(e): exp(-alpha^2 r^2) = 2^(c_exp r^2)
    float c_t;       // 0.3275911 alpha
    float c_g;       // (2 / sqrt(pi)) alpha
    float phi_self;  // the own particle's potential term: (eps^2)^{-1/2}, 0 at eps = 0
    float phi_same;  // another particle's at r = 0: less the limit of erf(alpha r) / r
};

__device__ __forceinline__ uint32_t fx_coord(double x, double scale)
{
    double q = rint(x * scale);  // an integer; exact below 2^53
    q -= 4294967296.0 * floor(q * 2.3283064365386963e-10);  // mod 2^32
    // a non-finite coordinate (or one beyond 2^21 L) takes 0 here, a defined
    // conversion; a NaN still reaches every field through the reciprocal sums
    return q >= 0.0 && q < 4294967296.0 ? (uint32_t)q : 0u;
}

__device__ __forceinline__ uint32_t wave_rotate_u(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x13C, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t wave_rotate_back_u(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x134, 0xF, 0xF, true);
}

// FP32 pairs.  With u = alpha r, Hastings' approximation (Abramowitz and
// Stegun 7.1.26; absolute error at most 1.5e-7, a few FP32 units of the
// kernel it enters) gives erf(u) = 1 - t p(t) g, t = 1 / (1 + 0.3275911 u),
// g = exp(-u^2), p of fourth degree, so that
// P(u) = erf(u) - (2 / sqrt(pi)) u g = 1 - g (t p + c_g r).  (Folding c_g
// into the exponent as 2^(c_exp r^2 + log2 c_g) would save the product c_g r
// but raises the exponent's rounding error sixfold.)  At r = 0 the pair's
// terms are selected (w = 0, psi = phi0), not branched to, so that the
// target rows interleave.
//
// 64 steps of one source chunk, in the phases of sym_chunk: separations; a
// burst of the two square roots and the exponential of every pair; the
// argument of t; a burst of the reciprocals with the rotations; weights and
// accumulations.  The polynomial's constants sit in vector registers
// (in_vgpr).  A piece of a diagonal (R = 1) takes four steps at a time.
struct EwaldFxRegs {
    float eps2, c_exp, c_t, c_g, one, k4, k3, k2, k1, k0;
};

__device__ __forceinline__ EwaldFxRegs ewald_fx_regs(const EwaldFx &E)
{
    return {in_vgpr(E.eps2),       in_vgpr(E.c_exp),       in_vgpr(E.c_t),
            in_vgpr(E.c_g),        in_vgpr(1.0f),          in_vgpr(1.061405429f),
            in_vgpr(-1.453152027f), in_vgpr(1.421413741f), in_vgpr(-0.284496736f),
            in_vgpr(0.254829592f)};
}

// r^2, the burst of square roots and exponentials, and the argument of t, of
// B pairs with separations (dx, dy, dz).
template <int B>
__device__ __forceinline__ void ewald_fx_roots(const EwaldFxRegs &C, const float (&dx)[B],
                                               const float (&dy)[B], const float (&dz)[B],
                                               float (&r2)[B], float (&rs)[B], float (&ri)[B],
                                               float (&r)[B], float (&g)[B], float (&t)[B])
{
#pragma unroll
    for (int b = 0; b < B; ++b) {
        r2[b] = fmaf(dx[b], dx[b], fmaf(dy[b], dy[b], dz[b] * dz[b]));
        rs[b] = r2[b] + C.eps2;
        g[b] = C.c_exp * r2[b];
    }
    burst_begin();
#pragma unroll
    for (int b = 0; b < B; ++b) {
        rs[b] = __builtin_amdgcn_rsqf(rs[b]);
        ri[b] = __builtin_amdgcn_rsqf(r2[b]);  // +inf at r = 0: not selected
        g[b] = __builtin_amdgcn_exp2f(g[b]);
    }
    burst_end();
#pragma unroll
    for (int b = 0; b < B; ++b) {
        r[b] = r2[b] * ri[b];
        t[b] = fmaf(C.c_t, r[b], C.one);
    }
}

// w (and psi) of one pair from its roots, t = 1 / (1 + 0.3275911 u).
template <bool PHI>
__device__ __forceinline__ float ewald_fx_weight(const EwaldFxRegs &C, float phi0, float r2,
                                                 float rs, float ri, float r, float g, float t,
                                                 float &psi)
{
    const float p = fmaf(t, fmaf(t, fmaf(t, fmaf(t, C.k4, C.k3), C.k2), C.k1), C.k0);
    const float P = fmaf(-g, fmaf(t, p, C.c_g * r), C.one);
    const bool nz = r2 > 0.0f;
    if constexpr (PHI) {
        const float erf_u = fmaf(-t * p, g, C.one);
        psi = select_value(nz, fmaf(-erf_u, ri, rs), phi0);
    }
    return select_value(nz, fmaf(-P, ri * (ri * ri), rs * (rs * rs)), 0.0f);
}

// Whether source chunk c of an item holds its targets (a piece of a diagonal part):
// each lane then meets its own particle in the chunk's first step.
__device__ __forceinline__ bool own_chunk(const WorkItem &w, int c)
{
    return w.j0 + (int64_t)c * 64 == w.i0;
}

template <int R, bool REACT, bool PHI>
__device__ __forceinline__ void ewald_chunk_fx(bool own, uint32_t sx, uint32_t sy, uint32_t sz,
                                               float sm, float &qx, float &qy, float &qz,
                                               float &qp, const uint32_t (&xi)[R],
                                               const uint32_t (&yi)[R], const uint32_t (&zi)[R],
                                               const float (&mi)[R], const EwaldFx &E,
                                               float (&ax)[R], float (&ay)[R], float (&az)[R],
                                               float (&ap)[R])
{
    constexpr int U = R == 1 && !REACT ? 4 : 1;
    constexpr int B = U * R;
    const EwaldFxRegs C = ewald_fx_regs(E);
    sm = wave_rotate_back(sm);
#pragma unroll 1
    for (int k = 0; k < 64; k += U) {
        float dx[B], dy[B], dz[B], r2[B], rs[B], ri[B], r[B], g[B], t[B], su[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int b = u * R + q;
                dx[b] = (float)(int32_t)(sx - xi[q]);
                dy[b] = (float)(int32_t)(sy - yi[q]);
                dz[b] = (float)(int32_t)(sz - zi[q]);
            }
            if (u + 1 < U) {
                sx = wave_rotate_u(sx);
                sy = wave_rotate_u(sy);
                sz = wave_rotate_u(sz);
            }
        }
        ewald_fx_roots<B>(C, dx, dy, dz, r2, rs, ri, r, g, t);
        burst_begin();
#pragma unroll
        for (int b = 0; b < B; ++b)
            t[b] = __builtin_amdgcn_rcpf(t[b]);
        phase_mark();
        sx = wave_rotate_u(sx);
        sy = wave_rotate_u(sy);
        sz = wave_rotate_u(sz);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sm = wave_rotate(sm);
            su[u] = sm;
        }
        if constexpr (REACT) {
            qx = wave_rotate(qx);
            qy = wave_rotate(qy);
            qz = wave_rotate(qz);
            if constexpr (PHI)
                qp = wave_rotate(qp);
        }
        burst_end();
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int b = u * R + q;
                float psi = 0.0f;
                const float phi0 = !REACT && own && k + u == 0 ? E.phi_self : E.phi_same;
                const float w = ewald_fx_weight<PHI>(C, phi0, r2[b], rs[b], ri[b], r[b], g[b], t[b],
                                                     psi);
                const float wt = su[u] * w;
                ax[q] = fmaf(wt, dx[b], ax[q]);
                ay[q] = fmaf(wt, dy[b], ay[q]);
                az[q] = fmaf(wt, dz[b], az[q]);
                if constexpr (PHI)
                    ap[q] = fmaf(su[u], psi, ap[q]);
                if constexpr (REACT) {
                    // the opposite sign until the end, as in sym_chunk
                    const float ws = mi[q] * w;
                    qx = fmaf(ws, dx[b], qx);
                    qy = fmaf(ws, dy[b], qy);
                    qz = fmaf(ws, dz[b], qz);
                    if constexpr (PHI)
                        qp = fmaf(mi[q], psi, qp);
                }
            }
        }
        phase_mark();
    }
    if constexpr (REACT) {
        qx = -wave_rotate(qx);
        qy = -wave_rotate(qy);
        qz = -wave_rotate(qz);
        if constexpr (PHI)
            qp = wave_rotate(qp);
    }
}

// A reaction piece (kind 2, FP32 pairs): the reactions of 64 sources, one per
// lane, from a part's targets, four per lane, which travel the other way
// around the wave.  A source meets the targets in the order in which a
// travelling source of a pair item does, so its sum has the same bits.
template <bool PHI>
__device__ __forceinline__ void ewald_react_fx(const WorkItem &w, const double *__restrict__ X,
                                               const double *__restrict__ Y,
                                               const double *__restrict__ Z,
                                               const double *__restrict__ m, int64_t N,
                                               float *__restrict__ part,
                                               float *__restrict__ part_phi, const double sc,
                                               const EwaldFx &E)
{
    const int lane = threadIdx.x & 63;
    const EwaldFxRegs C = ewald_fx_regs(E);
    const int64_t j = w.j0 + lane;
    const bool jv = j < w.j1;
    const uint32_t sx = jv ? fx_coord(X[j], sc) : 0u, sy = jv ? fx_coord(Y[j], sc) : 0u,
                   sz = jv ? fx_coord(Z[j], sc) : 0u;
    uint32_t xi[4], yi[4], zi[4];
    float mi[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        const bool v = i < w.i1;
        xi[r] = v ? fx_coord(X[i], sc) : 0u;
        yi[r] = v ? fx_coord(Y[i], sc) : 0u;
        zi[r] = v ? fx_coord(Z[i], sc) : 0u;
        // one lane ahead: the masses rotate just before their use
        mi[r] = wave_rotate(v ? (float)m[i] : 0.0f);
    }
    float qx = 0.0f, qy = 0.0f, qz = 0.0f, qp = 0.0f;
#pragma unroll 1
    for (int k = 0; k < 64; ++k) {
        float dx[4], dy[4], dz[4], r2[4], rs[4], ri[4], r[4], g[4], t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dx[q] = (float)(int32_t)(sx - xi[q]);
            dy[q] = (float)(int32_t)(sy - yi[q]);
            dz[q] = (float)(int32_t)(sz - zi[q]);
        }
        ewald_fx_roots<4>(C, dx, dy, dz, r2, rs, ri, r, g, t);
        burst_begin();
#pragma unroll
        for (int q = 0; q < 4; ++q)
            t[q] = __builtin_amdgcn_rcpf(t[q]);
        phase_mark();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            xi[q] = wave_rotate_back_u(xi[q]);
            yi[q] = wave_rotate_back_u(yi[q]);
            zi[q] = wave_rotate_back_u(zi[q]);
            mi[q] = wave_rotate_back(mi[q]);
        }
        burst_end();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float psi = 0.0f;
            const float wq = ewald_fx_weight<PHI>(C, E.phi_same, r2[q], rs[q], ri[q], r[q], g[q],
                                                  t[q], psi);
            const float ws = mi[q] * wq;
            qx = fmaf(ws, dx[q], qx);
            qy = fmaf(ws, dy[q], qy);
            qz = fmaf(ws, dz[q], qz);
            if constexpr (PHI)
                qp = fmaf(mi[q], psi, qp);
        }
        phase_mark();
    }
    if (!jv)
        return;
    const double sf = sc * sc;
    const int64_t rs = (int64_t)w.rslice;
    part[(rs * 3 + 0) * N + j] = (float)(sf * (double)-qx);
    part[(rs * 3 + 1) * N + j] = (float)(sf * (double)-qy);
    part[(rs * 3 + 2) * N + j] = (float)(sf * (double)-qz);
    if constexpr (PHI)
        part_phi[rs * N + j] = (float)(sc * (double)qp);
}

__device__ __forceinline__ EwaldFx ewald_fx(double eps2, double sc, double alpha)
{
    const double a_fx = alpha / sc;  // alpha in fixed-point units
    EwaldFx E;
    E.eps2 = (float)(eps2 * sc * sc);
    E.c_exp = (float)(-a_fx * a_fx * 1.4426950408889634);
    E.c_t = (float)(0.3275911 * a_fx);
    E.c_g = (float)(1.1283791670955126 * a_fx);
    E.phi_self = E.eps2 > 0.0f ? __builtin_amdgcn_rsqf(E.eps2) : 0.0f;
    E.phi_same = E.phi_self - E.c_g;
    return E;
}

template <int R, bool REACT, bool PHI>
__device__ __forceinline__ void ewald_item_fx(const WorkItem &w, const double *__restrict__ X,
                                              const double *__restrict__ Y,
                                              const double *__restrict__ Z,
                                              const double *__restrict__ m, int64_t N,
                                              float *__restrict__ part,
                                              float *__restrict__ part_phi, const double sc,
                                              const EwaldFx &E)
{
    const int lane = threadIdx.x & 63;
    const double sf = sc * sc;  // force sums back to lengths
    uint32_t xi[R], yi[R], zi[R];
    float mi[R], ax[R], ay[R], az[R], ap[R];
    bool valid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        valid[r] = i < w.i1;
        if (valid[r]) {
            xi[r] = fx_coord(X[i], sc);
            yi[r] = fx_coord(Y[i], sc);
            zi[r] = fx_coord(Z[i], sc);
            mi[r] = (float)m[i];
        } else {
            xi[r] = yi[r] = zi[r] = 0u;
            mi[r] = 0.0f;
        }
        ax[r] = ay[r] = az[r] = ap[r] = 0.0f;
    }
    const int n_chunks = (int)((w.j1 - w.j0 + 63) / 64);
    for (int c = 0; c < n_chunks; ++c) {
        const int64_t j = w.j0 + (int64_t)c * 64 + lane;
        const bool jv = j < w.j1;
        uint32_t sx = 0u, sy = 0u, sz = 0u;
        float sm = 0.0f;
        if (jv) {
            sx = fx_coord(X[j], sc);
            sy = fx_coord(Y[j], sc);
            sz = fx_coord(Z[j], sc);
            sm = (float)m[j];
        }
        float qx = 0.0f, qy = 0.0f, qz = 0.0f, qp = 0.0f;
        ewald_chunk_fx<R, REACT, PHI>(own_chunk(w, c), sx, sy, sz, sm, qx, qy, qz, qp, xi, yi, zi,
                                      mi, E, ax, ay, az, ap);
        if constexpr (REACT) {
            if (jv) {
                const int64_t rs = (int64_t)w.rslice;
                part[(rs * 3 + 0) * N + j] = (float)(sf * (double)qx);
                part[(rs * 3 + 1) * N + j] = (float)(sf * (double)qy);
                part[(rs * 3 + 2) * N + j] = (float)(sf * (double)qz);
                if constexpr (PHI)
                    part_phi[rs * N + j] = (float)(sc * (double)qp);
            }
        }
    }
    const int64_t slot = (int64_t)w.slice;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!valid[r])
            continue;
        const int64_t i = w.i0 + (int64_t)(r * 64 + lane);
        part[(slot * 3 + 0) * N + i] = (float)(sf * (double)ax[r]);
        part[(slot * 3 + 1) * N + i] = (float)(sf * (double)ay[r]);
        part[(slot * 3 + 2) * N + i] = (float)(sf * (double)az[r]);
        if constexpr (PHI)
            part_phi[slot * N + i] = (float)(sc * (double)ap[r]);
    }
}

template <bool PHI>
__global__ __launch_bounds__(64) void ewald_real_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const WorkItem *__restrict__ items, int n_items, float *__restrict__ part,
    float *__restrict__ part_phi, int64_t *__restrict__ step_inc, double L, double alpha)
{
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    if (step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *step_inc += 1;
    const int it = (int)blockIdx.x;
    if (it >= n_items)
        return;
    const WorkItem w = items[it];
    const double sc = 4294967296.0 / L;  // fixed-point units per length
    const EwaldFx E = ewald_fx(w.eps2, sc, alpha);
    if (w.kind == 0)
        ewald_item_fx<4, true, PHI>(w, X, Y, Z, m, N, part, part_phi, sc, E);
    else if (w.kind == 1)
        ewald_item_fx<1, false, PHI>(w, X, Y, Z, m, N, part, part_phi, sc, E);
    else
        ewald_react_fx<PHI>(w, X, Y, Z, m, N, part, part_phi, sc, E);
}

template <bool PHI>
__global__ __launch_bounds__(64) void ewald_real64_kernel(
    const double *__restrict__ x, const double *__restrict__ m, int64_t N,
    const WorkItem *__restrict__ items, int n_items, double *__restrict__ part,
    double *__restrict__ part_phi, int64_t *__restrict__ step_inc, EwaldReal E)
{
    const double *X = x, *Y = x + N, *Z = x + 2 * N;
    if (step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *step_inc += 1;
    constexpr int kPoly = 2 * kWindowDegree + 3;
    __shared__ alignas(16) double spoly[kPoly];
    const int it = (int)blockIdx.x;
    if (it >= n_items)
        return;
    if ((int)threadIdx.x < kPoly)
        spoly[threadIdx.x] = E.poly[threadIdx.x];
    __syncthreads();
    WorkItem w = items[it];
    if (w.kind == 0) {
        ewald_item<4, true, PHI>(w, X, Y, Z, m, N, part, part_phi, E, spoly);
        return;
    }
    if (w.kind == 2) {
        // the other side of a pair: its sources as targets
        const int64_t i0 = w.i0, i1 = w.i1;
        w.i0 = w.j0;
        w.i1 = w.j1;
        w.j0 = i0;
        w.j1 = i1;
        w.slice = w.rslice;
    }
    ewald_item<1, false, PHI>(w, X, Y, Z, m, N, part, part_phi, E, spoly);
}

}  // namespace

hipError_t launch_zero_counter(int *counter, hipStream_t stream)
{
    hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, stream, counter);
    return hipGetLastError();
}

hipError_t launch_pair_sweep(int precision, int form, const TileCfg &cfg, bool with_phi,
                             bool mask_self, const double *x, const double *m, int64_t N,
                             const WorkItem *items, int n_items, int *counter, bool persistent,
                             const double *box_mass, double *part, double *part_phi,
                             int64_t *step_inc, hipStream_t stream)
{
    if (n_items <= 0)
        return hipSuccess;
    const FwdArgs a{x, m, N, items, n_items, counter, persistent, box_mass, part, part_phi,
                    step_inc, stream};
    switch (precision) {
    case kFP64:
        if (form == 2)
            return dispatch_sym<double, kDirect>(cfg, with_phi, mask_self, a);
        return dispatch_fwd_shape<double, kDirect, 0>(cfg, with_phi, mask_self, a);
    case kMixedTwoSum:
        return dispatch_fwd_form<float, kTwoSum>(form, cfg, with_phi, mask_self, a);
    case kMixedF64Acc:
        return dispatch_fwd_form<float, kFold64>(form, cfg, with_phi, mask_self, a);
    case kFP32:
        return dispatch_fwd_form<float, kDirect>(form, cfg, with_phi, mask_self, a);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_ewald_real(int precision, bool with_phi, const double *x, const double *m,
                             int64_t N, const WorkItem *items, int n_items, double *part,
                             double *part_phi, int64_t *step_inc, double L, double alpha,
                             const double *poly, hipStream_t stream)
{
    if (n_items <= 0)
        return hipSuccess;
    const dim3 grid((unsigned)n_items), block(64);
    if (precision == kFP64) {
        const double rc = 0.5 * L;
        const EwaldReal E{L, 1.0 / L, rc * rc, -2.0 / (rc * rc), poly};
        if (with_phi)
            hipLaunchKernelGGL(ewald_real64_kernel<true>, grid, block, 0, stream, x, m, N, items,
                               n_items, part, part_phi, step_inc, E);
        else
            hipLaunchKernelGGL(ewald_real64_kernel<false>, grid, block, 0, stream, x, m, N, items,
                               n_items, part, part_phi, step_inc, E);
        return hipGetLastError();
    }
    float *pf = reinterpret_cast<float *>(part), *pp = reinterpret_cast<float *>(part_phi);
    if (with_phi)
        hipLaunchKernelGGL(ewald_real_kernel<true>, grid, block, 0, stream, x, m, N, items,
                           n_items, pf, pp, step_inc, L, alpha);
    else
        hipLaunchKernelGGL(ewald_real_kernel<false>, grid, block, 0, stream, x, m, N, items,
                           n_items, pf, pp, step_inc, L, alpha);
    return hipGetLastError();
}

// box_mass[b] = the common mass of box b, or NaN if its masses differ (or one
// is not positive).  A block per box compares a box's masses with its first;
// boxes too large (kMassBlock) or too many (kMassBoxes) for that take two passes
// over the whole grid: every box takes its first mass, then every particle whose
// mass differs marks the box NaN.  Those marks all store the same value, so the
// result does not depend on their order.  One launch against two: a cached step
// of 5000 particles 36 -> 33 us, forces of 5000 24.3 -> 23.7, but of 8000 34.1 ->
// 34.3 and of 32000 179 -> 182 (one block's loads take longer than a launch); the
// kernels alone, 2000 boxes of 200 7.6 / 9.6 us, 10 000 boxes of 30 29 / 9.4,
// 100 000 of 10 268 / 18 (a block of 1024 is mostly idle there).
constexpr int64_t kMassBlock = 6144;
constexpr int kMassBoxes = 2048;

__global__ __launch_bounds__(1024) void box_mass_kernel(const double *__restrict__ m,
                                                        const int64_t *__restrict__ off,
                                                        double *__restrict__ box_mass)
{
    const int64_t o0 = off[blockIdx.x], o1 = off[blockIdx.x + 1];
    const double m0 = m[o0];
    int differ = !(m0 > 0.0);
#pragma unroll 8
    for (int64_t i = o0 + threadIdx.x; i < o1; i += 1024)
        differ |= m[i] != m0;
    differ = __syncthreads_or(differ);
    if (threadIdx.x == 0)
        box_mass[blockIdx.x] = differ ? NAN : m0;
}

__global__ void box_mass_seed_kernel(const double *__restrict__ m,
                                     const int64_t *__restrict__ off, int n_boxes,
                                     double *__restrict__ box_mass)
{
    const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (b >= n_boxes)
        return;
    const double m0 = m[off[b]];
    box_mass[b] = m0 > 0.0 ? m0 : NAN;
}

__global__ void box_mass_check_kernel(const double *__restrict__ m,
                                      const int64_t *__restrict__ off, int n_boxes, int64_t N,
                                      double *__restrict__ box_mass)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    // the box holding particle i: the last b with off[b] <= i
    int lo = 0, hi = n_boxes - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    const double mi = m[i];
    if (mi != m[off[lo]] || !(mi > 0.0))
        box_mass[lo] = NAN;
}

hipError_t launch_box_mass(const double *m, const int64_t *box_offsets, int n_boxes, int64_t N,
                           int64_t max_n, double *box_mass, hipStream_t stream)
{
    if (n_boxes < 1 || N < 1)
        return hipErrorInvalidValue;
    if (max_n <= kMassBlock && n_boxes <= kMassBoxes) {
        hipLaunchKernelGGL(box_mass_kernel, dim3((unsigned)n_boxes), dim3(1024), 0, stream, m,
                           box_offsets, box_mass);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(box_mass_seed_kernel, dim3((unsigned)((n_boxes + 63) / 64)), dim3(64), 0,
                       stream, m, box_offsets, n_boxes, box_mass);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(box_mass_check_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0,
                       stream, m, box_offsets, n_boxes, N, box_mass);
    return hipGetLastError();
}

hipError_t launch_adjoint_sweep(int precision, const TileCfg &cfg, bool mask_self,
                                const double *x, const double *m, int64_t N, int n_cot,
                                const double *lam, const WorkItem *items, int n_items,
                                int *counter, bool persistent, const double *box_mass,
                                double *part, hipStream_t stream)
{
    if (n_items <= 0)
        return hipSuccess;
    if (cfg.form == 3)
        return precision == kFP64 && cfg.R * cfg.tpb == 64
                   ? launch_adjoint_matrix(mask_self, x, m, N, n_cot, lam, items, n_items, part,
                                           stream)
                   : hipErrorInvalidValue;
    switch (precision) {
    case kFP64:
        return dispatch_adj<double, kDirect>(cfg, mask_self, x, m, N, n_cot, lam, items,
                                             n_items, counter, persistent, box_mass, part, stream);
    case kMixedTwoSum:
        return dispatch_adj<float, kTwoSum>(cfg, mask_self, x, m, N, n_cot, lam, items,
                                            n_items, counter, persistent, box_mass, part, stream);
    case kMixedF64Acc:
        return dispatch_adj<float, kFold64>(cfg, mask_self, x, m, N, n_cot, lam, items,
                                            n_items, counter, persistent, box_mass, part, stream);
    case kFP32:
        return dispatch_adj<float, kDirect>(cfg, mask_self, x, m, N, n_cot, lam, items,
                                            n_items, counter, persistent, box_mass, part, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace colatus
