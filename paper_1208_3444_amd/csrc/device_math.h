// Device functions shared by the kernels: r^-1 and r^-3, the pair loops' phase
// marks, the external terms and the self term of the potential.
#ifndef COLATUS_DEVICE_MATH_H
#define COLATUS_DEVICE_MATH_H

#include "colatus_internal.h"

#include <math.h>

namespace colatus {

// The hardware estimate of s^{-1/2} alone, and the weights made from it: the
// pair loops issue the estimates of several pairs back to back and finish
// them afterwards (see sym_chunk).
__device__ __forceinline__ float rsq_raw(float s) { return __builtin_amdgcn_rsqf(s); }
__device__ __forceinline__ double rsq_raw(double s) { return __builtin_amdgcn_rsq(s); }
__device__ __forceinline__ float rsqrt_from(float, float y) { return y; }
__device__ __forceinline__ double rsqrt_from(double s, double y) { return rsqrt_refine(s, y); }

// s^{-3/2} for FP64 pairs that do not need s^{-1/2} itself: with
// y = v_rsq_f64(s) (relative error below 6e-8) and e = 1 - s y^2,
// s^{-3/2} = y^3 (1 - e)^{-3/2} = y^3 (1 + 3e/2 + O(e^2)).  The first-order
// correction applied to y^3 leaves about (15/8) e^2 < 3e-14 relative, one
// operation fewer than refining y (rsqrt_refine) and cubing it.
__device__ __forceinline__ double rinv3_from(double s, double y)
{
    const double y2 = y * y;
    const double e = fma(-s, y2, 1.0);
    const double y3 = y2 * y;
    return fma(1.5 * e, y3, y3);
}

// The same with one term more, two of (1 - e)^{-1/2} and of (1 - e)^{-3/2} (|e| < 1.2e-7),
// within rounding of exact: the periodic sum's pairs.
__device__ __forceinline__ double rsqrt_exact(double s, double y)
{
    const double e = fma(-s, y * y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double rinv3_exact(double s, double y)
{
    const double y2 = y * y;
    const double e = fma(-s, y2, 1.0);
    const double y3 = y2 * y;
    return fma(y3 * e, fma(1.875, e, 1.5), y3);
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }

// Phase marks of the pair loops.  Gfx950 issues two VALU instructions of two
// waves of a SIMD together (one each, 2.1 cycles per instruction) as long as
// both are in ordinary FP32 arithmetic; a v_rsq_f32 (8 cycles) or a DPP move of
// one wave stops the other's pairing, and spread over the loop they undo it:
// measured on registers alone, 56 FMAs with 4 v_rsq and 6 DPP moves take 265
// cycles, and 173 when the v_rsq and moves are issued back to back at a raised
// wave priority (s_setprio), which lets one wave finish its burst while the
// others wait at theirs and then run their FMAs side by side.  burst_begin /
// burst_end bracket such a run; neither lets the compiler move code across.
__device__ __forceinline__ void phase_mark() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void burst_begin()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
}
__device__ __forceinline__ void burst_end()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
}

// A constant held in a vector register: an FP32 instruction with a scalar or
// literal operand is never paired (4.1 cycles instead of 2.1).
__device__ __forceinline__ float in_vgpr(float c)
{
    asm("" : "+v"(c));
    return c;
}
__device__ __forceinline__ double in_vgpr(double c)
{
    asm("" : "+v"(c));
    return c;
}
// c ? v : other with v computed in every lane (a select, never a branch
// around v's computation).
__device__ __forceinline__ float select_value(bool c, float v, float other)
{
    asm volatile("" : "+v"(v));
    return c ? v : other;
}

// Orders the LDS accesses of a wave's lanes (no instruction is needed: a wave's LDS
// operations complete in order).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The potential sweep includes the self pair j == k, whose term is exactly
// m_k * rsqrt(eps^2) as the sweep computed it (zero separation); subtract
// that same value, rounded the same way, so no FP32-vs-FP64 residue of a
// large self term is left in phi.  Equal-mass boxes (mbox not NaN) were
// summed without m and scaled by mbox in FP64.  With eps == 0 the sweep
// masks the self pair.
__device__ __forceinline__ double self_potential(int precision, double m, double eps,
                                                 double mbox)
{
    if (!(eps > 0.0))
        return 0.0;
    const double eps2 = eps * eps;
    if (precision == kFP64)
        return m * rsqrt_refined(eps2);
    const float r = __builtin_amdgcn_rsqf((float)eps2);
    if (!isnan(mbox))
        return mbox * (double)r;
    return (double)((float)m * r);
}

__device__ __forceinline__ double box_mass_of(const double *box_mass, int box)
{
    return box_mass ? box_mass[box] : NAN;
}

// Eq. (10) attractor at particle position (px, py, pz), softening eps: adds
// its field S d r^-3 (d = x_psi - x, r^2 = |d|^2 + eps^2) to f and returns
// its potential -S / r.  FP64 with IEEE square root and division.
__device__ __forceinline__ double attractor_pull(const ExtField &A, double px, double py,
                                                 double pz, double eps, double (&f)[3])
{
    const double dx = A.x - px, dy = A.y - py, dz = A.z - pz;
    const double s = dx * dx + dy * dy + dz * dz + eps * eps;
    const double r = sqrt(s);
    const double r3 = 1.0 / (s * r);
    f[0] += A.S * dx * r3;
    f[1] += A.S * dy * r3;
    f[2] += A.S * dz * r3;
    return -A.S / r;
}

// Background term of Eq. (6): adds b (x - c) to f and returns its potential
// -b |x - c|^2 / 2.
__device__ __forceinline__ double background_pull(const ExtField &E, double px, double py,
                                                  double pz, double (&f)[3])
{
    const double dx = px - E.cx, dy = py - E.cy, dz = pz - E.cz;
    f[0] += E.b * dx;
    f[1] += E.b * dy;
    f[2] += E.b * dz;
    return -0.5 * E.b * (dx * dx + dy * dy + dz * dz);
}

// Every external term present: field added to f, potential returned.
__device__ __forceinline__ double ext_pull(const ExtField &E, double px, double py, double pz,
                                           double eps, double (&f)[3])
{
    double ph = 0.0;
    if (E.on)
        ph += attractor_pull(E, px, py, pz, eps, f);
    if (E.bg)
        ph += background_pull(E, px, py, pz, f);
    return ph;
}

}  // namespace colatus

#endif
