// Forward sweep of small boxes (form 4): one launch, no partial sums in memory.
//
// A block owns a few targets (kSmallT32, kSmallT64) and meets every source of
// their box, so that their sums are finished inside it and can be turned at
// once into accelerations, potentials and the closing kick of a step.  The
// general ordered sweep (a block per target tile and source slice, partial sums
// in memory, masses compared and slices added by kernels of their own) is four
// launches, and calls of a few thousand particles wait for the host to make
// them: forces of 1000 particles 20.5 -> 10.5 us a call, of 4096 20.6 -> 11.9
// (FP32 pairs) and 22.8 -> 16.1 (FP64), a cached step of 4096 36 -> 21 us.  A
// run takes one launch a step instead of two: 1000 particles 13.5 -> 11 us a
// step (FP64 14.9 -> 7.3), 4096 16.8 -> 13.1 (21.8 -> 16.7).
// So does the forward pass of an adjoint that keeps every position: five steps
// and their gradient, 1000 particles, FP32 pairs 323 -> 290 us.
//
// FP32 pairs keep the ordered sweep's bits: coordinates relative to the centre
// of the same tile of targets, one FP32 sum per tile of sources in order, the
// tiles' sums added in FP64 in the same order.  A lane is a target and a tile;
// a wave stages four tiles of sources in LDS, one for each of its rows of 16
// lanes, and the block meets only to add the tiles' sums.  With one or two
// waves a SIMD the loop waits on latencies: sources are read from LDS a group
// of eight ahead (11.4 -> 10.2 us at N = 1000 against four not ahead).  Four
// lanes sharing a target instead, a quarter of the pairs each and the ordered
// sum passed through DPP, took 9 us there but 20 at N = 4096 (14.0 so): the DPP
// moves and the transposed LDS reads cost more than the added waves gain.
//
// FP64 pairs: the lanes of a block hold different sources, loaded once
// straight to registers, and every lane meets the block's eight targets; the
// lanes' sums are added in a fixed order.  Bound by FP64 issue: 18 operations a
// pair, 8.8 of its 14.8 us at N = 4096.
#include "colatus_internal.h"
#include "device_math.h"

#include <math.h>

namespace colatus {
namespace {

// What a block does with its targets' finished sums.
__device__ __forceinline__ void small_finish(const SmallArgs &A, const WorkItem &w, int64_t i,
                                             double mbox, const double (&g)[3], double ph)
{
    const int64_t N = A.N;
    if (A.mode == kSmallSums) {
        for (int c = 0; c < 3; ++c)
            A.part[(int64_t)c * N + i] = g[c];
        if (A.part_phi)
            A.part_phi[i] = ph;
        return;
    }
    const double eps = A.ext.on || A.phi ? sqrt(w.eps2) : 0.0;
    if (A.mode == kSmallRun) {
        double gg[3], p[3], x[3];
        for (int c = 0; c < 3; ++c) {
            gg[c] = A.G * g[c];
            x[c] = A.x[(int64_t)c * N + i];
            if (A.row == 0) {
                const double a = A.coef[0].a0;
                p[c] = a * a * A.v[(int64_t)c * N + i];
            } else
                p[c] = A.p[(int64_t)c * N + i];
        }
        if (A.ext.on || A.ext.bg)
            (void)ext_pull(A.ext, x[0], x[1], x[2], eps, gg);
        if (A.row > 0) {
            const StepCoef cp = A.coef[A.row - 1];
            const int32_t t = A.track_slot ? A.track_slot[i] : -1;
            double *out = A.track + A.row * 6 * A.n_tracers + t;
            for (int c = 0; c < 3; ++c) {
                p[c] = fma(cp.k2, gg[c], p[c]);
                if (t >= 0) {
                    out[c * A.n_tracers] = x[c];
                    out[(3 + c) * A.n_tracers] = p[c] / (cp.a1 * cp.a1);
                }
                if (A.row == A.n_rows && A.v)
                    A.v[(int64_t)c * N + i] = p[c] / (cp.a1 * cp.a1);
            }
        }
        if (A.row < A.n_rows) {
            const StepCoef cf = A.coef[A.row];
            for (int c = 0; c < 3; ++c) {
                p[c] = fma(cf.k1, gg[c], p[c]);
                x[c] = fma(cf.d, p[c], x[c]);
                A.p[(int64_t)c * N + i] = p[c];
            }
        }
        if (A.x_out)
            for (int c = 0; c < 3; ++c)
                A.x_out[(int64_t)c * N + i] = x[c];
        return;
    }
    double f[3] = {0.0, 0.0, 0.0}, phe = 0.0;
    if (A.ext.on || A.ext.bg)
        phe = ext_pull(A.ext, A.x[i], A.x[N + i], A.x[2 * N + i], eps, f);
    for (int c = 0; c < 3; ++c) {
        const double gc = A.scale * g[c] + A.inv_a3 * f[c];
        A.acc[(int64_t)c * N + i] = gc;
        if (A.kick_v) {
            const StepCoef cf = A.kick_coef[0];
            const double pi = fma(cf.k2, gc, A.kick_p[(int64_t)c * N + i]);
            A.kick_v[(int64_t)c * N + i] = pi / (cf.a1 * cf.a1);
        }
    }
    if (A.phi)
        A.phi[i] = -A.G * (ph - self_potential(A.precision, A.m[i], eps, mbox)) + phe;
}

// The box's common mass, or NaN: from memory, or found here by the block.
__device__ __forceinline__ double small_mass(const SmallArgs &A, const WorkItem &w)
{
    if (A.box_mass)
        return A.box_mass[w.box];
    const double m0 = A.m[w.j0];
    int differ = !(m0 > 0.0);
#pragma unroll 4
    for (int64_t j = w.j0 + threadIdx.x; j < w.j1; j += blockDim.x)
        differ |= A.m[j] != m0;
    return __syncthreads_or(differ) ? NAN : m0;
}

// A tile's sources in order, eight at a time (the next eight on their way from
// LDS: few waves are there to hide the latencies), in the phases of sweep_tile.
template <bool PHI, bool MASK, bool EQM>
__device__ __forceinline__ void small_tile(const float4 *tile, int nt, float xi, float yi, float zi,
                                           float eps2, float &ax, float &ay, float &az, float &ph)
{
    constexpr int U = 8;
    float4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        q[u] = tile[u];
    for (int j = 0; j < nt; j += U) {
        float dx[U], dy[U], dz[U], s[U], y[U], mj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            dx[u] = q[u].x - xi;
            dy[u] = q[u].y - yi;
            dz[u] = q[u].z - zi;
            mj[u] = q[u].w;
            s[u] = fmaf(dx[u], dx[u], eps2);
            s[u] = fmaf(dy[u], dy[u], s[u]);
            s[u] = fmaf(dz[u], dz[u], s[u]);
        }
        const int jn = j + U < nt ? j + U : j;
#pragma unroll
        for (int u = 0; u < U; ++u)
            q[u] = tile[jn + u];
        burst_begin();
#pragma unroll
        for (int u = 0; u < U; ++u)
            y[u] = rsq_raw(s[u]);
        burst_end();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float mr = EQM ? y[u] : mj[u] * y[u];
            float w3 = mr * (y[u] * y[u]);
            if constexpr (MASK) {
                w3 = s[u] > 0.0f ? w3 : 0.0f;
                mr = s[u] > 0.0f ? mr : 0.0f;
            }
            ax = fmaf(w3, dx[u], ax);
            ay = fmaf(w3, dy[u], ay);
            az = fmaf(w3, dz[u], az);
            if constexpr (PHI)
                ph += mr;
        }
    }
}

// A wave takes four tiles at a time, its rows of 16 lanes one tile each, a lane
// one target.
template <bool PHI, bool MASK>
__global__ __launch_bounds__(64 * kSmallWaves) void small_box_kernel(SmallArgs A)
{
    constexpr int kT = kSmallT32, TPB = kSmallTile;
    static_assert(kT == 16, "a row of lanes per tile");
    __shared__ float4 st[kSmallWaves][4][TPB + 1];  // the odd row ends spread the banks
    __shared__ double sp[kSmallTiles][4][kT];       // a tile's sums: x, y, z, potential
    __shared__ double sg[4][4][kT];
    __shared__ double box[2][6];
    if (A.step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *A.step_inc += 1;
    const WorkItem w = A.items[blockIdx.x];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
    const int row = lane >> 4, t = lane & 15;
    const double *X = A.x, *Y = A.x + A.N, *Z = A.x + 2 * A.N;
    const int n_tiles = (int)((w.j1 - w.j0 + TPB - 1) / TPB);
    if (n_tiles > kSmallTiles)
        return;

    // sources of four tiles, eight a lane; the first are on their way meanwhile
    double vx[8], vy[8], vz[8], vm[8];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            int64_t j = w.j0 + (int64_t)t0 * TPB + 64 * r + lane;
            j = j < w.j1 ? j : w.j1 - 1;
            vx[r] = X[j];
            vy[r] = Y[j];
            vz[r] = Z[j];
            vm[r] = A.m[j];
        }
    };
    if (4 * wave < n_tiles)
        fetch(4 * wave);
    // centre of the bounding box of the tile of targets this block is part of
    const int64_t c0 = w.j0 + (w.i0 - w.j0) / TPB * TPB;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (wave < 2) {
        const int64_t k = c0 + 64 * wave + lane;
        if (k < w.j1) {
            const double q[3] = {X[k], Y[k], Z[k]};
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c] = q[c];
                hi[c] = q[c];
            }
        }
    }
    const int64_t i = w.i0 + t, ii = i < w.i1 ? i : w.i0;
    const double tx = X[ii], ty = Y[ii], tz = Z[ii];
    if (wave < 2) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c] = fmin(lo[c], __shfl_xor(lo[c], off, 64));
                hi[c] = fmax(hi[c], __shfl_xor(hi[c], off, 64));
            }
        }
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                box[wave][c] = lo[c];
                box[wave][3 + c] = hi[c];
            }
    }
    const double mbox = small_mass(A, w);
    __syncthreads();
    double cc[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        cc[c] = 0.5 * (fmin(box[0][c], box[1][c]) + fmax(box[0][3 + c], box[1][3 + c]));
    const float xi = (float)(tx - cc[0]), yi = (float)(ty - cc[1]), zi = (float)(tz - cc[2]);
    const float eps2 = (float)w.eps2;
    const bool eqm = !isnan(mbox);
    const double scale = eqm ? mbox : 1.0;

    for (int t0 = 4 * wave; t0 < n_tiles; t0 += 4 * n_waves) {
        const int64_t j0 = w.j0 + (int64_t)t0 * TPB;
        if (t0 != 4 * wave)
            fetch(t0);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            // padding so far away that the pair adds nothing
            const bool in = j0 + 64 * r + lane < w.j1;
            st[wave][r >> 1][(r & 1) * 64 + lane] =
                make_float4(in ? (float)(vx[r] - cc[0]) : 1e30f, in ? (float)(vy[r] - cc[1]) : 1e30f,
                            in ? (float)(vz[r] - cc[2]) : 1e30f, in ? (float)vm[r] : 0.0f);
        }
        wave_lds_fence();
        // the longest of the four tiles is the first
        const int nt = (int)(w.j1 - j0 < TPB ? w.j1 - j0 : TPB);
        float ax = 0.0f, ay = 0.0f, az = 0.0f, ph = 0.0f;
        if (eqm)
            small_tile<PHI, MASK, true>(st[wave][row], nt, xi, yi, zi, eps2, ax, ay, az, ph);
        else
            small_tile<PHI, MASK, false>(st[wave][row], nt, xi, yi, zi, eps2, ax, ay, az, ph);
        const int tile = t0 + row;
        if (tile < n_tiles) {
            sp[tile][0][t] = scale * (double)ax;
            sp[tile][1][t] = scale * (double)ay;
            sp[tile][2][t] = scale * (double)az;
            sp[tile][3][t] = PHI ? scale * (double)ph : 0.0;
        }
        wave_lds_fence();
    }
    __syncthreads();
    // the tiles' sums in the order of the slice sums of the O(N) kernels: four
    // interleaved groups, then the groups
    for (int q = wave; q < 4; q += n_waves) {
        double a = 0.0;
#pragma unroll 4
        for (int k = q; k < n_tiles; k += 4)
            a += sp[k][row][t];
        sg[q][row][t] = a;
    }
    __syncthreads();
    if (tid < kT && w.i0 + tid < w.i1) {
        double g[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            g[c] = ((sg[0][c][tid] + sg[1][c][tid]) + sg[2][c][tid]) + sg[3][c][tid];
        const double g3[3] = {g[0], g[1], g[2]};
        small_finish(A, w, w.i0 + tid, mbox, g3, g[3]);
    }
}

// a summed over the two halves of the wave (or of its rows of 16) into the first,
// b into the second.
template <int H> __device__ __forceinline__ double swap_add(double a, double b)
{
    const uint2 p = __builtin_bit_cast(uint2, a), q = __builtin_bit_cast(uint2, b);
    uint2 lo, hi;
    if constexpr (H == 32) {
        const auto x = __builtin_amdgcn_permlane32_swap(p.x, q.x, false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(p.y, q.y, false, false);
        lo = make_uint2(x[0], y[0]);
        hi = make_uint2(x[1], y[1]);
    } else {
        const auto x = __builtin_amdgcn_permlane16_swap(p.x, q.x, false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(p.y, q.y, false, false);
        lo = make_uint2(x[0], y[0]);
        hi = make_uint2(x[1], y[1]);
    }
    return __builtin_bit_cast(double, lo) + __builtin_bit_cast(double, hi);
}

// The value R lanes on in the row of 16.
template <int R> __device__ __forceinline__ double row_rotate(double v)
{
    const int2 p = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(
        double, make_int2(__builtin_amdgcn_update_dpp(0, p.x, 0x120 + R, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, p.y, 0x120 + R, 0xf, 0xf, true)));
}

// A lane's sources (every 512th, from j on) against the block's targets, FP64;
// the next source is loaded while this one is worked on.
template <int T, bool PHI, bool MASK, bool EQM>
__device__ __forceinline__ void small_loop64(const double *__restrict__ X,
                                             const double *__restrict__ Y,
                                             const double *__restrict__ Z,
                                             const double *__restrict__ M, int64_t j, int64_t j1,
                                             const double (&tx)[T], const double (&ty)[T],
                                             const double (&tz)[T], double eps2,
                                             double (&v)[(PHI ? 4 : 3) * T])
{
    double qx = X[j], qy = Y[j], qz = Z[j], qm = EQM ? 1.0 : M[j];
    for (; j < j1; j += 512) {
        const double px = qx, py = qy, pz = qz, pm = qm;
        const int64_t k = j + 512 < j1 ? j + 512 : j;
        qx = X[k];
        qy = Y[k];
        qz = Z[k];
        if constexpr (!EQM)
            qm = M[k];
        phase_mark();
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const double dx = px - tx[t], dy = py - ty[t], dz = pz - tz[t];
            const double s = fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2)));
            // s^{-3/2} from the estimate y, y^3 (1 - e)^{-3/2} to second order in
            // e = 1 - s y^2 (below 1.2e-7): as many operations as refining y first,
            // and 3e-15 closer
            const double y = rsq_raw(s), y2 = y * y, e = fma(-s, y2, 1.0), y3 = y2 * y;
            const double r3 = fma(y3, e * fma(1.875, e, 1.5), y3);
            double w3 = EQM ? r3 : pm * r3;
            if constexpr (MASK)
                w3 = s > 0.0 ? w3 : 0.0;
            v[t] = fma(w3, dx, v[t]);
            v[T + t] = fma(w3, dy, v[T + t]);
            v[2 * T + t] = fma(w3, dz, v[2 * T + t]);
            if constexpr (PHI) {
                // the self term is subtracted later as rsqrt_refined gives it
                const double rinv = rsqrt_refine(s, y);
                double mr = EQM ? rinv : pm * rinv;
                if constexpr (MASK)
                    mr = s > 0.0 ? mr : 0.0;
                v[3 * T + t] += mr;
            }
            if (t & 1)
                phase_mark();  // two targets' registers at a time
        }
    }
}

template <bool PHI, bool MASK>
__global__ __launch_bounds__(512, 4) void small_box64_kernel(SmallArgs A)
{
    constexpr int T = kSmallT64, V = (PHI ? 4 : 3) * T;
    __shared__ double red[8][V];
    __shared__ double sums[4 * T];
    if (A.step_inc && blockIdx.x == 0 && threadIdx.x == 0)
        *A.step_inc += 1;
    const WorkItem w = A.items[blockIdx.x];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double *X = A.x, *Y = A.x + A.N, *Z = A.x + 2 * A.N;
    // half of the targets' coordinates go through vector registers: all of them
    // in scalar ones would spill
    int none = 0;
    asm("" : "+v"(none));
    double tx[T], ty[T], tz[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int64_t k = w.i0 + t < w.i1 ? w.i0 + t : w.i1 - 1, i = t < T / 2 ? k : k + none;
        tx[t] = X[i];
        ty[t] = Y[i];
        tz[t] = Z[i];
    }
    const double mbox = small_mass(A, w);
    const bool eqm = !isnan(mbox);
    double v[V];
#pragma unroll
    for (int q = 0; q < V; ++q)
        v[q] = 0.0;
    if (w.j0 + tid < w.j1) {
        if (eqm)
            small_loop64<T, PHI, MASK, true>(X, Y, Z, A.m, w.j0 + tid, w.j1, tx, ty, tz, w.eps2, v);
        else
            small_loop64<T, PHI, MASK, false>(X, Y, Z, A.m, w.j0 + tid, w.j1, tx, ty, tz, w.eps2,
                                              v);
    }
    // the lanes' sums: halves of the wave exchange half of the values, then rows
    // of 16, and the 16 lanes left with the same values add them
    double u[V / 4];
#pragma unroll
    for (int q = 0; q < V / 2; ++q)
        v[q] = swap_add<32>(v[q], v[q + V / 2]);
#pragma unroll
    for (int q = 0; q < V / 4; ++q) {
        u[q] = swap_add<16>(v[q], v[q + V / 4]);
        u[q] += row_rotate<8>(u[q]);
        u[q] += row_rotate<4>(u[q]);
        u[q] += row_rotate<2>(u[q]);
        u[q] += row_rotate<1>(u[q]);
    }
    if ((lane & 15) == 0) {
        const int q0 = (lane & 32 ? V / 2 : 0) + (lane & 16 ? V / 4 : 0);
#pragma unroll
        for (int q = 0; q < V / 4; ++q)
            red[wave][q0 + q] = u[q];
    }
    __syncthreads();
    if (tid < V) {
        double a = red[0][tid];
#pragma unroll
        for (int k = 1; k < 8; ++k)
            a += red[k][tid];
        sums[tid] = (eqm ? mbox : 1.0) * a;
    }
    __syncthreads();
    if (tid < T && w.i0 + tid < w.i1) {
        const double g[3] = {sums[tid], sums[T + tid], sums[2 * T + tid]};
        small_finish(A, w, w.i0 + tid, mbox, g, PHI ? sums[3 * T + tid] : 0.0);
    }
}

template <bool PHI, bool MASK>
hipError_t launch_small(int precision, int64_t max_n, int n_items, const SmallArgs &A,
                        hipStream_t s)
{
    const dim3 grid((unsigned)n_items);
    // waves for the largest box's tiles, four at a time
    const int64_t groups = (max_n + 4 * kSmallTile - 1) / (4 * kSmallTile);
    const int waves = (int)(groups < 2 ? 2 : groups < kSmallWaves ? groups : kSmallWaves);
    if (precision == kFP64)
        hipLaunchKernelGGL((small_box64_kernel<PHI, MASK>), grid, dim3(512), 0, s, A);
    else
        hipLaunchKernelGGL((small_box_kernel<PHI, MASK>), grid, dim3(64 * waves), 0, s, A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_small_box(const TileCfg &cfg, bool with_phi, bool mask_self, int64_t max_n,
                            int n_items, const SmallArgs &A, hipStream_t stream)
{
    if (n_items <= 0)
        return hipSuccess;
    const int T = A.precision == kFP64 ? kSmallT64 : kSmallT32;
    if (cfg.form != 4 || cfg.R != T || cfg.tpb != kSmallTile ||
        (A.precision != kFP64 && max_n > (int64_t)kSmallTiles * kSmallTile))
        return hipErrorInvalidValue;
    if (with_phi)
        return mask_self ? launch_small<true, true>(A.precision, max_n, n_items, A, stream)
                         : launch_small<true, false>(A.precision, max_n, n_items, A, stream);
    return mask_self ? launch_small<false, true>(A.precision, max_n, n_items, A, stream)
                     : launch_small<false, false>(A.precision, max_n, n_items, A, stream);
}

}  // namespace colatus
