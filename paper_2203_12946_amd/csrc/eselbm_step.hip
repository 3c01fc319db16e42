// The step's dispatch (by storage type and lane mapping; the kernel is in
// step_kernel.hpp), the equilibrium initialiser, and the double-precision
// diagnostics (moments, H function, the statistics' reset).
#include "step_kernel.hpp"

namespace eselbm {

// Lanes along rows, or (flat) through whole planes.  Rows are addressed by
// scalars; a row of partial waves, or of a short last block, wastes lanes, and
// its stores leave partial lines.  256-lane blocks whatever the row also keep
// the FP64 D3Q27 step at its three waves per SIMD (its 48 KiB of parked values
// belong to a block).  Rows against planes, per step, periodic:
//   D3Q27 F32:  250x120x130 223 / 159 us, 300x128x100 252 / 149, 320x128x100
//               205 / 165, 100x90x110 74 / 63; 256^3 627 / 621, 128^3
//               107.5 / 110, 64^3 13.5 / 14.1; 32^3 5.7 / 6.1;
//   D3Q27 FP64: 48^3 27.9 / 13.0, 64^3 59 / 35, 128^3 267 / 222, 192^3 573 /
//               568, 250x120x130 411 / 341; 16^3 6.8 / 7.2;
//   D2Q9:       1500^2 66 / 63 (FP64), 33.5 / 30.9 (F32); 256^2 5.6 / 5.7,
//               3.9 / 4.2; 1024^2 34.5 / 36.6, 16.7 / 16.6.
//   cavities, D3Q27 F32: 192^3 308 / 288, 64^3 26.7 / 24.3, 128^3 101 / 110;
//   rows of 192 cells, D3Q27: 192^3 F32 286 / 278, F32-shifted 291 / 283,
//               F16-shifted 158 / 159, ES-BGK F32 445 / 404, cavity F32-shifted
//               324 / 306; 192x48x48 F32 23.9 / 23.8; in place F32 306 / 307,
//               F32-shifted 310 / 313;
//   cavities with rows of 64: 64x200x100 F32 62.7 / 61.3, 64^3 F16-shifted
//               17.9 / 17.0, F32-shifted 19.8 / 19.6, 64x40x40 F32 13.0 / 13.0.
// So planes where rows are ragged and the grid is beyond the smallest (whose
// step is latency), in D3Q27 also for rows of three waves (192 cells; not in
// place, and not the periodic F16-shifted step) and the walled step's rows of
// one, and for the FP64 D3Q27 step below 256 cells a row.
static bool use_flat(int dtype, int D, const StepArgs &a)
{
    if ((long long)a.nx * a.ny > kMaxFlatPlane) return false;
    const bool ragged = a.nx % 64 != 0 || (a.nx > 256 && a.nx % 256 != 0);
    if (D == 2) return ragged && a.N >= 1 << 18;
    if (dtype == 0) return (ragged || a.nx < 256) && a.N >= 1 << 15;
    const bool three = a.nx == 192 && a.aa == 0 && (dtype != 2 || a.walls || a.cpr != 0.0);
    return (ragged || three || (a.walls && a.nx == 64)) && a.N >= 1 << 16;
}

hipError_t launch_step(int dtype, int D, int mode, bool diag, const StepArgs &a, hipStream_t s)
{
    if (use_flat(dtype, D, a)) {
        switch (dtype) {
        case 0: return launch_step_flat_f64(D, mode, diag, a, s);
        case 1: return launch_step_flat_f32(D, mode, diag, a, s);
        case 2: return launch_step_flat_f16s(D, mode, diag, a, s);
        case 3: return launch_step_flat_f32s(D, mode, diag, a, s);
        }
        return hipErrorInvalidValue;
    }
    switch (dtype) {
    case 0: return launch_step_f64(D, mode, diag, a, s);
    case 1: return launch_step_f32(D, mode, diag, a, s);
    case 2: return launch_step_f16s(D, mode, diag, a, s);
    case 3: return launch_step_f32s(D, mode, diag, a, s);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Statistics reset (a fill kernel rather than a memset, so that the step
// sequence stays capturable in a graph).
// ---------------------------------------------------------------------------
__global__ void k_reset_stats(DevStats *st)
{
    const int k = threadIdx.x;
    if (k < kStatSlots) {
        DevStats z{};
        z.alpha_min_bits = 0x7FF0000000000000ull;
        z.alpha_max_bits = 0;
        st[k] = z;
    }
}

hipError_t launch_reset_stats(DevStats *st, hipStream_t s)
{
    hipLaunchKernelGGL(k_reset_stats, dim3(1), dim3(64), 0, s, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Equilibrium initial state from double rho, u fields.
// ---------------------------------------------------------------------------
template <int D, typename S>
__global__ __launch_bounds__(256) void k_init_eq(Grid g, const double *__restrict__ rho,
                                                 const double *__restrict__ u, S *__restrict__ f)
{
    using T = typename Storage<S>::T;
    constexpr int Q = Lat<D>::Q;
    const long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= g.N) return;
    const T drho = (T)(rho[cell] - 1.0);
    T uu[3] = {(T)u[cell], (T)u[g.N + cell], D == 3 ? (T)u[2 * g.N + cell] : T(0)};
    T feqt[Q];
    equilibrium_shifted<D, T>(drho, uu, feqt);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T w = T(Lat<D>::w(i));
        f[(long long)i * g.N + cell] = Storage<S>::from_T(Storage<S>::kShifted ? feqt[i] : w + feqt[i]);
    }
}

template <int D>
static hipError_t launch_init_eq_d(int dtype, const Grid &g, const double *rho, const double *u, void *f,
                                   hipStream_t s)
{
    const dim3 grid((unsigned)((g.N + 255) / 256)), block(256);
    switch (dtype) {
    case 0: hipLaunchKernelGGL((k_init_eq<D, double>), grid, block, 0, s, g, rho, u, (double *)f); break;
    case 1: hipLaunchKernelGGL((k_init_eq<D, float>), grid, block, 0, s, g, rho, u, (float *)f); break;
    case 2: hipLaunchKernelGGL((k_init_eq<D, _Float16>), grid, block, 0, s, g, rho, u, (_Float16 *)f); break;
    case 3: hipLaunchKernelGGL((k_init_eq<D, f32s>), grid, block, 0, s, g, rho, u, (f32s *)f); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_init_eq(int dtype, const Grid &g, const double *rho, const double *u, void *f,
                          hipStream_t s)
{
    return g.D == 2 ? launch_init_eq_d<2>(dtype, g, rho, u, f, s) : launch_init_eq_d<3>(dtype, g, rho, u, f, s);
}

// ---------------------------------------------------------------------------
// Density and velocity in double (diagnostics, parity).
// ---------------------------------------------------------------------------
template <int D, typename S>
__global__ __launch_bounds__(256) void k_moments(Grid g, const S *__restrict__ f, const float *__restrict__ force,
                                                 double *__restrict__ rho, double *__restrict__ u)
{
    constexpr int Q = Lat<D>::Q;
    const long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= g.N) return;
    double dr = 0.0, j[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double w = Lat<D>::w(i);
        const double v = Storage<S>::full(f[(long long)i * g.N + cell], w) - w;
        dr += v;
#pragma unroll
        for (int c = 0; c < D; ++c) j[c] += Lat<D>::c(i, c) * v;
    }
    const double r = 1.0 + dr;
    rho[cell] = r;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        double jc = j[c];
        if (force) jc += 0.5 * (double)force[(long long)c * g.N + cell];
        u[(long long)c * g.N + cell] = jc / r;
    }
}

template <int D>
static hipError_t launch_moments_d(int dtype, const Grid &g, const void *f, const float *force, double *rho,
                                   double *u, hipStream_t s)
{
    const dim3 grid((unsigned)((g.N + 255) / 256)), block(256);
    switch (dtype) {
    case 0: hipLaunchKernelGGL((k_moments<D, double>), grid, block, 0, s, g, (const double *)f, force, rho, u); break;
    case 1: hipLaunchKernelGGL((k_moments<D, float>), grid, block, 0, s, g, (const float *)f, force, rho, u); break;
    case 2: hipLaunchKernelGGL((k_moments<D, _Float16>), grid, block, 0, s, g, (const _Float16 *)f, force, rho, u); break;
    case 3: hipLaunchKernelGGL((k_moments<D, f32s>), grid, block, 0, s, g, (const f32s *)f, force, rho, u); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_moments(int dtype, const Grid &g, const void *f, const float *force, double *rho, double *u,
                          hipStream_t s)
{
    return g.D == 2 ? launch_moments_d<2>(dtype, g, f, force, rho, u, s)
                    : launch_moments_d<3>(dtype, g, f, force, rho, u, s);
}

// ---------------------------------------------------------------------------
// H function sum_x <f, log(f/w) - 1> (Eq. hdef), double precision.
// ---------------------------------------------------------------------------
// The terms v (log(v / w) - 1) of one cell.  log(v/w) = 2 atanh(z),
// z = (v - w) / (v + w), by its series to z^41 where every |z| of the wave is
// below 0.38 (v between 0.45 and 2.2 of w; remainder below 1e-18 of the
// logarithm), else the logarithm.  The test is in single precision and the
// values are read afresh (empty asm), so that no Q-array of doubles is live.
template <int D, typename S>
__device__ inline double H_cell(const S (&f)[Lat<D>::Q])
{
    using T = typename Storage<S>::T;
    constexpr int Q = Lat<D>::Q;
    constexpr bool SH = Storage<S>::kShifted;
    double h = 0.0;
    bool near = true;
    auto full = [&](int i) {
        T t = Storage<S>::to_T(f[i]);
        asm volatile("" : "+v"(t));
        return SH ? Lat<D>::w(i) + (double)t : (double)t;
    };
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        // |z| <= 0.375 as bounds on v: false for a non-positive, infinite or NaN
        // population, and for a double beyond the range of float
        const float w = (float)Lat<D>::w(i), t = (float)Storage<S>::to_T(f[i]), v = SH ? w + t : t;
        near = near && v >= float(5.0 / 11.0) * w && v <= 2.2f * w;
    }
    if (__ballot(!near) == 0ull) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double w = Lat<D>::w(i), v = full(i);
            const double z = (v - w) * rcp_(v + w), z2 = z * z;
            double s = 1.0 / 41.0;
#pragma unroll
            for (int k = 39; k >= 1; k -= 2) s = fma_(s, z2, 1.0 / k);
            h += v * fma_(2.0 * z, s, -1.0);
            asm volatile("" : "+v"(h));
            if (i % 3 == 2) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double v = full(i);
            h += v * (log(v / Lat<D>::w(i)) - 1.0);
            asm volatile("" : "+v"(h));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return h;
}

// A bounded grid strides over the cells, one atomic per block.  Bound by FP64
// issue; 128^3 with a logarithm and a division per population at two waves per
// SIMD: F32 194 us, F16-shifted 193; with the series at seven: 83 and 81.
constexpr unsigned kHBlocks = 4096;
template <int D, typename S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_H(Grid g, const S *__restrict__ f, DevStats *st)
{
    constexpr int Q = Lat<D>::Q;
    __shared__ double part[4];
    double h = 0.0;
    for (long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x; cell < g.N; cell += (long long)gridDim.x * blockDim.x) {
        S v[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = f[(long long)i * g.N + cell];
        h += H_cell<D, S>(v);
    }
    h = wave_sum(h);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) t += part[w];
        atomicAdd(&st[blockIdx.x % kStatSlots].H, t);
    }
}

__global__ void k_zero_H(DevStats *st)
{
    if (threadIdx.x < kStatSlots) st[threadIdx.x].H = 0.0;
}

template <int D>
static hipError_t launch_H_d(int dtype, const Grid &g, const void *f, DevStats *st, bool zero, hipStream_t s)
{
    const long long blocks = (g.N + 255) / 256;
    const dim3 grid(blocks < kHBlocks ? (unsigned)blocks : kHBlocks), block(256);
    if (zero) hipLaunchKernelGGL(k_zero_H, dim3(1), dim3(64), 0, s, st);
    switch (dtype) {
    case 0: hipLaunchKernelGGL((k_H<D, double>), grid, block, 0, s, g, (const double *)f, st); break;
    case 1: hipLaunchKernelGGL((k_H<D, float>), grid, block, 0, s, g, (const float *)f, st); break;
    case 2: hipLaunchKernelGGL((k_H<D, _Float16>), grid, block, 0, s, g, (const _Float16 *)f, st); break;
    case 3: hipLaunchKernelGGL((k_H<D, f32s>), grid, block, 0, s, g, (const f32s *)f, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_H(int dtype, const Grid &g, const void *f, DevStats *st, bool zero, hipStream_t s)
{
    return g.D == 2 ? launch_H_d<2>(dtype, g, f, st, zero, s) : launch_H_d<3>(dtype, g, f, st, zero, s);
}

}  // namespace eselbm
