// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eselbm {

// Diagnostic accumulators.  Several copies ("slots") spread the block-level
// atomics of one step over distinct addresses; the host adds the slots.
struct DevStats {
    double mass, mom[3], kinetic, alpha_sum, H, pad0;
    unsigned long long alpha_min_bits, alpha_max_bits;
    unsigned long long n_cells, n_gated, n_guard, n_nonpos, n_lt2, n_exact;
    unsigned long long n_iter, n_fallback;  // mirror modes
    unsigned long long pad1[14];
};
static_assert(sizeof(DevStats) == 256, "DevStats is two 128-byte lines");
constexpr int kStatSlots = 32;
constexpr int kWallEq = 6 * 27;  // doubles of the wall equilibrium table

struct Grid {
    int D, Q, nx, ny, nz;
    long long N;  // cells
};

// What every step reads comes first, in one 64-byte line: a line more is a
// read more that a small grid's step, a few microseconds long, waits for (per
// step against one reference build: D2Q9 64^2 FP64 1.028 -> 0.993 of its time,
// 128^2 F32 1.056 -> 1.028, D3Q27 22^3 FP64 1.026 -> 1.023).  112 bytes in all,
// and the kernels read no launch dimensions, of which the compiler would append
// 256 bytes: the host's time to enqueue a launch, which bounds the smallest
// grids, steps up between 112 and 120 bytes (a kernel of 64 blocks, 100 launches
// after a synchronisation: 3.1 us a launch up to 112 bytes, 3.7-4.4 from 120,
// 4.1-4.7 with 144 and the dimensions).
struct StepArgs {
    const void *fin;
    void *fout;          // in place: fin, or for the local half a second copy of its output
    int nx, ny, nz;
    unsigned walls : 8;  // bit a: axis a bounded by diffuse walls, else periodic
    unsigned cached : 8; // bit 0: plain stores, else non-temporal ones (cached_stores); bit 1: of the second copy
    unsigned aa : 16;    // 0: two lattices (fin -> fout); in place: 1 the pull half, 2 the local half
    long long N;         // cells
    double beta;
    double inv_nx;       // 1 / nx, for the plane-mapped launches
    const float *force;  // [D][N] or null
    const double *wall_eq;   // [2 D][Q]: feq_i(1, u_wall) - w_i of wall 2 a + side
    double cpr;          // ES-BGK stress factor c_Pr; 0: the equilibrium itself
    void *alpha_out;     // [N] compute type or null
    void *nut_out;       // [N] compute type or null: nu_T of Eq. nuT
    float *uv_out;       // [D + 1][N] or null: u (with the half-force shift) and rho of the output state
    DevStats *stats;     // kStatSlots slots or null
};
static_assert(sizeof(StepArgs) == 112, "at most 112 bytes (above)");

// Launchers (return the hipError_t of the launch).
hipError_t launch_step(int dtype, int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
// the step for one storage type (step_<type>.hip)
hipError_t launch_step_f64(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_f32(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_f16s(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_f32s(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
// the same with the lanes running through whole planes (step_flat_<type>.hip)
hipError_t launch_step_flat_f64(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_flat_f32(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_flat_f16s(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_step_flat_f32s(int D, int mode, bool diag, const StepArgs &a, hipStream_t s);
hipError_t launch_reset_stats(DevStats *st, hipStream_t s);
hipError_t launch_init_eq(int dtype, const Grid &g, const double *rho, const double *u, void *f,
                          hipStream_t s);
hipError_t launch_moments(int dtype, const Grid &g, const void *f, const float *force, double *rho,
                          double *u, hipStream_t s);
// (zero: clears the slots' H first, needed unless a reset is all that ran on them)
hipError_t launch_H(int dtype, const Grid &g, const void *f, DevStats *st, bool zero, hipStream_t s);

struct AdjArgs {
    const void *fn;
    const void *lam_next;
    void *lam_n;
    Grid g;
    double beta;
    const float *force;
    float *force_grad;
    const void *seed;  // compute type [1 + D][N] or null: lam_next_i += s0 + c_i . s
    // or null; else float [D + 1][N], the velocity and density field of the
    // state after the step, whose dissipation-loss seed (weight seed_w) the
    // kernel forms and adds as it would add seed (seed must then be null)
    const float *seed_uv = nullptr;
    double seed_w = 0.0;
};
hipError_t launch_adjoint(int dtype, int mode, const AdjArgs &a, hipStream_t s);
// Scratch of the losses, owned by a handle (so by its device) and grown on
// demand: velocity and density of the state, and one partial sum per block.
struct LossScratch {
    float *u = nullptr;      // [D][N], u = (j + F/2) / rho
    float *rho = nullptr;    // [N]
    double *part = nullptr;  // one partial sum per block
    long long cells = 0, parts = 0;
};
hipError_t free_loss_scratch(LossScratch &sc);
hipError_t launch_kinetic_loss(LossScratch &sc, int dtype, const Grid &g, const void *f, double *loss, void *lam,
                               double scale, hipStream_t s);
// The kinetic loss for callers that cannot allocate: its partial sums in a
// file-scope device array of kNoAllocParts doubles per device (grids of up to
// 256 * kNoAllocParts cells).  noalloc_scratch looks up that array's device
// address on `device`, which must be current, once, and returns it after.
constexpr long long kNoAllocParts = 1 << 16;
constexpr int kMaxDevices = 256;
hipError_t noalloc_scratch(int device, double **out);
hipError_t launch_kinetic_loss_noalloc(double *parts, int dtype, const Grid &g, const void *f, double *loss,
                                       void *lam, double scale, hipStream_t s);
// The dissipation loss from a state f (its velocity and density formed by a
// pass over f), or, with f null, from uv, the [D + 1][N] velocity and
// density field a step wrote (eselbm_set_velocity_field).
hipError_t launch_dissipation_loss(LossScratch &sc, int dtype, const Grid &g, const void *f, const float *uv,
                                   const float *force, double *loss, void *lam, void *seed, double weight,
                                   float *force_grad, hipStream_t s);
hipError_t launch_equilibrium_vjp(int dtype, const Grid &g, const double *rho, const double *u,
                                  const void *lam, double *grad_u, hipStream_t s);

// Cells of a plane that the plane-mapped launches address by a 32-bit byte
// offset (8-byte populations).
constexpr long long kMaxFlatPlane = 1LL << 28;

// Plain stores of a step's output (true), or non-temporal ones, which stream
// past the caches.  Streaming is the faster way out of a grid whose two
// lattices exceed the 256 MB last-level cache, and out of one of some tens of
// MB, whose dirty lines the L2s would write back at the end of the launch.
// Plain stores are faster (per step, streaming / plain; lattices are pairs)
//  - out of the smallest grids, whose stores the end of the launch would wait
//    for: D2Q9 F32 64^2 3.31 / 3.06 us, 256^2 (4.7 MB) 4.36 / 4.12, FP64 192^2
//    4.89 / 4.65, F16-shifted 384^2 4.69 / 4.47; D3Q27 F32 24^3 8.43 / 8.20,
//    F16-shifted 32^3 7.34 / 7.07; beyond the line F16-shifted 36^3 (5.04 MB)
//    10.2 / 10.8, F32 320^2 4.83 / 5.02, 512^2 6.25 / 7.81, FP64 256^2 6.33 / 6.55;
//  - where the two lattices fit the last-level cache, from which the next step
//    then reads, and the step waits for memory.  The line lies where the
//    slowest of a type's steps has reached it:
//    D2Q9   4 bytes: 50 MB F32 12.0 / 11.0 us but F32-shifted 13.4 / 14.0,
//                    58 MB F32 14.1 / 12.8, 231 MB 41.9 / 37.8
//           8 bytes: 59 MB 15.8 / 16.2, 71 MB 18.2 / 16.6, 236 MB 46.6 / 41.6
//           2 bytes: 71 MB 17.7 / 18.9, 85 MB 20.9 / 20.5, 116 MB 25.8 / 26.7,
//                    151 MB 35.9 / 33.6, 236 MB 48.5 / 47.8
//    D3Q27  4 bytes: 57 MB F32 14.1 / 13.3 us but F32-shifted 13.8 / 15.1, 81 MB
//                    20.7 / 17.2 and 20.8 / 19.4, 243 MB 48.4 / 44.0
//           8 bytes: 113 MB 33.5 / 35.1, 161 MB 46.7 / 48.1, 221 MB 60.6 / 60.3
//           2 bytes: 122 MB 38.4 / 39.5, 152 MB 40.1 / 38.6, 227 MB 51.0 / 46.5;
//  - where the populations' fields do not start on cache lines (N elements no
//    multiple of 128 bytes): a wave's row then ends in the middle of a line,
//    which streams out in two partial writes and merges in the L2 (255x253x251
//    F32 979 / 805 us, FP64 1732 / 1558, F16-shifted 558 / 439; 203x97x131 F32
//    141 / 130; 101x99x97 F32 54 / 46); in D2Q9 4- and 2-byte types not between
//    320 MB and 1 GB (F32 302 MB 74.8 / 67.7, 450 MB 85.9 / 90.7, 648 MB 129.5 /
//    132.8, 1152 MB 238 / 226; F16-shifted 576 MB 130 / 134; FP64 604 MB 138 / 128).
// In place the same holds, by the same lines (128^3 F16-shifted 54.8 / 52.3 us,
// 96^3 F32 36.8 / 35.0, 1024^2 FP64 32.1 / 29.1, 101x99x97 F32 46.6 / 42.3,
// 203x97x131 F32 125 / 121), but D2Q9 beyond the last-level cache streams
// (2049x2047 F32 56.7 / 62.4; larger ones within 2% either way).
inline long long lattices_bytes(const Grid &g, int elem) { return 2LL * g.Q * g.N * elem; }
constexpr long long kLastLevelCache = 256LL << 20;
inline bool cached_stores(const Grid &g, int elem, bool in_place)
{
    const long long bytes = lattices_bytes(g, elem);
    if (bytes < 5000000LL) return true;
    const long long line = g.D == 2 ? (elem == 2 ? 80 : elem == 4 ? 55 : 65) : (elem == 2 ? 140 : elem == 4 ? 70 : 210);
    const bool odd = g.N * elem % 128 != 0;
    if (bytes < (odd ? (g.D == 2 ? 55 : 110) : line) * 1000000LL) return false;
    if (bytes <= kLastLevelCache) return true;
    return odd && !(g.D == 2 && (in_place || (elem < 8 && bytes > 320000000LL && bytes < 1000000000LL)));
}

// The second copy of an even count's last step: plain where the lattices fit the
// last-level cache, from which the caller's next step then reads it.  Two steps a
// call, its stores streaming / plain: D2Q9 1024^2 FP64 65.7 / 62.0 us, F32 36.8 /
// 36.1, 512^2 FP64 22.5 / 21.1, D3Q27 64^3 FP64 75.8 / 67.0, 128^3 F16-shifted
// 108.1 / 103.1; beyond it 203x97x131 F32 310 / 340, 2999x3001 F32 339 / 370, 241^3
// FP64 3440 / 3572, 256^3 F32 1698 / 1730 (F16-shifted 241^3 1066 / 997).
inline bool cached_copy(const Grid &g, int elem) { return lattices_bytes(g, elem) <= kLastLevelCache; }

// Block shape along x: 64-lane waves, up to 4 per block, enough to cover nx;
// of a plane-mapped launch.
constexpr unsigned kFlatBlock = 256;
__host__ __device__ inline int block_x(int nx)
{
    int w = (nx + 63) / 64;
    if (w > 4) w = 4;
    return 64 * w;
}

}  // namespace eselbm
