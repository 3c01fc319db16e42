// The fused pull-stream + entropic collision step kernel and its launch
// templates, instantiated once per storage type in step_<type>.hip.
//
// Mapping: one lattice cell per lane.  A block is 64..256 lanes along one
// x-row and the grid (x-blocks, y, z), or 256 lanes through a whole plane and
// the grid (plane blocks, 1, z) (FLAT; use_flat says where).  Each lane pulls
// its Q populations from the neighbouring rows (Eq. advection): a population's
// loads of a wave are consecutive elements of a row (of two or more where a
// plane-mapped wave crosses row ends), shifted by at most one element, so loads
// stay coalesced; the stores are consecutive and unshifted, and start on cache
// lines where the fields do (cached_stores).  Each element of f_in is read
// exactly once over the whole grid, so there is no reuse for LDS or an
// XCD-aware block order to capture.
#pragma once

#include "internal.hpp"
#include "lattice.hpp"
#include "quasi_eq.hpp"

#include <type_traits>

namespace eselbm {

template <typename V>
__device__ inline V wave_sum(V v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// min and max over the wave of the bits of doubles, as unsigned numbers: the
// order of positive doubles, with a NaN beyond them (a floating-point maximum
// would drop it)
__device__ inline unsigned long long wave_min(unsigned long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long t = __shfl_xor(v, o, 64);
        v = t < v ? t : v;
    }
    return v;
}
__device__ inline unsigned long long wave_max(unsigned long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long t = __shfl_xor(v, o, 64);
        v = t > v ? t : v;
    }
    return v;
}

// Per-lane diagnostic contributions, reduced over the block and added to
// one accumulator slot with one atomic per quantity per block.
struct LaneStats {
    double mass = 0, mom[3] = {0, 0, 0}, ke = 0, asum = 0;
    unsigned long long amin = 0x7FF0000000000000ull, amax = 0;  // bits, of the cells that collided
    bool n = false, gated = false, guard = false, nonpos = false, lt2 = false, exact = false, fallback = false;
    int iters = 0;
};

// A lane's counts are zero or one: a ballot and a population count per wave
// take the place of a six-step exchange each (128^3, the step with its
// statistics: F32 94.6 -> 91.4 us, F16-shifted 83 -> 71 us).
template <bool ITER>
__device__ inline void block_reduce_stats(LaneStats &s, DevStats *slot, int nw)
{
    constexpr int NU = 8;  // counters
    __shared__ double red_d[4][6];
    __shared__ unsigned long long red_u[4][NU + 2];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double v[6] = {s.mass, s.mom[0], s.mom[1], s.mom[2], s.ke, s.asum};
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = wave_sum(v[k]);
    const unsigned long long mn = wave_min(s.amin), mx = wave_max(s.amax);
    auto count = [](bool c) { return (unsigned long long)__popcll(__ballot(c)); };
    const unsigned long long c[NU] = {count(s.n), count(s.gated), count(s.guard), count(s.nonpos), count(s.lt2),
                                      count(s.exact), ITER ? (unsigned long long)wave_sum(s.iters) : 0ull,
                                      ITER ? count(s.fallback) : 0ull};
    if (lane == 0) {
        for (int k = 0; k < 6; ++k) red_d[wid][k] = v[k];
        for (int k = 0; k < NU; ++k) red_u[wid][k] = c[k];
        red_u[wid][NU] = mn;
        red_u[wid][NU + 1] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        DevStats *st = slot;
        double t[6] = {0, 0, 0, 0, 0, 0};
        unsigned long long u[NU] = {0, 0, 0, 0, 0, 0, 0, 0};
        unsigned long long tmn = red_u[0][NU], tmx = red_u[0][NU + 1];
        for (int w = 0; w < nw; ++w) {
            for (int k = 0; k < 6; ++k) t[k] += red_d[w][k];
            for (int k = 0; k < NU; ++k) u[k] += red_u[w][k];
            tmn = red_u[w][NU] < tmn ? red_u[w][NU] : tmn;
            tmx = red_u[w][NU + 1] > tmx ? red_u[w][NU + 1] : tmx;
        }
        atomicAdd(&st->mass, t[0]);
        atomicAdd(&st->mom[0], t[1]);
        atomicAdd(&st->mom[1], t[2]);
        atomicAdd(&st->mom[2], t[3]);
        atomicAdd(&st->kinetic, t[4]);
        atomicAdd(&st->alpha_sum, t[5]);
        atomicAdd(&st->n_cells, u[0]);
        if (u[1]) atomicAdd(&st->n_gated, u[1]);
        if (u[2]) atomicAdd(&st->n_guard, u[2]);
        if (u[3]) atomicAdd(&st->n_nonpos, u[3]);
        if (u[4]) atomicAdd(&st->n_lt2, u[4]);
        if (u[5]) atomicAdd(&st->n_exact, u[5]);
        if (u[6]) atomicAdd(&st->n_iter, u[6]);
        if (u[7]) atomicAdd(&st->n_fallback, u[7]);
        atomicMin(&st->alpha_min_bits, tmn);
        atomicMax(&st->alpha_max_bits, tmx);
    }
}

// ---------------------------------------------------------------------------
// The fused step.
// ---------------------------------------------------------------------------
// Per-storage policy: the occupancy floor and the precision of the parts of
// a single-precision step whose rounding would otherwise dominate the
// error.  Measured against the oracle rounded to the storage format after
// every step (the storage floor), on the 64^2, 1024x136 and 3-D parity
// workloads and on a rough near-inviscid state (|x| up to 0.1, beta 0.9998):
//  - moment sums rho, j and the equilibrium deviation d = feq - g: their
//    single-precision rounding is a fixed function of the cell's state, a
//    bias that accumulates over steps.  With F32-shifted storage (f - w in
//    float, a floor 20x lower than plain F32) it reaches 10-30x the floor
//    (2e-6 relative on u after 1000 steps), so both are double there (1-3x
//    the floor); plain F32 stays within 1.0-2.5x of its floor in single
//    precision;
//  - alpha on the exact rational path (cells far from equilibrium): the
//    update multiplies an error of alpha by x relative to g; single-
//    precision sums leave 11x the floor after 5 steps of the rough state,
//    double sums about 1.3x, for both F32 formats;
//  - alpha beta as a two-term sum (F32-shifted): a rounded 2 beta in every
//    gated cell would shift the viscosity of the whole flow by its relative
//    rounding, visible above the shifted floor;
//  - F16-shifted: storage rounding (1e-3 of the deviation) dwarfs all
//    arithmetic rounding, and the power series of the path-length sums is
//    cut at the order that rounding allows (SeriesCfgF16).  It also skips
//    the exact-moment fix of d (conserve_moments): the bias that fix
//    removes, about 1e-8 of w per step, lies far below the unbiased storage
//    rounding of every stored deviation (about 1e-5 of w per step), which
//    conserves mass and momentum only on average anyway, and the step is
//    bound by VALU issue.  For the same reason it drops two register devices
//    that cost it moves (pin_dev false, zeros_in_branch true: 55 fewer VALU
//    instructions per wave); in the other formats those choices leave the
//    registers as they are (F32-shifted spills on its common path without
//    them) or make no measurable difference; F64: every part is double
//    already.
// The kernel is a stream of Q loads and Q stores per lane and needs several
// waves per SIMD in flight to cover HBM latency: 4 waves (<= 128 VGPRs) for
// the 4- and 2-byte formats; the double moments and equilibrium of
// F32-shifted fit there too without scratch on the common path.
//
// Double precision: the Q stored values alone take 54 VGPRs in D3Q27, and
// with d and the path-length sums the step needs about 210, i.e. two waves
// per SIMD, too few to hide the memory latency behind its arithmetic (about
// 1,900 VALU issue slots per wave).  The periodic closed-form steps
// therefore park 24 of the 27 stored values in LDS once the moments are
// formed (stash = 24: 48 KiB per 256-lane block, three blocks per CU) and
// run at three waves (stash_waves): 1.44-1.50 -> 1.38 ms at 256^3.
template <typename S>
struct StepPolicy {
    static constexpr int waves = 4;
    static constexpr bool mom_f64 = false, eq_f64 = false, ab_split = false, conserve = true;
    static constexpr bool pin_dev = true, zeros_in_branch = false;
    static constexpr int stash = 0, stash_waves = 0;
    using Series = SeriesCfg<typename Storage<S>::T>;
    using Exact = double;
};
template <>
struct StepPolicy<f32s> {
    static constexpr int waves = 4;
    static constexpr bool mom_f64 = true, eq_f64 = true, ab_split = true, conserve = true;
    static constexpr bool pin_dev = true, zeros_in_branch = false;
    static constexpr int stash = 0, stash_waves = 0;
    using Series = SeriesCfg<float>;
    using Exact = double;
};
template <>
struct StepPolicy<_Float16> {
    static constexpr int waves = 4;
    static constexpr bool mom_f64 = false, eq_f64 = false, ab_split = false, conserve = false;
    static constexpr bool pin_dev = false, zeros_in_branch = true;
    static constexpr int stash = 0, stash_waves = 0;
    using Series = SeriesCfgF16;
    using Exact = float;
};
template <>
struct StepPolicy<double> {
    static constexpr int waves = 2;
    static constexpr bool mom_f64 = true, eq_f64 = true, ab_split = false, conserve = true;
    static constexpr bool pin_dev = true, zeros_in_branch = false;
    static constexpr int stash = 24, stash_waves = 3;
    using Series = SeriesCfg<double>;
    using Exact = double;
};

// a if A, else b (both by reference)
template <bool A, typename X, typename Y>
__device__ inline const auto &pick(const X &a, const Y &b)
{
    if constexpr (A) return a;
    else return b;
}

// Stored values a step parks in LDS (PopAccess): the policy's count for the
// two-lattice D3Q27 steps, periodic or walled (cavity 256^3 FP64: 1567 us at
// two waves without parking, 1478 parked at three), with a path length; none for
// alpha = 2 (BGK fits two waves' registers and is memory-bound there: parked
// at three waves it measured 2% slower), the in-place halves (parked at
// three waves, 3-5% slower than at two), and the ES-BGK step, which keeps its
// own occupancy.
template <int D, typename S, int MODE, bool WALL, bool QE, int AA>
constexpr int stash_pops()
{
    return (D == 3 && !QE && AA == 0 && (MODE == MODE_HIGHER || MODE == MODE_LOWER || is_mirror_mode(MODE))) ? StepPolicy<S>::stash : 0;
}

// d = feq - g of one cell, with moments and equilibrium in EQ, rounded to T,
// and (CONSERVE) its mass and momentum then made exact to rounding.
// With POLY the equilibrium is the polynomial one of Eq. histeq (the classic
// LBGK mode): feq_i - w_i = w_i (drho + rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2)).
template <int D, typename T, typename EQ, bool POLY, bool CONSERVE, bool PIN, typename Dev>
__device__ inline void form_deviation(Dev dev, EQ drho, const EQ (&j)[3], T (&d)[Lat<D>::Q])
{
    const EQ rho = EQ(1) + drho, ir = rcp_(rho);
    const EQ u[3] = {quot_(j[0], rho, ir), quot_(j[1], rho, ir), D == 3 ? quot_(j[2], rho, ir) : EQ(0)};
    const Equilibrium<D, EQ> eq(drho, u);
    const EQ uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
#pragma unroll
    for (int i = 0; i < Lat<D>::Q; ++i) {
        // the stored deviation is formed again rather than kept live since
        // the moment sums (PIN: the empty asm hides it from
        // common-subexpression elimination and emits nothing; shifted storage
        // holds the deviation itself, which there is nothing to form again,
        // and the asm would only copy it)
        T v = dev(i);
        if constexpr (PIN) asm volatile("" : "+v"(v));
        EQ fe;
        if (POLY) {
            EQ cu = EQ(0);
#pragma unroll
            for (int a = 0; a < D; ++a) cu += EQ(Lat<D>::c(i, a)) * u[a];
            fe = EQ(Lat<D>::w(i)) * (drho + rho * (EQ(3) * cu + EQ(4.5) * cu * cu - EQ(1.5) * uu));
        } else {
            fe = eq.dev(i);
        }
        d[i] = T(fe - EQ(v));
    }
    if constexpr (CONSERVE) conserve_moments<D, T>(d);
}

// The ES-BGK quasi-equilibrium solve holds a K x K factor, its moments and
// the Newton state besides the two Q-arrays: two waves per SIMD for D2Q9 in
// single precision, one for D3Q27 (K = 10) or where the solve runs in double.
template <int D, typename S, int MODE, bool QE>
constexpr int step_waves_qe()
{
    return QE ? ((StepPolicy<S>::eq_f64 || D == 3) ? 1 : 2) : StepPolicy<S>::waves;
}

// The walled step runs the periodic pull in all but the boundary layers, so
// it takes the periodic step's occupancy floor, at most three waves per SIMD
// (the wall node's mass balance adds live values; the closed-form modes then
// still fit four waves in FP32 and F16 without scratch).
template <int D, typename S, int MODE, bool WALL, bool QE, int AA>
constexpr int step_waves_k()
{
    return stash_pops<D, S, MODE, WALL, QE, AA>() > 0 ? StepPolicy<S>::stash_waves
           : WALL ? (step_waves_qe<D, S, MODE, QE>() > 3 ? 3 : step_waves_qe<D, S, MODE, QE>())
                  : step_waves_qe<D, S, MODE, QE>();
}

// Pull with diffuse walls (the boundary rule of the lid-driven cavity,
// Sec. V C; the paper cites Ansumali and Karlin for it): on an axis whose
// bit is set in walls the domain is bounded by walls half-way outside the
// first and last nodes.  A population whose source lies in a wall is
// re-emitted by the wall of the first such axis (order x, y, z) as
// rho_w feq_i(1, u_wall), one rho_w per node, such that the re-emitted
// populations carry exactly the mass that the node's post-collision
// populations sent into the walls.  Interior populations are pulled as in the
// periodic case; sources outside are never loaded.
// Straight-line code: a wall test and a load behind a branch per population
// made the rows on a wall wait for some 60 loads in turn, about 15 us, in the
// first plane and, worse, the last.  Per step, rows of 256-lane blocks:
// D3Q27 cavity 256^3 752 -> 672 us (F32), 1949 -> 1571 (FP64), 531 -> 425
// (F16-shifted); 64^3 45 -> 27 us (F32); 32^3 22 -> 12 us.
template <int D, typename S>
__device__ inline void pull_walls(const StepArgs &a, int x, int y, int z, typename Storage<S>::T (&p)[Lat<D>::Q])
{
    using T = typename Storage<S>::T;
    constexpr int Q = Lat<D>::Q;
    constexpr bool SH = Storage<S>::kShifted;
    const int n[3] = {a.nx, a.ny, a.nz};
    const int xc[3] = {x, y, z};
    const long long N = a.N, cell = ((long long)z * n[1] + y) * n[0] + x;
    const S *__restrict__ fin = (const S *)a.fin;
    // per axis and velocity component c (at c + 1): the source coordinate,
    // wrapped, and the wall beyond which it lies (2 k + side, -1: none);
    // selects throughout, so that no load waits behind a branch
    int sc[3][3], wc[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const bool walled = k < D && (a.walls >> k & 1);
#pragma unroll
        for (int c = -1; c <= 1; ++c) {
            const int v = xc[k] - c, lo = v < 0, hi = v >= n[k];
            sc[k][c + 1] = v + (lo ? n[k] : 0) - (hi ? n[k] : 0);
            wc[k][c + 1] = c != 0 && walled && (lo || hi) ? 2 * k + hi : -1;
        }
    }
    auto wall_of = [&](int i) {
        const int wx = wc[0][Lat<D>::c(i, 0) + 1], wy = wc[1][Lat<D>::c(i, 1) + 1];
        const int wz = D == 3 ? wc[2][Lat<D>::c(i, 2) + 1] : -1;
        return wx >= 0 ? wx : (wy >= 0 ? wy : wz);
    };
    // deviations from the weights, so that the shifted formats keep their
    // precision: mass out of the node minus the weights of the outgoing
    // populations, and the re-emitted equilibrium minus its weights; in
    // double where the storage policy forms the moments in double (the
    // re-emission is a moment computation of the wall node)
    using E = typename std::conditional<StepPolicy<S>::mom_f64, double, T>::type;
    // every load before any use: the population's source, or for one that a
    // wall re-emits, the opposite population that left this node into the
    // same wall
    // (masks in place of selects, which the compiler would make branches)
    T out[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int none = wall_of(i) >> 31;  // all ones where no wall emits it
        const int px = x + ((sc[0][Lat<D>::c(i, 0) + 1] - x) & none);
        const int py = y + ((sc[1][Lat<D>::c(i, 1) + 1] - y) & none);
        const int pz = z + ((sc[2][Lat<D>::c(i, 2) + 1] - z) & none);
        const int q = (Q - 1 - i) + ((2 * i - (Q - 1)) & none);
        out[i] = Storage<S>::to_T(fin[q * N + ((long long)pz * n[1] + py) * n[0] + px]);
    }
    E out_dev = E(0), in_dev = E(0), in_w = E(0), em[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int wl = wall_of(i);
        em[i] = E(a.wall_eq[(wl & ~(wl >> 31)) * Q + i]);  // feq_i(1, u_wall) - w_i
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const bool wall = wall_of(i) >= 0;
        in_dev += wall ? em[i] : E(0);
        in_w += wall ? E(Lat<D>::w(i)) : E(0);
        out_dev += wall ? (SH ? E(out[i]) : E(out[i]) - E(Lat<D>::w(Q - 1 - i))) : E(0);
    }
    // rho_w = (in_w + out_dev) / (in_w + in_dev), as 1 + drho_w
    const E drw = (out_dev - in_dev) * rcp_(in_w + in_dev);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const E dev = fma_(drw, E(Lat<D>::w(i)) + em[i], em[i]);  // rho_w feq_i - w_i
        const T emitted = SH ? T(dev) : T(E(Lat<D>::w(i)) + dev);
        p[i] = wall_of(i) >= 0 ? emitted : out[i];
    }
}

// The same rule for a cell whose only sources outside the domain lie across
// one x wall (SIDE 0: the cell at x = 0, whose populations with c_x = +1
// come from the wall; SIDE 1: x = nx - 1, c_x = -1), in a row that is
// interior along y and z, after the periodic pull has loaded every
// population: those populations are replaced, with the same sums in the same
// order as pull_walls forms them, so the result is the same to the bit.  The
// population set is fixed at compile time, so the loads issue together.
template <int D, typename S, int SIDE>
__device__ inline void fix_x_wall(const StepArgs &a, long long cell, typename Storage<S>::T (&p)[Lat<D>::Q])
{
    using T = typename Storage<S>::T;
    constexpr int Q = Lat<D>::Q;
    constexpr bool SH = Storage<S>::kShifted;
    constexpr int CS = SIDE == 0 ? 1 : -1;
    const long long N = a.N;
    const S *__restrict__ fin = (const S *)a.fin;
    using E = typename std::conditional<StepPolicy<S>::mom_f64, double, T>::type;
    E out_dev = E(0), in_dev = E(0), in_w = E(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if (Lat<D>::c(i, 0) != CS) continue;
        in_dev += E(a.wall_eq[SIDE * Q + i]);
        in_w += E(Lat<D>::w(i));
        const int j = Q - 1 - i;
        const E v = E(Storage<S>::to_T(fin[(long long)j * N + cell]));
        out_dev += SH ? v : v - E(Lat<D>::w(j));
    }
    const E drw = (out_dev - in_dev) * rcp_(in_w + in_dev);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if (Lat<D>::c(i, 0) != CS) continue;
        const E e = E(a.wall_eq[SIDE * Q + i]);
        const E dev = fma_(drw, E(Lat<D>::w(i)) + e, e);
        p[i] = SH ? T(dev) : T(E(Lat<D>::w(i)) + dev);
    }
}

// In-place (AA) stepping on one lattice: pairs of launches, the first of
// which reads every population from its source cell x - c_i (as the
// two-lattice pull) and writes the post-collision population i back to the
// slot it read for the opposite direction, slot opp(i) of cell x + c_i; the
// second reads the populations of its own cell from the opposite slots and
// writes them to their own slots.  Each launch touches every location from
// one lane only (the one it reads is the one it writes), so it runs in place,
// and after the pair the lattice holds the post-collision state in the
// two-lattice layout.  kAAPull / kAALocal select the two launches.
// On two lattices an even count of steps ends with such a pair in f_in, whose
// local half also writes f_out: the newest state is then in both, as after a
// copy, for one more write of a state instead of a read and a write (256^3, 20
// steps F32 12.67 -> 12.32 ms, 10 steps FP64 14.09 -> 13.38).
enum AAKind { kTwoLattice = 0, kAAPull = 1, kAALocal = 2 };

template <int D, typename S, int MODE, bool DIAG, bool FORCE, bool WALL = false, bool QE = false, int AA = kTwoLattice, bool FLAT = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(step_waves_k<D, S, MODE, WALL, QE, AA>()))) void k_step(StepArgs a)
{
    using T = typename Storage<S>::T;
    using Pol = StepPolicy<S>;
    constexpr int Q = Lat<D>::Q;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const long long N = a.N;
    const int z = (int)blockIdx.z;
    // the lane's offset in its row, or (FLAT) in its plane
    const unsigned bx = FLAT ? kFlatBlock : (unsigned)block_x(nx);
    const unsigned lx = blockIdx.x * bx + threadIdx.x;
    // in place the two pointers are the same buffer: no restrict there
    using InP = typename std::conditional<AA == kTwoLattice, const S *__restrict__, const S *>::type;
    using OutP = typename std::conditional<AA == kTwoLattice, S *__restrict__, S *>::type;
    InP fin = (const S *)a.fin;
    OutP fout = (S *)a.fout;
    const T beta = (T)a.beta;
    // the end of the step needs these two: read now, with the other arguments
    // (an input of an empty asm), and not on first use, where a small grid's
    // step waits for them (D2Q9 F32, per step of a graph: 64^2 2.98 -> 2.95 us,
    // 128^2 3.11 -> 3.07)
    const unsigned cached = a.cached;
    asm volatile("" :: "s"(fout), "s"(cached));
    // the LDS columns of the stored values a double-precision step parks
    __shared__ T stash[stash_pops<D, S, MODE, WALL, QE, AA>() > 0 ? stash_pops<D, S, MODE, WALL, QE, AA>() * kStashStride : 1];

    LaneStats ls;
    if (lx < (unsigned)(FLAT ? nx * ny : nx)) {
        // source rows and x offsets of the pull (and, in place, the
        // neighbours the pull half stores to)
        const auto pix = [&]() {
            if constexpr (FLAT) return FlatIndex<D>(lx, z, nx, ny, nz, a.inv_nx);
            else return PullIndex<D>((int)lx, (int)blockIdx.y, z, nx, ny, nz);
        }();
        const int x = [&]() { if constexpr (FLAT) return pix.x; else return (int)lx; }();
        const int y = [&]() { if constexpr (FLAT) return pix.y; else return (int)blockIdx.y; }();
        const long long row0 = pix.row0;
        const long long cell = row0 + lx;

        // p: the stored values as arithmetic type -- the populations g, or
        // their deviations g - w for shifted storage.  Only p and d = feq - g
        // stay live as Q-arrays; g and g - w are formed on the fly (g - w is
        // exact in floating point for g within a factor two of w).
        // Each population's source row is block-uniform; only the x offset
        // varies per lane.
        constexpr bool SH = Storage<S>::kShifted;
        T p[Q];
        auto pull = [&]() {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const S *rowp = fin + ((long long)i * N + pix.src_row(i));
                p[i] = Storage<S>::to_T(*lane_ptr(rowp, pix.src_x(i)));
            }
        };
        if constexpr (WALL) {
            // A row in the first or last layer along a walled y or z axis
            // (block-uniform) takes the walled pull throughout.  Every other
            // row pulls as in the periodic step, with the row's coalesced
            // loads, and only its cells at a walled x boundary then replace
            // the populations whose source lies beyond it.
            // (A row one cell long between x walls has both at one cell.)
            const bool wall_row = ((a.walls & 2) && (y == 0 || y == ny - 1)) ||
                                  (D == 3 && (a.walls & 4) && (z == 0 || z == nz - 1)) ||
                                  ((a.walls & 1) && nx == 1);
            if (wall_row) {
                pull_walls<D, S>(a, x, y, z, p);
            } else {
                pull();
                if (a.walls & 1) {
                    if (x == 0) fix_x_wall<D, S, 0>(a, cell, p);
                    else if (x == nx - 1) fix_x_wall<D, S, 1>(a, cell, p);
                }
            }
        } else if constexpr (AA == kAALocal) {
#pragma unroll
            for (int i = 0; i < Q; ++i) p[i] = Storage<S>::to_T(fin[(long long)(Q - 1 - i) * N + cell]);
        } else {
            pull();
        }
        auto dev = [&](int i) { return SH ? p[i] : p[i] - T(Lat<D>::w(i)); };

        // Moments: rho and j feed the equilibrium, and a rounded
        // single-precision sum is a fixed function of the cell's state, i.e.
        // a bias on the equilibrium's stress that accumulates over steps;
        // summed in double where the storage is precise enough to see it.
        using E = typename std::conditional<Pol::mom_f64, double, T>::type;
        E drhoE, jE[3];
        row_moments<D, E>([&](int i) { return E(dev(i)); }, drhoE, jE);
        // positivity by comparisons (a min over raw loaded values would make
        // the compiler keep quieted copies of all of them); of a shifted value
        // against -w, which has the sign of w + p without the sum
        bool pos = true;
#pragma unroll
        for (int i = 0; i < Q; ++i) pos = pos && (p[i] > (SH ? -T(Lat<D>::w(i)) : T(0)));
        // from here on the stored values are read through pa: in registers,
        // or mostly parked in LDS (the empty asm's memory clobber keeps the
        // compiler from forwarding the parked registers to their reads)
        constexpr int NST = stash_pops<D, S, MODE, WALL, QE, AA>();
        PopAccess<T, Q, (NST > 0 ? NST : 1)> parked;
        if constexpr (NST > 0) {
#pragma unroll
            for (int i = 0; i < NST; ++i) stash[i * kStashStride + threadIdx.x] = p[i];
            asm volatile("" ::: "memory");
            parked.col = &stash[threadIdx.x];
#pragma unroll
            for (int i = NST; i < Q; ++i) parked.tail[i - NST] = p[i];
        }
        const auto &pa = pick<NST == 0>(p, parked);
        auto pdev = [&](int i) { return SH ? pa[i] : pa[i] - T(Lat<D>::w(i)); };
        const T drho = T(drhoE);
        const T j[3] = {T(jE[0]), T(jE[1]), T(jE[2])};
        // NaN in any population fails its comparison and propagates into drho.
        // The classic LBGK needs no logarithm: it collides every finite cell,
        // non-positive populations included (they are still counted).
        const bool finite = abs_(drhoE) < E(1e30);
        const bool ok = (pos || MODE == MODE_LBGK) && finite;
        const T rho = T(1) + drho;
        T alpha = T(0);
        CellInfo info{0, 0, 0, 0, 0};
        T dd[Q];
        // the output is p + (ab + ab_lo) dd; where the policy asks for it,
        // alpha beta is a two-term sum so that its rounding to single
        // precision is not a bias shared by every cell (with alpha = 2 in
        // all gated cells, a rounded 2 beta would shift the viscosity of the
        // whole flow by its relative rounding)
        T ab = T(0), ab_lo = T(0);
        if (ok) {
            // d = feq - g with the equilibrium in double where the policy asks
            // for it: the rounding of a single-precision equilibrium is a
            // fixed function of the cell's state, so it acts as a bias that
            // accumulates over steps.  The path length stays in T.
            using EQ = typename std::conditional<Pol::eq_f64, double, T>::type;
            form_deviation<D, T, EQ, MODE == MODE_LBGK, Pol::conserve, Pol::pin_dev>(pdev, EQ(drhoE),
                                                                                    {EQ(jE[0]), EQ(jE[1]), EQ(jE[2])}, dd);
            // ES-BGK: the quasi-equilibrium replaces the equilibrium, and the
            // path length is found from x = f^QE / g - 1 as before
            int qe_it = 0;
            bool qe_ok = true;
            if constexpr (QE) {
                const EQ rq = EQ(1) + EQ(drhoE), ir = rcp_(rq);
                const EQ uq[3] = {EQ(jE[0]) * ir, EQ(jE[1]) * ir, D == 3 ? EQ(jE[2]) * ir : EQ(0)};
                qe_ok = quasi_equilibrium<D, T, EQ, SH>(p, dd, rq, uq, EQ(a.cpr), qe_it);
            }
            alpha = path_length<D, T, typename Pol::Exact, MODE, SH, typename Pol::Series>(pa, dd, a.beta, info);
            if constexpr (QE) {
                info.iters = qe_it;
                info.fallback = !qe_ok;
            }
            if (Pol::ab_split) {
                const double abE = double(alpha) * a.beta;
                ab = T(abE);
                ab_lo = T(abE - double(ab));
            } else {
                ab = alpha * beta;
            }
            if (FORCE) {
                const T ir = rcp_(rho);
                const T u[3] = {quot_(j[0], rho, ir), quot_(j[1], rho, ir), D == 3 ? quot_(j[2], rho, ir) : T(0)};
                T du[3] = {T(0), T(0), T(0)};
#pragma unroll
                for (int c = 0; c < D; ++c) du[c] = (T)a.force[(long long)c * N + cell] * ir;
#pragma unroll
                for (int i = 0; i < Q; ++i) dd[i] = (ab + ab_lo) * dd[i];
                ForceTerm<D, T>(rho, u, du).add(dd);
                ab = T(1);
                ab_lo = T(0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                dd[i] = T(0);
                // (zeros_in_branch: the empty asm keeps the zeros in this
                // branch; hoisted above it, they cost every wave Q moves that
                // only uncollided lanes need)
                if constexpr (Pol::zeros_in_branch) asm volatile("" : "+v"(dd[i]));
            }
        }
        // post-collision value p + alpha beta (feq - g) [+ force term], in the
        // storage type before any branch (a 2-byte value then takes its one
        // rounding from the multiply-add in every variant of the step)
        S res[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i)
            res[i] = Storage<S>::from_T(Pol::ab_split || FORCE ? fma_(ab, dd[i], fma_(ab_lo, dd[i], pa[i])) : fma_(ab, dd[i], pa[i]));
        auto put = [&](OutP out, auto store) {
            // (the fields' distance as a value of this branch's own: shared,
            // the Q field addresses are formed ahead of the branch and spill.
            // In place they are the addresses of the loads: 256^3, per step,
            // formed again / shared FP64 1481 / 1474 us, F32 659.6 / 657.7,
            // F16-shifted 374.8 / 373.1)
            long long n1 = N;
            if constexpr (AA == kTwoLattice) asm volatile("" : "+s"(n1));
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                if constexpr (AA == kAAPull) {
                    // slot opp(i) of cell x + c_i, the location this lane read
                    // population opp(i) from
                    store(lane_ptr(out + uniform64((Q - 1 - i) * n1 + pix.dst_row(i)), pix.dst_x(i)), res[i]);
                } else {
                    store(lane_ptr(out + uniform64(i * n1 + row0), lx), res[i]);
                }
            }
        };
        // (the empty asm keeps the compiler from joining the branches' stores
        // and dropping the hint)
        OutP own = AA == kAALocal ? (OutP)a.fin : fout;
        if (cached & 1) {
            put(own, [](S *q, S v) { *q = v; });
            asm volatile("; end of cached stores");
        } else {
            put(own, [](S *q, S v) { Storage<S>::store_nt(q, v); });
        }
        if constexpr (AA == kAALocal) {
            // the last of an even count of steps on two lattices leaves its
            // state in both (the kind of stores: cached_copy)
            if (fout != own) {
                if (cached & 2) {
                    put(fout, [](S *q, S v) { *q = v; });
                    asm volatile("; end of cached stores");
                } else {
                    put(fout, [](S *q, S v) { Storage<S>::store_nt(q, v); });
                }
            }
        }

        // the velocity and density of the output state, for a loss that
        // depends on f through them: u = (sum_i c_i f_out,i + F/2) / rho,
        // where the output's momentum is j, plus F in a collided forced cell
        // (the force term adds F exactly); formed here from the moments the
        // step already holds, in place of a pass that re-reads the state
        if ((DIAG || FORCE) && a.uv_out) {
            const T r = T(1) + drho, ir = rcp_(r);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                T jc = j[c];
                if (FORCE) jc += (ok ? T(1.5) : T(0.5)) * (T)a.force[(long long)c * N + cell];
                a.uv_out[(long long)c * N + cell] = (float)quot_(jc, r, ir);
            }
            a.uv_out[(long long)D * N + cell] = (float)r;
        }

        if (DIAG) {
            if (a.alpha_out) ((T *)a.alpha_out)[cell] = ok ? alpha : T(__builtin_nan(""));
            // nu_T = theta (2 - alpha) / (2 alpha beta), theta = 1/3 (Eq. nuT)
            if (a.nut_out)
                ((T *)a.nut_out)[cell] = ok ? (T(2) - alpha) * rcp_(T(6) * alpha * beta) : T(__builtin_nan(""));
            if (ok) {
                const double r = 1.0 + (double)drho;
                ls.mass = r;
                double jj = 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    ls.mom[c] = (double)j[c];
                    jj += (double)j[c] * (double)j[c];
                }
                ls.ke = 0.5 * jj / r;
                ls.asum = (double)alpha;
                ls.amin = ls.amax = (unsigned long long)__double_as_longlong((double)alpha);
                ls.n = true;
                ls.gated = info.gated;
                ls.guard = info.guarded;
                ls.lt2 = alpha < T(2);
                ls.exact = info.exact;
                ls.iters = info.iters;
                ls.fallback = info.fallback;
                ls.nonpos = !pos;
            } else {
                ls.nonpos = true;
            }
        }
    }
    if (DIAG && a.stats) block_reduce_stats<QE || is_mirror_mode(MODE)>(ls, a.stats + ((FLAT ? blockIdx.x : blockIdx.y) + blockIdx.z) % kStatSlots, (int)(bx >> 6));
}

// Occupancy cap of the D3Q27 alpha = 2 steps in the 4- and 2-byte formats.
// With their fewer registers the hardware would run five waves per SIMD (F32:
// 94 VGPRs), which measured slower than four at 256^3 (F32 0.635 -> 0.627 ms,
// F16-shifted 0.337 -> 0.324 ms; the closed-form steps run at four already):
// past four waves the added concurrent streams (27 per wave) cost the HBM
// more than they hide.  D2Q9, with 9 streams per wave, keeps the hardware's
// occupancy.  Dynamic LDS that the kernel never touches bounds the blocks per
// CU.  Four waves per SIMD are 16 per CU, so a block of w waves gets a 16 / w
// share of the CU's 160 KiB, less 1 KiB for the kernel's own static LDS (the
// statistics reduction's 544 bytes).
template <int D, typename S, int MODE>
static unsigned occupancy_cap_lds(int bx)
{
    if constexpr (D == 3 && (MODE == MODE_BGK || MODE == MODE_LBGK) &&
                  !std::is_same<typename Storage<S>::T, double>::value) {
        const int blocks = 16 / (bx / 64);  // bx is 64, 128, 192 or 256
        return (unsigned)((160 * 1024 / blocks - 1024) & ~511);
    }
    return 0;
}

template <int D, typename S, int MODE, bool FLAT>
static hipError_t launch_step_t(bool diag, const StepArgs &a, hipStream_t s)
{
    // (x-block, y, z), or (plane block, 1, z); the API limits ny and nz to the
    // grid's 65535
    const int bx = FLAT ? (int)kFlatBlock : block_x(a.nx);
    if (a.ny > 65535 || a.nz > 65535) return hipErrorInvalidConfiguration;
    const long long line = FLAT ? (long long)a.nx * a.ny : a.nx;
    const dim3 grid((unsigned)((line + bx - 1) / bx), FLAT ? 1u : (unsigned)a.ny, (unsigned)a.nz), block(bx);
    const bool force = a.force != nullptr;
    if (a.aa != kTwoLattice) {
        // in place: periodic, the closed-form and alpha = 2 modes
        if constexpr (MODE == MODE_HIGHER || MODE == MODE_LOWER || MODE == MODE_BGK || MODE == MODE_LBGK) {
            if (a.walls || a.cpr != 0.0) return hipErrorInvalidValue;
            if (force && !std::is_same<S, float>::value) return hipErrorInvalidValue;
#define ESELBM_AA_LAUNCH(KIND)                                                                          \
    do {                                                                                                \
        if (force) {                                                                                    \
            if constexpr (std::is_same<S, float>::value) {                                              \
                if (diag) hipLaunchKernelGGL((k_step<D, S, MODE, true, true, false, false, KIND, FLAT>), grid, block, 0, s, a);  \
                else hipLaunchKernelGGL((k_step<D, S, MODE, false, true, false, false, KIND, FLAT>), grid, block, 0, s, a);      \
            }                                                                                           \
        } else if (diag) {                                                                              \
            hipLaunchKernelGGL((k_step<D, S, MODE, true, false, false, false, KIND, FLAT>), grid, block, 0, s, a);              \
        } else {                                                                                        \
            hipLaunchKernelGGL((k_step<D, S, MODE, false, false, false, false, KIND, FLAT>), grid, block, 0, s, a);             \
        }                                                                                               \
    } while (0)
            if (a.aa == kAAPull) ESELBM_AA_LAUNCH(kAAPull);
            else ESELBM_AA_LAUNCH(kAALocal);
#undef ESELBM_AA_LAUNCH
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (a.cpr != 0.0) {
        // ES-BGK: periodic, unforced, path lengths alpha_Higher, alpha_Lower, 2
        if constexpr (MODE == MODE_HIGHER || MODE == MODE_LOWER || MODE == MODE_BGK) {
            if (force || a.walls) return hipErrorInvalidValue;
            if (diag) hipLaunchKernelGGL((k_step<D, S, MODE, true, false, false, true, kTwoLattice, FLAT>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((k_step<D, S, MODE, false, false, false, true, kTwoLattice, FLAT>), grid, block, 0, s, a);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (a.walls) {
        if (force) return hipErrorInvalidValue;
        if (diag) hipLaunchKernelGGL((k_step<D, S, MODE, true, false, true, false, kTwoLattice, FLAT>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_step<D, S, MODE, false, false, true, false, kTwoLattice, FLAT>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    if (force) {
        if constexpr (std::is_same<S, float>::value) {
            if (diag) hipLaunchKernelGGL((k_step<D, S, MODE, true, true, false, false, kTwoLattice, FLAT>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((k_step<D, S, MODE, false, true, false, false, kTwoLattice, FLAT>), grid, block, 0, s, a);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    const unsigned lds = occupancy_cap_lds<D, S, MODE>(bx);
    if (diag) hipLaunchKernelGGL((k_step<D, S, MODE, true, false, false, false, kTwoLattice, FLAT>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((k_step<D, S, MODE, false, false, false, false, kTwoLattice, FLAT>), grid, block, lds, s, a);
    return hipGetLastError();
}

template <int D, typename S, bool FLAT>
static hipError_t launch_step_m(int mode, bool diag, const StepArgs &a, hipStream_t s)
{
    switch (mode) {
    case MODE_HIGHER: return launch_step_t<D, S, MODE_HIGHER, FLAT>(diag, a, s);
    case MODE_BGK: return launch_step_t<D, S, MODE_BGK, FLAT>(diag, a, s);
    case MODE_LBGK: return launch_step_t<D, S, MODE_LBGK, FLAT>(diag, a, s);
    case MODE_LOWER: return launch_step_t<D, S, MODE_LOWER, FLAT>(diag, a, s);
    case MODE_ELBM: return launch_step_t<D, S, MODE_ELBM, FLAT>(diag, a, s);
    case MODE_ITERATE1: return launch_step_t<D, S, MODE_ITERATE1, FLAT>(diag, a, s);
    }
    return hipErrorInvalidValue;
}

// One storage type S and lane mapping: every lattice, mode and variant of the
// step.
template <typename S, bool FLAT>
inline hipError_t launch_step_storage(int D, int mode, bool diag, const StepArgs &a, hipStream_t s)
{
    return D == 2 ? launch_step_m<2, S, FLAT>(mode, diag, a, s) : launch_step_m<3, S, FLAT>(mode, diag, a, s);
}

}  // namespace eselbm
