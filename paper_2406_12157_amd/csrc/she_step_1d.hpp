#pragma once

// Step kernels of 1D batches whose waves hold whole rods or shares of them, and
// their typed launchers: explicit batches, and the rods of up to kRodAlone cells of
// batches with implicit ones.  Included by the translation units that instantiate
// them (one per state type, mode and kernel).
//
// Scheme (Garcia et al., Sec. 3): face flux F_f = r (U_f - U_{f-1}) + w sigma A N_f
// through the low face f of cell f, update U_i += F_{i+1} - F_i (FE), or the
// predictor-corrector U = (U + U* + Delta(U*; same N)) / 2 (PC).  Dirichlet
// walls: F_0 = 2 r (U_0 - U_L) + sqrt(2) sigma A(U_L) N_0 and mirrored at the
// right wall (ghost stencil U_1 - 3U_0 + 2U_L of the Dirichlet paragraph).
// Material varying along the rod (composite-rod exercise, Sec. 6; MODE 1): a
// conductance r_f and noise factor s_f per face and a factor w_i per cell.
//
// A lane holds a unit of CPL consecutive cells in registers for the whole
// launch, and neighbouring units sit in neighbouring lanes, so a stage (the FE
// step, or either half of a PC step) moves one cell value and one face flux
// across by a DPP wave shift: no LDS access and no barrier.  A face is evaluated in
// the lane that owns it and taken over by its neighbour, so the sum is conserved
// bit for bit; where two waves of k_rods meet, each evaluates the face between
// them, from the same values by the same code, whose multiply-adds are written out
// so that every copy of it rounds alike.  Two kernels differ in where the numbers
// come from:
//
// k_rods: every wave draws its own numbers, four cells per Philox call.  An
//   instance takes whole waves of a workgroup (small instances share one).
//   Where it takes several, each wave also carries copies of its neighbours'
//   edge units (the halo lanes), with their numbers, and advances them
//   redundantly: a halo of 4 cells stays valid for 4 stages, so the waves of an
//   instance exchange edges through LDS once per 4 stages (between neighbours
//   only, by flags, the numbers of the next step being drawn meanwhile).
//   Bound by VALU issue once a SIMD has four waves: 92 vector instructions per
//   FE step of a wave (60 of them the numbers) and 136 per PC step, about 480
//   and 640 cycles.  FP32, us per step: 256 rods of 3967 cells FE 0.93 and PC
//   1.28, i.e. 1.10e12 and 7.9e11 cell-updates/s; the 1000 ragged rods (64 to
//   4096 cells, FE and PC) 1.38 against 2.09 with one LDS exchange and barrier
//   per stage.
// k_rods_ahead: the numbers do not depend on the state, so one wave of the
//   workgroup only advances the state and the others draw the numbers of the
//   next steps into LDS, (step, block) pairs packed over all lanes, and take
//   the samples.  The step is then the state's own dependent chain: 26 vector
//   instructions per FE and 53 per PC step with 2 cells per lane.  For rods of
//   up to 256 cells; us per step, against one wave that draws its own numbers:
//   one FP32 PC rod of 128 cells 0.12 (0.93 with statistics before, 0.14 now),
//   1024 of them 0.21 (1.02), one FP64 FE ring of 64 cells 0.10 (1.66).
#include <climits>
#include <type_traits>

#include "she_internal.hpp"
#include "she_rng.hpp"
#include "she_wave.hpp"

namespace she {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Noise amplitude of a face with value v: v (SHE), sqrt(v) (DK),
// sqrt(v (1 - v)) (Burgers); a negative radicand is clamped and counted.
template <typename T>
__device__ __forceinline__ T face_amp(int eq, T v, uint32_t &clamps)
{
    if (eq == 0) return v;
    const T q = eq == 2 ? v * (T(1) - v) : v;
    if (q < T(0)) {
        ++clamps;
        return T(0);
    }
    return amp_sqrt(q);
}

__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f64x4 mfma16x16x4(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// C[N x N] += X^T X for a full block X[256 x N] (row = snapshot).  Tiles of
// 16 x 16 over the upper triangle are spread over the instance's waves
// (wave = 0 .. nwave-1); each lane accumulates four outputs of its tile over
// K = 256 in the matrix-core accumulator type and adds them to the FP64 sum
// (both triangles).
// Operand layout of the 16x16x4 instructions: lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; output element v of lane l is D[4(l/16)+v][l%16] for
// the FP32 form and D[(l/16)+4v][l%16] for the FP64 form.
template <typename T>
__device__ void xtx_block(const T *__restrict__ X, double *__restrict__ Cm, int N, int wave, int nwave)
{
    using acc_t = typename std::conditional<std::is_same<T, float>::value, f32x4, f64x4>::type;
    const int lane = threadIdx.x & 63;
    const int nt = (N + 15) >> 4;
    const int ntiles = nt * (nt + 1) / 2;
    for (int t = wave; t < ntiles; t += nwave) {
        int ti = 0, rem = t;
        while (rem >= nt - ti) {
            rem -= nt - ti;
            ++ti;
        }
        const int tj = ti + rem;
        // rows and columns beyond N only reach outputs that are dropped: their
        // operands may be any (the last cell's)
        const uint32_t i = (lane >> 4) * N + min(16 * ti + (lane & 15), N - 1);
        const uint32_t j = (lane >> 4) * N + min(16 * tj + (lane & 15), N - 1);
        acc_t acc = {0, 0, 0, 0};
        // eight K-steps of operands are loaded before their eight products, so
        // the loads overlap instead of each product waiting for its own
        constexpr int kB = 8;
        for (int k0 = 0; k0 < kCorrBlock; k0 += 4 * kB) {
            T a[kB], b[kB];
#pragma unroll
            for (int q = 0; q < kB; ++q) {
                const T *row = X + static_cast<int64_t>(k0 + 4 * q) * N;  // uniform
                a[q] = row[i];
                b[q] = row[j];
            }
#pragma unroll
            for (int q = 0; q < kB; ++q) acc = mfma16x16x4(a[q], b[q], acc);
        }
        const int col = 16 * tj + (lane & 15);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            // output rows: FP32 form 4(l/16)+v, FP64 form (l/16)+4v (measured on gfx950)
            const int row = 16 * ti + (std::is_same<T, float>::value ? 4 * (lane >> 4) + v : (lane >> 4) + 4 * v);
            if (row < N && col < N) {
                const double val = static_cast<double>(acc[v]);
                Cm[(int64_t)row * N + col] += val;
                if (ti != tj) Cm[(int64_t)col * N + row] += val;
            }
        }
    }
}

// ------------------------------------------------------------------ lanes

// v of the lane to the left (lane - 1) or right; the lane without one gets edge.
template <int CTRL>
__device__ __forceinline__ float dpp_shift(float edge, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), CTRL, 0xf, 0xf, false));
}

template <int CTRL>
__device__ __forceinline__ double dpp_shift(double edge, double v)
{
    const long long e = __double_as_longlong(edge), u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(static_cast<int>(e & 0xffffffffLL), static_cast<int>(u & 0xffffffffLL),
                                               CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(static_cast<int>(e >> 32), static_cast<int>(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

template <typename T>
__device__ __forceinline__ T from_left(T edge, T v) { return dpp_shift<0x138>(edge, v); }  // wave_shr:1

template <typename T>
__device__ __forceinline__ T from_right(T edge, T v) { return dpp_shift<0x130>(edge, v); }  // wave_shl:1

// v of one lane (the same for the whole wave).
__device__ __forceinline__ float of_lane(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

__device__ __forceinline__ double of_lane(double v, int lane)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// A cell's flux divergence with its capacity factor, rounded by itself.  Left to
// the compiler, the product contracts with the sum that takes it wherever the two
// end up in one basic block, so that a composite rod's last bits depended on the
// kernel and even on the wave that held the cell.
template <typename T>
__device__ __forceinline__ T cell_flux(T w, T d)
{
#pragma clang fp contract(off)
    return w * d;
}

// c ? a : b on values: a select between array elements as lvalues would become
// an address select and move the array to private memory.
template <typename T>
__device__ __forceinline__ T sel(bool c, T a, T b) { return c ? a : b; }

// Entry k (0 .. C-1) of a register array.
template <typename T, int C>
__device__ __forceinline__ T pick(const T (&a)[C], int k)
{
    T v = a[0];
#pragma unroll
    for (int l = 1; l < C; ++l) v = sel(k >= l, a[l], v);
    return v;
}

// Ends of the rod that a wave holds; each kind has its own copy of the step
// loop, so an interior wave carries none of the end code.
enum Ends {
    kInterior = 0,  // none: every neighbour is in the next lane
    kWalls = 1,     // Dirichlet walls, last unit full
    kAny = 2,       // any, the last unit not full among them
    kRing = 3       // periodic rod held by the wave alone, last unit full
};

// The solve of an explicit step.
struct NoSolve {
    template <int C>
    __device__ __forceinline__ void operator()(double (&)[C]) const {}
};

// Modes of a batch.  0: any uniform rods (the face kind is looked up in each
// stage); 3, 4, 5: every rod uniform, with instantaneous noise and of one
// equation, heat, Dean-Kawasaki or Burgers (one face path: fewer registers, no
// branches); 1: material coefficients; 2 and 6: implicit rods among them, 2 with
// and 6 without material coefficients (which take 6 registers per cell in FP64).
// A rod has the same bits in every mode that holds it.
constexpr bool material(int mode) { return mode == 1 || mode == 2; }
constexpr bool implicit(int mode) { return mode == 2 || mode == 6; }
constexpr bool one_face(int mode) { return mode >= 3 && mode <= 5; }

// What one wave knows of its instance: the uniform parameters, the unit of
// each lane and where the ends of the rod lie.
template <typename T, int CPL, int MODE>
struct Rod {
    static constexpr bool VARC = material(MODE), IMPL = implicit(MODE);
    int N;
    bool dir;
    int eq, noise, kind;
    T r, sg, hs, uL, uR, u0, nu;
    T ampL, ampR;    // wall noise factors: sqrt(2) sigma A(U_wall), 0 without noise
    T rwL, rwR;      // wall conductances, doubled
    T r0;            // conductance of the lane's first face: the wall's in its lane
    int lane, unit;  // this lane's unit: cells CPL unit .. CPL unit + CPL - 1
    int nc;          // cells of the rod from the unit's first on (<= 0: none)
    bool own;        // the unit is this wave's (not a halo copy)
    bool wrap1;      // periodic rod held by this wave alone
    bool left_wall;  // Dirichlet and lane 0 holds cell 0
    int lg, m;       // lane of the unit of the last cell (-1: not here), its cells
    bool partial;    // that unit is here and not full
    T ex, rex;       // implicit: weight 1 - theta of the state-dependent deterministic flux; r of that
    T Rf[VARC ? CPL : 1], Sf[VARC ? CPL : 1], Wc[VARC ? CPL : 1];

    // Lane l holds unit first + l (wrapped on a periodic rod); lanes
    // [own0, own1) hold units of the wave's own; lanes up to last hold a unit.
    __device__ __forceinline__ void init(const Inst1D &d, const T *__restrict__ coef, int first, int own0, int own1,
                                         int last, bool alone)
    {
        N = d.n;
        dir = d.bc == 1;
        eq = d.eq;
        noise = d.noise;
        // face kinds: 0 heat with instantaneous noise; 1 deterministic or no
        // noise (any equation); 2 Dean-Kawasaki; 3 Burgers (both instantaneous)
        kind = noise != 0 ? 1 : (eq == 0 ? 0 : eq + 1);
        r = static_cast<T>(d.r);
        sg = static_cast<T>(d.sigma);
        hs = T(0.5) * sg;
        uL = static_cast<T>(d.uL);
        uR = static_cast<T>(d.uR);
        u0 = static_cast<T>(d.u0);
        nu = static_cast<T>(eq == 2 ? d.nu : 0.0);
        lane = threadIdx.x & 63;
        const int units = (N + CPL - 1) / CPL, glast = units - 1;
        unit = first + lane;
        if (!dir) {
            if (unit < 0) unit += units;
            if (unit >= units && lane <= last) unit -= units;
        }
        nc = N - CPL * unit;
        own = lane >= own0 && lane < own1;
        wrap1 = !dir && alone;
        left_wall = dir && first == 0;
        lg = -1;
        m = N - CPL * glast;
        for (int w = -1; w <= 1; ++w) {  // the last cell's unit, on a periodic rod also as a halo
            const int l = glast - first + w * units;
            if ((w == 0 || !dir) && l >= 0 && l <= last && l < 64) lg = lg < 0 ? l : lg;
        }
        partial = lg >= 0 && m < CPL;
        T sw = static_cast<T>(d.sigma * 1.41421356237309504880), swR = sw, rl = r, rr = r;
        ex = static_cast<T>(IMPL && d.scheme >= 2 ? 1.0 - d.theta : 1.0);
        rex = r * ex;
        if constexpr (VARC) {
            const int nf = dir ? N + 1 : N;
            const T *k = d.k_off >= 0 ? coef + d.k_off : nullptr;
#pragma unroll
            for (int l = 0; l < CPL; ++l) {
                const int f = CPL * unit + l;
                const bool wall = dir && (f == 0 || f == N);
                Rf[l] = ex * ((k && f >= 0 && f < nf) ? k[f] : r);
                Sf[l] = (k && f >= 0 && f < nf) ? k[nf + f] : (wall ? sw : sg);
                Wc[l] = (k && f >= 0 && f < N) ? k[2 * nf + f] : T(1);
            }
            if (k && dir) {
                rl = k[0];
                rr = k[N];
                sw = k[nf];
                swR = k[nf + N];
            }
        }
        uint32_t c = 0;
        ampL = noise != 2 ? sw * face_amp<T>(eq, uL, c) : T(0);
        ampR = noise != 2 ? swR * face_amp<T>(eq, uR, c) : T(0);
        rwL = T(2) * rl;
        rwR = T(2) * rr;
        r0 = left_wall && lane == 0 ? rwL : r;
    }

    __device__ __forceinline__ int ends() const
    {
        if (!left_wall && lg < 0) return kInterior;
        if (!one_face(MODE)) return kAny;  // the mixed modes compile two loops only
        if (dir) return partial ? kAny : kWalls;
        return wrap1 && !partial ? kRing : (wrap1 || partial ? kAny : kInterior);
    }

    template <int K>
    __device__ __forceinline__ T face(T lo, T hi, T z, int l, uint32_t &clamps) const
    {
        const T rf = VARC ? Rf[VARC ? l : 0] : (IMPL ? rex : r);
        const T sf = VARC ? Sf[VARC ? l : 0] : sg;
        const T df = hi - lo;
        if constexpr (K == 0) {
            // sf (lo + hi) / 2 z + r (hi - lo): the half goes into the factor
            // (exact), and the multiply-add is written out so that every copy
            // of this code rounds alike
            return fma((VARC ? T(0.5) * sf : hs) * (lo + hi), z, rf * df);
        } else {
            const T cf = T(0.5) * (lo + hi);
            const int f = CPL * unit + l;
            // clamps are counted on the faces of this wave's own cells
            const bool mine = own && l < nc && !(dir && f == 0);
            if constexpr (K == 1) {
                T am = T(0);
                if (noise == 1) {
                    const T v = dir ? uL + (uR - uL) * static_cast<T>(f) / static_cast<T>(N) : u0;
                    uint32_t c = 0;
                    am = face_amp<T>(eq, v, c);
                    if (mine) clamps += c;
                }
                return fma(sf * am, z, fma(-nu * cf, T(1) - cf, rf * df));
            } else if constexpr (K == 2) {
                const bool neg = cf < T(0);
                if (mine && neg) ++clamps;
                const T am = neg ? T(0) : amp_sqrt(cf);
                return fma(sf * am, z, rf * df);
            } else {
                const T q = cf * (T(1) - cf);
                const bool neg = q < T(0);
                if (mine && neg) ++clamps;
                const T am = neg ? T(0) : amp_sqrt(q);
                return fma(sf * am, z, fma(-nu, q, rf * df));
            }
        }
    }

    // Flux divergence dv of the state V; z: the numbers of the lane's faces, zN:
    // in the lane of the last cell that of the right wall.
    template <int E, int K>
    __device__ __forceinline__ void stage_k(const T (&V)[CPL], const T (&z)[CPL], T zN, T (&dv)[CPL],
                                            uint32_t &clamps) const
    {
        constexpr bool WALLS = E == kWalls || E == kAny;
        T lastv = V[CPL - 1];
        if (E == kAny && CPL > 1 && partial) lastv = sel(lane == lg, pick<T, CPL>(V, m - 1), lastv);
        T edge = uL;
        if (E == kRing || (E == kAny && wrap1)) edge = of_lane(lastv, lg);
        const T left = from_left(edge, lastv);
        T F[CPL + 1];
        // walls: F_0 = 2 r (U_0 - U_L) + sqrt 2 sigma A(U_L) N_0, mirrored at face N
        const bool wall0 = WALLS && left_wall && lane == 0;
        if constexpr (WALLS && K == 0 && !VARC && !IMPL) {
            // the left wall is a face like any other but for its factors
            const T w = sel(wall0, ampL, hs * (left + V[0]));
            F[0] = fma(w, z[0], r0 * (V[0] - left));
        } else {
            F[0] = face<K>(left, V[0], z[0], 0, clamps);
            if (WALLS && left_wall) {
                T w = rwL * ((IMPL ? ex * V[0] : V[0]) - uL);
                if constexpr (K != 0 && K != 2) w = fma(-nu * uL, T(1) - uL, w);
                w = fma(ampL, z[0], w);
                F[0] = sel(wall0, w, F[0]);
            }
        }
#pragma unroll
        for (int l = 1; l < CPL; ++l) F[l] = face<K>(V[l - 1], V[l], z[l], l, clamps);
        T Fr = F[0];
        if (E == kWalls || (E == kAny && dir)) {
            T w = rwR * (uR - (IMPL ? ex * lastv : lastv));
            if constexpr (K != 0 && K != 2) w = fma(-nu * uR, T(1) - uR, w);
            w = fma(ampR, zN, w);
            Fr = sel(lane == lg, w, from_right(w, F[0]));
        } else {
            Fr = from_right(F[0], F[0]);
            if (E == kRing || (E == kAny && wrap1)) Fr = sel(lane == lg, of_lane(F[0], 0), Fr);
        }
        F[CPL] = Fr;
        if (E == kAny && CPL > 1 && partial) {
#pragma unroll
            for (int l = 1; l < CPL; ++l) F[l] = sel(lane == lg && l == m, Fr, F[l]);
        }
#pragma unroll
        for (int l = 0; l < CPL; ++l) dv[l] = VARC ? cell_flux(Wc[VARC ? l : 0], F[l + 1] - F[l]) : F[l + 1] - F[l];
    }

    template <int E>
    __device__ __forceinline__ void stage(const T (&V)[CPL], const T (&z)[CPL], T zN, T (&dv)[CPL],
                                          uint32_t &clamps) const
    {
        if constexpr (one_face(MODE)) {
            stage_k<E, MODE == 3 ? 0 : MODE - 2>(V, z, zN, dv, clamps);
        } else {
            switch (kind) {
            case 0: stage_k<E, 0>(V, z, zN, dv, clamps); break;
            case 1: stage_k<E, 1>(V, z, zN, dv, clamps); break;
            case 2: stage_k<E, 2>(V, z, zN, dv, clamps); break;
            default: stage_k<E, 3>(V, z, zN, dv, clamps); break;
            }
        }
    }

    // One step (SCHEME 0 FE, 1 PC, 2 implicit: solve) with the numbers z.
    template <int E, int SCHEME, typename Solve>
    __device__ __forceinline__ void step(T (&u)[CPL], const T (&z)[CPL], T zN, uint32_t &clamps, const Solve &solve) const
    {
        T dv[CPL];
        stage<E>(u, z, zN, dv, clamps);
        if constexpr (SCHEME == 2) {
            double x[CPL];
#pragma unroll
            for (int l = 0; l < CPL; ++l) x[l] = l < nc ? static_cast<double>(u[l] + dv[l]) : 0.0;
            solve(x);
#pragma unroll
            for (int l = 0; l < CPL; ++l) u[l] = static_cast<T>(x[l]);
        } else if constexpr (SCHEME == 0) {
#pragma unroll
            for (int l = 0; l < CPL; ++l) u[l] = u[l] + dv[l];
        } else {
            T us[CPL];
#pragma unroll
            for (int l = 0; l < CPL; ++l) us[l] = u[l] + dv[l];
            stage<E>(us, z, zN, dv, clamps);
#pragma unroll
            for (int l = 0; l < CPL; ++l) u[l] = T(0.5) * ((u[l] + us[l]) + dv[l]);
        }
    }

    // f(ends, scheme) for this wave's kind of ends and the instance's scheme, as
    // compile-time constants.
    template <typename Fn>
    __device__ __forceinline__ void by_kind(int scheme, Fn &&f) const
    {
        auto g = [&](auto e) __attribute__((always_inline)) {
            if (scheme == 0) f(e, std::integral_constant<int, 0>{});
            else if (!IMPL || scheme == 1) f(e, std::integral_constant<int, 1>{});
            else if constexpr (IMPL) f(e, std::integral_constant<int, 2>{});
        };
        const int e = ends();
        if (e == kInterior) {
            g(std::integral_constant<int, kInterior>{});
            return;
        }
        if constexpr (one_face(MODE)) {
            if (e == kWalls) {
                g(std::integral_constant<int, kWalls>{});
                return;
            }
            if (e == kRing) {
                g(std::integral_constant<int, kRing>{});
                return;
            }
        }
        g(std::integral_constant<int, kAny>{});
    }
};

// First sample after step0 as a step count of the launch: the smallest k >= 1
// with step0 + k > burn_in and (step0 + k) % every == 0 (clipped to 2^30).
__device__ __forceinline__ int first_sample(int64_t step0, int64_t burn_in, int32_t every)
{
    const int64_t a0 = (step0 > burn_in ? step0 : burn_in) + 1;
    const int64_t rm = a0 % every;
    const int64_t k = (rm == 0 ? a0 : a0 + (every - rm)) - step0;
    return k < (1 << 30) ? static_cast<int>(k) : (1 << 30);
}

// ------------------------------------------------------------------ every wave its own numbers

// CMAX: the largest cells per lane of the batch's waves: 4 alone, 4 and 8
// side by side, or 16 alone.  FP32 kernels that fit or nearly fit 64 VGPRs are kept
// to eight waves per SIMD, two workgroups of 1024 threads on a CU.
template <typename T, int CMAX, int MODE>
constexpr int rods_occupancy()
{
    return std::is_same<T, float>::value && (one_face(MODE) ? CMAX <= 8 : CMAX == 4) ? 8 : 4;
}

// Wait until the flags (LDS, one per wave of the instance) of waves a and b
// reach seq.  Every wave of the instance is resident and publishes seq before
// it waits for it, so the wait ends.
__device__ __forceinline__ void wait_flags(const int *flag, int a, int b, int seq)
{
    const int lane = threadIdx.x & 63;
    const int w = lane & 1 ? b : a;
    for (;;) {
        const int v = __hip_atomic_load(flag + w, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__all(v >= seq)) break;
        __builtin_amdgcn_s_sleep(1);
    }
}

// Wait until the flags of all nw waves of the instance reach seq.
__device__ __forceinline__ void wait_all(const int *flag, int nw, int seq)
{
    const int lane = threadIdx.x & 63;
    for (;;) {
        const int v = __hip_atomic_load(flag + min(lane, nw - 1), __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__all(v >= seq)) break;
        __builtin_amdgcn_s_sleep(1);
    }
}

// All nw waves of the instance meet (LDS and global accesses of each before it
// are seen by all after it).
__device__ __forceinline__ void inst_sync(int *flag, int lw, int nw, int seq)
{
    if (nw == 1) return;
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag + lw, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    wait_all(flag, nw, seq);
}

// Exchange step of wave_totals: lanes whose bit is set keep b and give a, the
// others keep a and give b; the value that lane `CTRL` (a DPP move) gives is added.
template <int CTRL>
__device__ __forceinline__ double keep_give(bool bit, double a, double b)
{
    const double give = sel(bit, a, b);
    return sel(bit, b, a) + dpp_shift<CTRL>(give, give);
}

// Sums of n = 8 or 16 values over the wave, that of x[q] in the lanes with
// lane % n = q: the lanes of a row halve the values they hold at each exchange, then
// the rows are added (16 values: 115 instructions; 16 scans take 288).  Every value
// is added in the same order of lanes (mirrors first: they pair the same lanes
// whichever of the two keeps the sum), so its bits do not depend on q.
template <int n>
__device__ __forceinline__ double wave_totals(const double (&x)[n])
{
    const int lane = threadIdx.x & 63;
    double y[8], z[4], w[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (n == 16) y[i] = keep_give<0x140>(lane & 8, x[i], x[i + 8]);               // row_mirror
        else y[i] = x[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = keep_give<0x141>(lane & 4, y[i], y[i + 4]);              // row_half_mirror
#pragma unroll
    for (int i = 0; i < 2; ++i) w[i] = keep_give<0xB1>(lane & 1, z[2 * i], z[2 * i + 1]);       // quad_perm 1 0 3 2
    double v = keep_give<0x4E>(lane & 2, w[0], w[1]);                                           // quad_perm 2 3 0 1
    if constexpr (n == 8) v += dpp_shift<0x128>(v, v);                                          // row_ror:8
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// The statistics of a launch's samples, from the sampled states that the waves of
// an instance left in the ring, at the launch's end: by then the registers of the
// steps are free and no wave waits for another at a sample.  Batches of kB
// samples; a lane takes whole cells (one load and store of their sums per batch)
// and forms its part of the kB spatial sums on the way (4 samples in the kernels of
// 64 registers, 8 in the others: more would spill).  With the statistics
// updated at each sample the kernels spilled up to 768 bytes per lane, and rods
// with 8 or 16 cells per lane updated their sums at a stride of as many doubles.
// Us per step with a sample every step (that form / now; every tenth step in
// brackets): FP32 moments 16 x 1000 cells 2.18 / 1.71 (0.86 / 0.80), 900 x 1000
// 6.5 / 3.4, 256 x 7800 55 / 6.9 (5.9 / 2.8); FP64 covariance 1 x 1000 6.2 / 2.3.
// Not gained: FP64 batches whose sampled states exceed the caches, 900 x 2000 with
// spatial sums only 13.5 / 16.7.
// bad: LDS, the first sample with a non-finite value (INT_MAX: none); red: LDS,
// [2][nw][16].  The multiply-adds are written out, so that a sample's share has the
// same bits in a full batch and in the last one.
template <typename T, int kB>
__device__ __forceinline__ void take_samples(const Inst1D &d, int inst, int lw, int nw, uint32_t clamps, T *gU,
                                             uint32_t mask, const Stats1D &st, const SampleRing &ring, InstAcc *acc,
                                             int *mflag, const int *bad, double *red)
{
    const int count = ring.count;
    auto count_clamps = [&]() {
        if (clamps) atomicAdd(reinterpret_cast<unsigned long long *>(&acc->clamp_count), static_cast<unsigned long long>(clamps));
    };
    if (count == 0) {
        count_clamps();
        return;
    }
    const int N = d.n, lane = threadIdx.x & 63;
    const bool dir = d.bc == 1;
    const int64_t n0 = acc->n_samples;
    // reference profile of the deviations: u0, or the linear wall profile
    const double ref0 = dir ? d.uL : d.u0, ref_slope = dir ? (d.uR - d.uL) / N : 0.0;
    const T *rows = static_cast<const T *>(ring.rows) + ring_first(d.off, inst) * ring.cap;
    const int stride = ring_row(N);
    int seq = 0;
    __threadfence_block();
    inst_sync(mflag, lw, nw, ++seq);  // the sampled states, the final state, n_samples and bad
    // a non-finite sample: keep the statistics as they were before it and freeze
    // the state there
    const int good = min(count, __builtin_amdgcn_readfirstlane(*bad));
    const bool moments = (mask & 1u) && st.s1 != nullptr;
    const bool corr = (mask & 2u) && d.x_off >= 0;
    const bool tcorr = (mask & 16u) && d.h_off >= 0;
    T *X = corr ? static_cast<T *>(st.xblk) + d.x_off + n0 % kCorrBlock * N : nullptr;  // (no launch goes beyond an X block)
    T *H = tcorr ? static_cast<T *>(st.hist) + d.h_off : nullptr;
    double *s1 = moments ? st.s1 + d.off : nullptr, *s2 = moments ? st.s2 + d.off : nullptr;
    double sp_mean = acc->sp_mean, sp_sq = acc->sp_sq, sp_var = acc->sp_var;
    for (int j0 = 0; j0 < good; j0 += kB) {
        const int nb = min(kB, good - j0);  // samples of the batch
        double x[2 * kB];
#pragma unroll
        for (int q = 0; q < 2 * kB; ++q) x[q] = 0.0;
        const T *u = rows + static_cast<int64_t>(j0) * stride;
        T *const Xb = corr ? X + static_cast<int64_t>(j0) * N : nullptr;
        const int h0 = tcorr ? static_cast<int>((n0 + j0) % st.hist_rows) : 0;
        auto cells = [&](auto full) __attribute__((always_inline)) {
            // kE cells at a time, their loads ahead of all
            constexpr int kE = kB == 8 ? 2 : 1;
            for (uint32_t i = 64 * lw + lane; i < static_cast<uint32_t>(N); i += 64 * nw * kE) {
                T v[kE][kB];
                double m1[kE], m2[kE];
#pragma unroll
                for (int e = 0; e < kE; ++e) {
                    const uint32_t c = i + 64 * nw * e, k = c < static_cast<uint32_t>(N) ? c : i;
#pragma unroll
                    for (int q = 0; q < kB; ++q) v[e][q] = (u + (full ? q : min(q, nb - 1)) * stride)[k];
                    m1[e] = moments ? s1[k] : 0.0;
                    m2[e] = moments ? s2[k] : 0.0;
                }
#pragma unroll
                for (int e = 0; e < kE; ++e) {
                    const uint32_t k = i + 64 * nw * e;
                    if (k >= static_cast<uint32_t>(N)) break;
                    const double ref = fma(ref_slope, k + 0.5, ref0);
#pragma unroll
                    for (int q = 0; q < kB; ++q)
                        if (full || q < nb) {
                            const double dl = static_cast<double>(v[e][q]) - ref;
                            x[q] += dl;
                            x[kB + q] = fma(dl, dl, x[kB + q]);
                            m1[e] += dl;
                            m2[e] = fma(dl, dl, m2[e]);
                            if (corr) (Xb + q * N)[k] = static_cast<T>(dl);
                            if (tcorr) (H + static_cast<int64_t>(h0 + q - (h0 + q >= st.hist_rows ? st.hist_rows : 0)) * N)[k] = static_cast<T>(dl);
                        }
                    if (moments) {
                        s1[k] = m1[e];
                        s2[k] = m2[e];
                    }
                }
            }
        };
        if (nb == kB) cells(std::true_type{});
        else cells(std::false_type{});
        double tot = wave_totals<2 * kB>(x);
        if (nw > 1) {
            // (the slots alternate: a wave writes a set again two meetings later)
            double *rd = red + (seq & 1) * 2 * kB * nw;
            if (lane < 2 * kB) rd[2 * kB * lw + lane] = tot;
            inst_sync(mflag, lw, nw, ++seq);
            if (lw == 0) {
                tot = 0.0;
                for (int w = 0; w < nw; ++w) tot += rd[2 * kB * w + (lane & (2 * kB - 1))];
            }
        }
        if (lw == 0) {
            tot /= N;
#pragma unroll
            for (int q = 0; q < kB; ++q)
                if (q < nb) {
                    const double a = of_lane(tot, q), b = of_lane(tot, kB + q);
                    sp_mean += a;
                    sp_sq += b;
                    sp_var += fma(-a, a, b);
                }
        }
    }
    if (good < count) {
        for (int i = 64 * lw + lane; i < N; i += 64 * nw) gU[i] = rows[static_cast<int64_t>(good) * stride + i];
    } else {
        count_clamps();
    }
    if (corr && good == count && n0 % kCorrBlock + count == kCorrBlock) {
        __threadfence_block();
        inst_sync(mflag, lw, nw, ++seq);
        xtx_block<T>(static_cast<const T *>(st.xblk) + d.x_off, st.c + d.c_off, N, lw, nw);
    }
    if (lw == 0 && lane == 0) {
        acc->sp_mean = sp_mean;
        acc->sp_sq = sp_sq;
        acc->sp_var = sp_var;
        acc->n_samples = n0 + good;
        if (good < count) acc->nonfinite = 1;
    }
}

// First unit (of CPL cells) of wave lw's own: nf faces in blocks of four over nw
// waves, the middle nbig of which ("big" waves, 8 cells per lane) take 124
// blocks each; the rest is shared evenly, a Dirichlet end wave, which needs no
// halo lane at its wall, taking one more.  Big waves start at even blocks.
template <int CPL>
__device__ __forceinline__ int rod_split(int nf, bool dir, int nw, int nbig, int lw)
{
    if (nbig == 0) {
        const int units = (nf + CPL - 1) / CPL;
        if (lw == 0) return 0;
        if (lw == nw) return units;
        return dir ? 1 + lw * (units - 2) / nw : lw * units / nw;
    }
    const int blocks = (nf + 3) / 4, small = nw - nbig, lo = small / 2;
    const int rest = blocks - 124 * nbig, even = (lo * rest / small) & ~1;
    int b = lw < lo ? lw * rest / small : even + 124 * (lw - lo);
    if (lw > lo + nbig) b = even + 124 * nbig + (lw - lo - nbig) * (rest - even) / (small - lo);
    return b / (CPL / 4);
}

// kB: the kernel's batch of samples (all waves of an instance must agree).
template <typename T, int CPL, bool STATS, int MODE, int kB>
__device__ __forceinline__ void rod_waves(const Seg1D seg, int wave, const Inst1D *__restrict__ tab, T *__restrict__ pool,
                                          const T *__restrict__ coef, int64_t step0, int32_t nsteps, int64_t burn_in,
                                          int32_t every, uint32_t mask, const Stats1D &st, const SampleRing &ring,
                                          unsigned char *lds)
{
    constexpr int S = CPL / 4;  // Philox calls of a lane per step
    const Inst1D d = tab[seg.inst];
    InstAcc *acc = st.acc + seg.inst;
    const int nw = seg.nw, lw = wave - seg.w0;
    // LDS of the instance (rod_lds): edge flags, meeting flags, first bad sample;
    // sums of a batch of samples; edges
    constexpr int HC = rod_edge(CPL);  // edge cells a wave publishes at either end
    int *eflag = reinterpret_cast<int *>(lds), *mflag = eflag + 16, *bad = eflag + 32;
    double *red = reinterpret_cast<double *>(lds + kRodFlags);               // [2][nw][16]
    T *edges = reinterpret_cast<T *>(lds + kRodFlags + 2 * nw * 16 * 8);  // [2][nw][first HC cells, last HC cells]

    // the wave's units: [s0, s1) of its own, on lanes own0 .., halo copies beside them
    const int N = d.n;
    const bool dir = d.bc == 1;
    const int s0 = rod_split<CPL>(dir ? N + 1 : N, dir, nw, seg.nbig, lw);
    const int s1 = rod_split<CPL>(dir ? N + 1 : N, dir, nw, seg.nbig, lw + 1);
    const bool part_u = !dir && N % CPL != 0;
    const int hl = nw == 1 || (dir && lw == 0) ? 0 : (part_u && lw == 0 ? 2 : 1);
    const int hr = nw == 1 || (dir && lw == nw - 1) ? 0 : 1;
    const int own0 = hl, own1 = hl + s1 - s0;
    Rod<T, CPL, MODE> rod;
    rod.init(d, coef, s0 - hl, own0, own1, own1 + hr - 1, nw == 1);
    const int lane = rod.lane;

    T *gU = pool + d.off;
    T u[CPL];
#pragma unroll
    for (int l = 0; l < CPL; ++l) u[l] = l < rod.nc && lane < own1 + hr ? gU[CPL * rod.unit + l] : T(0);

    if (lane < 33 && lw == 0) eflag[lane] = lane < 32 ? 0 : INT_MAX;
    __syncthreads();  // flags cleared, and the halo cells read before any wave writes its own back

    const PhiloxKey key = make_key(d.seed);
    const bool pc = d.scheme == 1;
    constexpr int kStages = CPL == 16 ? 16 : 4;  // a halo lasts this many (all waves of an instance alike)
    int left = pc ? kStages / 2 : kStages;       // steps it still lasts
    int seq = 0;
    T *row = static_cast<T *>(ring.rows) + ring_first(d.off, seg.inst) * ring.cap;  // where the next sampled state goes
    int taken = 0;
    int k_next = STATS ? first_sample(step0, burn_in, every) : (1 << 30);
    every = min(every, 1 << 29);  // sample steps beyond the launch: no overflow
    uint32_t clamps = 0;
    // Fresh halos: publish the first and the last cells of the wave's own,
    // draw the step's numbers meanwhile, then take the neighbours'.
    const int wl = lw == 0 ? nw - 1 : lw - 1, wr = lw == nw - 1 ? 0 : lw + 1;
    auto publish = [&]() __attribute__((always_inline)) {
        T *head = edges + ((seq & 1) * nw + lw) * (2 * HC), *tail = head + HC;
        ++seq;
        if (lane >= own0 && lane < own0 + HC / CPL) {
#pragma unroll
            for (int l = 0; l < CPL; ++l) head[(lane - own0) * CPL + l] = u[l];
        }
        if (lane < own1 && lane >= own1 - HC / CPL) {
#pragma unroll
            for (int l = 0; l < CPL; ++l) tail[HC - (own1 - lane) * CPL + l] = u[l];
        }
        if (lane == 0) __hip_atomic_store(eflag + lw, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto collect = [&]() __attribute__((always_inline)) {
        wait_flags(eflag, hl ? wl : lw, hr ? wr : lw, seq);
        if (lane < own0 || (hr && lane == own1)) {
            const T *eb = edges + ((seq - 1) & 1) * nw * (2 * HC);
            const T *src = lane == own1 ? eb + wr * (2 * HC) : eb + wl * (2 * HC) + 2 * HC - (own0 - lane) * CPL;
#pragma unroll
            for (int l = 0; l < CPL; ++l) u[l] = src[l];
        }
    };
    int k = 0;
    while (k < nsteps) {
        // the steps up to the next sample (or the end of the launch)
        const int k_end = min(nsteps, k_next);
        rod.by_kind(d.scheme, [&](auto ec, auto sc) __attribute__((always_inline)) {
            constexpr int E = decltype(ec)::value;
            constexpr bool PC = decltype(sc)::value == 1;
            constexpr int per = PC ? kStages / 2 : kStages;
            for (; k < k_end; ++k) {
                const bool fresh = nw > 1 && left == 0;
                if (fresh) {
                    publish();
                    left = per;
                }
                --left;
                const uint64_t n = static_cast<uint64_t>(step0 + k);
                T z[CPL];
                if (one_face(MODE) || rod.noise != 2) {
#pragma unroll
                    for (int s = 0; s < S; ++s) {
                        const Normals4<T> nz = block_normals<T, true>(static_cast<uint32_t>(S * rod.unit + s),
                                                                      static_cast<uint32_t>(n), ctr_word2(n, 0u),
                                                                      d.realisation, key);
#pragma unroll
                        for (int l = 0; l < 4; ++l) z[4 * s + l] = nz.z[l];
                    }
                } else {
#pragma unroll
                    for (int l = 0; l < CPL; ++l) z[l] = T(0);
                }
                // number of the right wall's face: the unit's own, or the next one's first
                T zN = T(0);
                if (E == kWalls) zN = from_right(T(0), z[0]);
                else if (E == kAny && dir) zN = rod.partial ? pick<T, CPL>(z, rod.m) : from_right(T(0), z[0]);
                if (fresh) collect();
                rod.template step<E, PC>(u, z, zN, clamps, NoSolve{});
            }
        });

        if (STATS && k == k_next) {
            k_next += every;
            bool finite = true;
#pragma unroll
            for (int l = 0; l < CPL; l += 4)
                if (rod.own && l < rod.nc) {  // (what goes beyond the last cell is in the row's pad)
                    typedef T vec __attribute__((ext_vector_type(4)));
                    *reinterpret_cast<vec *>(row + CPL * rod.unit + l) = vec{u[l], u[l + 1], u[l + 2], u[l + 3]};
                }
#pragma unroll
            for (int l = 0; l < CPL; ++l)
                if (rod.own && l < rod.nc) finite = finite && isfinite(u[l]);
            if (!__all(finite) && lane == 0) atomicMin(bad, taken);
            ++taken;
            row += ring_row(N);
        }
    }

#pragma unroll
    for (int l = 0; l < CPL; ++l)
        if (rod.own && l < rod.nc) gU[CPL * rod.unit + l] = u[l];
    if constexpr (STATS)
        take_samples<T, kB>(d, seg.inst, lw, nw, clamps, gU, mask, st, ring, acc, mflag, bad, red);
}

template <typename T, int CMAX, bool STATS, int MODE>
__global__ void __launch_bounds__(1024, (rods_occupancy<T, CMAX, MODE>()))
    k_rods(const Inst1D *__restrict__ tab, const Seg1D *__restrict__ segs, T *__restrict__ pool,
           const T *__restrict__ coef, int64_t step0, int32_t nsteps, int64_t burn_in, int32_t every, uint32_t mask,
           Stats1D st, SampleRing ring)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const Seg1D seg = segs[static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + wave];
    if (seg.inst < 0) return;                   // idle wave (barriers count the waves still running)
    if (st.acc[seg.inst].nonfinite) return;     // frozen after a non-finite sample
    unsigned char *lds = smem_raw + seg.lds;
    constexpr int kB = rods_occupancy<T, CMAX, MODE>() == 8 ? 4 : 8;
    if constexpr (CMAX == 8) {
        if (seg.cpl == 8) {
            rod_waves<T, 8, STATS, MODE, kB>(seg, wave, tab, pool, coef, step0, nsteps, burn_in, every, mask, st, ring,
                                            lds);
            return;
        }
    }
    rod_waves<T, CMAX == 16 ? 16 : 4, STATS, MODE, kB>(seg, wave, tab, pool, coef, step0, nsteps, burn_in, every, mask, st,
                                                   ring, lds);
}

// ------------------------------------------------------------------ implicit solve

// v of lane - S or lane + S (any value where that is no lane: its factor is 0).
template <int S>
__device__ __forceinline__ double lane_below(double v)
{
    if constexpr (S == 1) return from_left(v, v);
    else return __shfl_up(v, S, 64);
}

template <int S>
__device__ __forceinline__ double lane_above(double v)
{
    if constexpr (S == 1) return from_right(v, v);
    else return __shfl_down(v, S, 64);
}

// M x = d for the constant tridiagonal M = I - theta W A of an implicit rod, C
// consecutive cells per lane, in FP64.  Within a lane the rows are eliminated
// until cells 1 .. C-1 depend only on the left lane's last cell x_0 and the
// lane's own last one; the last cells then form a tridiagonal system of one row
// per lane, solved by cyclic reduction over the lanes (r -= k1 r(l - s) + k2 r(l
// + s), s = 1, 2, 4, ..), and the others follow.  The host forms all factors
// once (lane_factors); M is diagonally dominant, so k1 and k2 fall quadratically
// from level to level, and levels whose factors are below 2^-64 are left out.
// A periodic rod takes the Sherman-Morrison correction x -= f z of its cyclic
// part.  The factors stay in registers: a reduction through LDS over all cells,
// its factors read from L2 and two barriers per level, took 8.4 us per step of
// 1024 Crank-Nicolson rods of 256 cells at r = 2; this takes 0.90 (64 cells: 5.5,
// 0.75).  Bound by the chain of lane exchanges, one LDS-pipe permute pair each.
template <int C>
struct LaneSolve {
    double m[C], n[C], ib[C], p[C], q[C], z[C];  // in-lane elimination and substitution, cyclic vector
    double g, k1[6], k2[6], invb;
    double sq, sc;  // cyclic part: f = (x_0 + sq x_(N-1)) sc
    int levels, lg, ml;
    bool ring;

    __device__ __forceinline__ void load(const double *__restrict__ f, int nlev, bool periodic, int last_lane, int last)
    {
        const int lane = threadIdx.x & 63;
        levels = nlev;
        ring = periodic;
        lg = last_lane;
        ml = last;
        f += lane;
#pragma unroll
        for (int l = 0; l < C; ++l) {
            m[l] = f[64 * (0 * C + l)];
            n[l] = f[64 * (1 * C + l)];
            ib[l] = f[64 * (2 * C + l)];
            p[l] = f[64 * (3 * C + l)];
            q[l] = f[64 * (4 * C + l)];
            z[l] = f[64 * (5 * C + l)];
        }
        f += 64 * 6 * C;
        g = f[0];
        invb = f[64];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            k1[k] = f[64 * (2 + k)];
            k2[k] = f[64 * (8 + k)];
        }
        sq = f[64 * 14];
        sc = f[64 * 15];
    }

    template <int K>
    __device__ __forceinline__ void level(double &r) const
    {
        if (levels > K) r = fma(-k2[K], lane_above<(1 << K)>(r), fma(-k1[K], lane_below<(1 << K)>(r), r));
    }

    __device__ __forceinline__ void operator()(double (&x)[C]) const
    {
#pragma unroll
        for (int l = 1; l < C; ++l) x[l] = fma(-m[l], x[l - 1], x[l]);
#pragma unroll
        for (int l = C - 3; l >= 0; --l) x[l] = fma(-n[l], x[l + 1], x[l]);
        double r = x[C - 1];
        if constexpr (C > 1) r = fma(-g, from_right(x[0], x[0]), r);
        level<0>(r);
        level<1>(r);
        level<2>(r);
        level<3>(r);
        level<4>(r);
        level<5>(r);
        r *= invb;
        const double x0 = from_left(r, r);
#pragma unroll
        for (int l = 0; l < C - 1; ++l) x[l] = fma(-q[l], r, fma(-p[l], x0, x[l] * ib[l]));
        x[C - 1] = r;
        if (ring) {
            const double f = (of_lane(x[0], 0) + sq * of_lane(pick<double, C>(x, ml - 1), lg)) * sc;
#pragma unroll
            for (int l = 0; l < C; ++l) x[l] = fma(-f, z[l], x[l]);
        }
    }
};

// ------------------------------------------------------------------ numbers drawn ahead

// One instance per workgroup, CPL cells per lane of wave 0 (N <= 64 CPL; CPL 8
// for batches with implicit rods only).  The
// steps go in chunks of up to K.  While wave 0 advances chunk c with the
// numbers in one LDS buffer and leaves the sampled states in LDS, the other
// waves draw the numbers of chunk c + 1 into the other buffer, and wave 1 first
// adds the samples of chunk c - 1 to the statistics; one barrier per chunk.  A
// sample that completes an X block is the last of its chunk, so that every
// wave can join the contraction before the next sample's row is written.
//
// What bounds it: the dependent chain of wave 0, one wave on its SIMD; from four
// workgroups per CU on, VALU issue.  Four waves in FP32 draw faster than wave 0
// steps; FP64 numbers take about four times as long, so it has eight.
template <typename T, int CPL, bool STATS, int MODE>
__device__ __forceinline__ void rod_ahead(int inst, const Inst1D *__restrict__ tab, T *__restrict__ pool,
                                          const T *__restrict__ coef, const double *__restrict__ pcr, int64_t step0,
                                          int32_t nsteps, int64_t burn_in, int32_t every, uint32_t mask,
                                          const Stats1D &st, int32_t K, int32_t zrow, int32_t slots,
                                          unsigned char *smem_raw)
{
    const int W = blockDim.x >> 6, lane = threadIdx.x & 63;
    // Wave 0 advances the state.  The hardware starts successive workgroups of a
    // CU on successive SIMDs, so these waves do not share one (measured).
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const Inst1D d = tab[inst];
    InstAcc *acc = st.acc + inst;
    if (acc->nonfinite) return;  // frozen after a non-finite sample
    // LDS: frozen flags of even and odd chunks; numbers [2][K][zrow], pad; sampled states [2][slots][64 CPL]
    int *frozen = reinterpret_cast<int *>(smem_raw);
    T *zbuf = reinterpret_cast<T *>(smem_raw + 16);
    T *sbuf = zbuf + 2 * K * zrow + 64 * CPL + 4;  // reads a row ahead end in the pad
    const int N = d.n;
    const bool dir = d.bc == 1;
    const int nfg = ((dir ? N + 1 : N) + 3) >> 2;
    const uint32_t magic = ((1u << 20) + nfg - 1) / nfg;  // q / nfg for q nfg < 2^20
    const PhiloxKey key = make_key(d.seed);
    T *gU = pool + d.off;
    if (threadIdx.x < 2) frozen[threadIdx.x] = 0;

    // numbers of steps [k0, k0 + kc), this thread the tasks q0, q0 + dq, ...
    auto draw = [&](T *buf, int k0, int kc, int q0, int dq) __attribute__((always_inline)) {
        for (int q = q0; q < kc * nfg; q += dq) {
            const int kk = static_cast<int>((static_cast<uint32_t>(q) * magic) >> 20), g = q - kk * nfg;
            const uint64_t n = static_cast<uint64_t>(step0 + k0 + kk);
            Normals4<T> nz{};
            if (one_face(MODE) || d.noise != 2)
                nz = block_normals<T>(static_cast<uint32_t>(g), static_cast<uint32_t>(n), ctr_word2(n, 0u),
                                      d.realisation, key);
            T *p = buf + kk * zrow + 4 * g;
#pragma unroll
            for (int l = 0; l < 4; ++l) p[l] = nz.z[l];
        }
    };

    // The chunks, the same in every wave: up to K steps, `slots` samples, the
    // launch's end and the sample that completes an X block.
    const bool corr = STATS && (mask & 2u) && d.x_off >= 0;
    struct Chunk {
        int k, len, k_next, row, prev;  // steps done, length, next sample (steps), its X row, samples of the chunk before
        bool full;                      // those complete an X block
    } ck;
    const int32_t ev = min(every, 1 << 29);  // sample steps beyond the launch: no overflow
    auto chunk_len = [&](int k, int kn, int row) {
        int len = min(K, nsteps - k);
        if (STATS && corr) {
            const int64_t full = kn + static_cast<int64_t>(kCorrBlock - 1 - row) * ev;  // completes the block
            if (full < k + len) len = static_cast<int>(full) - k;
        }
        return len;
    };
    auto samples_in = [&](const Chunk &q) {
        return !STATS || q.k_next > q.k + q.len ? 0 : (q.k + q.len - q.k_next) / ev + 1;
    };
    auto after = [&](const Chunk &q) {
        Chunk r;
        r.prev = samples_in(q);
        r.k = q.k + q.len;
        r.k_next = q.k_next + r.prev * ev;
        r.row = (q.row + r.prev) % kCorrBlock;
        r.full = corr && r.prev > 0 && r.row == 0;
        r.len = chunk_len(r.k, r.k_next, r.row);
        return r;
    };
    ck.k = 0;
    ck.row = STATS ? static_cast<int>(acc->n_samples % kCorrBlock) : 0;
    ck.k_next = STATS ? first_sample(step0, burn_in, every) : (1 << 30);
    ck.prev = 0;
    ck.full = false;
    ck.len = chunk_len(0, ck.k_next, ck.row);

    // The chunk loop of a wave with its own part `work` (one loop per role, so
    // that each role holds only its own registers).  Returns whether the
    // instance froze.  With statistics an empty chunk follows the last one,
    // for the samples of that.
    auto chunks = [&](auto &&work) __attribute__((always_inline)) {
        for (int c = 0;; ++c) {
            const Chunk nx = after(ck);
            work(c, ck, nx);
            __threadfence_block();
            __syncthreads();
            if (STATS && frozen[c & 1]) return true;
            if (STATS && ck.full) {
                xtx_block<T>(static_cast<const T *>(st.xblk) + d.x_off, st.c + d.c_off, N, wave, W);
                __syncthreads();
            }
            if (STATS ? ck.len == 0 : nx.len == 0) return false;
            ck = nx;
        }
    };
    auto zb = [&](int c) { return zbuf + (c & 1) * K * zrow; };
    auto sb = [&](int c) { return sbuf + (c & 1) * slots * (64 * CPL); };
    auto draw_next = [&](int c, const Chunk &nx) __attribute__((always_inline)) {
        if (nx.len > 0) draw(zb(c + 1), nx.k, nx.len, (W - 1 - wave) * 64 + lane, 64 * (W - 1));
    };
    const int cell0 = CPL * lane, nc = N - cell0;

    draw(zbuf, 0, ck.len, threadIdx.x, blockDim.x);
    __syncthreads();
    if (wave == 0) {
        Rod<T, CPL, MODE> rod;
        const int units = (N + CPL - 1) / CPL;
        rod.init(d, coef, 0, 0, units, units - 1, true);
        typename std::conditional<implicit(MODE), LaneSolve<CPL>, NoSolve>::type solve;
        if constexpr (implicit(MODE)) {
            if (d.scheme >= 2) solve.load(pcr + d.p_off, d.pcr_levels, !dir, rod.lg, rod.m);
        }
        uint32_t clamps = 0;
        T u[CPL];
#pragma unroll
        for (int l = 0; l < CPL; ++l) u[l] = l < nc ? gU[cell0 + l] : T(0);
        // the steps of a chunk; sampled states go to out.  The next step's
        // numbers are read a step ahead of their use (past the chunk's last row
        // what is read is not used; the buffers are padded).
        auto advance = [&](auto ec, auto sc, const T *buf, T *out, const Chunk &q) __attribute__((always_inline)) {
            constexpr int E = decltype(ec)::value;
            constexpr int SCHEME = decltype(sc)::value;
            constexpr bool WN = E == kWalls || E == kAny;
            T za[CPL], zz[CPL], wa = T(0), wz = T(0);
            const T *p = buf + cell0, *pn = buf + N;
            auto load = [&](T (&z)[CPL], T &w) __attribute__((always_inline)) {
#pragma unroll
                for (int l = 0; l < CPL; ++l) z[l] = p[l];
                if (WN) w = *pn;
                p += zrow;
                pn += zrow;
            };
            load(za, wa);
            for (int kk = 0, ks = STATS ? q.k_next - q.k : (1 << 30); kk < q.len;) {
                // the steps up to the next sample (or the end of the chunk)
                const int ke = min(q.len, ks);
                for (; kk + 2 <= ke; kk += 2) {
                    load(zz, wz);
                    rod.template step<E, SCHEME>(u, za, wa, clamps, solve);
                    load(za, wa);
                    rod.template step<E, SCHEME>(u, zz, wz, clamps, solve);
                }
                if (kk < ke) {
                    load(zz, wz);
                    rod.template step<E, SCHEME>(u, za, wa, clamps, solve);
                    ++kk;
#pragma unroll
                    for (int l = 0; l < CPL; ++l) za[l] = zz[l];
                    wa = wz;
                }
                if (STATS && kk == ks) {
                    ks += ev;
#pragma unroll
                    for (int l = 0; l < CPL; ++l) out[cell0 + l] = u[l];
                    out += 64 * CPL;
                }
            }
        };
        const bool gone = chunks([&](int c, const Chunk &q, const Chunk &) __attribute__((always_inline)) {
            rod.by_kind(d.scheme, [&](auto ec, auto sc) __attribute__((always_inline)) { advance(ec, sc, zb(c), sb(c), q); });
        });
        if (gone) return;
#pragma unroll
        for (int l = 0; l < CPL; ++l)
            if (l < nc) gU[cell0 + l] = u[l];
        if (STATS && clamps) atomicAdd(reinterpret_cast<unsigned long long *>(&acc->clamp_count),
                                       static_cast<unsigned long long>(clamps));
        return;
    }
    if constexpr (STATS) {
        if (wave == 1) {
            const bool tcorr = (mask & 16u) && d.h_off >= 0;
            const bool moments = (mask & 1u) && st.s1 != nullptr;
            int64_t nsamp = acc->n_samples;
            double sp_mean = acc->sp_mean, sp_sq = acc->sp_sq, sp_var = acc->sp_var;
            double s1r[CPL], s2r[CPL];
#pragma unroll
            for (int l = 0; l < CPL; ++l) {
                s1r[l] = moments && l < nc ? st.s1[d.off + cell0 + l] : 0.0;
                s2r[l] = moments && l < nc ? st.s2[d.off + cell0 + l] : 0.0;
            }
            // reference profile of the deviations: u0, or the linear wall profile
            const double ref0 = dir ? d.uL : d.u0, ref_slope = dir ? (d.uR - d.uL) / N : 0.0;
            // the samples of a finished chunk, in order
            auto take = [&](const T *in, int count, int *flag) __attribute__((always_inline)) {
                for (int j = 0; j < count; ++j) {
                    double a = 0.0, b = 0.0;
                    int bad = 0;
                    T v[CPL];
                    double del[CPL];
                    T *X = corr ? static_cast<T *>(st.xblk) + d.x_off + (nsamp % kCorrBlock) * N : nullptr;
                    T *H = tcorr ? static_cast<T *>(st.hist) + d.h_off + (nsamp % st.hist_rows) * N : nullptr;
#pragma unroll
                    for (int l = 0; l < CPL; ++l) {
                        v[l] = in[j * (64 * CPL) + cell0 + l];
                        del[l] = static_cast<double>(v[l]) - fma(ref_slope, cell0 + l + 0.5, ref0);
                        if (l < nc) {
                            if (!isfinite(v[l])) bad = 1;
                            a += del[l];
                            b += del[l] * del[l];
                        }
                    }
                    a = wave_total(a);
                    b = wave_total(b);
                    if (__any(bad)) {
                        // a non-finite sample: keep the statistics as they were
                        // before it and freeze the state
#pragma unroll
                        for (int l = 0; l < CPL; ++l)
                            if (l < nc) gU[cell0 + l] = v[l];
                        if (lane == 0) {
                            acc->nonfinite = 1;
                            *flag = 1;
                        }
                        return;
                    }
#pragma unroll
                    for (int l = 0; l < CPL; ++l)
                        if (l < nc) {
                            s1r[l] += del[l];
                            s2r[l] += del[l] * del[l];
                            if (corr) X[cell0 + l] = static_cast<T>(del[l]);
                            if (tcorr) H[cell0 + l] = static_cast<T>(del[l]);
                        }
                    a /= N;
                    b /= N;
                    sp_mean += a;
                    sp_sq += b;
                    sp_var += b - a * a;
                    ++nsamp;
                }
            };
            (void)chunks([&](int c, const Chunk &q, const Chunk &nx) {
                if (q.prev > 0) take(sb(c + 1), q.prev, frozen + (c & 1));
                draw_next(c, nx);
            });
            if (moments) {
#pragma unroll
                for (int l = 0; l < CPL; ++l)
                    if (l < nc) {
                        st.s1[d.off + cell0 + l] = s1r[l];
                        st.s2[d.off + cell0 + l] = s2r[l];
                    }
            }
            if (lane == 0) {
                acc->n_samples = nsamp;
                acc->sp_mean = sp_mean;
                acc->sp_sq = sp_sq;
                acc->sp_var = sp_var;
            }
            return;
        }
    }
    (void)chunks([&](int c, const Chunk &, const Chunk &nx) { draw_next(c, nx); });
}

template <typename T, int CPL, bool STATS, int MODE>
__global__ void __launch_bounds__(512, CPL == 8 ? 2 : 4)
    k_rods_ahead(const Inst1D *__restrict__ tab, const Seg1D *__restrict__ segs, T *__restrict__ pool,
                 const T *__restrict__ coef, const double *__restrict__ pcr, int64_t step0, int32_t nsteps,
                 int64_t burn_in, int32_t every, uint32_t mask, Stats1D st, int32_t K, int32_t zrow, int32_t slots)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int inst = implicit(MODE) ? segs[blockIdx.x].inst : static_cast<int>(blockIdx.x);
    rod_ahead<T, CPL, STATS, MODE>(inst, tab, pool, coef, pcr, step0, nsteps, burn_in, every, mask, st, K, zrow, slots,
                                   smem_raw);
}

// The same where the implicit rods of a batch ask for different counts of cells
// per lane, CMAX the largest: each rod takes that of its own length.  The order of
// its elimination, and so its last bits, follows from that split, and taken from
// the longest rod it would make a rod's field depend on the others.  (Explicit rods
// have the same bits with any split.)  Us per step, CMAX's split for every rod
// with material coefficients in registers / each its own without, Crank-Nicolson at
// r = 2: 700 rods of 3 to 256 cells FP32 0.96 / 0.88, FP64 2.96 / 1.51; of 3 to 512
// cells 1.92 / 1.65 and 4.5 / 2.2.  A kernel with one split holds its factors in
// fewer registers (1024 rods of 256 cells with statistics, FP64, material
// coefficients: 3.4, 4.3 with this one) and serves the batches it can.
template <typename T, int CMAX, bool STATS, int MODE>
__global__ void __launch_bounds__(512, CMAX == 8 ? 2 : 4)
    k_rods_mixed(const Inst1D *__restrict__ tab, const Seg1D *__restrict__ segs, T *__restrict__ pool,
                 const T *__restrict__ coef, const double *__restrict__ pcr, int64_t step0, int32_t nsteps,
                 int64_t burn_in, int32_t every, uint32_t mask, Stats1D st, int32_t K, int32_t zrow, int32_t slots)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const Seg1D seg = segs[blockIdx.x];
    auto run = [&](auto cpl) __attribute__((always_inline)) {
        rod_ahead<T, decltype(cpl)::value, STATS, MODE>(seg.inst, tab, pool, coef, pcr, step0, nsteps, burn_in, every, mask,
                                                        st, K, zrow, slots, smem_raw);
    };
    if (seg.cpl == 1) {
        run(std::integral_constant<int, 1>{});
        return;
    }
    if constexpr (CMAX > 2) {
        if (seg.cpl == 2) {
            run(std::integral_constant<int, 2>{});
            return;
        }
    }
    if constexpr (CMAX > 4) {
        if (seg.cpl == 4) {
            run(std::integral_constant<int, 4>{});
            return;
        }
    }
    run(std::integral_constant<int, CMAX>{});
}

// ------------------------------------------------------------------ typed launchers

template <typename T, bool STATS, int MODE>
static hipError_t rods_m(const Launch1D &a)
{
#define SHE_RODS(C)                                                                                              \
    hipLaunchKernelGGL((k_rods<T, C, STATS, MODE>), dim3(a.n_blocks), dim3(a.block), a.smem, a.s, a.tab, a.segs, \
                       static_cast<T *>(a.pool), static_cast<const T *>(a.coef), a.step0, a.nsteps, a.burn_in,   \
                       a.every, a.mask, a.st, a.ring)
    switch (a.cpl) {
    case 4: SHE_RODS(4); break;
    case 8: SHE_RODS(8); break;
    case 16:
        if constexpr (std::is_same<T, float>::value) {
            SHE_RODS(16);
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
#undef SHE_RODS
    return hipGetLastError();
}

#define SHE_AHEAD_K(KERNEL)                                                                                  \
    hipLaunchKernelGGL(KERNEL, dim3(a.n_blocks), dim3(a.block), a.smem, a.s, a.tab, a.segs,                  \
                       static_cast<T *>(a.pool), static_cast<const T *>(a.coef), a.pcr, a.step0, a.nsteps,   \
                       a.burn_in, a.every, a.mask, a.st, a.ahead, a.zrow, a.slots)

template <typename T, bool STATS, int MODE>
static hipError_t mixed_m(const Launch1D &a)
{
    switch (a.cpl) {
    case 2: SHE_AHEAD_K((k_rods_mixed<T, 2, STATS, MODE>)); break;
    case 4: SHE_AHEAD_K((k_rods_mixed<T, 4, STATS, MODE>)); break;
    case 8: SHE_AHEAD_K((k_rods_mixed<T, 8, STATS, MODE>)); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, bool STATS, int MODE>
static hipError_t ahead_m(const Launch1D &a)
{
#define SHE_AHEAD(C) SHE_AHEAD_K((k_rods_ahead<T, C, STATS, MODE>))
    switch (a.cpl) {
    case 1: SHE_AHEAD(1); break;
    case 2: SHE_AHEAD(2); break;
    case 4: SHE_AHEAD(4); break;
    case 8:
        if constexpr (implicit(MODE)) {
            SHE_AHEAD(8);
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
#undef SHE_AHEAD
    return hipGetLastError();
}

template <typename T, int MODE>
hipError_t rods_mixed_t(const Launch1D &a)
{
    return a.stats ? mixed_m<T, true, MODE>(a) : mixed_m<T, false, MODE>(a);
}

// Each in a unit of its own per state type, mode and kernel (they compile in parallel).
template <typename T, int MODE, bool AHEAD>
hipError_t rods_t(const Launch1D &a)
{
    if constexpr (AHEAD) return a.stats ? ahead_m<T, true, MODE>(a) : ahead_m<T, false, MODE>(a);
    else return a.stats ? rods_m<T, true, MODE>(a) : rods_m<T, false, MODE>(a);
}

}  // namespace she
