// 1D batches: the step kernel of the long instances of batches with implicit
// ones, the time correlation, initial state, finalisation, batch means and the
// verification kernels.  All others step in she_step_1d.hpp, whose comment states
// the scheme.
//
// Implicit schemes (backward Euler theta = 1, Crank-Nicolson theta = 1/2;
// the implicit-scheme exercise, Sec. 6): the flux pass weights the
// state-dependent deterministic flux by 1 - theta, giving the right-hand side
// U + W [(1 - theta) A U + b + noise]; M = I - theta W A is constant, so the
// host precomputes in FP64 the factors of parallel cyclic reduction (log2 N
// levels of d_i -= k1 d_(i-s) + k2 d_(i+s), then d_i / b_i) and, for periodic
// rods, the Sherman-Morrison vector of the cyclic part.  The reduction runs in
// FP64 for either state type (an FP64 array in LDS), so only the final state
// is rounded: rounded factors would bias the conserved sum a little every step.
//
// Statistics on sample steps: per-cell FP64 sums of dU and dU^2 kept in
// registers for the whole launch, spatial sums reduced over the instance, and
// (optionally) the shifted state written as one row of a 256-row X block;
// a full block is contracted on the matrix cores, C += X^T X, with
// v_mfma_f32_16x16x4f32 (FP32 state) or v_mfma_f64_16x16x4f64 (FP64 state),
// and added to the FP64 N x N sum.  For the time correlation each sample row
// also goes to a per-instance history ring; after the launch, k_tcorr adds the
// lag products of the new rows (one thread per cell and lag, FP64).
#include "she_step_1d.hpp"

namespace she {

// Value of the last of the first `m` (1..4) entries, chosen among values
// (a select of array elements as lvalues would become an address select and
// move the array to private memory).
template <typename T>
__device__ __forceinline__ T last_of(int m, T a0, T a1, T a2, T a3)
{
    return m >= 4 ? a3 : (m == 3 ? a2 : (m == 2 ? a1 : a0));
}

// The instances above kRodAlone cells of a batch with an implicit one (explicit and
// composite ones may be among them; the others, and explicit batches, run the wave
// kernels of she_step_1d.hpp).
//
// Thread t of an instance's waves owns Philox blocks g = t + s TS (s < MAXG,
// TS the instance's thread count): the faces 4g..4g+3 and the cells 4g..4g+3,
// whose values stay in registers.  A stage (the FE step, or either half of a
// PC step) publishes each block's first and last cell value (and, once per
// step, the number of its face 4g) in LDS, passes one barrier, reads the
// values next to its block and computes five fluxes: its own four faces and
// the face after its last cell, which the next block computes as its face 0
// as well (same inputs, same code, so the two agree bit for bit and the sum
// is conserved).  The exchange arrays alternate between two buffers, so one
// barrier per stage suffices.
template <typename T, int BLOCK, int MAXG, bool STATS>
__device__ __forceinline__ void step1d_body(const Inst1D *__restrict__ tab, const Seg1D *__restrict__ segs,
                                            T *__restrict__ pool, const T *__restrict__ coef,
                                            const double *__restrict__ pcr, int64_t step0, int32_t nsteps,
                                            int64_t burn_in, int32_t every, uint32_t mask, Stats1D st)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const Seg1D seg = segs[static_cast<int64_t>(blockIdx.x) * (BLOCK / 64) + wave];
    if (seg.inst < 0) return;  // idle wave (barriers count the waves still running)
    const int inst = seg.inst;
    const Inst1D d = tab[inst];
    InstAcc *acc = st.acc + inst;
    if (acc->nonfinite) return;  // frozen after a non-finite sample

    const int N = d.n;
    const bool dir = d.bc == 1;
    const int nf = dir ? N + 1 : N;
    const int nfg = (nf + 3) >> 2, nfgp = (nfg + 3) & ~3;
    const int glast = (N - 1) >> 2;  // block of the last cell
    const int TS = 64 * seg.nw;
    const int t = static_cast<int>(threadIdx.x) - 64 * seg.w0;
    const int lw = wave - seg.w0;
    const SegLds lay = seg_lds(N, nf, static_cast<int32_t>(sizeof(T)), 2);
    unsigned char *base = smem_raw + seg.lds;
    T *xch = reinterpret_cast<T *>(base + lay.xch);
    double *red = reinterpret_cast<double *>(base + lay.red);  // [3][16] wave sums of a sample
    T *Rf = reinterpret_cast<T *>(base + lay.rf);  // VARC: conductance per face (periodic: [N] = [0])
    T *Sf = reinterpret_cast<T *>(base + lay.sf);  // VARC: noise factor per face (walls: sqrt 2 included)
    T *Wc = reinterpret_cast<T *>(base + lay.wc);  // VARC: capacity factor per cell
    double *PD = reinterpret_cast<double *>(base + lay.pd);  // implicit: FP64 reduction array

    const T r = static_cast<T>(d.r);
    const T sg = static_cast<T>(d.sigma);
    const T sgw = static_cast<T>(d.sigma * 1.41421356237309504880);
    const T uL = static_cast<T>(d.uL), uR = static_cast<T>(d.uR), u0 = static_cast<T>(d.u0);
    const int eq = d.eq, noise = d.noise;
    const T nu = static_cast<T>(eq == 2 ? d.nu : 0.0);  // Burgers hyperbolic flux nu c_f (1 - c_f)
    const PhiloxKey key = make_key(d.seed);
    T *gU = pool + d.off;

    T u[MAXG][4];
#pragma unroll
    for (int s = 0; s < MAXG; ++s)
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int i = 4 * (t + s * TS) + l;
            u[s][l] = i < N ? gU[i] : T(0);
        }
    if (d.k_off >= 0) {
        const T *k = coef + d.k_off;
        for (int f = t; f < nf; f += TS) {
            Rf[f] = k[f];
            Sf[f] = k[nf + f];
        }
        for (int i = t; i < N; i += TS) Wc[i] = k[2 * nf + i];
        if (!dir && t == 0) {
            Rf[N] = k[0];
            Sf[N] = k[nf];
        }
    } else {
        for (int f = t; f < nf; f += TS) {
            Rf[f] = r;
            Sf[f] = (dir && (f == 0 || f == N)) ? sgw : sg;
        }
        for (int i = t; i < N; i += TS) Wc[i] = T(1);
        if (!dir && t == 0) {
            Rf[N] = r;
            Sf[N] = sg;
        }
    }

    // wall amplitudes (deterministic)
    uint32_t clamps = 0;
    const T amp_uL = face_amp<T>(eq, uL, clamps);
    const T amp_uR = face_amp<T>(eq, uR, clamps);
    clamps = 0;

    // Per-cell sums of dU and dU^2: in registers for the launch with one
    // Philox block per thread; with more, updated in memory on each sample
    // (registers for the stage matter more there: they set how many
    // workgroups of a packed batch are resident at once).
    constexpr bool kRegSums = MAXG == 1;
    double s1[MAXG][4], s2[MAXG][4];
    const bool moments = STATS && (mask & 1u) && st.s1 != nullptr;
    const bool corr = STATS && (mask & 2u) && d.x_off >= 0;
    const bool tcorr = STATS && (mask & 16u) && d.h_off >= 0;
    int64_t nsamp = STATS ? acc->n_samples : 0;
    // spatial sums of the instance, carried in registers over the launch
    double sp_mean = STATS ? acc->sp_mean : 0.0, sp_sq = STATS ? acc->sp_sq : 0.0,
           sp_var = STATS ? acc->sp_var : 0.0;
    // first sample of the launch: the smallest t > burn_in, t > step0 with
    // t % every == 0 (t = steps completed); later ones follow every `every`
    int64_t t_next = -1;
    if (STATS && every > 0) {
        const int64_t a0 = (step0 > burn_in ? step0 : burn_in) + 1;
        const int64_t rm = a0 % every;
        t_next = rm == 0 ? a0 : a0 + (every - rm);
    }
    // reference profile of the deviations: u0, or the linear wall profile
    const double ref0 = dir ? d.uL : d.u0, ref_slope = dir ? (d.uR - d.uL) / N : 0.0;
#pragma unroll
    for (int s = 0; s < MAXG; ++s)
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int i = 4 * (t + s * TS) + l;
            s1[s][l] = (kRegSums && moments && i < N) ? st.s1[d.off + i] : 0.0;
            s2[s][l] = (kRegSums && moments && i < N) ? st.s2[d.off + i] : 0.0;
        }
    __syncthreads();

    // implicit schemes: weight of the state-dependent deterministic flux
    const bool impl = d.scheme >= 2;
    const T ex = static_cast<T>(impl ? 1.0 - d.theta : 1.0);
    // face kinds: 0 heat with instantaneous noise; 1 deterministic or no
    // noise (any equation); 2 Dean-Kawasaki; 3 Burgers (both instantaneous)
    const int kind = noise != 0 ? 1 : (eq == 0 ? 0 : eq + 1);

    int ph = 0;  // exchange buffer of the next stage
    // Flux divergence dv of the state V (registers) for every owned cell.
    // first: the stage that also exchanges the face-0 numbers (rnz: the
    // number of the face after each block, kept for the second PC stage).
    auto stage = [&](const T (&V)[MAXG][4], const T (&z)[MAXG][4], T (&rnz)[MAXG], T (&dv)[MAXG][4],
                     bool first) __attribute__((always_inline)) {
        T *Uf = xch + (3 * ph) * nfgp, *Ul = Uf + nfgp, *Zf = Ul + nfgp;
        ph ^= 1;
#pragma unroll
        for (int s = 0; s < MAXG; ++s) {
            const int g = t + s * TS;
            if (g < nfg) {
                const int nc = N - 4 * g;
                Uf[g] = V[s][0];
                Ul[g] = last_of<T>(nc, V[s][0], V[s][1], V[s][2], V[s][3]);
                if (first) Zf[g] = z[s][0];
            }
        }
        __syncthreads();
        auto faces = [&](auto kc) __attribute__((always_inline)) {
            constexpr int K = decltype(kc)::value;
#pragma unroll
            for (int s = 0; s < MAXG; ++s) {
                const int g = t + s * TS;
                const int nc = N - 4 * g;  // cells from this block's first on
                if (nc <= 0) continue;     // no cells (a Dirichlet block holding only face N)
                const bool inner = nc > 4;
                const T lnb = Ul[g == 0 ? glast : g - 1];
                const T left = (dir && g == 0) ? uL : lnb;
                const T rnb = Uf[inner ? g + 1 : 0];
                const T right = (dir && !inner) ? uR : rnb;
                if (first) {
                    const T zn = Zf[inner || (dir && nc == 4) ? g + 1 : 0];
                    // Dirichlet, N not a multiple of 4: face N is this block's own
                    rnz[s] = (dir && nc < 4) ? last_of<T>(nc + 1, z[s][0], z[s][1], z[s][2], z[s][3]) : zn;
                }
                T lo[5], hi[5], zz[5];
                lo[0] = left;
#pragma unroll
                for (int l = 0; l < 4; ++l) {
                    lo[l + 1] = V[s][l];
                    hi[l] = V[s][l];
                    zz[l] = z[s][l];
                }
                hi[4] = right;
                zz[4] = rnz[s];
                if (nc < 4) {  // the block of the last cell when 4 does not divide N
#pragma unroll
                    for (int l = 1; l < 4; ++l)
                        if (l >= nc) {
                            hi[l] = right;
                            zz[l] = rnz[s];
                        }
                }
                T F[5];
#pragma unroll
                for (int l = 0; l < 5; ++l) {
                    const int f = 4 * g + l;
                    const T rf = Rf[f] * ex;
                    const T sf = Sf[f];
                    const T df = hi[l] - lo[l];
                    const T cf = T(0.5) * (lo[l] + hi[l]);
                    // clamps are counted on the faces this block owns
                    const bool own = l < 4 && l < nc && !(dir && f == 0);
                    if constexpr (K == 0) {
                        F[l] = fma(sf * cf, zz[l], rf * df);
                    } else if constexpr (K == 1) {
                        T am = T(0);
                        if (noise == 1) {
                            const T v = dir ? uL + (uR - uL) * static_cast<T>(f) / static_cast<T>(N) : u0;
                            uint32_t c = 0;
                            am = face_amp<T>(eq, v, c);
                            if (own) clamps += c;
                        }
                        F[l] = fma(sf * am, zz[l], fma(-nu * cf, T(1) - cf, rf * df));
                    } else if constexpr (K == 2) {
                        const bool neg = cf < T(0);
                        if (own && neg) ++clamps;
                        const T am = neg ? T(0) : amp_sqrt(cf);
                        F[l] = fma(sf * am, zz[l], rf * df);
                    } else {
                        const T q = cf * (T(1) - cf);
                        const bool neg = q < T(0);
                        if (own && neg) ++clamps;
                        const T am = neg ? T(0) : amp_sqrt(q);
                        F[l] = fma(sf * am, zz[l], fma(-nu, q, rf * df));
                    }
                }
                if (dir) {
                    // walls: F_0 = 2 r (U_0 - U_L) + sqrt 2 sigma A(U_L) N_0, mirrored at
                    // face N (the state term weighted by 1 - theta in implicit schemes)
                    if (g == 0) {
                        const T rw = Rf[0];
                        const T sw = Sf[0];
                        const T dwl = fma(-nu * uL, T(1) - uL, T(2) * rw * (ex * V[s][0] - uL));
                        F[0] = noise != 2 ? fma(sw * amp_uL, zz[0], dwl) : dwl;
                    }
                    if (!inner) {
                        const int m = nc < 4 ? nc : 4;
                        const T vl = last_of<T>(m, V[s][0], V[s][1], V[s][2], V[s][3]);
                        const T rw = Rf[N];
                        const T sw = Sf[N];
                        const T dwr = fma(-nu * uR, T(1) - uR, T(2) * rw * (uR - ex * vl));
                        const T w = noise != 2 ? fma(sw * amp_uR, rnz[s], dwr) : dwr;
#pragma unroll
                        for (int l = 1; l < 5; ++l)
                            if (l == m) F[l] = w;
                    }
                }
#pragma unroll
                for (int l = 0; l < 4; ++l) dv[s][l] = cell_flux(Wc[4 * g + l], F[l + 1] - F[l]);
            }
        };
        switch (kind) {
        case 0: faces(std::integral_constant<int, 0>{}); break;
        case 1: faces(std::integral_constant<int, 1>{}); break;
        case 2: faces(std::integral_constant<int, 2>{}); break;
        default: faces(std::integral_constant<int, 3>{}); break;
        }
    };

    for (int k = 0; k < nsteps; ++k) {
        const uint64_t n = static_cast<uint64_t>(step0 + k);
        T z[MAXG][4];
#pragma unroll
        for (int s = 0; s < MAXG; ++s) {
            const int g = t + s * TS;
            if (noise != 2 && g < nfg) {
                const Normals4<T> nz = block_normals<T, true>(static_cast<uint32_t>(g), static_cast<uint32_t>(n),
                                                              ctr_word2(n, 0u), d.realisation, key);
#pragma unroll
                for (int l = 0; l < 4; ++l) z[s][l] = nz.z[l];
            } else {
#pragma unroll
                for (int l = 0; l < 4; ++l) z[s][l] = T(0);
            }
        }
        T rnz[MAXG], dv[MAXG][4];
#pragma unroll
        for (int s = 0; s < MAXG; ++s) rnz[s] = T(0);
        stage(u, z, rnz, dv, true);
        if (impl) {
            // right-hand side in FP64, then M U' = rhs by parallel cyclic
            // reduction in the FP64 LDS array (same cells per thread)
            double x[MAXG][4];
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) {
                    const int i = 4 * (t + s * TS) + l;
                    x[s][l] = static_cast<double>(u[s][l] + dv[s][l]);
                    if (i < N) PD[i] = x[s][l];
                }
            const double *P = pcr + d.p_off;
            const int L = d.pcr_levels;
            // factors of the current level in registers; the next level's are
            // loaded before this level's barriers so their latency overlaps
            double f1[MAXG][4], f2[MAXG][4];
            auto load_level = [&](int lv, double (&a)[MAXG][4], double (&b)[MAXG][4]) __attribute__((always_inline)) {
                const double *k1 = P + static_cast<int64_t>(lv) * N, *k2 = P + static_cast<int64_t>(L + lv) * N;
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        a[s][l] = i < N ? k1[i] : 0.0;
                        b[s][l] = i < N ? k2[i] : 0.0;
                    }
            };
            if (L > 0) load_level(0, f1, f2);
            __syncthreads();
            for (int lv = 0; lv < L; ++lv) {
                const int sh = 1 << lv;
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        if (i < N) {
                            double v = PD[i];
                            if (i >= sh) v -= f1[s][l] * PD[i - sh];
                            if (i + sh < N) v -= f2[s][l] * PD[i + sh];
                            x[s][l] = v;
                        }
                    }
                if (lv + 1 < L) load_level(lv + 1, f1, f2);
                __syncthreads();
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        if (i < N) PD[i] = x[s][l];
                    }
                __syncthreads();
            }
            const double *invb = P + static_cast<int64_t>(2 * L) * N;
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) {
                    const int i = 4 * (t + s * TS) + l;
                    if (i < N) x[s][l] *= invb[i];
                }
            if (!dir) {
                // cyclic part: x = y - f z, f = (y_0 + q y_(N-1)) / (1 + z_0 + q z_(N-1))
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        if (i < N) PD[i] = x[s][l];
                    }
                __syncthreads();
                const double *zv = invb + N;
                const double f = (PD[0] + zv[N] * PD[N - 1]) * zv[N + 1];
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        if (i < N) x[s][l] -= f * zv[i];
                    }
            }
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) u[s][l] = static_cast<T>(x[s][l]);
        } else if (d.scheme == 0) {
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) u[s][l] = u[s][l] + dv[s][l];
        } else {
            T us[MAXG][4];
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) us[s][l] = u[s][l] + dv[s][l];
            stage(us, z, rnz, dv, false);
#pragma unroll
            for (int s = 0; s < MAXG; ++s)
#pragma unroll
                for (int l = 0; l < 4; ++l) u[s][l] = T(0.5) * ((u[s][l] + us[s][l]) + dv[s][l]);
        }

        if (STATS) {
            if (step0 + k + 1 == t_next) {
                t_next += every;
                double a = 0.0, b = 0.0;
                int bad = 0;
                double del[MAXG][4];
                const int row = static_cast<int>(nsamp % kCorrBlock);
                T *X = corr ? static_cast<T *>(st.xblk) + d.x_off : nullptr;
                T *Hrow = tcorr ? static_cast<T *>(st.hist) + d.h_off + (nsamp % st.hist_rows) * N : nullptr;
#pragma unroll
                for (int s = 0; s < MAXG; ++s)
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        const int i = 4 * (t + s * TS) + l;
                        del[s][l] = 0.0;
                        if (i < N) {
                            const T v = u[s][l];
                            if (!isfinite(v)) bad = 1;
                            const double dl = static_cast<double>(v) - fma(ref_slope, i + 0.5, ref0);
                            del[s][l] = dl;
                            a += dl;
                            b += dl * dl;
                            if (corr) X[(int64_t)row * N + i] = static_cast<T>(dl);
                            if (tcorr) Hrow[i] = static_cast<T>(dl);
                        }
                    }
                // sums over the instance (fixed order): DPP within each wave,
                // then (several waves) the wave sums through LDS, added by every
                // thread in the same order
                a = wave_total(a);
                b = wave_total(b);
                bad = __any(bad) ? 1 : 0;
                if (seg.nw > 1) {
                    if ((t & 63) == 0) {
                        red[lw] = a;
                        red[16 + lw] = b;
                        red[32 + lw] = static_cast<double>(bad);
                    }
                    __syncthreads();
                    a = b = 0.0;
                    bad = 0;
                    for (int w = 0; w < seg.nw; ++w) {
                        a += red[w];
                        b += red[16 + w];
                        bad |= red[32 + w] != 0.0;
                    }
                }
                if (bad) {
                    // a non-finite sample: keep the statistics as they were
                    // before it and freeze the state
#pragma unroll
                    for (int s = 0; s < MAXG; ++s)
#pragma unroll
                        for (int l = 0; l < 4; ++l) {
                            const int i = 4 * (t + s * TS) + l;
                            if (i < N) {
                                gU[i] = u[s][l];
                                if (kRegSums && moments) {
                                    st.s1[d.off + i] = s1[s][l];
                                    st.s2[d.off + i] = s2[s][l];
                                }
                            }
                        }
                    if (t == 0) {
                        acc->nonfinite = 1;
                        acc->n_samples = nsamp;
                        acc->sp_mean = sp_mean;
                        acc->sp_sq = sp_sq;
                        acc->sp_var = sp_var;
                    }
                    return;
                }
                a /= N;
                b /= N;
                sp_mean += a;
                sp_sq += b;
                sp_var += b - a * a;
                if (kRegSums) {
#pragma unroll
                    for (int s = 0; s < MAXG; ++s)
#pragma unroll
                        for (int l = 0; l < 4; ++l) {
                            s1[s][l] += del[s][l];
                            s2[s][l] += del[s][l] * del[s][l];
                        }
                } else if (moments) {
#pragma unroll
                    for (int s = 0; s < MAXG; ++s)
#pragma unroll
                        for (int l = 0; l < 4; ++l) {
                            const int i = 4 * (t + s * TS) + l;
                            if (i < N) {
                                st.s1[d.off + i] += del[s][l];
                                st.s2[d.off + i] += del[s][l] * del[s][l];
                            }
                        }
                }
                ++nsamp;
                if (corr && row == kCorrBlock - 1) {
                    __threadfence_block();
                    __syncthreads();
                    xtx_block<T>(X, st.c + d.c_off, N, lw, seg.nw);
                    __syncthreads();
                }
            }
        }
    }

#pragma unroll
    for (int s = 0; s < MAXG; ++s)
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int i = 4 * (t + s * TS) + l;
            if (i < N) gU[i] = u[s][l];
        }
    if (kRegSums && moments) {
#pragma unroll
        for (int s = 0; s < MAXG; ++s)
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const int i = 4 * (t + s * TS) + l;
                if (i < N) {
                    st.s1[d.off + i] = s1[s][l];
                    st.s2[d.off + i] = s2[s][l];
                }
            }
    }
    if (STATS) {
        if (clamps) atomicAdd(reinterpret_cast<unsigned long long *>(&acc->clamp_count),
                              static_cast<unsigned long long>(clamps));
        if (t == 0) {
            acc->n_samples = nsamp;
            acc->sp_mean = sp_mean;
            acc->sp_sq = sp_sq;
            acc->sp_var = sp_var;
        }
    }
}

template <typename T, int BLOCK, int MAXG, bool STATS>
__global__ void __launch_bounds__(BLOCK)
    k_step1d(const Inst1D *__restrict__ tab, const Seg1D *__restrict__ segs, T *__restrict__ pool,
             const T *__restrict__ coef, const double *__restrict__ pcr, int64_t step0, int32_t nsteps,
             int64_t burn_in, int32_t every, uint32_t mask, Stats1D st)
{
    step1d_body<T, BLOCK, MAXG, STATS>(tab, segs, pool, coef, pcr, step0, nsteps, burn_in, every, mask, st);
}

// ------------------------------------------------------------------ time correlation

// grid: (ceil(nmax L / 256), n_inst); thread (m, i) with i fastest, so the
// ring rows are read coalesced.  Sample n sits in ring row n mod hist_rows;
// the host keeps each launch's new samples plus L - 1 older ones in the ring.
template <typename T>
__global__ void __launch_bounds__(256)
    k_tcorr(const Inst1D *__restrict__ tab, const T *__restrict__ hist, int32_t hist_rows, int32_t lags, int64_t n0,
            int64_t count, double *__restrict__ tc, const InstAcc *__restrict__ acc)
{
    const int inst = blockIdx.y;
    const Inst1D d = tab[inst];
    if (d.h_off < 0) return;
    const int N = d.n;
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= static_cast<int64_t>(N) * lags) return;
    const int i = static_cast<int>(e % N), m = static_cast<int>(e / N);
    const int64_t n1 = min(n0 + count, acc[inst].n_samples);  // a frozen instance stopped sampling
    const int64_t nb = max(n0, static_cast<int64_t>(m));
    if (nb >= n1) return;
    const T *h = hist + d.h_off + i;
    int64_t a = nb % hist_rows, b = (nb - m) % hist_rows;
    double sum = 0.0;
    for (int64_t n = nb; n < n1; ++n) {
        sum += static_cast<double>(h[a * N]) * static_cast<double>(h[b * N]);
        if (++a == hist_rows) a = 0;
        if (++b == hist_rows) b = 0;
    }
    tc[d.tc_off + static_cast<int64_t>(m) * N + i] += sum;
}

__global__ void __launch_bounds__(256)
    k_fin_tc(int n, int lags, const double *__restrict__ s1, const double *__restrict__ tc, int64_t M,
             double *__restrict__ out)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= static_cast<int64_t>(n) * lags) return;
    const int i = static_cast<int>(e % n), m = static_cast<int>(e / n);
    if (M <= m) {
        out[e] = __builtin_nan("");
        return;
    }
    const double mu = s1[i] / static_cast<double>(M);
    out[e] = tc[e] / static_cast<double>(M - m) - mu * mu;
}

hipError_t launch_tcorr1d(int prec, int n_inst, int nmax, int lags, hipStream_t s, const Inst1D *tab,
                          const void *hist, int32_t hist_rows, int64_t n0, int64_t count, double *tc,
                          const InstAcc *acc)
{
    const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(nmax) * lags + 255) / 256), n_inst);
    if (prec == 0)
        hipLaunchKernelGGL(k_tcorr<float>, grid, dim3(256), 0, s, tab, static_cast<const float *>(hist), hist_rows,
                           lags, n0, count, tc, acc);
    else
        hipLaunchKernelGGL(k_tcorr<double>, grid, dim3(256), 0, s, tab, static_cast<const double *>(hist),
                           hist_rows, lags, n0, count, tc, acc);
    return hipGetLastError();
}

hipError_t launch_fin_tc(hipStream_t s, int n, int lags, const double *s1, const double *tc, int64_t M,
                         double *out)
{
    const int64_t tot = static_cast<int64_t>(n) * lags;
    hipLaunchKernelGGL(k_fin_tc, dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, s, n, lags, s1, tc, M,
                       out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ init

template <typename T>
__global__ void __launch_bounds__(256)
    k_init1d(const Inst1D *__restrict__ tab, const double *__restrict__ init_sd, T *__restrict__ pool)
{
    const int inst = blockIdx.x;
    const Inst1D d = tab[inst];
    const int i = blockIdx.y * 256 + threadIdx.x;
    if (i >= d.n) return;
    const double ref = d.bc == 1 ? d.uL + (d.uR - d.uL) * (i + 0.5) / d.n : d.u0;
    double v = ref;
    const double sd = init_sd[inst];
    if (sd > 0.0) {
        const Normals4<double> nz = init_normals(static_cast<uint32_t>(i >> 2), d.realisation, make_key(d.seed));
        v = ref + sd * nz.z[i & 3];
    }
    pool[d.off + i] = static_cast<T>(v);
}

// ------------------------------------------------------------------ finalisation

// m2[i][j] = (C[i][j] + sum over the rows of the open block X_b,i X_b,j) / M and
// cov[i][j] = m2[i][j] - m_i m_j.  One thread per entry; the open rows are loaded
// eight ahead of their (ordered) products, which otherwise each wait for
// their own loads.
template <typename T>
__global__ void __launch_bounds__(256)
    k_fin_m2(const T *__restrict__ X, const double *__restrict__ C, const double *__restrict__ s1, int N,
             const InstAcc *__restrict__ q, double *__restrict__ m2, double *__restrict__ cov)
{
    const int64_t M = max(q->n_samples, static_cast<int64_t>(1));
    const int rows = static_cast<int>(q->n_samples % kCorrBlock);  // open rows of the X block
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= static_cast<int64_t>(N) * N) return;
    const int i = static_cast<int>(e / N), j = static_cast<int>(e - static_cast<int64_t>(i) * N);
    double acc = C[e];
    int b = 0;
    for (; b + 8 <= rows; b += 8) {
        T x[8], y[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            x[k] = X[static_cast<int64_t>(b + k) * N + i];
            y[k] = X[static_cast<int64_t>(b + k) * N + j];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += static_cast<double>(x[k]) * static_cast<double>(y[k]);
    }
    for (; b < rows; ++b)
        acc += static_cast<double>(X[static_cast<int64_t>(b) * N + i]) * static_cast<double>(X[static_cast<int64_t>(b) * N + j]);
    const double inv = 1.0 / static_cast<double>(M), v = acc / static_cast<double>(M);
    m2[e] = v;
    if (cov) cov[e] = v - (s1[i] * inv) * (s1[j] * inv);
}

// mean, variance per cell, sum(U) of the current field
template <typename T>
__global__ void __launch_bounds__(256)
    k_fin_cells(const Inst1D *__restrict__ tab, int inst, const T *__restrict__ pool,
                const double *__restrict__ s1, const double *__restrict__ s2, const InstAcc *__restrict__ acc, Fin1D out)
{
    const Inst1D d = tab[inst];
    const int N = d.n;
    const double inv = 1.0 / static_cast<double>(max(acc->n_samples, static_cast<int64_t>(1)));
    if (threadIdx.x < sizeof(InstAcc) / 8)
        reinterpret_cast<uint64_t *>(out.acc)[threadIdx.x] = reinterpret_cast<const uint64_t *>(acc)[threadIdx.x];
    double a = 0.0;
    for (int i = threadIdx.x; i < N; i += 256) {
        const double ref = d.bc == 1 ? d.uL + (d.uR - d.uL) * (i + 0.5) / N : d.u0;
        const double m = s1 ? s1[d.off + i] * inv : 0.0;
        out.mean[i] = ref + m;
        out.var[i] = s2 ? s2[d.off + i] * inv - m * m : 0.0;
        a += static_cast<double>(pool[d.off + i]);
    }
    __shared__ double red[256];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out.sum = red[0];
}

// <|U_k|^2> = |R_k|^2 + 2 Re(conj(R_k) sum_j m_j w^{jk}) + sum_ij m2_ij cos(2 pi k (i-j)/N),
// R_k = DFT of the reference profile, m = E[dU], m2 = E[dU dU^T].  The double
// sum is sum_d c(d) cos(2 pi k d/N) over the circulant sums c(d) = sum_i
// m2[i][(i - d) mod N], formed once for all k: N^2 additions and N^2 cosines in
// all, where evaluating it per k takes N^3 of each (N = 128: 6050 us on one
// workgroup before, 7.7 us for both kernels now).
// One wave per d: lane l adds i = l, l + 64, ... in order, then the wave.
__global__ void __launch_bounds__(256) k_fin_circ(int N, const double *__restrict__ m2, double *__restrict__ circ)
{
    const int d = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (d >= N) return;
    double a = 0.0;
    for (int i = lane; i < N; i += 64) {
        const int j = i - d < 0 ? i - d + N : i - d;
        a += m2[static_cast<int64_t>(i) * N + j];
    }
    a = wave_total(a);
    if (lane == 0) circ[d] = a;
}

// One wave per k: lane l takes j = l, l + 64, ... of the three sums.
__global__ void __launch_bounds__(256)
    k_fin_sk(const Inst1D *__restrict__ tab, int inst, const double *__restrict__ s1, const double *__restrict__ circ,
             const InstAcc *__restrict__ acc, double *__restrict__ sk)
{
    const int64_t M = max(acc->n_samples, static_cast<int64_t>(1));
    const Inst1D d = tab[inst];
    const int N = d.n;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k >= N) return;
    const double inv = 1.0 / static_cast<double>(M);
    double rr = 0.0, ri = 0.0, mr = 0.0, mi = 0.0, q = 0.0;
    for (int j = lane; j < N; j += 64) {
        const int idx = (j * k) % N;  // N <= 1024
        double sn, cs;
        sincospi(-2.0 * static_cast<double>(idx) / N, &sn, &cs);
        const double ref = d.bc == 1 ? d.uL + (d.uR - d.uL) * (j + 0.5) / N : d.u0;
        const double m = s1[d.off + j] * inv;
        rr += ref * cs;
        ri += ref * sn;
        mr += m * cs;
        mi += m * sn;
        q += circ[j] * cs;
    }
    rr = wave_total(rr);
    ri = wave_total(ri);
    mr = wave_total(mr);
    mi = wave_total(mi);
    q = wave_total(q);
    if (lane == 0) sk[k] = (rr * rr + ri * ri) + 2.0 * (rr * mr + ri * mi) + q;
}

// ------------------------------------------------------------------ batch means

// Whether the last launch completed batch n_batches + 1 of this instance.
__device__ __forceinline__ bool batch_done(const InstAcc &q, int32_t len)
{
    return len > 0 && !q.nonfinite && q.n_samples >= (q.n_batches + 1) * static_cast<int64_t>(len);
}

// S_k of the batch, from its covariance sums: Cb = (C + the open X rows) -
// csnap, its circulant sums c(d) = sum_i Cb[i][(i - d) mod N] (so that
// sum_ij Cb_ij cos(2 pi k (i - j)/N) = sum_d c(d) cos(2 pi k d/N)), and the
// batch mean m_b of dU: S_k = |R_k|^2 + 2 Re(conj(R_k) DFT(m_b)_k) +
// sum_d c(d) cos(2 pi k d/N) / L, R the DFT of the reference profile (the
// formula of k_fin_sk for one batch).  Then csnap takes the current sums.
// One block per instance; runs before k_fold_cells1d (it reads the s1
// snapshot that kernel moves on).
template <typename T>
__global__ void __launch_bounds__(256)
    k_fold_sk1d(const Inst1D *__restrict__ tab, const T *__restrict__ xblk, const double *__restrict__ c,
                const double *__restrict__ s1, const InstAcc *__restrict__ acc, Batch1D bk)
{
    const int inst = blockIdx.x;
    const Inst1D d = tab[inst];
    const InstAcc q = acc[inst];
    if (d.c_off < 0 || !batch_done(q, bk.len)) return;
    __shared__ double cd[1024], mb[1024];
    const int N = d.n;
    const int rows = static_cast<int>(q.n_samples % kCorrBlock);  // open rows of the X block
    const T *X = xblk + d.x_off;
    const double *C = c + d.c_off;
    double *Cs = bk.csnap + d.c_off;
    const double *s1s = bk.cell;
    const double L = static_cast<double>(bk.len);
    auto ctot = [&](int i, int j) {
        double v = C[static_cast<int64_t>(i) * N + j];
        for (int r = 0; r < rows; ++r)
            v += static_cast<double>(X[static_cast<int64_t>(r) * N + i]) * static_cast<double>(X[static_cast<int64_t>(r) * N + j]);
        return v;
    };
    for (int dd = threadIdx.x; dd < N; dd += 256) {
        double a = 0.0;
        for (int i = 0; i < N; ++i) {
            const int j = i - dd < 0 ? i - dd + N : i - dd;
            a += ctot(i, j) - Cs[static_cast<int64_t>(i) * N + j];
        }
        cd[dd] = a;
    }
    for (int i = threadIdx.x; i < N; i += 256) mb[i] = (s1[d.off + i] - s1s[d.off + i]) / L;
    __syncthreads();
    for (int64_t e = threadIdx.x; e < static_cast<int64_t>(N) * N; e += 256) {
        const int i = static_cast<int>(e / N), j = static_cast<int>(e - static_cast<int64_t>(i) * N);
        Cs[e] = ctot(i, j);
    }
    const double b = static_cast<double>(q.n_batches + 1);
    for (int k = threadIdx.x; k < N; k += 256) {
        double rr = 0.0, ri = 0.0, mr = 0.0, mi = 0.0, qq = 0.0;
        for (int j = 0; j < N; ++j) {
            const int64_t idx = (static_cast<int64_t>(j) * k) % N;
            double sn, cs;
            sincospi(-2.0 * static_cast<double>(idx) / N, &sn, &cs);
            const double ref = d.bc == 1 ? d.uL + (d.uR - d.uL) * (j + 0.5) / N : d.u0;
            rr += ref * cs;
            ri += ref * sn;
            mr += mb[j] * cs;
            mi += mb[j] * sn;
            qq += cd[j] * cs;   // cos(2 pi k d / N) for d = j
        }
        const double x = (rr * rr + ri * ri) + 2.0 * (rr * mr + ri * mi) + qq / L;
        welford(x, b, bk.skw[d.off + k], bk.skw[bk.total_cells + d.off + k]);
    }
}

// Per-cell batch mean and variance of dU, folded into their Welford sums;
// the s1 / s2 snapshots move to the current sums.
__global__ void __launch_bounds__(256)
    k_fold_cells1d(const Inst1D *__restrict__ tab, const double *__restrict__ s1, const double *__restrict__ s2,
                   const InstAcc *__restrict__ acc, Batch1D bk)
{
    const int inst = blockIdx.x;
    const Inst1D d = tab[inst];
    const InstAcc q = acc[inst];
    const int i = blockIdx.y * 256 + threadIdx.x;
    if (i >= d.n || !batch_done(q, bk.len)) return;
    const int64_t tc = bk.total_cells, e = d.off + i;
    double *cl = bk.cell;
    const double L = static_cast<double>(bk.len), b = static_cast<double>(q.n_batches + 1);
    const double m = (s1[e] - cl[e]) / L;
    const double v = (s2[e] - cl[tc + e]) / L - m * m;
    welford(m, b, cl[2 * tc + e], cl[3 * tc + e]);
    welford(v, b, cl[4 * tc + e], cl[5 * tc + e]);
    cl[e] = s1[e];
    cl[tc + e] = s2[e];
}

// Spatial statistics of the batch and the batch count (last of the folds).
__global__ void __launch_bounds__(64) k_fold_acc1d(int n_inst, InstAcc *__restrict__ acc, int32_t len)
{
    const int inst = blockIdx.x * 64 + threadIdx.x;
    if (inst >= n_inst) return;
    InstAcc q = acc[inst];
    if (!batch_done(q, len)) return;
    fold_spatial(q, len);
    acc[inst] = q;
}

hipError_t launch_fold1d(int prec, int n_inst, int nmax, hipStream_t s, const Inst1D *tab, const void *xblk,
                         const double *c, const double *s1, const double *s2, InstAcc *acc, const Batch1D &bk)
{
    if (bk.csnap) {
        if (prec == 0)
            hipLaunchKernelGGL(k_fold_sk1d<float>, dim3(n_inst), dim3(256), 0, s, tab,
                               static_cast<const float *>(xblk), c, s1, acc, bk);
        else
            hipLaunchKernelGGL(k_fold_sk1d<double>, dim3(n_inst), dim3(256), 0, s, tab,
                               static_cast<const double *>(xblk), c, s1, acc, bk);
    }
    if (bk.cell)
        hipLaunchKernelGGL(k_fold_cells1d, dim3(n_inst, (nmax + 255) / 256), dim3(256), 0, s, tab, s1, s2, acc, bk);
    hipLaunchKernelGGL(k_fold_acc1d, dim3((n_inst + 63) / 64), dim3(64), 0, s, n_inst, acc, bk.len);
    return hipGetLastError();
}

// ------------------------------------------------------------------ launchers

struct Step1DLaunch {
    int n_blocks;
    size_t smem;
    hipStream_t s;
    const Inst1D *tab;
    const Seg1D *segs;
    void *pool;
    const void *coef;
    const double *pcr;
    int64_t step0;
    int32_t nsteps;
    int64_t burn_in;
    int32_t every;
    uint32_t mask;
    Stats1D st;
};

template <typename T, int BLOCK, int MAXG, bool STATS>
static hipError_t step1d_k(const Step1DLaunch &a)
{
    hipLaunchKernelGGL((k_step1d<T, BLOCK, MAXG, STATS>), dim3(a.n_blocks), dim3(BLOCK), a.smem, a.s, a.tab, a.segs,
                       static_cast<T *>(a.pool), static_cast<const T *>(a.coef), a.pcr, a.step0, a.nsteps, a.burn_in,
                       a.every, a.mask, a.st);
    return hipGetLastError();
}

template <typename T, int BLOCK, int MAXG>
static hipError_t step1d_t(bool stats, const Step1DLaunch &a)
{
    return stats ? step1d_k<T, BLOCK, MAXG, true>(a) : step1d_k<T, BLOCK, MAXG, false>(a);
}

// Launch shapes (threads per workgroup, Philox blocks per thread) the
// planner chooses: 256 x {1, 2}, 512 x {1, 2, 4}.
template <typename T>
static hipError_t step1d_p(int block, int maxg, bool stats, const Step1DLaunch &a)
{
    if (block == 256 && maxg == 1) return step1d_t<T, 256, 1>(stats, a);
    if (block == 256 && maxg == 2) return step1d_t<T, 256, 2>(stats, a);
    if (block == 512 && maxg == 1) return step1d_t<T, 512, 1>(stats, a);
    if (block == 512 && maxg == 2) return step1d_t<T, 512, 2>(stats, a);
    if (block == 512 && maxg == 4) return step1d_t<T, 512, 4>(stats, a);
    return hipErrorInvalidValue;
}

hipError_t launch_step1d(int prec, int block, int maxg, bool stats, int n_blocks, size_t smem, hipStream_t s,
                         const Inst1D *tab, const Seg1D *segs, void *pool, const void *coef, const double *pcr,
                         int64_t step0, int32_t nsteps, int64_t burn_in, int32_t every, uint32_t mask, Stats1D st)
{
    const Step1DLaunch a{n_blocks, smem, s, tab, segs, pool, coef, pcr, step0, nsteps, burn_in, every, mask, st};
    return prec == 0 ? step1d_p<float>(block, maxg, stats, a) : step1d_p<double>(block, maxg, stats, a);
}

// Typed launchers of the explicit batches, instantiated in she_k1d_f*.hip.
extern template hipError_t rods_t<float, 0, false>(const Launch1D &);
extern template hipError_t rods_t<float, 0, true>(const Launch1D &);
extern template hipError_t rods_t<float, 1, false>(const Launch1D &);
extern template hipError_t rods_t<float, 1, true>(const Launch1D &);
extern template hipError_t rods_t<float, 2, true>(const Launch1D &);
extern template hipError_t rods_t<double, 2, true>(const Launch1D &);
extern template hipError_t rods_t<float, 3, false>(const Launch1D &);
extern template hipError_t rods_t<float, 3, true>(const Launch1D &);
extern template hipError_t rods_t<double, 0, false>(const Launch1D &);
extern template hipError_t rods_t<double, 0, true>(const Launch1D &);
extern template hipError_t rods_t<double, 1, false>(const Launch1D &);
extern template hipError_t rods_t<double, 1, true>(const Launch1D &);
extern template hipError_t rods_t<double, 3, false>(const Launch1D &);
extern template hipError_t rods_t<double, 3, true>(const Launch1D &);
extern template hipError_t rods_t<float, 4, false>(const Launch1D &);
extern template hipError_t rods_t<float, 4, true>(const Launch1D &);
extern template hipError_t rods_t<float, 5, false>(const Launch1D &);
extern template hipError_t rods_t<float, 5, true>(const Launch1D &);
extern template hipError_t rods_t<double, 4, false>(const Launch1D &);
extern template hipError_t rods_t<double, 4, true>(const Launch1D &);
extern template hipError_t rods_t<double, 5, false>(const Launch1D &);
extern template hipError_t rods_t<double, 5, true>(const Launch1D &);
extern template hipError_t rods_t<float, 6, true>(const Launch1D &);
extern template hipError_t rods_t<double, 6, true>(const Launch1D &);
extern template hipError_t rods_mixed_t<float, 2>(const Launch1D &);
extern template hipError_t rods_mixed_t<float, 6>(const Launch1D &);
extern template hipError_t rods_mixed_t<double, 2>(const Launch1D &);
extern template hipError_t rods_mixed_t<double, 6>(const Launch1D &);

template <typename T>
static hipError_t rods_p(const Launch1D &a)
{
    const bool ahead = a.ahead > 0;
    switch (a.mode) {
    case 0: return ahead ? rods_t<T, 0, true>(a) : rods_t<T, 0, false>(a);
    case 1: return ahead ? rods_t<T, 1, true>(a) : rods_t<T, 1, false>(a);
    case 2: return !ahead ? hipErrorInvalidValue : (a.mixed ? rods_mixed_t<T, 2>(a) : rods_t<T, 2, true>(a));
    case 3: return ahead ? rods_t<T, 3, true>(a) : rods_t<T, 3, false>(a);
    case 4: return ahead ? rods_t<T, 4, true>(a) : rods_t<T, 4, false>(a);
    case 5: return ahead ? rods_t<T, 5, true>(a) : rods_t<T, 5, false>(a);
    case 6: return !ahead ? hipErrorInvalidValue : (a.mixed ? rods_mixed_t<T, 6>(a) : rods_t<T, 6, true>(a));
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_rods(const Launch1D &a) { return a.prec == 0 ? rods_p<float>(a) : rods_p<double>(a); }

hipError_t launch_init1d(int prec, int n_inst, int nmax, hipStream_t s, const Inst1D *tab, const double *init_sd,
                         void *pool)
{
    const dim3 grid(n_inst, (nmax + 255) / 256);
    if (prec == 0)
        hipLaunchKernelGGL(k_init1d<float>, grid, dim3(256), 0, s, tab, init_sd, static_cast<float *>(pool));
    else
        hipLaunchKernelGGL(k_init1d<double>, grid, dim3(256), 0, s, tab, init_sd, static_cast<double *>(pool));
    return hipGetLastError();
}

hipError_t launch_fin1d(int prec, hipStream_t s, const Inst1D *tab, int inst, int n, const void *pool,
                        const double *s1, const double *s2, int64_t off, const void *xblk, const double *c,
                        const InstAcc *acc, bool corr, const Fin1D &out)
{
    const int64_t nn = static_cast<int64_t>(n) * n;
    if (prec == 0)
        hipLaunchKernelGGL(k_fin_cells<float>, dim3(1), dim3(256), 0, s, tab, inst, static_cast<const float *>(pool),
                           s1, s2, acc, out);
    else
        hipLaunchKernelGGL(k_fin_cells<double>, dim3(1), dim3(256), 0, s, tab, inst,
                           static_cast<const double *>(pool), s1, s2, acc, out);
    if (corr) {
        const dim3 nb(static_cast<unsigned>((nn + 255) / 256)), nw((n + 3) / 4);
        if (prec == 0)
            hipLaunchKernelGGL(k_fin_m2<float>, nb, dim3(256), 0, s, static_cast<const float *>(xblk), c, s1 + off, n,
                               acc, out.m2, out.cov);
        else
            hipLaunchKernelGGL(k_fin_m2<double>, nb, dim3(256), 0, s, static_cast<const double *>(xblk), c, s1 + off, n,
                               acc, out.m2, out.cov);
        hipLaunchKernelGGL(k_fin_circ, nw, dim3(256), 0, s, n, out.m2, out.circ);
        hipLaunchKernelGGL(k_fin_sk, nw, dim3(256), 0, s, tab, inst, s1, out.circ, acc, out.sk);
    }
    return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(256) k_widen(const T *__restrict__ f, int64_t n, double *__restrict__ out)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) out[i] = static_cast<double>(f[i]);
}

hipError_t launch_widen(int prec, hipStream_t s, const void *field, int64_t n, double *out)
{
    const dim3 g(static_cast<unsigned>((n + 255) / 256));
    if (prec == 0)
        hipLaunchKernelGGL(k_widen<float>, g, dim3(256), 0, s, static_cast<const float *>(field), n, out);
    else
        hipLaunchKernelGGL(k_widen<double>, g, dim3(256), 0, s, static_cast<const double *>(field), n, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ verification

__global__ void __launch_bounds__(256)
    k_debug_philox(uint64_t seed, const uint32_t *__restrict__ ctr, int64_t count, uint32_t *__restrict__ out)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= count) return;
    const Words4 w = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], make_key(seed));
    for (int l = 0; l < 4; ++l) out[4 * i + l] = w.w[l];
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_debug_normals(uint64_t seed, uint32_t real, uint32_t tag, uint64_t step, uint64_t face0, int64_t count,
                    double *__restrict__ out)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= count) return;
    const uint64_t f = face0 + static_cast<uint64_t>(i);
    if constexpr (std::is_same<T, double>::value) {
        if (tag == 1) {  // as the initial state is drawn
            out[i] = init_normals(static_cast<uint32_t>(f >> 2), real, make_key(seed), step).z[f & 3];
            return;
        }
    }
    const Normals4<T> nz = block_normals<T>(static_cast<uint32_t>(f >> 2), static_cast<uint32_t>(step),
                                            ctr_word2(step, tag), real, make_key(seed));
    out[i] = static_cast<double>(nz.z[f & 3]);
}

hipError_t launch_debug_philox(hipStream_t s, uint64_t seed, const uint32_t *ctr, int64_t count, uint32_t *out)
{
    hipLaunchKernelGGL(k_debug_philox, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, seed, ctr,
                       count, out);
    return hipGetLastError();
}

hipError_t launch_debug_normals(hipStream_t s, int prec, uint64_t seed, uint32_t realisation, uint32_t tag,
                                uint64_t step, uint64_t face0, int64_t count, double *out)
{
    const dim3 grid(static_cast<unsigned>((count + 255) / 256));
    if (prec == 0)
        hipLaunchKernelGGL(k_debug_normals<float>, grid, dim3(256), 0, s, seed, realisation, tag, step, face0, count,
                           out);
    else
        hipLaunchKernelGGL(k_debug_normals<double>, grid, dim3(256), 0, s, seed, realisation, tag, step, face0, count,
                           out);
    return hipGetLastError();
}

}  // namespace she
