// 2D / 3D periodic grids: launch dispatch, sample reductions, initial state
// and finalisation.  The step kernels themselves are in she_step_nd.hpp.
#include "she_internal.hpp"
#include "she_rng.hpp"

namespace she {

// Typed launchers, instantiated in she_k2d_*.hip / she_k3d_*.hip.
template <typename T, int CX>
hipError_t step2d_e(int eq, int scheme, int n_blocks, hipStream_t s, const ParamsND &p, const void *src,
                    void *dst, const StepArg &sa, double *part, InstAcc *acc, const SkRows *skr);
template <typename T, int CX>
hipError_t step3d_e(int eq, int stage, int ty, int n_blocks, size_t smem, hipStream_t s, const ParamsND &p,
                    const void *src, const void *base, void *dst, const StepArg &sa, double *part, InstAcc *acc);

template <typename T>
static hipError_t step2d_c(int cx, int eq, int scheme, int n_blocks, hipStream_t s, const ParamsND &p,
                           const void *src, void *dst, const StepArg &sa, double *part, InstAcc *acc,
                           const SkRows *skr)
{
    switch (cx) {
    case 4: return step2d_e<T, 4>(eq, scheme, n_blocks, s, p, src, dst, sa, part, acc, skr);
    case 8: return step2d_e<T, 8>(eq, scheme, n_blocks, s, p, src, dst, sa, part, acc, skr);
    case 16: return step2d_e<T, 16>(eq, scheme, n_blocks, s, p, src, dst, sa, part, acc, skr);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step2d(int prec, int cx, int eq, int scheme, int n_blocks, hipStream_t s, const ParamsND &p,
                         const void *src, void *dst, const StepArg &sa, double *part, InstAcc *acc,
                         const SkRows *skr)
{
    ParamsND q = p;
    q.by_lx = fast_div(p.nx / cx);
    q.by_parts = fast_div((p.ny + p.chunk - 1) / p.chunk);
    if (prec == 0) return step2d_c<float>(cx, eq, scheme, n_blocks, s, q, src, dst, sa, part, acc, skr);
    return step2d_c<double>(cx, eq, scheme, n_blocks, s, q, src, dst, sa, part, acc, skr);
}

hipError_t launch_step3d(int prec, int cx, int eq, int stage, int ty, int n_blocks, size_t smem, hipStream_t s,
                         const ParamsND &p, const void *src, const void *base, void *dst, const StepArg &sa,
                         double *part, InstAcc *acc)
{
    ParamsND q = p;
    q.by_lx = fast_div(p.nx / cx);
    q.by_yt = fast_div(p.ny / ty);
    q.by_parts = fast_div(q.by_yt.d * ((p.nz + p.chunk - 1) / p.chunk));
    if (prec == 0) {
        if (cx == 4) return step3d_e<float, 4>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
        if (cx == 8) return step3d_e<float, 8>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
        if (cx == 16) return step3d_e<float, 16>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
    } else {
        if (cx == 4) return step3d_e<double, 4>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
        if (cx == 8) return step3d_e<double, 8>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
        if (cx == 16)
            return step3d_e<double, 16>(eq, stage, ty, n_blocks, smem, s, q, src, base, dst, sa, part, acc);
    }
    return hipErrorInvalidValue;
}

// Per-instance reduction of the sample partials, fixed order.
__global__ void __launch_bounds__(64)
    k_reduce_parts(StepArg sarg, SpatialParts sp)
{
    int64_t step;
    int sample;
    resolve_step(sarg, step, sample);
    if (!sample) return;
    reduce_spatial_wave(sp, blockIdx.x, threadIdx.x);
}

// ------------------------------------------------------------------ init / finalisation

template <typename T>
__global__ void __launch_bounds__(256)
    k_initnd(ParamsND p, int64_t cells, T *__restrict__ field)
{
    const int inst = blockIdx.y;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= cells) return;
    const InstND ipar = p.ip[inst];
    double v = ipar.u0;
    if (ipar.init_sd > 0.0) {
        const Normals4<double> nz = init_normals(static_cast<uint32_t>(c >> 2), ipar.realisation, make_key(p.seed));
        v += ipar.init_sd * nz.z[c & 3];
    }
    field[static_cast<int64_t>(inst) * cells + c] = static_cast<T>(v);
}

// Sum of cells [c0, c1) of a field over a block of 256 threads (FP64, fixed
// order; the result in thread 0).  16-byte loads, four in flight per thread:
// a single block that takes one cell per load waits out the memory latency
// once per 256 cells.  c0 is a multiple of 4 and so is the field's cell count.
template <typename T>
__device__ __forceinline__ double block_sum(const T *__restrict__ f, int64_t c0, int64_t c1)
{
    constexpr int V = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(V)));
    __shared__ double red[256];
    const vec *v = reinterpret_cast<const vec *>(f + c0);
    const int64_t nv = (c1 - c0) / V;
    double a = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 768 < nv; i += 1024) {
        vec x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = v[i + 256 * q];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int l = 0; l < V; ++l) a += static_cast<double>(x[q][l]);
    }
    for (; i < nv; i += 256) {
        const vec x = v[i];
#pragma unroll
        for (int l = 0; l < V; ++l) a += static_cast<double>(x[l]);
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

// Partial sums of one instance's field: block b the cells [b span, (b + 1) span).
template <typename T>
__global__ void __launch_bounds__(256)
    k_sum_parts(const T *__restrict__ field, int64_t cells, int64_t span, double *__restrict__ part)
{
    const int64_t c0 = blockIdx.x * span, c1 = min(c0 + span, cells);
    const double a = block_sum<T>(field, c0, c1);
    if (threadIdx.x == 0) part[blockIdx.x] = a;
}

// part: nparts partial sums of the field (k_sum_parts), or nparts = 0: the
// field is small and this block sums it itself.
template <typename T>
__global__ void __launch_bounds__(256)
    k_finnd(ParamsND p, int inst, int64_t cells, const T *__restrict__ field, const InstAcc *__restrict__ acc,
            const double *__restrict__ sk_sums, const double *__restrict__ sk_modes, int nbins,
            const double *__restrict__ part, int nparts, double *__restrict__ out)
{
    const double total = nparts > 0 ? block_sum<double>(part, 0, nparts)
                                    : block_sum<T>(field + static_cast<int64_t>(inst) * cells, 0, cells);
    if (threadIdx.x < sizeof(InstAcc) / 8)
        reinterpret_cast<uint64_t *>(out)[threadIdx.x] = reinterpret_cast<const uint64_t *>(acc + inst)[threadIdx.x];
    out += kFinAcc;
    const double u0 = p.ip[inst].u0;
    if (threadIdx.x == 0) {
        const InstAcc q = acc[inst];
        const double M = q.n_samples > 0 ? static_cast<double>(q.n_samples) : 1.0;
        out[0] = u0 + q.sp_mean / M;
        out[1] = q.sp_var / M;
        out[2] = total;
    }
    // shell averages; the k = 0 mode of U = u0 + dU is
    // sum_samples (N u0 + sum dU)^2 = M N^2 u0^2 + 2 N u0 (N sp_mean) + sum (sum dU)^2
    if (nbins > 0) {
        const InstAcc q = acc[inst];
        const double M = q.n_samples > 0 ? static_cast<double>(q.n_samples) : 1.0;
        const double N = static_cast<double>(cells);
        const double *ss = sk_sums + static_cast<int64_t>(inst) * nbins;
        for (int b = threadIdx.x; b < nbins; b += 256) {
            double v = ss[b];
            if (b == 0) v += M * N * N * u0 * u0 + 2.0 * N * u0 * (N * q.sp_mean);
            out[3 + b] = sk_modes[b] > 0 ? v / (M * sk_modes[b]) : 0.0;
        }
    }
}

// ------------------------------------------------------------------ launchers

hipError_t launch_reduce_parts(int n_inst, hipStream_t s, const StepArg &sa, const double *part, int32_t nparts,
                               double inv_cells, int32_t batch_len, InstAcc *acc)
{
    const SpatialParts sp{part, acc, inv_cells, nparts, batch_len};
    hipLaunchKernelGGL(k_reduce_parts, dim3(n_inst), dim3(64), 0, s, sa, sp);
    return hipGetLastError();
}

__global__ void k_set_step(int64_t *ctr, int64_t value)
{
    if (threadIdx.x == 0) *ctr = value;
}

__global__ void k_add_step(int64_t *ctr, int64_t k)
{
    if (threadIdx.x == 0) *ctr += k;
}

hipError_t launch_set_step(hipStream_t s, int64_t *ctr, int64_t value)
{
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(64), 0, s, ctr, value);
    return hipGetLastError();
}

hipError_t launch_add_step(hipStream_t s, int64_t *ctr, int64_t k)
{
    hipLaunchKernelGGL(k_add_step, dim3(1), dim3(64), 0, s, ctr, k);
    return hipGetLastError();
}

hipError_t launch_initnd(int prec, hipStream_t s, const ParamsND &p, int64_t cells, void *field)
{
    const dim3 grid(static_cast<unsigned>((cells + 255) / 256), p.n_inst);
    if (prec == 0)
        hipLaunchKernelGGL(k_initnd<float>, grid, dim3(256), 0, s, p, cells, static_cast<float *>(field));
    else
        hipLaunchKernelGGL(k_initnd<double>, grid, dim3(256), 0, s, p, cells, static_cast<double *>(field));
    return hipGetLastError();
}

// Fields above 16384 cells are summed by one block per 8192 cells (more cells
// per block from 8 Mi cells on, kFinParts blocks at most) ahead of the final
// kernel; up to there the one block is as fast as the extra launch.  One block
// for any field, one cell per load, took 17.7 ms for 256^3 cells, 409 us
// for 512 x 512 and 13.6 us for 128 x 128; now 15.5 us and 8.5 us (two
// launches) and 4.2 us.
template <typename T>
static void finnd_t(hipStream_t s, const ParamsND &p, int inst, int64_t cells, const void *field, const InstAcc *acc,
                    const double *sk_sums, const double *sk_modes, int nbins, double *part, double *out)
{
    const T *f = static_cast<const T *>(field);
    int nparts = 0;
    if (cells > 16384) {
        int64_t span = 8192;
        while ((cells + span - 1) / span > kFinParts) span *= 2;
        nparts = (static_cast<int>((cells + span - 1) / span) + 1) & ~1;  // an even count of doubles; the pad sums nothing
        hipLaunchKernelGGL(k_sum_parts<T>, dim3(nparts), dim3(256), 0, s, f + static_cast<int64_t>(inst) * cells, cells,
                           span, part);
    }
    hipLaunchKernelGGL(k_finnd<T>, dim3(1), dim3(256), 0, s, p, inst, cells, f, acc, sk_sums, sk_modes, nbins, part,
                       nparts, out);
}

hipError_t launch_finnd(int prec, hipStream_t s, const ParamsND &p, int inst, int64_t cells, const void *field,
                        const InstAcc *acc, const double *sk_sums, const double *sk_modes, int nbins, double *part,
                        double *out)
{
    if (prec == 0)
        finnd_t<float>(s, p, inst, cells, field, acc, sk_sums, sk_modes, nbins, part, out);
    else
        finnd_t<double>(s, p, inst, cells, field, acc, sk_sums, sk_modes, nbins, part, out);
    return hipGetLastError();
}

}  // namespace she
