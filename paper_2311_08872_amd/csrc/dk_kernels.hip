// dk_kernels.hip -- gfx950 kernels of the MLMC Dean--Kawasaki hot path: the resident level
// kernel (grids up to 128 x 128; its building blocks and the scheme it implements are described
// in dk_level.h), the ordered moment reduction, field evaluation and the noise dump.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "dk_internal.h"
#include "dk_level.h"
#include "dk_rng.h"

namespace dk {

// ---------------------------------------------------------------------------------------
// The resident level kernel: one block-iteration per block.
// ---------------------------------------------------------------------------------------
template <typename Real, int NF, int R, int C, bool PAIR, int FLUX, int SPW>
__global__ void __launch_bounds__(SPW * (NF / C) * (NF / R))
level_kernel(const LevelArgs A)
{
    __shared__ __align__(16) Real halo[SPW * halo_elems<Real, NF, R, PAIR, SPW>()];
    level_body<Real, NF, R, C, PAIR, FLUX, SPW>(A, (uint64_t)blockIdx.x * SPW, halo, (int)threadIdx.x);
}

// ---------------------------------------------------------------------------------------
// Launches: the tile shape of a batch by its variant (shape_rows in dk_tuning.cpp).
// ---------------------------------------------------------------------------------------
template <typename Real, int NF, int R, bool PAIR, int FLUX, int X = 1>
static hipError_t launch_R(const LevelArgs& A, hipStream_t s)
{
    using S = ShapeOf<NF, R, X>;
    const uint64_t blocks = (A.count + S::SPW - 1) / S::SPW;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL((level_kernel<Real, NF, R, S::C, PAIR, FLUX, S::SPW>), dim3((unsigned)blocks), dim3(S::SPW * S::TS), 0, s,
                       A);
    return hipGetLastError();
}

template <typename Real, int NF, bool PAIR, int FLUX>
static hipError_t launch_variants(const LevelArgs& A, int v, hipStream_t s)
{
    constexpr bool F32 = std::is_same<Real, float>::value;
    if constexpr (NF == 4) {
        // 4 x 4 (the level 0 of the paper's own hierarchy): 2 lanes per sample, 4 rows each
        return launch_R<Real, 4, 4, PAIR, FLUX>(A, s);
    } else if constexpr (NF == 8) {
        if constexpr (!PAIR) if (v == 4) return launch_R<Real, 8, 1, PAIR, FLUX>(A, s);
        if (v == 1) return launch_R<Real, 8, 2, PAIR, FLUX>(A, s);
        if (v == 2) return launch_R<Real, 8, 4, PAIR, FLUX>(A, s);
        if constexpr (F32) if (v == 3) return launch_R<Real, 8, 8, PAIR, FLUX, 4>(A, s);
        return launch_R<Real, 8, 8, PAIR, FLUX>(A, s);
    } else if constexpr (NF == 16) {
        if (v == 1) return launch_R<Real, 16, 4, PAIR, FLUX>(A, s);
        if constexpr (!PAIR) if (v == 4) return launch_R<Real, 16, 1, PAIR, FLUX>(A, s);
        if (v == 2) return launch_R<Real, 16, 2, PAIR, FLUX>(A, s);
        if constexpr (F32) if (v == 3) return launch_R<Real, 16, 8, PAIR, FLUX, 4>(A, s);
        return launch_R<Real, 16, 8, PAIR, FLUX>(A, s);
    } else if constexpr (NF == 32) {
        if (v == 1) return launch_R<Real, 32, 4, PAIR, FLUX>(A, s);
        if (v == 4) return launch_R<Real, 32, 2, PAIR, FLUX>(A, s);
        if constexpr (F32) {
            if (v == 2) return launch_R<Real, 32, 16, PAIR, FLUX>(A, s);
            if (v == 3) return launch_R<Real, 32, 8, PAIR, FLUX, 4>(A, s);
        }
        return launch_R<Real, 32, 8, PAIR, FLUX>(A, s);
    } else if constexpr (NF == 64) {
        if (v == 3) return launch_R<Real, 64, 4, PAIR, FLUX>(A, s);
        if (v == 4) return launch_R<Real, 64, 2, PAIR, FLUX>(A, s);
        if constexpr (F32) {
            if (v == 1) return launch_R<Real, 64, 16, PAIR, FLUX>(A, s);
            if (v == 2) return launch_R<Real, 64, 8, PAIR, FLUX, 4>(A, s);
        }
        return launch_R<Real, 64, 8, PAIR, FLUX>(A, s);
    } else {
        if (v == 1) return launch_R<Real, 128, 16, PAIR, FLUX>(A, s);
        return launch_R<Real, 128, 8, PAIR, FLUX>(A, s);
    }
}

template <typename Real, bool PAIR, int FLUX>
static hipError_t launch_nf(const LevelArgs& A, int v, hipStream_t s)
{
    switch (A.nf) {
        case 4: return launch_variants<Real, 4, PAIR, FLUX>(A, v, s);
        case 8: return launch_variants<Real, 8, PAIR, FLUX>(A, v, s);
        case 16: return launch_variants<Real, 16, PAIR, FLUX>(A, v, s);
        case 32: return launch_variants<Real, 32, PAIR, FLUX>(A, v, s);
        case 64: return launch_variants<Real, 64, PAIR, FLUX>(A, v, s);
        case 128: return launch_variants<Real, 128, PAIR, FLUX>(A, v, s);
        default: return hipErrorInvalidValue;
    }
}

bool level_supported(int nf) { return nf == 4 || nf == 8 || nf == 16 || nf == 32 || nf == 64 || nf == 128; }

hipError_t launch_level(const LevelKind& k, const LevelArgs& A, hipStream_t s)
{
    const bool f64 = k.precision == DK_PREC_F64;
    const int v = shape_run(A.nf, k.shape, f64, k.pair);
    const bool stag = k.flux == DK_FLUX_STAGGERED;
    if (!f64 && !stag) return k.pair ? launch_nf<float, true, DK_FLUX_CENTRAL>(A, v, s)
                                     : launch_nf<float, false, DK_FLUX_CENTRAL>(A, v, s);
    if (!f64 && stag) return k.pair ? launch_nf<float, true, DK_FLUX_STAGGERED>(A, v, s)
                                    : launch_nf<float, false, DK_FLUX_STAGGERED>(A, v, s);
    if (f64 && !stag) return k.pair ? launch_nf<double, true, DK_FLUX_CENTRAL>(A, v, s)
                                    : launch_nf<double, false, DK_FLUX_CENTRAL>(A, v, s);
    return k.pair ? launch_nf<double, true, DK_FLUX_STAGGERED>(A, v, s)
                  : launch_nf<double, false, DK_FLUX_STAGGERED>(A, v, s);
}

// ---------------------------------------------------------------------------------------
// Ordered compensated moment sums.  One block per observable and moment; thread t sums the samples
// t, t + T, t + 2T, .. with compensated summation, then the threads' sums are merged in a fixed pairwise
// tree.  The result depends only on (count, data).  One block for all six moments of an observable ran
// at the FP64 rate of one compute unit and read with a stride: 47 us on average over the batches of an
// Algorithm-1 run (up to 8e4 samples), now 4 us (up to 4096 samples) and 18 us (above).
// ---------------------------------------------------------------------------------------
template <int T>
__global__ void __launch_bounds__(T) moments_kernel(const double* __restrict__ ps, uint64_t count, int n_obs,
                                                    double* __restrict__ out)
{
    const int j = blockIdx.x, k = blockIdx.y;
    const int t = threadIdx.x;
    const int q = k / 2;                             // Y, P_fine, P_coarse
    double s = 0.0, c = 0.0;
#pragma unroll 4
    for (uint64_t i = t; i < count; i += T) {
        const double pf = ps[(i * n_obs + j) * 2 + 0];
        const double pc = ps[(i * n_obs + j) * 2 + 1];
        const double v = q == 0 ? pf - pc : (q == 1 ? pf : pc);
        neumaier(s, c, (k & 1) ? v * v : v);
    }
    __shared__ double sh[T][2];
    sh[t][0] = s;
    sh[t][1] = c;
    __syncthreads();
    for (int w = T / 2; w >= 1; w >>= 1) {
        if (t < w) {
            neumaier(s, c, sh[t + w][0]);
            c += sh[t + w][1];
            sh[t][0] = s;
            sh[t][1] = c;
        }
        __syncthreads();
    }
    if (t == 0) {
        out[(j * DK_NMOM + k) * 2 + 0] = s;
        out[(j * DK_NMOM + k) * 2 + 1] = c;
    }
}

hipError_t launch_moments(const double* per_sample, uint64_t count, int n_obs, double* out, hipStream_t s)
{
    const dim3 grid(n_obs, DK_NMOM);
    if (count <= 4096)
        hipLaunchKernelGGL(moments_kernel<256>, grid, dim3(256), 0, s, per_sample, count, n_obs, out);
    else
        hipLaunchKernelGGL(moments_kernel<1024>, grid, dim3(1024), 0, s, per_sample, count, n_obs, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Field evaluation (I_h of an analytic field), FP64.
// ---------------------------------------------------------------------------------------
__global__ void field_eval_kernel(const FieldDev f, double box, int n, void* out, int as_double)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * n) return;
    const int ix = idx % n, iy = idx / n;
    const double h = box / n;
    const double x = ix * h, y = iy * h;
    const double two_pi = 6.28318530717958647692;
    double v = f.c0;
    if (f.kind == DK_FIELD_MODES || f.kind == DK_FIELD_CLIPPED) {
        for (int k = 0; k < f.n_modes; ++k) v += f.amp[k] * cos(two_pi * (f.kx[k] * x + f.ky[k] * y) / box + f.phase[k]);
        if (f.kind == DK_FIELD_CLIPPED) v = fmax(v, 0.0) + f.floor_add;
    } else if (f.kind == DK_FIELD_BUMP) {
        double dx = fmod(fabs(x - f.bump_cx), box);
        dx = fmin(dx, box - dx);
        double dy = fmod(fabs(y - f.bump_cy), box);
        dy = fmin(dy, box - dy);
        v += f.bump_amp * exp(-(dx * dx + dy * dy) / (2.0 * f.bump_sigma * f.bump_sigma));
    } else {
        const double sx = sin(x - f.es_x0), sy = sin(y - f.es_y0);
        v = f.es_scale * (f.es_a + f.es_b * exp(-(sx * sx + sy * sy) / (2.0 * f.es_s)));
    }
    if (as_double) ((double*)out)[idx] = v;
    else ((float*)out)[idx] = (float)v;
}

hipError_t launch_field_eval(const FieldDev& f, double box, int n, void* out, bool as_double, hipStream_t s)
{
    const int total = n * n;
    hipLaunchKernelGGL(field_eval_kernel, dim3((total + 255) / 256), dim3(256), 0, s, f, box, n, out, (int)as_double);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Noise dump: out[sample][step][y][x][r] (one thread per site pair and step)
// ---------------------------------------------------------------------------------------
__global__ void noise_dump_kernel(uint64_t seed, uint32_t tag, int level, int n, uint64_t first_sample,
                                  uint32_t n_samples, int first_step, int n_steps, float* out)
{
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t pairs = (uint64_t)(n / 2) * n;
    const uint64_t total = pairs * n_steps * n_samples;
    if (idx >= total) return;
    const uint64_t p = idx % pairs;
    const uint64_t ms = (idx / pairs) % n_steps;
    const uint64_t si = idx / (pairs * n_steps);
    const NoiseKey key = make_key(seed, tag, level, first_sample + si);
    float a0, a1, b0, b1;
    site_pair_normals(key, (uint32_t)p, (uint32_t)(first_step + ms), a0, a1, b0, b1);
    const uint64_t y = p / (n / 2), x = 2 * (p % (n / 2));
    float* o = out + (((si * n_steps + ms) * n + y) * n + x) * 2;
    o[0] = a0;
    o[1] = a1;
    o[2] = b0;
    o[3] = b1;
}

hipError_t launch_noise_dump(uint64_t seed, uint32_t tag, int level, int n, uint64_t first_sample, uint32_t n_samples,
                             int first_step, int n_steps, float* out, hipStream_t s)
{
    const uint64_t total = (uint64_t)(n / 2) * n * n_steps * n_samples;
    if (total == 0) return hipSuccess;
    const uint64_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(noise_dump_kernel, dim3((unsigned)blocks), dim3(256), 0, s, seed, tag, level, n, first_sample,
                       n_samples, first_step, n_steps, out);
    return hipGetLastError();
}

__global__ void gauss_kernel(const uint32_t* __restrict__ a, const uint32_t* __restrict__ b, uint64_t count,
                             float* __restrict__ z0, float* __restrict__ z1)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    float u, v;
    box_muller(a[i], b[i], u, v);
    z0[i] = u;
    z1[i] = v;
}

__global__ void root_kernel(const double* __restrict__ x, uint64_t count, double* __restrict__ out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = pos_sqrt(x[i]);
}

hipError_t launch_root(const double* x, uint64_t count, double* out, hipStream_t s)
{
    const uint64_t blocks = (count + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(root_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, count, out);
    return hipGetLastError();
}

hipError_t launch_gauss(const uint32_t* a, const uint32_t* b, uint64_t count, float* z0, float* z1, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    const uint64_t blocks = (count + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gauss_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, b, count, z0, z1);
    return hipGetLastError();
}

}  // namespace dk
