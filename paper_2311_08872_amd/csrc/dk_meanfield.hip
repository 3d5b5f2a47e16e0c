// dk_meanfield.hip -- the noise-free scheme to its final time (the discrete mean field of Sec. 3,
// which centres the observables) and its inner products with the test functions, in FP64: stepped, or in
// the scheme's eigenbasis.
//
// rho^M = (I + (mu/2) Lap_h)^M rho^0 is diagonal in the discrete Fourier basis, with the factor
// g^M = (1 - 2 mu (sin^2(pi kx/n) + sin^2(pi ky/n)))^M (Appendix A, operator A_h), so M steps cost the
// way into that basis and back whatever M is.  The basis used is the real one of the Hartley
// transform, cas t = cos t + sin t: cas(2 pi k x/n) is an eigenvector of the periodic second
// difference with the eigenvalue of cos and sin, the matrix C[k][x] = cas(2 pi k x/n) is symmetric and
// C C = n I, so rho^M = n^-2 C (g^M .* (C rho^0 C)) C: four real n x n products on the FP64 matrix
// cores (v_mfma_f64_16x16x4_f64).  One pass forms C X^T, so two passes are C X C and the rows read are
// always contiguous; C itself is never stored, its entries are a table of n values in LDS indexed by
// k x mod n.
//
// Bound by the FP64 matrix rate for n >= 1024 and by the latency of four dependent passes below.
// One launch per step took 118 ms at 512 x 512 with 26624 steps (4.7 us a launch); now four of 18 us (145 us a call).
// g^M comes from exp(M log1p(-lambda)), whose error does not grow with M.  The transform takes the field's difference
// from a constant near its mean, which no step changes: 0.5 to 1.1e-16 of the field (2-norm, 16 x 16 to 128 x 128)
// against 1.0 to 1.6e-16 for the steps, and 0.9 to 2.4e-16 with the constant in it.
//
// The field of the two ways agrees to its rounding, and so do the inner products, relative to the size of their
// terms.  An inner product that cancels (an even datum and an odd test function) is the rounding itself, and has no
// digit in common between them.  The steps define its value: the caller takes the transform's result only where no
// inner product is below kCancelled of its terms' size, and steps the field otherwise.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dk_internal.h"
#include "dk_level.h"

namespace dk {

namespace {

typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kOneBlock = 64;      // grids up to this size run in one block, the field in LDS

__device__ __forceinline__ void cas_table(double* tab, int n)
{
    for (int m = threadIdx.x; m < n; m += blockDim.x) {
        double s, c;
        sincospi(2.0 * m / n, &s, &c);
        tab[m] = c + s;
    }
}

// g^M of mode (kx, ky), a = mu / 2.  1 - g = 4 a (sin^2 + sin^2) lies in [0, 2]; beyond 1 (mu > 1/4) the
// factor is negative and its size is 1 - (2 - (1 - g)).
__device__ __forceinline__ double mode_power(int kx, int ky, int n, double a, int M)
{
    const double sx = sinpi((double)kx / n), sy = sinpi((double)ky / n);
    const double lam = 4.0 * a * (sx * sx + sy * sy);
    if (lam <= 1.0) return exp(M * log1p(-lam));
    const double p = exp(M * log1p(lam - 2.0));
    return (M & 1) ? -p : p;
}

// Tile rows k0.., columns y0.. of C X^T: sum over x of cas(k x) X[y][x].  The order of the 16 x of one
// product group over lanes and products is the same for both operands: lane group q takes x0 + 4 q + j.
// G groups are loaded ahead of the G being multiplied (the rows come from L2 with one wavefront per
// SIMD).  SHIFT: of X - shift.  Returns D[row 4 r + q][column lane & 15].
template <int G, bool SHIFT>
__device__ __forceinline__ doublex4 cas_tile(const double* X, int pitch, int n, const double* tab, int k0, int y0, int lane,
                                             double shift)
{
    const int i = lane & 15, q = lane >> 4;
    const int k = min(k0 + i, n - 1), y = min(y0 + i, n - 1);
    const double* row = X + (size_t)y * pitch;
    const int step = (16 * k) % n;
    int idx = (4 * q * k) % n;
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
    doublex2 nxt[G][2];
    auto load = [&](int x0) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) {                // beyond the row: zeros (n is even)
                const int x = x0 + 16 * g + 4 * q + 2 * h;
                nxt[g][h] = doublex2{0.0, 0.0};
                if (x < n) nxt[g][h] = *(const doublex2*)(row + x) - (SHIFT ? doublex2{shift, shift} : doublex2{0.0, 0.0});
            }
    };
    load(0);
    for (int x0 = 0; x0 < n; x0 += 16 * G) {
        doublex2 cur[G][2];
#pragma unroll
        for (int g = 0; g < G; ++g) { cur[g][0] = nxt[g][0]; cur[g][1] = nxt[g][1]; }
        load(x0 + 16 * G);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            int id = idx;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(tab[id], cur[g][j >> 1][j & 1], acc, 0, 0, 0);
                id += k;
                id -= id >= n ? n : 0;
            }
            idx += step;
            idx -= idx >= n ? n : 0;
        }
    }
    return acc;
}

// Grids up to 64 x 64: all four passes in one block, a wavefront per 16 x 16 tile.
__global__ void __launch_bounds__(1024) meanfield_block_kernel(double* __restrict__ rho, int n, double a, int steps, double shift)
{
    constexpr int PMAX = kOneBlock + 2;
    __shared__ __align__(16) double fld[2][kOneBlock * PMAX];
    __shared__ double tab[kOneBlock];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int P = n + 2;                                  // rows start two banks apart
    const int T = (n + 15) / 16;
    const int k0 = 16 * (wave / T), y0 = 16 * (wave % T);
    cas_table(tab, n);
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) fld[0][(e / n) * P + e % n] = rho[e] - shift;
    __syncthreads();
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
        const doublex4 d = cas_tile<1, false>(fld[pass & 1], P, n, tab, k0, y0, lane, 0.0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = k0 + 4 * r + (lane >> 4), y = y0 + (lane & 15);
            if (k >= n || y >= n) continue;
            const double v = pass == 1 ? d[r] * (mode_power(y, k, n, a, steps) / ((double)n * n)) : d[r];
            fld[(pass + 1) & 1][k * P + y] = v;
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) rho[e] = fld[0][(e / n) * P + e % n] + shift;
}

// Larger grids: one pass per launch.  The four wavefronts of a block share their columns y, so the rows
// of X are read through one L1.
template <int PASS>
__global__ void __launch_bounds__(256) cas_pass_kernel(const double* __restrict__ X, double* __restrict__ out, int n, double a,
                                                       int steps, double shift)
{
    extern __shared__ double tab[];
    cas_table(tab, n);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int T = (n + 15) / 16, TK = (T + 3) / 4;
    const int kt = 4 * (blockIdx.x % TK) + (threadIdx.x >> 6);
    if (kt >= T) return;
    const int k0 = 16 * kt, y0 = 16 * (blockIdx.x / TK);
    const doublex4 d = cas_tile<4, PASS == 0>(X, n, n, tab, k0, y0, lane, shift);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int k = k0 + 4 * r + (lane >> 4), y = y0 + (lane & 15);
        if (k >= n || y >= n) continue;
        double v = d[r];
        if constexpr (PASS == 1) v *= mode_power(y, k, n, a, steps) / ((double)n * n);
        if constexpr (PASS == 3) v += shift;
        out[(size_t)k * n + y] = v;
    }
}

// The steps of a resident grid (4, 8, .. 128) and the inner products, in one block: the tiles of the level
// kernels (2 columns and R rows per lane, the rows above and below through LDS, one barrier a step).  A step of
// 128 x 128 takes 1.74 us, the latency of a lane's 16 rows.
template <int N>
struct Resident {
    static constexpr int R = N == 4 ? 4 : (N == 128 ? 16 : 8), NPL = N / 2, G = N / R, TS = NPL * G;
};

template <int N>
__global__ void __launch_bounds__(Resident<N>::TS) meanfield_steps_kernel(double* __restrict__ field, double a, int steps,
                                                                        const double* __restrict__ phi, int n_obs, double h2,
                                                                        double* __restrict__ out)
{
#pragma clang fp contract(off)
    constexpr int R = Resident<N>::R, NPL = Resident<N>::NPL, G = Resident<N>::G, TS = Resident<N>::TS;
    constexpr bool WL = TS <= 64;
    __shared__ __align__(16) double halo[2][G][2][N];
    __shared__ double red[(TS + 63) / 64];
    const int t = threadIdx.x, cl = t % NPL, g = t / NPL, lane = t & 63;
    const int addr_l = (lane - cl + (cl + NPL - 1) % NPL) * 4, addr_r = (lane - cl + (cl + 1) % NPL) * 4;
    const int gu = g == 0 ? G - 1 : g - 1, gd = g == G - 1 ? 0 : g + 1;
    double rho[R][2];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) rho[i][c] = field[(R * g + i) * N + 2 * cl + c];
#pragma unroll 1
    for (int m = 0; m < steps; ++m) {
        auto& buf = halo[m & 1];
        double prev[2], below[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            buf[g][0][2 * cl + c] = rho[0][c];
            buf[g][1][2 * cl + c] = rho[R - 1][c];
        }
        sample_sync<WL>();               // the other buffer is written next: one barrier a step
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            prev[c] = buf[gu][1][2 * cl + c];
            below[c] = buf[gd][0][2 * cl + c];
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const double o0 = rho[i][0], o1 = rho[i][1];
            const double n0 = i + 1 < R ? rho[i + 1 < R ? i + 1 : 0][0] : below[0];
            const double n1 = i + 1 < R ? rho[i + 1 < R ? i + 1 : 0][1] : below[1];
            const double l = lane_get(addr_l, o1), r = lane_get(addr_r, o0);
            rho[i][0] = o0 + a * fma(-4.0, o0, (l + o1) + (prev[0] + n0));
            rho[i][1] = o1 + a * fma(-4.0, o1, (o0 + r) + (prev[1] + n1));
            prev[0] = o0;
            prev[1] = o1;
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) field[(R * g + i) * N + 2 * cl + c] = rho[i][c];
    for (int j = 0; j < n_obs; ++j) {
        const double* ph = phi + (size_t)j * N * N;
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) v = fma(rho[i][c], ph[(R * g + i) * N + 2 * cl + c], v);
#pragma unroll
        for (int off = (TS < 64 ? TS : 64) / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if constexpr (!WL) {
            if (lane == 0) red[t >> 6] = v;
            __syncthreads();
            v = 0.0;
            for (int w = 0; w < TS / 64; ++w) v += red[w];
            __syncthreads();
        }
        if (t == 0) out[j] = h2 * v;
    }
}

// One step of any other grid
__global__ void heat_step_kernel(const double* __restrict__ in, double* __restrict__ out, int n, double a)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= n) return;
    const int xm = x == 0 ? n - 1 : x - 1, xp = x == n - 1 ? 0 : x + 1;
    const int ym = y == 0 ? n - 1 : y - 1, yp = y == n - 1 ? 0 : y + 1;
    const double c = in[(size_t)y * n + x];
    const double lap = (in[(size_t)y * n + xm] + in[(size_t)y * n + xp]) + (in[(size_t)ym * n + x] + in[(size_t)yp * n + x]) - 4.0 * c;
    out[(size_t)y * n + x] = c + a * lap;
}

__device__ __forceinline__ double block_sum(double v, double* sh)
{
    __syncthreads();
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    return sh[0];
}

// Part p of the inner product with observable j and of the size of its terms (grid: parts x observables).  One part:
// the results themselves.  out: [products][sizes][parts of both, 2 per block].
__global__ void __launch_bounds__(256) inner_kernel(const double* __restrict__ rho, int nn, const double* __restrict__ phi,
                                                    double h2, double* __restrict__ out)
{
    __shared__ double sh[256];
    const int j = blockIdx.y, parts = gridDim.x, nobs = gridDim.y;
    const double* ph = phi + (size_t)j * nn;
    double acc = 0.0, size = 0.0;
#pragma unroll 4
    for (int i = blockIdx.x * 256 + threadIdx.x; i < nn; i += 256 * parts) {
        const double r = rho[i], f = ph[i];
        acc = fma(r, f, acc);
        size = fma(fabs(r), fabs(f), size);
    }
    const double s = block_sum(acc, sh), z = block_sum(size, sh);
    if (threadIdx.x != 0) return;
    if (parts == 1) {
        out[j] = h2 * s;
        out[nobs + j] = h2 * z;
    } else {
        double* part = out + 2 * nobs + 2 * (j * parts + blockIdx.x);
        part[0] = s;
        part[1] = z;
    }
}

__global__ void __launch_bounds__(256) inner_finish_kernel(int parts, double h2, double* __restrict__ out)
{
    __shared__ double sh[256];
    const int j = blockIdx.x, nobs = gridDim.x, t = threadIdx.x;
    const double* part = out + 2 * nobs + 2 * j * parts;
    const double s = block_sum(t < parts ? part[2 * t] : 0.0, sh), z = block_sum(t < parts ? part[2 * t + 1] : 0.0, sh);
    if (t != 0) return;
    out[j] = h2 * s;
    out[nobs + j] = h2 * z;
}

template <int N>
hipError_t resident_steps(double a, int steps, double* field, const double* phi, int n_obs, double h2, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(meanfield_steps_kernel<N>, dim3(1), dim3(Resident<N>::TS), 0, s, field, a, steps, phi, n_obs, h2, out);
    return hipGetLastError();
}

}  // namespace

bool meanfield_steps_cheaper(int n, int steps)
{
    // Microseconds on MI355X: the four passes 4 (4^2) .. 30 (64^2) in one block, 31 (128^2), 46 (256^2), 105 (512^2)
    // in four launches; a step 0.27 (4^2), 0.45 (8^2 .. 32^2), 0.60 (64^2), 1.74 (128^2) in one block, 3.5 (to 256^2),
    // 4.4 (512^2), 60 (4096^2) as a launch.  25 more lie between the passes and the steps where both are needed.
    const double passes = n <= kOneBlock ? 2.0 + 0.4 * n : 24.0 + 2.2e-7 * (double)n * n * n;
    const double step = level_supported(n) ? 0.4 + 8e-5 * (double)n * n : 3.5 + 3.5e-6 * (double)n * n;
    return steps * step <= passes + 25.0;
}

hipError_t launch_meanfield_steps(int n, double a, int steps, double* buf0, double* buf1, const double* phi, int n_obs, double h2,
                                  double* out, double** result, hipStream_t s)
{
    if (n < 2 || (n & 1) || n > 4096 || steps < 0) return hipErrorInvalidValue;
    *result = buf0;
    switch (n) {
    case 4: return resident_steps<4>(a, steps, buf0, phi, n_obs, h2, out, s);
    case 8: return resident_steps<8>(a, steps, buf0, phi, n_obs, h2, out, s);
    case 16: return resident_steps<16>(a, steps, buf0, phi, n_obs, h2, out, s);
    case 32: return resident_steps<32>(a, steps, buf0, phi, n_obs, h2, out, s);
    case 64: return resident_steps<64>(a, steps, buf0, phi, n_obs, h2, out, s);
    case 128: return resident_steps<128>(a, steps, buf0, phi, n_obs, h2, out, s);
    default: break;
    }
    double *in = buf0, *to = buf1;
    const dim3 grid((n + 255) / 256, n);
    for (int m = 0; m < steps; ++m) {
        hipLaunchKernelGGL(heat_step_kernel, grid, dim3(256), 0, s, in, to, n, a);
        double* t = in; in = to; to = t;
    }
    *result = in;
    hipLaunchKernelGGL(inner_kernel, dim3(1, n_obs), dim3(256), 0, s, in, n * n, phi, h2, out);
    return hipGetLastError();
}

hipError_t launch_meanfield_transform(int n, double a, int steps, double shift, double* buf0, double* buf1, const double* phi,
                                      int n_obs, double h2, double* out, hipStream_t s)
{
    if (n < 2 || (n & 1) || n > 4096 || steps < 1) return hipErrorInvalidValue;
    const int T = (n + 15) / 16;
    if (n <= kOneBlock) {
        hipLaunchKernelGGL(meanfield_block_kernel, dim3(1), dim3(64 * T * T), 0, s, buf0, n, a, steps, shift);
    } else {
        const dim3 grid((unsigned)(T * ((T + 3) / 4)));
        const size_t lds = sizeof(double) * n;
        hipLaunchKernelGGL(cas_pass_kernel<0>, grid, dim3(256), lds, s, buf0, buf1, n, a, steps, shift);
        hipLaunchKernelGGL(cas_pass_kernel<1>, grid, dim3(256), lds, s, buf1, buf0, n, a, steps, shift);
        hipLaunchKernelGGL(cas_pass_kernel<2>, grid, dim3(256), lds, s, buf0, buf1, n, a, steps, shift);
        hipLaunchKernelGGL(cas_pass_kernel<3>, grid, dim3(256), lds, s, buf1, buf0, n, a, steps, shift);
    }
    // above 128 x 128 one block per observable would read its megabytes alone (320 us at 512 x 512)
    const int parts = n <= 128 ? 1 : kInnerParts;
    hipLaunchKernelGGL(inner_kernel, dim3(parts, n_obs), dim3(256), 0, s, buf0, n * n, phi, h2, out);
    if (parts > 1) hipLaunchKernelGGL(inner_finish_kernel, dim3(n_obs), dim3(256), 0, s, parts, h2, out);
    return hipGetLastError();
}

}  // namespace dk
