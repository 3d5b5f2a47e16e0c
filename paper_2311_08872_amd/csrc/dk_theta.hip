// dk_theta.hip -- level kernel of eq. (FullyDiscreteDK) with an implicit weight b0 > 0.
//
// One step solves (I - tau b0/2 Lap_h) rho^m = (I + tau b1/2 Lap_h) rho^{m-1} + noise term
// (b1 = 1 - b0).  Writing d for the increment of the explicit scheme (b0 = 0), the same step is
// rho^m = rho^{m-1} + S d with S = (I - tau b0/2 Lap_h)^{-1}: the right-hand side minus
// (I - tau b0/2 Lap_h) rho^{m-1} is exactly d.  So a step computes d with the per-cell arithmetic
// of the other kernels, filters it with S -- diagonal in the discrete Fourier basis, with
// eigenvalue 1 / (1 + 2 b0 mu (sin^2(pi kx/n) + sin^2(pi ky/n))) from a host table -- and adds
// the filtered increment with the compensated sum of the FP32 kernels (FP64: plain sum).
// Pairs are NN-coupled (Sec. 3.2): the coarse grid takes the same scheme every 4 fine steps
// with the restricted noise (the sum over the 2 x 2 block and the 4 steps, in state precision).
//
// The filter on the matrix cores.  cas t = cos t + sin t diagonalises the periodic second difference as
// the complex exponential does, with a real symmetric matrix C[k][x] = cas(2 pi k x/n), C C = n I, so
// S d = n^-2 C (s .* (C d C)) C: four real n x n products.  The even frequencies of a transform over n
// points are a transform over n/2 of the sums f(x) + f(x + n/2), the odd ones a product by n/2 columns of
// C with the differences, down to one tile of 16: for n = 64 a product costs 24 instead of 64 instructions
// per 16 columns.  The frequencies stay in the order this leaves (theta_frequency).
//
// FP32 adds d and (S - I) d, with the products on the second part only: S - I is small where the observables
// look, at long waves, and so are the rounding errors that pass it (a sum of 32 products rounds more often
// than five butterflies; 4000 pairs of 32 x 32 at N = 1e4: 6.8e-7 of the observable's RMS with S d, 4.2e-7 so,
// 6.1e-7 by butterflies).
//
// Bound by the vector ALU (generator and addresses: instructions active in half of the SIMDs' cycles at 64 x 64)
// and the FP64 matrix cores (busy in a third); two wavefronts per SIMD overlap the two in part.  1000 pairs of
// 64 x 64 in FP64 with one lane per butterfly point: 38.3 ms; here 8.0 ms (1.5e11 cell updates/s).
//
// Layout: cells are owned as the products return them: register i of lane (q, c) = (lane / 16, lane % 16)
// of a 16 x 16 tile is row M::row(i, q) of column c.  The same register is the operand B of a product that
// contracts over those rows (C X) and, as A, of the transposed one (X^T C), so a grid of one tile goes
// through all four products in registers: X^T C, C (.), s, (.)^T C, C (.).  A wavefront owns the n/16
// tiles of 16 columns; between the two directions the tiles change hands through LDS.  Grids below
// 16 x 16 share a tile, with C block-diagonal.  C's entries come from a table of n values in LDS.
// Density and fluxes reach the neighbouring cells through two LDS planes.  The horizontal site pair of
// one generator call lies in two neighbouring lanes: each draws one of two rows, and they swap.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "dk_level.h"
#include "dk_mma.h"
#include "dk_sum.h"
#include "dk_theta.h"

namespace dk {

namespace {
template <int N>
struct TG {
    static constexpr int TN = N < 16 ? 16 : N;        // extent of the tiles of a wavefront group
    static constexpr int T = TN / 16;                 // tiles per column, wavefronts of a group
    static constexpr int SIDE = TN / N;               // samples per tile side
    static constexpr int SLOTS = SIDE * SIDE;         // samples of a group
    static constexpr bool WL = T == 1;                // a group inside one wavefront
    static constexpr int WPB = WL ? 4 : T;            // wavefronts of a block
    static constexpr int GPB = WL ? WPB : 1;          // groups of a block
    static constexpr int SPB = GPB * SLOTS;           // samples of a block
    // 64 x 64 in FP64: 64 KB of planes, two blocks of four wavefronts per compute unit
    static constexpr int WAVES = T == 4 ? 2 : 4;
};

__device__ __forceinline__ double root(double x) { return pos_sqrt_f64(x); }
__device__ __forceinline__ float root(float x) { return sqrt(x > 0.0f ? x : 0.0f); }

// the value of the neighbouring lane of an even-odd pair
__device__ __forceinline__ float swap_pair(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

// The lanes' view of one grid of N x N: its planes in LDS and the lane's place.  NT: length of the table of
// C's entries (N, or 2 N for the coarse grid of a pair).
template <typename Real, int N, int NT>
struct Grid {
    typedef Mma<Real> M;
    typedef typename M::Acc Acc;
    typedef TG<N> G;
    static constexpr int T = G::T, TN = G::TN;
    static constexpr bool F64 = std::is_same<Real, double>::value;
    // Planes are [TN][P].  The 16 columns of four (FP32) or two (FP64, half a wavefront at a time) rows that
    // one access touches lie in different banks: by the pitch for one tile, else by swapping groups of 16.
    static constexpr int P = T == 1 && !F64 ? 20 : TN;
    static constexpr int PLANE = TN * P;
    static __device__ __forceinline__ int cell(int y, int x)
    {
        const int swap = T == 1 ? 0 : 16 * (F64 ? (y & 1) : (y >> 2) & (T - 1));
        return y * P + (x ^ swap);
    }

    // cell(row(t, i), x), and the cells above and below it: one address for a lane and a constant, but for the
    // rows where a sample's edge or the swap of the next four rows falls
    __device__ __forceinline__ int at(int t, int i, int x) const
    {
        const int swap = T == 1 ? 0 : 16 * (F64 ? (q & 1) : q & (T - 1));
        return M::row(0, q) * P + (x ^ swap) + (16 * t + (F64 ? 4 * i : i)) * P;
    }
    __device__ __forceinline__ int above(int t, int i, int x) const
    {
        const int y = row(t, i);
        if (F64 ? (16 * t + 4 * i) % N == 0 : i == 0) return cell(y % N == 0 ? y + N - 1 : y - 1, x);
        if (!F64) return at(t, i, x) - P;
        return (q - 1) * P + (x ^ (T == 1 ? 0 : 16 * (1 - (q & 1)))) + (16 * t + 4 * i) * P;
    }
    __device__ __forceinline__ int below(int t, int i, int x) const
    {
        const int y = row(t, i);
        if (F64 ? (16 * t + 4 * i + 4) % N == 0 : i == 3) return cell(y % N == N - 1 ? y + 1 - N : y + 1, x);
        if (!F64) return at(t, i, x) + P;
        return (q + 1) * P + (x ^ (T == 1 ? 0 : 16 * (1 - (q & 1)))) + (16 * t + 4 * i) * P;
    }

    Real *p0, *p1;
    const Real* cas;           // cas(2 pi j / NT), j < NT, in LDS
    int w, q, c;               // column tile, lane group, lane column
    Real creg[4];              // one tile: C[row(i, q)][c], block-diagonal for N < 16

    // The place is derived again for every step: the addresses that follow from it, kept across the steps,
    // would take the registers of the tiles.
    __device__ __forceinline__ void place()
    {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        w = TG<NT>::WL ? 0 : tid >> 6;
        q = (tid >> 4) & 3;
        c = tid & 15;
    }
    __device__ __forceinline__ int col() const { return 16 * w + c; }
    __device__ __forceinline__ int row(int t, int i) const { return 16 * t + M::row(i, q); }

    __device__ __forceinline__ void init()
    {
        if constexpr (T == 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = M::row(i, q);
                creg[i] = r / N == c / N ? cas[(r % N) * (c % N) * (NT / N) & (NT - 1)] : Real(0);
            }
    }

    // D += the part of H tiles of a product with frequencies FS * position + F0 (in units of the table),
    // the rows of X contracted: over the points (INV: the frequencies).  LEFT: D = C X, else X^T C.
    template <int H, int FS, int F0, bool INV, bool LEFT>
    __device__ __forceinline__ void part(const Acc* X, Acc* D) const
    {
#pragma unroll
        for (int J = 0; J < H; ++J) {
            Acc acc = {0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < H; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    Real e;
                    if constexpr (T == 1) {
                        e = creg[i];
                    } else {
                        const int o = 16 * J + c, k = 16 * t + M::row(i, q);
                        e = cas[(INV ? (FS * k + F0) * o : (FS * o + F0) * k) & (NT - 1)];
                    }
                    acc = LEFT ? M::mul(e, X[t][i], acc) : M::mul(X[t][i], e, acc);
                }
            D[J] = acc;
        }
    }

    // one direction of the transform of H tiles (16 H points of the N), forward or inverse
    template <int H, bool INV, bool LEFT>
    __device__ __forceinline__ void transform(const Acc* X, Acc* D) const
    {
        constexpr int STEP = NT / (16 * H);              // its first frequency
        if constexpr (H == 1) {
            part<1, STEP, 0, INV, LEFT>(X, D);
        } else {
            constexpr int L = H / 2;
            Acc e[L], o[L];
            if constexpr (!INV) {
#pragma unroll
                for (int t = 0; t < L; ++t) {
                    e[t] = X[t] + X[t + L];
                    o[t] = X[t] - X[t + L];
                }
                transform<L, INV, LEFT>(e, D);
                part<L, 2 * STEP, STEP, INV, LEFT>(o, D + L);
            } else {
                transform<L, INV, LEFT>(X, e);
                part<L, 2 * STEP, STEP, INV, LEFT>(X + L, o);
#pragma unroll
                for (int t = 0; t < L; ++t) {
                    D[t] = e[t] + o[t];
                    D[t + L] = e[t] - o[t];
                }
            }
        }
    }

    // hand the tiles over: D (this wavefront's 16 rows, all columns) -> X (all rows, its 16 columns)
    __device__ __forceinline__ void exchange(Real* p, const Acc* D, Acc* X, bool on) const
    {
        if (on)
#pragma unroll
            for (int J = 0; J < T; ++J)
#pragma unroll
                for (int i = 0; i < 4; ++i) p[cell(16 * w + M::row(i, q), 16 * J + c)] = D[J][i];
        __syncthreads();
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) X[t][i] = p[at(t, i, col())];
    }

    // v <- S v (FP32: S v - v); sol: [position of kx][position of ky], 1 / N^2 included.  Every wavefront of a block comes
    // here; those that are not `on` own no tile of this grid.  Issued ahead of the other wavefronts' vector work,
    // so that the matrix cores' queue does not run dry (1000 pairs of 64 x 64: 9.5 to 8.5 ms).
    __device__ __forceinline__ void filter(Acc (&v)[T], const Real* __restrict__ sol, bool on) const
    {
        __builtin_amdgcn_s_setprio(2);
        if constexpr (G::SIDE == 1) {
            products(v, sol, on);
        } else {
            // The zeros of C beside the samples' blocks do not keep a value that is not finite from the other samples
            // of the tile: then each sample is filtered alone, with zeros in the others' places.
            const Acc in = v[0];
            products(v, sol, on);
            bool finite = true;
#pragma unroll
            for (int i = 0; i < 4; ++i) finite = finite && isfinite(v[0][i]);
            if (__any(!finite)) {
                Acc all = v[0];
#pragma unroll 1
                for (int s = 0; s < G::SLOTS; ++s) {
                    bool mine[4];
                    Acc one[1];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        mine[i] = (row(0, i) / N) * G::SIDE + c / N == s;
                        one[0][i] = mine[i] ? in[i] : Real(0);
                    }
                    products(one, sol, on);
#pragma unroll
                    for (int i = 0; i < 4; ++i) all[i] = mine[i] ? one[0][i] : all[i];
                }
                v[0] = all;
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }

    // the four products and the multipliers between them
    __device__ __forceinline__ void products(Acc (&v)[T], const Real* __restrict__ sol, bool on) const
    {
        Acc u[T];
        if (on) transform<T, false, false>(v, u);
        if constexpr (T > 1) exchange(p0, u, v, on);
        if (on) {
            if constexpr (T == 1) v[0] = u[0];
            transform<T, false, true>(v, u);
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) u[t][i] *= sol[(row(t, i) % N) * N + col() % N];
            transform<T, true, false>(u, v);
        }
        if constexpr (T > 1) exchange(p1, v, u, on);
        if (on) {
            if constexpr (T == 1) u[0] = v[0];
            transform<T, true, true>(u, v);
        }
    }

    // d <- the explicit increment of rho with the unit noise w0, w1 (float: fine normals; Real: restricted
    // sums).  The first barrier ends the reads of the planes before it.
    template <bool WL, typename NW>
    __device__ __forceinline__ void increment(const Real (&rho)[T][4], const NW (&w0)[T][4], const NW (&w1)[T][4], Real a,
                                              Real kappa, Acc (&d)[T], bool on) const
    {
#pragma clang fp contract(off)
        Real f1[T][4], dx[T][4];
        const int x = col(), xl = x % N == 0 ? x + N - 1 : x - 1, xr = x % N == N - 1 ? x + 1 - N : x + 1;
        sample_sync<WL>();
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = at(t, i, x);
                    const Real s = root(rho[t][i]);
                    p0[k] = rho[t][i];
                    p1[k] = s * (Real)w0[t][i];
                    f1[t][i] = s * (Real)w1[t][i];
                }
        sample_sync<WL>();
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int l = at(t, i, xl), r = at(t, i, xr);
                    const Real lap = fma(Real(-4), rho[t][i], (p0[l] + p0[r]) + (p0[above(t, i, x)] + p0[below(t, i, x)]));
                    d[t][i] = a * lap;
                    dx[t][i] = p1[r] - p1[l];
                }
        sample_sync<WL>();
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) p1[at(t, i, x)] = f1[t][i];
        sample_sync<WL>();
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Real dy = p1[below(t, i, x)] - p1[above(t, i, x)];
                    d[t][i] = fma(kappa, dx[t][i] + dy, d[t][i]);
                }
    }

    // rho += u
    static __device__ __forceinline__ void advance(Real (&rho)[T][4], Real (&cmp)[T][4], const Acc (&u)[T])
    {
#pragma clang fp contract(off)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (F64) {
                    rho[t][i] = rho[t][i] + u[t][i];
                } else {
                    const Real yk = u[t][i] - cmp[t][i];
                    const Real tv = rho[t][i] + yk;
                    cmp[t][i] = (tv - rho[t][i]) - yk;
                    rho[t][i] = tv;
                }
            }
    }

    // sum of rho * phi over the sample in row sr of the tile's samples, valid in the lanes of lane group 0.
    // Products and sums carry their rounding errors: the centring that follows cancels most digits.
    __device__ __forceinline__ Sum inner(const Real (&rho)[T][4], const double* __restrict__ phi, int sr, bool on) const
    {
        Sum acc;
        if (on)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int y = row(t, i);
                    if (T == 1 && y / N != sr) continue;
                    acc.add_product((double)rho[t][i], phi[(y % N) * N + col() % N]);
                }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            if (off >= 16 || off < N) acc.add(__shfl_xor(acc.hi, off, 64), __shfl_xor(acc.lo, off, 64));
        return acc;
    }
};
}  // namespace

template <typename Real, int N, bool PAIR>
__global__ void __launch_bounds__(64 * TG<N>::WPB, TG<N>::WAVES) theta_kernel(const ThetaArgs A)
{
#pragma clang fp contract(off)
    constexpr int NC = PAIR ? N / 2 : N;                     // single paths: names a grid that is not used
    typedef TG<N> G;
    typedef Grid<Real, N, N> Fine;
    typedef Grid<Real, NC, N> Coarse;
    constexpr int T = G::T, TC = Coarse::T, TN = G::TN;
    constexpr bool WL = G::WL;
    constexpr int PLANE = Fine::PLANE > Coarse::PLANE ? Fine::PLANE : Coarse::PLANE;
    __shared__ Real planes[G::GPB * 2 * PLANE];
    __shared__ Real cas[N];
    __shared__ double red[G::WPB][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = lane >> 4, c = lane & 15, w = WL ? 0 : wave, p = c & 1;
    Real* p0 = planes + (WL ? wave : 0) * 2 * PLANE;
    Fine F{p0, p0 + PLANE, cas, w, q, c, {}};
    Coarse K{p0, p0 + PLANE, cas, w, q, c, {}};
    const bool on_c = w < TC;                                // wavefronts that own a tile of the coarse grid
    const Real a = (Real)A.a, kf = (Real)A.kf, kc = (Real)A.kc;

    for (int e = threadIdx.x; e < N; e += blockDim.x) cas[e] = ((const Real*)A.cas)[e];
    __syncthreads();
    F.init();
    if constexpr (PAIR) K.init();

    // sample of a tile slot; slots past the batch repeat its first sample and write nothing
    const uint64_t base = ((uint64_t)blockIdx.x * G::GPB + (WL ? wave : 0)) * G::SLOTS;
    auto sample = [&](int y, int x) { return base + (uint64_t)((y / N) * G::SIDE + x / N); };

    Real rho[T][4], cmp[T][4], rhoc[TC][4], cmpc[TC][4];
    Real Z[PAIR ? T : 1][2][2];                              // sums over the drawn site pairs and the steps
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rho[t][i] = ((const Real*)A.rho0_f)[(F.row(t, i) % N) * N + F.col() % N];
            cmp[t][i] = Real(0);
        }
        if constexpr (PAIR) Z[t][0][0] = Z[t][0][1] = Z[t][1][0] = Z[t][1][1] = Real(0);
    }
    if constexpr (PAIR)
#pragma unroll
        for (int t = 0; t < TC; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                rhoc[t][i] = on_c ? ((const Real*)A.rho0_c)[(K.row(t, i) % NC) * NC + K.col() % NC] : Real(0);
                cmpc[t][i] = Real(0);
            }
    // rows 16 t + row(2 d + p, q), d = 0, 1, are the lane's to draw
    NoiseKey key[2];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const uint64_t s = sample(Mma<Real>::row(2 * d + p, q), F.col());
        key[d] = make_key(A.seed, A.tag, A.level_id, A.first + (s < A.count ? s : 0));
    }

#pragma unroll 1
    for (int m = 0; m < A.steps; ++m) {
        F.place();
        const int q = F.q, p = F.c & 1;
        float w0[T][4], w1[T][4];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int y = 16 * t + Mma<Real>::row(2 * d + p, q);
                uint32_t idx = (uint32_t)((F.col() % N) / 2 + (N / 2) * (y % N));
                asm volatile("" : "+v"(idx));                // recomputed every step rather than kept live
                float a0, a1, b0, b1;
                site_pair_normals(key[G::SIDE > 1 ? d : 0], idx, (uint32_t)m, a0, a1, b0, b1);
                if constexpr (PAIR) {
                    Z[t][d][0] += (Real)a0 + (Real)b0;
                    Z[t][d][1] += (Real)a1 + (Real)b1;
                }
                const float r0 = swap_pair(p ? a0 : b0), r1 = swap_pair(p ? a1 : b1);
                w0[t][2 * d] = p ? r0 : a0;
                w0[t][2 * d + 1] = p ? b0 : r0;
                w1[t][2 * d] = p ? r1 : a1;
                w1[t][2 * d + 1] = p ? b1 : r1;
            }
        typename Fine::Acc u[T];
        F.template increment<WL, float>(rho, w0, w1, a, kf, u, true);
        if constexpr (!Fine::F64) Fine::advance(rho, cmp, u);
        F.filter(u, (const Real*)A.sol_f, true);
        Fine::advance(rho, cmp, u);
        if constexpr (PAIR) {
            if ((m & 3) == 3) {
                constexpr int H = TN / 2;                    // the coarse cells are the first H rows and columns
                F.place();
                K.place();
                const int q = F.q, p = F.c & 1;
                sample_sync<WL>();                           // the planes are read
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const int k = (16 * t + Mma<Real>::row(2 * d + p, q)) * H + F.col() / 2;
                        F.p0[k] = Z[t][d][0];
                        F.p1[k] = Z[t][d][1];
                        Z[t][d][0] = Z[t][d][1] = Real(0);
                    }
                sample_sync<WL>();
                Real z0[TC][4], z1[TC][4];
#pragma unroll
                for (int t = 0; t < TC; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int y = K.row(t, i), x = K.col(), k = 2 * y * H + x;
                        const bool in = y < H && x < H;
                        z0[t][i] = in ? F.p0[k] + F.p0[k + H] : Real(0);
                        z1[t][i] = in ? F.p1[k] + F.p1[k + H] : Real(0);
                    }
                typename Coarse::Acc v[TC];
                K.template increment<WL, Real>(rhoc, z0, z1, a, kc, v, on_c);
                if constexpr (!Fine::F64)
                    if (on_c) Coarse::advance(rhoc, cmpc, v);
                K.filter(v, (const Real*)A.sol_c, on_c);
                if (on_c) Coarse::advance(rhoc, cmpc, v);
            }
        }
    }

    // observables of eq. (eqn_MLMCLevels): FP64 inner products, the wavefronts' sums in their order
    auto write = [&](int j, int grid, uint64_t si, Sum L) {
        const double* ob = (grid == 0 ? A.obs_f : A.obs_c) + 3 * j;
        const double X = ob[0] * L.centred(grid == 0 ? A.h2f : A.h2c, ob[1]);
        double* dst = A.out + (si * A.n_obs + j) * 2;
        dst[grid] = ob[2] != 0.0 ? X * X : X;
        if (!PAIR) dst[1] = 0.0;
    };
    for (int j = 0; j < A.n_obs; ++j)
#pragma unroll
        for (int grid = 0; grid < (PAIR ? 2 : 1); ++grid)
#pragma unroll 1
            for (int sr = 0; sr < G::SIDE; ++sr) {
                Sum L;
                if (grid == 0) L = F.inner(rho, A.phi_f + (size_t)j * N * N, sr, true);
                else L = K.inner(rhoc, A.phi_c + (size_t)j * NC * NC, sr, on_c);
                const int n = grid == 0 ? N : NC;
                if constexpr (WL) {
                    const int sc = c / n;
                    const uint64_t si = base + (uint64_t)(sr * G::SIDE + sc);
                    if (q == 0 && c % n == 0 && sc < G::SIDE && si < A.count) write(j, grid, si, L);
                } else {
                    if (lane == 0) {
                        red[wave][0] = L.hi;
                        red[wave][1] = L.lo;
                    }
                    __syncthreads();
                    if (threadIdx.x == 0) {
                        Sum sum;
                        for (int k = 0; k < (grid == 0 ? T : TC); ++k) sum.add(red[k][0], red[k][1]);
                        if (base < A.count) write(j, grid, base, sum);
                    }
                    __syncthreads();
                }
            }
}

bool theta_supported(int n, bool pair) { return (n == 4 && !pair) || n == 8 || n == 16 || n == 32 || n == 64; }

template <int N>
static int blocks_of(uint64_t count) { return (int)std::min<uint64_t>((count + TG<N>::SPB - 1) / TG<N>::SPB, 0x7FFFFFFFull); }

int theta_grid(int n, int precision, uint64_t count)
{
    (void)precision;
    switch (n) {
    case 4: return blocks_of<4>(count);
    case 8: return blocks_of<8>(count);
    case 16: return blocks_of<16>(count);
    case 32: return blocks_of<32>(count);
    default: return blocks_of<64>(count);
    }
}

template <typename Real, int N, bool PAIR>
static hipError_t launch(const ThetaArgs& A, int grid, hipStream_t s)
{
    if ((uint64_t)grid * TG<N>::SPB < A.count) return hipErrorInvalidValue;
    hipLaunchKernelGGL((theta_kernel<Real, N, PAIR>), dim3(grid), dim3(64 * TG<N>::WPB), 0, s, A);
    return hipGetLastError();
}

template <typename Real, bool PAIR>
static hipError_t launch_n(const ThetaArgs& A, int grid, hipStream_t s)
{
    switch (A.n) {
    case 4: if constexpr (!PAIR) return launch<Real, 4, false>(A, grid, s); return hipErrorInvalidValue;
    case 8: return launch<Real, 8, PAIR>(A, grid, s);
    case 16: return launch<Real, 16, PAIR>(A, grid, s);
    case 32: return launch<Real, 32, PAIR>(A, grid, s);
    case 64: return launch<Real, 64, PAIR>(A, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_theta(const ThetaArgs& A, int precision, bool pair, int grid, hipStream_t s)
{
    if (!theta_supported(A.n, pair) || grid < 1 || (pair && A.steps % 4 != 0) || !A.cas || !A.sol_f || (pair && !A.sol_c))
        return hipErrorInvalidValue;
    if (precision == DK_PREC_F64) return pair ? launch_n<double, true>(A, grid, s) : launch_n<double, false>(A, grid, s);
    return pair ? launch_n<float, true>(A, grid, s) : launch_n<float, false>(A, grid, s);
}

}  // namespace dk
