// dk_fourier.hip -- level kernel of the Fourier coupling (Sec. 3.1): h_{l-1} = 3 h_l and
// tau_{l-1} = 9 tau_l, grids n_l = n_0 3^l up to 108 x 108.
//
// The fine level runs the scheme of eq. (FullyDiscreteDK) with the nodal noise of every other
// level (the same generator and counters): in the orthonormal Fourier basis of the grid
// functions its coefficients are exactly the family of complex Brownian increments of
// Sec. 3.1.  The coarse level reuses the coefficients of the frequencies it resolves, summed
// over its 9 fine steps; in real space that is the fine normals summed over the coarse step,
// projected onto the coarse frequencies and read at the coarse nodes, i.e. the separable map
// S -> K S K^T with the [nc][nf] kernel K[ic][i] = k(3 ic - i), k even and periodic (a sum of cosines;
// on the coarse Nyquist frequency the two fine aliases enter with weight 2^{-1/2} each, which makes
// the coarse noise real with the coarse level's own law).  The projected sums have unit variance
// per coarse node, so the coarse noise coefficient is kc = kf h_f / h_c.
//
// Layout: the register tiles of the resident level kernel (tile_step in dk_level.h) on grids that are
// not powers of two.  A lane owns C columns and R rows; a row group of n / C lanes sits inside one
// wavefront (54 of 64 lanes at 108 x 108), whose remaining lanes repeat its first lane's work, writes
// included.  A lane keeps the running sums of its cells' normals beside the state.  At the end of a
// coarse step the sums of one direction go to LDS and the matrix cores form K S K^T in one go: a
// wavefront multiplies 16 rows of S by K^T (A = S from LDS, B from the table k), and the product's
// registers are, as they stand, the right operand of the product by K that follows
// (v_mfma_f64_16x16x4_f64 returns row 4 i + q of its result where it takes row 4 i + q of its second
// factor), so the half-projected sums are never stored.  The coarse state is in LDS, a cell per lane.
//
// Bound by the vector ALU (Philox, Box--Muller, one FP64 root per cell).  The first kernel held the
// state and the normals in LDS, four roots a cell and five barriers a step, and projected through L2:
// 500 pairs of 108 x 108 took 63.8 ms (6.7e10 cell updates/s), now 16.8 ms (2.5e11).  Rows per lane: the most
// that leave the sums in registers at 108 x 108 (9 x 2 cells, three wavefronts per SIMD); four on the
// small grids, whose batches rarely fill the chip.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "dk_fourier.h"
#include "dk_level.h"
#include "dk_mma.h"
#include "dk_sum.h"

namespace dk {

namespace {
template <int NF>
struct FG {
    static constexpr int C = NF == 72 ? 4 : 2;                       // 72: 18 lanes a row, three rows a wavefront
    static constexpr int R = NF == 108 ? 9 : (NF == 24 || NF == 72 ? 6 : 4);
    static constexpr int NPL = NF / C, G = NF / R;                   // lanes per row group, row groups
    static constexpr int GPW = 64 / NPL;                             // row groups a wavefront can hold
    static constexpr bool WL = G <= GPW;                             // a sample (or several) per wavefront
    static constexpr int SEG = NPL * (WL ? G : GPW);                 // lanes of a sample in a wavefront
    static constexpr int SPW = WL ? 64 / SEG : 1;                    // samples per wavefront
    static constexpr int W = WL ? 1 : G / GPW;                       // wavefronts of a sample
    static constexpr int WPB = WL ? 4 : W;                           // wavefronts of a block
    static constexpr int SPB = WL ? WPB * SPW : 1;                   // samples of a block
    static constexpr int NC = NF / 3, NCC = NC * NC;
    static constexpr int PITCH = NF + 2;                             // sums in LDS: 16 rows without bank conflicts
    static constexpr int YT = (NF + 15) / 16, CT = (NC + 15) / 16;   // 16 x 16 tiles of the products
    static constexpr int PARTS = W / CT > 0 ? W / CT : 1;            // wavefronts that share a column tile
    static_assert(NF % R == 0 && (WL || G % GPW == 0) && (WL || W % CT == 0), "whole tiles");
    // Reals of one sample's LDS: halo rows, the sums of one direction or partial products; z, rho_c
    static constexpr int HALO = 2 * G * 4 * NF;
    static constexpr int SUMS = NF * PITCH;
    static constexpr int PARTIAL = WL ? 0 : PARTS * CT * CT * 256;
    static constexpr int AREA1 = HALO;                               // single paths
    static constexpr int AREA2 = HALO > SUMS ? (HALO > PARTIAL ? HALO : PARTIAL) : (SUMS > PARTIAL ? SUMS : PARTIAL);
};

// The fine normals of a tile, added to the running sums of the coarse step.
template <typename Real, int R, int C, bool PAIR>
struct FourierNoise {
    NoiseKey key;
    uint32_t step, pair_base, pairs_per_row;
    Real (*S)[C][2];
    using W = float;
    static __device__ __forceinline__ Real root(Real x)
    {
        if constexpr (std::is_same<Real, double>::value) return pos_sqrt_f64(x);
        else return sqrt(x > Real(0) ? x : Real(0));
    }

    template <int I>
    __device__ __forceinline__ void row(W (&w0)[C], W (&w1)[C])
    {
#pragma unroll
        for (int cp = 0; cp < C / 2; ++cp) {
            float a0, a1, b0, b1;
            uint32_t idx = pair_base + (uint32_t)I * pairs_per_row + cp;
            asm volatile("" : "+v"(idx));      // recomputed every step rather than kept live (see FineNoise)
            site_pair_normals(key, idx, step, a0, a1, b0, b1);
            w0[2 * cp] = a0;
            w1[2 * cp] = a1;
            w0[2 * cp + 1] = b0;
            w1[2 * cp + 1] = b1;
            if constexpr (PAIR) {
                S[I][2 * cp][0] += Real(a0);
                S[I][2 * cp][1] += Real(a1);
                S[I][2 * cp + 1][0] += Real(b0);
                S[I][2 * cp + 1][1] += Real(b1);
            }
        }
    }
};

// acc[jt] += K[16 jt ..][y] (S K^T)[y][16 ct ..] over the row tiles part, part + parts, ..
template <typename Real, int NF>
__device__ __forceinline__ void project(const Real* S, const Real* ktab, int ct, int part, int lane,
                                        typename Mma<Real>::Acc (&acc)[FG<NF>::CT])
{
    typedef Mma<Real> M;
    typedef FG<NF> F;
    const int i16 = lane & 15, q = lane >> 4;
    const int ic = 3 * (16 * ct + i16) % NF;
#pragma unroll 1
    for (int yt = part; yt < F::YT; yt += F::PARTS) {
        const Real* row = S + min(16 * yt + i16, NF - 1) * F::PITCH + q;
        int d = ic - q;
        d += d < 0 ? NF : 0;
        typename M::Acc t = {0, 0, 0, 0};
#pragma unroll 3
        for (int x = 0; x < NF; x += 4) {
            t = M::mul(row[x], ktab[d], t);
            d -= 4;
            d += d < 0 ? NF : 0;
        }
#pragma unroll
        for (int jt = 0; jt < F::CT; ++jt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int y = 16 * yt + M::row(i, q);
                int e = 3 * (16 * jt + i16) % NF - (y < NF ? y : 0);
                e += e < 0 ? NF : 0;
                acc[jt] = M::mul(y < NF ? ktab[e] : Real(0), t[i], acc[jt]);
            }
    }
}
}  // namespace

template <typename Real, int NF, bool PAIR>
__global__ void __launch_bounds__(64 * FG<NF>::WPB) fourier_kernel(const FourierArgs A)
{
#pragma clang fp contract(off)
    typedef FG<NF> F;
    typedef Mma<Real> M;
    constexpr int R = F::R, C = F::C, NPL = F::NPL, G = F::G, NC = F::NC, NCC = F::NCC;
    constexpr bool WL = F::WL, COMP = std::is_same<Real, float>::value;
    constexpr int AREA = PAIR ? F::AREA2 : F::AREA1;
    constexpr int CSLOTS = (NCC + F::SEG * F::W - 1) / (F::SEG * F::W);    // coarse cells per lane
    __shared__ __align__(16) Real area[F::SPB * AREA];
    __shared__ Real zc_[PAIR ? F::SPB * 2 * NCC : 1];
    __shared__ Real rhoc_[PAIR ? F::SPB * NCC : 1];
    __shared__ Real ktab[PAIR ? NF : 1];
    __shared__ double red[F::SPW > 1 ? F::WPB * 64 : F::WPB][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // lanes beyond the wavefront's samples repeat lane 0
    const bool own = lane < F::SPW * F::SEG;
    const int l = own ? lane : 0;
    const int slot = l / F::SEG, ls = l % F::SEG;
    const int g = (WL ? 0 : wave * F::GPW) + ls / NPL, cl = ls % NPL;
    const int addr_l = (l - cl + (cl + NPL - 1) % NPL) * 4, addr_r = (l - cl + (cl + 1) % NPL) * 4;
    const int row0 = R * g, col0 = C * cl;
    const int sb = WL ? wave * F::SPW + slot : 0;            // sample of the block
    const uint64_t local = (uint64_t)blockIdx.x * F::SPB + sb;
    const bool active = local < A.count;
    const uint64_t si = active ? local : 0;
    Real* my = area + sb * AREA;
    Real* zc = zc_ + (PAIR ? sb * 2 * NCC : 0);
    Real* rhoc = rhoc_ + (PAIR ? sb * NCC : 0);
    const int cc0 = WL ? ls : wave * F::SEG + ls;            // first coarse cell of the lane

    Real rho[R][C], cmp[R][C], S[PAIR ? R : 1][C][2], cmpc[CSLOTS];
    {
        const Real* r0 = (const Real*)A.rho0_f;
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                rho[i][c] = r0[(row0 + i) * NF + col0 + c];
                cmp[i][c] = Real(0);
                if constexpr (PAIR) S[i][c][0] = S[i][c][1] = Real(0);
            }
    }
    if constexpr (PAIR) {
        const Real* r0 = (const Real*)A.rho0_c;
        for (int k = 0; k < CSLOTS; ++k) {
            cmpc[k] = Real(0);
            const int c = cc0 + k * F::SEG * F::W;
            if (c < NCC) rhoc[c] = r0[c];
        }
        for (int e = threadIdx.x; e < NF; e += blockDim.x) ktab[e] = ((const Real*)A.K)[e];
        __syncthreads();
    }
    const NoiseKey key = make_key(A.seed, A.tag, A.level_id, A.first + si);
    const Real a = (Real)A.a, kf = (Real)A.kf, kc = (Real)A.kc;

    auto fine_step = [&](int m) {
        FourierNoise<Real, R, C, PAIR> fn{key, (uint32_t)m, (uint32_t)(col0 / 2 + row0 * (NF / 2)), (uint32_t)(NF / 2),
                                          PAIR ? S : nullptr};
        tile_step<Real, R, C, DK_FLUX_CENTRAL, COMP, true, WL>(rho, cmp, fn, a, kf, my + (m & 1) * G * 4 * NF, g, G, cl, NF, addr_l,
                                                               addr_r);
    };
    if constexpr (!PAIR) {
#pragma unroll 1
        for (int m = 0; m < A.steps; ++m) fine_step(m);
    } else {
#pragma unroll 1
        for (int m0 = 0; m0 < A.steps; m0 += 9) {
#pragma unroll 1
            for (int j = 0; j < 9; ++j) fine_step(m0 + j);
            // the coarse step: its noise, one direction after the other
            // Everything the coarse step derives from the lane index is derived again here: kept across the
            // fine steps it would take the registers that the sums need.
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63, wave = tid >> 6;
            const int l = lane < F::SPW * F::SEG ? lane : 0;
            const int slot = l / F::SEG, ls = l % F::SEG;
            const int g = (WL ? 0 : wave * F::GPW) + ls / NPL, cl = ls % NPL, row0 = R * g, col0 = C * cl;
            const int sb = WL ? wave * F::SPW + slot : 0, cc0 = WL ? ls : wave * F::SEG + ls;
            Real* my = area + sb * AREA;
            Real* zc = zc_ + sb * 2 * NCC;
            Real* rhoc = rhoc_ + sb * NCC;
            sample_sync<WL>();                               // the last step's halo is read
#pragma unroll
            for (int r = 0; r < 2; ++r) {
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        my[(row0 + i) * F::PITCH + col0 + c] = S[i][c][r];
                        S[i][c][r] = Real(0);
                    }
                sample_sync<WL>();
                const int ct = WL ? 0 : wave % F::CT, part = WL ? 0 : wave / F::CT;
                if constexpr (WL) {
                    for (int s = 0; s < F::SPW; ++s) {       // every sample of the wavefront in turn
                        typename M::Acc z[F::CT] = {};
                        project<Real, NF>(area + (wave * F::SPW + s) * AREA, ktab, 0, 0, lane, z);
                        Real* zs = zc_ + (wave * F::SPW + s) * 2 * NCC + r * NCC;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int jc = M::row(i, lane >> 4), ic = lane & 15;
                            if (jc < NC && ic < NC) zs[jc * NC + ic] = z[0][i];
                        }
                    }
                    sample_sync<WL>();
                } else {
                    typename M::Acc z[F::CT] = {};
                    project<Real, NF>(my, ktab, ct, part, lane, z);
                    __syncthreads();                         // the sums are read; their place takes the partial products
#pragma unroll
                    for (int jt = 0; jt < F::CT; ++jt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            my[((part * F::CT + ct) * F::CT + jt) * 256 + M::row(i, lane >> 4) * 16 + (lane & 15)] = z[jt][i];
                    __syncthreads();
                    for (int c = tid; c < NCC; c += 64 * F::WPB) {
                        const int jc = c / NC, ic = c % NC;
                        Real v = Real(0);
#pragma unroll
                        for (int p = 0; p < F::PARTS; ++p)
                            v += my[((p * F::CT + ic / 16) * F::CT + jc / 16) * 256 + (jc % 16) * 16 + ic % 16];
                        zc[r * NCC + c] = v;
                    }
                    __syncthreads();
                }
            }
            Real nv[CSLOTS];
#pragma unroll
            for (int k = 0; k < CSLOTS; ++k) {
                const int c = cc0 + k * F::SEG * F::W;
                nv[k] = Real(0);
                if (c >= NCC) continue;
                const int x = c % NC, y = c / NC;
                const int xl = x == 0 ? c + NC - 1 : c - 1, xr = x == NC - 1 ? c + 1 - NC : c + 1;
                const int yu = y == 0 ? c + NCC - NC : c - NC, yd = y == NC - 1 ? c + NC - NCC : c + NC;
                auto flux = [&](int r, int at) { return FourierNoise<Real, R, C, PAIR>::root(rhoc[at]) * zc[r * NCC + at]; };
                const Real rv = rhoc[c];
                const Real dx = flux(0, xr) - flux(0, xl), dy = flux(1, yd) - flux(1, yu);
                const Real lap = fma(Real(-4), rv, (rhoc[xl] + rhoc[xr]) + (rhoc[yu] + rhoc[yd]));
                const Real d = fma(kc, dx + dy, a * lap);
                if constexpr (COMP) {
                    const Real yk = d - cmpc[k];
                    const Real tv = rv + yk;
                    cmpc[k] = (tv - rv) - yk;
                    nv[k] = tv;
                } else {
                    nv[k] = rv + d;
                }
            }
            sample_sync<WL>();
#pragma unroll
            for (int k = 0; k < CSLOTS; ++k) {
                const int c = cc0 + k * F::SEG * F::W;
                if (c < NCC) rhoc[c] = nv[k];
            }
            // read again after the next coarse step's barriers
        }
    }

    // observables of eq. (eqn_MLMCLevels): FP64 inner products; the lanes' sums in lane order, then the
    // wavefronts' in theirs
    __syncthreads();
    for (int j = 0; j < A.n_obs; ++j) {
#pragma unroll
        for (int grid = 0; grid < (PAIR ? 2 : 1); ++grid) {
            Sum acc;
            if (grid == 0) {
                const double* ph = A.phi_f + (size_t)j * NF * NF;
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int c = 0; c < C; ++c) acc.add_product((double)rho[i][c], ph[(row0 + i) * NF + col0 + c]);
            } else {
                const double* ph = A.phi_c + (size_t)j * NCC;
                for (int c = cc0; c < NCC; c += F::SEG * F::W) acc.add_product((double)rhoc[c], ph[c]);
            }
            Sum L;
            if constexpr (F::SPW > 1) {
                red[threadIdx.x][0] = acc.hi;
                red[threadIdx.x][1] = acc.lo;
                sample_sync<WL>();
                if (own && ls == 0)
                    for (int k = 0; k < F::SEG; ++k) L.add(red[threadIdx.x + k][0], red[threadIdx.x + k][1]);
                sample_sync<WL>();
            } else {
                acc.hi = own ? acc.hi : 0.0;
                acc.lo = own ? acc.lo : 0.0;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) acc.add(__shfl_xor(acc.hi, off, 64), __shfl_xor(acc.lo, off, 64));
                L = acc;
                if constexpr (F::W > 1) {
                    if (lane == 0) {
                        red[wave][0] = acc.hi;
                        red[wave][1] = acc.lo;
                    }
                    __syncthreads();
                    L = Sum();
                    for (int w = 0; w < F::W; ++w) L.add(red[w][0], red[w][1]);
                    __syncthreads();
                }
            }
            if (own && active && ls == 0 && (WL || wave == 0)) {
                const double* ob = (grid == 0 ? A.obs_f : A.obs_c) + 3 * j;
                const double X = ob[0] * L.centred(grid == 0 ? A.h2f : A.h2c, ob[1]);
                double* dst = A.out + (si * A.n_obs + j) * 2;
                dst[grid] = ob[2] != 0.0 ? X * X : X;
                if (!PAIR) dst[1] = 0.0;
            }
        }
    }
}

bool fourier_supported(int nf, bool pair)
{
    switch (nf) {
    case 4: case 8: return !pair;
    case 12: case 24: case 36: case 72: case 108: return true;
    default: return false;
    }
}

template <int NF>
static int blocks_of(uint64_t count) { return (int)std::min<uint64_t>((count + FG<NF>::SPB - 1) / FG<NF>::SPB, 0x7FFFFFFFull); }

int fourier_grid(int nf, int precision, uint64_t count)
{
    (void)precision;
    switch (nf) {
    case 4: return blocks_of<4>(count);
    case 8: return blocks_of<8>(count);
    case 12: return blocks_of<12>(count);
    case 24: return blocks_of<24>(count);
    case 36: return blocks_of<36>(count);
    case 72: return blocks_of<72>(count);
    default: return blocks_of<108>(count);
    }
}

template <typename Real, int NF, bool PAIR>
static hipError_t launch(const FourierArgs& A, int grid, hipStream_t s)
{
    if ((uint64_t)grid * FG<NF>::SPB < A.count) return hipErrorInvalidValue;
    hipLaunchKernelGGL((fourier_kernel<Real, NF, PAIR>), dim3(grid), dim3(64 * FG<NF>::WPB), 0, s, A);
    return hipGetLastError();
}

template <typename Real, bool PAIR>
static hipError_t launch_nf(const FourierArgs& A, int grid, hipStream_t s)
{
    switch (A.nf) {
    case 4: if constexpr (!PAIR) return launch<Real, 4, false>(A, grid, s); return hipErrorInvalidValue;
    case 8: if constexpr (!PAIR) return launch<Real, 8, false>(A, grid, s); return hipErrorInvalidValue;
    case 12: return launch<Real, 12, PAIR>(A, grid, s);
    case 24: return launch<Real, 24, PAIR>(A, grid, s);
    case 36: return launch<Real, 36, PAIR>(A, grid, s);
    case 72: return launch<Real, 72, PAIR>(A, grid, s);
    case 108: return launch<Real, 108, PAIR>(A, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fourier(const FourierArgs& A, int precision, bool pair, int grid, hipStream_t s)
{
    if (!fourier_supported(A.nf, pair) || grid < 1 || (pair && (A.steps % 9 != 0 || !A.K))) return hipErrorInvalidValue;
    if (precision == DK_PREC_F64) return pair ? launch_nf<double, true>(A, grid, s) : launch_nf<double, false>(A, grid, s);
    return pair ? launch_nf<float, true>(A, grid, s) : launch_nf<float, false>(A, grid, s);
}

}  // namespace dk
