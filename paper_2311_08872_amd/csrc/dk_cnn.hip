// dk_cnn.hip -- the control-variate network on gfx950: forward, backward and Adam.
//
// Network (coarse final field -> prediction of the level correction Y):
//   conv 3x3 1->16 (circular) + ReLU, conv 3x3 16->16 + ReLU, conv 3x3 16->16 + ReLU,
//   global average pool, dense 16->64 + ReLU, dense 64->1.
// Parameters are FP32 masters, flat in the order W1 b1 W2 b2 W3 b3 U1 c1 U2 c2 with conv
// weights [o][c][ky][kx] and dense weights [out][in] (5953 values).
//
// Numbers: the 16->16 convolutions multiply BF16 operands on v_mfma_f32_16x16x32_bf16 with FP32
// accumulation; each layer's output (and each gradient at a layer's output) is rounded to BF16
// once; the first layer and its weight gradient (v_mfma_f32_16x16x4_f32), pooling and the dense head
// are FP32 throughout.
//
// Forward (one block per tile of at most 32 x 16 pixels): the tile of x with a halo of 3 comes to
// LDS once, the first layer writes its 16 channels there with a halo of 2, the second reads it and
// writes beside it, the third adds its outputs to the tile's channel sums (several samples in a block: by
// way of LDS): nothing but x is read from HBM and nothing but 16 sums per tile is written (the training
// pass writes the three activations and a 16-bit ReLU mask per pixel instead).  Grids of at most 16 x 16
// put several samples into one block.  A layer as its own pass over HBM moved 64 B per pixel and
// layer and summed the pool in one thread per (sample, channel): 4.64 ms for 4000 inputs of 64 x 64
// (0.85 ms per 1024 of it the pool) against 0.51 ms now, bound by the vector ALU (roundings and packing, ReLU,
// addresses) and the five LDS reads of 1 KB per 16 pixels and layer.
// An activation image is two planes of 8 channels, 16 B per pixel each, so the 16 pixels of an MFMA
// operand are 256 consecutive bytes.  The register bounds keep the accumulators among the vector registers:
// without them the compiler puts them into the second file and moves every result (4 % of the kernel).
//
// Backward: per layer one kernel whose blocks stride over tiles (halo 1) and hold the weight
// gradient in MFMA accumulators for their whole run: A = gradient [o][pixel], B = activation
// [pixel][c], both from LDS images transposed to [channel][pixel]; the nine neighbour shifts are the
// three rows of the image times {funnel shift left, none, funnel shift right} of one 16-byte row
// piece.  The bias gradient is a tenth product with a column of ones.  The same kernel convolves the
// gradient back to the layer's input.  Per-block partial sums are added in block order by the last
// kernel, which also forms the dense head's gradients.  Loss and gradient at 64 x 64, batch 256:
// 4.01 ms with one kernel per product (2-byte gathers, serial column sums, 27 launches), 0.29 ms now.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "dk_cnn.h"

namespace dk {
namespace cnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// rounded to nearest even by the hardware conversion (a pair is one instruction, where the integer
// sequence takes nine)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

// x / d for 0 <= x < 2^16 and 1 <= d < 2^11 in three full-rate instructions: (x + 1/2) / d is at least 1 / (2 d)
// away from an integer, its two roundings at most x / d 2^-22 (a 32-bit high product takes four times as long)
struct Div {
    float inv, half;
    __host__ __device__ Div(uint32_t v = 1) : inv(1.0f / (float)(v < 1 ? 1 : v)), half(0.5f * inv) {}
    __device__ __forceinline__ int q(int x) const { return (int)fmaf((float)x, inv, half); }
};

__device__ __forceinline__ int wrapn(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// ---------------------------------------------------------------------------------------
// Tiles.  A sample's n x n pixels are cut into tx x ty tiles of tw x th pixels (the last ones may
// be smaller); a block holds S samples when one tile covers a sample, one tile otherwise.
// ---------------------------------------------------------------------------------------
struct Geo {
    int n, batch, tw, th, tx, ty, S;
    int H;              // halo of the image
    int P, img, L;      // image pitch, pixels of one sample's image, of all S
    int groups;         // ceil(batch / S) x tiles per sample: work items
    Div dP, dImg, dTw, dTile;
};

constexpr int kTileW = 32, kTileH = 16;
constexpr int kFwdThreads = 256;    // three blocks per compute unit (LDS); 512 threads run at the same speed
constexpr int kFwdL = 728;          // image pixels (halo 2) of a forward block: 36 x 20 fit
constexpr int kFwdX = 1040;         // x pixels (halo 3)
constexpr int kBwdL = 616;          // image pixels (halo 1) of a backward block: 34 x 18 fit
constexpr int kBwdA = 872;          // transposed activation image: pixels per channel (18 rows of 48 fit)
constexpr int kBwdZ = 520;          // transposed gradient tile: pixels per channel
constexpr int kForwardTiles = 1 << 17;   // of one forward pass: 8 MB of sums
constexpr int kBlocks = 512;        // two blocks per compute unit: the backward grid, and what small grids are spread to

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

static Geo make_geo(int n, int batch, int H)
{
    Geo g;
    g.n = n;
    g.batch = batch;
    g.H = H;
    g.tx = cdiv(n, kTileW);
    g.tw = 4 * cdiv(n / 4, g.tx);
    g.tx = cdiv(n, g.tw);
    g.ty = cdiv(n, kTileH);
    g.th = cdiv(n, g.ty);
    g.ty = cdiv(n, g.th);
    g.P = g.tw + 2 * H;
    g.img = g.P * (g.th + 2 * H);
    g.S = 1;
    if (g.tx * g.ty == 1) {
        const int units = cdiv(g.tw, 8), rp = 8 * units + 16;
        int most;
        if (H == 2) most = std::min(kFwdL / g.img, kFwdX / ((g.tw + 6) * (g.th + 6)));
        else most = std::min({kBwdL / g.img, (kBwdA - 8) / ((g.th + 2) * rp), (kBwdZ - 8) / (g.th * units * 8)});
        // as many samples as fit, unless that leaves compute units idle
        g.S = std::max(1, std::min(most, cdiv(batch, kBlocks)));
    }
    g.L = g.S * g.img;
    g.groups = cdiv(batch, g.S) * g.tx * g.ty;
    g.dP = Div(g.P);
    g.dImg = Div(g.img);
    g.dTw = Div(g.tw);
    g.dTile = Div(g.tw * g.th);
    return g;
}

struct TileAt {
    int b0, x0, y0, tw, th;     // first sample, first pixel, pixels of this tile
};

__device__ __forceinline__ TileAt tile_at(const Geo& g, int item)
{
    const int tiles = g.tx * g.ty;
    const int grp = item / tiles, t = item - grp * tiles;
    const int ty = t / g.tx, txx = t - ty * g.tx;
    TileAt a;
    a.b0 = grp * g.S;
    a.x0 = txx * g.tw;
    a.y0 = ty * g.th;
    a.tw = min(g.tw, g.n - a.x0);
    a.th = min(g.th, g.n - a.y0);
    return a;
}

// MFMA operand of the weights: row i of the packed layout [16][160], k = 32 s + 8 kg ..
__device__ __forceinline__ void load_weights(uint4 (&w)[5], const uint16_t* __restrict__ Wk, int lane)
{
#pragma unroll
    for (int s = 0; s < 5; ++s) w[s] = *(const uint4*)(Wk + (lane & 15) * 160 + 32 * s + 8 * (lane >> 4));
}

// 3x3 16->16 products of 16 consecutive image pixels starting at idx0: D[row = output channel]
// [column = pixel], K = 9 neighbours x 16 channels = 144 padded to 160.  off[s]: the lane's
// neighbour offset of K-step s.
__device__ __forceinline__ floatx4 conv16(const uint4* __restrict__ img, int plane, int idx0, const int (&off)[5],
                                          const uint4 (&w)[5], int lane)
{
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    const int i = lane & 15, kg = lane >> 4;
    const uint4* p = img + (kg & 1) * plane + idx0 + i;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        uint4 v = p[off[s]];
        if (s == 4 && kg >= 2) v = make_uint4(0, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s]), __builtin_bit_cast(bf16x8, v), acc, 0,
                                                       0, 0);
    }
    return acc;
}

__device__ __forceinline__ void neighbour_offsets(int (&off)[5], int P, int lane, int sign)
{
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        const int pos = 2 * s + (lane >> 5);
        off[s] = pos < 9 ? sign * ((pos / 3 - 1) * P + (pos % 3 - 1)) : 0;
    }
}

// ---------------------------------------------------------------------------------------
// Forward: the three convolutions of one tile.  KEEP (training): writes the activations a1, a2, a3 ([pixel][16]
// BF16) and the third layer's ReLU mask.  Else gpart[sample][tile][16] receives the tile's channel sums.
// ---------------------------------------------------------------------------------------
template <bool KEEP>
__global__ void __launch_bounds__(kFwdThreads, 3) conv_fwd(const Geo g, const float* __restrict__ x, const float* __restrict__ prm,
                                                const uint16_t* __restrict__ wt2, const uint16_t* __restrict__ wt3,
                                                float* __restrict__ gpart, uint16_t* __restrict__ a1g,
                                                uint16_t* __restrict__ a2g, uint16_t* __restrict__ a3g,
                                                uint16_t* __restrict__ m3g)
{
    constexpr int PL = kFwdL + 16;                 // plane: the last group of 16 reads past the image
    __shared__ float sx[kFwdX];
    __shared__ uint4 sA[2 * PL];
    __shared__ uint4 sB[2 * PL];
    constexpr int WAVES = kFwdThreads / 64;
    __shared__ float sred[WAVES * 16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const TileAt T = tile_at(g, blockIdx.x);
    const int n = g.n, P = g.P, L = g.L;
    const size_t nn = (size_t)n * n;
    // x with halo 3
    {
        const int xp = g.tw + 6, xi = xp * (g.th + 6);
        const Div dxp(xp), dxi(xi);
        for (int e = t; e < g.S * xi; e += kFwdThreads) {
            const int s = dxi.q(e), r = e - s * xi, yy = dxp.q(r), xx = r - yy * xp;
            const int b = min(T.b0 + s, g.batch - 1);
            sx[e] = x[b * nn + (size_t)wrapn(T.y0 + yy - 3, n) * n + wrapn(T.x0 + xx - 3, n)];
        }
    }
    uint4 w2[5], w3[5];
    load_weights(w2, wt2, lane);
    load_weights(w3, wt3, lane);
    __syncthreads();
    const int i = lane & 15, kg = lane >> 4;
    // First layer on the whole image (halo 2): 16 pixels by 16 outputs, K = 9 neighbours padded to 12 on the FP32
    // matrix instruction, which adds its four products in order, each fused and rounded, as nine multiply-adds do.
    // A fused multiply-add of its own per product took a third of the kernel's vector instructions.
    {
        const int xp = g.tw + 6, xi = xp * (g.th + 6);
        float w1[3], b1[4];
        int o[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int pos = min(4 * k + kg, 8);
            w1[k] = 4 * k + kg < 9 ? prm[OFF_W1 + 9 * i + pos] : 0.0f;
            o[k] = (pos / 3) * xp + pos % 3;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) b1[r] = prm[OFF_B1 + 4 * kg + r];
        for (int g0 = 16 * wave; g0 < L; g0 += 16 * WAVES) {
            const int e = min(g0 + i, L - 1), s = g.dImg.q(e), r = e - s * g.img, yy = g.dP.q(r), xx = r - yy * P;
            const float* c = sx + s * xi + yy * xp + xx;
            floatx4 acc = {b1[0], b1[1], b1[2], b1[3]};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float v = c[o[k]];
                if (k == 2 && kg > 0) v = 0.0f;
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[k], v, acc, 0, 0, 0);
            }
            ((uint2*)&sA[(kg >> 1) * PL + e])[kg & 1] =
                make_uint2(pack2(fmaxf(acc[0], 0.0f), fmaxf(acc[1], 0.0f)), pack2(fmaxf(acc[2], 0.0f), fmaxf(acc[3], 0.0f)));
        }
    }
    __syncthreads();
    int off[5];
    neighbour_offsets(off, P, lane, 1);
    // One layer: image pixels [lo, hi) of src -> dst, over the image's linear index (tile rows and their halo columns
    // alike; what comes out in halo columns is not used).  The neighbours are added row by row, as by the backward
    // pass: with two rows of outputs from one operand (5 % faster) they were added column by column, other BF16
    // roundings followed, and outputs moved by up to 4e-5 of their RMS on small grids.
    // POOL (one sample a block): the outputs inside the tile are added to v4 and not written.
    float v4[4] = {0.f, 0.f, 0.f, 0.f};
    auto layer = [&](const uint4* src, uint4* dst, const uint4 (&w)[5], const float* bias, int lo, int hi, auto pool) {
        constexpr bool POOL = decltype(pool)::value;
        float b4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) b4[r] = bias[4 * kg + r];
        for (int g0 = lo + 16 * wave; g0 < hi; g0 += 16 * WAVES) {
            const floatx4 acc = conv16(src, PL, g0, off, w, lane);
            const uint2 o = make_uint2(pack2(fmaxf(acc[0] + b4[0], 0.0f), fmaxf(acc[1] + b4[1], 0.0f)),
                                       pack2(fmaxf(acc[2] + b4[2], 0.0f), fmaxf(acc[3] + b4[3], 0.0f)));
            if constexpr (!POOL) ((uint2*)&dst[(kg >> 1) * PL + g0 + i])[kg & 1] = o;
            if constexpr (POOL) {
                const int q = g0 + i, yy = g.dP.q(q), xx = q - yy * P - 2;
                const bool in = q < hi && (unsigned)(yy - 2) < (unsigned)T.th && (unsigned)xx < (unsigned)T.tw;
                v4[0] += __uint_as_float(in ? o.x << 16 : 0u);
                v4[1] += __uint_as_float(in ? o.x & 0xFFFF0000u : 0u);
                v4[2] += __uint_as_float(in ? o.y << 16 : 0u);
                v4[3] += __uint_as_float(in ? o.y & 0xFFFF0000u : 0u);
            }
        }
    };
    // interior pixels of an image in LDS to global memory, 16 B per thread
    auto keep = [&](const uint4* src, uint16_t* dst) {
        const int tile = g.tw * g.th;
        for (int e = t; e < g.S * tile * 2; e += kFwdThreads) {
            const int h = e & 1, q = e >> 1, s = g.dTile.q(q), r = q - s * tile, yy = g.dTw.q(r), xx = r - yy * g.tw;
            if (T.b0 + s < g.batch && yy < T.th && xx < T.tw)
                *(uint4*)(dst + ((T.b0 + s) * nn + (size_t)(T.y0 + yy) * n + T.x0 + xx) * 16 + 8 * h) =
                    src[h * PL + s * g.img + (yy + 2) * P + xx + 2];
        }
    };
    layer(sA, sB, w2, prm + OFF_B2, P + 1, L - P - 1, std::false_type());
    if constexpr (KEEP) keep(sA, a1g);
    __syncthreads();
    if (!KEEP && g.S == 1) layer(sB, sA, w3, prm + OFF_B3, 2 * P + 2, L - 2 * P - 2, std::true_type());
    else layer(sB, sA, w3, prm + OFF_B3, 2 * P + 2, L - 2 * P - 2, std::false_type());
    if constexpr (KEEP) keep(sB, a2g);
    __syncthreads();
    if constexpr (KEEP) {
        keep(sA, a3g);
        const int tile = g.tw * g.th;
        for (int q = t; q < g.S * tile; q += kFwdThreads) {
            const int s = g.dTile.q(q), r = q - s * tile, yy = g.dTw.q(r), xx = r - yy * g.tw;
            const int c = s * g.img + (yy + 2) * P + xx + 2;
            uint32_t m = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 v = sA[h * PL + c];
                const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    m |= (uint32_t)((d[k] & 0x7FFFu) != 0) << (8 * h + 2 * k);
                    m |= (uint32_t)((d[k] & 0x7FFF0000u) != 0) << (8 * h + 2 * k + 1);
                }
            }
            if (T.b0 + s < g.batch && yy < T.th && xx < T.tw)
                m3g[(T.b0 + s) * nn + (size_t)(T.y0 + yy) * n + T.x0 + xx] = (uint16_t)m;
        }
        return;
    }
    // channel sums.  One sample a block: of the third layer's lanes, over the block
    if (g.S == 1) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) v4[k] += __shfl_xor(v4[k], o, 64);
        if (i == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) sred[wave * 16 + 4 * kg + k] = v4[k];
        __syncthreads();
        if (t < 16) {
            const int ntile = g.tx * g.ty;
            float a = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) a += sred[16 * w + t];
            gpart[((size_t)T.b0 * ntile + blockIdx.x % ntile) * 16 + t] = a;
        }
        return;
    }
    // several: of the image in LDS, a sample per wavefront; lanes of one parity hold one plane's 8 channels
    const int h = t & 1, px = T.tw * T.th;
    const Div dw(T.tw);
    for (int s = wave; s < g.S; s += WAVES) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = 0.f;
        for (int q = lane >> 1; q < px; q += 32) {
            const int yy = dw.q(q), xx = q - yy * T.tw;
            const uint4 u = sA[h * PL + s * g.img + (yy + 2) * P + xx + 2];
            const uint32_t d[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[2 * k] += __uint_as_float(d[k] << 16);
                v[2 * k + 1] += __uint_as_float(d[k] & 0xFFFF0000u);
            }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int o = 32; o >= 2; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
        if (lane < 2 && T.b0 + s < g.batch)
#pragma unroll
            for (int k = 0; k < 8; ++k) gpart[(size_t)(T.b0 + s) * 16 + 8 * h + k] = v[k];
    }
}

// ---------------------------------------------------------------------------------------
// Dense head: 64 lanes per sample, lane k the hidden unit k.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float head_hidden(const float* gs, const float* __restrict__ prm, int k)
{
    float s = prm[OFF_C1 + k];
#pragma unroll
    for (int c = 0; c < 16; ++c) s = fmaf(prm[OFF_U1 + k * 16 + c], gs[c], s);
    return s;
}

__device__ __forceinline__ float head_out(const float* hs, const float* __restrict__ prm)
{
    float v = prm[OFF_C2];
#pragma unroll 16
    for (int q = 0; q < 64; ++q) v = fmaf(prm[OFF_U2 + q], hs[q], v);
    return v;
}

__global__ void __launch_bounds__(256) head_fwd(const float* __restrict__ gpart, int ntile, float nn, const float* __restrict__ prm,
                                                int batch, float* __restrict__ gout, float* __restrict__ r)
{
    __shared__ float sg[4][16];
    __shared__ __align__(16) float sh[4][64];
    const int k = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int b = blockIdx.x * 4 + w;
    const bool on = b < batch;
    if (on && k < 16) {
        float s = 0.f;
        for (int q = 0; q < ntile; ++q) s += gpart[((size_t)b * ntile + q) * 16 + k];
        s /= nn;
        sg[w][k] = s;
        gout[(size_t)b * 16 + k] = s;
    }
    __syncthreads();
    if (on) sh[w][k] = fmaxf(head_hidden(sg[w], prm, k), 0.f);
    __syncthreads();
    if (on && k == 0) r[b] = head_out(sh[w], prm);
}

// The head of a training pass, a block per sample.  The gradient at the third layer is rounded to BF16, so the last
// bit of an output turns one of its roundings in 20000 and moves the gradient of a small batch by up to 1e-4: in
// training a channel's mean adds its pixels one after the other, whatever the tiles are, and the output its hidden
// units.  Bound by that chain: 19 us for 4096 pixels.  Three wavefronts load 384 pixels ahead and turn them over
// in LDS, the fourth adds (its own loads, or all four taking turns, left the chain waiting: 65 to 115 us).
__global__ void __launch_bounds__(256) head_train(const uint16_t* __restrict__ a3, int nn, const float* __restrict__ prm,
                                                  float* __restrict__ gout, float* __restrict__ r)
{
    constexpr int PX = 384, PITCH = PX + 4, LOADS = PX * 2 / 192;
    __shared__ __align__(16) float sp[2][16 * PITCH];            // [channel][pixel]
    __shared__ float sg[16];
    __shared__ __align__(16) float sh[64];
    const int k = threadIdx.x & 63, w = threadIdx.x >> 6, t = (int)threadIdx.x - 64;
    const uint4* src = (const uint4*)(a3 + (size_t)blockIdx.x * nn * 16);
    uint4 next[LOADS];
    auto load = [&](int p0) {
#pragma unroll
        for (int q = 0; q < LOADS; ++q) next[q] = src[min(2 * p0 + t + 192 * q, 2 * nn - 1)];
    };
    if (w > 0) load(0);
    float s = 0.f;
    for (int p0 = 0, par = 0; p0 < nn; p0 += PX, par ^= 1) {
        if (w > 0) {
#pragma unroll
            for (int q = 0; q < LOADS; ++q) {
                const int e = t + 192 * q, px = e >> 1, h = e & 1;
                const uint32_t d[4] = {next[q].x, next[q].y, next[q].z, next[q].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    sp[par][(8 * h + 2 * j) * PITCH + px] = __uint_as_float(d[j] << 16);
                    sp[par][(8 * h + 2 * j + 1) * PITCH + px] = __uint_as_float(d[j] & 0xFFFF0000u);
                }
            }
            load(p0 + PX);
        }
        __syncthreads();          // the other buffer's reader came here, too, after its last read
        if (w == 0 && k < 16) {
            const float4* v = (const float4*)(sp[par] + k * PITCH);
            const int m = min(PX, nn - p0) >> 2;                 // a multiple of 4
#pragma unroll 8
            for (int q = 0; q < m; ++q) {
                const float4 d = v[q];
                s += d.x;
                s += d.y;
                s += d.z;
                s += d.w;
            }
        }
    }
    if (w == 0 && k < 16) {
        s /= (float)nn;
        sg[k] = s;
        gout[(size_t)blockIdx.x * 16 + k] = s;
    }
    __syncthreads();
    if (w == 0) sh[k] = fmaxf(head_hidden(sg, prm, k), 0.f);
    __syncthreads();
    if (threadIdx.x == 0) r[blockIdx.x] = head_out(sh, prm);
}

// Per sample: squared error, dL/dr, the hidden layer's gradient dh and dr relu(h) (for U1, c1, U2), and
// the gradient at the third convolution's output, dg / nn in BF16.
__global__ void __launch_bounds__(256) head_bwd(const float* __restrict__ g, const float* __restrict__ r,
                                                const float* __restrict__ y, const float* __restrict__ prm, int batch, float nn,
                                                float* __restrict__ sq, float* __restrict__ drs, float* __restrict__ dh,
                                                float* __restrict__ da, uint16_t* __restrict__ dgs)
{
    __shared__ float sg[4][16], sd[4][64];
    const int k = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int b = blockIdx.x * 4 + w;
    const bool on = b < batch;
    if (on && k < 16) sg[w][k] = g[(size_t)b * 16 + k];
    __syncthreads();
    if (on) {
        const float e = r[b] - y[b];
        const float dr = 2.0f * e / (float)batch;
        const float hk = head_hidden(sg[w], prm, k);
        const float d = hk > 0.f ? dr * prm[OFF_U2 + k] : 0.f;
        sd[w][k] = d;
        dh[(size_t)b * 64 + k] = d;
        da[(size_t)b * 64 + k] = dr * fmaxf(hk, 0.f);
        if (k == 0) { sq[b] = e * e; drs[b] = dr; }
    }
    __syncthreads();
    if (on && k < 16) {
        float s = 0.f;
#pragma unroll 8
        for (int q = 0; q < 64; ++q) s = fmaf(prm[OFF_U1 + q * 16 + k], sd[w][q], s);
        dgs[(size_t)b * 16 + k] = f2bf(s / nn);
    }
}

// ---------------------------------------------------------------------------------------
// Backward of one 16->16 convolution.
//   LAYER 3: the gradient at its output is dgs[b][c] where the ReLU mask m3 is set; writes the
//            gradient at its input (masked by act > 0) to dzo.
//   LAYER 2: the gradient at its output is dzi; the gradient at its input stays in LDS and gives the
//            first layer's weight gradient with x.
// part [block][10][256]: the weight gradient per neighbour [o][c] and, last, the bias gradient in
// column 0; part1 [block][256]: the first layer's [o][position 0..8 | 9: bias].
// ---------------------------------------------------------------------------------------
template <int LAYER>
__global__ void __launch_bounds__(256, 2) conv_bwd(const Geo g, const uint16_t* __restrict__ wb, const uint16_t* __restrict__ act,
                                                const uint16_t* __restrict__ m3, const uint16_t* __restrict__ dgs,
                                                const uint16_t* __restrict__ dzi, uint16_t* __restrict__ dzo,
                                                const float* __restrict__ x, float* __restrict__ part,
                                                float* __restrict__ part1)
{
    constexpr int PL = kBwdL + 24;
    __shared__ uint4 sZ[2 * PL];                         // gradient image (halo 1), two planes
    __shared__ __align__(16) uint16_t aT[16 * kBwdA];    // activation image, [channel][row][8 + pixel]
    __shared__ __align__(16) uint16_t zT[16 * kBwdZ];    // gradient tile, [channel][8-pixel units]
    __shared__ float sx[LAYER == 2 ? kBwdL + 64 : 1];    // x image (halo 1)
    __shared__ uint16_t utab[kBwdZ / 8];                 // a unit's place in a row of aT
    __shared__ uint16_t sdg[LAYER == 3 ? 64 * 16 : 1];
    static_assert(16 * kBwdA * 2 >= 2560 * 4, "the block's sums reuse the activation image");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, i = lane & 15, kg = lane >> 4;
    const int n = g.n, P = g.P, L = g.L, S = g.S;
    const size_t nn = (size_t)n * n;
    const int upr = (g.tw + 7) >> 3, rp = 8 * upr + 16, rows = S * (g.th + 2), U = S * g.th * upr;
    // channel strides of an odd number of 16-byte pieces: the 16 channels of an operand read without bank conflicts
    const int ca = 8 * ((rows * rp / 8) | 1), cz = 8 * (U | 1);
    const Div dU(upr), dRow(g.th), dRp(rp), dRows(g.th + 2), dUs(g.th * upr);
    uint4 w[5];
    load_weights(w, wb, lane);
    int off[5];
    neighbour_offsets(off, P, lane, -1);
    for (int u = t; u < U; u += 256) {
        const int row = dU.q(u), s = dRow.q(row);
        utab[u] = (uint16_t)((row + 2 * s + 1) * rp + 8 + 8 * (u - row * upr));
    }
    if constexpr (LAYER == 2)
        for (int e = L + t; e < kBwdL + 64; e += 256) sx[e] = 0.f;
    floatx4 acc[10], acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int pos = 0; pos < 10; ++pos) acc[pos] = floatx4{0.f, 0.f, 0.f, 0.f};
    const uint4 ones = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);

    for (int item = blockIdx.x; item < g.groups; item += gridDim.x) {
        const TileAt T = tile_at(g, item);
        __syncthreads();                                 // the previous tile's readers are done
        if constexpr (LAYER == 3) {
            for (int e = t; e < S * 16; e += 256) sdg[e] = T.b0 + (e >> 4) < g.batch ? dgs[(size_t)T.b0 * 16 + e] : (uint16_t)0;
            __syncthreads();
        }
        // the gradient's 8 channels h of pixel (s, y, x)
        auto grad8 = [&](int s, int gy, int gx, int h) -> uint4 {
            const size_t p = (size_t)(T.b0 + s) * nn + (size_t)gy * n + gx;
            if (T.b0 + s >= g.batch) return make_uint4(0, 0, 0, 0);
            if constexpr (LAYER == 3) {
                const uint32_t m = (uint32_t)m3[p] >> (8 * h);
                uint32_t d[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t v = *(const uint32_t*)(sdg + s * 16 + 8 * h + 2 * k);
                    d[k] = ((m >> (2 * k)) & 1u ? v & 0xFFFFu : 0u) | ((m >> (2 * k + 1)) & 1u ? v & 0xFFFF0000u : 0u);
                }
                return make_uint4(d[0], d[1], d[2], d[3]);
            } else {
                return *(const uint4*)(dzi + p * 16 + 8 * h);
            }
        };
        auto scatter8 = [](uint16_t* dst, int stride, uint4 v) {
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                dst[(2 * k) * stride] = (uint16_t)d[k];
                dst[(2 * k + 1) * stride] = (uint16_t)(d[k] >> 16);
            }
        };
        for (int e = t; e < 2 * L; e += 256) {
            const int h = e >= L ? 1 : 0, q = e - h * L, s = g.dImg.q(q), r = q - s * g.img, yy = g.dP.q(r), xx = r - yy * P;
            sZ[h * PL + q] = grad8(s, wrapn(T.y0 + yy - 1, n), wrapn(T.x0 + xx - 1, n), h);
        }
        for (int e = t; e < 16 * U; e += 256) {          // (half, unit, pixel)
            const int h = e >= 8 * U ? 1 : 0, q = e - h * 8 * U, u = q >> 3, row = dU.q(u), s = dRow.q(row);
            const int yy = row - s * g.th, xx = 8 * (u - row * upr) + (q & 7);
            const bool in = yy < T.th && xx < T.tw;
            scatter8(zT + 8 * h * cz + q, cz, in ? grad8(s, T.y0 + yy, T.x0 + xx, h) : make_uint4(0, 0, 0, 0));
        }
        for (int e = t; e < 2 * rows * rp; e += 256) {   // (half, row, place)
            const int h = e >= rows * rp ? 1 : 0, q = e - h * rows * rp, row = dRp.q(q), s = dRows.q(row);
            const int yy = row - s * (g.th + 2) - 1, xx = q - row * rp - 8;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (xx >= -1 && xx <= g.tw && T.b0 + s < g.batch)
                v = *(const uint4*)(act + ((T.b0 + s) * nn + (size_t)wrapn(T.y0 + yy, n) * n + wrapn(T.x0 + xx, n)) * 16 + 8 * h);
            scatter8(aT + 8 * h * ca + q, ca, v);
        }
        if constexpr (LAYER == 2) {
            for (int e = t; e < L; e += 256) {
                const int s = g.dImg.q(e), r = e - s * g.img, yy = g.dP.q(r), xx = r - yy * P;
                const int b = min(T.b0 + s, g.batch - 1);
                sx[e] = x[b * nn + (size_t)wrapn(T.y0 + yy - 1, n) * n + wrapn(T.x0 + xx - 1, n)];
            }
        }
        __syncthreads();
        // weight and bias gradients: 4 units of 8 pixels per MFMA
        for (int u0 = 4 * wave; u0 < U; u0 += 16) {
            const int u = u0 + kg;
            uint4 za = make_uint4(0, 0, 0, 0);
            int place = 8;
            if (u < U) {
                za = *(const uint4*)(zT + i * cz + 8 * u);
                place = utab[u];
            }
            const bf16x8 A = __builtin_bit_cast(bf16x8, za);
            const uint16_t* base = aT + i * ca + place;
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                const int ro = u < U ? dy * rp : 0;
                const uint4 c = *(const uint4*)(base + ro);
                const uint32_t lf = *(const uint32_t*)(base + ro - 2), rt = *(const uint32_t*)(base + ro + 8);
                const uint32_t f0 = __builtin_amdgcn_alignbit(c.x, lf, 16), f1 = __builtin_amdgcn_alignbit(c.y, c.x, 16),
                               f2 = __builtin_amdgcn_alignbit(c.z, c.y, 16), f3 = __builtin_amdgcn_alignbit(c.w, c.z, 16),
                               f4 = __builtin_amdgcn_alignbit(rt, c.w, 16);
                const int p0 = 3 * (dy + 1);
                acc[p0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, make_uint4(f0, f1, f2, f3)), acc[p0], 0, 0, 0);
                acc[p0 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, c), acc[p0 + 1], 0, 0, 0);
                acc[p0 + 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, make_uint4(f1, f2, f3, f4)), acc[p0 + 2], 0, 0, 0);
            }
            acc[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8, ones), acc[9], 0, 0, 0);
        }
        if constexpr (LAYER == 2) __syncthreads();       // zT is overwritten below
        // the gradient at the layer's input
        for (int g0 = P + 1 + 16 * wave; g0 < L - P - 1; g0 += 64) {
            const floatx4 d = conv16(sZ, PL, g0, off, w, lane);
            const int q = g0 + i, s = g.dImg.q(q), r = q - s * g.img, yy = g.dP.q(r) - 1, xx = r - (yy + 1) * P - 1;
            const bool in = s < S && T.b0 + s < g.batch && yy >= 0 && yy < T.th && xx >= 0 && xx < T.tw;
            if (!in) continue;
            const size_t p = (size_t)(T.b0 + s) * nn + (size_t)(T.y0 + yy) * n + T.x0 + xx;
            const uint16_t* am = aT + (4 * kg) * ca + (s * (g.th + 2) + yy + 1) * rp + 8 + xx;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (am[k * ca] & 0x7FFFu) != 0 ? d[k] : 0.0f;
            if constexpr (LAYER == 3) {
                *(uint2*)(dzo + p * 16 + 4 * kg) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
            } else {
                uint16_t* z = zT + 4 * kg * cz + ((s * g.th + yy) * upr) * 8 + xx;
#pragma unroll
                for (int k = 0; k < 4; ++k) z[k * cz] = f2bf(v[k]);
            }
        }
        if constexpr (LAYER == 2) {
            __syncthreads();
            // first layer: dW1[o][pos] = sum_p dz1[p][o] x[p + d(pos)], FP32 products; 4 pixels per MFMA
            const int dpos = i < 9 ? (i / 3 - 1) * P + (i % 3 - 1) : 0;
            for (int u = wave; u < U; u += 4) {
                const int row = dU.q(u), s = dRow.q(row);
                const int xi = s * g.img + (row - s * g.th + 1) * P + 1 + 8 * (u - row * upr) + kg;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float za = bf2f(zT[i * cz + 8 * u + 4 * j + kg]);
                    const float xv = i < 9 ? sx[xi + 4 * j + dpos] : (i == 9 ? 1.0f : 0.0f);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(za, xv, acc1, 0, 0, 0);
                }
            }
        }
    }
    // the block's sums, wavefront by wavefront
    __syncthreads();
    float* red = (float*)aT;
    float* red1 = (float*)zT;
    for (int v = 0; v < 4; ++v) {
        if (wave == v) {
#pragma unroll
            for (int pos = 0; pos < 10; ++pos)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float* d = red + pos * 256 + (4 * kg + r) * 16 + i;
                    *d = v == 0 ? acc[pos][r] : *d + acc[pos][r];
                }
            if constexpr (LAYER == 2)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float* d = red1 + (4 * kg + r) * 16 + i;
                    *d = v == 0 ? acc1[r] : *d + acc1[r];
                }
        }
        __syncthreads();
    }
    for (int e = t; e < 2560; e += 256) part[(size_t)blockIdx.x * 2560 + e] = red[e];
    if constexpr (LAYER == 2) part1[(size_t)blockIdx.x * 256 + t] = red1[t];
}

// Sums of the blocks' partials, 16 slices of blocks per output in a fixed order, into the flat
// gradient; and the dense head's gradients, a block per hidden unit over the batch.
constexpr int kSumBlocks = (2 * 2560 + 256) / 64;

__global__ void __launch_bounds__(1024) finish_grad(const float* __restrict__ p3, const float* __restrict__ p2,
                                                    const float* __restrict__ p1, int nb, const float* __restrict__ g,
                                                    const float* __restrict__ dh, const float* __restrict__ da,
                                                    const float* __restrict__ drs, int batch, float* __restrict__ grad)
{
    __shared__ float sh[64 * 18];
    const int t = threadIdx.x;
    if ((int)blockIdx.x < kSumBlocks) {
        const int lane = t & 63, sl = t >> 6, e = blockIdx.x * 64 + lane;
        const float* src = e < 2560 ? p3 + e : (e < 5120 ? p2 + (e - 2560) : p1 + (e - 5120));
        const size_t stride = e < 5120 ? 2560 : 256;
        const int b0 = nb * sl / 16, b1 = nb * (sl + 1) / 16;
        float s = 0.f;
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += src[b * stride];
        sh[sl * 64 + lane] = s;
        __syncthreads();
        if (sl != 0) return;
        s = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) s += sh[k * 64 + lane];
        if (e < 5120) {
            const int q = e < 2560 ? e : e - 2560, pos = q >> 8, o = (q >> 4) & 15, c = q & 15;
            if (pos < 9) grad[(e < 2560 ? OFF_W3 : OFF_W2) + o * 144 + c * 9 + pos] = s;
            else if (c == 0) grad[(e < 2560 ? OFF_B3 : OFF_B2) + o] = s;
        } else {
            const int q = e - 5120, o = q >> 4, pos = q & 15;
            if (pos < 9) grad[OFF_W1 + o * 9 + pos] = s;
            else if (pos == 9) grad[OFF_B1 + o] = s;
        }
        return;
    }
    const int k = (int)blockIdx.x - kSumBlocks;          // hidden unit; 64: the output bias
    const int c = t & 15, sl = t >> 4;
    float s = 0.f, sa = 0.f, sb = 0.f;
    if (k < 64) {
        for (int b = sl; b < batch; b += 64) {
            const float d = dh[(size_t)b * 64 + k];
            s += d * g[(size_t)b * 16 + c];
            if (c == 0) { sa += da[(size_t)b * 64 + k]; sb += d; }
        }
    } else if (c == 0) {
        for (int b = sl; b < batch; b += 64) sa += drs[b];
    }
    sh[sl * 18 + c] = s;
    if (c == 0) { sh[sl * 18 + 16] = sa; sh[sl * 18 + 17] = sb; }
    __syncthreads();
    if (t >= 18) return;
    s = 0.f;
    for (int q = 0; q < 64; ++q) s += sh[q * 18 + t];
    if (k == 64) { if (t == 16) grad[OFF_C2] = s; return; }
    if (t < 16) grad[OFF_U1 + k * 16 + t] = s;
    else if (t == 16) grad[OFF_U2 + k] = s;
    else grad[OFF_C1 + k] = s;
}

// Adam (Kingma & Ba) with bias correction; t is the 1-based step.
__global__ void adam(float* __restrict__ p, const float* __restrict__ gr, float* __restrict__ m, float* __restrict__ v,
                     int n, float lr, float b1, float b2, float eps, int t)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float gk = gr[k];
    const float mk = b1 * m[k] + (1.f - b1) * gk;
    const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const float mh = mk / (1.f - powf(b1, (float)t));
    const float vh = vk / (1.f - powf(b2, (float)t));
    p[k] -= lr * mh / (sqrtf(vh) + eps);
}

// BF16 GEMM layouts of the two 16->16 convs: fwd[o][pos*16+c], bwd[c][pos*16+o] (rows of 160)
__global__ void pack_weights(const float* __restrict__ prm, uint16_t* __restrict__ fwd2, uint16_t* __restrict__ bwd2,
                             uint16_t* __restrict__ fwd3, uint16_t* __restrict__ bwd3)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;   // 2 * 16 * 160
    if (t >= 2 * 16 * 160) return;
    const bool third = t >= 16 * 160;
    if (third) t -= 16 * 160;
    const int off = third ? OFF_W3 : OFF_W2;
    uint16_t* fwd = third ? fwd3 : fwd2;
    uint16_t* bwd = third ? bwd3 : bwd2;
    const int row = t / 160, k = t % 160;
    if (k >= 144) { fwd[t] = 0; bwd[t] = 0; return; }
    const int pos = k / 16, col = k % 16;
    fwd[t] = f2bf(prm[off + row * 144 + col * 9 + pos]);   // W[o=row][c=col][pos]
    bwd[t] = f2bf(prm[off + col * 144 + row * 9 + pos]);   // W[o=col][c=row][pos]
}

// x = scale (rho - rho_bar) (FP32 or FP64 fields; rho_bar FP64 [nn])
__global__ void normalize_fields(const void* __restrict__ rho, int is_double, const double* __restrict__ rbar, int nn,
                                 size_t total, double scale, float* __restrict__ x)
{
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const double v = is_double ? ((const double*)rho)[t] : (double)((const float*)rho)[t];
    x[t] = (float)(scale * (v - rbar[t % nn]));
}

// Y = P_f - P_c of observable j as float targets
__global__ void extract_y_kernel(const double* __restrict__ ps, int nobs, int j, int count, float* __restrict__ y)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    y[i] = (float)(ps[((size_t)i * nobs + j) * 2] - ps[((size_t)i * nobs + j) * 2 + 1]);
}

// Z_i = (Y_i - r_i) + (1/k) sum_{j<k} r'_{k i + j}, written as (Z, 0) pairs for the moment kernel
__global__ void combine_cv_kernel(const double* __restrict__ ps, int nobs, int jobs, const float* __restrict__ r,
                                  const float* __restrict__ rco, int k, int count, double* __restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const double y = ps[((size_t)i * nobs + jobs) * 2] - ps[((size_t)i * nobs + jobs) * 2 + 1];
    double m = 0.0;
    for (int t = 0; t < k; ++t) m += (double)rco[(size_t)i * k + t];
    out[2 * (size_t)i] = (y - (double)r[i]) + m / (double)k;
    out[2 * (size_t)i + 1] = 0.0;
}

hipError_t extract_y(const double* ps, int nobs, int j, int count, float* y, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(extract_y_kernel, dim3((count + 255) / 256), dim3(256), 0, s, ps, nobs, j, count, y);
    return hipGetLastError();
}

hipError_t combine_cv(const double* ps, int nobs, int j, const float* r, const float* rco, int k, int count, double* out,
                      hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(combine_cv_kernel, dim3((count + 255) / 256), dim3(256), 0, s, ps, nobs, j, r, rco, k, count, out);
    return hipGetLastError();
}

// acc[0] += sum of v, in double: 256 strided partial sums, then a fixed tree
__global__ void __launch_bounds__(256) sum_into(const float* __restrict__ v, int n, double* __restrict__ acc)
{
    __shared__ double sh[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += (double)v[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) acc[0] += sh[0];
}

hipError_t accumulate_sq(const Workspace& W, int batch, double* acc, hipStream_t s)
{
    hipLaunchKernelGGL(sum_into, dim3(1), dim3(256), 0, s, W.sq, batch, acc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Host-side launch sequences
// ---------------------------------------------------------------------------------------
static inline unsigned blocks_for(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

int forward_batch(int n)
{
    const Geo g = make_geo(n, 1, 2);
    return std::max(1, kForwardTiles / (g.tx * g.ty));
}

// The pool's sums grow with the forward batch, the rest with the training batch, so a program that
// alternates evaluation and training on one grid size allocates once for each.
hipError_t Workspace::reserve(int n_, int batch_)
{
    if (n_ != n) release();
    n = n_;
    hipError_t e;
    auto take = [&](auto*& ptr, size_t bytes) {
        if (ptr) (void)hipFree(ptr);
        ptr = nullptr;
        return hipMalloc((void**)&ptr, bytes);
    };
#define TAKE(ptr, bytes) if ((e = take(ptr, bytes)) != hipSuccess) { release(); return e; }
    if (!wt2) {
        TAKE(wt2, 16 * 160 * 2);
        TAKE(wb2, 16 * 160 * 2);
        TAKE(wt3, 16 * 160 * 2);
        TAKE(wb3, 16 * 160 * 2);
    }
    if (batch_ > batch) {
        const Geo g = make_geo(n_, batch_, 2);
        TAKE(gpart, (size_t)batch_ * g.tx * g.ty * 16 * 4);
        TAKE(g_, (size_t)batch_ * 16 * 4);
        batch = batch_;
    }
    if (keep && batch_ > kept) {
        const size_t npix = (size_t)batch_ * n_ * n_;
        TAKE(a1, npix * 16 * 2);
        TAKE(a2, npix * 16 * 2);
        TAKE(a3, npix * 16 * 2);
        TAKE(dz2, npix * 16 * 2);
        TAKE(m3, npix * 2);
        TAKE(sq, (size_t)batch_ * 4);
        TAKE(drs, (size_t)batch_ * 4);
        TAKE(dh, (size_t)batch_ * 64 * 4);
        TAKE(da, (size_t)batch_ * 64 * 4);
        TAKE(dgs, (size_t)batch_ * 16 * 2);
        TAKE(part, (size_t)kBlocks * (2 * 2560 + 256) * 4);
        kept = batch_;
    }
#undef TAKE
    return hipSuccess;
}

void Workspace::release()
{
    void* ptrs[] = {gpart, g_, wt2, wb2, wt3, wb3, a1, a2, a3, dz2, m3, sq, drs, dh, da, dgs, part};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    gpart = g_ = sq = drs = dh = da = part = nullptr;
    wt2 = wb2 = wt3 = wb3 = a1 = a2 = a3 = dz2 = m3 = dgs = nullptr;
    n = batch = kept = 0;
}

hipError_t pack(Workspace& W, const float* prm, hipStream_t s)
{
    hipLaunchKernelGGL(pack_weights, dim3(blocks_for(2 * 16 * 160, 256)), dim3(256), 0, s, prm, W.wt2, W.wb2, W.wt3, W.wb3);
    return hipGetLastError();
}

hipError_t forward(Workspace& W, const float* prm, const float* x, int batch, float* r, hipStream_t s)
{
    if (batch < 1) return hipSuccess;
    const Geo g = make_geo(W.n, batch, 2);
    const dim3 grid((unsigned)g.groups);
    uint16_t* none = nullptr;
    if (W.keep) {
        hipLaunchKernelGGL(conv_fwd<true>, grid, dim3(kFwdThreads), 0, s, g, x, prm, W.wt2, W.wt3, W.gpart, W.a1, W.a2, W.a3, W.m3);
        hipLaunchKernelGGL(head_train, dim3(batch), dim3(256), 0, s, W.a3, W.n * W.n, prm, W.g_, r);
    } else {
        hipLaunchKernelGGL(conv_fwd<false>, grid, dim3(kFwdThreads), 0, s, g, x, prm, W.wt2, W.wt3, W.gpart, none, none, none, none);
        hipLaunchKernelGGL(head_fwd, dim3(blocks_for(batch, 4)), dim3(256), 0, s, W.gpart, g.tx * g.ty, (float)(W.n * W.n), prm, batch,
                           W.g_, r);
    }
    return hipGetLastError();
}

hipError_t backward(Workspace& W, const float* prm, const float* x, const float* r, const float* y, int batch, float* grad,
                    hipStream_t s)
{
    if (W.kept < batch) return hipErrorInvalidValue;
    const Geo g = make_geo(W.n, batch, 1);
    const int nb = std::min(g.groups, kBlocks);
    float* p3 = W.part;
    float* p2 = p3 + (size_t)kBlocks * 2560;
    float* p1 = p2 + (size_t)kBlocks * 2560;
    hipLaunchKernelGGL(head_bwd, dim3(blocks_for(batch, 4)), dim3(256), 0, s, W.g_, r, y, prm, batch, (float)(W.n * W.n), W.sq,
                       W.drs, W.dh, W.da, W.dgs);
    hipLaunchKernelGGL(conv_bwd<3>, dim3(nb), dim3(256), 0, s, g, W.wb3, W.a2, W.m3, W.dgs, (const uint16_t*)nullptr, W.dz2,
                       (const float*)nullptr, p3, (float*)nullptr);
    hipLaunchKernelGGL(conv_bwd<2>, dim3(nb), dim3(256), 0, s, g, W.wb2, W.a1, (const uint16_t*)nullptr,
                       (const uint16_t*)nullptr, W.dz2, (uint16_t*)nullptr, x, p2, p1);
    hipLaunchKernelGGL(finish_grad, dim3(kSumBlocks + 65), dim3(1024), 0, s, p3, p2, p1, nb, W.g_, W.dh, W.da, W.drs, batch, grad);
    return hipGetLastError();
}

hipError_t adam_update(float* prm, const float* grad, float* m, float* v, float lr, int t, hipStream_t s)
{
    hipLaunchKernelGGL(adam, dim3(blocks_for(NPARAM, 256)), dim3(256), 0, s, prm, grad, m, v, NPARAM, lr, 0.9f, 0.999f,
                       1e-8f, t);
    return hipGetLastError();
}

hipError_t normalize(const void* rho, bool is_double, const double* rbar, int nn, size_t total, double scale, float* x,
                     hipStream_t s)
{
    hipLaunchKernelGGL(normalize_fields, dim3(blocks_for(total, 256)), dim3(256), 0, s, rho, (int)is_double, rbar, nn, total,
                       scale, x);
    return hipGetLastError();
}

}  // namespace cnn
}  // namespace dk
