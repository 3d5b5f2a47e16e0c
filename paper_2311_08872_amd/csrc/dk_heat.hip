// dk_heat.hip -- the noise-free FP32 scheme rho <- rho + (mu/2) Lap_h rho on a batch of fields
// (dk_heat_steps): many steps per pass over memory, the fields in registers.
//
// A pass per step moves 8 B a cell and step and is bound by HBM (6.16 ms for 64 steps of 1000 fields of
// 256 x 256, 5.45 TB/s); the five operations of a cell and step take a fifteenth of that.  A lane holds
// 16 rows x 4 columns, so one block of 1024 lanes holds 256 x 256 cells, half of a compute unit's
// registers, and takes any number of steps between one read and one write of the field:
//   n <= 256       a block per field (several fields per wavefront where a field's row groups fit into
//                  one), in place, all steps in one launch up to the work of one launch
//   n > 256        256 x 256 windows with a halo of T <= 16 cells, T steps a pass, two buffers in turn
// Rows of a lane are swept in registers; the columns at a lane's edges come from the neighbouring lanes
// (ds_bpermute), the rows at its top and bottom through LDS, double-buffered by step, one barrier a step,
// none where a field lies in one wavefront.  The same 64 steps of 1000 fields now take 0.58 ms (7.2e12 cell
// steps/s; 8.3e12 at 128 x 128, where four blocks share a compute unit): bound by the 330 vector and 36 LDS
// instructions of a wavefront's step and, at one block per compute unit, by its barrier.  Windows: 512 x 512
// 2.2e12 (7.6e11 with a pass per step), 1024 x 1024 3.5e12 (6.3e11).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "dk_host.h"

namespace dk {
namespace {

constexpr int R = 16;             // rows per lane (4 columns each)
constexpr int kWin = 256;         // window and largest resident field
constexpr int kMaxT = 16;         // steps of a pass over windows

struct HeatGeo {
    int n, batch, T;
    int q;                        // lanes per row
    int G;                        // row groups of a field (or window)
    int gpw;                      // row groups per wavefront
    int F;                        // fields per wavefront; 0: one field (window) per block
    int H, tx, ty, vx, vy;        // windows: halo, count and interior size
};

// A neighbouring lane's value, whatever the row's length.  Whole-wavefront DPP rotations, which a 256-cell
// row could use, run 14 % slower; 16-lane ones, for 64-cell rows only, 9 % faster.
__device__ __forceinline__ float lane_value(float v, int addr)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}

// by component, so that the row array stays in registers
__device__ __forceinline__ float4 pick(bool first, const float4 a, const float4 b)
{
    return make_float4(first ? a.x : b.x, first ? a.y : b.y, first ? a.z : b.z, first ? a.w : b.w);
}

// EXACT: n is a multiple of R; else the last row group holds n % R rows.  BLOCK: a field spans the block's
// wavefronts.  WINDOW: the block's 256 x 256 cells are a window of a larger field.
template <bool EXACT, bool BLOCK, bool WINDOW>
__global__ void __launch_bounds__(BLOCK ? 1024 : 256) heat_kernel(const HeatGeo A, const float* in, float* out,
                                                                  float a /* in and out: the same fields, or two */)
{
#pragma clang fp contract(off)
    extern __shared__ float4 halo[];            // per field [parity][row group][top, bottom][lane]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = A.q, G = A.G, n = A.n;
    const int grp = lane / q, cl = lane - grp * q;
    int g = 0, x0 = 4 * cl, y0 = 0, H = 0;
    size_t field;
    bool on = grp < A.gpw;
    float4* mine = halo;
    if constexpr (BLOCK) {
        g = wave * A.gpw + grp;
        on = on && g < G;
        if constexpr (WINDOW) {
            const int per = A.tx * A.ty;
            field = blockIdx.x / per;
            const int t = blockIdx.x - (unsigned)field * per;
            H = A.H;
            x0 += (t % A.tx) * A.vx - H;
            y0 = (t / A.tx) * A.vy - H;
        } else {
            field = blockIdx.x;
        }
    } else {
        const int f = grp / G;
        g = grp - f * G;
        on = on && f < A.F;
        const int slot = wave * A.F + (f < A.F ? f : 0);
        field = (size_t)blockIdx.x * (blockDim.x >> 6) * A.F + slot;
        on = on && field < (size_t)A.batch;
        mine = halo + (size_t)slot * 4 * G * q;
    }
    if (!on) { g = 0; field = BLOCK ? field : 0; }
    const int rows = EXACT ? R : min(R, n - g * R);
    const int src_l = (lane - cl + (cl == 0 ? q - 1 : cl - 1)) * 4, src_r = (lane - cl + (cl == q - 1 ? 0 : cl + 1)) * 4;
    // a window's rows beyond its interior and halo feed nothing that is kept: its wavefronts only meet the barriers
    const bool work = !WINDOW || g * R < A.vy + 2 * H;
    auto wrap = [n](int v) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    // R + 1 row slots: before an even step row i is in slot i + 1, and the sweep goes down and leaves it in
    // slot i (the slot of the row above, whose old value is used up); an odd step sweeps up and puts it back.
    // In-place rows would need a copy of every cell (60 of 380 instructions a step).
    float4 v[R + 1];
    {
        const float* f = in + field * (size_t)n * n;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            v[i + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!work || (!EXACT && i >= rows)) continue;
            const int y = WINDOW ? wrap(y0 + g * R + i) : g * R + i, x = WINDOW ? wrap(x0) : x0;
            if (on) v[i + 1] = *(const float4*)(f + (size_t)y * n + x);
        }
    }
    const int gu = g == 0 ? G - 1 : g - 1, gd = g == G - 1 ? 0 : g + 1;
    // one cell row: c between u above and d below
    auto update = [&](const float4 u, const float4 c, const float4 d) {
        const float l = lane_value(c.w, src_l), r = lane_value(c.x, src_r);
        float4 o;
        o.x = fmaf(a, fmaf(-4.0f, c.x, (l + c.y) + (u.x + d.x)), c.x);
        o.y = fmaf(a, fmaf(-4.0f, c.y, (c.x + c.z) + (u.y + d.y)), c.y);
        o.z = fmaf(a, fmaf(-4.0f, c.z, (c.y + c.w) + (u.z + d.z)), c.z);
        o.w = fmaf(a, fmaf(-4.0f, c.w, (c.z + r) + (u.w + d.w)), c.w);
        // row by row: with the rows interleaved the old and new cells of many rows would be live at once
        asm volatile("" : "+v"(o.x), "+v"(o.y), "+v"(o.z), "+v"(o.w));
        return o;
    };
    // rows of parity S in slots 1 - S + i
    auto step = [&](auto par) {
        constexpr int S = decltype(par)::value, O = 1 - S;
        float4* buf = mine + S * 2 * G * q;
        float4 last = v[R - 1 + O];
        if constexpr (!EXACT) {
#pragma unroll
            for (int i = 0; i < R - 1; ++i)
                last = pick(i == rows - 1, v[i + O], last);
        }
        if (on) {
            buf[(2 * g) * q + cl] = v[O];
            buf[(2 * g + 1) * q + cl] = last;
        }
        if constexpr (BLOCK) __syncthreads();
        else asm volatile("" ::: "memory");      // one wavefront: its LDS accesses are served in order
        if (!work) return;
        const float4 above = buf[(2 * gu + 1) * q + cl], below = buf[(2 * gd) * q + cl];
        auto next = [&](int i) {
            float4 d = i + 1 < R ? v[i + 1 < R ? i + 1 + O : O] : below;
            if constexpr (!EXACT) {
                d = pick(i == rows - 1, below, d);
            }
            return d;
        };
        if constexpr (S == 0) {
            v[0] = above;
#pragma unroll
            for (int i = 0; i < R; ++i) v[i] = update(v[i], v[i + 1], next(i));
        } else {
#pragma unroll
            for (int i = R - 1; i >= 0; --i) v[i + 1] = update(i > 0 ? v[i > 0 ? i - 1 : 0] : above, v[i], next(i));
        }
    };
    int m = 0;
#pragma unroll 1
    for (; m + 2 <= A.T; m += 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    if (m < A.T) {
        step(std::integral_constant<int, 0>{});
#pragma unroll
        for (int i = R; i >= 1; --i) v[i] = v[i - 1];
    }
    if (!on || !work) return;
    float* f = out + field * (size_t)n * n;
    if constexpr (WINDOW) {
        const int x = x0, xe = min((x0 - 4 * cl + H) + A.vx, n), ye = min(y0 + H + A.vy, n);
        if (4 * cl < H || x >= xe) return;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int y = y0 + g * R + i;
            if (g * R + i >= H && y < ye) *(float4*)(f + (size_t)y * n + x) = v[i + 1];
        }
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (EXACT || i < rows) *(float4*)(f + (size_t)(g * R + i) * n + x0) = v[i + 1];
    }
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

// `steps` steps of fields that fit one block, in place
hipError_t heat_resident(float* rho, int n, int batch, int steps, float a, hipStream_t s)
{
    HeatGeo A{};
    A.n = n;
    A.batch = batch;
    A.T = steps;
    A.q = n / 4;
    A.G = cdiv(n, R);
    A.gpw = 64 / A.q;
    const bool exact = n % R == 0;
    if (A.G > A.gpw) {
        const int waves = cdiv(A.G, A.gpw);
        const size_t lds = sizeof(float4) * 4 * A.G * A.q;
        const dim3 grid(batch), block(64 * waves);
        if (exact) hipLaunchKernelGGL((heat_kernel<true, true, false>), grid, block, lds, s, A, rho, rho, a);
        else hipLaunchKernelGGL((heat_kernel<false, true, false>), grid, block, lds, s, A, rho, rho, a);
        return hipGetLastError();
    }
    A.F = A.gpw / A.G;
    // four wavefronts a block, fewer where that leaves compute units idle
    const int waves = std::max(1, std::min(4, cdiv(cdiv(batch, A.F), 256)));
    const size_t lds = sizeof(float4) * 4 * A.G * A.q * A.F * waves;
    const dim3 grid(cdiv(batch, A.F * waves)), block(64 * waves);
    if (exact) hipLaunchKernelGGL((heat_kernel<true, false, false>), grid, block, lds, s, A, rho, rho, a);
    else hipLaunchKernelGGL((heat_kernel<false, false, false>), grid, block, lds, s, A, rho, rho, a);
    return hipGetLastError();
}

// one pass of T <= kMaxT steps over windows
hipError_t heat_windows(const float* in, float* out, int n, int batch, int T, float a, hipStream_t s)
{
    HeatGeo A{};
    A.n = n;
    A.batch = batch;
    A.T = T;
    A.q = 64;
    A.G = kWin / R;
    A.gpw = 1;
    A.H = 4 * cdiv(T, 4);
    const int v = kWin - 2 * A.H;
    A.tx = A.ty = cdiv(n, v);
    A.vx = 4 * cdiv(n / 4, A.tx);
    A.vy = cdiv(n, A.ty);
    const uint64_t blocks = (uint64_t)A.tx * A.ty * batch;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL((heat_kernel<true, true, true>), dim3((unsigned)blocks), dim3(64 * A.G),
                       sizeof(float4) * 4 * A.G * A.q, s, A, in, out, a);
    return hipGetLastError();
}

}  // namespace
}  // namespace dk

using namespace dkh;

extern "C" int dk_heat_steps(dk_context* ctx, int32_t n, int32_t batch, int32_t steps, double mu, float* rho, float* work,
                             double* kernel_ms, void* stream)
{
    if (!ctx || !rho || !work) return fail(DK_EINVAL, "NULL argument");
    if (n < 4 || n % 4 || batch < 1 || steps < 0) return fail(DK_EINVAL, "n must be a multiple of 4, batch >= 1");
    if (!(mu > 0) || mu > 0.5) return fail(DK_EINVAL, "mu outside (0, 1/2]");
    HIP_TRY(hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const float a = (float)(0.5 * mu);
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    HIP_TRY(hipEventRecord(e0, s));
    float* from = rho;
    if (n <= dk::kWin) {
        // no launch longer than a level's may be
        const double most = std::max(1.0, ctx->max_launch_cells / ((double)n * n * batch));
        for (int done = 0; done < steps;) {
            const int T = (int)std::min<double>(steps - done, most);
            HIP_TRY(dk::heat_resident(rho, n, batch, T, a, s));
            done += T;
        }
    } else {
        // passes in pairs, so that the fields end in rho; a single step is a pass and a copy
        int passes = (steps + dk::kMaxT - 1) / dk::kMaxT;
        if (passes % 2 && steps > 1) ++passes;
        float* to = work;
        for (int done = 0, k = 0; k < passes; ++k) {
            const int T = (steps - done + passes - k - 1) / (passes - k);
            HIP_TRY(dk::heat_windows(from, to, n, batch, T, a, s));
            done += T;
            std::swap(from, to);
        }
    }
    HIP_TRY(hipEventRecord(e1, s));
    if (from != rho) HIP_TRY(hipMemcpyAsync(rho, from, sizeof(float) * (size_t)n * n * batch, hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));       // the copy, too: rho and work are the caller's again
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
    if (kernel_ms) *kernel_ms = ms;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return DK_OK;
}
