// dk_tuning.cpp -- tile-shape choice for the resident kernels (forced, cached, or timed on a
// short batch) and the JSON text of the choices.
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <regex>
#include <sstream>

#include "dk_host.h"

// ------------------------------------------------------------------------------------------
// Tile shapes.  A lane owns C = 2 columns and R rows; a sample uses (n/2) x (n/R) lanes and a
// block holds S samples (about 256 lanes, or four times as many samples in 1024-lane blocks).
// Several (R, S) per grid size are compiled; choose_shape picks one by the size of the batch, or by
// timing them for large jobs.  FP64 states have the shapes of at most 8 rows and 256 lanes per block's worth of
// samples (16 rows at 128 x 128); the others stand for their shape 0.  One-row shapes are for single paths
// (a pair's coarse cell needs two rows): pairs run them with two (shape_run).
// ------------------------------------------------------------------------------------------
namespace dk {

// rows per lane of shape variant v for grid size nf (0 = no such variant); variant 0 is the
// default (8 rows: the fastest measured on MI355X for every grid size of the hierarchy)
int shape_rows(int nf, int v)
{
    switch (nf) {
        case 4: return v == 0 ? 4 : 0;
        case 8: { const int r[] = {8, 2, 4, 8, 1}; return v >= 0 && v < 5 ? r[v] : 0; }
        case 16: { const int r[] = {8, 4, 2, 8, 1}; return v >= 0 && v < 5 ? r[v] : 0; }
        case 32: { const int r[] = {8, 4, 16, 8, 2}; return v >= 0 && v < 5 ? r[v] : 0; }
        case 64: { const int r[] = {8, 16, 8, 4, 2}; return v >= 0 && v < 5 ? r[v] : 0; }
        case 128: { const int r[] = {8, 16}; return v >= 0 && v < 2 ? r[v] : 0; }
        default: return 0;
    }
}

namespace {
bool wide_shape(int nf, int v) { return (nf == 8 || nf == 16 || nf == 32) ? v == 3 : (nf == 64 && v == 2); }
}  // namespace

// samples per block of shape variant v
int shape_spw(int nf, int v)
{
    const int r = shape_rows(nf, v);
    if (r == 0) return 0;
    const int ts = (nf / 2) * (nf / r);
    const int base = ts >= 256 ? 1 : 256 / ts;
    return wide_shape(nf, v) ? 4 * base : base;
}

int shape_run(int nf, int v, bool f64, bool pair)
{
    if (pair && shape_rows(nf, v) == 1) {
        v = 0;
        while (shape_rows(nf, v) != 2) ++v;
    }
    return f64 && nf < 128 && (shape_rows(nf, v) > 8 || wide_shape(nf, v)) ? 0 : v;
}

}  // namespace dk

namespace dkh {

namespace {

std::string device_arch(int device)
{
    hipDeviceProp_t pr;
    if (hipGetDeviceProperties(&pr, device) != hipSuccess) return "unknown";
    std::string a = pr.gcnArchName;
    const size_t c = a.find(':');
    return c == std::string::npos ? a : a.substr(0, c);
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Tile-shape choices as JSON text:
//   {"format": "dk-tile-shapes-1", "arch": "gfx950",
//    "shapes": [{"n": 128, "pair": 1, "flux": 0, "rows": 8, "spw": 1}, ...]}
// ("spw", samples per block, may be left out: then the shape with that R and ~256-lane blocks)
// ------------------------------------------------------------------------------------------
std::string tuning_json(const dk_context* ctx)
{
    std::ostringstream o;
    o << "{\"format\": \"dk-tile-shapes-1\", \"arch\": \"" << device_arch(ctx->device) << "\", \"shapes\": [";
    bool first = true;
    for (const auto& kv : ctx->tuned) {
        const int nf = (int)(kv.first >> 8), pair = (int)((kv.first >> 4) & 0xF), flux = (int)(kv.first & 0xF);
        o << (first ? "" : ", ") << "{\"n\": " << nf << ", \"pair\": " << pair << ", \"flux\": " << flux
          << ", \"rows\": " << dk::shape_rows(nf, kv.second) << ", \"spw\": " << dk::shape_spw(nf, kv.second) << "}";
        first = false;
    }
    for (const auto& kv : ctx->tuned_depth) {
        const int nf = (int)(kv.first >> 8), pair = (int)((kv.first >> 4) & 0xF), flux = (int)(kv.first & 0xF);
        o << (first ? "" : ", ") << "{\"n\": " << nf << ", \"pair\": " << pair << ", \"flux\": " << flux
          << ", \"depth\": " << kv.second << "}";
        first = false;
    }
    o << "]}";
    return o.str();
}

int load_tuning_json(dk_context* ctx, const std::string& text)
{
    static const std::regex fmt("\"format\"\\s*:\\s*\"dk-tile-shapes-1\"");
    static const std::regex arch("\"arch\"\\s*:\\s*\"([^\"]*)\"");
    static const std::regex entry("\\{\\s*\"n\"\\s*:\\s*(\\d+)\\s*,\\s*\"pair\"\\s*:\\s*(\\d+)\\s*,\\s*\"flux\"\\s*:\\s*(\\d+)"
                                  "\\s*,\\s*\"rows\"\\s*:\\s*(\\d+)(?:\\s*,\\s*\"spw\"\\s*:\\s*(\\d+))?\\s*\\}");
    if (!std::regex_search(text, fmt)) return fail(DK_EINVAL, "tuning JSON: missing \"format\": \"dk-tile-shapes-1\"");
    std::smatch m;
    if (!std::regex_search(text, m, arch)) return fail(DK_EINVAL, "tuning JSON: missing \"arch\"");
    const std::string dev = device_arch(ctx->device);
    if (m[1].str() != dev) return fail(DK_EINVAL, "tuning JSON is for %s, the device is %s", m[1].str().c_str(), dev.c_str());
    static const std::regex dentry("\\{\\s*\"n\"\\s*:\\s*(\\d+)\\s*,\\s*\"pair\"\\s*:\\s*(\\d+)\\s*,\\s*\"flux\"\\s*:\\s*(\\d+)"
                                   "\\s*,\\s*\"depth\"\\s*:\\s*(\\d+)\\s*\\}");
    std::map<long, int> got, gotd;
    for (auto it = std::sregex_iterator(text.begin(), text.end(), dentry); it != std::sregex_iterator(); ++it) {
        const int nf = std::stoi((*it)[1]), pair = std::stoi((*it)[2]), flux = std::stoi((*it)[3]);
        const int depth = std::stoi((*it)[4]);
        if (pair > 1 || (flux != DK_FLUX_CENTRAL && flux != DK_FLUX_STAGGERED) || !dk::stream_supported(nf) ||
            !dk::stream_depth_supported(depth))
            return fail(DK_EINVAL, "tuning JSON: bad streaming entry for n = %d", nf);
        gotd[((long)nf << 8) | ((long)pair << 4) | (long)flux] = depth;
    }
    for (auto it = std::sregex_iterator(text.begin(), text.end(), entry); it != std::sregex_iterator(); ++it) {
        const int nf = std::stoi((*it)[1]), pair = std::stoi((*it)[2]), flux = std::stoi((*it)[3]);
        const int rows = std::stoi((*it)[4]);
        if (pair > 1 || (flux != DK_FLUX_CENTRAL && flux != DK_FLUX_STAGGERED))
            return fail(DK_EINVAL, "tuning JSON: bad entry for n = %d", nf);
        int v = 0;
        while (dk::shape_rows(nf, v) > 0 && dk::shape_rows(nf, v) != rows) ++v;
        if (dk::shape_rows(nf, v) == 0) return fail(DK_EINVAL, "tuning JSON: no %d-row shape for n = %d", rows, nf);
        if ((*it)[5].matched) {
            const int spw = std::stoi((*it)[5]);
            while (dk::shape_rows(nf, v) > 0 && !(dk::shape_rows(nf, v) == rows && dk::shape_spw(nf, v) == spw)) ++v;
            if (dk::shape_rows(nf, v) == 0)
                return fail(DK_EINVAL, "tuning JSON: no %d-row shape with %d samples per block for n = %d", rows, spw, nf);
        }
        got[((long)nf << 8) | ((long)pair << 4) | (long)flux] = dk::shape_run(nf, v, false, pair != 0);
    }
    for (const auto& kv : got) ctx->tuned[kv.first] = kv.second;
    for (const auto& kv : gotd) ctx->tuned_depth[kv.first] = kv.second;
    return DK_OK;
}

// DK_TUNE_CACHE: the file the context loads when created and rewrites after every new choice
void save_tuning_cache(const dk_context* ctx)
{
    const char* path = std::getenv("DK_TUNE_CACHE");
    if (!path || !*path) return;
    const std::string tmp = std::string(path) + ".tmp";
    {
        std::ofstream f(tmp);
        if (!f) return;
        f << tuning_json(ctx) << "\n";
    }
    std::rename(tmp.c_str(), path);
}

// Rows per lane for a batch that leaves the GPU's wavefront slots partly empty (1024 SIMDs, 4 wavefronts
// each at these register counts).  A step then takes a wavefront's own latency, about 0.4 us a row, so the
// fewest rows are the fastest until the extra wavefronts of the smaller tiles (which repeat the halo and
// lane-exchange work more often) fill the chip.  The lines lie where the measured times of one step cross
// (MI355X, pairs; us at 2 / 4 / 8 rows):
//   FP32   8^2: 4096 samples 1.2 / 2.0 / 3.5, 32768 4.8 / 4.7 / 5.1, 65536 8.7 / 8.2 / 8.6
//         16^2: 1024 samples 1.1 / 1.9 / 3.6, 8192 4.7 / 5.1 / 5.2, 32768 15.9 / 16.7 / 15.2
//         32^2: 1024 samples 2.7 / 2.8 / 3.9, 3456 7.5 / 7.5 / 8.5, 7776 15.8 / 15.7 / 15.1
//         64^2: 256 samples 2.7 / 2.7 / 3.6, 257 4.7 / 4.2 / 4.1, 1536 14.3 / 12.5 / 11.3
//   FP64   8^2: 4096 samples 1.5 / 2.4 / 3.9, 16384 3.9 / 3.8 / 4.2, 32768 7.2 / 6.6 / 6.5
//         16^2: 2048 samples 2.4 / 2.4 / 4.1, 8192 7.3 / 6.9 / 7.2, 16384 13.4 / 12.5 / 12.7
//         32^2: 512 samples 2.2 / 2.4 / 4.0, 1024 3.8 / 3.7 / 4.2, 7776 23.5 / 22.8 / 21.3
//         64^2: 256 samples 4.0 / 3.6 / 4.0, 257 7.1 / 6.1 / 5.7, 1000 14.4 / 11.9 / 11.9
// (4^2 and 128^2 have no smaller tile.)  Single paths cross at the same sizes within a few percent, and
// can run one row per lane:
//   FP32   8^2: 1024 samples 0.69 against 1.0 at 2 rows, 8192 1.5 / 1.4;  16^2: 512 samples 0.72 / 0.98, 2048 1.6 / 1.5
//   FP64   8^2: 1024 samples 1.1 / 1.5, 4096 1.6 / 1.6;  16^2: 512 samples 1.1 / 1.4, 1024 1.6 / 1.6
int small_batch_rows(int nf, bool f64, bool pair, uint64_t count)
{
    struct Line { int n; uint64_t one, two, four; };
    static const Line f32[] = {{8, 6000, 24000, 80000}, {16, 1200, 20000, 0}, {32, 0, 2500, 6000}, {64, 0, 256, 0}};
    static const Line d64[] = {{8, 3000, 8192, 20000}, {16, 800, 3000, 10000}, {32, 0, 600, 6000}, {64, 0, 0, 256}};
    for (const Line& l : f64 ? d64 : f32)
        if (l.n == nf) return !pair && count <= l.one ? 1 : (count <= l.two ? 2 : (count <= l.four ? 4 : 0));
    return 0;
}

// Tile-shape choice: a forced variant, the rows of a small batch, and for batches that fill the chip a choice that
// was timed or loaded (FP32), the fastest variant on a tuning batch (FP32 jobs of 1e11 cell updates; same tables, at
// most 2048 fine steps, samples from the requested range, the outputs discarded), or the default shape.  The timed
// choice is one of full chips, so the batch's size comes first: 1000 pairs of 32 x 32 take 1.28 ms with their two
// rows and 1.86 ms with the eight of a full chip.
int choose_shape(dk_context* ctx, const dk_problem* p, bool pair, const dk::LevelArgs& A, uint64_t count,
                 double cells_per_sample, hipStream_t s, int* variant)
{
    *variant = 0;
    const int nf = A.nf;
    auto f = ctx->forced_shape.find(nf);
    if (f != ctx->forced_shape.end() && f->second >= 0) {
        if (dk::shape_rows(nf, f->second) == 0) return fail(DK_EINVAL, "no tile-shape variant %d for n = %d", f->second, nf);
        *variant = f->second;
        return DK_OK;
    }
    const bool f64 = p->precision == DK_PREC_F64;
    if (const int rows = small_batch_rows(nf, f64, pair, count)) {
        while (dk::shape_rows(nf, *variant) != rows) ++*variant;
        return DK_OK;
    }
    if (f64) return DK_OK;
    const long key = ((long)nf << 8) | ((long)pair << 4) | (long)p->flux;
    auto t = ctx->tuned.find(key);
    if (t != ctx->tuned.end()) { *variant = t->second; return DK_OK; }
    if ((double)count * cells_per_sample < 1e11) return DK_OK;
    int nvar = 0;
    while (dk::shape_rows(nf, nvar) > 0) ++nvar;
    if (nvar < 2) { ctx->tuned[key] = 0; save_tuning_cache(ctx); return DK_OK; }
    // The batch resembles a production launch: the level's own horizon (capped at 2048 steps;
    // a much shorter one favours shapes whose per-sample setup is cheaper, not their time loop)
    // and about one full round of blocks (256 CUs) of the larger grids.
    dk::LevelArgs T = A;
    T.count = std::min<uint64_t>(count, nf <= 32 ? 8192 : (nf == 64 ? 1024 : 256));
    T.steps = std::min(A.steps, 2048);
    // on 8^2 and 16^2 it is a small batch itself, on which fewer rows win as they do not on a full chip
    const bool small = small_batch_rows(nf, false, pair, T.count) != 0;
    T.field_f = nullptr;
    T.field_c = nullptr;
    int rc = ctx->per_sample.ensure(sizeof(double) * 2 * A.n_obs * T.count);
    if (rc) return rc;
    T.out = (double*)ctx->per_sample.p;
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    ctx->tune_log.clear();
    double best = 1e300;
    int bestv = 0;
    for (int v = 0; v < nvar; ++v) {
        if (dk::shape_run(nf, v, false, pair) != v || (small && dk::shape_rows(nf, v) < 8)) continue;
        dk::LevelKind K{p->precision, pair, p->flux, v};
        HIP_TRY(dk::launch_level(K, T, s));   // warm-up
        HIP_TRY(hipEventRecord(e0, s));
        HIP_TRY(dk::launch_level(K, T, s));
        HIP_TRY(dk::launch_level(K, T, s));
        HIP_TRY(hipEventRecord(e1, s));
        HIP_TRY(hipEventSynchronize(e1));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
        ctx->tune_log.push_back(std::make_pair(v, (double)ms));
        if (ms < best) { best = ms; bestv = v; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    ctx->tuned[key] = bestv;
    save_tuning_cache(ctx);
    if (std::getenv("DK_LOG")) {
        std::fprintf(stderr, "[dk] tuned n=%d pair=%d flux=%d:", nf, (int)pair, p->flux);
        for (auto& kv : ctx->tune_log)
            std::fprintf(stderr, " R=%d/S=%d %.3f ms", dk::shape_rows(nf, kv.first), dk::shape_spw(nf, kv.first), kv.second);
        std::fprintf(stderr, " -> R=%d/S=%d\n", dk::shape_rows(nf, bestv), dk::shape_spw(nf, bestv));
        std::fflush(stderr);
    }
    *variant = bestv;
    return DK_OK;
}

}  // namespace dkh
