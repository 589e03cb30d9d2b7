// Plans: batches of sonar and camera frames prepared once and launched many
// times (frame tables uploaded once, launch sequences optionally captured in
// HIP graphs), and the launch-shape autotuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/oceansim.h"
#include "device.hpp"
#include "host.hpp"
#include "launch.hpp"

using namespace osim;
using namespace osim::host;

struct oceansim_plan {
    std::vector<oceansim_sonar_frame> sonar;
    std::vector<oceansim_uw_frame> camera;
    const oceansim_sonar_params *sp = nullptr;
    int n_srows = 0;
    const float *refl = nullptr;
    int n_mat = 1;
    const oceansim_water_params *wp = nullptr;
    int n_wrows = 0;
    float *g_refl = nullptr, *g_sp = nullptr, *g_wp = nullptr;
    int flags = 0;
    Tuning tune;
    SonarPlan sf, sb;
    UwPlan uf, ub;
    char *mem = nullptr;        // workspaces and frame tables
    char *stencil_mem = nullptr;
    char *savedp_mem = nullptr;   // binned sums of range-normalised frames (backward plans)
    // transposed fan operators of the sonar frames (backward plans), per frame
    // (nullptr where a frame has none)
    char *fant_mem = nullptr;
    std::vector<const int *> fant_ptr;
    std::vector<const FanEntry *> fant_ent;
    char *ws_sf = nullptr, *ws_sb = nullptr, *ws_uf = nullptr, *ws_ub = nullptr;
    hipStream_t cap = nullptr;   // capture stream (default priority)
    // with both kinds of frames the camera frames ride along in the forward
    // launches of the sonar frames
    bool fused = false;
    // the backward runs from the forward's material pairs (k_pair_bwd)
    bool pair = false;
    hipGraphExec_t g_fwd = nullptr, g_bwd = nullptr;
};

namespace {

// ---------------------------------------------------------------------------
// Agreement check of a tuning candidate against the reference outputs:
// counts elements with |a - b| > rtol * max(|a|, |b|) (NaN counts).
// ---------------------------------------------------------------------------
__global__ void k_count_disagree(const float *a, const float *b, long long n, float rtol, unsigned *bad) {
    unsigned local = 0;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float x = a[i], y = b[i];
        const float m = fmaxf(fabsf(x), fabsf(y));
        if (!(fabsf(x - y) <= rtol * m)) ++local;
    }
    if (local) atomicAdd(bad, local);
}

UwCompanion companion(const oceansim_plan *p, const UwDev *table) {
    UwCompanion c;
    c.table = table;
    c.n = (int)p->camera.size();
    c.blocks = p->uf.blocks;
    for (const UwDev &d : p->uf.dev) c.pixels += d.npix;
    c.params = p->wp;
    return c;
}

hipError_t camera_forward(oceansim_plan *p, hipStream_t st) {
    if (p->camera.empty() || p->uf.blocks == 0) return hipSuccess;
    return uw_forward_table(reinterpret_cast<const UwDev *>(p->ws_uf + p->uf.off_table), (int)p->camera.size(),
                            p->uf.blocks, p->wp, st);
}

hipError_t camera_reduce(oceansim_plan *p, hipStream_t st) {
    double *part = reinterpret_cast<double *>(p->ws_ub + p->ub.off_part);
    int *row = reinterpret_cast<int *>(p->ws_ub + p->ub.off_part_row);
    return reduce_rows(part, row, p->ub.blocks, 9, p->n_wrows, p->g_wp, OCEANSIM_WATER_GRAD_WIDTH, st);
}

hipError_t camera_backward(oceansim_plan *p, hipStream_t st) {
    if (p->camera.empty()) return hipSuccess;
    if (p->ub.blocks > 0) {
        hipError_t e = uw_backward_table(reinterpret_cast<const UwDev *>(p->ws_ub + p->ub.off_table),
                                         (int)p->camera.size(), p->ub.blocks, p->wp,
                                         reinterpret_cast<double *>(p->ws_ub + p->ub.off_part),
                                         reinterpret_cast<int *>(p->ws_ub + p->ub.off_part_row), st);
        if (e != hipSuccess) return e;
    }
    return camera_reduce(p, st);
}

hipError_t launch_forward(oceansim_plan *p, hipStream_t st) {
    if (p->sonar.empty()) return camera_forward(p, st);
    const UwCompanion c = p->fused ? companion(p, reinterpret_cast<const UwDev *>(p->ws_uf + p->uf.off_table)) : UwCompanion{};
    hipError_t e = sonar_forward_table(reinterpret_cast<const SonarDev *>(p->ws_sf + p->sf.off_table),
                                       (int)p->sonar.size(), p->sf.grid, p->sp, p->refl, p->n_mat, st,
                                       p->fused ? &c : nullptr);
    if (e != hipSuccess || p->fused) return e;
    return camera_forward(p, st);
}

// Sonar backward, then camera backward; with both, the camera workgroups run
// in the sonar return-gather launch and the two fixed-order reductions are
// one launch.
hipError_t launch_backward(oceansim_plan *p, hipStream_t st) {
    if (p->sonar.empty()) return camera_backward(p, st);
    const bool lane_hist = p->n_mat <= kLaneHistMats;
    const bool pair = !p->camera.empty() && p->ub.blocks > 0;
    SonarReduce sr;
    double *part = pair ? reinterpret_cast<double *>(p->ws_ub + p->ub.off_part) : nullptr;
    int *row = pair ? reinterpret_cast<int *>(p->ws_ub + p->ub.off_part_row) : nullptr;
    // the camera backward rides along in the sonar return-gather launch
    UwBwdCompanion uwb;
    if (pair) {
        uwb.table = reinterpret_cast<const UwDev *>(p->ws_ub + p->ub.off_table);
        uwb.n = (int)p->camera.size();
        uwb.blocks = p->ub.blocks;
        uwb.params = p->wp;
        uwb.part = part;
        uwb.part_row = row;
    }
    hipError_t e = sonar_backward_table(reinterpret_cast<const SonarDev *>(p->ws_sb + p->sb.off_table),
                                        (int)p->sonar.size(), p->sb.grid, p->sp, p->n_srows, p->refl, p->n_mat,
                                        reinterpret_cast<double *>(p->ws_sb + p->sb.off_part),
                                        lane_hist ? reinterpret_cast<double *>(p->ws_sb + p->sb.off_refl_part)
                                                  : nullptr,
                                        p->g_sp, p->g_refl, st, pair ? &sr : nullptr, pair ? &uwb : nullptr);
    if (e != hipSuccess) return e;
    if (!pair) return camera_backward(p, st);
    RowsReduce rr;
    rr.part = part;
    rr.row = row;
    rr.n_slots = p->ub.blocks;
    rr.width = 9;
    rr.out = p->g_wp;
    rr.out_stride = OCEANSIM_WATER_GRAD_WIDTH;
    rr.blocks = p->n_wrows * OCEANSIM_WATER_GRAD_WIDTH;
    return reduce_pair(sr, rr, st);
}

// ---------------------------------------------------------------------------
// Tuning cache: per process, optionally persisted as JSON
// ({"key": [fwd_tile_bins, chunk, fant_bpt], ...}).
// ---------------------------------------------------------------------------
std::mutex g_tune_mu;
std::map<std::string, Tuning> g_tune;
bool g_tune_loaded = false;

const char *tune_file() {
    const char *p = getenv("OCEANSIM_TUNE_CACHE");
    return (p && *p) ? p : nullptr;
}

void tune_load_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char *path = tune_file();
    if (!path) return;
    FILE *fh = fopen(path, "r");
    if (!fh) return;
    std::string text;
    char buf[4096];
    size_t n;
    while ((n = fread(buf, 1, sizeof buf, fh)) > 0) text.append(buf, n);
    fclose(fh);
    size_t pos = 0;
    while ((pos = text.find('"', pos)) != std::string::npos) {
        size_t end = text.find('"', pos + 1);
        if (end == std::string::npos) break;
        std::string key = text.substr(pos + 1, end - pos - 1);
        Tuning t;
        if (sscanf(text.c_str() + end + 1, " : [ %d , %d , %d ]", &t.fwd_tile_bins, &t.chunk, &t.fant_bpt) == 3) {
            if (t.fant_bpt != 1 && t.fant_bpt != 2 && t.fant_bpt != 4) t.fant_bpt = 0;
            g_tune[key] = t;
        }
        pos = end + 1;
    }
}

void tune_save_locked() {
    const char *path = tune_file();
    if (!path) return;
    std::string tmp = std::string(path) + ".tmp";
    FILE *fh = fopen(tmp.c_str(), "w");
    if (!fh) return;
    fprintf(fh, "{\n");
    size_t k = 0;
    for (auto &kv : g_tune)
        fprintf(fh, "  \"%s\": [%d, %d, %d]%s\n", kv.first.c_str(), kv.second.fwd_tile_bins, kv.second.chunk,
                kv.second.fant_bpt, ++k < g_tune.size() ? "," : "");
    fprintf(fh, "}\n");
    fclose(fh);
    rename(tmp.c_str(), path);
}

int ilog2(long long v) {
    int e = 0;
    while (v > 1) {
        v >>= 1;
        ++e;
    }
    return e;
}

// Everything the choice depends on: the device, the sizes (powers of two), the
// kernels' materials path, and since the camera's forward blocks ride in the
// launches that are timed, and the operator rows per thread follow the fans'
// density and layout, those too.  k: counted up when a change to these kernels
// makes shapes timed before worth nothing (a file's older entries stay unread).
constexpr int kTuneKernels = 2;
std::string tune_key(const oceansim_plan *p) {
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    hipDeviceProp_t prop;
    std::string arch = "gfx";
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) arch = prop.gcnArchName;
    arch = arch.substr(0, arch.find(':'));
    long long n = 0, nb = 0, px = 0;
    for (auto &f : p->sonar) {
        n += f.n_returns;
        nb += (long long)f.n_range * f.n_azimuth;
        px += (long long)f.fan_h * f.fan_w;
    }
    int layout = 0;
    const int density = fan_density(p->sonar.data(), (int)p->sonar.size(), layout);
    const int cam = p->fused && p->uf.blocks > 0 ? 1 + ilog2(p->uf.blocks) : 0;
    char buf[256];
    snprintf(buf, sizeof buf, "%s/%dcu/k%d-s%d-r%d-b%d-f%d-d%d-l%d-c%d-m%d-bw%d", arch.c_str(), cus, kTuneKernels,
             ilog2(p->sonar.size()), ilog2(n), ilog2(nb), ilog2(px), density, layout, cam,
             p->n_mat <= kLaneHistMats ? 0 : 1, (p->flags & OCEANSIM_PLAN_BACKWARD) ? 1 : 0);
    return buf;
}

struct Candidate {
    Tuning t;
    SonarPlan f, b;
    double us = 1e30;
    bool ok = false;
};

// Times `fn` (5 launches after `warm` warm-up launches) on stream st, in
// microseconds.
template <class F>
double time_us(F fn, hipStream_t st, int warm = 1) {
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return 1e30;
    if (hipEventCreate(&b) != hipSuccess) {
        (void)hipEventDestroy(a);
        return 1e30;
    }
    for (int k = 0; k < warm; ++k) fn();
    (void)hipEventRecord(a, st);
    for (int k = 0; k < 5; ++k) fn();
    (void)hipEventRecord(b, st);
    float ms = 1e30f;
    if (hipEventSynchronize(b) == hipSuccess) (void)hipEventElapsedTime(&ms, a, b);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    return ms * 1e3 / 5.0;
}

void attach_fan_transposes(const oceansim_plan *p, SonarPlan &P);

// Chooses p->tune by timing candidates: forward tile and chunk sizes, then
// the bins per thread of the backward through the transposed fan operators
// (built before tuning).
int autotune(oceansim_plan *p, hipStream_t st) {
    const std::string key = tune_key(p);
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        tune_load_locked();
        auto it = g_tune.find(key);
        if (it != g_tune.end()) {
            p->tune = it->second;
            return OCEANSIM_OK;
        }
    }
    const int n = (int)p->sonar.size();
    std::vector<Candidate> cands;
    cands.push_back(Candidate{});   // the default shape is the reference
    for (int ft : {1024, 2048, 4096, 8192, 16384})
        for (int ch : {512, 1024, 2048, 4096, 8192}) {
            Candidate c;
            c.t.fwd_tile_bins = ft;
            c.t.chunk = ch;
            cands.push_back(c);
        }
    // A pair backward runs one workgroup per forward tile: with it, the tile
    // and chunk sizes are timed on the forward and the backward together.
    const bool with_bwd = p->pair && (p->flags & OCEANSIM_PLAN_BACKWARD);
    size_t ws = 0, wsb_pair = 0;
    for (auto &c : cands) {
        int rc = plan_sonar(p->sonar.data(), n, p->n_srows, p->n_mat, false, c.f, &c.t, true, p->pair);
        if (rc) return rc;
        ws = std::max(ws, c.f.bytes);
        if (with_bwd) {
            rc = plan_sonar(p->sonar.data(), n, p->n_srows, p->n_mat, true, c.b, &c.t, true, true);
            if (rc) return rc;
            attach_fan_transposes(p, c.b);
            wsb_pair = std::max(wsb_pair, c.b.bytes);
        }
    }
    // reference outputs
    size_t out_elems = 0;
    for (auto &f : p->sonar) {
        if (f.polar) out_elems += (size_t)f.n_range * f.n_azimuth;
        if (f.fan) out_elems += (size_t)f.fan_h * f.fan_w;
    }
    char *tmp = nullptr, *tmp_b = nullptr;
    float *ref = nullptr;
    unsigned *bad = nullptr;
    // with camera frames the forward carries them along (in the binning or
    // the tile launch, by shape), so candidates are timed with them
    UwDev *uw_table = nullptr;
    UwCompanion uwc;
    if (p->fused && p->uf.blocks > 0) {
        hipError_t ue = hipMalloc((void **)&uw_table, sizeof(UwDev) * p->uf.dev.size());
        if (ue == hipSuccess)
            ue = hipMemcpyAsync(uw_table, p->uf.dev.data(), sizeof(UwDev) * p->uf.dev.size(), hipMemcpyHostToDevice,
                                st);
        if (ue != hipSuccess) {
            if (uw_table) (void)hipFree(uw_table);
            return hip_fail(ue, "autotune camera table");
        }
        uwc = companion(p, uw_table);
    }
    hipError_t e = hipMalloc(&tmp, ws + 256);
    if (e != hipSuccess) {
        if (uw_table) (void)hipFree(uw_table);
        return hip_fail(e, "autotune workspace");
    }
    if (with_bwd) {
        e = hipMalloc(&tmp_b, wsb_pair + 256);
        if (e != hipSuccess) {
            (void)hipFree(tmp);
            if (uw_table) (void)hipFree(uw_table);
            return hip_fail(e, "autotune workspace");
        }
    }
    e = hipMalloc(&ref, std::max<size_t>(out_elems, 1) * sizeof(float) + 256);
    if (e == hipSuccess) e = hipMalloc(&bad, sizeof(unsigned));
    if (e != hipSuccess) {
        (void)hipFree(tmp);
        if (tmp_b) (void)hipFree(tmp_b);
        if (ref) (void)hipFree(ref);
        if (uw_table) (void)hipFree(uw_table);
        return hip_fail(e, "autotune buffers");
    }
    auto copy_outputs = [&](bool to_ref) -> hipError_t {
        size_t off = 0;
        for (auto &f : p->sonar) {
            const size_t a = f.polar ? (size_t)f.n_range * f.n_azimuth : 0;
            const size_t b = f.fan ? (size_t)f.fan_h * f.fan_w : 0;
            hipError_t r = hipSuccess;
            if (a) {
                if (to_ref) r = hipMemcpyAsync(ref + off, f.polar, a * 4, hipMemcpyDeviceToDevice, st);
                else hipLaunchKernelGGL(k_count_disagree, dim3(256), dim3(256), 0, st, f.polar, ref + off,
                                        (long long)a, 1e-5f, bad);
                off += a;
            }
            if (r == hipSuccess && b) {
                if (to_ref) r = hipMemcpyAsync(ref + off, f.fan, b * 4, hipMemcpyDeviceToDevice, st);
                else hipLaunchKernelGGL(k_count_disagree, dim3(256), dim3(256), 0, st, f.fan, ref + off,
                                        (long long)b, 1e-5f, bad);
                off += b;
            }
            if (r != hipSuccess) return r;
        }
        return hipGetLastError();
    };
    int rc = OCEANSIM_OK;
    for (size_t k = 0; k < cands.size() && rc == OCEANSIM_OK; ++k) {
        Candidate &c = cands[k];
        carve_sonar(c.f, tmp, false);
        e = upload_table(c.f.dev, tmp, c.f.off_table, st);
        const SonarDev *table = reinterpret_cast<const SonarDev *>(tmp + c.f.off_table);
        const SonarDev *table_b = nullptr;
        if (with_bwd && e == hipSuccess) {
            carve_sonar(c.b, tmp_b, true);
            link_pairs(c.b, c.f);
            e = upload_table(c.b.dev, tmp_b, c.b.off_table, st);
            table_b = reinterpret_cast<const SonarDev *>(tmp_b + c.b.off_table);
        }
        auto fwd = [&]() {
            return sonar_forward_table(table, n, c.f.grid, p->sp, p->refl, p->n_mat, st, uw_table ? &uwc : nullptr);
        };
        auto run = [&]() {
            hipError_t r = fwd();
            if (r == hipSuccess && table_b)
                r = sonar_backward_table(table_b, n, c.b.grid, p->sp, p->n_srows, p->refl, p->n_mat,
                                         reinterpret_cast<double *>(tmp_b + c.b.off_part),
                                         reinterpret_cast<double *>(tmp_b + c.b.off_refl_part), p->g_sp,
                                         p->g_refl, st);
            return r;
        };
        if (e == hipSuccess) e = fwd();
        if (e == hipSuccess && k == 0) e = copy_outputs(true);
        unsigned nbad = 0;
        if (e == hipSuccess && k > 0) {
            e = hipMemsetAsync(bad, 0, sizeof(unsigned), st);
            if (e == hipSuccess) e = copy_outputs(false);
            if (e == hipSuccess) e = hipMemcpyAsync(&nbad, bad, sizeof(unsigned), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
        }
        if (e != hipSuccess) {
            rc = hip_fail(e, "autotune forward");
            break;
        }
        c.ok = nbad == 0;
        // the first candidate also brings the GPU to its working clocks: on a
        // fresh box the first few large launches run up to a quarter slower,
        // which would favour the candidates timed later
        if (c.ok) c.us = time_us(run, st, k == 0 ? 10 : 1);
    }
    // One pass over the candidates is at the mercy of clock and power drift
    // along the sweep: the three fastest are timed again, interleaved over
    // three rounds, and each keeps its best time.
    if (rc == OCEANSIM_OK) {
        std::vector<size_t> top;
        for (size_t k = 0; k < cands.size(); ++k)
            if (cands[k].ok) top.push_back(k);
        std::sort(top.begin(), top.end(), [&](size_t a, size_t b) { return cands[a].us < cands[b].us; });
        if (top.size() > 3) top.resize(3);
        for (int round = 0; round < 3 && top.size() > 1; ++round)
            for (size_t k : top) {
                Candidate &c = cands[k];
                carve_sonar(c.f, tmp, false);
                e = upload_table(c.f.dev, tmp, c.f.off_table, st);
                const SonarDev *table = reinterpret_cast<const SonarDev *>(tmp + c.f.off_table);
                const SonarDev *table_b = nullptr;
                if (with_bwd && e == hipSuccess) {
                    carve_sonar(c.b, tmp_b, true);
                    link_pairs(c.b, c.f);
                    e = upload_table(c.b.dev, tmp_b, c.b.off_table, st);
                    table_b = reinterpret_cast<const SonarDev *>(tmp_b + c.b.off_table);
                }
                if (e != hipSuccess) break;
                auto run = [&]() {
                    hipError_t r = sonar_forward_table(table, n, c.f.grid, p->sp, p->refl, p->n_mat, st,
                                                       uw_table ? &uwc : nullptr);
                    if (r == hipSuccess && table_b)
                        r = sonar_backward_table(table_b, n, c.b.grid, p->sp, p->n_srows, p->refl, p->n_mat,
                                                 reinterpret_cast<double *>(tmp_b + c.b.off_part),
                                                 reinterpret_cast<double *>(tmp_b + c.b.off_refl_part), p->g_sp,
                                                 p->g_refl, st);
                    return r;
                };
                c.us = std::min(c.us, time_us(run, st));
            }
        if (e != hipSuccess) rc = hip_fail(e, "autotune re-timing");
    }
    size_t best = 0;
    for (size_t k = 1; k < cands.size(); ++k)
        if (cands[k].ok && cands[k].us < cands[best].us) best = k;
    Tuning chosen = cands[best].t;   // zeros: the built-in heuristic won

    if (rc == OCEANSIM_OK && (p->flags & OCEANSIM_PLAN_BACKWARD)) {
        // backward: bins per thread through the transposed fan operators,
        // after one forward under the chosen shape
        SonarPlan fp;
        rc = plan_sonar(p->sonar.data(), n, p->n_srows, p->n_mat, false, fp, &chosen, true, p->pair);
        if (rc == OCEANSIM_OK && fp.bytes > ws) rc = fail(OCEANSIM_E_WORKSPACE, "autotune: forward workspace");
        std::vector<Candidate> bc;
        for (int bpt : {0, 1, 2, 4}) {   // 0: the size heuristic, the reference
            Candidate c;
            c.t = chosen;
            c.t.fant_bpt = bpt;
            bc.push_back(c);
        }
        size_t wsb = 0;
        for (auto &c : bc) {
            if (rc) break;
            rc = plan_sonar(p->sonar.data(), n, p->n_srows, p->n_mat, true, c.b, &c.t, true, p->pair);
            attach_fan_transposes(p, c.b);
            wsb = std::max(wsb, c.b.bytes);
        }
        char *tb = nullptr;
        if (rc == OCEANSIM_OK) {
            e = hipMalloc(&tb, wsb + 256);
            if (e != hipSuccess) rc = hip_fail(e, "autotune workspace");
        }
        if (rc == OCEANSIM_OK) {
            carve_sonar(fp, tmp, false);
            e = upload_table(fp.dev, tmp, fp.off_table, st);
            if (e == hipSuccess)
                e = sonar_forward_table(reinterpret_cast<const SonarDev *>(tmp + fp.off_table), n, fp.grid, p->sp,
                                        p->refl, p->n_mat, st);
            std::vector<float> ref_g;
            const size_t ng = (size_t)p->n_mat + (size_t)p->n_srows * OCEANSIM_SONAR_GRAD_WIDTH;
            const bool lane_hist = p->n_mat <= kLaneHistMats;
            for (size_t k = 0; k < bc.size() && e == hipSuccess; ++k) {
                Candidate &c = bc[k];
                carve_sonar(c.b, tb, true);
                if (p->pair) link_pairs(c.b, fp);
                e = upload_table(c.b.dev, tb, c.b.off_table, st);
                const SonarDev *table = reinterpret_cast<const SonarDev *>(tb + c.b.off_table);
                auto run = [&]() {
                    return sonar_backward_table(table, n, c.b.grid, p->sp, p->n_srows, p->refl, p->n_mat,
                                                reinterpret_cast<double *>(tb + c.b.off_part),
                                                lane_hist ? reinterpret_cast<double *>(tb + c.b.off_refl_part)
                                                          : nullptr,
                                                p->g_sp, p->g_refl, st);
                };
                if (e == hipSuccess) e = run();
                std::vector<float> g(ng);
                if (e == hipSuccess)
                    e = hipMemcpyAsync(g.data(), p->g_refl, sizeof(float) * p->n_mat, hipMemcpyDeviceToHost, st);
                if (e == hipSuccess)
                    e = hipMemcpyAsync(g.data() + p->n_mat, p->g_sp,
                                       sizeof(float) * p->n_srows * OCEANSIM_SONAR_GRAD_WIDTH,
                                       hipMemcpyDeviceToHost, st);
                if (e == hipSuccess) e = hipStreamSynchronize(st);
                if (e != hipSuccess) break;
                if (k == 0) ref_g = g;
                float peak = 0.0f;
                for (float v : ref_g) peak = std::max(peak, std::fabs(v));
                // an all-zero reference (zero loss gradients) checks nothing:
                // then only the default shape is accepted
                c.ok = k == 0 || peak > 0.0f;
                for (size_t i = 0; i < ng; ++i)
                    if (!(std::fabs(g[i] - ref_g[i]) <= 1e-5f * std::max(std::fabs(ref_g[i]), 1e-3f * peak)))
                        c.ok = false;
                if (c.ok) c.us = time_us(run, st);
            }
            if (e != hipSuccess) rc = hip_fail(e, "autotune backward");
            size_t bbest = 0;
            for (size_t k = 1; k < bc.size(); ++k)
                if (bc[k].ok && bc[k].us < bc[bbest].us) bbest = k;
            chosen.fant_bpt = bc[bbest].t.fant_bpt;
        }
        if (tb) (void)hipFree(tb);
    }
    (void)hipStreamSynchronize(st);
    (void)hipFree(tmp);
    if (tmp_b) (void)hipFree(tmp_b);
    (void)hipFree(ref);
    (void)hipFree(bad);
    if (uw_table) (void)hipFree(uw_table);
    if (rc) return rc;
    p->tune = chosen;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[key] = chosen;
    tune_save_locked();
    return OCEANSIM_OK;
}

void free_plan(oceansim_plan *p) {
    if (!p) return;
    (void)hipDeviceSynchronize();
    if (p->g_fwd) (void)hipGraphExecDestroy(p->g_fwd);
    if (p->g_bwd) (void)hipGraphExecDestroy(p->g_bwd);
    if (p->cap) (void)hipStreamDestroy(p->cap);
    if (p->mem) (void)hipFree(p->mem);
    if (p->stencil_mem) (void)hipFree(p->stencil_mem);
    if (p->savedp_mem) (void)hipFree(p->savedp_mem);
    if (p->fant_mem) (void)hipFree(p->fant_mem);
    delete p;
}

// ---------------------------------------------------------------------------
// Transposed fan operators.  The fan of a frame is a fixed linear map of its
// polar image (bilinear weights that depend on the geometry alone), so its
// adjoint is a fixed sparse matrix: for each polar bin, the fan pixels that
// read it and their weights.  It is built once per plan, on the host, from
// the stencil records the fan kernel writes (the same bins and weights the
// forward pass uses), in bin-major order with each bin's entries in pixel
// order; the backward pass then gathers instead of scattering.
// ---------------------------------------------------------------------------

// Weight w and 1 - w of a stencil code (the device decoding, in FP32).
void decode_code(float e, float &w, float &omw) {
    if (std::signbit(e)) {
        w = 1.0f + e;
        omw = -e;
    } else {
        w = e;
        omw = 1.0f - e;
    }
}

struct HostRec {
    int i0, j0, ct, cl;
};

// Visits the entries of one frame's transposed operator in pixel order:
// fn(range row i, first column j0, pixel row v, pixel column u, weight on bin
// (i, j0), weight on bin (i, j0 + 1)); a grid of one column has no second bin
// (weight 0).  The corners and the mirror pixel follow the backward tile
// kernel's reading of a saved stencil.
template <class Fn>
void for_each_entry(const oceansim_sonar_frame &f, const std::vector<HostRec> &recs, Fn fn) {
    const int W = f.fan_w, half_w = (f.fan_w + 1) / 2, n_az = f.n_azimuth;
    const bool one_row = f.n_range == 1, one_col = n_az == 1;
    for (int v = 0; v < f.fan_h; ++v)
        for (int u = 0; u < half_w; ++u) {
            const HostRec &r = recs[(size_t)v * half_w + u];
            if (r.i0 < 0) continue;
            float ct, cl, t, omt;
            std::memcpy(&ct, &r.ct, 4);
            std::memcpy(&cl, &r.cl, 4);
            decode_code(ct, t, omt);
            const int um = W - 1 - u;
            for (int side = 0; side < 2; ++side) {
                if (side == 1 && um == u) break;
                const int j0 = side == 0 || one_col ? r.j0 : n_az - 2 - r.j0;
                float sw, omsw;
                decode_code(side == 0 || one_col ? cl : -cl, sw, omsw);
                const int pu = side == 0 ? u : um;
                for (int a = 0; a < (one_row ? 1 : 2); ++a) {
                    const double wa = a == 0 ? omt : t;
                    fn(r.i0 + a, j0, v, pu, (float)(wa * (double)omsw), one_col ? 0.0f : (float)(wa * (double)sw));
                }
            }
        }
}

// Whether two frames have the same fan operator: everything the stencils and
// the operator's layout are made from (for frames that have one).
bool same_fan_operator(const oceansim_sonar_frame &a, const oceansim_sonar_frame &b) {
    return a.fan_h == b.fan_h && a.fan_w == b.fan_w && a.n_range == b.n_range && a.n_azimuth == b.n_azimuth &&
           a.r_min == b.r_min && a.r_max == b.r_max && a.fov_az == b.fov_az &&
           fan_operator_layout(a) == fan_operator_layout(b);
}

// Stencils of the frames that need an operator, then the operators; the
// plan's own stencil memory is released afterwards (the forward pass then
// saves none).
int build_fan_transposes(oceansim_plan *p, hipStream_t st) {
    const int n = (int)p->sonar.size();
    p->fant_ptr.assign(n, nullptr);
    p->fant_ent.assign(n, nullptr);
    std::vector<int> need;
    for (int i = 0; i < n; ++i)
        if (fan_operator_layout(p->sonar[i]) != 0) {
            // the backward launch shapes assume an operator for every such frame
            if (!p->sonar[i].fan_stencil) return fail(OCEANSIM_E_INVALID_ARG, "frame %d: no fan stencil", i);
            need.push_back(i);
        }
    if (need.empty()) return OCEANSIM_OK;
    // frames of one fan geometry (a batch from one sensor) share one operator:
    // built once, held once, and read from the caches by all frames but the first
    std::vector<size_t> same(need.size());
    for (size_t k = 0; k < need.size(); ++k) {
        same[k] = k;
        for (size_t j = 0; j < k; ++j)
            if (same[j] == j && same_fan_operator(p->sonar[need[j]], p->sonar[need[k]])) {
                same[k] = j;
                break;
            }
    }
    SonarPlan fp;
    int rc = plan_sonar(p->sonar.data(), n, p->n_srows, p->n_mat, false, fp, nullptr, true);
    if (rc) return rc;
    char *ws = nullptr;
    hipError_t e = hipMalloc(&ws, fp.bytes + 256);
    if (e != hipSuccess) return hip_fail(e, "fan operator workspace");
    carve_sonar(fp, ws, false);
    e = upload_table(fp.dev, ws, fp.off_table, st);
    if (e == hipSuccess)
        e = sonar_fan_stencils_table(reinterpret_cast<const SonarDev *>(ws + fp.off_table), n, fp.grid, st);
    std::vector<std::vector<HostRec>> recs(need.size());
    for (size_t k = 0; k < need.size() && e == hipSuccess; ++k) {
        if (same[k] != k) continue;
        const oceansim_sonar_frame &f = p->sonar[need[k]];
        recs[k].resize((size_t)f.fan_h * ((f.fan_w + 1) / 2));
        e = hipMemcpyAsync(recs[k].data(), f.fan_stencil, recs[k].size() * sizeof(HostRec), hipMemcpyDeviceToHost,
                           st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(ws);
    if (e != hipSuccess) return hip_fail(e, "fan stencils");
    // row-major layout: counts, offsets, then the entries in pixel order
    std::vector<std::vector<int>> ptr(need.size());
    std::vector<std::vector<FanEntry>> ent(need.size());
    size_t bytes = 0;
    std::vector<size_t> off_ptr(need.size()), off_ent(need.size());
    for (size_t k = 0; k < need.size(); ++k) {
        if (same[k] != k) continue;
        const oceansim_sonar_frame &f = p->sonar[need[k]];
        const bool mirror = fan_operator_layout(f) == 2;
        const int n_az = f.n_azimuth, ncol = mirror ? (n_az + 1) / 2 : n_az;
        const long long nrow = (long long)f.n_range * ncol;
        // A cell is in the operator if its first bin has a row (mirrored layout:
        // the others are read through their partners).  The size limit counts
        // the weights on rows.
        std::vector<int> &P = ptr[k];
        P.assign(nrow + 1, 0);
        long long weights = 0;
        for_each_entry(f, recs[k], [&](int i, int j0, int, int, float, float) {
            if (j0 >= ncol) return;
            ++P[(long long)i * ncol + j0 + 1];
            weights += j0 + 1 < ncol ? 2 : 1;
        });
        if (weights > INT32_MAX || (long long)f.fan_h * f.fan_w > INT32_MAX)
            return fail(OCEANSIM_E_UNSUPPORTED, "frame %d: fan operator too large", need[k]);
        for (long long h = 0; h < nrow; ++h) P[h + 1] += P[h];
        std::vector<int> cur(P.begin(), P.end() - 1);
        ent[k].resize((size_t)P[nrow]);
        for_each_entry(f, recs[k], [&](int i, int j0, int v, int u, float w0, float w1) {
            if (j0 >= ncol) return;
            const unsigned pix = mirror ? ((unsigned)v << 16) | (unsigned)u : (unsigned)((long long)v * f.fan_w + u);
            ent[k][cur[(long long)i * ncol + j0]++] = FanEntry{pix, w0, w1};
        });
        off_ptr[k] = bytes;
        bytes = (bytes + sizeof(int) * P.size() + kWsAlign - 1) / kWsAlign * kWsAlign;
        off_ent[k] = bytes;
        bytes = (bytes + sizeof(FanEntry) * std::max<size_t>(1, ent[k].size()) + kWsAlign - 1) / kWsAlign * kWsAlign;
    }
    e = hipMalloc(&p->fant_mem, bytes);
    if (e != hipSuccess) return hip_fail(e, "fan operator memory");
    for (size_t k = 0; k < need.size() && e == hipSuccess; ++k) {
        if (same[k] != k) {
            p->fant_ptr[need[k]] = p->fant_ptr[need[same[k]]];
            p->fant_ent[need[k]] = p->fant_ent[need[same[k]]];
            continue;
        }
        e = hipMemcpyAsync(p->fant_mem + off_ptr[k], ptr[k].data(), sizeof(int) * ptr[k].size(),
                           hipMemcpyHostToDevice, st);
        if (e == hipSuccess && !ent[k].empty())
            e = hipMemcpyAsync(p->fant_mem + off_ent[k], ent[k].data(), sizeof(FanEntry) * ent[k].size(),
                               hipMemcpyHostToDevice, st);
        p->fant_ptr[need[k]] = reinterpret_cast<const int *>(p->fant_mem + off_ptr[k]);
        p->fant_ent[need[k]] = reinterpret_cast<const FanEntry *>(p->fant_mem + off_ent[k]);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "fan operator upload");
    return OCEANSIM_OK;
}

// Backward tables of a plan read the frames' transposed operators.
void attach_fan_transposes(const oceansim_plan *p, SonarPlan &P) {
    for (size_t i = 0; i < P.dev.size() && i < p->fant_ptr.size(); ++i) {
        P.dev[i].ft_ptr = gcast(p->fant_ptr[i]);
        P.dev[i].ft_ent = gcast(p->fant_ent[i]);
    }
    P.grid.use_fant = 1;
}

int capture(oceansim_plan *p, bool backward, hipGraphExec_t *out) {
    set_capturing(true);
    hipError_t e = hipStreamBeginCapture(p->cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        const hipError_t le = backward ? launch_backward(p, p->cap) : launch_forward(p, p->cap);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(p->cap, &g);
        if (e == hipSuccess) e = le;
        if (e == hipSuccess) e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
        if (g) (void)hipGraphDestroy(g);
    }
    set_capturing(false);
    return e == hipSuccess ? OCEANSIM_OK : hip_fail(e, "graph capture");
}

}  // namespace

extern "C" {

int oceansim_plan_create(const oceansim_sonar_frame *sonar, int32_t n_sonar, const oceansim_uw_frame *camera,
                         int32_t n_camera, const oceansim_sonar_params *sonar_params_dev, int32_t n_sonar_rows,
                         const float *refl_dev, int32_t n_materials,
                         const oceansim_water_params *water_params_dev, int32_t n_water_rows,
                         float *grad_refl_dev, float *grad_sonar_params_dev, float *grad_water_params_dev,
                         int32_t flags, void *stream, oceansim_plan **plan) {
    if (!plan) return fail(OCEANSIM_E_INVALID_ARG, "plan is NULL");
    *plan = nullptr;
    if (n_sonar < 0 || n_camera < 0) return fail(OCEANSIM_E_INVALID_ARG, "negative frame count");
    if ((n_sonar > 0 && !sonar) || (n_camera > 0 && !camera))
        return fail(OCEANSIM_E_INVALID_ARG, "frames is NULL");
    if (n_sonar + n_camera == 0) return fail(OCEANSIM_E_INVALID_ARG, "a plan needs at least one frame");
    if (flags & ~(OCEANSIM_PLAN_BACKWARD | OCEANSIM_PLAN_GRAPH | OCEANSIM_PLAN_AUTOTUNE))
        return fail(OCEANSIM_E_INVALID_ARG, "unknown plan flags 0x%x", flags);
    const bool bwd = (flags & OCEANSIM_PLAN_BACKWARD) != 0;
    if (n_sonar > 0 && (!sonar_params_dev || !refl_dev))
        return fail(OCEANSIM_E_INVALID_ARG, "sonar parameters or reflectivities are NULL");
    if (n_camera > 0 && !water_params_dev) return fail(OCEANSIM_E_INVALID_ARG, "water parameters are NULL");
    if (bwd && n_sonar > 0 && (!grad_refl_dev || !grad_sonar_params_dev))
        return fail(OCEANSIM_E_INVALID_ARG, "sonar gradient outputs are NULL");
    if (bwd && n_camera > 0 && !grad_water_params_dev)
        return fail(OCEANSIM_E_INVALID_ARG, "water gradient output is NULL");
    // a backward plan gathers the fan gradient through the operator it builds
    // from the frame's rendered fan: a fan gradient needs the fan output
    if (bwd)
        for (int i = 0; i < n_sonar; ++i)
            if (sonar[i].grad_fan && !sonar[i].fan)
                return fail(OCEANSIM_E_INVALID_ARG, "frame %d: a backward plan reads grad_fan only with the fan output",
                            i);
    hipStream_t st = static_cast<hipStream_t>(stream);

    oceansim_plan *p = new oceansim_plan;
    p->sonar.assign(sonar, sonar + n_sonar);
    p->camera.assign(camera, camera + n_camera);
    p->sp = sonar_params_dev;
    p->n_srows = std::max(1, n_sonar_rows);
    p->refl = refl_dev;
    p->n_mat = n_materials;
    p->wp = water_params_dev;
    p->n_wrows = std::max(1, n_water_rows);
    p->g_refl = grad_refl_dev;
    p->g_sp = grad_sonar_params_dev;
    p->g_wp = grad_water_params_dev;
    p->flags = flags;

    // validation of both directions before anything is allocated
    int rc = OCEANSIM_OK;
    if (n_sonar > 0) {
        rc = plan_sonar(p->sonar.data(), n_sonar, n_sonar_rows, n_materials, false, p->sf, nullptr);
        if (!rc && bwd) rc = plan_sonar(p->sonar.data(), n_sonar, n_sonar_rows, n_materials, true, p->sb, nullptr);
    }
    p->fused = n_sonar > 0 && n_camera > 0;
    p->pair = bwd && n_sonar > 0 && pair_backward_ok(p->sonar.data(), n_sonar, n_materials);
    if (!rc && n_camera > 0) {
        rc = plan_uw(p->camera.data(), n_camera, n_water_rows, false, p->uf, true);
        if (!rc && bwd) rc = plan_uw(p->camera.data(), n_camera, n_water_rows, true, p->ub, true);
    }
    if (rc) {
        delete p;
        return rc;
    }
    // the binned sums a range-normalised frame's backward reads, where the
    // caller keeps none
    if (bwd) {
        size_t sp_bytes = 0;
        std::vector<size_t> sp_off(n_sonar, (size_t)-1);
        for (int i = 0; i < n_sonar; ++i)
            if (p->sonar[i].range_norm && !p->sonar[i].saved_p) {
                sp_off[i] = sp_bytes;
                sp_bytes += (sizeof(float) * (size_t)p->sonar[i].n_range * p->sonar[i].n_azimuth + kWsAlign - 1) /
                            kWsAlign * kWsAlign;
            }
        if (sp_bytes) {
            hipError_t se = hipMalloc(&p->savedp_mem, sp_bytes);
            if (se != hipSuccess) {
                free_plan(p);
                return hip_fail(se, "plan binned-sum memory");
            }
            for (int i = 0; i < n_sonar; ++i)
                if (sp_off[i] != (size_t)-1) p->sonar[i].saved_p = reinterpret_cast<float *>(p->savedp_mem + sp_off[i]);
        }
    }
    // saved fan stencils for frames rendered with a fan whose gradient is read
    size_t st_bytes = 0;
    std::vector<size_t> st_off(n_sonar, (size_t)-1);
    if (bwd)
        for (int i = 0; i < n_sonar; ++i) {
            auto &f = p->sonar[i];
            if (f.fan && f.grad_fan && !f.fan_stencil) {
                st_off[i] = st_bytes;
                st_bytes += (oceansim_fan_stencil_size(f.fan_h, f.fan_w) + kWsAlign - 1) / kWsAlign * kWsAlign;
            }
        }
    hipError_t e = hipSuccess;
    if (st_bytes) {
        e = hipMalloc(&p->stencil_mem, st_bytes);
        if (e != hipSuccess) {
            free_plan(p);
            return hip_fail(e, "plan stencil memory");
        }
        for (int i = 0; i < n_sonar; ++i)
            if (st_off[i] != (size_t)-1) p->sonar[i].fan_stencil = p->stencil_mem + st_off[i];
    }
    if (bwd && n_sonar > 0) {
        rc = build_fan_transposes(p, st);
        // the stencils were needed for the operators only
        for (int i = 0; i < n_sonar; ++i)
            if (st_off[i] != (size_t)-1) p->sonar[i].fan_stencil = nullptr;
        if (p->stencil_mem) {
            (void)hipFree(p->stencil_mem);
            p->stencil_mem = nullptr;
        }
        if (rc) {
            free_plan(p);
            return rc;
        }
    }
    const char *shape_env = getenv("OCEANSIM_PLAN_SHAPE");
    if (shape_env && *shape_env && n_sonar > 0) {
        // a fixed launch shape "tile_bins,chunk" in place of the heuristic or
        // the autotuner
        int tb = 0, ch = 0;
        if (sscanf(shape_env, "%d,%d", &tb, &ch) != 2 || tb < 1 || tb > kMaxFwdTileBins ||
            (ch != 512 && ch != 1024 && ch != 2048 && ch != 4096 && ch != 8192)) {
            free_plan(p);
            return fail(OCEANSIM_E_INVALID_ARG,
                        "OCEANSIM_PLAN_SHAPE must be \"tile_bins,chunk\" with tile_bins in 1..%d and chunk one of "
                        "512, 1024, 2048, 4096, 8192",
                        kMaxFwdTileBins);
        }
        p->tune.fwd_tile_bins = tb;
        p->tune.chunk = ch;
    } else if ((flags & OCEANSIM_PLAN_AUTOTUNE) && n_sonar > 0) {
        rc = autotune(p, st);
        if (rc) {
            free_plan(p);
            return rc;
        }
    }
    // final shapes
    if (n_sonar > 0) {
        rc = plan_sonar(p->sonar.data(), n_sonar, n_sonar_rows, n_materials, false, p->sf, &p->tune, true, p->pair);
        if (!rc && bwd) {
            rc = plan_sonar(p->sonar.data(), n_sonar, n_sonar_rows, n_materials, true, p->sb, &p->tune, true,
                            p->pair);
            attach_fan_transposes(p, p->sb);
        }
        if (rc) {
            free_plan(p);
            return rc;
        }
    }
    auto up = [](size_t v) { return (v + kWsAlign - 1) / kWsAlign * kWsAlign; };
    const size_t b_sf = n_sonar ? up(p->sf.bytes) : 0, b_sb = (n_sonar && bwd) ? up(p->sb.bytes) : 0;
    const size_t b_uf = n_camera ? up(p->uf.bytes) : 0, b_ub = (n_camera && bwd) ? up(p->ub.bytes) : 0;
    e = hipMalloc(&p->mem, std::max<size_t>(b_sf + b_sb + b_uf + b_ub, kWsAlign));
    if (e != hipSuccess) {
        free_plan(p);
        return hip_fail(e, "plan memory");
    }
    p->ws_sf = p->mem;
    p->ws_sb = p->ws_sf + b_sf;
    p->ws_uf = p->ws_sb + b_sb;
    p->ws_ub = p->ws_uf + b_uf;
    if (n_sonar > 0) {
        carve_sonar(p->sf, p->ws_sf, false);
        e = upload_table(p->sf.dev, p->ws_sf, p->sf.off_table, st);
        if (e == hipSuccess && bwd) {
            carve_sonar(p->sb, p->ws_sb, true);
            if (p->pair) link_pairs(p->sb, p->sf);
            e = upload_table(p->sb.dev, p->ws_sb, p->sb.off_table, st);
        }
    }
    if (e == hipSuccess && n_camera > 0) {
        e = upload_table(p->uf.dev, p->ws_uf, p->uf.off_table, st);
        if (e == hipSuccess && bwd) e = upload_table(p->ub.dev, p->ws_ub, p->ub.off_table, st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        free_plan(p);
        return hip_fail(e, "plan tables");
    }
    if (flags & OCEANSIM_PLAN_GRAPH) {
        e = hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking);
        if (e != hipSuccess) {
            free_plan(p);
            return hip_fail(e, "capture stream");
        }
        rc = capture(p, false, &p->g_fwd);
        if (!rc && bwd) rc = capture(p, true, &p->g_bwd);
        if (rc) {
            free_plan(p);
            return rc;
        }
    }
    *plan = p;
    return ok();
}

int oceansim_plan_forward(oceansim_plan *p, void *stream) {
    if (!p) return fail(OCEANSIM_E_INVALID_ARG, "plan is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = p->g_fwd ? hipGraphLaunch(p->g_fwd, st) : launch_forward(p, st);
    return e == hipSuccess ? ok() : hip_fail(e, "plan forward");
}

int oceansim_plan_backward(oceansim_plan *p, void *stream) {
    if (!p) return fail(OCEANSIM_E_INVALID_ARG, "plan is NULL");
    if (!(p->flags & OCEANSIM_PLAN_BACKWARD))
        return fail(OCEANSIM_E_INVALID_ARG, "plan was created without OCEANSIM_PLAN_BACKWARD");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = p->g_bwd ? hipGraphLaunch(p->g_bwd, st) : launch_backward(p, st);
    return e == hipSuccess ? ok() : hip_fail(e, "plan backward");
}

int oceansim_plan_shape(const oceansim_plan *p, int32_t shape[4]) {
    if (!p || !shape) return fail(OCEANSIM_E_INVALID_ARG, "NULL argument");
    shape[0] = p->sf.grid.max_tile_bins;
    shape[1] = p->sf.grid.chunk;
    // operator rows per thread times the workgroup's threads (a workgroup takes
    // kFantRows times them: each wave's first lane has no rows of its own)
    shape[2] = (p->flags & OCEANSIM_PLAN_BACKWARD) && !p->sonar.empty() ? kBlock * p->sb.grid.fant_bpt : 0;
    shape[3] = p->g_fwd ? 1 : 0;
    return ok();
}

int oceansim_plan_destroy(oceansim_plan *p) {
    free_plan(p);
    return ok();
}

}  // extern "C"
