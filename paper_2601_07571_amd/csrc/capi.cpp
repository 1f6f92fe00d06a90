// capi.cpp -- the C ABI (include/gazemap.h): argument checks, scene upload,
// device scratch management and the launch sequence of each entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "gazemap.h"
#include "gm_host.h"
#include "gm_internal.h"

using namespace gm;

namespace gm {

namespace {
thread_local std::string g_error;
}  // namespace

gm_status fail(gm_status st, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_error = buf;
    return st;
}

void clear_error() { g_error.clear(); }
const char* last_error() { return g_error.c_str(); }

}  // namespace gm

namespace gm {

gm_status check_device(const gm_scene* sc)
{
    int dev = -1;
    GM_HIP(hipGetDevice(&dev));
    if (dev != sc->device)
        return fail(GM_ERR_INVALID_ARGUMENT, "scene lives on device %d but device %d is current", sc->device, dev);
    return GM_OK;
}

namespace {
__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
}  // namespace

// fills by a kernel (also safe inside captured graphs)
void fill_u32(void* p, int64_t n, uint32_t v, hipStream_t s)
{
    if (n > 0) k_fill_u32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(static_cast<uint32_t*>(p), n, v);
}

void zero(void* p, size_t bytes, hipStream_t s) { fill_u32(p, (int64_t)((bytes + 3) / 4), 0u, s); }

}  // namespace gm

namespace {

// Boxes per closed mesh: kSolidScene over the meshes that have any, within kSolidLeast and
// kSolidMost, and at most one for every kSolidPer triangles of the mesh or its share of one for
// every kSolidShare triangles of the scene, whichever is more (so their tree stays a thousandth of
// the scene's).  More boxes settle more occluded pairs but each packet walks their tree.  Map time
// at 0 / 1 / 4 / 10 / 16 / 48 boxes a mesh: three objects and a terrain, 2M samples x 6,000
// fixations, 25.6 / 25.3 / 24.9 / 25.2 / 25.2 / 26.0 ms; 25 spheres of 20,000 triangles, 400,003 x
// 12,000, 18.2 / 14.8 / 14.1 / 14.3 / 14.6 / 16.2 ms.
// A mesh of fewer than kSolidPer triangles is so shallow a tree that walking its boxes costs as
// much as the descents they save.  150,000 samples x 1,500 fixations, 144 spheres of 320 / 720 /
// 1,280 / 5,120 triangles, 0.35 of their spacing wide: 1.00 / 1.24 / 1.43 / 2.12 ms with one box
// each, 0.94 / 1.20 / 1.41 / 2.21 without; 0.7 wide: 1.16 / 1.35 / 1.57 / 2.31 and 1.17 / 1.43 / 1.72
// / 2.74; 2,304 of 180 triangles: 2.52 and 2.81 with, 2.22 and 2.69 without.  But a coarse mesh
// among fine ones is worth its boxes: the objects (one is a cube) take 1 to 5 % longer when the
// cube has none.
// Self occlusion has none: what a point's own boxes could settle, the back-face rule has settled
// (the triangle tests stay the same); 100 spheres of 8,000 triangles 10.24 ms with, 9.87 without.
constexpr int kSolidLeast = 4;
constexpr int kSolidMost = 12;
constexpr int kSolidScene = 128;
constexpr int64_t kSolidPer = 1000;
constexpr int64_t kSolidShare = 20000;

// a1 + a2 on the device, once per scene: areas, weights, their scan and the per-mesh
// totals and scale exponents, the last two read back to the host (blocking, once).
gm_status ensure_weights(gm_scene* sc, hipStream_t s)
{
    if (sc->weights_ready) return GM_OK;
    const int64_t T = sc->T;
    const int32_t M = sc->M;
    GM_HIP(sc->area.ensure(sizeof(double) * T));
    GM_HIP(sc->W.ensure(8 * T));
    GM_HIP(sc->C.ensure(8 * T));
    GM_HIP(sc->max_bits.ensure(8 * M));
    GM_HIP(sc->S.ensure(4 * M));
    GM_HIP(sc->scan_tmp.ensure(scan_tmp_bytes(T)));
    GM_HIP(sc->counts.ensure(8 * M));
    GM_HIP(sc->offsets.ensure(8 * (M + 1)));
    GM_HIP(sc->mesh_total.ensure(8 * M));
    GM_HIP(sc->tbegin(kStageSample, s));
    zero(sc->max_bits.p, 8 * (size_t)M, s);
    launch_tri_area(sc->V.as<float>(), sc->I.as<int32_t>(), sc->tri_mesh.as<int32_t>(), T, sc->area.as<double>(),
                    sc->max_bits.as<unsigned long long>(), s);
    launch_mesh_scale(sc->max_bits.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(), M, sc->S.as<int32_t>(), s);
    launch_tri_weight(sc->area.as<double>(), sc->tri_mesh.as<int32_t>(), sc->S.as<int32_t>(), T,
                      sc->W.as<unsigned long long>(), s);
    launch_inclusive_scan_u64(sc->W.as<unsigned long long>(), sc->C.as<unsigned long long>(), T, sc->scan_tmp.p, s);
    // the totals (the counts of density 0 are unused)
    launch_mesh_counts(sc->C.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(), sc->S.as<int32_t>(), M, 0.0,
                       sc->counts.as<int64_t>(), sc->offsets.as<int64_t>(), sc->mesh_total.as<unsigned long long>(), s);
    GM_HIP(hipGetLastError());
    GM_HIP(sc->tend(kStageSample, s));
    sc->mesh_total_h.assign((size_t)M, 0ull);
    sc->S_h.assign((size_t)M, 0);
    GM_HIP(hipMemcpyAsync(sc->mesh_total_h.data(), sc->mesh_total.p, 8 * (size_t)M, hipMemcpyDeviceToHost, s));
    GM_HIP(hipMemcpyAsync(sc->S_h.data(), sc->S.p, 4 * (size_t)M, hipMemcpyDeviceToHost, s));
    GM_HIP(hipStreamSynchronize(s));
    // the guide table: per mesh about one bucket per triangle (a power of two >= its
    // triangle count, at most 2^24), each 2^gsh targets wide, plus a closing entry
    std::vector<int64_t> goff((size_t)M + 1, 0);
    std::vector<int32_t> gsh((size_t)M, 0);
    for (int32_t m = 0; m < M; ++m) {
        const int64_t nt = sc->tri_off[(size_t)m + 1] - sc->tri_off[(size_t)m];
        int g = 0;
        while (g < 24 && ((int64_t)1 << g) < nt) ++g;
        const unsigned long long tot = sc->mesh_total_h[(size_t)m];
        int len = 0;  // bit length of tot - 1: targets lie in [0, tot)
        for (unsigned long long v = tot > 1 ? tot - 1 : 0; v; v >>= 1) ++len;
        gsh[(size_t)m] = std::max(0, len - g);
        const int64_t buckets = tot > 0 ? (int64_t)((tot - 1) >> gsh[(size_t)m]) + 1 : 1;
        goff[(size_t)m + 1] = goff[(size_t)m] + buckets + 1;
    }
    GM_HIP(sc->goff.ensure(8 * ((size_t)M + 1)));
    GM_HIP(sc->gsh.ensure(4 * (size_t)M));
    GM_HIP(sc->guide.ensure(4 * (size_t)goff[(size_t)M]));
    GM_HIP(hipMemcpyAsync(sc->goff.p, goff.data(), 8 * ((size_t)M + 1), hipMemcpyHostToDevice, s));
    GM_HIP(hipMemcpyAsync(sc->gsh.p, gsh.data(), 4 * (size_t)M, hipMemcpyHostToDevice, s));
    launch_sample_guide(sc->C.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(), sc->goff.as<int64_t>(),
                        sc->gsh.as<int32_t>(), M, goff[(size_t)M], sc->guide.as<int32_t>(), s);
    GM_HIP(hipGetLastError());
    GM_HIP(hipStreamSynchronize(s));  // the host vectors above go out of scope
    sc->weights_ready = true;
    return GM_OK;
}

// Per-mesh counts round(k * W_m 2^-S_m), evaluated on the host exactly as k_mesh_counts
// evaluates them on the device (the same FP64 operations in the same order).
gm_status sample_counts(gm_scene* sc, double k, hipStream_t s, std::vector<int64_t>& counts)
{
    if (!(k > 0.0) || !std::isfinite(k)) return fail(GM_ERR_INVALID_ARGUMENT, "samples_per_m2 must be finite and > 0");
    gm_status st = ensure_weights(sc, s);
    if (st != GM_OK) return st;
    counts.assign((size_t)sc->M, 0);
    for (int32_t m = 0; m < sc->M; ++m) {
        const unsigned long long tot = sc->mesh_total_h[(size_t)m];
        const double area = std::ldexp((double)tot, -sc->S_h[(size_t)m]);
        counts[(size_t)m] = tot ? (int64_t)std::floor(area * k + 0.5) : 0;
    }
    return GM_OK;
}

// Lattice sampler counts: areas (a1, cached), Eq. (4) resolutions and Eq. (1) counts
// per triangle, their inclusive scan in sc->lat_C, per-mesh totals (blocking).
gm_status lattice_counts(gm_scene* sc, double k, hipStream_t s, std::vector<int64_t>& counts)
{
    if (!(k > 0.0) || !(k <= 1e12)) return fail(GM_ERR_INVALID_ARGUMENT, "samples_per_m2 must be in (0, 1e12]");
    gm_status st = ensure_weights(sc, s);
    if (st != GM_OK) return st;
    const int64_t T = sc->T;
    const int32_t M = sc->M;
    GM_HIP(sc->lat_C.ensure(8 * T));
    // the totals go straight to host memory (with the counts formed inside the scan, a call of
    // 1,000,003 points on 200,000 triangles 55.4 -> 46.1 us)
    if (!sc->lat_totals) GM_HIP(hipHostMalloc(reinterpret_cast<void**>(&sc->lat_totals), 8 * (size_t)M, hipHostMallocMapped));
    GM_HIP(sc->tbegin(kStageSample, s));
    launch_lattice_scan(sc->area.as<double>(), k, sc->lat_C.as<unsigned long long>(), T, sc->scan_tmp.p, s);
    launch_lattice_mesh_counts(sc->lat_C.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(), M, sc->lat_totals, s);
    GM_HIP(hipGetLastError());
    GM_HIP(sc->tend(kStageSample, s));
    GM_HIP(hipStreamSynchronize(s));
    counts.assign(sc->lat_totals, sc->lat_totals + M);
    return GM_OK;
}

// mesh m's entry of DensityLaunch::solid_mbox under its present flag
void solid_mbox_entry(const gm_scene* sc, int32_t m, float (&e)[8])
{
    for (int c = 0; c < 8; ++c) {
        const float open = (c & 3) == 3 ? 0.0f : (c < 4 ? -INFINITY : INFINITY);
        e[c] = sc->closed[(size_t)m] ? sc->mbox[(size_t)8 * m + c] : open;
    }
}

bool finite3(const float* p) { return std::isfinite(p[0]) && std::isfinite(p[1]) && std::isfinite(p[2]); }

}  // namespace

namespace gm {

gm_status check_density_args(const gm_scene* sc, const float* pos, int64_t n, const gm_fixations* fix,
                             double theta_deg, uint32_t flags)
{
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    if (!fix) return fail(GM_ERR_INVALID_ARGUMENT, "fixations is NULL");
    if (n < 0 || n >= ((int64_t)1 << 31)) return fail(GM_ERR_INVALID_ARGUMENT, "n must be in [0, 2^31)");
    if (n > 0 && !pos) return fail(GM_ERR_INVALID_ARGUMENT, "pos is NULL");
    if (fix->n < 0) return fail(GM_ERR_INVALID_ARGUMENT, "fixation count < 0");
    if (fix->n > 0 && (!fix->eye || !fix->gaze || !fix->duration))
        return fail(GM_ERR_INVALID_ARGUMENT, "fixation arrays must not be NULL");
    if (!(theta_deg > 0.0 && theta_deg < 45.0)) return fail(GM_ERR_INVALID_ARGUMENT, "theta_deg must be in (0, 45)");
    const uint32_t mode = flags & GM_OCC_MASK;
    if (mode > GM_OCC_FULL || (flags & ~GM_OCC_MASK)) return fail(GM_ERR_INVALID_ARGUMENT, "unknown flags 0x%x", flags);
    return check_device(sc);
}

gm_status density_reserve(DensityWork& w, int64_t n, int32_t F)
{
    // spatial buckets: about one sample per bucket of the scene's box, at most 2^21; launches
    // of more than 2^20 points take 2^24, of more than 2^23 points 2^27.  Samples lie on
    // surfaces, so an occupied bucket of the coarser grid holds about a hundred of them in no
    // particular order (the scatter's atomic cursor) and a wave's 64 segments would start
    // anywhere in it: the finer grids cut node visits by 6 % on the paper-shaped map (2M
    // points) and by 10 % on the scale-up map (20M points).
    int bits = 1;
    while (bits < 7 && ((int64_t)1 << (3 * bits)) < n) ++bits;
    if (n > ((int64_t)1 << 20)) bits = 8;
    if (n > ((int64_t)1 << 23)) bits = 9;
    w.bits = bits;
    w.buckets = (int64_t)1 << (3 * bits);
    const int64_t nn = std::max<int64_t>(n, 1);
    GM_HIP(w.fix.ensure(sizeof(FixRec) * (size_t)std::max(F, 1)));
    GM_HIP(w.fx_shift.ensure(16));
    GM_HIP(w.key.ensure(4 * nn));
    GM_HIP(w.hist.ensure(4 * w.buckets));
    GM_HIP(w.cursor.ensure(4 * w.buckets));
    GM_HIP(w.scan_tmp.ensure(scan_tmp_bytes(w.buckets)));
    GM_HIP(w.spos.ensure(16 * nn));
    GM_HIP(w.smesh.ensure(4 * nn));
    GM_HIP(w.inv.ensure(4 * nn));
    GM_HIP(w.acc.ensure(8 * nn));
    GM_HIP(w.max_acc.ensure(8));
    GM_HIP(w.stats.ensure(8 * kDensityStats));
    return GM_OK;
}

void density_sort(gm_scene* sc, DensityWork& w, const float* pos, const int32_t* tri, const int32_t* mesh,
                  int64_t n, hipStream_t s, int64_t off, bool zeroed)
{
    if (n <= 0) return;
    if (!zeroed) {
        zero(w.acc.as<unsigned long long>() + off, 8 * (size_t)n, s);
        zero(w.hist.p, 4 * (size_t)w.buckets, s);
    }
    float lo[3];
    float ext = 0.0f;
    for (int c = 0; c < 3; ++c) {
        lo[c] = sc->bvh.lo[c];
        ext = std::max(ext, sc->bvh.hi[c] - sc->bvh.lo[c]);
    }
    const int cells = 1 << w.bits;
    const float inv_cell = ext > 0.0f ? (float)cells / ext : 1.0f;
    launch_morton(pos, tri, mesh, sc->tri_mesh.as<int32_t>(), n, lo, inv_cell, w.bits, w.key.as<uint32_t>(),
                  w.hist.as<uint32_t>(), w.inv.as<int32_t>() + off, s);
    launch_exclusive_scan_u32(w.hist.as<uint32_t>(), w.cursor.as<uint32_t>(), w.buckets, w.scan_tmp.p, s);
    launch_scatter(pos, tri, mesh, sc->tri_mesh.as<int32_t>(), sc->T, n, w.key.as<uint32_t>(),
                   w.cursor.as<uint32_t>(), w.spos.as<float4>() + off, w.smesh.as<int32_t>() + off,
                   w.inv.as<int32_t>() + off, (int32_t)off, s);
}

int32_t auto_fix_per_chunk(const gm_scene* sc, int64_t tiles, int32_t F, double tile_fixations, uint32_t mode)
{
    // The cost of a (tile, chunk) item varies a lot (how many of its fixations see the tile),
    // so a large grid holds many small items: at least ~512k of them and at most 1024
    // fixations each, but chunks of no fewer than 128 fixations (512 without a visibility
    // test, where an item costs little beyond its fixed part: its samples, the staging and
    // the tile cone test of every fixation, the flush; the paper-shaped gate takes 2.43 ms at
    // 128, 1.71 ms at 512, 1.74 ms at 1024).
    // A launch of few tiles must cut its fixations finer to fill 256 CUs: the best chunk
    // measured grows like the square root of the launch's (tile, fixation) pairs, which
    // balances the items' fixed parts against the tail of the last ones.  Full occlusion,
    // map time at chunks of 4 / 8 / 16 / 32 / 64 / 128 fixations: 25 tiles x 100 fixations
    // 100 / 110 / 132 / 153 / 196 / 252 us; 47 x 2,501 1.17 / 1.11 / 1.17 / 1.22 / 1.43 /
    // 1.97 ms; 196 x 1,000 1.32 / 1.25 / 1.34 / 1.68 / 2.05 / 3.25 ms; 1,173 x 3,000 6.8 /
    // 5.2 / 4.2 / 3.7 / 3.7 / 4.4 ms; 1,563 x 12,000 38.9 / 29.7 / 24.2 / 21.1 / 19.7 / 19.4
    // ms.  The smallest, at 1 / 2 / 4 / 8: 25 x 100 82 / 80 / 88 / 91 us; 47 x 100 on a fine mesh
    // (60,000 triangles) 242 / 275 / 364 / 382; 59 x 100 in a room 250 / 256 / 316 / 379; 196 x
    // 100 340 / 352 / 417 / 421.  Without: 40 x 1,000 157 / 110 / 82 / 78 / 92 / 132 us; 391 x
    // 3,000 2.17 / 1.48 / 0.93 / 0.56 / 0.33 / 0.27 ms (0.32 at 256, 0.46 at 512).
    // Those with occlusion are of scenes of 60,000 triangles and more but for the 25 tiles; in a
    // shallow tree or a flat scene a pair costs little more than without, and the line lies between the two.  235
    // tiles x 1,000 at 12 / 16 / 32 / 64 / 128: a cube (12 triangles) 305 / 242 / 182 / 174 / 179 us,
    // spheres of 320 triangles 320 / 277 / 267 / 270 / 322, of 5,120 467 / 438 / 472 / 456 / 560, of
    // 20,480 693 / 665 / 731 / 754 / 870; 1,172 x 1,000 at 27 / 64 / 128: a cube 638 / 520 / 481.
    const bool occ = mode != GM_OCC_NONE;
    const double root = std::sqrt(std::max(1.0, tile_fixations));
    const double parts = occ ? std::min(40.0, 8.0 + 3.5 * sc->walk_levels) : 8.0;
    const int64_t min_chunk = std::min<int64_t>(occ ? 128 : 512, std::max<int64_t>(occ ? 1 : 16, (int64_t)(root / parts)));
    const int64_t max_chunks = std::max<int64_t>(1, (F + min_chunk - 1) / min_chunk);
    const int64_t want = std::max<int64_t>((524288 + tiles - 1) / tiles, (F + 1023) / 1024);
    // the grid is tiles x chunks: chunks <= 65535 (grid y) and tiles x chunks < 2^31
    const int64_t cap = std::min<int64_t>(65535, std::max<int64_t>(1, INT32_MAX / tiles));
    const int64_t chunks = std::min<int64_t>(std::min(max_chunks, cap), std::max<int64_t>(1, want));
    return (int32_t)std::max<int64_t>(1, (F + chunks - 1) / chunks);
}

void density_args(const gm_scene* sc, const DensityWork& w, int64_t n, int32_t F, double sigma, uint32_t mode,
                  int spl, int32_t fix_per_chunk, DensityLaunch& a)
{
    a.spos = w.spos.as<float4>();
    a.smesh = w.smesh.as<int32_t>();
    a.n = n;
    a.fix = w.fix.as<FixRec>();
    a.F = F;
    a.nodes = sc->nodes.as<BvhNode>();
    a.node_stride = (int64_t)sc->bvh.nodes.size();
    a.tris = sc->tris.as<BvhTri>();
    a.tri_stride = (int64_t)sc->bvh.tris.size();
    a.occ_mode = (int32_t)mode;
    a.cone2 = (float)(16.0 * sigma * sigma);
    a.kexp = (float)(1.0 / (2.0 * sigma * sigma * std::log(2.0)));
    a.fx_shift = w.fx_shift.as<int32_t>();
    a.acc = w.acc.as<unsigned long long>();
    a.stats = w.stats.as<unsigned long long>();
    a.spl = spl;
    const int64_t tiles = std::max<int64_t>(1, (n + 256 * spl - 1) / (256 * spl));
    if (fix_per_chunk <= 0) fix_per_chunk = auto_fix_per_chunk(sc, tiles, F, (double)tiles * (double)F, mode);
    a.fix_per_chunk = fix_per_chunk;
    a.n_chunks = F > 0 ? (int32_t)((F + fix_per_chunk - 1) / fix_per_chunk) : 0;
    a.F_live = nullptr;
    if (w.backface && mode != GM_OCC_NONE) {
        a.bface = w.bface.as<float4>();
        a.bcand = w.bcand.as<int32_t>();
        a.mbox = sc->mbox_d.as<float4>();
        a.bf_tris = sc->tris.as<BvhTri>() + 2 * sc->bvh.tris.size();
        a.bf_L2max = backface_l2max(sc);
        if (w.horizon) {
            a.hz = w.hz.as<float>();
            a.hz_reach = sc->hz_reach;
        }
        if (mode == GM_OCC_FULL && sc->solid_n > 0 && sc->any_closed()) {
            a.solid = sc->solid.as<BvhNode>();
            a.solid_stride = sc->solid_n;
            a.solid_mbox = sc->solid_mbox_d.as<float4>();
        }
    }
}

float backface_l2max(const gm_scene* sc)
{
    // the rule's longest segment: its last kEpsV stretch stays 1e-3 inside rmax
    const double lmax = (double)sc->bf_rmax / kEpsV * (1.0 - 1e-3);
    return (float)(lmax * lmax);
}

gm_status density_backface(gm_scene* sc, DensityWork& w, int64_t n, uint32_t mode, bool normals, hipStream_t s,
                           int64_t off)
{
    w.backface = false;
    if (mode == GM_OCC_NONE || (!sc->any_closed() && !normals) || n <= 0) return GM_OK;
    GM_HIP(w.bface.ensure(16 * (size_t)(off + n)));
    GM_HIP(w.bcand.ensure(backface_list_bytes(sc, off + n)));
    launch_backface_prep(w.spos.as<float4>() + off, w.smesh.as<int32_t>() + off, n, sc->V.as<float>(),
                         sc->I.as<int32_t>(), sc->closed_d.as<uint8_t>(), sc->M, sc->nodes.as<BvhNode>(),
                         sc->tris.as<BvhTri>() + 2 * sc->bvh.tris.size(), sc->bf_rmax, sc->solid_near,
                         w.bface.as<float4>() + off,
                         w.bcand.as<int32_t>() + kBfCand * off, s);
    GM_HIP(hipGetLastError());
    w.backface = true;
    return GM_OK;
}

bool stream_captures(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

size_t backface_list_bytes(const gm_scene* sc, int64_t n)
{
    for (uint8_t c : sc->closed_topology)
        if (c) return 4 * (size_t)kBfCand * (size_t)n;
    return 0;
}

bool horizon_room(const gm_scene* sc, DensityWork& w, int64_t n, hipStream_t s)
{
    const size_t bf = 16 * (size_t)n, bc = backface_list_bytes(sc, n), hz = 4 * (size_t)n;
    if (w.bface.bytes >= bf && w.bcand.bytes >= bc && w.hz.bytes >= hz) return true;
    if (!stream_captures(s) && w.bface.ensure(bf) == hipSuccess && w.bcand.ensure(bc) == hipSuccess &&
        w.hz.ensure(hz) == hipSuccess)
        return true;
    (void)hipGetLastError();
    return false;
}

bool horizon_pays(const gm_scene* sc, int64_t n, int64_t F, double sigma, uint32_t mode)
{
    // A point's walked pairs grow with F sigma^2 (its share of the cones), its horizon costs
    // one walk of its neighbourhood.  Map time without / with: three objects and a terrain,
    // 300,021 points, 2,500 fixations at 1 degree (F sigma^2 = 0.76) 3.68 / 3.97 ms; a sphere,
    // 12,007 points, 2,501 at 1.2 degrees (1.1) 1.13 / 1.01; 2M points, 6,000 at 1 degree (1.8)
    // 34.0 / 29.5; 25 spheres, 400,003 points, 12,000 (3.7) 15.4 / 14.3.
    // Few points, a wave each, have theirs for 40 to 150 us: a sphere, 30,000 points, 300 / 600 /
    // 1,200 / 2,400 fixations at 1 degree (0.09 / 0.18 / 0.37 / 0.73) 509 / 551 / 784 / 1,244 us
    // without, 469 / 543 / 661 / 901 with; 25 spheres 520 / 714 / 832 / 1,122 and 568 / 593 /
    // 735 / 1,033; 120,000 points at 0.37 / 0.73 1,249 / 1,909 and 1,420 / 1,989.
    // Those are scenes of 60,000 triangles and more.  60,000 points at 0.3 / 3.0: spheres of 20,480
    // triangles 693 / 3,987 without, 604 / 2,508 with; 5,120 467 / 2,559 and 493 / 1,754; 1,280 359 /
    // 1,890 and 452 / 1,389; 80 317 / 1,375 and 385 / 1,108; a cube 305 / 1,108 and 384 / 1,208; a flat
    // plate of 2,048 289 / 1,317 and 390 / 1,542.  The fewest triangles and flat scenes never pay:
    // a segment leaves their boxes at once.  Flat is up to 5e-5 of the scene's extent (walk_levels):
    // a plate of 20,000 triangles with waves 2e-5 / 2e-4 / 6e-4 / 2e-3 of it high, at 3.0, 1.25 / 2.97 /
    // 4.55 / 6.11 ms without, 1.47 / 2.59 / 3.43 / 4.53 with.
    if (mode == GM_OCC_NONE || sc->walk_levels < 2.0) return false;
    return (double)F * sigma * sigma >= (n <= 65536 && sc->T >= 8192 ? 0.2 : 1.0);
}

gm_status density_horizon(gm_scene* sc, DensityWork& w, int64_t n, hipStream_t s)
{
    w.horizon = false;
    if (!w.backface || n <= 0) return GM_OK;
    GM_HIP(w.hz.ensure(4 * (size_t)n));
    launch_horizon(w.spos.as<float4>(), w.bface.as<float4>(), n, sc->nodes.as<BvhNode>(),
                   sc->tris.as<BvhTri>() + 2 * sc->bvh.tris.size(), sc->hz_reach, w.hz.as<float>(), s);
    GM_HIP(hipGetLastError());
    w.horizon = true;
    return GM_OK;
}

gm_status density_prep(gm_scene* sc, DensityWork& w, const float* pos, const int32_t* tri, const int32_t* mesh,
                       int64_t n, const gm_fixations* fix, double theta_deg, uint32_t mode, int spl,
                       int32_t fix_per_chunk, DensityLaunch& a, hipStream_t s)
{
    const int32_t F = fix->n;
    const double sigma = std::tan(theta_deg * M_PI / 180.0);
    MapBegin begin;
    begin.eye = fix->eye;
    begin.gaze = fix->gaze;
    begin.dur = fix->duration;
    begin.F = F;
    begin.rec = w.fix.as<FixRec>();
    begin.fx_shift = w.fx_shift.as<int32_t>();
    begin.acc = w.acc.as<unsigned long long>();
    begin.stats = w.stats.as<unsigned long long>();
    begin.max_acc = w.max_acc.as<unsigned long long>();
    begin.n = n;
    begin.hist = w.hist.as<uint32_t>();
    begin.buckets = w.buckets;
    launch_map_begin(begin, sigma, kGateWiden, s);
    density_sort(sc, w, pos, tri, mesh, n, s, 0, true);
    const bool horizon = n > 0 && horizon_pays(sc, n, F, sigma, mode) && horizon_room(sc, w, n, s);
    w.horizon = false;
    gm_status st = density_backface(sc, w, n, mode, horizon, s);
    if (st == GM_OK && horizon) st = density_horizon(sc, w, n, s);
    if (st != GM_OK) return st;
    density_args(sc, w, n, F, sigma, mode, spl, fix_per_chunk, a);
    GM_HIP(hipGetLastError());
    return GM_OK;
}

gm_status density_finalize(DensityWork& w, int64_t n, float* density, float* density_norm, float* max_out,
                           hipStream_t s)
{
    launch_finalize(w.acc.as<unsigned long long>(), w.inv.as<int32_t>(), n, w.fx_shift.as<int32_t>(),
                    w.max_acc.as<unsigned long long>(), density, density_norm, max_out, s);
    GM_HIP(hipGetLastError());
    return GM_OK;
}

}  // namespace gm

extern "C" {

const char* gm_last_error(void) { return gm::last_error(); }

int32_t gm_version(void) { return (1 << 16) | 0; }

gm_status gm_scene_create(const gm_mesh* meshes, int32_t n_meshes, gm_scene** out)
{
    gm::clear_error();
    if (!out) return fail(GM_ERR_INVALID_ARGUMENT, "out is NULL");
    *out = nullptr;
    if (!meshes || n_meshes < 1 || n_meshes > 4096)
        return fail(GM_ERR_INVALID_ARGUMENT, "n_meshes must be in [1, 4096] (got %d)", n_meshes);
    int64_t T = 0, NV = 0;
    for (int32_t m = 0; m < n_meshes; ++m) {
        const gm_mesh& g = meshes[m];
        if (!g.vertices || !g.indices || g.n_vertices < 3 || g.n_triangles < 1)
            return fail(GM_ERR_INVALID_ARGUMENT, "mesh %d: needs >= 3 vertices and >= 1 triangle", m);
        for (int64_t v = 0; v < g.n_vertices; ++v)
            if (!finite3(g.vertices + 3 * v)) return fail(GM_ERR_INVALID_ARGUMENT, "mesh %d: vertex %lld not finite", m, (long long)v);
        for (int64_t t = 0; t < 3 * (int64_t)g.n_triangles; ++t)
            if (g.indices[t] < 0 || g.indices[t] >= g.n_vertices)
                return fail(GM_ERR_INVALID_ARGUMENT, "mesh %d: index %d out of range", m, g.indices[t]);
        T += g.n_triangles;
        NV += g.n_vertices;
    }
    if (T >= (int64_t)1 << 31) return fail(GM_ERR_INVALID_ARGUMENT, "more than 2^31 - 1 triangles");
    gm_scene* sc = new (std::nothrow) gm_scene();
    if (!sc) return fail(GM_ERR_OUT_OF_MEMORY, "host allocation failed");
    if (const char* e = std::getenv("GM_FIX_PER_CHUNK")) sc->fix_per_chunk = std::max(0, std::atoi(e));
    if (const char* e = std::getenv("GM_SAMPLES_PER_LANE")) {
        const int v = std::atoi(e);
        if (v == 1 || v == 2 || v == 4) sc->spl = v;
    }
    hipError_t he = hipGetDevice(&sc->device);
    if (he != hipSuccess) {
        delete sc;
        return fail(GM_ERR_DEVICE, "hipGetDevice: %s", hipGetErrorString(he));
    }
    sc->M = n_meshes;
    sc->T = T;
    sc->NV = NV;
    std::vector<float> V((size_t)NV * 3);
    std::vector<int32_t> I((size_t)T * 3), tm((size_t)T);
    sc->tri_off.assign((size_t)n_meshes + 1, 0);
    int64_t vb = 0, tb = 0;
    for (int32_t m = 0; m < n_meshes; ++m) {
        const gm_mesh& g = meshes[m];
        std::memcpy(V.data() + 3 * vb, g.vertices, sizeof(float) * 3 * (size_t)g.n_vertices);
        for (int64_t t = 0; t < g.n_triangles; ++t) {
            for (int k = 0; k < 3; ++k) I[(size_t)(3 * (tb + t) + k)] = (int32_t)(g.indices[3 * t + k] + vb);
            tm[(size_t)(tb + t)] = m;
        }
        sc->tri_off[(size_t)m] = tb;
        vb += g.n_vertices;
        tb += g.n_triangles;
    }
    sc->tri_off[(size_t)n_meshes] = tb;
    int leaf_max = kLeafMax;
    if (const char* e = std::getenv("GM_BVH_LEAF")) {
        const int v = std::atoi(e);
        if (v >= 1 && v <= kLeafMax) leaf_max = v;
    }
    build_bvh(V.data(), I.data(), tm.data(), T, sc->bvh, leaf_max);
    // meshes that bound a solid, their boxes, and the back-face rule's neighbour radius:
    // kEpsV of twice the scene's diagonal plus 4 m (segments up to that length, eyes within
    // a few metres of the scene, use the rule)
    sc->closed.assign((size_t)n_meshes, 0);
    std::vector<float> mbox((size_t)8 * n_meshes, 0.0f);
    for (int32_t m = 0; m < n_meshes; ++m) {
        const gm_mesh& g = meshes[m];
        sc->closed[(size_t)m] = mesh_is_closed(g.vertices, g.n_vertices, g.indices, g.n_triangles) ? 1 : 0;
        float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        for (int64_t t = 0; t < 3 * (int64_t)g.n_triangles; ++t)
            for (int c = 0; c < 3; ++c) {
                const float v = g.vertices[3 * (int64_t)g.indices[t] + c];
                lo[c] = std::min(lo[c], v);
                hi[c] = std::max(hi[c], v);
            }
        for (int c = 0; c < 3; ++c) {
            mbox[(size_t)8 * m + c] = lo[c];
            mbox[(size_t)8 * m + 4 + c] = hi[c];
        }
    }
    {
        double sum = 0.0;
        for (const BvhTri& r : sc->bvh.tris) {
            if (r.id < 0) continue;
            for (int c = 0; c < 3; ++c)
                sum += std::max(r.v0[c], std::max(r.v1[c], r.v2[c])) - std::min(r.v0[c], std::min(r.v1[c], r.v2[c]));
        }
        // four mean triangle extents: the map of 2M points x 6,000 fixations takes 33.1 / 31.6 /
        // 31.3 ms at 2 / 4 / 8 (its horizons 1.4 / 2.1 / 3.3 of them), a sphere of 12,007 x 2,501
        // 1.08 / 1.09 / 1.33
        sc->hz_reach = (float)(4.0 * sum / (3.0 * (double)T));
    }
    {
        double least = INFINITY, most = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double e = (double)sc->bvh.hi[a] - sc->bvh.lo[a];
            least = std::min(least, e);
            most = std::max(most, e);
        }
        sc->walk_levels = least <= 5e-5 * most ? 0.0 : std::max(0.0, std::log2((double)T / 16.0));
    }
    sc->closed_topology = sc->closed;
    sc->mbox = mbox;
    std::vector<BvhNode> solid8;
    {
        double scale = 0.0;
        for (int c = 0; c < 3; ++c)
            scale = std::max(scale, std::max(std::fabs((double)sc->bvh.lo[c]), std::fabs((double)sc->bvh.hi[c])));
        int32_t n_closed = 0;
        for (uint8_t f : sc->closed) n_closed += f;
        const int64_t share = T / (kSolidShare * std::max(1, n_closed));
        auto boxes_of = [&](int32_t m) -> int64_t {
            const int64_t t = meshes[m].n_triangles;
            return sc->closed[(size_t)m] ? std::max(share, t / kSolidPer) : 0;
        };
        int32_t n_solid = 0;
        for (int32_t m = 0; m < n_meshes; ++m) n_solid += boxes_of(m) > 0;
        const int64_t most = std::max(kSolidLeast, std::min(kSolidMost, kSolidScene / std::max(1, n_solid)));
        double near = INFINITY;
        std::vector<SolidBox> boxes;
        for (int32_t m = 0; m < n_meshes; ++m)
            near = std::min(near, solid_boxes(meshes[m].vertices, meshes[m].indices, meshes[m].n_triangles, scale,
                                              (int)std::min(most, boxes_of(m)), m, boxes));
        sc->solid_near = (float)(0.5 * near);
        std::vector<BvhNode> nodes;
        build_solid_tree(std::move(boxes), nodes);
        sc->solid_n = (int64_t)nodes.size();
        if (sc->solid_n > 0) octant_node_copies(nodes, solid8);
    }
    std::vector<float> solid_mbox((size_t)8 * n_meshes);
    for (int32_t m = 0; m < n_meshes; ++m) {
        float v[8];
        solid_mbox_entry(sc, m, v);
        std::copy(v, v + 8, solid_mbox.begin() + (size_t)8 * m);
    }
    {
        double d2 = 0.0;
        for (int c = 0; c < 3; ++c) d2 += ((double)sc->bvh.hi[c] - sc->bvh.lo[c]) * ((double)sc->bvh.hi[c] - sc->bvh.lo[c]);
        sc->bf_rmax = (float)(kEpsV * (2.0 * std::sqrt(d2) + 4.0));
    }

    auto up = [&](DevBuf& b, const void* src, size_t bytes) -> hipError_t {
        hipError_t e = b.ensure(bytes);
        if (e != hipSuccess) return e;
        return hipMemcpy(b.p, src, bytes, hipMemcpyHostToDevice);
    };
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = up(sc->V, V.data(), V.size() * 4);
    if (e == hipSuccess) e = up(sc->I, I.data(), I.size() * 4);
    if (e == hipSuccess) e = up(sc->tri_mesh, tm.data(), tm.size() * 4);
    if (e == hipSuccess) e = up(sc->tri_off_d, sc->tri_off.data(), sc->tri_off.size() * 8);
    std::vector<BvhNode> node8;
    octant_node_copies(sc->bvh.nodes, node8);
    if (e == hipSuccess) e = up(sc->nodes, node8.data(), node8.size() * sizeof(BvhNode));
    std::vector<BvhTri> tri3;
    permute_tri_copies(sc->bvh.tris, tri3);
    if (e == hipSuccess) e = up(sc->tris, tri3.data(), tri3.size() * sizeof(BvhTri));
    if (e == hipSuccess) e = up(sc->closed_d, sc->closed.data(), sc->closed.size());
    if (e == hipSuccess) e = up(sc->mbox_d, mbox.data(), mbox.size() * 4);
    if (e == hipSuccess && sc->solid_n > 0) e = up(sc->solid, solid8.data(), solid8.size() * sizeof(BvhNode));
    if (e == hipSuccess) e = up(sc->solid_mbox_d, solid_mbox.data(), solid_mbox.size() * 4);
    if (e != hipSuccess) {
        delete sc;
        return fail(e == hipErrorOutOfMemory ? GM_ERR_OUT_OF_MEMORY : GM_ERR_DEVICE, "scene upload: %s",
                    hipGetErrorString(e));
    }
    *out = sc;
    return GM_OK;
}

gm_status gm_scene_destroy(gm_scene* scene)
{
    gm::clear_error();
    if (scene) {
        (void)hipDeviceSynchronize();
        delete scene;
    }
    return GM_OK;
}

gm_status gm_scene_info(const gm_scene* sc, int64_t* n_triangles, int32_t* n_meshes, int64_t* n_bvh_nodes,
                        int32_t* bvh_depth, float* bbox)
{
    gm::clear_error();
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    if (n_triangles) *n_triangles = sc->T;
    if (n_meshes) *n_meshes = sc->M;
    if (n_bvh_nodes) *n_bvh_nodes = (int64_t)sc->bvh.nodes.size();
    if (bvh_depth) *bvh_depth = sc->bvh.depth;
    if (bbox)
        for (int a = 0; a < 3; ++a) {
            bbox[a] = sc->bvh.lo[a];
            bbox[3 + a] = sc->bvh.hi[a];
        }
    return GM_OK;
}

gm_status gm_scene_mesh_closed(const gm_scene* sc, uint8_t* closed)
{
    gm::clear_error();
    if (!sc || !closed) return fail(GM_ERR_INVALID_ARGUMENT, "scene and closed must not be NULL");
    std::memcpy(closed, sc->closed.data(), sc->closed.size());
    return GM_OK;
}

gm_status gm_scene_set_mesh_closed(gm_scene* sc, int32_t mesh, int32_t closed)
{
    gm::clear_error();
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    if (mesh < 0 || mesh >= sc->M) return fail(GM_ERR_INVALID_ARGUMENT, "mesh %d outside [0, %d)", mesh, sc->M);
    if (closed && !sc->closed_topology[(size_t)mesh])
        return fail(GM_ERR_INVALID_ARGUMENT, "mesh %d does not bound a solid (gm_mesh_closed)", mesh);
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    GM_HIP(hipDeviceSynchronize());
    sc->closed[(size_t)mesh] = closed ? 1 : 0;
    GM_HIP(hipMemcpy(sc->closed_d.as<uint8_t>() + mesh, &sc->closed[(size_t)mesh], 1, hipMemcpyHostToDevice));
    float v[8];
    solid_mbox_entry(sc, mesh, v);
    GM_HIP(hipMemcpy(sc->solid_mbox_d.as<float>() + (size_t)8 * mesh, v, sizeof(v), hipMemcpyHostToDevice));
    return GM_OK;
}

gm_status gm_count_lattice_samples(gm_scene* sc, double k, int64_t* n_per_mesh, void* stream)
{
    gm::clear_error();
    if (!sc || !n_per_mesh) return fail(GM_ERR_INVALID_ARGUMENT, "scene and n_per_mesh must not be NULL");
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    std::vector<int64_t> counts;
    st = lattice_counts(sc, k, (hipStream_t)stream, counts);
    if (st != GM_OK) return st;
    std::memcpy(n_per_mesh, counts.data(), 8 * counts.size());
    return GM_OK;
}

gm_status build_lattice_samples(gm_scene* sc, double k, int32_t* tri, int32_t* mesh, float* bary, float* pos,
                                int64_t capacity, int64_t* n_out, void* stream)
{
    gm::clear_error();
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    if (capacity < 0) return fail(GM_ERR_INVALID_ARGUMENT, "capacity < 0");
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    std::vector<int64_t> counts;
    st = lattice_counts(sc, k, s, counts);
    if (st != GM_OK) return st;
    int64_t N = 0;
    for (int64_t c : counts) N += c;
    if (n_out) *n_out = N;
    if (N > capacity) return fail(GM_ERR_CAPACITY, "%lld samples do not fit capacity %lld", (long long)N, (long long)capacity);
    if (N >= (int64_t)1 << 31) return fail(GM_ERR_INVALID_ARGUMENT, "more than 2^31 - 1 samples");
    GM_HIP(sc->tbegin(kStageSample, s));
    launch_lattice_sample(sc->V.as<float>(), sc->I.as<int32_t>(), sc->tri_mesh.as<int32_t>(), sc->area.as<double>(),
                          sc->lat_C.as<unsigned long long>(), sc->T, N, k, tri, mesh, bary, pos, s);
    GM_HIP(hipGetLastError());
    GM_HIP(sc->tend(kStageSample, s));
    return GM_OK;
}

gm_status gm_count_surface_samples(gm_scene* sc, double k, int64_t* n_per_mesh, void* stream)
{
    gm::clear_error();
    if (!sc || !n_per_mesh) return fail(GM_ERR_INVALID_ARGUMENT, "scene and n_per_mesh must not be NULL");
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    std::vector<int64_t> counts;
    st = sample_counts(sc, k, (hipStream_t)stream, counts);
    if (st != GM_OK) return st;
    std::memcpy(n_per_mesh, counts.data(), 8 * counts.size());
    return GM_OK;
}

gm_status build_surface_samples(gm_scene* sc, double k, uint64_t seed, int32_t* tri, int32_t* mesh, float* bary,
                                float* pos, int64_t capacity, int64_t* n_out, void* stream)
{
    gm::clear_error();
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    if (capacity < 0) return fail(GM_ERR_INVALID_ARGUMENT, "capacity < 0");
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    std::vector<int64_t> counts;
    st = sample_counts(sc, k, s, counts);
    if (st != GM_OK) return st;
    int64_t N = 0;
    for (int64_t c : counts) N += c;
    if (n_out) *n_out = N;
    if (N > capacity) return fail(GM_ERR_CAPACITY, "%lld samples do not fit capacity %lld", (long long)N, (long long)capacity);
    if (N >= (int64_t)1 << 31) return fail(GM_ERR_INVALID_ARGUMENT, "more than 2^31 - 1 samples");
    GM_HIP(sc->tbegin(kStageSample, s));
    launch_mesh_counts(sc->C.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(), sc->S.as<int32_t>(), sc->M, k,
                       sc->counts.as<int64_t>(), sc->offsets.as<int64_t>(), sc->mesh_total.as<unsigned long long>(), s);
    launch_sample(sc->V.as<float>(), sc->I.as<int32_t>(), sc->C.as<unsigned long long>(), sc->tri_off_d.as<int64_t>(),
                  sc->offsets.as<int64_t>(), sc->mesh_total.as<unsigned long long>(), sc->guide.as<int32_t>(),
                  sc->goff.as<int64_t>(), sc->gsh.as<int32_t>(), sc->M, N, seed, tri, mesh, bary, pos, s);
    GM_HIP(hipGetLastError());
    GM_HIP(sc->tend(kStageSample, s));
    return GM_OK;
}

gm_status accumulate_density(gm_scene* sc, const float* pos, const int32_t* tri, const int32_t* mesh, int64_t n,
                             const gm_fixations* fix, double theta_deg, uint32_t flags, float* density,
                             float* density_norm, float* max_out, void* stream)
{
    gm::clear_error();
    gm_status st = check_density_args(sc, pos, n, fix, theta_deg, flags);
    if (st != GM_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    DensityWork& w = sc->work;
    st = density_reserve(w, n, fix->n);
    if (st != GM_OK) return st;
    DensityLaunch a;
    GM_HIP(sc->tbegin(kStagePrep, s));
    const int spl = sc->spl ? sc->spl : ((flags & GM_OCC_MASK) != GM_OCC_NONE ? 1 : 2);
    st = density_prep(sc, w, pos, tri, mesh, n, fix, theta_deg, flags & GM_OCC_MASK, spl, sc->fix_per_chunk, a, s);
    if (st != GM_OK) return st;

    GM_HIP(sc->tend(kStagePrep, s));
    if (n > 0 && fix->n > 0) {
        GM_HIP(sc->tbegin(kStageDensity, s));
        launch_density(a, s);
        GM_HIP(sc->tend(kStageDensity, s));
    }
    GM_HIP(sc->tbegin(kStageFinalize, s));
    st = density_finalize(w, n, density, density_norm, max_out, s);
    if (st != GM_OK) return st;
    GM_HIP(sc->tend(kStageFinalize, s));
    return GM_OK;
}

gm_status gm_debug_sqrt_f64(const double* x, double* y, int64_t n, void* stream)
{
    gm::clear_error();
    if (n < 0 || (n > 0 && (!x || !y))) return fail(GM_ERR_INVALID_ARGUMENT, "NULL argument or negative size");
    launch_sqrt_f64(x, y, n, (hipStream_t)stream);
    GM_HIP(hipGetLastError());
    return GM_OK;
}

gm_status gm_debug_pair_values(const float* pos, int64_t n_points, const gm_fixations* fix, double theta_deg,
                               const int32_t* pair_s, const int32_t* pair_f, int64_t m, float* g_out, void* stream)
{
    gm::clear_error();
    if (!fix || (m > 0 && (!pos || !pair_s || !pair_f || !g_out)) || m < 0 || n_points < 0 || fix->n < 0)
        return fail(GM_ERR_INVALID_ARGUMENT, "NULL argument or negative size");
    if (!(theta_deg > 0.0 && theta_deg < 45.0)) return fail(GM_ERR_INVALID_ARGUMENT, "theta_deg must be in (0, 45)");
    hipStream_t s = (hipStream_t)stream;
    const double sigma = std::tan(theta_deg * M_PI / 180.0);
    DevBuf rec, sh;
    GM_HIP(rec.ensure(sizeof(FixRec) * (size_t)std::max(fix->n, 1)));
    GM_HIP(sh.ensure(16));
    zero(sh.p, 16, s);
    launch_fix_prep(fix->eye, fix->gaze, fix->duration, fix->n, sigma, kGateWiden, rec.as<FixRec>(), nullptr,
                    sh.as<int32_t>(), s);
    launch_pair_values(pos, rec.as<FixRec>(), pair_s, pair_f, m, n_points, fix->n, (float)(16.0 * sigma * sigma),
                       (float)(1.0 / (2.0 * sigma * sigma * std::log(2.0))), g_out, s);
    hipError_t e = hipStreamSynchronize(s);
    rec.release();
    sh.release();
    GM_HIP(e);
    GM_HIP(hipGetLastError());
    return GM_OK;
}

gm_status gm_debug_pair_visibility(gm_scene* sc, const float* pos, const int32_t* tri, const int32_t* mesh,
                                   int64_t n_points, const float* eye, const float* gaze, int32_t n_eyes,
                                   const int32_t* pair_s, const int32_t* pair_f, int64_t m, uint32_t flags,
                                   uint8_t* vis_out, void* stream)
{
    gm::clear_error();
    if (!sc || m < 0 || n_points < 0 || n_eyes < 0 || (m > 0 && (!pos || !eye || !pair_s || !pair_f || !vis_out)))
        return fail(GM_ERR_INVALID_ARGUMENT, "NULL argument or negative size");
    const uint32_t mode = flags & GM_OCC_MASK;
    if (mode > GM_OCC_FULL) return fail(GM_ERR_INVALID_ARGUMENT, "unknown occlusion mode");
    gm_status st = check_device(sc);
    if (st != GM_OK) return st;
    BackfaceArgs bf;
    {
        bf.V = sc->V.as<float>();
        bf.I = sc->I.as<int32_t>();
        bf.closed = sc->closed_d.as<uint8_t>();
        bf.n_meshes = sc->M;
        bf.mbox = sc->mbox_d.as<float4>();
        bf.rmax = sc->bf_rmax;
        bf.l2max = backface_l2max(sc);
        bf.near = sc->solid_near;
        if (mode == GM_OCC_FULL && sc->solid_n > 0) bf.solid = sc->solid.as<BvhNode>();
        bf.solid_mbox = sc->solid_mbox_d.as<float4>();
    }
    launch_pair_visibility(pos, tri, mesh, sc->tri_mesh.as<int32_t>(), eye, gaze, pair_s, pair_f, m, n_points, n_eyes,
                           sc->T, sc->nodes.as<BvhNode>(), sc->tris.as<BvhTri>() + 2 * sc->bvh.tris.size(),
                           (int32_t)mode, bf, vis_out, (hipStream_t)stream);
    GM_HIP(hipGetLastError());
    return GM_OK;
}

gm_status gm_density_counters(gm_scene* sc, int64_t* out, int32_t n_out)
{
    gm::clear_error();
    if (!sc || !out) return fail(GM_ERR_INVALID_ARGUMENT, "scene and out must not be NULL");
    if (n_out < 0) return fail(GM_ERR_INVALID_ARGUMENT, "n_out < 0");
    const int n = std::min<int32_t>(n_out, kDensityStats);
    for (int i = 0; i < n_out; ++i) out[i] = 0;
    if (!sc->work.stats.p) return GM_OK;
    GM_HIP(hipDeviceSynchronize());
    unsigned long long v[kDensityStats];
    GM_HIP(hipMemcpy(v, sc->work.stats.p, sizeof(v), hipMemcpyDeviceToHost));
    for (int i = 0; i < n; ++i) out[i] = (int64_t)v[i];
    return GM_OK;
}

gm_status gm_density_stats(gm_scene* sc, int64_t* out) { return gm_density_counters(sc, out, 4); }

gm_status gm_profile_enable(gm_scene* sc, int32_t on)
{
    gm::clear_error();
    if (!sc) return fail(GM_ERR_INVALID_ARGUMENT, "scene is NULL");
    for (auto& t : sc->timers) {
        GM_HIP(t.collect());
        t.clear();
    }
    sc->profiling = on != 0;
    return GM_OK;
}

gm_status gm_profile_read(gm_scene* sc, const char* stage, double* total_ms, int64_t* launches)
{
    gm::clear_error();
    if (!sc || !stage) return fail(GM_ERR_INVALID_ARGUMENT, "scene and stage must not be NULL");
    for (int i = 0; i < kStages; ++i) {
        if (std::strcmp(stage, kStageNames[i]) != 0) continue;
        GM_HIP(sc->timers[i].collect());
        if (total_ms) *total_ms = sc->timers[i].total_ms;
        if (launches) *launches = sc->timers[i].launches;
        return GM_OK;
    }
    return fail(GM_ERR_INVALID_ARGUMENT, "unknown stage '%s'", stage);
}

}  // extern "C"
