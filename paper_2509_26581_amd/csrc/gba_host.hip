// Problem images, union planning, batch build and the per-problem
// Levenberg-Marquardt driver.
#include "gba_host.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>

namespace gba {

#define HIP_OR(msgv, call)                                                        \
    do {                                                                          \
        hipError_t e_ = (call);                                                   \
        if (e_ != hipSuccess) {                                                   \
            msgv = std::string(#call) + ": " + hipGetErrorString(e_);             \
            return GBA_ERR_HIP;                                                   \
        }                                                                         \
    } while (0)

bool HostProblem::any_free() const {
    for (unsigned char f : cam_fixed)
        if (!f) return true;
    for (unsigned char f : pt_fixed)
        if (!f) return true;
    return false;
}

void* Allocator::allocate(size_t bytes) const {
    if (alloc) return alloc(bytes, ctx);
    void* p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
    return p;
}

void Allocator::release(void* p) const {
    if (!p) return;
    if (free_fn)
        free_fn(p, ctx);
    else
        (void)hipFree(p);
}

void Batch::drop_graphs() {
    for (auto& row : pcg_graph)
        for (auto& pg : row) {
            if (pg.exec) (void)hipGraphExecDestroy(pg.exec);
            pg = PcgGraph{};
        }
    pcg_warm = false;
}

void Batch::release() {
    drop_graphs();
    if (side) (void)hipStreamSynchronize(side);   // a step that failed may have left work there
    if (arena && owns_arena) {
        (void)hipStreamSynchronize(stream);
        allocator.release(arena);
    }
    arena = nullptr;
    arena_bytes = 0;
    P = 0;
}

hipError_t Batch::ensure_side() {
    hipError_t r = hipSuccess;
    if (!side) r = hipStreamCreateWithFlags(&side, hipStreamNonBlocking);
    if (r == hipSuccess && !ev_fork) r = hipEventCreateWithFlags(&ev_fork, hipEventDisableTiming);
    if (r == hipSuccess && !ev_join) r = hipEventCreateWithFlags(&ev_join, hipEventDisableTiming);
    return r;
}

gba_status Batch::ensure_mirrors(int n, std::string& msg) {
    if (n <= h_cap) return GBA_OK;
    if (h_scal) (void)hipHostFree(h_scal);
    if (h_pcg) (void)hipHostFree(h_pcg);
    if (h_lam) (void)hipHostFree(h_lam);
    if (h_accept) (void)hipHostFree(h_accept);
    h_scal = nullptr;
    h_pcg = nullptr;
    h_lam = nullptr;
    h_accept = nullptr;
    h_cap = 0;
    d_scal_host = nullptr;
    d_pcg_host = nullptr;
    // the per-trial and per-chunk results come back through mapped, coherent
    // pinned memory that the finishing kernels write (no copy per readback)
    const unsigned mapped = hipHostMallocMapped | hipHostMallocCoherent;
    if (hipHostMalloc((void**)&h_scal, sizeof(TrialScalars) * n, mapped) != hipSuccess ||
        hipHostMalloc((void**)&h_pcg, sizeof(PcgState) * n, mapped) != hipSuccess ||
        hipHostMalloc((void**)&h_lam, sizeof(double) * n, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&h_accept, sizeof(int) * n, hipHostMallocDefault) != hipSuccess ||
        hipHostGetDevicePointer((void**)&d_scal_host, h_scal, 0) != hipSuccess ||
        hipHostGetDevicePointer((void**)&d_pcg_host, h_pcg, 0) != hipSuccess) {
        msg = "pinned host allocation failed";
        return GBA_ERR_HIP;
    }
    std::memset(h_scal, 0, sizeof(TrialScalars) * n);
    std::memset(h_pcg, 0, sizeof(PcgState) * n);
    h_cap = n;
    return GBA_OK;
}

Batch::~Batch() {
    release();
    if (cap_stream) (void)hipStreamDestroy(cap_stream);
    if (side) (void)hipStreamDestroy(side);
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (ev_join) (void)hipEventDestroy(ev_join);
    if (h_scal) (void)hipHostFree(h_scal);
    if (h_pcg) (void)hipHostFree(h_pcg);
    if (h_lam) (void)hipHostFree(h_lam);
    if (h_accept) (void)hipHostFree(h_accept);
}

hipError_t Timers::init() {
    ev.resize(4 + 2 * 64);
    for (auto& e : ev) {
        hipError_t r = hipEventCreate(&e);
        if (r != hipSuccess) return r;
    }
    return hipSuccess;
}

Timers::~Timers() {
    for (auto& e : ev)
        if (e) (void)hipEventDestroy(e);
}

// ---------------------------------------------------------------- images
// Centre -R^T t of a camera (rotation vector, translation first).
static void camera_centre(const double* cam, double* c) {
    const double w2 = cam[0] * cam[0] + cam[1] * cam[1] + cam[2] * cam[2], th = std::sqrt(w2);
    const double a = th > 1e-8 ? std::sin(th) / th : 1.0, b = th > 1e-8 ? (1.0 - std::cos(th)) / w2 : 0.5;
    const double *w = cam, *t = cam + 3;
    const double wt = w[0] * t[0] + w[1] * t[1] + w[2] * t[2];
    // R^T t = t - a (w x t) + b (w x (w x t))
    const double x[3] = {w[1] * t[2] - w[2] * t[1], w[2] * t[0] - w[0] * t[2], w[0] * t[1] - w[1] * t[0]};
    for (int k = 0; k < 3; ++k) c[k] = -(t[k] - a * x[k] + b * (w[k] * wt - w2 * t[k]));
}

// Squared sine of the angle at X between the rays from two centres (0 for
// coinciding or non-finite ones).
static double ray_sin2(const double* X, const double* c1, const double* c2) {
    const double u[3] = {X[0] - c1[0], X[1] - c1[1], X[2] - c1[2]};
    const double v[3] = {X[0] - c2[0], X[1] - c2[1], X[2] - c2[2]};
    const double x[3] = {u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]};
    const double n = (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double s = (x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) / n;
    return s > 0.0 ? s : 0.0;
}

gba_status make_image(const HostProblem& h, HostImage& img, std::string& msg) {
    img = HostImage{};
    const int nc = h.nc(), np = h.np();
    std::vector<int> act;
    act.reserve(h.n_edges());
    for (int e = 0; e < h.n_edges(); ++e)
        if (h.e_active[e]) act.push_back(e);
    const int ne = (int)act.size();
    const bool info = !h.e_info.empty();

    // point-major order: counting sort by point, camera order inside a point,
    // insertion order for ties
    std::vector<int> cnt(np + 1, 0);
    for (int e : act) cnt[h.e_pt[e] + 1]++;
    for (int j = 0; j < np; ++j) cnt[j + 1] += cnt[j];
    std::vector<int> pm(ne);
    {
        std::vector<int> pos(cnt.begin(), cnt.end() - 1);
        for (int e : act) pm[pos[h.e_pt[e]]++] = e;
        for (int j = 0; j < np; ++j)
            std::stable_sort(pm.begin() + cnt[j], pm.begin() + cnt[j + 1],
                             [&](int a, int c) { return h.e_cam[a] < h.e_cam[c]; });
    }
    img.e_cam.resize(ne);
    img.e_pt.resize(ne);
    img.obs.resize(2 * (size_t)ne);
    for (int q = 0; q < ne; ++q) {
        const int e = pm[q];
        img.e_cam[q] = h.e_cam[e];
        img.e_pt[q] = h.e_pt[e];
        img.obs[q] = h.e_uv[2 * (size_t)e];
        img.obs[(size_t)ne + q] = h.e_uv[2 * (size_t)e + 1];
    }
    // tiles of whole points (<= 64 edges) or one long point
    img.tile_off.push_back(0);
    {
        std::vector<double> centre;
        if (nc <= kRayCams) {
            centre.resize(3 * (size_t)nc);
            for (int i = 0; i < nc; ++i) camera_centre(&h.cam_params[9 * (size_t)i], &centre[3 * (size_t)i]);
        }
        int cur = 0;
        for (int j = 0; j < np; ++j) {
            const int c = cnt[j + 1] - cnt[j];
            if (c == 0) continue;
            img.n.pairs += (long long)c * (c - 1) / 2;
            img.n.min_views = img.n.min_views == 0 ? c : std::min(img.n.min_views, c);
            if (c == 2 && nc <= kRayCams)
                img.n.ray_sin2 = std::min(img.n.ray_sin2,
                                          ray_sin2(&h.pt_params[3 * (size_t)j], &centre[3 * (size_t)img.e_cam[cnt[j]]],
                                                   &centre[3 * (size_t)img.e_cam[cnt[j] + 1]]));
            if (c > kTileEdges) {
                if (cur > 0) {
                    img.tile_off.push_back(img.tile_off.back() + cur);
                    cur = 0;
                }
                img.tile_off.push_back(img.tile_off.back() + c);
            } else {
                if (cur + c > kTileEdges) {
                    img.tile_off.push_back(img.tile_off.back() + cur);
                    cur = 0;
                }
                cur += c;
            }
        }
        if (cur > 0) img.tile_off.push_back(img.tile_off.back() + cur);
    }
    // camera-major order (point order inside a camera), runs of equal
    // (camera, point), chunks of at most kChunkRuns runs of one camera
    std::vector<int> ccount(nc + 1, 0);
    for (int q = 0; q < ne; ++q) ccount[img.e_cam[q] + 1]++;
    for (int i = 0; i < nc; ++i) ccount[i + 1] += ccount[i];
    std::vector<int> cm(ne);  // camera-major position -> point-major position
    {
        std::vector<int> pos(ccount.begin(), ccount.end() - 1);
        for (int q = 0; q < ne; ++q) cm[pos[img.e_cam[q]]++] = q;
    }
    img.cam_chunk_off.assign(nc + 1, 0);
    for (int i = 0; i < nc; ++i) {
        img.cam_chunk_off[i] = (int)img.chunk_cam.size();
        int runs_in_chunk = 0;
        for (int c = ccount[i]; c < ccount[i + 1]; ++c) {
            const bool new_run = c == ccount[i] || img.e_pt[cm[c]] != img.e_pt[cm[c - 1]];
            if (!new_run) continue;
            if (runs_in_chunk == 0) {
                img.chunk_run_off.push_back((int)img.cm_run_off.size());
                img.chunk_cam.push_back(i);
            }
            img.cm_run_off.push_back(c);
            if (++runs_in_chunk == kChunkRuns) runs_in_chunk = 0;
        }
    }
    img.cam_chunk_off[nc] = (int)img.chunk_cam.size();
    const int n_runs = (int)img.cm_run_off.size();
    img.cm_run_off.push_back(ne);
    img.chunk_run_off.push_back(n_runs);
    img.cm_pt.resize(ne);
    img.cm_obs.resize(2 * (size_t)ne);
    for (int c = 0; c < ne; ++c) {
        const int q = cm[c];
        img.cm_pt[c] = img.e_pt[q];
        img.cm_obs[c] = img.obs[q];
        img.cm_obs[(size_t)ne + c] = img.obs[(size_t)ne + q];
    }
    // square-root information factors (Omega = A^T A, A upper triangular)
    if (info) {
        img.sinfo.resize(3 * (size_t)ne);
        img.cm_sinfo.resize(3 * (size_t)ne);
        for (int q = 0; q < ne; ++q) {
            const int e = pm[q];
            const double o00 = h.e_info[3 * (size_t)e], o01 = h.e_info[3 * (size_t)e + 1],
                         o11 = h.e_info[3 * (size_t)e + 2];
            if (!(o00 > 0.0)) {
                msg = "information matrix not positive definite";
                return GBA_ERR_INVALID_ARG;
            }
            const double a00 = std::sqrt(o00), a01 = o01 / a00, d = o11 - a01 * a01;
            if (!(d > 0.0)) {
                msg = "information matrix not positive definite";
                return GBA_ERR_INVALID_ARG;
            }
            img.sinfo[q] = a00;
            img.sinfo[(size_t)ne + q] = a01;
            img.sinfo[2 * (size_t)ne + q] = std::sqrt(d);
        }
        for (int c = 0; c < ne; ++c)
            for (int k = 0; k < 3; ++k)
                img.cm_sinfo[(size_t)k * ne + c] = img.sinfo[(size_t)k * ne + cm[c]];
    }
    img.pm_edge = std::move(pm);
    img.n.nc = nc;
    for (int i = 0; i < nc; ++i) {
        if (!h.cam_fixed[i]) ++img.n.free_cams;
        img.n.cam_edges = std::max(img.n.cam_edges, ccount[i + 1] - ccount[i]);
    }
    img.n.np = np;
    img.n.ne = ne;
    img.n.n_tiles = (int)img.tile_off.size() - 1;
    img.n.n_runs = n_runs;
    img.n.n_chunks = (int)img.chunk_cam.size();
    img.n.info = info;
    return GBA_OK;
}

// ---------------------------------------------------------------- planning
// In the mixed modes S is formed only where the points' places don't hang on
// rounding.  Where two nearly parallel rays are all there is, a point runs off
// along them, and in FP32 its place then follows the rounding of every camera
// step: on whole solves the two forms, and any two orders of the launched
// products' own sums, end up 1e-5 to 0.5 of the points' norm apart, each as far
// from a 64-bit solve (2 of 16 scenes of 203 cameras, 30,011 points and tracks of
// two and more; 5 of 16 bursts of 48 local requests of 5 to 40 keyframes and
// tracks of two to ten).  So every point has three edges (52 solves of 7 to 273
// cameras: at most 6e-9 apart), or there are at most kRayCams cameras and the
// rays of every point of two edges are 0.57 degrees apart, squared sine 1e-4, at
// the start (of 266 requests of up to 20 keyframes six had points that ran off,
// which began at 2.6e-6 to 8.5e-5; 78% of such requests pass, and 64 that do end
// at most 6e-7 apart; windows of more keyframes end a trial's PCG at its limit
// and are 1e-5 apart without such points).  Other solves keep the launched
// products' results.
static bool rays_fix_points(const ImageCounts& n, int precision) {
    if (precision == GBA_FP64 || n.min_views >= 3) return true;
    return n.min_views == 2 && n.nc <= kRayCams && n.ray_sin2 >= 1e-4;
}

// The explicit reduced system (gba_reduced.hip): when the camera sums are
// left to the library, the points are eliminated, no camera observes a point
// twice (the rank bitmaps hold one edge per camera and point), S has at most
// reduced_max rows and the mode's rounding leaves the points where they are
// (above).  A launched PCG iteration takes 14-16 us for small
// problems whatever their size; one workgroup's iteration on S takes 1.6 us at
// 12 cameras, 4.4 at 18 and 6.6 at 28 (FP64: S then comes from the L2 in part).
// Past 28 cameras one CU's reads of S set the pace: in FP64, whole solves at 32,
// 40 and 48 cameras are 1.0, 0.85 and 0.73 times as fast as with launched
// iterations.  The mixed modes read half the bytes: requests of 18, 29, 40 and
// 56 cameras with three-view tracks (100 points a camera) are 2.6, 1.7, 1.4 and
// 1.1 times as fast as with launched iterations.  A single problem has launched
// iterations on S as well (below).
// A block of S is one workgroup's walk over its first camera's edges, 6.5 ns
// (mixed) to 8 ns (FP64) an edge, so few cameras with many edges are bounded
// too: four-trial solves at 2,000, 10,000, 16,000 and 24,000 edges a camera are
// 1.9-2.1, 1.2-1.4, 1.0-1.2 and 0.8-0.95 times as fast with 8 iterations a step
// (2.9-3.6, 1.9-2.7, 1.6-2.6 and 1.2-2.4 with about 25), and with one free
// camera, whose step takes one iteration, 1.2-1.5 at 2,000, 1.0-1.2 at 5,000 and
// 0.8-1.0 at 10,000 (0.2 at 200,000).
bool reduced_rule(const ImageCounts& n, const Tuning& tune, int precision) {
    if (tune.accumulation != GBA_ACC_AUTO || tune.deterministic || tune.solver == GBA_SOLVER_FULL) return false;
    if (!rays_fix_points(n, precision)) return false;
    return n.nc > 0 && n.ne > 0 && n.n_runs == n.ne && 9 * n.nc <= reduced_max(precision) &&
           n.cam_edges <= (n.free_cams > 1 ? 20'000 : 5'000);
}

// The same for a single larger problem, whose launched PCG iterations then
// multiply by S instead of taking the point pass and its reduction.  From 29
// (mixed: 33) cameras on that is faster than one workgroup: mixed, whole solves
// of 1,600 to 25,600 points, one workgroup and launched, 1.49-1.76 and 1.46-1.80
// ms at 32 cameras, 1.85-2.03 and 1.54-1.91 at 40, 2.14-2.69 and 1.75-2.09 at 48.
// Whole solves (8 trials of about 35 iterations, mixed FP32 and FP64) against the
// point passes: 1.5 and 1.6 times as fast at 60 and 90 cameras, 1.4 and 1.5 at
// 130, 1.3 and 1.4 at 203, 1.25 and 1.25 at 240, 1.2 and 0.98 at 300, mixed 1.1
// at 340: S is read in every iteration, so it is bounded to 40 MB (248 cameras,
// mixed 348).  Forming it takes about 60 ps (mixed) and 120 ps (FP64) a pair of a
// point's edges and step (FP64, 260 cameras, 2M pairs: no gain left), so the
// pairs are bounded too.
bool reduced_wide_rule(const ImageCounts& n, const Tuning& tune, int precision) {
    if (tune.accumulation != GBA_ACC_AUTO || tune.deterministic || tune.solver == GBA_SOLVER_FULL) return false;
    if (!rays_fix_points(n, precision)) return false;
    if (n.nc <= 0 || n.ne <= 0 || n.n_runs != n.ne || n.nc <= (precision == GBA_FP64 ? 28 : 32)) return false;
    const long long word = precision == GBA_FP64 ? 8 : 4;
    return 9LL * n.nc * reduced_ld(9 * n.nc) * word <= 40'000'000 && n.pairs * word <= 12'000'000;
}

// S pays when forming it takes no longer than a step's PCG iterations save.
// Iterations of a step: at most the limit, about four a decade of a relative
// tolerance, 25 where neither says less.  Forming a wide S takes 8 us and 60 ps
// an edge and 65 ps a pair of a point's edges (FP64: 150 and 130); a launched
// iteration is 12 us and 17 ps an edge (FP64: 15 and 30) above one on S but for
// the read of S (4 us, or 5.2 MB a us).  Four-trial solves against the launched
// products with 3 and 8 iterations a step, mixed / FP64: 29 cameras, 110,000
// edges 0.95 and 1.16 / 0.88 and 1.06, 550,000 edges 0.75 and 0.98 / 0.63 and
// 0.84; 240 cameras, 161,000 edges 0.74 and 0.85 / 0.61 and 0.77 (with about 30
// iterations 1.1 to 1.5 for all of these).  The one-workgroup form also saves a
// host check, about 50 us.
bool reduced_pays(const ImageCounts& n, int precision, const gba_options& o) {
    double its = std::min(25, o.pcg_max_iters);
    if (o.pcg_tol_relative && o.pcg_tol > 0.0) its = std::min(its, std::max(1.0, -4.0 * std::log10(o.pcg_tol)));
    const bool f64 = precision == GBA_FP64;
    const double ne = n.ne;
    if (!n.wide) return 0.008 * n.cam_edges <= 50.0 + 12.0 * its;
    const double form = 8.0 + (f64 ? 150e-6 : 60e-6) * ne + (f64 ? 130e-6 : 65e-6) * (double)n.pairs;
    const double s_mb = 9.0 * n.nc * reduced_ld(9 * n.nc) * (f64 ? 8e-6 : 4e-6);
    const double saved = (f64 ? 15.0 : 12.0) + (f64 ? 30e-6 : 17e-6) * ne - std::max(4.0, s_mb / 5.2);
    return form <= its * saved;
}

namespace {

// Problem-aligned decomposition of item ranges [off[p], off[p+1]) into
// workgroups of at most `per_block` items, split evenly inside a problem.
HostDecomp make_decomp(const std::vector<int>& off, long long per_block, bool aligned = false) {
    HostDecomp d;
    const int P = (int)off.size() - 1;
    d.prob_blk.resize(P + 1);
    per_block = std::max<long long>(1, per_block);
    for (int p = 0; p < P; ++p) {
        d.prob_blk[p] = d.nblk();
        const long long n = (long long)off[p + 1] - off[p];
        if (n <= 0) continue;
        const long long nb = (n + per_block - 1) / per_block;
        for (long long q = 0; q < nb; ++q) {
            // even split, or full blocks from the problem's start (aligned)
            const long long b = aligned ? per_block * q : n * q / nb;
            const long long e = aligned ? std::min(n, per_block * (q + 1)) : n * (q + 1) / nb;
            d.blk.push_back((int)(off[p] + b));
            d.blk.push_back((int)(off[p] + e));
            d.blk.push_back(p);
        }
    }
    d.prob_blk[P] = d.nblk();
    return d;
}

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

// Sequential layout of 256-byte aligned arrays; with a null base it only
// counts bytes.
struct Planner {
    char* base;
    size_t off = 0;
    explicit Planner(void* b) : base((char*)b) {}
    template <typename T>
    void add(T*& slot, size_t bytes) {
        if (base) slot = (T*)(base + off);
        off += align_up(bytes ? bytes : 1);
    }
};

}  // namespace

gba_status plan_union(const std::vector<const ImageCounts*>& probs, const Tuning& tune,
                      const DeviceInfo& dev, int precision, UnionPlan& u, std::string& msg) {
    u = UnionPlan{};
    const int P = (int)probs.size();
    if (P < 1 || P > kMaxProblems) {
        msg = "a batch holds 1.." + std::to_string(kMaxProblems) + " problems";
        return GBA_ERR_INVALID_ARG;
    }
    u.P = P;
    u.cam_off.assign(P + 1, 0);
    u.pt_off.assign(P + 1, 0);
    u.edge_off.assign(P + 1, 0);
    u.tile_off.assign(P + 1, 0);
    u.run_off.assign(P + 1, 0);
    u.chunk_off.assign(P + 1, 0);
    long long sc = 0, sp = 0, se = 0, st = 0, sr = 0, sk = 0;
    for (int p = 0; p < P; ++p) {
        const ImageCounts& n = *probs[p];
        sc += n.nc;
        sp += n.np;
        se += n.ne;
        st += n.n_tiles;
        sr += n.n_runs;
        sk += n.n_chunks;
        if (se > std::numeric_limits<int>::max() / 32 || sp > std::numeric_limits<int>::max() / 16 ||
            sc > std::numeric_limits<int>::max() / 64) {
            msg = "batch too large for 32-bit indexing";
            return GBA_ERR_UNSUPPORTED;
        }
        u.cam_off[p + 1] = (int)sc;
        u.pt_off[p + 1] = (int)sp;
        u.edge_off[p + 1] = (int)se;
        u.tile_off[p + 1] = (int)st;
        u.run_off[p + 1] = (int)sr;
        u.chunk_off[p + 1] = (int)sk;
        u.tot.info = u.tot.info || n.info;
        u.max_cams = std::max(u.max_cams, n.nc);
    }
    u.tot.nc = (int)sc;
    u.tot.np = (int)sp;
    u.tot.ne = (int)se;
    u.tot.n_tiles = (int)st;
    u.tot.n_runs = (int)sr;
    u.tot.n_chunks = (int)sk;
    // the LDS camera sums of the point passes are FP64 in every mode
    (void)precision;
    const size_t lds = 9 * (size_t)u.max_cams * sizeof(double);
    const bool fits = lds + 1024 <= dev.max_lds;
    if (tune.accumulation == GBA_ACC_LDS && tune.deterministic) {
        msg = "fixed-order sums need the camera-major pass, not LDS partials";
        return GBA_ERR_INVALID_ARG;
    }
    if (tune.accumulation == GBA_ACC_LDS && !fits) {
        msg = "the camera vector of one problem does not fit in LDS (" +
              std::to_string(u.max_cams) + " cameras)";
        return GBA_ERR_UNSUPPORTED;
    }
    // the LDS partials are combined by atomics in a varying order; the
    // camera-major pass sums every camera in a fixed order
    u.deterministic = tune.deterministic != 0;
    u.full = tune.solver == GBA_SOLVER_FULL;
    u.dynamic = u.full && tune.dynamic != 0;
    if (u.full && (u.deterministic || tune.accumulation == GBA_ACC_CAMERA_PASS || !fits)) {
        msg = "the full-Hessian PCG sums the camera side in LDS (at most " +
              std::to_string((dev.max_lds - 1024) / 72) + " cameras per problem, no fixed-order mode)";
        return GBA_ERR_UNSUPPORTED;
    }
    u.cam_pass = tune.accumulation == GBA_ACC_CAMERA_PASS || tune.accumulation == GBA_ACC_CAMERA_BLOCKS ||
                 !fits || u.deterministic;
    u.lds_pp = u.cam_pass ? 0 : (int)lds;
    // the camera-blocked product pass: one problem, stored Jacobians, sums
    // by LDS atomics (so not in the fixed-order mode)
    u.cam_blocks = u.cam_pass && P == 1 && !u.deterministic && !u.full && u.tot.ne > 0 &&
                   (tune.accumulation == GBA_ACC_CAMERA_BLOCKS ||
                    (tune.accumulation == GBA_ACC_AUTO && u.tot.nc > kCamBlock));
    if (u.cam_blocks) {
        u.bo_nblk = (u.tot.nc + kCamBlock - 1) / kCamBlock;
        u.bo_target = std::max(4096, (u.tot.ne + dev.n_cu - 1) / std::max(1, dev.n_cu));
        u.bo_chunk_cap = u.bo_nblk + u.tot.ne / u.bo_target + 1;
    }
    // automatic: one point-pass workgroup per CU (each flushes one LDS camera
    // partial; the flush grows with the workgroup count, and smaller
    // workgroups measured slower in both schemes)
    // A workgroup of the Schur passes gets at least 16 tiles; the whole-system
    // products, with more work per edge (and a Jacobian to recompute when it is
    // dynamic), spread to four: a wavefront per SIMD on four times the CUs.
    // Whole solves in FP64 at 16 and at 4 tiles: dynamic 13.3 and 11.4 ms at 120
    // cameras and 1,000 tiles, 8.7 and 7.0 at 20 and 170; stored 11.0 and 10.5,
    // and 9.3 and 8.7 at 60 cameras.  Two tiles: 16.2, 6.8; 14.0, 11.5 ms.
    const long long least = u.full ? 4 : 16;
    const long long tpb = tune.tiles_per_block > 0
                              ? tune.tiles_per_block
                              : std::max<long long>(least, (st + dev.n_cu - 1) / std::max(1, dev.n_cu));
    const long long epb = tune.edges_per_block > 0 ? tune.edges_per_block
                                                   : std::max<long long>(256, (se + 2047) / 2048);
    const long long ppb = tune.pts_per_block > 0 ? tune.pts_per_block
                                                 : std::max<long long>(256, (sp + 2047) / 2048);
    std::vector<int> comp(P + 1);
    for (int p = 0; p <= P; ++p) comp[p] = 9 * u.cam_off[p];
    u.pp = make_decomp(u.tile_off, tpb);
    u.red = make_decomp(comp, kRedComps, true);   // 16-byte aligned partial reads
    u.cam = make_decomp(u.cam_off, kCamsPerBlock);
    u.edges = make_decomp(u.edge_off, epb);
    u.pts = make_decomp(u.pt_off, ppb);
    u.part_off.assign(std::max(1, u.pp.nblk()), 0);
    long long part = 0;
    for (int p = 0; p < P && !u.cam_pass; ++p) {
        const int ncp = u.cam_off[p + 1] - u.cam_off[p];
        for (int q = u.pp.prob_blk[p]; q < u.pp.prob_blk[p + 1]; ++q) {
            // one partial vector per workgroup, a problem's consecutive and
            // each padded to 4 entries (k_reduce computes the addresses
            // from this layout and reads 16 bytes per lane)
            u.part_off[q] = (int)part;
            part += (9LL * ncp + 3) / 4 * 4;
        }
    }
    if (part > std::numeric_limits<int>::max()) {
        msg = "camera partial buffer too large";
        return GBA_ERR_UNSUPPORTED;
    }
    u.part_total = part;
    u.xs_off.assign(P, -1);
    u.xs_rank_off.assign(P, 0);
    u.xs_all = true;
    if (P == 1) u.one = *probs[0];
    for (int p = 0; p < P; ++p) {
        const ImageCounts& n = *probs[p];
        if (!n.reduced && !(P == 1 && n.wide)) {
            u.xs_all = false;
            continue;
        }
        u.xs_wide = !n.reduced;
        if (u.xs_wide) u.xs_pairs = n.pairs;
        u.xs_off[p] = u.xs_total;
        u.xs_rank_off[p] = u.xs_rank_total;
        u.xs_total += 9LL * n.nc * reduced_ld(9 * n.nc);
        u.xs_rank_total += (long long)n.nc * rank_words(n.np);
        u.xs_cams = std::max(u.xs_cams, n.nc);
    }
    u.cam_prob.resize(sc);
    u.pt_prob.resize(sp);
    for (int p = 0; p < P; ++p) {
        for (int i = u.cam_off[p]; i < u.cam_off[p + 1]; ++i) u.cam_prob[i] = p;
        for (int j = u.pt_off[p]; j < u.pt_off[p + 1]; ++j) u.pt_prob[j] = p;
    }
    return GBA_OK;
}

size_t layout_union(const UnionPlan& u, int precision, void* base, DeviceGraph* dptr) {
    DeviceGraph tmp{};
    DeviceGraph& d = dptr ? *dptr : tmp;
    Planner L(dptr ? base : nullptr);
    const size_t NE = (size_t)u.tot.ne, NP = (size_t)u.tot.np, NC = (size_t)u.tot.nc;
    const int P = u.P;
    const size_t tsz = precision == GBA_FP64 ? 8 : 4;
    const size_t jsz = precision == GBA_FP64 ? 8 : (precision == GBA_MIXED_FP32 ? 4 : 2);
    auto decomp = [&](Decomp& dc, const HostDecomp& h) {
        L.add(dc.blk, sizeof(int) * std::max<size_t>(3, h.blk.size()));
        L.add(dc.prob_blk, sizeof(int) * h.prob_blk.size());
    };
    L.add(d.tile_off, sizeof(int) * (u.tot.n_tiles + 1));
    L.add(d.e_cam, sizeof(int) * NE);
    L.add(d.e_pt, sizeof(int) * NE);
    L.add(d.obs, sizeof(double) * 2 * NE);
    if (u.tot.info) L.add(d.sinfo, sizeof(double) * 3 * NE);
    L.add(d.cm_run_off, sizeof(int) * (u.tot.n_runs + 1));
    L.add(d.cm_pt, sizeof(int) * NE);
    L.add(d.cm_obs, sizeof(double) * 2 * NE);
    if (u.tot.info) L.add(d.cm_sinfo, sizeof(double) * 3 * NE);
    L.add(d.chunk_run_off, sizeof(int) * (u.tot.n_chunks + 1));
    L.add(d.chunk_cam, sizeof(int) * u.tot.n_chunks);
    L.add(d.cam_chunk_off, sizeof(int) * (NC + 1));
    L.add(d.cam_fixed, NC);
    L.add(d.pt_fixed, NP);
    L.add(d.cam_prob, sizeof(int) * NC);
    L.add(d.pt_prob, sizeof(int) * NP);
    L.add(d.prob_cam_off, sizeof(int) * (P + 1));
    L.add(d.lam, sizeof(double) * P);
    L.add(d.accept, sizeof(int) * P);
    L.add(d.pcg, sizeof(PcgState) * P);
    L.add(d.pcg_dec, sizeof(PcgState) * P);
    L.add(d.scal, sizeof(TrialScalars) * P);
    L.add(d.cam, sizeof(double) * 9 * NC);
    L.add(d.cam_c, sizeof(double) * 9 * NC);
    L.add(d.cam_init, sizeof(double) * 9 * NC);
    L.add(d.pt, sizeof(double) * 3 * NP);
    L.add(d.pt_c, sizeof(double) * 3 * NP);
    L.add(d.pt_init, sizeof(double) * 3 * NP);
    L.add(d.dpt, sizeof(double) * 3 * NP);
    const size_t NE64 = (NE + 63) / 64 * 64;   // the stored Jacobian pads to whole 64-edge groups
    if (!u.dynamic) L.add(d.jst, jsz * 24 * NE64);
    else if (dptr) d.jst = nullptr;
    L.add(d.rw, tsz * 2 * NE);
    L.add(d.hpp, tsz * 6 * NP);
    L.add(d.bp, tsz * 3 * NP);
    L.add(d.hcc, tsz * 45 * NC);
    L.add(d.bc, tsz * 9 * NC);
    L.add(d.hpp_inv, tsz * kHinvStride * NP);
    if (!u.dynamic) L.add(d.jst_cm, jsz * 24 * NE64);   // camera-major copy (preconditioner, two-pass products)
    else if (dptr) d.jst_cm = nullptr;
    if (u.cam_pass) L.add(d.zbuf, tsz * 4 * NP);
    if (u.cam_blocks) {
        const size_t cap = (size_t)u.bo_chunk_cap;
        L.add(d.bo_off, sizeof(int) * (cap + 1));
        L.add(d.bo_blk, sizeof(int) * cap);
        L.add(d.bo_blk_chunk, sizeof(int) * (u.bo_nblk + 1));
        L.add(d.bo_perm, sizeof(int) * NE);
        L.add(d.bo_pt, sizeof(int) * NE);
        L.add(d.bo_cam, sizeof(int) * NE);
        L.add(d.jst_bo, jsz * 24 * NE64);
        L.add(d.bo_partial, tsz * cap * kCamBlock * 9);
    } else if (dptr) {
        d.bo_off = d.bo_blk = d.bo_blk_chunk = d.bo_perm = d.bo_pt = d.bo_cam = nullptr;
        d.jst_bo = d.bo_partial = nullptr;
    }
    L.add(d.minv, tsz * 45 * NC);
    L.add(d.v_x, tsz * 9 * NC + 64);   // slack: 16-byte gathers (gather9); back-substitution
    L.add(d.v_r, tsz * 9 * NC);
    L.add(d.v_z, tsz * 9 * NC + 64);   // the product gathers z
    L.add(d.v_p, tsz * 9 * NC);
    L.add(d.v_q, tsz * 9 * NC);
    L.add(d.v_best, tsz * 9 * NC);
    decomp(d.dc_pp, u.pp);
    decomp(d.dc_red, u.red);
    decomp(d.dc_cam, u.cam);
    decomp(d.dc_edges, u.edges);
    decomp(d.dc_pts, u.pts);
    L.add(d.pp_part_off, sizeof(int) * u.part_off.size());
    L.add(d.cam_partial, sizeof(double) * std::max<long long>(1, u.part_total));
    L.add(d.pq_partial, sizeof(double) * std::max({1, u.red.nblk(), u.xs_wide ? reduced_row_blocks(9 * (int)NC) : 0}));
    L.add(d.dot_partial, sizeof(double) * 2 * std::max(1, u.cam.nblk()));
    L.add(d.camupd_partial, sizeof(double) * 3 * std::max(1, u.cam.nblk()));
    L.add(d.chunk_partial, sizeof(double) * 54 * std::max(1, u.tot.n_chunks));
    L.add(d.red_partial, sizeof(double) * 4 * std::max(1, u.pp.nblk()));
    L.add(d.cost_partial, sizeof(double) * std::max(1, u.edges.nblk()));
    L.add(d.damp_partial, sizeof(double) * std::max(1, u.pts.nblk()));
    if (u.xs_total > 0) {
        L.add(d.xs_off, sizeof(long long) * P);
        L.add(d.xs_rank_off, sizeof(long long) * P);
        L.add(d.prob_pt_off, sizeof(int) * (P + 1));
        L.add(d.xs_S, tsz * (size_t)u.xs_total);
        L.add(d.xs_diag, sizeof(double) * 45 * NC);
        L.add(d.xs_rank, sizeof(RankWord) * (size_t)u.xs_rank_total);
        if (u.xs_wide) {
            L.add(d.xs_pair_off, sizeof(int) * (NC * NC + 1));
            L.add(d.xs_pairs, sizeof(int2) * (size_t)u.xs_pairs);
            L.add(d.xs_edge, tsz * kEdgeRec * NE);
        }
    } else if (dptr) {
        d.xs_off = d.xs_rank_off = nullptr;
        d.prob_pt_off = nullptr;
        d.xs_S = nullptr;
        d.xs_diag = nullptr;
        d.xs_rank = nullptr;
    }
    L.add(d.gbar, sizeof(unsigned int) * kGbarWords);
    L.add(d.red_count, sizeof(unsigned int) * u.P);
    if (u.full) {
        for (void** v : {&d.w_x, &d.w_r, &d.w_z, &d.w_p, &d.w_q, &d.w_best})
            L.add(*v, tsz * 3 * NP + 64);
        L.add(d.pdot_partial, sizeof(double) * 2 * std::max(1, u.pts.nblk()));
        L.add(d.ppq_partial, sizeof(double) * std::max(1, u.pp.nblk()));
    } else if (dptr) {
        d.w_x = d.w_r = d.w_z = d.w_p = d.w_q = d.w_best = nullptr;
        d.pdot_partial = d.ppq_partial = nullptr;
    }
    return L.off;
}

void set_union_scalars(Batch& b, int precision, int loss, double delta) {
    const UnionPlan& u = b.plan;
    DeviceGraph& d = b.dg;
    d.nc = u.tot.nc;
    d.np = u.tot.np;
    d.ne = u.tot.ne;
    d.n_tiles = u.tot.n_tiles;
    d.n_runs = u.tot.n_runs;
    d.n_chunks = u.tot.n_chunks;
    d.n_probs = u.P;
    d.has_info = u.tot.info ? 1 : 0;
    d.loss = loss;
    d.delta = delta;
    d.mode = precision;
    d.pcg_host = b.d_pcg_host;
    d.scal_host = b.d_scal_host;
    d.lam_host = b.h_lam;
    d.accept_host = b.h_accept;
    d.jac_bytes = precision == GBA_FP64 ? 8 : (precision == GBA_MIXED_FP32 ? 4 : 2);
    d.block_pp = kPointPassBlock;
    d.cam_pass = u.cam_pass ? 1 : 0;
    d.deterministic = u.deterministic ? 1 : 0;
    d.full = u.full ? 1 : 0;
    d.dynamic = u.dynamic ? 1 : 0;
    d.lds_pp = u.lds_pp;
    d.fuse_apply = !u.full && u.max_cams <= kFuseApplyCams ? 1 : 0;
    d.xs_on = u.xs_total > 0 ? 1 : 0;
    d.xs_all = d.xs_on && u.xs_all ? 1 : 0;
    d.xs_cams = u.xs_cams;
    d.xs_wide = u.xs_wide ? 1 : 0;
    d.xs_pair_total = u.xs_pairs;
    d.xs_rows = 0;
    d.dc_pp.nblk = u.pp.nblk();
    d.dc_red.nblk = u.red.nblk();
    d.dc_cam.nblk = u.cam.nblk();
    d.dc_edges.nblk = u.edges.nblk();
    d.dc_pts.nblk = u.pts.nblk();
    b.P = u.P;
    b.precision = precision;
}

gba_status upload_plan(Batch& b, std::string& msg) {
    const UnionPlan& u = b.plan;
    const DeviceGraph& d = b.dg;
    hipStream_t s = b.stream;
    auto up = [&](const void* dst, const void* src, size_t bytes) -> hipError_t {
        if (!bytes) return hipSuccess;
        return hipMemcpyAsync((void*)dst, src, bytes, hipMemcpyHostToDevice, s);
    };
    auto up_decomp = [&](const Decomp& dc, const HostDecomp& h) -> hipError_t {
        hipError_t r = up(dc.blk, h.blk.data(), sizeof(int) * h.blk.size());
        if (r != hipSuccess) return r;
        return up(dc.prob_blk, h.prob_blk.data(), sizeof(int) * h.prob_blk.size());
    };
    HIP_OR(msg, up_decomp(d.dc_pp, u.pp));
    HIP_OR(msg, up_decomp(d.dc_red, u.red));
    HIP_OR(msg, up_decomp(d.dc_cam, u.cam));
    HIP_OR(msg, up_decomp(d.dc_edges, u.edges));
    HIP_OR(msg, up_decomp(d.dc_pts, u.pts));
    HIP_OR(msg, up(d.pp_part_off, u.part_off.data(), sizeof(int) * u.part_off.size()));
    HIP_OR(msg, up(d.cam_prob, u.cam_prob.data(), sizeof(int) * u.cam_prob.size()));
    HIP_OR(msg, up(d.pt_prob, u.pt_prob.data(), sizeof(int) * u.pt_prob.size()));
    HIP_OR(msg, up(d.prob_cam_off, u.cam_off.data(), sizeof(int) * u.cam_off.size()));
    if (u.xs_total > 0) {
        HIP_OR(msg, up(d.xs_off, u.xs_off.data(), sizeof(long long) * u.xs_off.size()));
        HIP_OR(msg, up(d.xs_rank_off, u.xs_rank_off.data(), sizeof(long long) * u.xs_rank_off.size()));
        HIP_OR(msg, up(d.prob_pt_off, u.pt_off.data(), sizeof(int) * u.pt_off.size()));
    }
    return GBA_OK;
}

gba_status build_batch(const std::vector<const HostProblem*>& probs, int precision, int loss,
                       double delta, const DeviceInfo& dev, const Tuning& tune,
                       const Allocator& alloc, hipStream_t stream, Batch& b, std::string& msg) {
    b.release();
    b.stream = stream;
    b.allocator = alloc;
    b.owns_arena = true;
    const int P = (int)probs.size();
    std::vector<HostImage> imgs(P);
    std::vector<const ImageCounts*> counts(P);
    for (int p = 0; p < P; ++p) {
        gba_status st = make_image(*probs[p], imgs[p], msg);
        if (st != GBA_OK) return st;
        imgs[p].n.wide = P == 1 && reduced_wide_rule(imgs[p].n, tune, precision);
        imgs[p].n.reduced = !imgs[p].n.wide && reduced_rule(imgs[p].n, tune, precision);
        counts[p] = &imgs[p].n;
    }
    gba_status st = plan_union(counts, tune, dev, precision, b.plan, msg);
    if (st != GBA_OK) return st;
    if ((st = b.ensure_mirrors(P, msg)) != GBA_OK) return st;
    const UnionPlan& u = b.plan;
    const size_t bytes = layout_union(u, precision, nullptr, nullptr);
    void* arena = alloc.allocate(bytes);
    if (!arena) {
        msg = "device allocation of " + std::to_string(bytes) + " bytes failed";
        return GBA_ERR_OOM;
    }
    b.arena = arena;
    b.arena_bytes = bytes;
    b.dg = DeviceGraph{};
    b.blocks_zeroed = false;
    b.reduced_built = false;
    b.persistent_ok = -1;
    layout_union(u, precision, arena, &b.dg);
    set_union_scalars(b, precision, loss, delta);
    DeviceGraph& d = b.dg;

    // concatenate the images with offsets (host), then upload
    const size_t NE = u.tot.ne, NP = u.tot.np, NC = u.tot.nc;
    std::vector<int> e_cam(NE), e_pt(NE), cm_pt(NE), tile_off(u.tot.n_tiles + 1),
        run_off(u.tot.n_runs + 1), chunk_run_off(u.tot.n_chunks + 1), chunk_cam(u.tot.n_chunks),
        cam_chunk_off(NC + 1);
    std::vector<double> obs(2 * NE), cm_obs(2 * NE), sinfo, cm_sinfo;
    if (u.tot.info) {
        sinfo.resize(3 * NE);
        cm_sinfo.resize(3 * NE);
    }
    std::vector<unsigned char> cfix(NC), pfix(NP);
    std::vector<double> cams(9 * NC), cams0(9 * NC), pts(3 * NP), pts0(3 * NP);
    b.pm_edge.assign(P, {});
    for (int p = 0; p < P; ++p) {
        const HostImage& im = imgs[p];
        const HostProblem& h = *probs[p];
        const int eo = u.edge_off[p], co = u.cam_off[p], po = u.pt_off[p];
        const int ne = im.n.ne;
        for (int q = 0; q < ne; ++q) {
            e_cam[eo + q] = im.e_cam[q] + co;
            e_pt[eo + q] = im.e_pt[q] + po;
            cm_pt[eo + q] = im.cm_pt[q] + po;
            for (int k = 0; k < 2; ++k) {
                obs[k * NE + eo + q] = im.obs[(size_t)k * ne + q];
                cm_obs[k * NE + eo + q] = im.cm_obs[(size_t)k * ne + q];
            }
            if (u.tot.info)
                for (int k = 0; k < 3; ++k) {
                    const double id = k == 1 ? 0.0 : 1.0;
                    sinfo[k * NE + eo + q] = im.n.info ? im.sinfo[(size_t)k * ne + q] : id;
                    cm_sinfo[k * NE + eo + q] = im.n.info ? im.cm_sinfo[(size_t)k * ne + q] : id;
                }
        }
        for (int t = 0; t < im.n.n_tiles; ++t) tile_off[u.tile_off[p] + t] = im.tile_off[t] + eo;
        for (int r = 0; r < im.n.n_runs; ++r) run_off[u.run_off[p] + r] = im.cm_run_off[r] + eo;
        for (int c = 0; c < im.n.n_chunks; ++c) {
            chunk_run_off[u.chunk_off[p] + c] = im.chunk_run_off[c] + u.run_off[p];
            chunk_cam[u.chunk_off[p] + c] = im.chunk_cam[c] + co;
        }
        for (int i = 0; i < im.n.nc; ++i) cam_chunk_off[co + i] = im.cam_chunk_off[i] + u.chunk_off[p];
        std::copy(h.cam_fixed.begin(), h.cam_fixed.end(), cfix.begin() + co);
        std::copy(h.pt_fixed.begin(), h.pt_fixed.end(), pfix.begin() + po);
        std::copy(h.cam_params.begin(), h.cam_params.end(), cams.begin() + 9 * (size_t)co);
        std::copy(h.cam_init.begin(), h.cam_init.end(), cams0.begin() + 9 * (size_t)co);
        std::copy(h.pt_params.begin(), h.pt_params.end(), pts.begin() + 3 * (size_t)po);
        std::copy(h.pt_init.begin(), h.pt_init.end(), pts0.begin() + 3 * (size_t)po);
        b.pm_edge[p] = std::move(imgs[p].pm_edge);
    }
    tile_off[u.tot.n_tiles] = (int)NE;
    run_off[u.tot.n_runs] = (int)NE;
    chunk_run_off[u.tot.n_chunks] = u.tot.n_runs;
    cam_chunk_off[NC] = u.tot.n_chunks;
    auto up = [&](const void* dst, const void* src, size_t n) -> hipError_t {
        if (!n) return hipSuccess;
        return hipMemcpyAsync((void*)dst, src, n, hipMemcpyHostToDevice, stream);
    };
    HIP_OR(msg, up(d.tile_off, tile_off.data(), sizeof(int) * tile_off.size()));
    HIP_OR(msg, up(d.e_cam, e_cam.data(), sizeof(int) * NE));
    HIP_OR(msg, up(d.e_pt, e_pt.data(), sizeof(int) * NE));
    // the camera-blocked order: the point-major edges bucketed by camera
    // block (so point order inside a block), each block cut into chunks of
    // about bo_target edges
    std::vector<int> bo_off, bo_blk, bo_blk_chunk, bo_perm, bo_pt, bo_cam;
    d.bo_chunks = 0;
    d.bo_nblk = 0;
    if (u.cam_blocks) {
        const int nb = u.bo_nblk;
        std::vector<int> bstart(nb + 1, 0);
        for (size_t e = 0; e < NE; ++e) ++bstart[e_cam[e] / kCamBlock + 1];
        for (int b = 0; b < nb; ++b) bstart[b + 1] += bstart[b];
        bo_perm.resize(NE);
        bo_pt.resize(NE);
        bo_cam.resize(NE);
        {
            std::vector<int> at(bstart.begin(), bstart.end() - 1);
            for (size_t e = 0; e < NE; ++e) {
                const int q = at[e_cam[e] / kCamBlock]++;
                bo_perm[q] = (int)e;
                bo_pt[q] = e_pt[e];
                bo_cam[q] = e_cam[e];
            }
        }
        bo_blk_chunk.assign(nb + 1, 0);
        for (int b = 0; b < nb; ++b) {
            bo_blk_chunk[b] = (int)bo_blk.size();
            const long long n_b = bstart[b + 1] - bstart[b];
            const long long k = std::max(1LL, (n_b + u.bo_target - 1) / u.bo_target);
            for (long long c = 0; c < k && n_b > 0; ++c) {
                bo_off.push_back(bstart[b] + (int)(n_b * c / k));
                bo_blk.push_back(b);
            }
        }
        bo_blk_chunk[nb] = (int)bo_blk.size();
        bo_off.push_back((int)NE);
        if ((int)bo_blk.size() > u.bo_chunk_cap) {
            msg = "camera-blocked chunk count above its bound";
            return GBA_ERR_STATE;
        }
        d.bo_chunks = (int)bo_blk.size();
        d.bo_nblk = nb;
        HIP_OR(msg, up(d.bo_off, bo_off.data(), sizeof(int) * bo_off.size()));
        HIP_OR(msg, up(d.bo_blk, bo_blk.data(), sizeof(int) * bo_blk.size()));
        HIP_OR(msg, up(d.bo_blk_chunk, bo_blk_chunk.data(), sizeof(int) * bo_blk_chunk.size()));
        HIP_OR(msg, up(d.bo_perm, bo_perm.data(), sizeof(int) * NE));
        HIP_OR(msg, up(d.bo_pt, bo_pt.data(), sizeof(int) * NE));
        HIP_OR(msg, up(d.bo_cam, bo_cam.data(), sizeof(int) * NE));
    }
    HIP_OR(msg, up(d.obs, obs.data(), sizeof(double) * 2 * NE));
    if (u.tot.info) {
        HIP_OR(msg, up(d.sinfo, sinfo.data(), sizeof(double) * 3 * NE));
        HIP_OR(msg, up(d.cm_sinfo, cm_sinfo.data(), sizeof(double) * 3 * NE));
    }
    HIP_OR(msg, up(d.cm_run_off, run_off.data(), sizeof(int) * run_off.size()));
    HIP_OR(msg, up(d.cm_pt, cm_pt.data(), sizeof(int) * NE));
    HIP_OR(msg, up(d.cm_obs, cm_obs.data(), sizeof(double) * 2 * NE));
    HIP_OR(msg, up(d.chunk_run_off, chunk_run_off.data(), sizeof(int) * chunk_run_off.size()));
    HIP_OR(msg, up(d.chunk_cam, chunk_cam.data(), sizeof(int) * chunk_cam.size()));
    HIP_OR(msg, up(d.cam_chunk_off, cam_chunk_off.data(), sizeof(int) * cam_chunk_off.size()));
    HIP_OR(msg, up(d.cam_fixed, cfix.data(), NC));
    HIP_OR(msg, up(d.pt_fixed, pfix.data(), NP));
    HIP_OR(msg, up(d.cam, cams.data(), sizeof(double) * 9 * NC));
    HIP_OR(msg, up(d.cam_init, cams0.data(), sizeof(double) * 9 * NC));
    HIP_OR(msg, up(d.pt, pts.data(), sizeof(double) * 3 * NP));
    HIP_OR(msg, up(d.pt_init, pts0.data(), sizeof(double) * 3 * NP));
    if ((st = upload_plan(b, msg)) != GBA_OK) return st;
    HIP_OR(msg, hipStreamSynchronize(stream));
    return GBA_OK;
}

// ---------------------------------------------------------------- LM driver
namespace {

// h_scal is written by k_finish / k_cost_finish through its mapping
gba_status read_scal(Batch& b, std::string& msg) {
    HIP_OR(msg, hipStreamSynchronize(b.stream));
    return GBA_OK;
}

}  // namespace

gba_status batch_linearize(Batch& b, const RawOut* raw, Timers* tm, std::string& msg) {
    const bool timing = tm && tm->on;
    b.dg.jacobian = b.jacobian;
    if (timing) HIP_OR(msg, hipEventRecord(tm->ev[0], b.stream));
    HIP_OR(msg, launch_linearize(b.dg, b.stream, raw, !b.blocks_zeroed));
    b.blocks_zeroed = true;
    if (!raw) HIP_OR(msg, launch_assemble(b.dg, b.stream));
    if (timing) {
        HIP_OR(msg, hipEventRecord(tm->ev[1], b.stream));
        HIP_OR(msg, hipEventSynchronize(tm->ev[1]));
        float ms = 0.f;
        HIP_OR(msg, hipEventElapsedTime(&ms, tm->ev[0], tm->ev[1]));
        tm->ms_phase[0] += ms;
    }
    return GBA_OK;
}

gba_status batch_damped_step(Batch& b, const gba_options& o, const Tuning& tune, Timers* tm,
                             std::string& msg) {
    b.dg.min_diag = o.min_diag;   // the full system's products damp the point rows
    b.dg.max_diag = o.max_diag;
    const DeviceGraph& d = b.dg;
    hipStream_t s = b.stream;
    const bool timing = tm && tm->on;
    if (timing) HIP_OR(msg, hipEventRecord(tm->ev[0], s));
    HIP_OR(msg, launch_damp(d, s, o.min_diag, o.max_diag));
    // the block-Jacobi pass forms the reduced RHS on its way (one-pass scheme)
    const int block_jacobi = o.precond == GBA_PRECOND_BLOCK_JACOBI ? 1 : 0;
    // the full system needs no reduced RHS (its PCG starts from -b)
    if (!d.full && !precond_forms_rhs(d, block_jacobi)) HIP_OR(msg, launch_rhs(d, s));
    HIP_OR(msg, launch_precond(d, s, o.min_diag, o.max_diag, block_jacobi, o.jacobi_scaling));
    if (timing) HIP_OR(msg, hipEventRecord(tm->ev[1], s));
    // explicit reduced systems: S, and the whole PCG of those problems in one
    // launch; with no other problem in the batch the trial runs to its end
    // without a host check (a forced schedule keeps the launched iterations,
    // the identity preconditioner has no diagonal blocks; phase timing takes
    // the same path as none)
    const bool reduced = d.xs_on && block_jacobi && o.pcg_schedule == GBA_PCG_AUTO &&
                         !b.launched_products && (b.P > 1 || reduced_pays(b.plan.one, d.mode, o));
    const bool wide = reduced && d.xs_wide;
    if (!reduced || !d.xs_all || wide) HIP_OR(msg, launch_pcg_init(d, s, o.pcg_tol, o.pcg_tol_relative));
    if (reduced && !b.reduced_built) {
        HIP_OR(msg, launch_reduced_build(d, (size_t)b.plan.xs_rank_total, (size_t)b.plan.xs_total, s));
        b.reduced_built = true;
    }
    // In a batch with other problems S is formed and its PCGs run beside those
    // problems' launched iterations, which take them for stopped: each leaves
    // most of the CUs idle and is a chain of its own.  (One after the other, 12
    // FP64 requests of 5 to 40 keyframes took 39.8 ms, 36.2 with launched
    // iterations alone.)
    const bool beside = reduced && !wide && !d.xs_all && !timing;
    hipStream_t rs = s;
    if (beside) {
        HIP_OR(msg, b.ensure_side());
        HIP_OR(msg, launch_pcg_reduced_mark(d, s));
        HIP_OR(msg, hipEventRecord(b.ev_fork, s));
        HIP_OR(msg, hipStreamWaitEvent(b.side, b.ev_fork, 0));
        rs = b.side;
    }
    if (reduced) HIP_OR(msg, launch_reduced_form(d, rs));
    if (reduced && !wide)
        HIP_OR(msg, launch_pcg_reduced(d, rs, o.pcg_tol, o.pcg_tol_relative, o.pcg_max_iters,
                                       o.pcg_rejection_ratio));
    if (beside) HIP_OR(msg, hipEventRecord(b.ev_join, b.side));
    // back-substitution, the candidate's cost and the trial's sums, and the
    // phase times
    auto finish_trial = [&]() -> gba_status {
        if (timing) HIP_OR(msg, hipEventRecord(tm->ev[2], s));
        HIP_OR(msg, launch_backsub(d, s));
        HIP_OR(msg, launch_cost(d, s, d.cam_c, d.pt_c));
        HIP_OR(msg, launch_finish(d, s));
        if (timing) HIP_OR(msg, hipEventRecord(tm->ev[3], s));
        gba_status st = read_scal(b, msg);
        if (st != GBA_OK) return st;
        if (timing) {
            float a = 0.f, c = 0.f, e = 0.f;
            HIP_OR(msg, hipEventElapsedTime(&a, tm->ev[0], tm->ev[1]));
            HIP_OR(msg, hipEventElapsedTime(&c, tm->ev[1], tm->ev[2]));
            HIP_OR(msg, hipEventElapsedTime(&e, tm->ev[2], tm->ev[3]));
            tm->ms_phase[1] += a;
            tm->ms_phase[2] += c;
            tm->ms_phase[3] += e;
        }
        return GBA_OK;
    };
    if (reduced && d.xs_all && !wide) return finish_trial();
    // one cooperative launch for every PCG iteration (the trial then runs to
    // its end without a host check), or chunks of launched iterations
    bool persistent = false;
    if (!timing && o.pcg_schedule == GBA_PCG_PERSISTENT) {
        if (b.persistent_ok < 0) b.persistent_ok = pcg_persistent_ok(d) ? 1 : 0;
        if (!b.persistent_ok) {
            msg = "the persistent PCG needs cooperative launches and a co-resident grid";
            return GBA_ERR_UNSUPPORTED;
        }
        persistent = true;
    }
    if (persistent) {
        HIP_OR(msg, launch_pcg_persistent(d, s, o.min_diag, o.max_diag, o.pcg_max_iters,
                                          o.pcg_rejection_ratio));
        if (timing) HIP_OR(msg, hipEventRecord(tm->ev[2], s));
        HIP_OR(msg, launch_backsub(d, s));
        HIP_OR(msg, launch_cost(d, s, d.cam_c, d.pt_c));
        HIP_OR(msg, launch_finish(d, s));
        gba_status st = read_scal(b, msg);
        if (st != GBA_OK) return st;
        int iters = 0;
        for (int p = 0; p < b.P; ++p) {
            if (b.h_scal[p].barrier_err) {
                msg = "persistent PCG: a grid barrier wait exceeded its bound";
                return GBA_ERR_HIP;
            }
            iters = std::max(iters, b.h_scal[p].pcg_iters);
        }
        b.last_pcg_iters = iters;
        return GBA_OK;
    }
    DeviceGraph di = d;   // of the launched iterations
    di.xs_rows = wide ? reduced_row_blocks(9 * d.nc) : 0;
    const int chunk = std::max(1, std::min(kMaxPcgChunk, tune.pcg_sync_every));
    // A PCG of k steps takes k + 1 launched iterations: an iteration decides
    // at its start whether the previous step ended the PCG.  The first chunk
    // is the previous step's launch count (successive LM trials need similar
    // counts; an idle iteration costs a few microseconds, a further host
    // check about thirty), replayed as a graph or launched directly, and the
    // rest are chunks of two.  Without a previous count: chunks of
    // pcg_sync_every.
    int first = chunk, rest = chunk;
    if (b.last_pcg_iters > 0) {
        first = std::min(kMaxPcgChunk, b.last_pcg_iters + 1);
        rest = std::min(chunk, 2);
    }
    const int max_launch = o.pcg_max_iters + 1;
    int launched = 0;
    int last_iters = 0;
    int products = 0;   // timing: launches that ran a product
    while (launched < max_launch) {
        const int c = std::min(launched == 0 ? first : rest, max_launch - launched);
        if (b.use_graphs && !timing && b.pcg_warm) {
            // replay the chunk as one graph (captured on first use, cached by length)
            // the dynamic product reads the parameters: one graph per
            // orientation of the current/candidate buffers
            const int orient = d.dynamic && d.cam > d.cam_c ? 1 : 0;
            Batch::PcgGraph& pg = b.pcg_graph[c][orient];
            const bool moved = d.dynamic && (pg.cam != d.cam || pg.pt != d.pt);
            if (pg.exec && (pg.iters != c || pg.max_iters != o.pcg_max_iters ||
                            pg.min_diag != o.min_diag || pg.max_diag != o.max_diag ||
                            pg.ratio != o.pcg_rejection_ratio || pg.wide != wide || moved)) {
                (void)hipGraphExecDestroy(pg.exec);
                pg = Batch::PcgGraph{};
            }
            if (!pg.exec) {
                // captured on a private stream, replayed on the batch stream
                if (!b.cap_stream)
                    HIP_OR(msg, hipStreamCreateWithFlags(&b.cap_stream, hipStreamNonBlocking));
                hipStream_t cs = b.cap_stream;
                hipGraph_t graph = nullptr;
                HIP_OR(msg, hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
                hipError_t r = hipSuccess;
                for (int k = 0; k < c && r == hipSuccess; ++k)
                    r = launch_pcg_iter(di, cs, o.min_diag, o.max_diag, o.pcg_max_iters,
                                        o.pcg_rejection_ratio, nullptr, nullptr);
                hipError_t r2 = hipStreamEndCapture(cs, &graph);
                HIP_OR(msg, r);
                HIP_OR(msg, r2);
                r = hipGraphInstantiate(&pg.exec, graph, nullptr, nullptr, 0);
                (void)hipGraphDestroy(graph);
                HIP_OR(msg, r);
                pg.iters = c;
                pg.max_iters = o.pcg_max_iters;
                pg.min_diag = o.min_diag;
                pg.max_diag = o.max_diag;
                pg.ratio = o.pcg_rejection_ratio;
                pg.wide = wide;
                pg.cam = d.cam;
                pg.pt = d.pt;
            }
            HIP_OR(msg, hipGraphLaunch(pg.exec, s));
        } else {
            for (int k = 0; k < c; ++k) {
                hipEvent_t e0 = timing ? tm->ev[4 + 2 * k] : nullptr;
                hipEvent_t e1 = timing ? tm->ev[5 + 2 * k] : nullptr;
                HIP_OR(msg, launch_pcg_iter(di, s, o.min_diag, o.max_diag, o.pcg_max_iters,
                                            o.pcg_rejection_ratio, e0, e1));
            }
            b.pcg_warm = true;
        }
        launched += c;
        // h_pcg is written by the apply kernels through its mapping
        HIP_OR(msg, hipStreamSynchronize(s));
        int max_iters_now = 0;
        bool all_done = true;
        for (int p = 0; p < b.P; ++p) {
            if (reduced && !wide && b.plan.xs_off[p] >= 0) continue;   // its own PCG
            max_iters_now = std::max(max_iters_now, b.h_pcg[p].iters);
            all_done = all_done && b.h_pcg[p].done != 0;
        }
        if (timing) {
            // only launches in which some problem still stepped time a
            // product: every launch until all PCGs have stopped, then as many
            // as the longest one took steps
            const int ran = std::min(c, std::max(0, (all_done ? max_iters_now : launched) - products));
            products += ran;
            for (int k = 0; k < ran; ++k) {
                float ms = 0.f;
                HIP_OR(msg, hipEventElapsedTime(&ms, tm->ev[4 + 2 * k], tm->ev[5 + 2 * k]));
                tm->ms_mv += ms;
                tm->n_mv += 1;
            }
        }
        last_iters = max_iters_now;
        if (all_done) break;
    }
    b.last_pcg_iters = last_iters;
    if (beside) HIP_OR(msg, hipStreamWaitEvent(s, b.ev_join, 0));
    return finish_trial();
}

gba_status batch_time_matvec(Batch& b, const gba_options& o, int launches, double* ms,
                             std::string& msg) {
    b.dg.min_diag = o.min_diag;
    b.dg.max_diag = o.max_diag;
    const DeviceGraph& d = b.dg;
    hipStream_t s = b.stream;
    HIP_OR(msg, launch_damp(d, s, o.min_diag, o.max_diag));
    // the block-Jacobi pass forms the reduced RHS on its way (one-pass scheme)
    const int block_jacobi = o.precond == GBA_PRECOND_BLOCK_JACOBI ? 1 : 0;
    // the full system needs no reduced RHS (its PCG starts from -b)
    if (!d.full && !precond_forms_rhs(d, block_jacobi)) HIP_OR(msg, launch_rhs(d, s));
    HIP_OR(msg, launch_precond(d, s, o.min_diag, o.max_diag, block_jacobi, o.jacobi_scaling));
    // tolerance 0 and no iteration limit: the products below run for every
    // problem with work.  One iteration first, so that they take the decision
    // of a later iteration, as in the PCG loop.
    constexpr int kNoLimit = 1 << 30;
    HIP_OR(msg, launch_pcg_init(d, s, 0.0, 0));
    HIP_OR(msg, launch_pcg_iter(d, s, o.min_diag, o.max_diag, kNoLimit, 0.0, nullptr, nullptr));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_OR(msg, hipEventCreate(&e0));
    hipError_t r = hipEventCreate(&e1);
    if (r == hipSuccess) r = hipEventRecord(e0, s);
    for (int k = 0; k < launches && r == hipSuccess; ++k) r = launch_matvec(d, s, kNoLimit, 0.0);
    if (r == hipSuccess) r = hipEventRecord(e1, s);
    if (r == hipSuccess) r = hipEventSynchronize(e1);
    float t = 0.f;
    if (r == hipSuccess) r = hipEventElapsedTime(&t, e0, e1);
    (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    HIP_OR(msg, r);
    *ms = launches > 0 ? (double)t / launches : 0.0;
    return GBA_OK;
}

gba_status batch_cost(Batch& b, std::string& msg) {
    HIP_OR(msg, launch_cost(b.dg, b.stream, b.dg.cam, b.dg.pt));
    HIP_OR(msg, launch_cost_finish(b.dg, b.stream));
    return read_scal(b, msg);
}

gba_status batch_begin(Batch& b, const std::vector<const HostProblem*>& probs,
                       std::vector<ProblemLM>& lm, const std::vector<char>& fresh,
                       const gba_options& o, Timers* tm, std::string& msg) {
    gba_status st = batch_cost(b, msg);
    if (st != GBA_OK) return st;
    bool any = false;
    for (int p = 0; p < b.P; ++p) {
        ProblemLM& s = lm[p];
        if (!fresh[p]) {
            any = any || s.running;
            continue;
        }
        const bool edges = b.plan.edge_off[p + 1] > b.plan.edge_off[p];
        s.F = edges ? b.h_scal[p].cost : 0.0;
        s.F0 = s.F;
        s.lam = o.initial_lambda;
        s.nu = 2.0;
        s.trials = s.accepted = s.pcg_total = 0;
        s.log.clear();
        s.running = false;
        if (!edges || !probs[p]->any_free()) {
            s.term = GBA_TERM_NO_WORK;
        } else if (s.max_iters <= 0) {
            s.term = GBA_TERM_MAX_ITERS;
        } else if (!std::isfinite(s.F)) {
            s.term = GBA_TERM_NUMERICAL_FAILURE;
        } else {
            s.term = GBA_TERM_NONE;
            s.running = true;
            any = true;
        }
    }
    if (any) return batch_linearize(b, nullptr, tm, msg);
    return GBA_OK;
}

gba_status batch_trial(Batch& b, std::vector<ProblemLM>& lm, const gba_options& o,
                       const Tuning& tune, Timers* tm, std::string& msg) {
    // idle problems (terminated or without work) carry a negative damping: the
    // device skips their PCG
    for (int p = 0; p < b.P; ++p) b.h_lam[p] = lm[p].running ? lm[p].lam : -o.initial_lambda;
    gba_status st = batch_damped_step(b, o, tune, tm, msg);
    if (st != GBA_OK) return st;
    bool any_accept = false, any_running = false;
    for (int p = 0; p < b.P; ++p) {
        b.h_accept[p] = 0;
        ProblemLM& s = lm[p];
        if (!s.running) continue;
        const TrialScalars& sc = b.h_scal[p];
        const double Fn = sc.cost;
        const double L = -(sc.b_dot_dx + 0.5 * sc.quad);
        const double dnorm = std::sqrt(sc.step2), xnorm = std::sqrt(sc.x2);
        const bool accepted = (L > 0.0) && (Fn < s.F);
        const double gain = L != 0.0 ? (s.F - Fn) / L : std::numeric_limits<double>::quiet_NaN();
        gba_trial tr;
        tr.cost = s.F;
        tr.candidate_cost = Fn;
        tr.lambda = s.lam;
        tr.model_decrease = L;
        tr.step_norm = dnorm;
        tr.accepted = accepted ? 1 : 0;
        tr.pcg_iters = sc.pcg_iters;
        s.log.push_back(tr);
        s.trials += 1;
        s.pcg_total += sc.pcg_iters;
        int stop = 0;
        if (accepted) {
            const double rel = (s.F - Fn) / s.F;
            s.F = Fn;
            const double t3 = 2.0 * gain - 1.0;
            s.lam *= std::max(1.0 / 3.0, 1.0 - t3 * t3 * t3);
            s.nu = 2.0;
            s.accepted += 1;
            b.h_accept[p] = 1;
            any_accept = true;
            if (rel < s.tol) stop = GBA_TERM_COST_TOL;
        } else {
            s.lam *= s.nu;
            s.nu *= 2.0;
        }
        if (!stop && dnorm <= s.tol * (xnorm + s.tol)) stop = GBA_TERM_STEP_TOL;
        if (!stop && s.lam > 1e32) stop = GBA_TERM_LAMBDA_OVERFLOW;
        if (!stop && s.trials >= s.max_iters) stop = GBA_TERM_MAX_ITERS;
        if (stop) {
            s.term = stop;
            s.running = false;
        }
        any_running = any_running || s.running;
    }
    if (any_accept) {
        if (b.P == 1) {
            // one problem: the candidate buffers become the current ones
            std::swap(b.dg.cam, b.dg.cam_c);
            std::swap(b.dg.pt, b.dg.pt_c);
        } else {
            HIP_OR(msg, launch_commit(b.dg, b.stream));
        }
        if (any_running) return batch_linearize(b, nullptr, tm, msg);
        HIP_OR(msg, hipStreamSynchronize(b.stream));
    }
    return GBA_OK;
}

gba_status batch_download(Batch& b, int p, double* cams, double* pts, std::string& msg) {
    const int c0 = b.plan.cam_off[p], c1 = b.plan.cam_off[p + 1];
    const int p0 = b.plan.pt_off[p], p1 = b.plan.pt_off[p + 1];
    if (cams && c1 > c0)
        HIP_OR(msg, hipMemcpyAsync(cams, b.dg.cam + 9 * (size_t)c0, sizeof(double) * 9 * (c1 - c0),
                                   hipMemcpyDeviceToHost, b.stream));
    if (pts && p1 > p0)
        HIP_OR(msg, hipMemcpyAsync(pts, b.dg.pt + 3 * (size_t)p0, sizeof(double) * 3 * (p1 - p0),
                                   hipMemcpyDeviceToHost, b.stream));
    HIP_OR(msg, hipStreamSynchronize(b.stream));
    return GBA_OK;
}

}  // namespace gba
