// Host-only checks of the explicit reduced systems' parts that run on both
// sides, built with a plain C++ compiler by tests/test_reduced_host.py.  No GPU
// is touched.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "gba_host.hip"
#include "gba_vi_rule.h"

// the buffers' allocations and copies, on the host
#include <map>
static std::map<char*, size_t> g_blocks;
static size_t g_limit = ~(size_t)0;
static hipError_t host_malloc(void** p, size_t n) {
    if (n > g_limit) return hipErrorOutOfMemory;
    *p = std::aligned_alloc(256, (n + 255) & ~(size_t)255);
    g_blocks[(char*)*p] = n;
    return hipSuccess;
}
static hipError_t host_free(void* p) {
    g_blocks.erase((char*)p);
    std::free(p);
    return hipSuccess;
}
static hipError_t host_copy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
#define hipMalloc host_malloc
#define hipFree host_free
#define hipMemcpy host_copy
#define hipGetLastError() hipSuccess
#include "gba_vi_bufs.h"
#undef hipMalloc
#undef hipFree
#undef hipMemcpy
#undef hipGetLastError

namespace gba {
#define GBA_STUB(name, ...)                                        \
    hipError_t name(__VA_ARGS__) {                                 \
        std::fprintf(stderr, "unexpected launch: %s\n", #name);    \
        std::abort();                                              \
    }
GBA_STUB(launch_linearize, const DeviceGraph&, hipStream_t, const RawOut*, bool)
GBA_STUB(launch_assemble, const DeviceGraph&, hipStream_t)
GBA_STUB(launch_cost, const DeviceGraph&, hipStream_t, const double*, const double*)
GBA_STUB(launch_cost_finish, const DeviceGraph&, hipStream_t)
GBA_STUB(launch_damp, const DeviceGraph&, hipStream_t, double, double)
GBA_STUB(launch_precond, const DeviceGraph&, hipStream_t, double, double, int, int)
GBA_STUB(launch_rhs, const DeviceGraph&, hipStream_t)
GBA_STUB(launch_pcg_init, const DeviceGraph&, hipStream_t, double, int)
GBA_STUB(launch_pcg_iter, const DeviceGraph&, hipStream_t, double, double, int, double, hipEvent_t,
         hipEvent_t)
GBA_STUB(launch_matvec, const DeviceGraph&, hipStream_t, int, double)
GBA_STUB(launch_backsub, const DeviceGraph&, hipStream_t)
GBA_STUB(launch_finish, const DeviceGraph&, hipStream_t)
GBA_STUB(launch_commit, const DeviceGraph&, hipStream_t)
bool precond_forms_rhs(const DeviceGraph&, int) { return false; }
}  // namespace gba

using namespace gba;

static int g_fail = 0;
#define CHECK(c)                                                                   \
    do {                                                                           \
        if (!(c)) {                                                                \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
            ++g_fail;                                                              \
        }                                                                          \
    } while (0)

// The blocks' point side J_p,i Hpp^-1 J_p,k^T of FP32 inverses up to condition
// 1e12 equals the product with the stored inverse itself (as the diagonal
// blocks have it) to the FP32 rounding of J_p Hpp^-1, six terms of at most one
// rounding each.  (A Cholesky factor of such an inverse is off by thousands of
// roundings where its condition passes 1e8.)
static void check_point_side() {
    std::mt19937_64 rng(1);
    std::normal_distribution<double> nrm;
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    for (int it = 0; it < 20000; ++it) {
        // H^-1 = Q diag(1, e1, e2) Q^T with e2 <= e1 <= 1
        double q[3][3];
        for (auto& r : q)
            for (double& v : r) v = nrm(rng);
        for (int a = 0; a < 3; ++a) {   // Gram-Schmidt
            for (int b = 0; b < a; ++b) {
                double d = 0.0;
                for (int c = 0; c < 3; ++c) d += q[a][c] * q[b][c];
                for (int c = 0; c < 3; ++c) q[a][c] -= d * q[b][c];
            }
            double n = 0.0;
            for (int c = 0; c < 3; ++c) n += q[a][c] * q[a][c];
            for (int c = 0; c < 3; ++c) q[a][c] /= std::sqrt(n);
        }
        const double e[3] = {1.0, std::pow(10.0, -12.0 * uni(rng)), std::pow(10.0, -12.0 * uni(rng))};
        float h[6];
        int at = 0;
        for (int r = 0; r < 3; ++r)
            for (int c = r; c < 3; ++c) {
                double v = 0.0;
                for (int k = 0; k < 3; ++k) v += e[k] * q[k][r] * q[k][c];
                h[at++] = (float)v;
            }
        float ji[2][3], jk[2][3], out[6];
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 3; ++c) {
                ji[r][c] = (float)nrm(rng);
                jk[r][c] = (float)nrm(rng);
            }
        point_side(ji, h, out);
        const int sym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 2; ++c) {
                double got = 0.0, want = 0.0, size = 0.0;
                for (int k = 0; k < 3; ++k) {
                    got += (double)out[3 * r + k] * (double)jk[c][k];
                    for (int m = 0; m < 3; ++m) {
                        const double t = (double)ji[r][m] * (double)h[sym[m][k]] * (double)jk[c][k];
                        want += t;
                        size += std::fabs(t);
                    }
                }
                CHECK(std::fabs(got - want) <= size * std::ldexp(1.0, -23));
            }
    }
}

// Which problems take which form: one workgroup's PCG up to 28 cameras (FP64)
// or 56 (mixed), for a single problem of more than 28 or 32 launched iterations
// on S (the one-workgroup form is the slower one there), the launched products
// where S or its forming costs too much.
static ImageCounts counts(int nc, int np, int ne, long long pairs) {
    ImageCounts n;
    n.free_cams = nc - 1;
    n.cam_edges = ne / nc;
    n.min_views = 3;
    n.nc = nc;
    n.np = np;
    n.ne = n.n_runs = ne;
    n.pairs = pairs;
    return n;
}
static void check_rules() {
    const Tuning t;
    for (int prec : {GBA_FP64, GBA_MIXED_FP32, GBA_MIXED_BF16})
        for (int nc = 2; nc <= 400; ++nc) {
            const ImageCounts n = counts(nc, 20 * nc, 100 * nc, 200 * nc);
            CHECK(reduced_rule(n, t, prec) == (nc <= (prec == GBA_FP64 ? 28 : 56)));
            CHECK(reduced_wide_rule(n, t, prec) ==
                  (prec == GBA_FP64 ? nc > 28 && nc <= 248 : nc > 32 && nc <= 348));
        }
    // points of two rays in the mixed modes: few cameras and rays apart only;
    // of one ray never
    for (int prec : {GBA_FP64, GBA_MIXED_FP32, GBA_MIXED_BF16})
        for (int nc : {10, 20, 21, 60, 200})
            for (int views : {1, 2})
                for (double sin2 : {0.0, 0.9e-4, 1.1e-4}) {
                    ImageCounts n = counts(nc, 20 * nc, 100 * nc, 200 * nc);
                    n.min_views = views;
                    n.ray_sin2 = sin2;
                    CHECK((reduced_rule(n, t, prec) || reduced_wide_rule(n, t, prec)) ==
                          (prec == GBA_FP64 || (views == 2 && nc <= 20 && sin2 > 1e-4)));
                }
    // few cameras with many edges: forming S would cost more than the PCG
    for (int nc : {2, 3, 8, 28})
        for (int per : {1'000, 4'000, 6'000, 19'000, 21'000, 200'000}) {
            const ImageCounts n = counts(nc, per, nc * per, per);
            CHECK(reduced_rule(n, t, GBA_FP64) == (per <= (nc == 2 ? 5'000 : 20'000)));
        }
}

// The rays' least squared sine and the fewest views, as an image counts them.
static void check_rays() {
    // cameras at known centres, turned arbitrarily: t = -R c
    std::mt19937_64 rng(2);
    std::normal_distribution<double> nrm;
    for (int it = 0; it < 200; ++it) {
        HostProblem h;
        const double off[2] = {std::pow(10.0, -3.0 + 3.0 * (it / 200.0)), 5.0};
        const double centre[3][3] = {{0, 0, 0}, {off[0], 0, 0}, {0, off[1], 0}};
        for (auto& c : centre) {
            const double w[3] = {it ? nrm(rng) : 0.0, it ? nrm(rng) : 0.0, it ? nrm(rng) : 0.0};
            const double th = std::sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
            const double k[3] = {th ? w[0] / th : 1, th ? w[1] / th : 0, th ? w[2] / th : 0};
            const double kc = k[0] * c[0] + k[1] * c[1] + k[2] * c[2];
            const double x[3] = {k[1] * c[2] - k[2] * c[1], k[2] * c[0] - k[0] * c[2], k[0] * c[1] - k[1] * c[0]};
            for (double v : w) h.cam_params.push_back(v);
            for (int a = 0; a < 3; ++a)
                h.cam_params.push_back(-(c[a] * std::cos(th) + x[a] * std::sin(th) + k[a] * kc * (1 - std::cos(th))));
            for (double v : {500.0, 0.0, 0.0}) h.cam_params.push_back(v);
            h.cam_fixed.push_back(0);
        }
        const double pts[3][3] = {{0, 0, 10}, {0, 0, 10}, {1, 1, 8}};
        for (auto& p : pts) {
            for (double v : p) h.pt_params.push_back(v);
            h.pt_fixed.push_back(0);
        }
        // point 0: cameras 0 and 1; point 1: 0 and 2; point 2: all (not counted)
        const int ec[] = {1, 0, 2, 0, 0, 1, 2}, ep[] = {0, 0, 1, 1, 2, 2, 2};
        for (int e = 0; e < 7; ++e) {
            h.e_cam.push_back(ec[e]);
            h.e_pt.push_back(ep[e]);
            h.e_uv.push_back(0.0);
            h.e_uv.push_back(0.0);
            h.e_active.push_back(1);
        }
        h.cam_init = h.cam_params;
        h.pt_init = h.pt_params;
        HostImage img;
        std::string msg;
        CHECK(make_image(h, img, msg) == GBA_OK);
        const double least = off[0] < off[1] ? off[0] : off[1];
        const double want = least * least / (least * least + 100.0);
        CHECK(img.n.min_views == 2);
        CHECK(std::fabs(img.n.ray_sin2 - want) <= 1e-9 * want + 1e-20);
    }
}

// S is formed where a step's iterations pay for it: not at a small iteration
// limit or with a loose tolerance, and always at those of a tight PCG.
static void check_pays() {
    gba_options o{};
    o.pcg_tol = 1e-6;
    o.pcg_tol_relative = 1;
    const int nc[] = {29, 240, 60}, ne[] = {550'000, 161'000, 80'000};
    const long long pairs[] = {1'380'000, 1'000'000, 760'000};
    for (int prec : {GBA_FP64, GBA_MIXED_FP32})
        for (int k = 0; k < 3; ++k) {
            ImageCounts n = counts(nc[k], 1'000, ne[k], pairs[k]);
            n.wide = true;
            o.pcg_max_iters = 100;
            o.pcg_tol = 1e-6;
            CHECK(reduced_pays(n, prec, o));
            o.pcg_max_iters = 3;
            CHECK(!reduced_pays(n, prec, o));
            o.pcg_max_iters = 100;
            o.pcg_tol = 0.2;
            CHECK(!reduced_pays(n, prec, o));
            o.pcg_tol_relative = 0;   // an absolute tolerance says nothing
            CHECK(reduced_pays(n, prec, o));
            o.pcg_tol_relative = 1;
            o.pcg_tol = 0.0;
            CHECK(reduced_pays(n, prec, o));
        }
    o.pcg_max_iters = 1;
    CHECK(!reduced_pays(counts(5, 20'000, 90'000, 120'000), GBA_FP64, o));
    CHECK(reduced_pays(counts(5, 500, 2'000, 3'000), GBA_FP64, o));
}

// Keyframe blocks: formed for windowed visibility and for scattered visibility
// of few blocks an observation, not where an iteration's blocks are more than
// the observations they replace, nor for a handful of iterations.
static void check_vi_blocks() {
    const auto pay = vi::vi_blocks_pay;
    for (int its : {50, 100, 4000}) {
        CHECK(pay(32'000, 112'000, 3'540, 0, its));              // 60 keyframes
        CHECK(pay(2'070'000, 7'000'000, 24'000, 0, its));        // 2,000, windowed
        CHECK(pay(400'000, 1'400'000, 938'000, 380'000, its));   // 1,000, at random
        CHECK(!pay(400'000, 1'400'000, 2'400'000, 390'000, its));   // 3,000, at random
        CHECK(!pay(240'000, 360'000, 528'000, 0, its));          // 12,000, few points
    }
    CHECK(pay(32'000, 112'000, 3'540, 0, 1));
    CHECK(!pay(2'070'000, 7'000'000, 24'000, 0, 1));
}

// Buffers of a call: 256-byte aligned, inside an allocation, disjoint while they
// live; scratch memory is reused after it is dropped, whatever the expected size
// and also where allocations of the expected size fail.
static void check_buffers() {
    std::mt19937_64 rng(7);
    for (int it = 0; it < 400; ++it) {
        g_limit = it % 4 == 3 ? 20'000 : ~(size_t)0;   // larger allocations fail
        {
            vi::DevBufs b(1 + rng() % 200'000);
            struct Live {
                char* p;
                size_t n;
                bool scratch;
            };
            std::vector<Live> live;
            std::vector<char> src(12'000, 'x');
            for (int k = 0; k < 60; ++k) {
                if (rng() % 12 == 0) {
                    b.drop_scratch();
                    live.erase(std::remove_if(live.begin(), live.end(), [](const Live& l) { return l.scratch; }),
                               live.end());
                    continue;
                }
                char* p = nullptr;
                const size_t n = rng() % 12'000;
                const bool scratch = rng() % 3 == 0, copy = rng() % 2 == 0;
                CHECK(scratch ? b.scratch(&p, copy ? src.data() : nullptr, n)
                              : b.up(&p, copy ? src.data() : nullptr, n));
                CHECK((uintptr_t)p % 256 == 0);
                auto blk = g_blocks.upper_bound(p);
                CHECK(blk != g_blocks.begin());
                --blk;
                CHECK(p + n <= blk->first + blk->second);
                for (const Live& l : live) CHECK(p + n <= l.p || l.p + l.n <= p || n == 0 || l.n == 0);
                live.push_back({p, n, scratch});
            }
        }
        CHECK(g_blocks.empty());
    }
}

// The residual exchange of the one-workgroup PCG stays among the entries that
// the wavefront's row owners have written, for every lane.
static void check_exchange() {
    CHECK(kOwnRows == 63);
    for (int l = 0; l < kWave; ++l) {
        const int first = own_first(l);
        CHECK(first >= 0 && first + 8 < kOwnRows && first % 9 == 0);
        CHECK(l >= kOwnRows || (first <= l && l < first + 9));
    }
}

int main() {
    check_exchange();
    check_vi_blocks();
    check_buffers();
    // the arguments of a recorded iteration's kernels without the explicit systems' part
    CHECK(sizeof(KernelGraph) <= 848 && sizeof(DeviceGraph) > sizeof(KernelGraph));
    check_point_side();
    check_rules();
    check_rays();
    check_pays();
    if (g_fail) {
        std::fprintf(stderr, "%d checks failed\n", g_fail);
        return 1;
    }
    std::printf("reduced checks passed\n");
    return 0;
}
