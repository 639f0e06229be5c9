// C ABI of libteuk.so (declared and documented in include/teuk.h).
//
// Host responsibilities: argument validation (before any device work),
// workspace layout, the 1-D coefficient tables of Eq. (1), extraction
// weights, launch geometry and ping-pong of the state buffers.  All step
// arithmetic runs in the gfx950 kernels of lw_kernels.hip.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/teuk.h"
#include "geometry.hpp"
#include "internal.hpp"

using namespace teuk;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) return fail(TEUK_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr size_t kAlign = 256;
constexpr int kMaxExtract = 4096;
constexpr int64_t kMaxSingleUserSource = 300000;  // points of a grid with user coefficients and a source
constexpr int kMaxFusedAdjointExtract = 16;  // extraction points handled inside the adjoint kernel
// Most points of a grid whose equal ones count as one in a tile.  Every
// wavefront looks through all points at its start, 80 ns each: with samples
// inside the three-step pass and in launches of their own after single steps,
// us per step, 64 equal points on 1600 x 128 8.8 and 10.3, on 6400 x 256 17.5 and
// 21.6; 256 points 20.8 and 30.6 inside; 4096 points 320 and 435.
constexpr int kMaxEqualExtract = 64;
constexpr int64_t kMaxNr = int64_t(1) << 24;
constexpr int64_t kMaxNth = int64_t(1) << 20;
constexpr int kMinDefaultBlockSteps = 4;  // the default block pass takes at least this many steps a launch

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    int pitch = 0;
    size_t state = 0;                 // bytes of one state [Phi, Pi][nth][pitch]
    size_t off_u[2]{};                // ping-pong state
    size_t off_rad = 0, off_ang = 0, off_x = 0;  // KERR tables; x = r - r_+ at their positions
    size_t off_uci = 0, off_uch = 0;  // USER tables
    size_t off_ext = 0, off_ext2 = 0, off_flag = 0;
    size_t total = 0;
};

int validate(const teuk_params* p) {
    if (!p) return fail(TEUK_E_INVALID_ARG, "params is NULL");
    if (!(p->a >= 0.0 && p->a < 1.0)) return fail(TEUK_E_INVALID_ARG, "spin a=%g outside [0, 1)", p->a);
    if (p->s < -2 || p->s > 2) return fail(TEUK_E_INVALID_ARG, "spin weight s=%d outside [-2, 2]", p->s);
    if (p->m < -1000 || p->m > 1000) return fail(TEUK_E_INVALID_ARG, "m=%d out of range", p->m);
    if (p->nr < 3 || p->nr > kMaxNr) return fail(TEUK_E_INVALID_ARG, "nr=%lld outside [3, 2^24]", (long long)p->nr);
    if (p->ntheta < 2 || p->ntheta > kMaxNth)
        return fail(TEUK_E_INVALID_ARG, "ntheta=%lld outside [2, 2^20]", (long long)p->ntheta);
    if (!std::isfinite(p->rstar_min) || !std::isfinite(p->rstar_max) || !(p->rstar_min < p->rstar_max))
        return fail(TEUK_E_INVALID_ARG, "need finite rstar_min < rstar_max");
    if (!std::isfinite(p->dt)) return fail(TEUK_E_INVALID_ARG, "dt=%g is not finite", p->dt);
    if (!(p->dt > 0.0) && p->coef_mode == TEUK_COEF_USER)
        return fail(TEUK_E_INVALID_ARG, "dt=%g: USER mode needs dt > 0", p->dt);
    if (p->coef_mode != TEUK_COEF_KERR && p->coef_mode != TEUK_COEF_USER)
        return fail(TEUK_E_INVALID_ARG, "coef_mode=%d unknown", p->coef_mode);
    if (p->n_extract < 0 || p->n_extract > kMaxExtract)
        return fail(TEUK_E_INVALID_ARG, "n_extract=%d outside [0, %d]", p->n_extract, kMaxExtract);
    if (p->n_extract > 0 && (!p->extract_rstar || !p->extract_theta))
        return fail(TEUK_E_INVALID_ARG, "extraction coordinates are NULL");
    const double nptr = (double)p->nr * (double)p->ntheta;
    if (nptr > 2.0e9) return fail(TEUK_E_INVALID_ARG, "nr*ntheta too large");
    for (int e = 0; e < p->n_extract; ++e) {
        const double r = p->extract_rstar[e], t = p->extract_theta[e];
        if (!(r >= p->rstar_min && r <= p->rstar_max))
            return fail(TEUK_E_INVALID_ARG, "extraction r*=%g outside the grid", r);
        if (!(t >= 0.0 && t <= M_PI)) return fail(TEUK_E_INVALID_ARG, "extraction theta=%g outside [0, pi]", t);
    }
    return TEUK_OK;
}

Layout make_layout(const teuk_params* p) {
    Layout L;
    const int nr = (int)p->nr, nth = (int)p->ntheta;
    L.pitch = (nr + 7) / 8 * 8;  // 128-byte rows of complex128
    L.state = align_up((size_t)nth * L.pitch * 2 * sizeof(double2));
    size_t o = 0;
    for (int k = 0; k < 2; ++k) {
        L.off_u[k] = o;
        o += L.state;
    }
    L.off_rad = o;
    o += align_up((size_t)kNumSRad * 2 * L.pitch * sizeof(double));
    L.off_ang = o;
    o += align_up((size_t)kNumAng * nth * sizeof(double));
    if (p->coef_mode == TEUK_COEF_KERR) {
        L.off_x = o;
        o += align_up((size_t)2 * L.pitch * sizeof(double));
    }
    if (p->coef_mode == TEUK_COEF_USER) {
        L.off_uci = o;
        o += align_up((size_t)kNumUser * nth * L.pitch * sizeof(double));
        L.off_uch = o;
        o += align_up((size_t)kNumUser * nth * L.pitch * sizeof(double));
    }
    L.off_ext = o;
    o += align_up(std::max(1, p->n_extract) * sizeof(ExtPoint));
    L.off_ext2 = o;
    o += align_up(kMaxExtract * sizeof(ExtPoint));
    L.off_flag = o;
    o += kAlign;
    L.total = o;
    return L;
}

// Bilinear weights of Phi at (r*, theta): columns col, col+1; rows rowa and
// rowb, with the pole ghost rows (sigma times the mirrored row) folded in.
ExtPoint ext_point(double rstar, double theta, double rmin, double dr, int nr, int nth, int sigma) {
    const double dth = M_PI / nth;
    const double pcol = (rstar - rmin) / dr;
    int col = (int)std::floor(pcol);
    col = std::min(std::max(col, 0), nr - 2);
    const double wr = pcol - col;
    const double qrow = theta / dth - 0.5;
    int j = (int)std::floor(qrow);
    j = std::min(std::max(j, -1), nth - 1);
    const double wt = qrow - j;
    ExtPoint E{};
    E.col = col;
    E.wr = wr;
    if (j < 0) {  // rows -1 (ghost of 0) and 0
        E.rowa = 0;
        E.wa = wt + sigma * (1.0 - wt);
        E.rowb = -1;
        E.wb = 0.0;
    } else if (j == nth - 1) {  // rows nth-1 and nth (ghost of nth-1)
        E.rowa = nth - 1;
        E.wa = (1.0 - wt) + sigma * wt;
        E.rowb = -1;
        E.wb = 0.0;
    } else {
        E.rowa = j;
        E.wa = 1.0 - wt;
        E.rowb = j + 1;
        E.wb = wt;
    }
    return E;
}

// Device scratch of teuk_extract_noalloc: the point records of one call,
// staged here instead of in a grid's workspace, so that the call needs no
// device memory from the caller beyond its output.  Every device the
// library runs on holds its own copy until the process ends.  Host code
// reaches a device's copy only through the address hipGetSymbolAddress
// returns for it with that device current (scratch_address), never through
// the array's name, which on the host is only a stand-in for the symbol.
constexpr int kNoAllocMaxPoints = kMaxExtract;
constexpr size_t kScratchBytes = (size_t)kNoAllocMaxPoints * sizeof(ExtPoint);  // 192 KiB
static __device__ __align__(256) char scratch[kScratchBytes];

std::mutex g_scratch_mu;
std::vector<void*> g_scratch_addr;  // by device ordinal; nullptr until resolved

// Resolve the scratch address of `device`, which must be the current device
// (called once per device, from teuk_init_grid).
int resolve_scratch(int device) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (device < 0) return fail(TEUK_E_HIP, "invalid device %d", device);
    if ((size_t)device < g_scratch_addr.size() && g_scratch_addr[device]) return TEUK_OK;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        return fail(TEUK_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", device, hipGetErrorString(e));
    if ((size_t)device >= g_scratch_addr.size()) g_scratch_addr.resize(device + 1, nullptr);
    g_scratch_addr[device] = p;
    return TEUK_OK;
}

void* scratch_address(int device) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return (device >= 0 && (size_t)device < g_scratch_addr.size()) ? g_scratch_addr[device] : nullptr;
}

// The passes that have a tile height of their own: 1, 2, 3 steps, and 3 with a
// source term (its kernel holds one wavefront on a SIMD, the others two).
constexpr int kPassKinds = kMaxPassSteps + 1;
constexpr int pass_kind(int steps, bool source) {
    return steps == kMaxPassSteps && source ? kMaxPassSteps : steps - 1;
}

// The adjoint-side kernels, each with a tile height of its own: one adjoint
// step with the spin gradient from states; one step otherwise; two steps; two
// with the tangents' dot products; the step that stores its tangent; the step
// with its spin derivative.
constexpr int kAdjWaves = 4;  // wavefronts a workgroup until teuk_set_adjoint_tile
enum AdjKind { kAdjStates, kAdjOne, kAdjTwo, kAdjTwoDot, kAdjTangent, kAdjSpinTangent, kAdjKinds };

}  // namespace

struct teuk_grid {
    teuk_params p{};
    std::vector<double> ext_r, ext_t;
    std::vector<ExtPoint> ext;
    Layout L;
    hipStream_t stream = nullptr;
    int device = 0;
    char* ws = nullptr;
    double dr = 0.0, dth = 0.0;
    int sigma = 1;
    int cur = 0;          // which ping-pong buffer holds the state
    int64_t steps = 0;
    int rows = 64;        // theta rows per wavefront tile
    int wpb = 4;          // wavefronts per workgroup
    // the same of the passes of 1, 2, 3 steps and of 3 with a source
    // (teuk_set_tile sets them all)
    int pass_rows[kPassKinds] = {64, 64, 64, 64}, pass_wpb[kPassKinds] = {4, 4, 4, 4};
    int steps_per_pass = 2;  // 2: several steps in one pass (temporal blocking)
    // runs with samples: the passes' tiles, whether they hold a point apiece, and
    // the most steps a pass takes, without and with a source
    int sample_rows[kPassKinds] = {64, 64, 64, 64}, sample_wpb[kPassKinds] = {4, 4, 4, 4};
    bool fused[kPassKinds] = {true, true, true, true};
    int sample_steps[2] = {3, 3};
    int tan_sample_rows = 32;  // the same of the step with its spin derivative
    bool tan_fused = true;
    int cus = 256;
    int block_steps = 0;     // teuk_set_block_launch: steps per launch of the block pass (0: off)
    int block_cols = 0;      // columns a block-pass workgroup holds (0: not set)
    TileShape tile_shape;    // the tile pass's shape and steps per launch (0: off)
    int tile_steps = 0;
    bool default_launch = true;  // tile and block launch as teuk_init_grid chose them
    int default_tile[2] = {0, 0}, default_block[2] = {0, 0};
    int default_rows[kPassKinds] = {}, default_wpb[kPassKinds] = {};
    int64_t check_every = 0;  // teuk_set_finite_check: steps between device checks of the state (0: off)
    char* sws = nullptr;      // source profile (teuk_set_source): [integer, half][nth][pitch] complex128
    bool coef_set = false;
    // adjoint (teuk_enable_adjoint)
    char* aws = nullptr;      // adjoint workspace
    size_t aoff_lam[2]{}, aoff_da = 0, aoff_slots = 0, aoff_sum = 0;
    int adj_rows = 32, adj_wpb = kAdjWaves, adj_strips = 0;  // the tile as teuk_get_adjoint_tile reports it
    int adj_pass_rows[kAdjKinds] = {}, adj_pass_wpb[kAdjKinds] = {};  // the kernels' tiles, and as teuk_init_grid chose them
    int default_adj_rows = 0, default_adj_pass_rows[kAdjKinds] = {}, default_adj_pass_wpb[kAdjKinds] = {};
    TileShape adj_tile;       // adjoint tile pass: shape and steps per launch (0: off)
    int adj_tile_steps = 0;
    bool adj_default = true;  // the adjoint tile is as teuk_init_grid chose it
    int cache_policy = TEUK_CACHE_AUTO;  // teuk_set_cache_policy
    // forward-mode spin derivative (teuk_enable_spin_tangent): v = du/da in two buffers
    char* tws = nullptr;
    int vcur = 0;

    double2* u(int k) const { return reinterpret_cast<double2*>(ws + L.off_u[k]); }
    double2* v(int k) const { return reinterpret_cast<double2*>(tws + (size_t)k * L.state); }
    template <class T>
    T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

namespace {

// What the device builds the grid's tables from: b and c carry dt/dr at the
// half points and half of it at the columns, the rest dt/2 and dt/4 (Stage).
TableArgs table_args(const teuk_grid* g) {
    TableArgs a{};
    a.a = g->p.a;
    a.rmin = g->p.rstar_min;
    a.dr = g->dr;
    a.dth = g->dth;
    for (int kind = 0; kind < 2; ++kind) {
        const double k = kind == 0 ? 0.5 : 1.0;
        a.d[kind] = k * g->p.dt / g->dr;
        a.t[kind] = 0.5 * k * g->p.dt;
    }
    a.nr = (int32_t)g->p.nr;
    a.nth = (int32_t)g->p.ntheta;
    a.pitch = g->L.pitch;
    a.s = g->p.s;
    a.m = g->p.m;
    return a;
}

// The extraction points in the order of a sweep's tiles: by strip of `cols`
// columns, row, and then so that equal ones are neighbours.
std::vector<ExtPoint> tile_order(const teuk_grid* g, int cols) {
    std::vector<std::pair<int64_t, int>> order(g->ext.size());
    for (size_t i = 0; i < order.size(); ++i)
        order[i] = {((int64_t)(g->ext[i].col / cols) << 32) + g->ext[i].rowa, (int)i};
    auto rest = [](const ExtPoint& e) { return std::make_tuple(e.col, e.rowb, e.wr, e.wa, e.wb); };
    std::sort(order.begin(), order.end(), [&](const auto& a, const auto& b) {
        return a.first != b.first ? a.first < b.first : rest(g->ext[a.second]) < rest(g->ext[b.second]);
    });
    std::vector<ExtPoint> E;
    for (const auto& o : order) E.push_back(g->ext[o.second]);
    return E;
}

// Fused extraction handles at most one point per tile (its state is held
// in scalar registers of the tile's wavefront); the forward passes also any
// number of points equal to it (observers that differ in azimuth alone), of
// kMaxEqualExtract points in all.  E: tile_order(g, cols).
bool one_point_a_tile(const std::vector<ExtPoint>& E, int cols, int rows, bool equal_ok) {
    equal_ok = equal_ok && (int)E.size() <= kMaxEqualExtract;
    for (size_t i = 1; i < E.size(); ++i) {
        const ExtPoint &a = E[i - 1], &b = E[i];
        const bool same = a.col == b.col && a.rowa == b.rowa && a.rowb == b.rowb && a.wr == b.wr && a.wa == b.wa && a.wb == b.wb;
        if (a.col / cols == b.col / cols && a.rowa / rows == b.rowa / rows && !(equal_ok && same)) return false;
    }
    return true;
}

// The adjoint passes take up to kRowHits points whose stencils touch a grid
// point: no point may share a row with more at its column or a neighbouring one.
bool fused_adjoint_ok(const teuk_grid* g) {
    const auto& E = g->ext;
    if ((int)E.size() > kMaxFusedAdjointExtract) return false;
    for (const ExtPoint& a : E) {
        int near = 0;
        for (const ExtPoint& b : E) {
            const bool row = a.rowa == b.rowa || a.rowa == b.rowb || (a.rowb >= 0 && (a.rowb == b.rowa || a.rowb == b.rowb));
            if (row && std::abs(a.col - b.col) <= 1) ++near;
        }
        if (near > kRowHits) return false;
    }
    return true;
}

// Two states (a pass's input and output) up to this size stay in the
// last-level cache (256 MB on MI355X) with room to spare for the tables.
constexpr size_t kKeepStatesBytes = (size_t)192 << 20;

// Whether the next state is written with cache-keeping stores.
bool keeps_states(const teuk_grid* g) {
    if (g->cache_policy == TEUK_CACHE_KEEP) return true;
    if (g->cache_policy == TEUK_CACHE_STREAM) return false;
    return 2 * g->L.state <= kKeepStatesBytes;
}

// 1 / x for the factor that undoes a step's own: the product with what a step of
// 1e-310 leaves of a coefficient (zero) has to be zero, not 0 x infinity.
double finite_inverse(double x) { return std::min(1.0 / x, std::numeric_limits<double>::max()); }

StepArgs step_args(const teuk_grid* g) {
    StepArgs a{};
    StepScalars& k = a.k;
    k.nr = (int)g->p.nr;
    k.nth = (int)g->p.ntheta;
    k.pitch = g->L.pitch;
    k.sigma = g->sigma;
    k.rows = g->rows;
    k.n_chunks = (k.nth + g->rows - 1) / g->rows;
    k.hdt = 0.5 * g->p.dt;
    k.qdt = 0.25 * g->p.dt;
    k.kap_h = finite_inverse(k.hdt);
    k.kap_i = finite_inverse(k.qdt);
    k.dt_dr = g->p.dt / g->dr;
    k.hdt_dr = 0.5 * g->p.dt / g->dr;
    k.inv_dth2 = 1.0 / (g->dth * g->dth);
    k.inv_2dth = 1.0 / (2.0 * g->dth);
    k.plane = (int64_t)k.nth * k.pitch;
    a.rad = g->at<double>(g->L.off_rad);
    a.ang = g->at<double>(g->L.off_ang);
    if (g->p.coef_mode == TEUK_COEF_USER) {
        a.uci = g->at<double>(g->L.off_uci);
        a.uch = g->at<double>(g->L.off_uch);
    }
    a.ext = g->at<ExtPoint>(g->L.off_ext);
    k.keep = keeps_states(g) ? 1 : 0;
    return a;
}

// Launch arguments of a pass of `steps` steps.  XCD runs of strips where each
// XCD gets at least 8 (measured: 0.6-0.8 % faster on 25600 x 512 at 32-64 row
// tiles, neutral on 6400 x 256).
StepArgs pass_args(const teuk_grid* g, int steps, bool source, bool sample) {
    const int kind = pass_kind(steps, source);
    StepArgs a = step_args(g);
    a.k.n_strips = (a.k.nr + strip_cols(steps) - 1) / strip_cols(steps);
    a.k.rows = sample ? g->sample_rows[kind] : g->pass_rows[kind];
    a.k.n_chunks = (a.k.nth + a.k.rows - 1) / a.k.rows;
    a.k.n_ext = sample ? g->p.n_extract : 0;
    a.k.order = steps > 1 && a.k.n_strips >= 64 ? kTileOrderXcdStrip : kTileOrderDispatch;
    return a;
}

int check_grid(const teuk_grid* g) {
    if (!g) return fail(TEUK_E_INVALID_ARG, "grid handle is NULL");
    return TEUK_OK;
}

// Bytes of one plane of the source profile ([nth][pitch] complex128).
size_t source_plane_bytes(const teuk_grid* g) { return align_up((size_t)g->p.ntheta * g->L.pitch * sizeof(double2)); }

// Status block of the workspace: [int] non-finite flag of teuk_check_finite,
// then at byte 8 the step count recorded by the first failing in-loop check
// (0: none).
long long* first_nonfinite(const teuk_grid* g) { return reinterpret_cast<long long*>(g->ws + g->L.off_flag + 8); }

// Default tile as teuk_get_tile reports it (until teuk_set_tile, the passes
// take their own heights), that of a two-step pass.  The device holds two of its wavefronts
// per SIMD, so its tiles run in rounds of 8 x CUs; a last round that is only
// partly filled leaves SIMDs idle, and a wavefront walks its tile's rows one
// after the other, so on a grid that fits one round shorter tiles finish
// sooner.  Take the fewest rounds k whose tiles, cut so that the grid's tiles
// just fit k rounds, have at most 64 rows.  Grids with fewer tiles than SIMDs
// take one wavefront per workgroup, to spread over the CUs.
void default_tile(int nr, int nth, int cus, int* rows, int* wpb) {
    const int64_t strips2 = (nr + kStripCols2 - 1) / kStripCols2;
    const int64_t slots = (int64_t)cus * 8;
    int64_t r = 64;
    for (int64_t k = 1; k <= 64; ++k) {
        const int64_t chunks = k * slots / strips2;
        if (chunks < 1) continue;
        const int64_t rk = (nth + chunks - 1) / chunks;
        if (rk <= 64) {
            r = rk;
            break;
        }
    }
    r = std::min<int64_t>(r, nth);
    const int64_t tiles = strips2 * ((nth + r - 1) / r);
    *rows = (int)r;
    *wpb = tiles < (int64_t)cus * 4 ? 1 : 4;
}

// What a sweep's tile height is chosen from, by kernel.  A wavefront walks its
// tile's rows one after the other: `steps` rows to fill the steps, then the
// tile's rows and `steps` more, in groups of `group`, after a start (tables and
// first rows) worth about three rows, `start2` where wavefronts overlap in it.
struct SweepCost {
    int steps, group;
    int waves;         // wavefronts a SIMD holds; two share its issue:
    double alone;      // a row takes 2 units of time beside another one, `alone` units without
    double start2;
    bool longer;       // of heights that cost the same the longer (fewer tiles); otherwise
                       // the shorter where the tiles have a SIMD each
    double us0, us;    // us of a pass: us0 + us for each unit of time (0: not used)
    double us_alone;   // (the same where the tiles have a SIMD each)
};

// Forward passes: of one and two steps; of three steps; with a source.
// Measured, us per step by rows: one step, 1600 x 128 at 2 / 4 / 5 rows 9.5 /
// 7.5 / 8.2, 6400 x 256 at 8 / 15 / 27 rows 21.8 / 19.8 / 19.2; two steps (store
// runs), 3200 x 128 at 4 / 7 / 9 rows 7.7 / 6.9 / 7.4; three steps, 6400 x 256
// at 15 / 17 / 29 rows 13.3 / 12.2 / 12.3, 5003 x 197 at 9 / 10 / 13 rows 9.6 /
// 10.9 / 10.1, 25600 x 512 at 57 / 103 rows 68 / 86.
constexpr SweepCost kForward[kPassKinds] = {{1, 1, 2, 1.2, 3.0, true, 4.1, 0.36, 0.38},
                                            {2, 1, 2, 1.2, 3.0, true, 2.8, 0.75, 0.75},
                                            {3, 4, 2, 1.3, 2.0, false, 8.4, 0.65, 0.5},
                                            {3, 4, 1, 1.3, 2.0, false, 3.2, 0.81, 0.91}};
// Adjoint-side kernels, in the order of AdjKind.
// Measured, us per step by rows: from states, 3200 x 128 at 4 / 5 / 7 rows 18.5 /
// 21.4 / 20.6, 1600 x 64 at 1 / 2 / 3 rows 11.8 / 10.2 / 12.3; one step, 1600 x
// 128 at 2 / 4 / 8 rows 8.2 / 6.8 / 8.2; two steps, 6400 x 256 at 9 / 14 / 29
// rows 16.0 / 14.9 / 18.2; with dot products 28.3 / 22.7 / 21.0; the step that
// stores its tangent, 1600 x 64 at 1 / 2 / 3 rows 8.6 / 7.1 / 7.8; the step with
// its spin derivative, 1600 x 64 9.6 / 8.3 / 10.5, 6400 x 256 at 15 / 17 / 29 rows
// 42.2 / 43.5 / 38.7.
constexpr SweepCost kAdjoint[kAdjKinds] = {{1, 1, 2, 1.4, 3.0, true, 0.0, 0.0, 0.0},
                                           {1, 1, 2, 1.3, 3.0, true, 0.0, 0.0, 0.0},
                                           {2, 1, 2, 1.3, 3.0, true, 3.4, 0.725, 0.725},
                                           {2, 1, 2, 1.0, 3.0, true, 0.0, 0.0, 0.0},
                                           {1, 1, 2, 1.2, 3.0, true, 0.0, 0.0, 0.0},
                                           {1, 1, 2, 1.0, 3.0, true, 4.9, 0.89, 1.08}};

// The tile height of the lowest cost, at most 128 rows, of those that ok(rows)
// allows (0 if none); us: the estimated time of a step.  Tiles beyond one round
// of wavefronts wait for a slot; with several rounds the last, partly filled
// one counts for less.
template <class Ok>
int sweep_rows(int nr, int nth, int cus, const SweepCost& c, double* us, Ok ok) {
    const int cols = strip_cols(c.steps);
    const int64_t strips = (nr + cols - 1) / cols;
    double best = 0.0;
    int rows = 0;
    for (int r = 1; r <= std::min(nth, 128); ++r) {
        if (!ok(r)) continue;
        const double x = (double)(strips * ((nth + r - 1) / r)) / (4.0 * cus);  // tiles per SIMD
        const int its = c.steps + (r + c.steps + c.group - 1) / c.group * c.group;
        double f = c.alone, rounds = 1.0;
        if (x > 1.0 && c.waves == 1) {
            rounds = std::ceil(x);
            f = c.alone * (x + (rounds - x) / std::max(1.0, rounds - 1.0));
        } else if (x > 1.0) {
            rounds = std::ceil(0.5 * x);
            const double over = x - 2.0 * (rounds - 1.0);
            const double whole = 2.0 * (rounds - 1.0) + (over > 1.0 ? 2.0 : c.alone);
            f = x + (whole - x) / std::max(1.0, rounds - 1.0);
        }
        const double t = (x > 1.0 && c.waves > 1 ? c.start2 : 3.0) * rounds + its * f;
        if (rows == 0 || t < best || (t == best && (x > 1.0 || c.longer))) {
            best = t;
            rows = r;
            if (us) *us = (c.us0 + (x > 1.0 ? c.us : c.us_alone) * its * f) / c.steps;
        }
    }
    return rows;
}

int sweep_rows(int nr, int nth, int cus, const SweepCost& c, double* us = nullptr) {
    return sweep_rows(nr, nth, cus, c, us, [](int) { return true; });
}

// Wavefronts a workgroup of a sweep: four, or one, to spread few tiles over the CUs.
int sweep_waves(int nr, int nth, int cus, int steps, int rows) {
    const int64_t tiles = (int64_t)((nr + strip_cols(steps) - 1) / strip_cols(steps)) * ((nth + rows - 1) / rows);
    return tiles < (int64_t)cus * 4 ? 1 : 4;
}

// A launch that samples between passes, per state, besides the passes' own time.
constexpr double kExtractUs = 2.5;

// The tiles of runs with samples, after a change of the tiles: a pass's own
// where each holds a point at most.  Otherwise, where the heights are the
// grid's choice, the best ones among those that part the points, and as many
// steps a pass as are estimated fastest with them, single steps with launches
// that sample among the choices.  (Two observers of one strip at rows 12 and 14,
// us per step in single steps, as their shared tile has it at the passes' own
// heights, and with the points parted: 6400 x 256 24.0 and 14.4, 5003 x 197 17.8
// and 10.5, 25600 x 512 172 and 87.)
void update_fusion(teuk_grid* g) {
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    const bool choose = g->rows == g->default_tile[0] && g->wpb == g->default_tile[1];
    double us[kPassKinds] = {};
    bool own[kPassKinds] = {};
    for (int i = 0; i < kPassKinds; ++i) {
        const int steps = kForward[i].steps, cols = strip_cols(steps);
        const std::vector<ExtPoint> E = tile_order(g, cols);
        g->sample_rows[i] = g->pass_rows[i];
        g->sample_wpb[i] = g->pass_wpb[i];
        own[i] = g->fused[i] = one_point_a_tile(E, cols, g->pass_rows[i], true);
        if (own[i] || !choose) continue;
        const int r = sweep_rows(nr, nth, g->cus, kForward[i], &us[i],
                                 [&](int rows) { return one_point_a_tile(E, cols, rows, true); });
        if (r == 0) continue;
        g->fused[i] = true;
        g->sample_rows[i] = r;
        g->sample_wpb[i] = sweep_waves(nr, nth, g->cus, steps, r);
    }
    // single steps: sampling inside or not, whichever is estimated faster
    double single_us = 0.0;
    sweep_rows(nr, nth, g->cus, kForward[0], &single_us);
    if (!own[0] && choose) {
        single_us += kExtractUs;
        if (g->fused[0] && us[0] < single_us) {
            single_us = us[0];
        } else {
            g->fused[0] = false;
        }
    }
    if (own[1]) sweep_rows(nr, nth, g->cus, kForward[1], &us[1]);
    for (int source = 0; source < 2; ++source) {
        const int three = pass_kind(3, source != 0);
        int& steps = g->sample_steps[source];
        steps = g->fused[three] ? 3 : g->fused[1] ? 2 : 1;
        if (!choose || own[three]) continue;
        // The estimates know no memory: passes of fewer steps, which move more of
        // it, have to be estimated the faster by a margin.  (With a source one
        // and two steps take 1.3 times their estimates: 6400 x 256 23.5 and 17.2.)
        const double f = source ? 1.3 : 1.0;
        if (steps == 3 && g->fused[1] && us[three] > 1.15 * f * us[1]) steps = 2;
        if (steps > 1 && us[steps == 3 ? three : 1] * (steps == 3 ? 1.0 : f) > 1.5 * f * single_us) steps = 1;
    }
    // the step with its spin derivative, which samples two series
    const SweepCost& c = kAdjoint[kAdjSpinTangent];
    const int cols = strip_cols(c.steps);
    const std::vector<ExtPoint> E = tile_order(g, cols);
    g->tan_sample_rows = g->adj_pass_rows[kAdjSpinTangent];
    g->tan_fused = one_point_a_tile(E, cols, g->tan_sample_rows, false);
    if (!g->tan_fused && g->adj_default) {
        double fused_us = 0.0, plain_us = 0.0;
        sweep_rows(nr, nth, g->cus, c, &plain_us);
        const int r = sweep_rows(nr, nth, g->cus, c, &fused_us, [&](int rows) { return one_point_a_tile(E, cols, rows, false); });
        if (r > 0 && fused_us < plain_us + 2.0 * kExtractUs) {
            g->tan_fused = true;
            g->tan_sample_rows = r;
        }
    }
}

// Shape and steps per launch of the tile pass with the lowest estimated time
// per step, which is returned (us); 0 steps if no shape applies.  A launch
// costs 2.5 us before its first workgroup; a workgroup starts (loads, builds
// its coefficients) and takes its steps, and with more workgroups than the
// device holds at once they run in rounds.  Measured: a step takes 0.54 us
// with one row a lane and two wavefronts a SIMD, 0.87 with four, 1.13 with
// three rows and two; a launch of 256 workgroups 5.7, 7.5 and 7.1 us besides.
// Estimate and measurement (us per step): 400 x 32 1.28 and 1.27, 1600 x 128
// 2.97 and 3.05, 3200 x 128 5.4 and 5.2, 1200 x 100 2.2 and 2.0; adjoint (three
// points) 1200 x 100 2.5 and 2.5, 3200 x 128 5.6 and 6.1, 5003 x 197 13.1 and
// 13.8 (sweeps: 7.1, 10.7, 16.7).  work: instructions per step, the forward's as 1.
double best_tile(int nr, int nth, int cus, double work, TileShape* shape, int* steps) {
    struct Kind {
        int cols, rows, most, per_cu;  // most wavefronts a workgroup and a CU
        double us;                     // per row and wavefront of a SIMD
    };
    constexpr Kind kinds[] = {{16, 1, 16, 20, 0.155}, {32, 1, 16, 20, 0.155}, {64, 1, 16, 20, 0.155},
                              {32, 2, 8, 8, 0.14},    {64, 2, 8, 8, 0.14},    {64, 3, 8, 8, 0.145}};
    double best = 0.0;
    *steps = 0;
    for (const Kind& c : kinds)
        for (int waves = 1; waves <= c.most; ++waves) {
            const int per = kWave / c.cols, rows = waves * per * c.rows;
            if (rows > nth && (c.rows != 1 || rows - per >= nth)) continue;
            for (int k = 1; k <= (c.cols - 2) / 2; ++k) {
                int chunks = 1;
                if (rows < nth) {
                    if (rows - 2 * k < 1) break;
                    chunks = 2 + std::max(0, (nth - 2 * (rows - k) + rows - 2 * k - 1) / (rows - 2 * k));
                }
                const int w = c.cols - 2 * k;
                const int64_t groups = (int64_t)((nr + w - 1) / w) * chunks;
                const int64_t at_once = (groups + cus - 1) / cus;  // per CU
                const int held = (int)std::min<int64_t>(at_once, std::max(1, c.per_cu / waves));
                const double rounds = std::ceil((double)groups / ((double)cus * held));
                const double load = c.rows * std::max(1.0, 0.25 * waves), all = c.rows * std::max(1.0, 0.25 * waves * held);
                const double t = (2.5 + rounds * ((1.5 + 0.35 * load) * held + 1.3 * std::min(1.0, (double)groups / cus) +
                                                  k * (0.25 + work * c.us * all))) / k;
                if (*steps == 0 || t < best) {
                    best = t;
                    *steps = k;
                    shape->cols = c.cols;
                    shape->rows = c.rows;
                    shape->waves = waves;
                }
            }
        }
    return best;
}

// Default tile height of an adjoint kernel: the shortest tiles of which
// `slots` wavefronts hold all (workgroups take consecutive tiles of the
// strip-major list, so any tile count packs), at most 16 rows.
int adjoint_rows(int nr, int nth, int64_t slots, int strip_cols) {
    const int64_t strips = (nr + strip_cols - 1) / strip_cols;
    const int64_t chunks = slots / strips;  // theta chunks per strip
    if (chunks < 1) return std::min(nth, 16);
    return (int)std::min<int64_t>(std::min<int64_t>((nth + chunks - 1) / chunks, 16), nth);
}

int set_device(const teuk_grid* g) {
    int cur = -1;
    HIP_TRY(hipGetDevice(&cur));
    if (cur != g->device) HIP_TRY(hipSetDevice(g->device));
    return TEUK_OK;
}

// Gershgorin bound of the largest |eigenvalue| of the discrete theta operator
// (rows of A2 (f+ - 2 f + f-)/dth^2 + A1 (f+ - f-)/(2 dth) - V0 f, ghost rows
// folded in) over all integer columns.
double angular_eig_bound(const teuk_params* p, double dr) {
    const int nr = (int)p->nr, nth = (int)p->ntheta;
    const double dth = M_PI / nth;
    const int sigma = (std::abs(p->m) % 2 == 0) ? 1 : -1;
    std::vector<double> ang((size_t)nth * kNumAng);
    for (int j = 0; j < nth; ++j) angular_fields(p->s, p->m, j, dth, &ang[(size_t)j * kNumAng]);
    double best = 0.0;
    for (int i = 0; i < nr; ++i) {
        double x;
        if (!tortoise_inverse(p->a, p->rstar_min + i * dr, &x)) continue;
        double R[kNumSRad];
        stage_fields<double>(p->a, p->s, p->m, x, dth, 1.0, 1.0, R);
        for (int j = 0; j < nth; ++j) {
            const double* G = &ang[(size_t)j * kNumAng];
            const double inv = 1.0 / (R[S_RHO2] - R[S_A2D] * G[A_SN2]);
            const double a2 = R[S_DL2] * inv, a1 = a2 * G[A_COTP];
            const double v0 = std::hypot((R[S_DL2] * G[A_PD] + R[S_VR]) * inv, R[S_VI] * inv);
            double lo = a2 - a1, hi = a2 + a1, diag = -2.0 * a2;  // weights of f-, f+, f
            if (j == 0) diag += sigma * lo, lo = 0.0;
            if (j == nth - 1) diag += sigma * hi, hi = 0.0;
            best = std::max(best, std::fabs(diag) + v0 + std::fabs(lo) + std::fabs(hi));
        }
    }
    return best;
}

}  // namespace

extern "C" {

const char* teuk_last_error(void) { return g_last_error.c_str(); }

size_t teuk_workspace_bytes(const teuk_params* p) {
    if (validate(p) != TEUK_OK) return 0;
    return make_layout(p).total;
}

int teuk_radius(double a, double rstar, double* h_r) {
    if (!(a >= 0.0 && a < 1.0)) return fail(TEUK_E_INVALID_ARG, "spin a=%g outside [0, 1)", a);
    if (!std::isfinite(rstar) || !h_r) return fail(TEUK_E_INVALID_ARG, "need a finite r* and an output pointer");
    double x;
    if (!tortoise_inverse(a, rstar, &x)) return fail(TEUK_E_INVALID_ARG, "tortoise inversion failed at r*=%g", rstar);
    *h_r = 1.0 + std::sqrt(1.0 - a * a) + x;
    return TEUK_OK;
}

int teuk_suggest_dt(const teuk_params* p, int64_t n_steps, double growth, double courant, double* h_dt) {
    if (validate(p) != TEUK_OK) return TEUK_E_INVALID_ARG;
    if (!h_dt) return fail(TEUK_E_INVALID_ARG, "h_dt is NULL");
    if (n_steps < 1 || !(growth > 1.0) || !(courant > 0.0))
        return fail(TEUK_E_INVALID_ARG, "need n_steps >= 1, growth > 1, courant > 0");
    const double dr = (p->rstar_max - p->rstar_min) / (double)(p->nr - 1);
    const double w = std::sqrt(angular_eig_bound(p, dr));
    double dt = courant * dr;
    if (w > 0.0) dt = std::min(dt, std::pow(8.0 * std::log(growth) / (double)n_steps, 0.25) / w);
    *h_dt = dt;
    return TEUK_OK;
}

namespace {

// The grid's time step: the policy step for dt <= 0, the strict-mode check
// for dt > 0 with a horizon (see teuk_params in teuk.h).
constexpr int64_t kPolicySteps = 10000;
constexpr double kPolicyGrowth = 10.0;

int resolve_dt(const teuk_params* p, double* dt) {
    *dt = p->dt;
    if (p->coef_mode != TEUK_COEF_KERR) return TEUK_OK;
    const int64_t n = p->stable_steps > 0 ? p->stable_steps : kPolicySteps;
    if (!(p->dt > 0.0)) return teuk_suggest_dt(p, n, kPolicyGrowth, 0.5, dt);
    if (p->stable_steps > 0) {
        double bound = 0.0;
        if (int rc = teuk_suggest_dt(p, n, kPolicyGrowth, 1.0, &bound)) return rc;
        if (p->dt > bound)
            return fail(TEUK_E_UNSTABLE_DT,
                        "dt=%g exceeds %g: the fastest angular mode would grow more than %gx over %lld steps "
                        "(or the r* Courant number exceed 1)",
                        p->dt, bound, kPolicyGrowth, (long long)n);
    }
    return TEUK_OK;
}

}  // namespace

int teuk_init_grid(const teuk_params* p, void* hip_stream, void* d_workspace, size_t workspace_bytes,
                   teuk_grid** out) {
    if (int rc = validate(p)) return rc;
    double dt = 0.0;
    if (int rc = resolve_dt(p, &dt)) return rc;
    if (!out) return fail(TEUK_E_INVALID_ARG, "out is NULL");
    if (!d_workspace) return fail(TEUK_E_INVALID_ARG, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(d_workspace) % kAlign)
        return fail(TEUK_E_WORKSPACE, "workspace not %zu-byte aligned", kAlign);
    const Layout L = make_layout(p);
    if (workspace_bytes < L.total)
        return fail(TEUK_E_WORKSPACE, "workspace has %zu bytes, needs %zu", workspace_bytes, L.total);

    const int nr = (int)p->nr, nth = (int)p->ntheta;
    const double dr = (p->rstar_max - p->rstar_min) / (double)(nr - 1);
    const double dth = M_PI / nth;

    teuk_grid* g = new teuk_grid();
    g->p = *p;
    g->p.dt = dt;
    g->L = L;
    g->stream = reinterpret_cast<hipStream_t>(hip_stream);
    g->ws = reinterpret_cast<char*>(d_workspace);
    g->dr = dr;
    g->dth = dth;
    g->sigma = (std::abs(p->m) % 2 == 0) ? 1 : -1;
    int cus = 0;
    double sweep_us = 0.0;  // estimated time of a step by the three-step pass
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        g->cus = cus;
        default_tile(nr, nth, cus, &g->rows, &g->wpb);
        // Each pass on a tile of its own: the strips of a pass of k steps are
        // 64 - 2 k columns, and the rows that fill the chip once differ.  With
        // the one-step pass's rows for all, source runs of 6400 x 256 (steps in
        // pairs) took 18.8 us a step, with their own 16.8; three steps a pass
        // with the rows of the pass without a source 18.7, with their own 15.4.
        for (int i = 0; i < kPassKinds; ++i) {
            const int k = kForward[i].steps;
            const int r = sweep_rows(nr, nth, cus, kForward[i], k == i + 1 ? &sweep_us : nullptr);
            g->pass_rows[i] = g->default_rows[i] = r;
            g->pass_wpb[i] = g->default_wpb[i] = sweep_waves(nr, nth, cus, k, r);
        }
    }
    // The block pass: one thread per point of (columns x all rows).  Default
    // launch: over workgroups of up to 256, 512 or 1024 threads (at most 64
    // columns), the most steps a launch (at least 4) whose workgroups fit the
    // device one per CU, scored by the per-step time measured on small grids
    // (400 x 16 .. 3200 x 32, 1600 x 64): about 0.8 ns per point a workgroup
    // holds plus 3.6 us per launch spread over its steps.
    if (nth <= kMaxBlockRows && g->p.coef_mode == TEUK_COEF_KERR) {
        double best = 0.0;
        for (int threads : {256, 512, 1024}) {
            const int c = std::min(64, threads / nth);
            if (c < 2 * kMinDefaultBlockSteps + 2) continue;
            for (int k = (c - 2) / 2; k >= kMinDefaultBlockSteps; --k) {
                const int64_t w = c - 2 * k;
                if ((nr + w - 1) / w > cus) continue;
                const double score = 0.8e-3 * c * nth + 3.6 / k;  // us per step
                if (g->block_steps == 0 || score < best) {
                    best = score;
                    g->block_steps = k;
                    g->block_cols = c;
                }
                break;  // the most steps for this width
            }
        }
    }
    // the tile pass where its estimate is below the sweeps'
    if (p->coef_mode == TEUK_COEF_KERR && best_tile(nr, nth, cus, 1.0, &g->tile_shape, &g->tile_steps) >= sweep_us)
        g->tile_steps = 0;
    g->default_tile[0] = g->rows;
    g->default_tile[1] = g->wpb;
    g->default_block[0] = g->block_steps;
    g->default_block[1] = g->block_cols;
    // The adjoint tile as it is reported; the kernels take heights of their own
    // until teuk_set_adjoint_tile.
    g->adj_rows = adjoint_rows(nr, nth, (int64_t)cus * 7, kStripCols);
    // (Wavefronts whose lanes hold their own factors go one to a workgroup while
    // there are few, the others share the workgroup's tables: us per step with
    // four and one, the step that stores its tangent 200 x 16 5.8 and 4.7, 400 x 32
    // 6.0 and 4.9; one cotangent step 5.4 and 4.7; with the spin gradient from
    // states 8.6 and 11.8.)
    for (int i = 0; i < kAdjKinds; ++i) {
        const int r = sweep_rows(nr, nth, cus, kAdjoint[i], i == kAdjTwo ? &sweep_us : nullptr);
        const bool own = i == kAdjOne || i == kAdjTangent;
        g->adj_pass_rows[i] = g->default_adj_pass_rows[i] = r;
        g->adj_pass_wpb[i] = g->default_adj_pass_wpb[i] = own ? sweep_waves(nr, nth, cus, kAdjoint[i].steps, r) : kAdjWaves;
    }
    g->default_adj_rows = g->adj_rows;
    // (the adjoint tile pass: 1.17 times the forward one's instructions.  us per
    // step, tile pass and sweeps: 2000 x 256 7.2 and 8.1, 12000 x 64 10.3 and 9.9,
    // 4000 x 200 10.4 and 9.8, 5003 x 197 12.9 and 11.1)
    if (best_tile(nr, nth, cus, 1.17, &g->adj_tile, &g->adj_tile_steps) >= 0.95 * sweep_us) g->adj_tile_steps = 0;
    g->adj_strips = ((int)p->nr + kStripCols - 1) / kStripCols;
    g->ext_r.assign(p->extract_rstar, p->extract_rstar + p->n_extract);
    g->ext_t.assign(p->extract_theta, p->extract_theta + p->n_extract);
    g->p.extract_rstar = g->ext_r.data();
    g->p.extract_theta = g->ext_t.data();
    for (int e = 0; e < p->n_extract; ++e)
        g->ext.push_back(ext_point(g->ext_r[e], g->ext_t[e], p->rstar_min, dr, nr, nth, g->sigma));
    update_fusion(g);
    g->coef_set = p->coef_mode == TEUK_COEF_KERR;

    auto bail = [&](int rc) {
        delete g;
        return rc;
    };
    hipError_t e = hipGetDevice(&g->device);
    if (e != hipSuccess) return bail(fail(TEUK_E_HIP, "hipGetDevice: %s", hipGetErrorString(e)));
    if (int rc = resolve_scratch(g->device)) return bail(rc);
    hipStream_t s = g->stream;
    e = hipMemsetAsync(g->ws, 0, L.off_rad, s);  // both state buffers
    if (e == hipSuccess) e = hipMemsetAsync(g->ws + L.off_flag, 0, kAlign, s);  // status flags
    // The tables, built on the device; the status block's third word tells of
    // a position without an r.
    const bool kerr = p->coef_mode == TEUK_COEF_KERR;
    int* d_failed = g->at<int>(L.off_flag + 16);
    int failed = 0;
    if (e == hipSuccess)
        e = launch_tables(table_args(g), kerr ? g->at<double>(L.off_x) : nullptr,
                          kerr ? g->at<double>(L.off_rad) : nullptr, g->at<double>(L.off_ang), d_failed, s);
    if (e == hipSuccess && kerr) e = hipMemcpyAsync(&failed, d_failed, sizeof(failed), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && !g->ext.empty())
        e = hipMemcpyAsync(g->ws + L.off_ext, g->ext.data(), g->ext.size() * sizeof(ExtPoint),
                           hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bail(fail(TEUK_E_HIP, "building tables: %s", hipGetErrorString(e)));
    if (failed) return bail(fail(TEUK_E_INVALID_ARG, "tortoise inversion failed on the grid's r* range"));
    *out = g;
    return TEUK_OK;
}

int teuk_set_coefficients(teuk_grid* g, const double* d_ci, const double* d_ch) {
    if (int rc = check_grid(g)) return rc;
    if (g->p.coef_mode != TEUK_COEF_USER) return fail(TEUK_E_STATE, "grid is not in TEUK_COEF_USER mode");
    if (!d_ci || !d_ch) return fail(TEUK_E_INVALID_ARG, "coefficient pointers are NULL");
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_pitch_copy(d_ci, g->at<double>(g->L.off_uci), kNumUser * nth, nr, g->L.pitch, g->stream));
    HIP_TRY(launch_pitch_copy(d_ch, g->at<double>(g->L.off_uch), kNumUser * nth, nr - 1, g->L.pitch, g->stream));
    g->coef_set = true;
    return TEUK_OK;
}

int teuk_set_initial_data(teuk_grid* g, const void* d_phi, const void* d_pi) {
    if (int rc = check_grid(g)) return rc;
    if (!d_phi || !d_pi) return fail(TEUK_E_INVALID_ARG, "initial data pointers are NULL");
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_import(static_cast<const double2*>(d_phi), static_cast<const double2*>(d_pi), g->u(0),
                          nr, nth, g->L.pitch, g->stream));
    g->cur = 0;
    g->steps = 0;
    return TEUK_OK;
}

namespace {

// Optional device check of the state every check_every steps (at the first
// pass boundary at or after each multiple) and at the end of a call: the
// first check that finds a non-finite value records its step count on the
// device; the call reads it once, at its end.
struct InLoopCheck {
    teuk_grid* g;
    long long* first_bad;
    int64_t start, last_check, next_check;
    explicit InLoopCheck(teuk_grid* grid)
        : g(grid), first_bad(first_nonfinite(grid)), start(grid->steps), last_check(grid->steps),
          next_check(grid->steps + grid->check_every) {}
    int check(const double2* u) {
        HIP_TRY(launch_nonfinite_step(u, (int)g->p.nr, (int)g->p.ntheta, g->L.pitch, first_bad, g->steps,
                                      g->stream));
        last_check = g->steps;
        return TEUK_OK;
    }
    int maybe(const double2* u) {
        if (g->check_every <= 0 || g->steps < next_check) return TEUK_OK;
        next_check = start + ((g->steps - start) / g->check_every + 1) * g->check_every;
        return check(u);
    }
    // u: the state after the call's last step
    int finish(const double2* u) {
        if (g->check_every <= 0) return TEUK_OK;
        if (last_check != g->steps)
            if (int rc = check(u)) return rc;
        long long bad = 0;
        HIP_TRY(hipMemcpyAsync(&bad, first_bad, sizeof(bad), hipMemcpyDeviceToHost, g->stream));
        HIP_TRY(hipStreamSynchronize(g->stream));
        if (bad) {
            HIP_TRY(launch_zero_ints(reinterpret_cast<int*>(first_bad), 2, g->stream));
            return fail(TEUK_E_NONFINITE, "the state holds a non-finite value, first seen by the check after step %lld",
                        bad);
        }
        return TEUK_OK;
    }
};

// How the steps of a run go: launches of the tile pass, or of the block pass, or
// sweeps.
struct RunPlan {
    bool tile, block;
    bool three, two;  // sweeps take three, two steps a pass (single ones always)
    bool fused1;      // a single step samples its input
};

// The tile pass is for Kerr coefficients, neither a window, a source nor a
// check between steps, and a series of no more points than it samples; so is
// the block pass, which may check.  Sweeps run several steps to a pass: three
// where the pass has a kernel for it (Kerr coefficients, no window, three rows
// or more) and no check falls between them.
RunPlan run_plan(const teuk_grid* g, bool series, bool source, bool window) {
    const bool kerr = g->p.coef_mode == TEUK_COEF_KERR, multi = g->steps_per_pass == 2;
    const bool in_launch = kerr && !window && !source && (!series || g->p.n_extract <= kMaxBlockExt);
    RunPlan p{};
    p.tile = in_launch && multi && g->tile_steps > 0 && g->default_launch && g->check_every == 0;
    p.block = in_launch && g->block_steps > 0;
    const int most = series ? g->sample_steps[source] : kMaxPassSteps;
    // user coefficients and a source at once leave the two-step pass no registers
    // to load them ahead: single steps on small grids (us per step, pairs and
    // single: 800 x 48 9.1 and 6.1, 1200 x 100 14.0 and 12.3, 1600 x 128 15.1 and
    // 13.8, 3200 x 128 18.5 and 19.1, 6400 x 256 53 and 75)
    const bool single = !kerr && source && g->p.nr * g->p.ntheta <= kMaxSingleUserSource;
    p.two = multi && most >= 2 && !single && (!series || g->fused[1]);
    p.three = multi && most == 3 && kerr && !window && g->p.ntheta >= 3 && g->check_every == 0;
    p.fused1 = g->fused[0];
    return p;
}

// Whether cotangents go by the adjoint tile pass.
bool adjoint_on_tiles(const teuk_grid* g) {
    return g->adj_tile_steps > 0 && g->adj_default && g->steps_per_pass == 2 && g->p.n_extract <= kMaxBlockExt;
}

// n steps; optional extraction series and optional window of input states
// (slot k = the state before step k, stride L.state bytes); h_f: the time
// factors of the source term for the n steps (4 doubles per step), or
// nullptr for the homogeneous equation.
int step_n_impl(teuk_grid* g, int64_t n, void* d_series, void* d_window, const double* h_f = nullptr) {
    if (int rc = check_grid(g)) return rc;
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (!g->coef_set) return fail(TEUK_E_STATE, "USER-mode coefficients not set");
    if (n == 0) return TEUK_OK;
    if (int rc = set_device(g)) return rc;
    const int ne = g->p.n_extract;
    double2* series = (ne > 0) ? static_cast<double2*>(d_series) : nullptr;
    const bool kerr = g->p.coef_mode == TEUK_COEF_KERR;
    StepArgs args[kMaxPassSteps];
    for (int m = 1; m <= kMaxPassSteps; ++m) {
        StepArgs& a = args[m - 1];
        a = pass_args(g, m, h_f != nullptr, series && g->fused[pass_kind(m, h_f != nullptr)]);
        if (h_f) {
            a.src_i = reinterpret_cast<const double2*>(g->sws);
            a.src_h = reinterpret_cast<const double2*>(g->sws + source_plane_bytes(g));
        }
    }
    const ExtPoint* ext = g->at<ExtPoint>(g->L.off_ext);
    char* win = static_cast<char*>(d_window);
    auto window_state = [&](int64_t k) { return reinterpret_cast<double2*>(win + (size_t)k * g->L.state); };
    // Without a window the state ping-pongs between the grid's two buffers.
    // With one, state k (0 < k < n) is written straight into window slot k,
    // the first step copies the grid's state into slot 0 on the way, and the
    // last step writes the grid's other buffer: no state is written twice.
    const int cur0 = g->cur;
    int cur = cur0;
    double2* in = g->u(cur0);
    auto next_buffer = [&](int64_t knext) -> double2* {
        if (win) return (knext < n) ? window_state(knext) : g->u(1 - cur0);
        return g->u(1 - cur);
    };
    auto advance = [&](double2* out) {
        if (!win) cur = 1 - cur;
        in = out;
    };
    // A call's last four steps run as two and two rather than three and one,
    // and the first step of a window run, which also copies its input, alone.
    const RunPlan plan = run_plan(g, series != nullptr, h_f != nullptr, win != nullptr);
    auto pass_steps = [&](int64_t k) -> int {
        const int64_t left = n - k;
        if (win && k == 0) return 1;
        if (plan.three && left >= 3 && (left != 4 || !plan.two)) return 3;
        return plan.two && left >= 2 ? 2 : 1;
    };
    // Sample of state j (after step j) goes to series row j-1.  Launches
    // with fused extraction sample their input and a pass its intermediate
    // states; otherwise a separate pass samples each new state.
    const bool fused = plan.fused1;
    int64_t sampled = 0;
    InLoopCheck chk(g);
    auto extract_state = [&](const double2* u, int64_t j) -> int {
        HIP_TRY(launch_extract(u, g->L.pitch, ext, ne, series + (j - 1) * ne, g->stream));
        sampled = j;
        return TEUK_OK;
    };
    for (int64_t k = 0; k < n;) {
        if (plan.tile) {  // in launches of about equal steps
            const int64_t left = n - k, launches = (left + g->tile_steps - 1) / g->tile_steps;
            const int m = (int)((left + launches - 1) / launches);
            double2* out = next_buffer(k + m);
            StepArgs at = step_args(g);
            at.u_in = in;
            at.u_out = out;
            at.k.bsteps = m;
            at.k.n_ext = series ? ne : 0;
            at.k.row0 = k - 1;  // state k + s goes to series row k + s - 1
            at.series = series;
            HIP_TRY(launch_tile(at, g->tile_shape, g->stream));
            if (series) sampled = k + m - 1;
            advance(out);
            k += m;
            g->steps += m;
            continue;
        }
        if (plan.block) {
            const int m = (int)std::min<int64_t>(g->block_steps, n - k);
            double2* out = next_buffer(k + m);
            StepArgs ab = step_args(g);
            ab.u_in = in;
            ab.u_out = out;
            ab.k.bsteps = m;
            ab.k.bcols = g->block_cols;
            ab.k.n_ext = series ? ne : 0;
            ab.k.row0 = k - 1;  // state k + s goes to series row k + s - 1
            ab.series = series;
            HIP_TRY(launch_block(ab, g->stream));
            if (series) sampled = k + m - 1;
            advance(out);
            k += m;
            g->steps += m;
            if (int rc = chk.maybe(in)) return rc;
            continue;
        }
        const int m = pass_steps(k);
        // a one-step launch that cannot sample leaves each new state to a
        // separate pass
        const bool sample = series && (m > 1 || fused);
        if (series && !sample && k > sampled)
            if (int rc = extract_state(in, k)) return rc;
        double2* out = next_buffer(k + m);
        StepArgs& a = args[m - 1];
        a.u_in = in;
        a.u_out = out;
        a.win = !win ? nullptr : m == 1 ? (k == 0 ? window_state(0) : nullptr) : window_state(k + 1);
        a.series = (sample && k > 0) ? series + (k - 1) * ne : nullptr;
        a.series_mid = sample ? series + k * ne : nullptr;
        if (h_f)
            for (int j = 0; j < 4 * m; ++j) a.k.sf[j] = g->p.dt * h_f[4 * k + j];
        const int kind = pass_kind(m, h_f != nullptr);
        HIP_TRY(launch_pass(a, m, kerr, std::min(sample ? g->sample_wpb[kind] : g->pass_wpb[kind], 4), g->stream));
        if (sample) sampled = k + m - 1;
        advance(out);
        k += m;
        g->steps += m;
        if (series && !sample)
            if (int rc = extract_state(out, k)) return rc;
        if (int rc = chk.maybe(in)) return rc;
    }
    if (series && sampled < n)
        if (int rc = extract_state(in, n)) return rc;
    g->cur = win ? 1 - cur0 : cur;
    return chk.finish(in);
}

}  // namespace

int teuk_step_n(teuk_grid* g, int64_t n, void* d_series) { return step_n_impl(g, n, d_series, nullptr); }

size_t teuk_source_workspace_bytes(const teuk_grid* g) {
    if (!g) {
        fail(TEUK_E_INVALID_ARG, "grid handle is NULL");
        return 0;
    }
    return 2 * source_plane_bytes(g);
}

int teuk_set_source(teuk_grid* g, void* d_src_workspace, size_t bytes, const void* d_gi, const void* d_gh) {
    if (int rc = check_grid(g)) return rc;
    if (!d_gi && !d_gh) {
        g->sws = nullptr;
        return TEUK_OK;
    }
    if (!d_gi || !d_gh) return fail(TEUK_E_INVALID_ARG, "give both source profiles or neither");
    if (!d_src_workspace) return fail(TEUK_E_INVALID_ARG, "source workspace is NULL");
    if (reinterpret_cast<uintptr_t>(d_src_workspace) % kAlign)
        return fail(TEUK_E_WORKSPACE, "source workspace not %zu-byte aligned", kAlign);
    if (bytes < 2 * source_plane_bytes(g))
        return fail(TEUK_E_WORKSPACE, "source workspace has %zu bytes, needs %zu", bytes, 2 * source_plane_bytes(g));
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta, P = g->L.pitch;
    char* ws = static_cast<char*>(d_src_workspace);
    // complex128 rows as pairs of doubles: dense [nth][cols] -> pitched [nth][pitch]
    HIP_TRY(launch_pitch_copy(static_cast<const double*>(d_gi), reinterpret_cast<double*>(ws), nth, 2 * nr, 2 * P,
                              g->stream));
    HIP_TRY(launch_pitch_copy(static_cast<const double*>(d_gh), reinterpret_cast<double*>(ws + source_plane_bytes(g)),
                              nth, 2 * (nr - 1), 2 * P, g->stream));
    g->sws = ws;
    return TEUK_OK;
}

int teuk_step_n_source(teuk_grid* g, int64_t n, void* d_series, const double* h_f) {
    if (int rc = check_grid(g)) return rc;
    if (!g->sws) return fail(TEUK_E_STATE, "no source profile: call teuk_set_source first");
    if (n > 0 && !h_f) return fail(TEUK_E_INVALID_ARG, "time factors are NULL");
    for (int64_t j = 0; j < 4 * n; ++j)
        if (!std::isfinite(h_f[j])) return fail(TEUK_E_INVALID_ARG, "time factor %lld is not finite", (long long)j);
    return step_n_impl(g, n, d_series, nullptr, h_f);
}

size_t teuk_window_bytes(const teuk_grid* g, int64_t n) {
    if (!g || n < 0) {
        fail(TEUK_E_INVALID_ARG, "need a grid and n >= 0");
        return 0;
    }
    return g->L.state * (size_t)n;
}

int teuk_step_n_store(teuk_grid* g, int64_t n, void* d_series, void* d_window) {
    if (n > 0 && !d_window) return fail(TEUK_E_INVALID_ARG, "window is NULL");
    if (d_window && reinterpret_cast<uintptr_t>(d_window) % kAlign)
        return fail(TEUK_E_WORKSPACE, "window not %zu-byte aligned", kAlign);
    return step_n_impl(g, n, d_series, d_window);
}

namespace {

// Host check of the extraction requests of teuk_extract / teuk_extract_noalloc.
int check_extract_args(const teuk_grid* g, int32_t n, int32_t max_n, const double* h_rstar, const double* h_theta,
                       const void* d_out) {
    if (int rc = check_grid(g)) return rc;
    if (n < 0 || n > max_n) return fail(TEUK_E_INVALID_ARG, "n=%d outside [0, %d]", n, max_n);
    if (n == 0) return TEUK_OK;
    if (!h_rstar || !h_theta || !d_out) return fail(TEUK_E_INVALID_ARG, "NULL pointer");
    for (int e = 0; e < n; ++e) {
        if (!(h_rstar[e] >= g->p.rstar_min && h_rstar[e] <= g->p.rstar_max))
            return fail(TEUK_E_INVALID_ARG, "r*=%g outside the grid", h_rstar[e]);
        if (!(h_theta[e] >= 0.0 && h_theta[e] <= M_PI))
            return fail(TEUK_E_INVALID_ARG, "theta=%g outside [0, pi]", h_theta[e]);
    }
    return TEUK_OK;
}

ExtPoint grid_ext_point(const teuk_grid* g, double rstar, double theta) {
    return ext_point(rstar, theta, g->p.rstar_min, g->dr, (int)g->p.nr, (int)g->p.ntheta, g->sigma);
}

}  // namespace

int teuk_get_window_slot(teuk_grid* g, const void* d_window, int64_t k, void* d_phi, void* d_pi) {
    if (int rc = check_grid(g)) return rc;
    if (!d_window || !d_phi || !d_pi) return fail(TEUK_E_INVALID_ARG, "NULL pointer");
    if (k < 0) return fail(TEUK_E_INVALID_ARG, "slot %lld < 0", (long long)k);
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    const double2* u = reinterpret_cast<const double2*>(static_cast<const char*>(d_window) + (size_t)k * g->L.state);
    HIP_TRY(launch_export(u, static_cast<double2*>(d_phi), static_cast<double2*>(d_pi), nr, nth, g->L.pitch, g->stream));
    return TEUK_OK;
}

int teuk_extract(teuk_grid* g, int32_t n, const double* h_rstar, const double* h_theta, void* d_out) {
    if (int rc = check_extract_args(g, n, kMaxExtract, h_rstar, h_theta, d_out)) return rc;
    if (n == 0) return TEUK_OK;
    std::vector<ExtPoint> pts(n);
    for (int e = 0; e < n; ++e) pts[e] = grid_ext_point(g, h_rstar[e], h_theta[e]);
    if (int rc = set_device(g)) return rc;
    ExtPoint* dp = g->at<ExtPoint>(g->L.off_ext2);
    HIP_TRY(hipMemcpyAsync(dp, pts.data(), n * sizeof(ExtPoint), hipMemcpyHostToDevice, g->stream));
    HIP_TRY(launch_extract(g->u(g->cur), g->L.pitch, dp, n, static_cast<double2*>(d_out), g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));  // `pts` is released on return
    return TEUK_OK;
}

int teuk_extract_noalloc(teuk_grid* g, int32_t n, const double* h_rstar, const double* h_theta, void* d_out) {
    if (int rc = check_extract_args(g, n, kNoAllocMaxPoints, h_rstar, h_theta, d_out)) return rc;
    if (n == 0) return TEUK_OK;
    if (int rc = set_device(g)) return rc;
    char* d_scratch = static_cast<char*>(scratch_address(g->device));
    if (!d_scratch) return fail(TEUK_E_STATE, "no scratch address for device %d", g->device);
    // The point records are built in stack chunks and staged into this
    // device's scratch; a chunk buffer is reused only once its copy is done.
    constexpr int kChunk = 256;
    ExtPoint buf[kChunk];
    for (int e0 = 0; e0 < n; e0 += kChunk) {
        const int c = std::min(kChunk, n - e0);
        for (int k = 0; k < c; ++k) buf[k] = grid_ext_point(g, h_rstar[e0 + k], h_theta[e0 + k]);
        HIP_TRY(hipMemcpyAsync(d_scratch + (size_t)e0 * sizeof(ExtPoint), buf, c * sizeof(ExtPoint),
                               hipMemcpyHostToDevice, g->stream));
        HIP_TRY(hipStreamSynchronize(g->stream));
    }
    HIP_TRY(launch_extract(g->u(g->cur), g->L.pitch, reinterpret_cast<const ExtPoint*>(d_scratch), n,
                           static_cast<double2*>(d_out), g->stream));
    // the scratch is free for the next call once this one returns
    HIP_TRY(hipStreamSynchronize(g->stream));
    return TEUK_OK;
}

int teuk_get_state(teuk_grid* g, void* d_phi, void* d_pi) {
    if (int rc = check_grid(g)) return rc;
    if (!d_phi || !d_pi) return fail(TEUK_E_INVALID_ARG, "output pointers are NULL");
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_export(g->u(g->cur), static_cast<double2*>(d_phi), static_cast<double2*>(d_pi), nr, nth, g->L.pitch, g->stream));
    return TEUK_OK;
}

int teuk_check_finite(teuk_grid* g) {
    if (int rc = check_grid(g)) return rc;
    if (int rc = set_device(g)) return rc;
    int* flag = g->at<int>(g->L.off_flag);
    HIP_TRY(launch_zero_ints(flag, 1, g->stream));
    HIP_TRY(launch_nonfinite(g->u(g->cur), (int)g->p.nr, (int)g->p.ntheta, g->L.pitch, flag, g->stream));
    int h = 0;
    HIP_TRY(hipMemcpyAsync(&h, flag, sizeof(h), hipMemcpyDeviceToHost, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    if (h) return fail(TEUK_E_NONFINITE, "state holds a non-finite value after %lld steps", (long long)g->steps);
    return TEUK_OK;
}

int teuk_set_finite_check(teuk_grid* g, int64_t every) {
    if (int rc = check_grid(g)) return rc;
    if (every < 0) return fail(TEUK_E_INVALID_ARG, "every=%lld < 0", (long long)every);
    g->check_every = every;
    return TEUK_OK;
}

int64_t teuk_steps_taken(const teuk_grid* g) { return g ? g->steps : -1; }

double teuk_get_dt(const teuk_grid* g) { return g ? g->p.dt : 0.0; }

namespace {

// After a change of the tile or the block launch: with both as teuk_init_grid
// chose them the grid's own choice among the passes is back (the passes' own
// tiles and the tile pass); otherwise the sweeps take the tile given.
// off: the block pass was turned off, which leaves the sweeps.
void select_launch(teuk_grid* g, bool off) {
    const bool tile = g->rows == g->default_tile[0] && g->wpb == g->default_tile[1];
    const bool block = g->block_steps == g->default_block[0] &&
                       (g->block_steps == 0 || g->block_cols == g->default_block[1]);  // off: whatever its columns
    g->default_launch = tile && block && !off;
    for (int k = 0; k < kPassKinds; ++k) {
        g->pass_rows[k] = tile ? g->default_rows[k] : g->rows;
        g->pass_wpb[k] = tile ? g->default_wpb[k] : g->wpb;
    }
}

}  // namespace

int teuk_set_tile(teuk_grid* g, int32_t rows_per_tile, int32_t waves_per_block) {
    if (int rc = check_grid(g)) return rc;
    if (rows_per_tile < 1 || rows_per_tile > g->p.ntheta)
        return fail(TEUK_E_INVALID_ARG, "rows_per_tile=%d outside [1, ntheta]", rows_per_tile);
    if (waves_per_block != 1 && waves_per_block != 2 && waves_per_block != 4 && waves_per_block != 8)
        return fail(TEUK_E_INVALID_ARG, "waves_per_block=%d not in {1, 2, 4, 8}", waves_per_block);
    g->rows = rows_per_tile;
    g->wpb = waves_per_block;
    select_launch(g, false);
    update_fusion(g);
    return TEUK_OK;
}

int teuk_set_steps_per_pass(teuk_grid* g, int32_t steps_per_pass) {
    if (int rc = check_grid(g)) return rc;
    if (steps_per_pass != 1 && steps_per_pass != 2)
        return fail(TEUK_E_INVALID_ARG, "steps_per_pass=%d not in {1, 2}", steps_per_pass);
    g->steps_per_pass = steps_per_pass;
    return TEUK_OK;
}

int teuk_get_steps_per_pass(const teuk_grid* g, int32_t* steps_per_pass) {
    if (int rc = check_grid(g)) return rc;
    if (steps_per_pass) *steps_per_pass = g->steps_per_pass;
    return TEUK_OK;
}

int teuk_set_block_launch(teuk_grid* g, int32_t steps, int32_t cols) {
    if (int rc = check_grid(g)) return rc;
    if (steps == 0) {
        g->block_steps = 0;
        select_launch(g, true);
        return TEUK_OK;
    }
    const int nth = (int)g->p.ntheta;
    if (g->p.coef_mode != TEUK_COEF_KERR || nth > kMaxBlockRows)
        return fail(TEUK_E_INVALID_ARG, "the block pass needs Kerr coefficients and ntheta <= %d", kMaxBlockRows);
    if (cols == 0) cols = g->block_cols > 0 ? g->block_cols : std::min(64, 1024 / nth);
    if (cols < 4 || cols > 64 || cols * nth > 1024)
        return fail(TEUK_E_INVALID_ARG, "block cols=%d outside [4, min(64, 1024/ntheta=%d)]", cols, 1024 / nth);
    if (steps < 0 || steps > (cols - 2) / 2)
        return fail(TEUK_E_INVALID_ARG, "block steps=%d outside [0, %d] for %d columns", steps, (cols - 2) / 2, cols);
    g->block_steps = steps;
    g->block_cols = cols;
    select_launch(g, false);
    return TEUK_OK;
}

int teuk_get_block_launch(const teuk_grid* g, int32_t* steps, int32_t* cols) {
    if (int rc = check_grid(g)) return rc;
    if (steps) *steps = g->block_steps;
    if (cols) *cols = g->block_cols;
    return TEUK_OK;
}

int teuk_set_cache_policy(teuk_grid* g, int32_t policy) {
    if (int rc = check_grid(g)) return rc;
    if (policy != TEUK_CACHE_AUTO && policy != TEUK_CACHE_KEEP && policy != TEUK_CACHE_STREAM)
        return fail(TEUK_E_INVALID_ARG, "cache policy %d not in {0, 1, 2}", policy);
    g->cache_policy = policy;
    return TEUK_OK;
}

int teuk_get_cache_policy(const teuk_grid* g, int32_t* policy, int32_t* keeps) {
    if (int rc = check_grid(g)) return rc;
    if (policy) *policy = g->cache_policy;
    if (keeps) *keeps = keeps_states(g) ? 1 : 0;
    return TEUK_OK;
}

int teuk_get_tile(const teuk_grid* g, int32_t* rows_per_tile, int32_t* waves_per_block) {
    if (int rc = check_grid(g)) return rc;
    if (rows_per_tile) *rows_per_tile = g->rows;
    if (waves_per_block) *waves_per_block = g->wpb;
    return TEUK_OK;
}

int teuk_set_adjoint_tile(teuk_grid* g, int32_t rows_per_tile, int32_t waves_per_block) {
    if (int rc = check_grid(g)) return rc;
    if (rows_per_tile < 1 || rows_per_tile > g->p.ntheta)
        return fail(TEUK_E_INVALID_ARG, "rows_per_tile=%d outside [1, ntheta]", rows_per_tile);
    if (waves_per_block != 1 && waves_per_block != 2 && waves_per_block != 4)
        return fail(TEUK_E_INVALID_ARG, "waves_per_block=%d not in {1, 2, 4}", waves_per_block);
    g->adj_rows = rows_per_tile;
    g->adj_wpb = waves_per_block;
    // the tile as teuk_init_grid chose it: the kernels' own heights and the tile pass again
    g->adj_default = rows_per_tile == g->default_adj_rows && waves_per_block == kAdjWaves;
    for (int i = 0; i < kAdjKinds; ++i) {
        g->adj_pass_rows[i] = g->adj_default ? g->default_adj_pass_rows[i] : rows_per_tile;
        g->adj_pass_wpb[i] = g->adj_default ? g->default_adj_pass_wpb[i] : waves_per_block;
    }
    update_fusion(g);
    return TEUK_OK;
}

int teuk_get_adjoint_tile(const teuk_grid* g, int32_t* rows_per_tile, int32_t* waves_per_block) {
    if (int rc = check_grid(g)) return rc;
    if (rows_per_tile) *rows_per_tile = g->adj_rows;
    if (waves_per_block) *waves_per_block = g->adj_wpb;
    return TEUK_OK;
}

int teuk_get_pass(const teuk_grid* g, int32_t run, teuk_pass* out) {
    if (int rc = check_grid(g)) return rc;
    if (!out) return fail(TEUK_E_INVALID_ARG, "output pointer is NULL");
    if (run < TEUK_RUN_STEPS || run > TEUK_RUN_SPIN_TANGENT) return fail(TEUK_E_INVALID_ARG, "run=%d unknown", run);
    auto tile = [&](const TileShape& t, int steps) {
        *out = {TEUK_PASS_TILE, steps, t.cols, t.rows, t.waves, 1};
        return TEUK_OK;
    };
    if (run == TEUK_RUN_COTANGENTS) {
        if (adjoint_on_tiles(g)) return tile(g->adj_tile, g->adj_tile_steps);
        const bool two = fused_adjoint_ok(g) && g->steps_per_pass == 2;
        const AdjKind kind = two ? kAdjTwo : kAdjOne;
        const int steps = kAdjoint[kind].steps;
        *out = {TEUK_PASS_SWEEP, steps, strip_cols(steps), g->adj_pass_rows[kind], g->adj_pass_wpb[kind],
                fused_adjoint_ok(g)};
        return TEUK_OK;
    }
    if (run == TEUK_RUN_SPIN_TANGENT) {
        *out = {TEUK_PASS_SWEEP, 1, kStripCols, g->tan_sample_rows, g->adj_pass_wpb[kAdjSpinTangent], g->tan_fused};
        return TEUK_OK;
    }
    const bool series = run == TEUK_RUN_SERIES || run == TEUK_RUN_SOURCE_SERIES;
    const bool source = run == TEUK_RUN_SOURCE || run == TEUK_RUN_SOURCE_SERIES;
    const RunPlan p = run_plan(g, series, source, false);
    if (p.tile) return tile(g->tile_shape, g->tile_steps);
    if (p.block) {
        *out = {TEUK_PASS_BLOCK, g->block_steps, g->block_cols, (int32_t)g->p.ntheta,
                (int32_t)(g->block_cols * g->p.ntheta + kWave - 1) / kWave, 1};
        return TEUK_OK;
    }
    const int steps = p.three ? 3 : p.two ? 2 : 1, kind = pass_kind(steps, source);
    const bool samples = steps > 1 || p.fused1, sample = series && samples;
    *out = {TEUK_PASS_SWEEP, steps, strip_cols(steps), sample ? g->sample_rows[kind] : g->pass_rows[kind],
            std::min(sample ? g->sample_wpb[kind] : g->pass_wpb[kind], 4), samples};
    return TEUK_OK;
}

namespace {

void adjoint_layout(teuk_grid* g, size_t* total) {
    const int nth = (int)g->p.ntheta;
    size_t o = 0;
    for (int k = 0; k < 2; ++k) {
        g->aoff_lam[k] = o;
        o += g->L.state;
    }
    g->aoff_da = o;
    o += align_up((size_t)kNumSRad * 2 * g->L.pitch * sizeof(double));
    g->aoff_slots = o;
    // one slot per tile of either adjoint tiling, for any tile rows
    const size_t strips2 = ((size_t)g->p.nr + kStripCols2 - 1) / kStripCols2;
    o += align_up(std::max<size_t>(g->adj_strips, strips2) * nth * sizeof(double));
    g->aoff_sum = o;
    o += kAlign;
    *total = o;
}

}  // namespace

size_t teuk_adjoint_workspace_bytes(teuk_grid* g) {
    if (!g) {
        fail(TEUK_E_INVALID_ARG, "grid handle is NULL");
        return 0;
    }
    size_t total;
    adjoint_layout(g, &total);
    return total;
}

int teuk_enable_adjoint(teuk_grid* g, void* d_adj_workspace, size_t bytes) {
    if (int rc = check_grid(g)) return rc;
    if (g->p.coef_mode != TEUK_COEF_KERR) return fail(TEUK_E_STATE, "the adjoint needs TEUK_COEF_KERR coefficients");
    if (!d_adj_workspace) return fail(TEUK_E_INVALID_ARG, "adjoint workspace is NULL");
    if (reinterpret_cast<uintptr_t>(d_adj_workspace) % kAlign)
        return fail(TEUK_E_WORKSPACE, "adjoint workspace not %zu-byte aligned", kAlign);
    size_t total;
    adjoint_layout(g, &total);
    if (bytes < total) return fail(TEUK_E_WORKSPACE, "adjoint workspace has %zu bytes, needs %zu", bytes, total);
    if (int rc = set_device(g)) return rc;
    g->aws = static_cast<char*>(d_adj_workspace);
    HIP_TRY(hipMemsetAsync(g->aws, 0, total, g->stream));
    // a-derivatives of the radial tables at fixed r* (dual numbers through
    // the tortoise inversion and every radial factor), from the x that
    // teuk_init_grid solved for at each position
    HIP_TRY(launch_tables_da(table_args(g), g->at<double>(g->L.off_x), reinterpret_cast<double*>(g->aws + g->aoff_da),
                             g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    return TEUK_OK;
}

namespace {

// Launch arguments of an adjoint-side kernel.
AdjArgs adjoint_args(const teuk_grid* g, AdjKind kind) {
    AdjArgs a{};
    const int nth = (int)g->p.ntheta;
    a.k.nr = (int)g->p.nr;
    a.k.nth = nth;
    a.k.pitch = g->L.pitch;
    a.k.sigma = g->sigma;
    const int cols = strip_cols(kAdjoint[kind].steps);
    a.k.rows = g->adj_pass_rows[kind];
    a.k.n_strips = (a.k.nr + cols - 1) / cols;
    a.k.n_chunks = (nth + a.k.rows - 1) / a.k.rows;
    a.k.zero = 0;
    a.k.keep = keeps_states(g) ? 1 : 0;
    a.k.plane = (int64_t)nth * g->L.pitch;
    a.k.hdt = 0.5 * g->p.dt;
    a.rad = g->at<double>(g->L.off_rad);
    a.rad_da = reinterpret_cast<const double*>(g->aws + g->aoff_da);
    a.k.qdt = 0.25 * g->p.dt;
    a.k.kap_h = finite_inverse(a.k.hdt);
    a.k.kap_i = finite_inverse(a.k.qdt);
    a.ang = g->at<double>(g->L.off_ang);
    a.ext = g->at<ExtPoint>(g->L.off_ext);
    return a;
}

}  // namespace

int teuk_step_n_tangent(teuk_grid* g, int64_t n, void* d_window) {
    if (int rc = check_grid(g)) return rc;
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (!g->aws) return fail(TEUK_E_STATE, "teuk_enable_adjoint has not been called");
    if (n > 0 && !d_window) return fail(TEUK_E_INVALID_ARG, "window is NULL");
    if (d_window && reinterpret_cast<uintptr_t>(d_window) % kAlign)
        return fail(TEUK_E_WORKSPACE, "window not %zu-byte aligned", kAlign);
    if (n == 0) return TEUK_OK;
    if (int rc = set_device(g)) return rc;
    const AdjArgs a = adjoint_args(g, kAdjTangent);
    char* win = static_cast<char*>(d_window);
    for (int64_t k = 0; k < n; ++k) {
        double2* t_out = reinterpret_cast<double2*>(win + (size_t)k * g->L.state);
        HIP_TRY(launch_tangent(g->u(g->cur), g->u(1 - g->cur), t_out, a, g->adj_pass_wpb[kAdjTangent], g->stream));
        g->cur = 1 - g->cur;
        g->steps += 1;
    }
    return TEUK_OK;
}

namespace {

// The reverse of a segment; dL/da goes to the host (h_acc: reduced,
// copied back, synchronised) or to a device accumulator (d_acc: added on the
// stream, asynchronous), or nowhere (both NULL: cotangents only).
int adjoint_impl(teuk_grid* g, int64_t n, void* d_lam_phi, void* d_lam_pi, const void* d_dL_dseries,
                 const void* d_window, int32_t flags, double* h_dL_da_accum, double* d_dL_da_accum) {
    if (int rc = check_grid(g)) return rc;
    if (!g->aws) return fail(TEUK_E_STATE, "teuk_enable_adjoint has not been called");
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (!d_lam_phi || !d_lam_pi) return fail(TEUK_E_INVALID_ARG, "cotangent pointers are NULL");
    // without a dL/da accumulator only the cotangents are computed, and they
    // do not depend on the forward states (the step is linear)
    const bool spin = h_dL_da_accum != nullptr || d_dL_da_accum != nullptr;
    if (n > 0 && spin && !d_window) return fail(TEUK_E_INVALID_ARG, "window is NULL");
    if (flags & ~(TEUK_ADJ_PROJECT_INITIAL | TEUK_ADJ_TANGENT_WINDOW))
        return fail(TEUK_E_INVALID_ARG, "unknown flags 0x%x", flags);
    // the window holds T_k = (dA/da) u^k (teuk_step_n_tangent) instead of u^k
    const bool tangent = spin && (flags & TEUK_ADJ_TANGENT_WINDOW);
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta, P = g->L.pitch;
    const int ne = g->p.n_extract;
    const double2* gs = (ne > 0) ? static_cast<const double2*>(d_dL_dseries) : nullptr;
    const ExtPoint* ext = g->at<ExtPoint>(g->L.off_ext);
    hipStream_t s = g->stream;
    auto lam = [&](int k) { return reinterpret_cast<double2*>(g->aws + g->aoff_lam[k]); };
    double* slots = reinterpret_cast<double*>(g->aws + g->aoff_slots);
    double* sum = reinterpret_cast<double*>(g->aws + g->aoff_sum);
    const AdjKind one = spin && !tangent ? kAdjStates : kAdjOne, two = tangent ? kAdjTwoDot : kAdjTwo;
    AdjArgs a = adjoint_args(g, one), a2 = adjoint_args(g, two);
    const int nslots = std::max(a.k.n_strips * a.k.n_chunks, a2.k.n_strips * a2.k.n_chunks);

    int c = 0;
    HIP_TRY(launch_import(static_cast<const double2*>(d_lam_phi), static_cast<const double2*>(d_lam_pi), lam(c),
                          nr, nth, P, s));
    if (spin) {
        HIP_TRY(hipMemsetAsync(slots, 0, (size_t)nslots * sizeof(double), s));
        if (!d_dL_da_accum) HIP_TRY(hipMemsetAsync(sum, 0, sizeof(double), s));
    }
    // the sample of the segment's last state
    if (gs && n > 0) HIP_TRY(launch_extract_adjoint(lam(c), P, ext, ne, gs + (n - 1) * ne, s));
    a.slots = a2.slots = slots;
    // the sample of the state an adjoint step produces is added by the
    // adjoint kernel itself for a few points, by a separate pass otherwise
    const bool fused = fused_adjoint_ok(g);
    a.k.n_ext = a2.k.n_ext = fused ? ne : 0;
    const char* win = static_cast<const char*>(d_window);
    auto slot = [&](int64_t k) { return reinterpret_cast<const double2*>(win + (size_t)k * g->L.state); };
    int64_t k = n - 1;
    if (!spin && adjoint_on_tiles(g)) {
        // cotangents on register tiles, in launches of about equal steps
        AdjArgs at = a;
        at.k.n_ext = ne;
        for (; k >= 0;) {
            const int64_t left = k + 1, launches = (left + g->adj_tile_steps - 1) / g->adj_tile_steps;
            const int m = (int)((left + launches - 1) / launches);
            at.nu_in = lam(c);
            at.lam_out = lam(1 - c);
            HIP_TRY(launch_adjoint_tile(at, gs, k - 1, m, g->adj_tile, s));
            c = 1 - c;
            k -= m;
        }
    }
    if ((!spin || tangent) && fused && g->steps_per_pass == 2) {
        // cotangents (and the tangents' dot products): two adjoint steps
        // (k, then k-1) per pass
        for (; k >= 1; k -= 2) {
            a2.nu_in = lam(c);
            a2.lam_out = lam(1 - c);
            a2.u_in = tangent ? slot(k) : nullptr;
            a2.gsample = gs ? reinterpret_cast<const double*>(gs + (k - 1) * ne) : nullptr;
            const double* gb = (gs && k >= 2) ? reinterpret_cast<const double*>(gs + (k - 2) * ne) : nullptr;
            HIP_TRY(launch_adjoint2(a2, gb, tangent ? slot(k - 1) : nullptr, g->adj_pass_wpb[two], s));
            c = 1 - c;
        }
    }
    const AdjMode mode = tangent ? AdjMode::kTangentDot : spin ? AdjMode::kSpin : AdjMode::kCotangent;
    for (; k >= 0; --k) {
        a.nu_in = lam(c);
        a.u_in = spin ? slot(k) : nullptr;
        a.lam_out = lam(1 - c);
        a.gsample = (gs && k >= 1 && fused) ? reinterpret_cast<const double*>(gs + (k - 1) * ne) : nullptr;
        HIP_TRY(launch_adjoint(a, g->adj_pass_wpb[one], mode, s));
        c = 1 - c;
        if (gs && k >= 1 && !fused) HIP_TRY(launch_extract_adjoint(lam(c), P, ext, ne, gs + (k - 1) * ne, s));
    }
    if (flags & TEUK_ADJ_PROJECT_INITIAL) HIP_TRY(launch_zero_radial_boundary(lam(c), nr, nth, P, s));
    HIP_TRY(launch_export(lam(c), static_cast<double2*>(d_lam_phi), static_cast<double2*>(d_lam_pi), nr, nth, P, s));
    if (!spin) return TEUK_OK;  // asynchronous
    if (d_dL_da_accum) {         // asynchronous: added on the stream, in call order
        HIP_TRY(launch_reduce_slots(slots, nslots, d_dL_da_accum, s));
        return TEUK_OK;
    }
    HIP_TRY(launch_reduce_slots(slots, nslots, sum, s));
    double h = 0.0;
    HIP_TRY(hipMemcpyAsync(&h, sum, sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    *h_dL_da_accum += h;
    return TEUK_OK;
}

}  // namespace

int teuk_adjoint_step_n(teuk_grid* g, int64_t n, void* d_lam_phi, void* d_lam_pi, const void* d_dL_dseries,
                        const void* d_window, int32_t flags, double* h_dL_da_accum) {
    return adjoint_impl(g, n, d_lam_phi, d_lam_pi, d_dL_dseries, d_window, flags, h_dL_da_accum, nullptr);
}

int teuk_adjoint_step_n_async(teuk_grid* g, int64_t n, void* d_lam_phi, void* d_lam_pi, const void* d_dL_dseries,
                              const void* d_window, int32_t flags, double* d_dL_da_accum) {
    if (!d_dL_da_accum) return fail(TEUK_E_INVALID_ARG, "the dL/da accumulator is NULL");
    return adjoint_impl(g, n, d_lam_phi, d_lam_pi, d_dL_dseries, d_window, flags, nullptr, d_dL_da_accum);
}

/* ---- forward-mode spin derivative ------------------------------------- */

size_t teuk_spin_tangent_workspace_bytes(const teuk_grid* g) {
    if (!g) {
        fail(TEUK_E_INVALID_ARG, "grid handle is NULL");
        return 0;
    }
    return 2 * g->L.state;
}

int teuk_enable_spin_tangent(teuk_grid* g, void* d_workspace, size_t bytes) {
    if (int rc = check_grid(g)) return rc;
    if (!g->aws) return fail(TEUK_E_STATE, "teuk_enable_adjoint has not been called (it builds the a-derivative tables)");
    if (!d_workspace) return fail(TEUK_E_INVALID_ARG, "spin-tangent workspace is NULL");
    if (reinterpret_cast<uintptr_t>(d_workspace) % kAlign)
        return fail(TEUK_E_WORKSPACE, "spin-tangent workspace not %zu-byte aligned", kAlign);
    if (bytes < 2 * g->L.state)
        return fail(TEUK_E_WORKSPACE, "spin-tangent workspace has %zu bytes, needs %zu", bytes, 2 * g->L.state);
    if (int rc = set_device(g)) return rc;
    g->tws = static_cast<char*>(d_workspace);
    g->vcur = 0;
    HIP_TRY(hipMemsetAsync(g->tws, 0, 2 * g->L.state, g->stream));
    return TEUK_OK;
}

int teuk_set_spin_tangent(teuk_grid* g, const void* d_vphi, const void* d_vpi) {
    if (int rc = check_grid(g)) return rc;
    if (!g->tws) return fail(TEUK_E_STATE, "teuk_enable_spin_tangent has not been called");
    if ((d_vphi == nullptr) != (d_vpi == nullptr)) return fail(TEUK_E_INVALID_ARG, "give both planes or neither");
    if (int rc = set_device(g)) return rc;
    g->vcur = 0;
    if (!d_vphi) {
        HIP_TRY(hipMemsetAsync(g->v(0), 0, g->L.state, g->stream));
        return TEUK_OK;
    }
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_import(static_cast<const double2*>(d_vphi), static_cast<const double2*>(d_vpi), g->v(0),
                          nr, nth, g->L.pitch, g->stream));
    return TEUK_OK;
}

int teuk_get_spin_tangent(teuk_grid* g, void* d_vphi, void* d_vpi) {
    if (int rc = check_grid(g)) return rc;
    if (!g->tws) return fail(TEUK_E_STATE, "teuk_enable_spin_tangent has not been called");
    if (!d_vphi || !d_vpi) return fail(TEUK_E_INVALID_ARG, "output pointers are NULL");
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_export(g->v(g->vcur), static_cast<double2*>(d_vphi), static_cast<double2*>(d_vpi), nr, nth, g->L.pitch, g->stream));
    return TEUK_OK;
}

int teuk_step_n_spin_tangent(teuk_grid* g, int64_t n, void* d_series, void* d_tseries) {
    if (int rc = check_grid(g)) return rc;
    if (!g->tws) return fail(TEUK_E_STATE, "teuk_enable_spin_tangent has not been called");
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (n == 0) return TEUK_OK;
    if (int rc = set_device(g)) return rc;
    const int ne = g->p.n_extract;
    double2* series = (ne > 0) ? static_cast<double2*>(d_series) : nullptr;
    double2* tseries = (ne > 0) ? static_cast<double2*>(d_tseries) : nullptr;
    const ExtPoint* ext = g->at<ExtPoint>(g->L.off_ext);
    AdjArgs a = adjoint_args(g, kAdjSpinTangent);
    // the launches sample their input (row k-1 of a series: the state after
    // step k); the call's last state, or every state when two extraction
    // points share a tile, by a separate pass
    const bool fused = (series || tseries) && g->tan_fused;
    if (fused) {
        a.k.rows = g->tan_sample_rows;
        a.k.n_chunks = (a.k.nth + a.k.rows - 1) / a.k.rows;
    }
    a.k.n_ext = fused ? ne : 0;
    auto extract = [&](int64_t j) -> int {
        if (series) HIP_TRY(launch_extract(g->u(g->cur), g->L.pitch, ext, ne, series + (j - 1) * ne, g->stream));
        if (tseries) HIP_TRY(launch_extract(g->v(g->vcur), g->L.pitch, ext, ne, tseries + (j - 1) * ne, g->stream));
        return TEUK_OK;
    };
    InLoopCheck chk(g);
    for (int64_t k = 0; k < n; ++k) {
        if (!fused && k > 0)
            if (int rc = extract(k)) return rc;
        double2* su = (series && fused && k > 0) ? series + (k - 1) * ne : nullptr;
        double2* sv = (tseries && fused && k > 0) ? tseries + (k - 1) * ne : nullptr;
        HIP_TRY(launch_spin_tangent(g->u(g->cur), g->v(g->vcur), g->u(1 - g->cur), g->v(1 - g->vcur), su, sv, a,
                                    g->adj_pass_wpb[kAdjSpinTangent], g->stream));
        g->cur = 1 - g->cur;
        g->vcur = 1 - g->vcur;
        g->steps += 1;
        if (int rc = chk.maybe(g->u(g->cur))) return rc;
    }
    if (int rc = extract(n)) return rc;
    return chk.finish(g->u(g->cur));
}

int teuk_spin_gradient(teuk_grid* g, int64_t n, const void* d_dL_dseries, const void* d_tseries,
                       double* d_dL_da_accum) {
    if (int rc = check_grid(g)) return rc;
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (!d_dL_da_accum) return fail(TEUK_E_INVALID_ARG, "the dL/da accumulator is NULL");
    const int64_t count = n * g->p.n_extract;
    if (count == 0) return TEUK_OK;
    if (!d_dL_dseries || !d_tseries) return fail(TEUK_E_INVALID_ARG, "series pointers are NULL");
    if (int rc = set_device(g)) return rc;
    HIP_TRY(launch_series_dot(static_cast<const double2*>(d_dL_dseries), static_cast<const double2*>(d_tseries),
                              count, d_dL_da_accum, g->stream));
    return TEUK_OK;
}

/* ---- batched evolutions ------------------------------------------------ */

struct teuk_batch {
    std::vector<teuk_grid*> members;
    std::vector<size_t> ws_off;     // member workspace offsets in the batch workspace
    size_t desc_off = 0;            // descriptor table offset
    size_t ext_off = 0;             // extraction point table offset
    int n_points = 0;               // extraction points of all members
    char* ws = nullptr;
    hipStream_t stream = nullptr;
    int device = 0;
    int rows = 64, wpb = 4, n_blocks = 0;  // default launch: 64-row tiles, four wavefronts per SIMD
    int total_tiles[kMaxPassSteps] = {};   // work lists of the passes of 1, 2, 3 steps
    int steps_per_pass = 2;
    int parity = 0;                 // which state buffer of every member is the input
    bool keep = false;              // next states with cache-keeping stores (set by batch_upload)
    bool fused = true;              // the passes can sample every member's points (set by batch_upload)
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;  // two launches (parity 0 then 1)
    hipStream_t cap = nullptr;      // private stream the graph is captured on
    int64_t steps = 0;
};

namespace {

size_t batch_layout(const teuk_params* members, int count, std::vector<size_t>* offs, size_t* desc_off,
                    size_t* ext_off = nullptr) {
    size_t o = 0;
    int64_t points = 0;
    for (int k = 0; k < count; ++k) {
        if (offs) offs->push_back(o);
        o += align_up(make_layout(&members[k]).total);
        points += members[k].n_extract;
    }
    if (desc_off) *desc_off = o;
    o += align_up((size_t)count * sizeof(BatchMember));
    if (ext_off) *ext_off = o;
    o += align_up((size_t)std::max<int64_t>(points, 1) * sizeof(BatchExtPoint));
    return o;
}

void batch_drop_graph(teuk_batch* b) {
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
}

// Descriptor table for the current tile rows; uploaded synchronously.
int batch_upload(teuk_batch* b) {
    std::vector<BatchMember> d(b->members.size());
    int tiles[kMaxPassSteps] = {};
    // one launch advances every member: their states share the cache
    size_t states = 0;
    for (const teuk_grid* g : b->members) states += 2 * g->L.state;
    const int keep = states <= kKeepStatesBytes ? 1 : 0;
    b->keep = keep != 0;
    b->fused = true;
    int64_t points = 0;
    for (size_t k = 0; k < b->members.size(); ++k) {
        teuk_grid* g = b->members[k];
        g->rows = std::min<int>(b->rows, (int)g->p.ntheta);
        StepArgs a = step_args(g);
        BatchMember& M = d[k];
        M.u[0] = g->u(0);
        M.u[1] = g->u(1);
        M.rad = a.rad;
        M.ang = a.ang;
        M.k = a.k;
        M.ext = a.ext;
        M.ext_off = points;
        points += g->p.n_extract;
        M.k.n_ext = g->p.n_extract;
        M.k.keep = keep;
        b->fused = b->fused && g->p.n_extract <= kMaxEqualExtract;
        for (int m = 1; m <= kMaxPassSteps; ++m)
            b->fused = b->fused && one_point_a_tile(tile_order(g, strip_cols(m)), strip_cols(m), g->rows, true);
        for (int m = 0; m < kMaxPassSteps; ++m) {
            M.strips[m] = (a.k.nr + strip_cols(m + 1) - 1) / strip_cols(m + 1);
            M.tile_begin[m] = tiles[m];
            tiles[m] += M.strips[m] * a.k.n_chunks;
        }
    }
    for (int m = 0; m < kMaxPassSteps; ++m) b->total_tiles[m] = tiles[m];
    HIP_TRY(hipMemcpyAsync(b->ws + b->desc_off, d.data(), d.size() * sizeof(BatchMember), hipMemcpyHostToDevice,
                           b->stream));
    HIP_TRY(hipStreamSynchronize(b->stream));
    return TEUK_OK;
}

int batch_launch(teuk_batch* b, int parity, int steps, hipStream_t s, const BatchSeries& series = {}) {
    const hipError_t e =
        launch_batch(reinterpret_cast<const BatchMember*>(b->ws + b->desc_off), (int)b->members.size(),
                     b->total_tiles[steps - 1], parity, b->n_blocks, b->wpb, steps, b->keep, series, s);
    return e == hipSuccess ? TEUK_OK : fail(TEUK_E_HIP, "batched step launch failed: %s", hipGetErrorString(e));
}

// Most steps of a launch: 1, or with several steps a pass, 3 (2 if a member
// has fewer than the three rows that pass needs).
int batch_pass_steps(const teuk_batch* b) {
    if (b->steps_per_pass == 1) return 1;
    for (const teuk_grid* g : b->members)
        if (g->p.ntheta < 3) return 2;
    return 3;
}

// Steps of the next launch with `left` to take (the last as in step_n_impl).
int batch_next_steps(int most, int64_t left) {
    return most == 3 && left >= 3 && left != 4 ? 3 : (int)std::min<int64_t>(left, std::min(most, 2));
}

// Capture two launches (parity 0, then 1) into a graph.  The capture runs on a
// private stream (capturing the caller's stream may not be allowed, e.g. the
// legacy default stream); the graph is launched on the caller's stream.
int batch_capture(teuk_batch* b) {
    if (!b->cap) HIP_TRY(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
    HIP_TRY(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
    const int rc0 = batch_launch(b, 0, batch_pass_steps(b), b->cap);
    const int rc1 = batch_launch(b, 1, batch_pass_steps(b), b->cap);
    hipGraph_t graph = nullptr;
    const hipError_t e = hipStreamEndCapture(b->cap, &graph);
    if (rc0 || rc1 || e != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        return fail(TEUK_E_HIP, "capturing the batched step graph failed: %s", hipGetErrorString(e));
    }
    b->graph = graph;
    HIP_TRY(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
    return TEUK_OK;
}

int batch_check(const teuk_batch* b, int member) {
    if (!b) return fail(TEUK_E_INVALID_ARG, "batch handle is NULL");
    if (member < 0 || member >= (int)b->members.size())
        return fail(TEUK_E_INVALID_ARG, "member %d outside [0, %zu)", member, b->members.size());
    return TEUK_OK;
}

}  // namespace

size_t teuk_batch_workspace_bytes(const teuk_params* members, int32_t count) {
    if (!members || count < 1) {
        fail(TEUK_E_INVALID_ARG, "need count >= 1 members");
        return 0;
    }
    for (int k = 0; k < count; ++k)
        if (validate(&members[k]) != TEUK_OK) return 0;
    return batch_layout(members, count, nullptr, nullptr);
}

int teuk_batch_init(const teuk_params* members, int32_t count, void* hip_stream, void* d_workspace, size_t bytes,
                    teuk_batch** out) {
    if (!members || count < 1 || !out) return fail(TEUK_E_INVALID_ARG, "need members, count >= 1 and out");
    for (int k = 0; k < count; ++k) {
        if (int rc = validate(&members[k])) return rc;
        if (members[k].coef_mode != TEUK_COEF_KERR)
            return fail(TEUK_E_INVALID_ARG, "member %d: batched members use TEUK_COEF_KERR", k);
    }
    if (!d_workspace || reinterpret_cast<uintptr_t>(d_workspace) % kAlign)
        return fail(TEUK_E_WORKSPACE, "batch workspace NULL or not %zu-byte aligned", kAlign);
    teuk_batch* b = new teuk_batch();
    const size_t need = batch_layout(members, count, &b->ws_off, &b->desc_off, &b->ext_off);
    if (bytes < need) {
        delete b;
        return fail(TEUK_E_WORKSPACE, "batch workspace has %zu bytes, needs %zu", bytes, need);
    }
    b->ws = static_cast<char*>(d_workspace);
    b->stream = reinterpret_cast<hipStream_t>(hip_stream);
    for (int k = 0; k < count; ++k) {
        teuk_grid* g = nullptr;
        const size_t mbytes = make_layout(&members[k]).total;
        if (int rc = teuk_init_grid(&members[k], hip_stream, b->ws + b->ws_off[k], mbytes, &g)) {
            for (teuk_grid* m : b->members) teuk_free(m);
            delete b;
            return rc;
        }
        b->members.push_back(g);
    }
    b->device = b->members[0]->device;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device) != hipSuccess || cus < 1)
        cus = 256;
    // four wavefronts per SIMD: two resident (the two-step kernel's
    // occupancy), and a second round that takes over as the first drains
    b->n_blocks = cus * 16 / b->wpb;
    // the extraction points of all members, in member order
    std::vector<BatchExtPoint> pts;
    for (teuk_grid* g : b->members)
        for (const ExtPoint& e : g->ext) {
            BatchExtPoint q{};
            q.u[0] = g->u(0);
            q.u[1] = g->u(1);
            q.pitch = g->L.pitch;
            q.e = e;
            pts.push_back(q);
        }
    b->n_points = (int)pts.size();
    hipError_t e = hipSuccess;
    if (!pts.empty()) {
        e = hipMemcpyAsync(b->ws + b->ext_off, pts.data(), pts.size() * sizeof(BatchExtPoint), hipMemcpyHostToDevice,
                           b->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    }
    if (e != hipSuccess) {
        for (teuk_grid* m : b->members) teuk_free(m);
        delete b;
        return fail(TEUK_E_HIP, "uploading the extraction points: %s", hipGetErrorString(e));
    }
    if (int rc = batch_upload(b)) {
        for (teuk_grid* m : b->members) teuk_free(m);
        delete b;
        return rc;
    }
    *out = b;
    return TEUK_OK;
}

int teuk_batch_set_initial_data(teuk_batch* b, int32_t member, const void* d_phi, const void* d_pi) {
    if (int rc = batch_check(b, member)) return rc;
    if (!d_phi || !d_pi) return fail(TEUK_E_INVALID_ARG, "initial data pointers are NULL");
    teuk_grid* g = b->members[member];
    if (int rc = set_device(g)) return rc;
    const int nr = (int)g->p.nr, nth = (int)g->p.ntheta;
    HIP_TRY(launch_import(static_cast<const double2*>(d_phi), static_cast<const double2*>(d_pi), g->u(b->parity),
                          nr, nth, g->L.pitch, g->stream));
    g->cur = b->parity;
    g->steps = 0;
    return TEUK_OK;
}

int teuk_batch_get_state(teuk_batch* b, int32_t member, void* d_phi, void* d_pi) {
    if (int rc = batch_check(b, member)) return rc;
    return teuk_get_state(b->members[member], d_phi, d_pi);
}

int teuk_batch_step_n(teuk_batch* b, int64_t n) {
    if (int rc = batch_check(b, 0)) return rc;
    if (n < 0) return fail(TEUK_E_INVALID_ARG, "n=%lld < 0", (long long)n);
    if (n == 0) return TEUK_OK;
    if (int rc = set_device(b->members[0])) return rc;
    // every launch flips the parity; whole graphs (two launches) start from
    // parity 0; the last steps run as in step_n_impl
    const int most = batch_pass_steps(b);
    int64_t left = n;
    while (left > 0) {
        if (b->parity == 0 && left >= 2 * most && !(most == 3 && left == 7)) {
            if (!b->exec)  // captured once per launch configuration
                if (int rc = batch_capture(b)) return rc;
            HIP_TRY(hipGraphLaunch(b->exec, b->stream));
            left -= 2 * most;
            continue;
        }
        const int m = batch_next_steps(most, left);
        if (int rc = batch_launch(b, b->parity, m, b->stream)) return rc;
        b->parity = 1 - b->parity;
        left -= m;
    }
    b->steps += n;
    for (teuk_grid* g : b->members) {
        g->cur = b->parity;
        g->steps += n;
    }
    return TEUK_OK;
}

int teuk_batch_step_samples(teuk_batch* b, int64_t n_samples, int64_t every, void* d_out) {
    if (int rc = batch_check(b, 0)) return rc;
    if (n_samples < 0 || every < 1) return fail(TEUK_E_INVALID_ARG, "need n_samples >= 0 and every >= 1");
    if (b->n_points == 0) return fail(TEUK_E_STATE, "no member has extraction points");
    if (n_samples > 0 && !d_out) return fail(TEUK_E_INVALID_ARG, "output pointer is NULL");
    if (every > INT64_MAX / std::max<int64_t>(n_samples, 1))
        return fail(TEUK_E_INVALID_ARG, "n_samples * every out of range");
    double2* out = static_cast<double2*>(d_out);
    if (!b->fused || every > 16) {  // points that share a tile, or samples too rare to cut the passes
        for (int64_t k = 0; k < n_samples; ++k) {
            if (int rc = teuk_batch_step_n(b, every)) return rc;
            if (int rc = teuk_batch_extract(b, out + k * b->n_points)) return rc;
        }
        return TEUK_OK;
    }
    if (int rc = set_device(b->members[0])) return rc;
    const int most = batch_pass_steps(b);
    const int64_t n = n_samples * every;
    for (int64_t k = 0; k < n;) {
        const int m = batch_next_steps(most, n - k);
        BatchSeries rows{};
        for (int j = 0; j < m; ++j) {  // the state after k + j steps
            const int64_t at = k + j;
            rows.row[j] = at > 0 && at % every == 0 ? out + (at / every - 1) * b->n_points : nullptr;
        }
        if (int rc = batch_launch(b, b->parity, m, b->stream, rows)) return rc;
        b->parity = 1 - b->parity;
        k += m;
    }
    b->steps += n;
    for (teuk_grid* g : b->members) {
        g->cur = b->parity;
        g->steps += n;
    }
    return n > 0 ? teuk_batch_extract(b, out + (n_samples - 1) * b->n_points) : TEUK_OK;
}

int teuk_batch_set_launch(teuk_batch* b, int32_t rows_per_tile, int32_t waves_per_block, int32_t n_blocks) {
    if (int rc = batch_check(b, 0)) return rc;
    if (rows_per_tile < 1 || rows_per_tile > 4096)
        return fail(TEUK_E_INVALID_ARG, "rows_per_tile=%d outside [1, 4096]", rows_per_tile);
    if (waves_per_block != 1 && waves_per_block != 2 && waves_per_block != 4 && waves_per_block != 8)
        return fail(TEUK_E_INVALID_ARG, "waves_per_block=%d not in {1, 2, 4, 8}", waves_per_block);
    if (n_blocks < 1 || n_blocks > (1 << 20)) return fail(TEUK_E_INVALID_ARG, "n_blocks=%d out of range", n_blocks);
    if (int rc = set_device(b->members[0])) return rc;
    HIP_TRY(hipStreamSynchronize(b->stream));  // in-flight launches read the old descriptors
    batch_drop_graph(b);
    b->rows = rows_per_tile;
    b->wpb = waves_per_block;
    b->n_blocks = n_blocks;
    return batch_upload(b);
}

int teuk_batch_set_steps_per_pass(teuk_batch* b, int32_t steps_per_pass) {
    if (int rc = batch_check(b, 0)) return rc;
    if (steps_per_pass != 1 && steps_per_pass != 2)
        return fail(TEUK_E_INVALID_ARG, "steps_per_pass=%d not in {1, 2}", steps_per_pass);
    if (steps_per_pass == b->steps_per_pass) return TEUK_OK;
    if (int rc = set_device(b->members[0])) return rc;
    HIP_TRY(hipStreamSynchronize(b->stream));
    batch_drop_graph(b);
    b->steps_per_pass = steps_per_pass;
    return TEUK_OK;
}

int teuk_batch_get_launch(const teuk_batch* b, int32_t* rows_per_tile, int32_t* waves_per_block,
                          int32_t* n_blocks) {
    if (int rc = batch_check(b, 0)) return rc;
    if (rows_per_tile) *rows_per_tile = b->rows;
    if (waves_per_block) *waves_per_block = b->wpb;
    if (n_blocks) *n_blocks = b->n_blocks;
    return TEUK_OK;
}

int teuk_batch_extract(teuk_batch* b, void* d_out) {
    if (int rc = batch_check(b, 0)) return rc;
    if (b->n_points == 0) return fail(TEUK_E_STATE, "no member has extraction points");
    if (!d_out) return fail(TEUK_E_INVALID_ARG, "output pointer is NULL");
    if (int rc = set_device(b->members[0])) return rc;
    HIP_TRY(launch_batch_extract(reinterpret_cast<const BatchExtPoint*>(b->ws + b->ext_off), b->n_points, b->parity,
                                 static_cast<double2*>(d_out), b->stream));
    return TEUK_OK;
}

int32_t teuk_batch_n_extract(const teuk_batch* b) { return b ? b->n_points : -1; }

int teuk_assemble_modes(int64_t n_samples, int32_t n_modes, const int32_t* h_m, int32_t n_obs, const double* h_phi,
                        const double* h_r, const void* d_samples, void* d_psi, void* hip_stream) {
    if (n_samples < 0) return fail(TEUK_E_INVALID_ARG, "n_samples=%lld < 0", (long long)n_samples);
    if (n_modes < 1 || n_modes > kMaxModes) return fail(TEUK_E_INVALID_ARG, "n_modes=%d outside [1, %d]", n_modes, kMaxModes);
    if (n_obs < 1 || n_obs > kMaxObservers) return fail(TEUK_E_INVALID_ARG, "n_obs=%d outside [1, %d]", n_obs, kMaxObservers);
    if (!h_m || !h_phi || !h_r) return fail(TEUK_E_INVALID_ARG, "mode or observer arrays are NULL");
    if (n_samples > 0 && (!d_samples || !d_psi)) return fail(TEUK_E_INVALID_ARG, "device pointers are NULL");
    AssembleArgs a{};
    a.n_modes = n_modes;
    a.n_obs = n_obs;
    for (int j = 0; j < n_modes; ++j) a.m[j] = h_m[j];
    for (int o = 0; o < n_obs; ++o) {
        if (!std::isfinite(h_phi[o]) || !std::isfinite(h_r[o]) || !(h_r[o] > 0.0))
            return fail(TEUK_E_INVALID_ARG, "observer %d: need finite phi and r > 0", o);
        a.phi[o] = h_phi[o];
        a.r3[o] = h_r[o] * h_r[o] * h_r[o];
    }
    HIP_TRY(launch_assemble(a, n_samples, static_cast<const double2*>(d_samples), static_cast<double2*>(d_psi),
                            reinterpret_cast<hipStream_t>(hip_stream)));
    return TEUK_OK;
}

int64_t teuk_batch_total_points(const teuk_batch* b) {
    if (!b) return -1;
    int64_t n = 0;
    for (const teuk_grid* g : b->members) n += g->p.nr * g->p.ntheta;
    return n;
}

int teuk_batch_free(teuk_batch* b) {
    if (!b) return TEUK_OK;
    hipError_t e = hipStreamSynchronize(b->stream);
    batch_drop_graph(b);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (teuk_grid* g : b->members) teuk_free(g);
    delete b;
    if (e != hipSuccess) return fail(TEUK_E_HIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    return TEUK_OK;
}

int teuk_free(teuk_grid* g) {
    if (!g) return TEUK_OK;
    hipError_t e = hipStreamSynchronize(g->stream);
    delete g;
    if (e != hipSuccess) return fail(TEUK_E_HIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    return TEUK_OK;
}

}  // extern "C"
