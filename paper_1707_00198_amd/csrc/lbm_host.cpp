// Host runtime of lbmcg: parameter validation, node classification, wall normals, memory
// layout, tile schedule and the C entry points declared in include/lbmcg.h.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "lbm_internal.h"
#include "lbmcg.h"

using namespace lbmcg;

static_assert(WET_SCHEME_B == LBM_WET_SCHEME_B && WET_SURFACE_ENERGY == LBM_WET_SURFACE_ENERGY,
              "device wetting flags follow the interface's");

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_OK(expr)                                                                      \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return fail(LBM_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));      \
    } while (0)

const int EXH[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
const int EYH[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
const double WH[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                      1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

size_t storage_bytes(int storage) { return storage == 0 ? 8 : (storage == 1 ? 4 : 2); }  // 2: f16, 3: c16
size_t colour_bytes(int storage) { return storage == 0 ? 8 : 4; }

// Byte offsets of every region, shared by query and create.
struct Layout {
    size_t plane = 0;         // elements per node plane
    size_t rows = 0;          // total rows (inlet / outlet arrays)
    size_t items_cap = 0;     // work-item capacity
    int bpd = 0;              // mass-reduction blocks per domain
    // state
    size_t buf[2] = {0, 0}, f_bytes = 0, c_off = 0, vx_off = 0, vy_off = 0, hist[2] = {0, 0};
    size_t state_bytes = 0;
    // scratch
    size_t mask = 0, ns = 0, inlet = 0, doms = 0, items = 0, partials = 0, flag = 0, scratch_bytes = 0;
};

int strips_of(const lbm_domain_desc &d, const TileShape &t, int storage) {
    return (d.nx + t.out(storage) - 1) / t.out(storage);
}

Layout make_layout(const lbm_domain_desc *d, int n, int storage) {
    Layout L;
    size_t nodes = 0, rows = 0, cap = 0;
    for (int i = 0; i < n; i++) {
        nodes += align_up((size_t)d[i].nx * d[i].ny, 64);
        rows += d[i].ny;
        cap += (size_t)strips_of(d[i], {64, 4, 1, 1}, 0) * ((d[i].ny + 7) / 8);  // the narrowest strips
    }
    L.plane = align_up(std::max<size_t>(nodes, 64), 128);
    L.rows = rows;
    L.items_cap = cap;
    // mass-reduction blocks per domain: about 4096 blocks in all (16 per CU), so that a single
    // large domain is not summed by a handful of blocks; 16 to 1024 per domain
    L.bpd = std::max(16, std::min(1024, (4096 + n - 1) / n));
    const size_t sb = storage_bytes(storage), cb = colour_bytes(storage);
    size_t o = 0;
    for (int b = 0; b < 2; b++) {
        L.buf[b] = o;
        o += align_up(9 * L.plane * sb, 256) + 3 * align_up(L.plane * cb, 256);
    }
    L.f_bytes = align_up(9 * L.plane * sb, 256);
    L.c_off = L.f_bytes;
    L.vx_off = L.c_off + align_up(L.plane * cb, 256);
    L.vy_off = L.vx_off + align_up(L.plane * cb, 256);
    for (int b = 0; b < 2; b++) {
        L.hist[b] = o;
        o += align_up(3 * rows * cb, 256);
    }
    L.state_bytes = o;
    o = 0;
    L.mask = o;
    o += align_up(L.plane * 2, 256);
    L.ns = o;  // wall normal (x, y) per node, interleaved
    o += align_up(2 * L.plane * cb, 256);
    L.inlet = o;
    o += align_up(rows * cb, 256);
    L.doms = o;
    o += align_up(n * sizeof(DomDev), 256);
    L.items = o;
    o += align_up(cap * sizeof(WorkItem), 256);
    L.partials = o;
    o += align_up((size_t)n * L.bpd * 2 * sizeof(double), 256);
    L.flag = o;
    o += 256;
    L.scratch_bytes = o;
    return L;
}

int validate(const lbm_domain_desc *d, int n, int storage) {
    if (!d || n <= 0) return fail(LBM_EINVAL, "need at least one domain");
    if (storage < 0 || storage > 3) return fail(LBM_EINVAL, "unknown storage %d", storage);
    for (int i = 0; i < n; i++) {
        const lbm_domain_desc &q = d[i];
        if (q.nx < 1 || q.ny < 1) return fail(LBM_EINVAL, "domain %d: bad extent %dx%d", i, q.nx, q.ny);
        if ((long long)q.nx * q.ny > (1LL << 31)) return fail(LBM_EINVAL, "domain %d too large", i);
        if (q.open_x && q.nx < 2) return fail(LBM_EINVAL, "domain %d: open x needs nx >= 2", i);
        if (q.wetting & ~(LBM_WET_SCHEME_B | LBM_WET_SURFACE_ENERGY))
            return fail(LBM_EINVAL, "domain %d: unknown wetting flags 0x%x", i, (unsigned)q.wetting);
        if (!q.solid || !q.rho_r0 || !q.rho_b0) return fail(LBM_EINVAL, "domain %d: missing array", i);
        if (q.open_x && !q.inlet_ux) return fail(LBM_EINVAL, "domain %d: open x needs inlet_ux", i);
        if (!(q.nu_r > 0) || !(q.nu_b > 0)) return fail(LBM_EINVAL, "domain %d: viscosity must be > 0 (tau > 1/2)", i);
        if (!(q.sigma >= 0)) return fail(LBM_EINVAL, "domain %d: sigma must be >= 0", i);
        if (!(q.beta >= 0 && q.beta <= 1)) return fail(LBM_EINVAL, "domain %d: beta outside [0, 1]", i);
        if (!(q.theta_deg >= 0 && q.theta_deg <= 180)) return fail(LBM_EINVAL, "domain %d: theta outside [0, 180]", i);
        for (double s : {q.s_e, q.s_eps, q.s_q})
            if (!(s > 0 && s < 2)) return fail(LBM_EINVAL, "domain %d: relaxation rate outside (0, 2)", i);
        if (!(q.rho0 > 0) || !(q.eps > 0) || !(q.outlet_u >= 0))
            return fail(LBM_EINVAL, "domain %d: rho0, eps must be > 0 and outlet_u >= 0", i);
        const size_t nn = (size_t)q.nx * q.ny;
        for (size_t k = 0; k < nn; k++) {
            if (q.solid[k]) continue;
            const double rr = q.rho_r0[k], rb = q.rho_b0[k];
            if (!(std::isfinite(rr) && std::isfinite(rb) && rr >= 0 && rb >= 0 && rr + rb > 0))
                return fail(LBM_EINVAL, "domain %d: invalid initial density at node %zu", i, k);
        }
        if (q.open_x)
            for (int y = 0; y < q.ny; y++)
                if (!(std::isfinite(q.inlet_ux[y]) && std::fabs(q.inlet_ux[y]) < 0.5))
                    return fail(LBM_EINVAL, "domain %d: inlet velocity must be finite and |u| < 0.5", i);
    }
    return LBM_OK;
}

// Eighth-order isotropic estimate of the wall normal (Eqs. 32-33), pointing into the solid.
// Beyond an open x edge the stencil sees fluid.
void e8_normal(const lbm_domain_desc &q, int x, int y, double &nx, double &ny) {
    double sx = 0.0, sy = 0.0;
    for (int cy = -2; cy <= 2; cy++)
        for (int cx = -2; cx <= 2; cx++) {
            const int r2 = cx * cx + cy * cy;
            double w;
            switch (r2) {
                case 1: w = 4.0 / 21.0; break;
                case 2: w = 4.0 / 45.0; break;
                case 4: w = 1.0 / 60.0; break;
                case 5: w = 2.0 / 315.0; break;
                case 8: w = 1.0 / 5040.0; break;
                default: continue;
            }
            int xx = x + cx;
            const int yy = ((y + cy) % q.ny + q.ny) % q.ny;
            if (q.open_x && (xx < 0 || xx >= q.nx)) continue;
            xx = ((xx % q.nx) + q.nx) % q.nx;
            if (!q.solid[(size_t)yy * q.nx + xx]) continue;
            sx += w * cx;
            sy += w * cy;
        }
    const double m = std::sqrt(sx * sx + sy * sy);
    nx = m > 0 ? sx / m : 0.0;
    ny = m > 0 ? sy / m : 0.0;
}

// Class word of node (x, y) (see lbm_internal.h) and, on outermost fluid nodes, the wall
// normal: the caller's analytic one (normalised) or the eighth-order estimate.
uint32_t node_class(const lbm_domain_desc &q, int x, int y, double &nsx, double &nsy) {
    auto solid_at = [&](int xx, int yy) -> bool {
        yy = ((yy % q.ny) + q.ny) % q.ny;
        if (q.open_x) xx = std::min(std::max(xx, 0), q.nx - 1);
        else xx = ((xx % q.nx) + q.nx) % q.nx;
        return q.solid[(size_t)yy * q.nx + xx] != 0;
    };
    const size_t k = (size_t)y * q.nx + x;
    const bool s = q.solid[k] != 0;
    uint32_t m = s ? SELF_SOLID : 0u;
    bool other = false;
    for (int a = 1; a < 9; a++) {
        const bool sn = solid_at(x + EXH[a], y + EYH[a]);
        if (sn) m |= 1u << (a - 1);
        if (sn != s) other = true;
    }
    if (other) m |= s ? SOLID_BND : FLUID_BND;
    nsx = nsy = 0.0;
    if (!s && other) {
        if (q.ns) {
            nsx = q.ns[2 * k];
            nsy = q.ns[2 * k + 1];
            const double mg = std::sqrt(nsx * nsx + nsy * nsy);
            nsx = mg > 0 ? nsx / mg : 0.0;
            nsy = mg > 0 ? nsy / mg : 0.0;
        } else {
            e8_normal(q, x, y, nsx, nsy);
        }
    }
    return m;
}

template <class T>
T encode(double v, float scale);
template <>
double encode<double>(double v, float) { return v; }
template <>
float encode<float>(double v, float) { return (float)v; }
template <>
__half encode<__half>(double v, float scale) { return __float2half_rn((float)(v * scale)); }
// The 16-bit format of C16 from exact double arithmetic (round to nearest, ties to even).
template <>
C16 encode<C16>(double v, float scale) {
    const double x = std::fabs(v * scale);
    uint32_t r;
    if (!(x >= 0x1p-6)) {
        r = (uint32_t)std::nearbyint(x * 0x1p17);  // subnormal; 2048 is the smallest normal
    } else {
        int ex;
        const double fr = std::frexp(x, &ex);  // x = fr 2^ex, fr in [0.5, 1)
        const int e = std::min(ex - 1 + 7, 16);
        // a rounding carry (fraction 2048) moves into the exponent
        r = ((uint32_t)e << 11) + (uint32_t)std::nearbyint((2.0 * fr - 1.0) * 2048.0);
    }
    r = std::min<uint32_t>(r, 0x7FFFu);
    return C16{(uint16_t)(r | (std::signbit(v) ? 0x8000u : 0u))};
}

}  // namespace

struct lbm_ctx {
    int n = 0, storage = 0;
    hipStream_t stream = nullptr;
    char *state = nullptr, *scratch = nullptr;
    Layout L;
    std::vector<lbm_domain_desc> desc;   // host pointers are not kept valid: sizes only
    std::vector<DomDev> doms;
    std::vector<WorkItem> items;
    // rows per work item, wavefronts (tile rows advanced per iteration), wavefronts side by side
    // in a tile row, and node columns per lane (2: pair kernel) of the step
    TileShape tile{0, 0, 1, 1};
    bool variants = false;  // some domain uses a wetting variant (LBM_WET_*)
    int parity = 0;   // buffer holding the current state
    int own = 1;      // current state is a node-local snapshot
    int64_t steps = 0;
    double *mass_host = nullptr;
    int *flag_host = nullptr;
    // diagnostics: caller's device buffer (lbm_diag_attach), pinned staging, snapshot state
    char *diag = nullptr;
    double *diag_host = nullptr;
    int *rows_host = nullptr;
    bool snap_valid = false;
    bool snap_first = false;  // the snapshot is the first of the two velocity buffers
    int max_fluid_bnd = 0;  // largest number of outermost fluid nodes in one domain
    size_t max_nodes = 1;   // nodes of the largest domain
    // step graphs: `graph_steps` step launches captured once on a private stream, one graph per
    // parity a replay starts from (graph_steps is even, so a replay ends on the same parity)
    int graph_steps = 0;
    hipStream_t cap = nullptr;
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    // device current at lbm_create, and its static staging array of lbm_diag_crossings_noalloc
    int device = 0;
    void *noalloc = nullptr;
};

namespace {

template <class T, class AT>
void fill_args(const lbm_ctx *c, int parity, StepArgs<T, AT> &A) {
    const Layout &L = c->L;
    A.doms = reinterpret_cast<const DomDev *>(c->scratch + L.doms);
    A.items = reinterpret_cast<const WorkItem *>(c->scratch + L.items);
    A.n_items = (int)c->items.size();
    A.own = c->own;
    char *bi = c->state + L.buf[parity], *bo = c->state + L.buf[1 - parity];
    A.fin = reinterpret_cast<const T *>(bi);
    A.cin = reinterpret_cast<const AT *>(bi + L.c_off);
    A.vxin = reinterpret_cast<const AT *>(bi + L.vx_off);
    A.vyin = reinterpret_cast<const AT *>(bi + L.vy_off);
    A.fout = reinterpret_cast<T *>(bo);
    A.cout = reinterpret_cast<AT *>(bo + L.c_off);
    A.vxout = reinterpret_cast<AT *>(bo + L.vx_off);
    A.vyout = reinterpret_cast<AT *>(bo + L.vy_off);
    A.hist_in = reinterpret_cast<const AT *>(c->state + L.hist[parity]);
    A.hist_out = reinterpret_cast<AT *>(c->state + L.hist[1 - parity]);
    A.mask = reinterpret_cast<const uint16_t *>(c->scratch + L.mask);
    A.ns = reinterpret_cast<const AT *>(c->scratch + L.ns);
    A.inlet = reinterpret_cast<const AT *>(c->scratch + L.inlet);
    A.plane = L.plane;
    A.flag = reinterpret_cast<int *>(c->scratch + L.flag);
    A.f_plane_bytes = (uint32_t)(L.plane * sizeof(T));
    A.f_set_bytes = (uint32_t)(9 * L.plane * sizeof(T));
    A.c_plane_bytes = (uint32_t)(L.vx_off - L.c_off);
    A.ns_bytes = (uint32_t)(2 * L.plane * sizeof(AT));
}

// Arguments for the current parity, as raw bytes of the storage's StepArgs instantiation.
struct AnyArgs {
    alignas(16) unsigned char bytes[sizeof(StepArgs<double, double>)];
};

// Layout of the diagnostics buffer: velocity (u_x, u_y planes at the colour-plane stride) and its
// snapshot, which change places when a snapshot is taken, reduction partials, and the contact-line
// counter and list (room for every outermost fluid node of the largest domain).  Results and row
// lists are in pinned host memory, which the kernels access directly.
struct DiagLayout {
    size_t u = 0, snap = 0, part = 0, cl_count = 0, cl_list = 0, bytes = 0;
};
DiagLayout diag_layout(const lbm_ctx *c) {
    DiagLayout D;
    const size_t cp = c->L.vx_off - c->L.c_off;
    size_t o = 0;
    D.u = c->snap_first ? 2 * cp : 0;
    D.snap = c->snap_first ? 0 : 2 * cp;
    o += 4 * cp;
    D.part = o;
    o += align_up(std::max<size_t>((size_t)c->n * DIAG_BLOCKS * 2, DIAG_BLOCKS * 4) * sizeof(double), 256);
    D.cl_count = o;
    o += 256;
    D.cl_list = o;
    o += align_up(std::max<size_t>((size_t)c->max_fluid_bnd, 1) * sizeof(int32_t), 256);
    D.bytes = o;
    return D;
}

template <class T, class AT>
void set_diag_t(StepArgs<T, AT> &A, void *u, void *cl_list, void *cl_count, int cl_cap, int cl_dom) {
    A.u_out = static_cast<AT *>(u);
    A.diag = 1;
    A.cl_list = static_cast<int32_t *>(cl_list);
    A.cl_count = static_cast<int *>(cl_count);
    A.cl_cap = cl_cap;
    A.cl_dom = cl_dom;
}

AnyArgs make_args(const lbm_ctx *c, int parity) {
    AnyArgs a;
    std::memset(&a, 0, sizeof a);
    if (c->storage == 0) fill_args(c, parity, *reinterpret_cast<StepArgs<double, double> *>(a.bytes));
    else if (c->storage == 1) fill_args(c, parity, *reinterpret_cast<StepArgs<float, float> *>(a.bytes));
    else if (c->storage == 2) fill_args(c, parity, *reinterpret_cast<StepArgs<__half, float> *>(a.bytes));
    else fill_args(c, parity, *reinterpret_cast<StepArgs<C16, float> *>(a.bytes));
    return a;
}

// Arguments of a diagnostic launch on the current state: velocity into the diagnostics buffer,
// and, for cl_dom >= 0, the contact-line list of that domain.
AnyArgs make_diag_args(const lbm_ctx *c, int cl_dom = -1) {
    AnyArgs a = make_args(c, c->parity);
    const DiagLayout DL = diag_layout(c);
    void *u = c->diag + DL.u;
    void *list = cl_dom >= 0 ? c->diag + DL.cl_list : nullptr;
    void *count = cl_dom >= 0 ? c->diag + DL.cl_count : nullptr;
    const int cap = c->max_fluid_bnd;
    if (c->storage == 0) set_diag_t(*reinterpret_cast<StepArgs<double, double> *>(a.bytes), u, list, count, cap, cl_dom);
    else if (c->storage == 1) set_diag_t(*reinterpret_cast<StepArgs<float, float> *>(a.bytes), u, list, count, cap, cl_dom);
    else if (c->storage == 2) set_diag_t(*reinterpret_cast<StepArgs<__half, float> *>(a.bytes), u, list, count, cap, cl_dom);
    else set_diag_t(*reinterpret_cast<StepArgs<C16, float> *>(a.bytes), u, list, count, cap, cl_dom);
    return a;
}

// Work items, in the order the step kernel takes them.  The kernel deals blocks round-robin to
// the 8 XCDs and gives XCD x the x-th of 8 equal consecutive runs of this list, so the order
// decides which items share an L2 and run at the same time.  Within a domain the items are
// band-major (all strips of a band of rows, then the next band): the blocks in flight then
// stream a narrow band of every plane, which measured markedly faster than a strip at a time.
// A domain with more items than one run is cut into strip groups of about one run each, so
// that every XCD works through a compact region and neighbouring strips share its L2.
std::vector<WorkItem> build_items(const std::vector<lbm_domain_desc> &d, const TileShape &t, int storage) {
    const int chunk = t.chunk;
    size_t total = 0;
    for (const auto &q : d) {
        const int nch = std::max(1, (q.ny + chunk - 1) / chunk);
        total += (size_t)strips_of(q, t, storage) * nch;
    }
    const size_t run = std::max<size_t>(1, total / 8);
    std::vector<WorkItem> out;
    out.reserve(total);
    for (int i = 0; i < (int)d.size(); i++) {
        const int ny = d[i].ny, S = strips_of(d[i], t, storage);
        const int nch = std::max(1, (ny + chunk - 1) / chunk);
        const int ch = ((ny + nch - 1) / nch + 3) / 4 * 4;
        const size_t items = (size_t)S * nch;
        const int groups = (int)std::min<size_t>(S, std::max<size_t>(1, (items + run / 2) / run));
        for (int g = 0; g < groups; g++) {
            const int s0 = (int)((long long)S * g / groups), s1 = (int)((long long)S * (g + 1) / groups);
            for (int k = 0; k < nch; k++) {
                const int y0 = k * ch, y1 = std::min(ny, y0 + ch);
                if (y0 >= y1) continue;
                for (int s = s0; s < s1; s++) out.push_back(WorkItem{i, s * t.out(storage), y0, y1});
            }
        }
    }
    return out;
}

// Tallest chunk, up to 64 rows, that still yields 4096 work items.  Taller chunks repeat fewer
// halo rows, but with the band-major order shorter bands measured faster on wide domains
// (16384 x 512: 32 rows best), and enough items keep every CU busy on small ones.  Below that,
// 16 or 12 rows as long as they give 512 items (two blocks per CU): batches of 60-row channels
// (15 or 44 of 630 x 60) ran 15-23 % faster in 16-row chunks than in 8-row ones, whose halo
// rows double the work, while a single 2000 x 100 channel (266 items at 16 rows) ran fastest
// in 8-row chunks, where more items outweigh the halo.  FP64 marches fewer blocks at a time and
// takes 32 rows from 2400 items on: 24 cylinder boxes 400 x 400 201 us against 220 in 16-row
// chunks, 16384 x 256 249 against 254, 30 channels of the sweep 396 against 417.
int auto_chunk(const std::vector<lbm_domain_desc> &d, TileShape t, int storage) {
    const auto items = [&](int ch) {
        t.chunk = ch;
        return build_items(d, t, storage).size();
    };
    for (int ch : {64, 48, 32, 24})
        if (items(ch) >= 4096) return ch;
    if (storage == 0 && items(32) >= 2400) return 32;
    for (int ch : {16, 12})
        if (items(ch) >= 512) return ch;
    return 8;
}

// Blocks of 4 tile rows (one wavefront per SIMD) measured at least as fast as blocks of 8 for
// every storage type.
constexpr int DEFAULT_WAVES = 4;
// One-wavefront tiles.  Tiles two wavefronts wide (120 output columns of 128; 118 with FP64
// arithmetic) repeat fewer halo columns but measured 6 % slower on the sweep (1.67 against 1.57 ms
// a step in binary16: 8-wavefront barriers, 2 blocks per CU).
constexpr int DEFAULT_COLS = 1;
// The built-in shape of a batch: the patch kernel, which takes a work item at once, while its
// repeated halo rows cost less than the march's iterations (us per step on an MI355X, patch
// against the best march):
//  FP32 arithmetic: items of 8 rows up to 1408 of them, then of 24.  Above, 24 rows won wherever
//    measured (15 channels 630 x 60, 1440 items of 8 rows, 20.8 / 22.4 against 22.7 / 22.5 in FP32 /
//    binary16, four cylinder boxes 400 x 400, 1600 items, 18.7 / 19.9 against 23.7 / 23.5); from 1050
//    on it depends on the lattices (12 channels 16.2 / 17.2 against 19.7 / 19.5, three boxes, 1200
//    items, 19.4 / 19.8 against 19.0 / 18.4); 234 items take 8.2 with 8 rows, the march 20.
//    Items of 24 rows against the march: 44 channels 42.5 / 42.5 against 63, 16384 x 512 218 / 176
//    against 250 / 186, 60 channels of the sweep, 13212 items, 386 / 317 against 449 / 328.  FP32 stays
//    ahead (150 of these channels 941 against 1056).  In the 16-bit storages up to 16384 items: 367
//    against 373 at 15414 items, 495 against 488 at 20919.
//  FP64: items of 8 rows up to 8192 (234 items 10.3 against 21.7, 4224 items 98 against 119, 8160
//    items, 85 channels, 202 against 208, 8000 items, 20 cylinder boxes, 180 against 189; 9600
//    items, 24 cylinder boxes, 213 against 201), with wetting variants likewise (4224 items 94
//    against 119, 7800 items, 200 closed boxes, 207 against 220).
//  Lattices of 25 to 31 rows are two items of less than two thirds of the 24 rows; beyond 8192 such
//    items the march, which takes each lattice as one of more than 4096 items, is faster: 500 channels
//    630 x 28 277 / 240 against 301 / 273 (FP32 / binary16, 12000 items), 270 of them 186 / 160
//    against 171 / 146 (6480 items); 500 channels of 36 rows 351 / 290 against 341 / 305.
constexpr size_t PATCH_ITEMS = 1408, PATCH_TALL_ITEMS_16 = 16384, PATCH_ITEMS_F64 = 8192, PATCH_HALF_ITEMS = 8192;
bool half_empty(const std::vector<lbm_domain_desc> &d, const TileShape &tall, int storage) {
    size_t items = 0, rows = 0;
    for (const auto &q : d)
        if (q.ny > PATCH_TALL_ROWS) {
            const size_t s = (size_t)strips_of(q, tall, storage);
            items += s * ((q.ny + PATCH_TALL_ROWS - 1) / PATCH_TALL_ROWS);
            rows += s * q.ny;
        }
    return items > PATCH_HALF_ITEMS && 3 * rows < 2 * PATCH_TALL_ROWS * items;
}
TileShape builtin_tile(const std::vector<lbm_domain_desc> &d, int storage) {
    const TileShape patch{PATCH_ROWS, 8, 1, 1}, tall{PATCH_TALL_ROWS, 8, 1, 1};
    if (build_items(d, patch, storage).size() <= (storage == 0 ? PATCH_ITEMS_F64 : PATCH_ITEMS)) return patch;
    if ((storage == 1 || (storage > 1 && build_items(d, tall, storage).size() <= PATCH_TALL_ITEMS_16)) &&
        !half_empty(d, tall, storage))
        return tall;
    TileShape t{0, DEFAULT_WAVES, DEFAULT_COLS, 1};
    t.chunk = auto_chunk(d, t, storage);
    return t;
}
// The pair kernel (two node columns per lane) needs FP32 arithmetic and an even width in every
// domain.  It is offered to lbm_set_tile and the autotuner but is not the built-in choice: at the
// two wavefronts per SIMD its register use allows, it measured slower than the one-column kernel
// at five (binary16 sweep 45.6 against 52.4 GLUPS).
bool pair_allowed(int storage, const std::vector<lbm_domain_desc> &d) {
    if (storage == 0) return false;
    for (const auto &q : d)
        if (q.nx % 2) return false;
    return true;
}

int upload_items(lbm_ctx *c) {
    if (c->items.size() > c->L.items_cap) return fail(LBM_EINVAL, "work-item table overflow");
    HIP_OK(hipMemcpyAsync(c->scratch + c->L.items, c->items.data(),
                          c->items.size() * sizeof(WorkItem), hipMemcpyHostToDevice, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

// One step launched directly on stream s, with the context's current arguments.
hipError_t step_once(lbm_ctx *c, hipStream_t s) {
    AnyArgs a = make_args(c, c->parity);
    const hipError_t e = launch_step(c->storage, a.bytes, (int)c->items.size(), c->tile, c->variants, s);
    if (e != hipSuccess) return e;
    c->parity ^= 1;
    c->own = 0;
    c->steps++;
    return hipSuccess;
}

void drop_graphs(lbm_ctx *c) {
    for (auto &g : c->gexec)
        if (g) {
            (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
}

// Capture graph_steps step launches starting from `parity` (the state then being no snapshot)
// on the private stream and instantiate them.  The context's parity, flags and step count are
// left as they were: lbm_step advances them per replay.
int build_graph(lbm_ctx *c, int parity) {
    if (!c->cap) HIP_OK(hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking));
    const int p0 = c->parity, own0 = c->own;
    const int64_t s0 = c->steps;
    HIP_OK(hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal));
    c->parity = parity;
    c->own = 0;
    hipError_t e = hipSuccess;
    for (int k = 0; k < c->graph_steps && e == hipSuccess; k++) e = step_once(c, c->cap);
    hipGraph_t g = nullptr;
    const hipError_t e2 = hipStreamEndCapture(c->cap, &g);
    c->parity = p0;
    c->own = own0;
    c->steps = s0;
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipGraphInstantiateWithFlags(&c->gexec[parity], g, 0);
    // upload now, on the context's stream: otherwise the first replay pays for it (measured
    // 4 ms for 20 launches of the 320-channel sweep, in front of that replay's first kernel)
    if (e == hipSuccess) e = hipGraphUpload(c->gexec[parity], c->stream);
    if (g) (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        c->gexec[parity] = nullptr;
        return fail(LBM_EDEVICE, "step graph: %s", hipGetErrorString(e));
    }
    return LBM_OK;
}

template <class T, class AT>
int create_t(lbm_ctx *c, const lbm_domain_desc *d) {
    const Layout &L = c->L;
    const size_t P = L.plane;
    std::vector<uint16_t> mask(P, (uint16_t)SELF_SOLID);
    std::vector<AT> ns(2 * P, AT(0)), inlet(std::max<size_t>(L.rows, 1), AT(0));
    std::vector<T> f(9 * P, encode<T>(0.0, 1.0f));
    std::vector<AT> col(3 * P, AT(0));  // c, vx, vy
    std::vector<AT> hist(3 * std::max<size_t>(L.rows, 1), AT(0));
    long long off = 0, io = 0;
    for (int i = 0; i < c->n; i++) {
        const lbm_domain_desc &q = d[i];
        DomDev &D = c->doms[i];
        const double th = q.theta_deg * M_PI / 180.0;
        D.off = off;
        D.nx = q.nx;
        D.ny = q.ny;
        D.open_x = q.open_x ? 1 : 0;
        D.wetting = q.wetting;
        D.io_off = io;
        DomPar<double> &PD = D.d;
        PD.inv2nu_r = 1.0 / (2.0 * q.nu_r);
        PD.inv2nu_b = 1.0 / (2.0 * q.nu_b);
        PD.half_sigma = 0.5 * q.sigma;
        PD.beta = q.beta;
        PD.cos_t = std::cos(th);
        PD.sin_t = std::sin(th);
        PD.s_e = q.s_e;
        PD.s_eps = q.s_eps;
        PD.s_q = q.s_q;
        PD.ke = 6.0 * (1.0 - 0.5 * q.s_e);
        PD.keps = 6.0 * (1.0 - 0.5 * q.s_eps);
        PD.kq = 1.0 - 0.5 * q.s_q;
        PD.rho0 = q.rho0;
        PD.eps = q.eps;
        PD.outlet_u = q.outlet_u;
        PD.w_rest = WH[0] * q.rho0;
        PD.w_axis = WH[1] * q.rho0;
        PD.w_diag = WH[5] * q.rho0;
        PD.pad[0] = PD.pad[1] = 0.0;
        const double *pd = &PD.rho0;
        float *pf = &D.f.rho0;
        for (size_t k = 0; k < sizeof(DomPar<double>) / sizeof(double); k++) pf[k] = (float)pd[k];
        int n_fluid_bnd = 0;
        for (int y = 0; y < q.ny; y++)
            for (int x = 0; x < q.nx; x++) {
                const size_t k = (size_t)y * q.nx + x, g = off + k;
                double vx, vy;
                const uint32_t m = node_class(q, x, y, vx, vy);
                const bool s = (m & SELF_SOLID) != 0;
                n_fluid_bnd += (m & FLUID_BND) ? 1 : 0;
                mask[g] = (uint16_t)m;
                ns[2 * g] = (AT)vx;
                ns[2 * g + 1] = (AT)vy;
                if (s) continue;
                const double rr = q.rho_r0[k], rb = q.rho_b0[k], rho = rr + rb;
                for (int a = 0; a < 9; a++)
                    f[a * P + g] = encode<T>(WH[a] * (rho - q.rho0), c->storage >= 2 ? fp16_scale(a) : 1.0f);
                col[g] = (AT)(rr / rho);
                if (q.open_x && x == q.nx - 1) {
                    hist[3 * (io + y) + 0] = (AT)(WH[3] * (rho - q.rho0));
                    hist[3 * (io + y) + 1] = (AT)(WH[6] * (rho - q.rho0));
                    hist[3 * (io + y) + 2] = (AT)(WH[7] * (rho - q.rho0));
                }
            }
        c->max_fluid_bnd = std::max(c->max_fluid_bnd, n_fluid_bnd);
        if (q.open_x)
            for (int y = 0; y < q.ny; y++) inlet[io + y] = (AT)q.inlet_ux[y];
        off += (long long)align_up((size_t)q.nx * q.ny, 64);
        io += q.ny;
    }
    hipStream_t s = c->stream;
    char *st = c->state + L.buf[0];
    HIP_OK(hipMemsetAsync(c->state, 0, L.state_bytes, s));
    HIP_OK(hipMemcpyAsync(st, f.data(), 9 * P * sizeof(T), hipMemcpyHostToDevice, s));
    HIP_OK(hipMemcpyAsync(st + L.c_off, col.data(), P * sizeof(AT), hipMemcpyHostToDevice, s));
    HIP_OK(hipMemcpyAsync(c->state + L.hist[0], hist.data(), 3 * L.rows * sizeof(AT),
                          hipMemcpyHostToDevice, s));
    HIP_OK(hipMemsetAsync(c->scratch, 0, L.scratch_bytes, s));
    HIP_OK(hipMemcpyAsync(c->scratch + L.mask, mask.data(), P * 2, hipMemcpyHostToDevice, s));
    HIP_OK(hipMemcpyAsync(c->scratch + L.ns, ns.data(), 2 * P * sizeof(AT), hipMemcpyHostToDevice, s));
    HIP_OK(hipMemcpyAsync(c->scratch + L.inlet, inlet.data(), L.rows * sizeof(AT),
                          hipMemcpyHostToDevice, s));
    HIP_OK(hipMemcpyAsync(c->scratch + L.doms, c->doms.data(), c->n * sizeof(DomDev),
                          hipMemcpyHostToDevice, s));
    HIP_OK(hipStreamSynchronize(s));
    return upload_items(c);
}

}  // namespace

extern "C" {

int lbm_query_bytes(const lbm_domain_desc *domains, int n, int storage, size_t *state_bytes,
                    size_t *scratch_bytes) {
    int rc = validate(domains, n, storage);
    if (rc) return rc;
    Layout L = make_layout(domains, n, storage);
    if (state_bytes) *state_bytes = L.state_bytes;
    if (scratch_bytes) *scratch_bytes = L.scratch_bytes;
    return LBM_OK;
}

int lbm_create(const lbm_domain_desc *domains, int n, int storage, void *state_dev,
               size_t state_bytes, void *scratch_dev, size_t scratch_bytes, void *hip_stream,
               lbm_ctx **out) {
    if (!out) return fail(LBM_EINVAL, "out is NULL");
    *out = nullptr;
    int rc = validate(domains, n, storage);
    if (rc) return rc;
    Layout L = make_layout(domains, n, storage);
    // The step kernel addresses the 9 population planes, the 3 colour-state planes and the
    // interleaved wall normals each as one buffer of fewer than 2^31 bytes.
    if (L.f_bytes >= (size_t(1) << 31) || 3 * (L.vx_off - L.c_off) >= (size_t(1) << 31) ||
        2 * L.plane * (storage == 0 ? 8 : 4) >= (size_t(1) << 31))
        return fail(LBM_EINVAL,
                    "%zu nodes exceed one context's limit (2^31 bytes for the 9 population planes "
                    "and for the 3 colour-state planes); split the domains over several contexts",
                    L.plane);
    if (!state_dev || !scratch_dev) return fail(LBM_EINVAL, "device buffers are NULL");
    if (state_bytes < L.state_bytes || scratch_bytes < L.scratch_bytes)
        return fail(LBM_ENOMEM, "buffers too small: need %zu state and %zu scratch bytes",
                    L.state_bytes, L.scratch_bytes);
    if (((uintptr_t)state_dev | (uintptr_t)scratch_dev) & 255)
        return fail(LBM_EINVAL, "device buffers must be 256-byte aligned");
    // the device's static staging array, looked up once per device with the device current
    int device = 0;
    void *noalloc = nullptr;
    HIP_OK(hipGetDevice(&device));
    HIP_OK(noalloc_scratch(device, &noalloc));
    lbm_ctx *c = new lbm_ctx();
    c->device = device;
    c->noalloc = noalloc;
    c->n = n;
    c->storage = storage;
    for (int i = 0; i < n; i++) {
        c->variants = c->variants || domains[i].wetting != 0;
        c->max_nodes = std::max(c->max_nodes, (size_t)domains[i].nx * domains[i].ny);
    }
    c->stream = (hipStream_t)hip_stream;
    c->state = (char *)state_dev;
    c->scratch = (char *)scratch_dev;
    c->L = L;
    c->desc.assign(domains, domains + n);
    c->doms.resize(n);
    c->tile = builtin_tile(c->desc, storage);
    c->items = build_items(c->desc, c->tile, storage);
    if (hipHostMalloc((void **)&c->mass_host, (2 * (size_t)n + 2) * sizeof(double)) != hipSuccess ||
        hipHostMalloc((void **)&c->flag_host, 64) != hipSuccess) {
        delete c;
        return fail(LBM_EDEVICE, "pinned host allocation failed");
    }
    if (storage == 0) rc = create_t<double, double>(c, domains);
    else if (storage == 1) rc = create_t<float, float>(c, domains);
    else if (storage == 2) rc = create_t<__half, float>(c, domains);
    else rc = create_t<C16, float>(c, domains);
    if (rc) {
        lbm_destroy(c);
        return rc;
    }
    *out = c;
    return LBM_OK;
}

int lbm_classify(const lbm_domain_desc *domain, uint8_t *classes_out, double *ns_out) {
    int rc = validate(domain, 1, 0);
    if (rc) return rc;
    const lbm_domain_desc &q = *domain;
    for (int y = 0; y < q.ny; y++)
        for (int x = 0; x < q.nx; x++) {
            double vx, vy;
            const uint32_t m = node_class(q, x, y, vx, vy);
            const size_t k = (size_t)y * q.nx + x;
            if (classes_out)
                classes_out[k] = (m & SELF_SOLID) ? ((m & SOLID_BND) ? 2 : 3) : ((m & FLUID_BND) ? 1 : 0);
            if (ns_out) {
                ns_out[2 * k] = vx;
                ns_out[2 * k + 1] = vy;
            }
        }
    return LBM_OK;
}

int lbm_step(lbm_ctx *c, int64_t n_steps) {
    if (!c) return fail(LBM_EINVAL, "null context");
    if (n_steps < 0) return fail(LBM_EINVAL, "negative step count");
    while (n_steps > 0) {
        // A replay needs the steady state of the arguments: a snapshot state (own) takes one
        // direct step first, and a remainder shorter than a graph is launched step by step.
        const int G = c->graph_steps;
        if (G > 0 && !c->own && n_steps >= G) {
            if (!c->gexec[c->parity]) {
                const int rc = build_graph(c, c->parity);
                if (rc) return rc;
            }
            HIP_OK(hipGraphLaunch(c->gexec[c->parity], c->stream));
            c->steps += G;
            n_steps -= G;
            continue;
        }
        HIP_OK(step_once(c, c->stream));
        n_steps--;
    }
    return LBM_OK;
}

int lbm_set_graph(lbm_ctx *c, int launches) {
    if (!c) return fail(LBM_EINVAL, "null context");
    if (launches != 0 && (launches < 2 || launches > 1024 || launches % 2))
        return fail(LBM_EINVAL, "launches per graph must be 0 or an even number in [2, 1024]");
    HIP_OK(hipStreamSynchronize(c->stream));
    drop_graphs(c);
    c->graph_steps = launches;
    // capture, instantiate and upload both graphs now, so that no replay pays for it
    for (int p = 0; p < 2 && launches > 0; p++) {
        const int rc = build_graph(c, p);
        if (rc) return rc;
    }
    HIP_OK(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

int lbm_autotune(lbm_ctx *c, int steps, void *save_dev, double *out_host) {
    if (!c || !save_dev) return fail(LBM_EINVAL, "null argument");
    if (steps < 1 || steps > 100000) return fail(LBM_EINVAL, "steps per trial must be in [1, 100000]");
    int rc = lbm_save_state(c, save_dev);
    if (rc) return rc;
    HIP_OK(hipMemcpyAsync(c->flag_host, c->scratch + c->L.flag, sizeof(int), hipMemcpyDeviceToHost,
                          c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    const int flag0 = *c->flag_host;
    struct Trial {
        TileShape tile;
        double ms;
    };
    std::vector<Trial> trials;
    // (waves, cols, node columns per lane); the pair-kernel shapes where the batch allows them
    const int shapes[5][3] = {{4, 1, 1}, {8, 1, 1}, {4, 2, 1}, {4, 1, 2}, {8, 1, 2}};
    const bool pairs = pair_allowed(c->storage, c->desc);
    for (const auto &sh : shapes) {
        if (sh[2] == 2 && !pairs) continue;
        std::vector<WorkItem> last[2];  // of the march and of the patch kernel
        for (int ch : {8, 12, 16, 24, 32, 48, 64}) {
            const TileShape t{ch, sh[0], sh[1], sh[2]};
            std::vector<WorkItem> it = build_items(c->desc, t, c->storage);
            // a taller chunk that cuts no domain differently is the same schedule of its kernel
            std::vector<WorkItem> &prev = last[t.patch(c->storage == 0)];
            if (it.size() == prev.size() &&
                std::equal(it.begin(), it.end(), prev.begin(), [](const WorkItem &a, const WorkItem &b) {
                    return a.dom == b.dom && a.x0 == b.x0 && a.y0 == b.y0 && a.y1 == b.y1;
                }))
                continue;
            trials.push_back({t, 0.0});
            prev.swap(it);
        }
    }
    hipEvent_t e0, e1;
    HIP_OK(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(LBM_EDEVICE, "hipEventCreate failed");
    }
    // one untimed step, then `steps` timed steps on the stream, per shape
    auto time_shape = [&](const Trial &t, double &ms) -> hipError_t {
        c->tile = t.tile;
        c->items = build_items(c->desc, t.tile, c->storage);
        if (upload_items(c)) return hipErrorInvalidValue;
        hipError_t e = step_once(c, c->stream);
        if (e == hipSuccess) e = hipEventRecord(e0, c->stream);
        for (int k = 0; k < steps && e == hipSuccess; k++) e = step_once(c, c->stream);
        if (e == hipSuccess) e = hipEventRecord(e1, c->stream);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float f = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&f, e0, e1);
        ms = f / steps;
        return e;
    };
    hipError_t e = hipSuccess;
    for (auto &t : trials)
        if (e == hipSuccess) e = time_shape(t, t.ms);
    // the three fastest again, ranked by the sum of both timings
    std::sort(trials.begin(), trials.end(), [](const Trial &a, const Trial &b) { return a.ms < b.ms; });
    const size_t top = std::min<size_t>(3, trials.size());
    for (size_t i = 0; i < top && e == hipSuccess; i++) {
        double ms = 0.0;
        e = time_shape(trials[i], ms);
        trials[i].ms += ms;
    }
    std::sort(trials.begin(), trials.begin() + top, [](const Trial &a, const Trial &b) { return a.ms < b.ms; });
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return fail(LBM_EDEVICE, "autotune: %s", hipGetErrorString(e));
    const Trial best = trials[0];
    c->tile = best.tile;
    c->items = build_items(c->desc, best.tile, c->storage);
    rc = upload_items(c);
    if (rc) return rc;
    drop_graphs(c);
    rc = lbm_load_state(c, save_dev);
    if (rc) return rc;
    *c->flag_host = flag0;
    HIP_OK(hipMemcpyAsync(c->scratch + c->L.flag, c->flag_host, sizeof(int), hipMemcpyHostToDevice,
                          c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    if (out_host) {
        out_host[0] = best.tile.chunk;
        out_host[1] = best.tile.waves;
        out_host[2] = best.tile.cols;
        out_host[3] = best.ms / 2.0;  // mean of the two timings
        out_host[4] = best.tile.npl;
    }
    return LBM_OK;
}

int lbm_read_fields(lbm_ctx *c, int domain, uint32_t which, double *out_dev, size_t out_count) {
    if (!c) return fail(LBM_EINVAL, "null context");
    if (domain < 0 || domain >= c->n) return fail(LBM_EINVAL, "domain %d out of range", domain);
    if (which == 0 || (which & ~31u)) return fail(LBM_EINVAL, "bad field selection %u", which);
    if (!out_dev) return fail(LBM_EINVAL, "output is NULL");
    if ((which & 24u) && !c->diag)
        return fail(LBM_ESTATE, "velocity fields need a diagnostics buffer (lbm_diag_attach)");
    const lbm_domain_desc &q = c->desc[domain];
    const size_t nn = (size_t)q.nx * q.ny;
    const size_t planes = ((which & 1u) ? 1 : 0) + ((which & 2u) ? 1 : 0) + ((which & 4u) ? 18 : 0) +
                          ((which & 8u) ? 1 : 0) + ((which & 16u) ? 1 : 0);
    if (out_count < planes * nn)
        return fail(LBM_ENOMEM, "output holds %zu doubles, need %zu", out_count, planes * nn);
    AnyArgs a = make_args(c, c->parity);
    size_t p = 0;
    if (which & 7u) {
        HIP_OK(launch_read(c->storage, a.bytes, domain, q.nx, q.ny, which & 7u, out_dev, c->stream));
        p = planes - ((which & 8u) ? 1 : 0) - ((which & 16u) ? 1 : 0);
    }
    if (which & 24u) {
        AnyArgs da = make_diag_args(c);
        HIP_OK(launch_step(c->storage, da.bytes, (int)c->items.size(), c->tile, c->variants, c->stream));
        double *ox = (which & 8u) ? out_dev + (p++) * nn : nullptr;
        double *oy = (which & 16u) ? out_dev + p * nn : nullptr;
        HIP_OK(launch_velocity_copy(c->storage, a.bytes, domain, c->diag + diag_layout(c).u, ox, oy,
                                    c->stream));
    }
    return LBM_OK;
}

int lbm_mass(lbm_ctx *c, double *out_host) {
    if (!c || !out_host) return fail(LBM_EINVAL, "null argument");
    AnyArgs a = make_args(c, c->parity);
    double *partials = reinterpret_cast<double *>(c->scratch + c->L.partials);
    // no more blocks per domain than the largest one fills
    const int bpd = (int)std::min<size_t>(c->L.bpd, (c->max_nodes + 255) / 256);
    HIP_OK(launch_mass(c->storage, a.bytes, c->n, partials, bpd, c->mass_host, c->flag_host, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    std::memcpy(out_host, c->mass_host, 2 * (size_t)c->n * sizeof(double));
    if (*c->flag_host) return fail(LBM_ENONFINITE, "a non-finite density or velocity appeared");
    return LBM_OK;
}

int64_t lbm_steps_taken(const lbm_ctx *c) { return c ? c->steps : -1; }

int lbm_set_tile(lbm_ctx *c, int chunk_rows, int waves, int cols, int cols_per_lane) {
    if (!c) return fail(LBM_EINVAL, "null context");
    if (chunk_rows != 0 && (chunk_rows < 8 || chunk_rows % 4))
        return fail(LBM_EINVAL, "chunk rows must be 0 or a multiple of 4 >= 8");
    if (waves != 0 && waves != 4 && waves != 8) return fail(LBM_EINVAL, "waves must be 0, 4 or 8");
    if (cols != 0 && cols != 1 && cols != 2) return fail(LBM_EINVAL, "cols must be 0, 1 or 2");
    if (cols_per_lane != 0 && cols_per_lane != 1 && cols_per_lane != 2)
        return fail(LBM_EINVAL, "cols_per_lane must be 0, 1 or 2");
    const int w = waves ? waves : DEFAULT_WAVES;
    const int npl = cols_per_lane ? cols_per_lane : 1;
    const int k = cols ? cols : DEFAULT_COLS;
    if (w == 8 && k == 2) return fail(LBM_EINVAL, "tiles of 8 x 2 wavefronts are not provided");
    if (npl == 2 && k != 1) return fail(LBM_EINVAL, "two columns per lane need one wavefront per tile row");
    if (npl == 2 && !pair_allowed(c->storage, c->desc))
        return fail(LBM_EINVAL, "two columns per lane need FP32 arithmetic and an even nx in every domain");
    HIP_OK(hipStreamSynchronize(c->stream));
    drop_graphs(c);
    TileShape t{chunk_rows, w, k, npl};
    if (!chunk_rows) {
        if (!waves && k == 1 && npl == 1) t = builtin_tile(c->desc, c->storage);
        else t.chunk = auto_chunk(c->desc, t, c->storage);
    }
    c->tile = t;
    c->items = build_items(c->desc, t, c->storage);
    return upload_items(c);
}

int lbm_get_tile(const lbm_ctx *c, int *shape_out) {
    if (!c || !shape_out) return fail(LBM_EINVAL, "null argument");
    shape_out[0] = c->tile.chunk;
    shape_out[1] = c->tile.waves;
    shape_out[2] = c->tile.cols;
    shape_out[3] = (int)c->items.size();
    shape_out[4] = c->tile.npl;
    return LBM_OK;
}

size_t lbm_state_size(const lbm_ctx *c) { return c ? c->L.state_bytes + 256 : 0; }

int lbm_save_state(lbm_ctx *c, void *dst_dev) {
    if (!c || !dst_dev) return fail(LBM_EINVAL, "null argument");
    HIP_OK(hipMemcpyAsync(dst_dev, c->state, c->L.state_bytes, hipMemcpyDeviceToDevice, c->stream));
    long long hdr[4] = {0x6c626d6367LL, c->parity, c->own, c->steps};
    HIP_OK(hipMemcpyAsync((char *)dst_dev + c->L.state_bytes, hdr, sizeof hdr,
                          hipMemcpyHostToDevice, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

int lbm_load_state(lbm_ctx *c, const void *src_dev) {
    if (!c || !src_dev) return fail(LBM_EINVAL, "null argument");
    long long hdr[4];
    HIP_OK(hipMemcpyAsync(hdr, (const char *)src_dev + c->L.state_bytes, sizeof hdr,
                          hipMemcpyDeviceToHost, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    if (hdr[0] != 0x6c626d6367LL || (hdr[1] & ~1LL) || (hdr[2] & ~1LL) || hdr[3] < 0)
        return fail(LBM_ESTATE, "not a saved state of this library");
    HIP_OK(hipMemcpyAsync(c->state, src_dev, c->L.state_bytes, hipMemcpyDeviceToDevice, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    c->parity = (int)hdr[1];
    c->own = (int)hdr[2];
    c->steps = hdr[3];
    return LBM_OK;
}

const char *lbm_last_error(void) { return g_err.c_str(); }

size_t lbm_diag_bytes(const lbm_ctx *c) { return c ? diag_layout(c).bytes : 0; }

int lbm_diag_attach(lbm_ctx *c, void *diag_dev, size_t bytes) {
    if (!c) return fail(LBM_EINVAL, "null context");
    HIP_OK(hipStreamSynchronize(c->stream));
    c->snap_valid = c->snap_first = false;
    if (!diag_dev) {
        c->diag = nullptr;
        return LBM_OK;
    }
    if (bytes < diag_layout(c).bytes)
        return fail(LBM_ENOMEM, "diagnostics buffer holds %zu bytes, need %zu", bytes, diag_layout(c).bytes);
    if ((uintptr_t)diag_dev & 255) return fail(LBM_EINVAL, "diagnostics buffer must be 256-byte aligned");
    if (!c->diag_host) {
        const size_t nd = std::max<size_t>(std::max<size_t>(2 * (size_t)c->n, 4), DIAG_MAX_ROWS);
        if (hipHostMalloc((void **)&c->diag_host, nd * sizeof(double)) != hipSuccess ||
            hipHostMalloc((void **)&c->rows_host, DIAG_MAX_ROWS * sizeof(int)) != hipSuccess)
            return fail(LBM_EDEVICE, "pinned host allocation failed");
    }
    c->diag = static_cast<char *>(diag_dev);
    return LBM_OK;
}

int lbm_diag_velocity(lbm_ctx *c, int snapshot, double *out_host) {
    if (!c || !out_host) return fail(LBM_EINVAL, "null argument");
    if (!c->diag) return fail(LBM_ESTATE, "no diagnostics buffer attached (lbm_diag_attach)");
    const DiagLayout DL = diag_layout(c);
    AnyArgs da = make_diag_args(c);
    HIP_OK(launch_step(c->storage, da.bytes, (int)c->items.size(), c->tile, c->variants, c->stream));
    HIP_OK(launch_velocity_stats(c->storage, da.bytes, c->n, c->diag + DL.u,
                                 c->snap_valid ? c->diag + DL.snap : nullptr,
                                 reinterpret_cast<double *>(c->diag + DL.part), c->diag_host, c->flag_host,
                                 c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    std::memcpy(out_host, c->diag_host, 2 * (size_t)c->n * sizeof(double));
    if (snapshot) {  // the buffer just written becomes the snapshot
        c->snap_valid = true;
        c->snap_first = !c->snap_first;
    }
    if (*c->flag_host) return fail(LBM_ENONFINITE, "a non-finite density or velocity appeared");
    return LBM_OK;
}

int lbm_diag_region_mass(lbm_ctx *c, int domain, const uint8_t *region_dev, double *out_host) {
    if (!c || !region_dev || !out_host) return fail(LBM_EINVAL, "null argument");
    if (domain < 0 || domain >= c->n) return fail(LBM_EINVAL, "domain %d out of range", domain);
    if (!c->diag) return fail(LBM_ESTATE, "no diagnostics buffer attached (lbm_diag_attach)");
    const DiagLayout DL = diag_layout(c);
    AnyArgs a = make_args(c, c->parity);
    HIP_OK(launch_region_mass(c->storage, a.bytes, domain, region_dev,
                              reinterpret_cast<double *>(c->diag + DL.part), c->diag_host, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    std::memcpy(out_host, c->diag_host, 4 * sizeof(double));
    return LBM_OK;
}

int lbm_diag_crossings(lbm_ctx *c, int domain, const int32_t *rows_host, int n_rows, double *out_host) {
    if (!c || !rows_host || !out_host) return fail(LBM_EINVAL, "null argument");
    if (domain < 0 || domain >= c->n) return fail(LBM_EINVAL, "domain %d out of range", domain);
    if (n_rows < 1 || n_rows > DIAG_MAX_ROWS) return fail(LBM_EINVAL, "row count %d outside [1, %d]", n_rows, DIAG_MAX_ROWS);
    if (!c->diag) return fail(LBM_ESTATE, "no diagnostics buffer attached (lbm_diag_attach)");
    for (int k = 0; k < n_rows; k++)
        if (rows_host[k] < 0 || rows_host[k] >= c->desc[domain].ny)
            return fail(LBM_EINVAL, "row %d outside the domain", rows_host[k]);
    std::memcpy(c->rows_host, rows_host, (size_t)n_rows * sizeof(int));
    AnyArgs a = make_args(c, c->parity);
    HIP_OK(launch_crossings(c->storage, a.bytes, domain, c->desc[domain].nx, c->rows_host, n_rows, c->diag_host,
                            c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    std::memcpy(out_host, c->diag_host, (size_t)n_rows * sizeof(double));
    return LBM_OK;
}

int lbm_diag_crossings_noalloc(lbm_ctx *c, int domain, const int32_t *rows_host, int n_rows,
                               double *out_host) {
    if (!c || !rows_host || !out_host) return fail(LBM_EINVAL, "null argument");
    if (domain < 0 || domain >= c->n) return fail(LBM_EINVAL, "domain %d out of range", domain);
    if (n_rows < 1 || n_rows > NOALLOC_ROWS)
        return fail(LBM_EINVAL, "row count %d outside [1, %d] (size of the static staging array)", n_rows,
                    NOALLOC_ROWS);
    for (int k = 0; k < n_rows; k++)
        if (rows_host[k] < 0 || rows_host[k] >= c->desc[domain].ny)
            return fail(LBM_EINVAL, "row %d outside the domain", rows_host[k]);
    if (!c->noalloc) return fail(LBM_ESTATE, "no static staging array for this context's device");
    // rows in, crossing kernel, results out, all on the context's stream; the caller's host
    // arrays are used directly (no pinned staging), and the stream is drained before returning
    HIP_OK(hipMemcpyAsync(c->noalloc, rows_host, (size_t)n_rows * sizeof(int32_t), hipMemcpyHostToDevice,
                          c->stream));
    AnyArgs a = make_args(c, c->parity);
    HIP_OK(launch_crossings_noalloc(c->storage, a.bytes, domain, c->desc[domain].nx, c->noalloc, n_rows, c->stream));
    HIP_OK(hipMemcpyAsync(out_host, static_cast<char *>(c->noalloc) + NOALLOC_OUT_OFFSET,
                          (size_t)n_rows * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

int lbm_diag_contact_line(lbm_ctx *c, int domain, int32_t *out_host, int cap, int *count) {
    if (!c || !count || (cap > 0 && !out_host)) return fail(LBM_EINVAL, "null argument");
    if (domain < 0 || domain >= c->n) return fail(LBM_EINVAL, "domain %d out of range", domain);
    if (cap < 0) return fail(LBM_EINVAL, "negative capacity");
    if (!c->diag) return fail(LBM_ESTATE, "no diagnostics buffer attached (lbm_diag_attach)");
    const DiagLayout DL = diag_layout(c);
    int *dcount = reinterpret_cast<int *>(c->diag + DL.cl_count);
    HIP_OK(hipMemsetAsync(dcount, 0, sizeof(int), c->stream));
    AnyArgs da = make_diag_args(c, domain);
    HIP_OK(launch_step(c->storage, da.bytes, (int)c->items.size(), c->tile, c->variants, c->stream));
    HIP_OK(hipMemcpyAsync(c->rows_host, dcount, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    const int n = c->rows_host[0];
    *count = n;
    if (n > c->max_fluid_bnd)  // each node is recorded once: cannot happen
        return fail(LBM_EDEVICE, "contact-line list overflow (%d entries)", n);
    if (n > cap) return fail(LBM_ENOMEM, "%d contact-line nodes, room for %d", n, cap);
    if (n > 0) {
        HIP_OK(hipMemcpy(out_host, c->diag + DL.cl_list, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost));
        std::sort(out_host, out_host + n);
    }
    return LBM_OK;
}

void lbm_destroy(lbm_ctx *c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    drop_graphs(c);
    if (c->cap) (void)hipStreamDestroy(c->cap);
    if (c->mass_host) (void)hipHostFree(c->mass_host);
    if (c->flag_host) (void)hipHostFree(c->flag_host);
    if (c->diag_host) (void)hipHostFree(c->diag_host);
    if (c->rows_host) (void)hipHostFree(c->rows_host);
    delete c;
}

}  // extern "C"
