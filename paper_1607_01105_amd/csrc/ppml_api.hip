// ppml_api.hip -- host implementation of the C ABI declared in include/ppml.h.
// Argument checking, launch geometry, and the enqueueing of the kernels of
// ppml_kernels.hip on the caller's stream.  No computation of the method
// happens on the host.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/ppml.h"
#include "ppml_gravity.hpp"
#include "ppml_sine.hpp"
#include "ppml_kernels.hpp"
#include "ppml_transfer.hpp"
#include "ppml_line.hpp"
#include "ppml_sheet.hpp"
#include "ppml_brick.hpp"

using namespace ppml;

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define HIPCHK(expr)                                                                                   \
    do {                                                                                               \
        hipError_t e_ = (expr);                                                                        \
        if (e_ != hipSuccess) return fail(PPML_EHIP, "%s: %s", #expr, hipGetErrorString(e_));          \
    } while (0)

// Work-group tile shapes (x extent, y extent) per dimensionality; index 0 is
// the default.  Every shape runs the same per-cell arithmetic, so results do
// not depend on the choice; the autotuner picks one per workload.
template <int X, int Y> struct Tile {
    static constexpr int tx = X, ty = Y, nt = X * Y;
};
constexpr int NTILE[4] = {0, 3, 4, 4};
constexpr int TILE_X[4][4] = {{0, 0, 0, 0}, {256, 128, 64, 0}, {32, 64, 16, 32}, {32, 64, 16, 32}};
constexpr int TILE_Y[4][4] = {{0, 0, 0, 0}, {1, 1, 1, 0}, {8, 4, 16, 4}, {8, 4, 16, 4}};

// Tile shape of the 3-D launches for the grids added: FP64 launches take 16x16
// for the default, whose Eulerian kernel fits a CU's LDS three times where 32x8
// fits twice, unless it takes more than TILE_FP64 times the cells to cover the
// grids.  us per step at 32x8 / 16x16 (cells of 16x16 over those of 32x8):
// 512x512x64 2648 / 2434 (1.00), 131x97x75 230 / 199 (0.97), 150^3 595 / 569
// (1.05), 100x40x200 182 / 188 (1.05), 224x88x100 341 / 320 (1.09), 200x40x120
// 204 / 206 and 200x40x40 87 / 102 (1.11), 512x72x64 432 / 409 (1.11), 160x56x100
// 177 / 182 (1.14), 512x40x64 238 / 251 (1.20), 400x23x100 181 / 203 (1.28).
constexpr double TILE_FP64 = 1.1;
struct TileRule {
    double cells[2] = {0.0, 0.0};  // of the tiles of 32x8, 16x16
    void add(const GridParams &gp)
    {
        cells[0] += (double)((gp.n[0] + 31) / 32 * 32) * ((gp.n[1] + 7) / 8 * 8) * gp.n[2];
        cells[1] += (double)((gp.n[0] + 15) / 16 * 16) * ((gp.n[1] + 15) / 16 * 16) * gp.n[2];
    }
    int tile(int prec, int v) const
    {
        return prec == PPML_FP64 && v == 0 && cells[1] <= TILE_FP64 * cells[0] ? 2 : v;
    }
};

// Calls f(Tile<tx, ty>{}) for launch tile v of dimensionality NDIM (the tables
// above, spelled out as template arguments).
template <int NDIM, typename F> void with_tile(int v, F &&f)
{
    if constexpr (NDIM == 1) {
        switch (v) {
        case 1: f(Tile<128, 1>{}); break;
        case 2: f(Tile<64, 1>{}); break;
        default: f(Tile<256, 1>{}); break;
        }
    } else {
        switch (v) {
        case 1: f(Tile<64, 4>{}); break;
        case 2: f(Tile<16, 16>{}); break;
        case 3: f(Tile<32, 4>{}); break;
        default: f(Tile<32, 8>{}); break;
        }
    }
}

// Rows per wave the 2-D kernels are compiled for; FP64 spills past two.
constexpr int SHEET_ROWS[] = {1, 2, 3, 4, 8};
template <typename T, typename F> void with_rows(int r, F &&f)
{
    if constexpr (sizeof(T) == 4) {
        switch (r) {
        case 8: return f(std::integral_constant<int, 8>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 3: return f(std::integral_constant<int, 3>{});
        }
    }
    if (r == 2) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 1>{});
}

// Fields per LDS pass of the Lagrangian kernel (all six in FP32; FP64 in
// two passes to keep two work groups per CU).
template <typename T> struct LG {
    static constexpr int g = sizeof(T) == 4 ? 6 : 3;
};

int nfields(const ppml_desc *d) { return 3 + d->ndim; }

size_t elem(const ppml_desc *d) { return d->prec == PPML_FP64 ? sizeof(double) : sizeof(float); }

long long ncells(const ppml_desc *d)
{
    return (long long)d->n[0] * (long long)d->n[1] * (long long)d->n[2];
}

int validate(const ppml_desc *d)
{
    if (!d) return fail(PPML_EINVAL, "descriptor is NULL");
    if (d->ndim < 1 || d->ndim > 3) return fail(PPML_EINVAL, "ndim must be 1, 2 or 3 (got %d)", d->ndim);
    if (d->prec != PPML_FP32 && d->prec != PPML_FP64) return fail(PPML_EINVAL, "prec must be PPML_FP32 or PPML_FP64");
    for (int a = 0; a < 3; a++) {
        if (a < d->ndim) {
            if (d->n[a] < 1 || d->n[a] > (1 << 20)) return fail(PPML_EINVAL, "n[%d] out of range", a);
            if (!(d->hi[a] > d->lo[a])) return fail(PPML_EINVAL, "hi[%d] must exceed lo[%d]", a, a);
            for (int s = 0; s < 2; s++) {
                int b = s ? d->bc_hi[a] : d->bc_lo[a];
                if (b != PPML_PERIODIC && b != PPML_OUTFLOW && b != PPML_REFLECT && b != PPML_INFLOW)
                    return fail(PPML_EINVAL, "bad boundary code on axis %d", a);
                if (b == PPML_REFLECT && d->n[a] < 3) return fail(PPML_EINVAL, "reflecting axis %d needs n >= 3", a);
                if (b == PPML_INFLOW) {
                    const double *st = d->inflow[2 * a + s];
                    for (int q = 0; q < 5; q++)
                        if (!std::isfinite(st[q])) return fail(PPML_EINVAL, "inflow state of face %d is not finite", 2 * a + s);
                    if (!(st[0] > 0.0) || !(st[4] > 0.0))
                        return fail(PPML_EINVAL, "inflow face %d needs rho > 0 and p > 0", 2 * a + s);
                }
            }
            if ((d->bc_lo[a] == PPML_PERIODIC) != (d->bc_hi[a] == PPML_PERIODIC))
                return fail(PPML_EINVAL, "axis %d: periodic must be set on both faces", a);
        } else if (d->n[a] != 1) {
            return fail(PPML_EINVAL, "n[%d] must be 1 for an unused axis", a);
        }
    }
    if (ncells(d) > (1ll << 31) - 1) return fail(PPML_EINVAL, "grid too large (%lld cells)", ncells(d));
    if (!(d->gamma > 1.0) || !std::isfinite(d->gamma)) return fail(PPML_EINVAL, "gamma must be > 1");
    if (!(d->cfl > 0.0 && d->cfl < 1.0)) return fail(PPML_EINVAL, "cfl must lie in (0, 1)");
    if (!(d->vacuum_ratio >= 0.0)) return fail(PPML_EINVAL, "vacuum_ratio must be >= 0");
    if (d->potential != PPML_POT_NONE && d->potential != PPML_POT_LOG && d->potential != PPML_POT_UNIFORM &&
        d->potential != PPML_POT_HALO)
        return fail(PPML_EINVAL, "bad potential code");
    if (d->potential == PPML_POT_LOG && !(d->pot[2] > 0.0)) return fail(PPML_EINVAL, "log potential needs q > 0");
    if (d->potential == PPML_POT_HALO && !(d->pot[1] > 0.0 && d->pot[2] > 0.0))
        return fail(PPML_EINVAL, "halo potential needs r0 > 0 and rh > 0");
    if (d->potential == PPML_POT_HALO && d->ndim != 3) return fail(PPML_EINVAL, "the halo potential needs ndim = 3");
    if (d->flags & ~(PPML_FLAG_FIRST_ORDER | PPML_FLAG_ISOTHERMAL)) return fail(PPML_EINVAL, "unknown flags 0x%x", d->flags);
    if ((d->flags & PPML_FLAG_ISOTHERMAL) && !(d->iso_cs > 0.0 && std::isfinite(d->iso_cs)))
        return fail(PPML_EINVAL, "the isothermal variant needs iso_cs > 0");
    if (d->tile < 0 || d->tile >= NTILE[d->ndim])
        return fail(PPML_EINVAL, "tile %d out of range [0, %d) for ndim %d", d->tile, NTILE[d->ndim], d->ndim);
    if (d->self_gravity != 0 && d->self_gravity != 1) return fail(PPML_EINVAL, "self_gravity must be 0 or 1");
    if (d->self_gravity) {
        if (d->ndim != 3) return fail(PPML_EINVAL, "self-gravity needs ndim = 3");
        const double h0 = (d->hi[0] - d->lo[0]) / (double)d->n[0];
        for (int a = 1; a < 3; a++) {
            const double ha = (d->hi[a] - d->lo[a]) / (double)d->n[a];
            if (std::fabs(ha - h0) > 1e-12 * h0) return fail(PPML_EINVAL, "self-gravity needs cubic cells");
        }
        if (!(d->grav_G > 0.0) || !std::isfinite(d->grav_G)) return fail(PPML_EINVAL, "grav_G must be > 0");
        // the multipole expansion about the origin is undefined at the origin
        int on_grid = 1, on_shell = 0;
        for (int a = 0; a < 3; a++) {
            const double u = (0.0 - d->lo[a]) / h0 - 0.5;  // origin in cell units
            const double ur = std::nearbyint(u);
            if (std::fabs(u - ur) > 1e-9 || ur < -1.0 || ur > (double)d->n[a]) on_grid = 0;
            if (ur == -1.0 || ur == (double)d->n[a]) on_shell = 1;
        }
        if (on_grid && on_shell) return fail(PPML_EINVAL, "the origin (the multipole centre) is a shell cell centre");
    }
    return PPML_OK;
}

constexpr size_t ALIGN = 256;
size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

// Totals reduction: fixed number of blocks so the summation order is fixed.
int totals_blocks(long long n) { return (int)std::min<long long>(1024, (n + 4095) / 4096 > 0 ? (n + 4095) / 4096 : 1); }

// Bytes behind the control block for the maxima slots (two sets), and how many
// slots a set has there: about one per 43 work groups of 256 cells, at most
// one per lane of the wave that folds them.
size_t maxima_bytes(long long n) { return align_up((size_t)totals_blocks(n) * 6 * sizeof(double)); }
int maxima_slots(long long n)
{
    return (int)std::min<size_t>(MSLOT_MAX, maxima_bytes(n) / (2 * MSLOT_BYTES));
}

struct ScratchLayout {
    size_t half, ctrl, maxima, totals;
    // self-gravity: padded potential, two work arrays, sine matrices,
    // eigenvalue factors, moment partials, shell terms of the outer layer
    size_t phi, wx, wy, sx, sy, sz, fx, fy, fz, gpart, gedge;
    size_t total;
};

// Moment reduction of the self-gravity solve: fixed block count (fixed order).
int grav_blocks(long long n) { return (int)std::min<long long>(1024, (n + 2047) / 2048 > 0 ? (n + 2047) / 2048 : 1); }

// The kernels of ppml_sine.hpp hold a line's two halves in registers, in the
// z pass its results too: up to SINE_TILES blocks of 16 a half, axes of 256
// cells.  A grid with a longer axis takes library products.  The solve,
// library against kernels, in us: FP64 160^3 338 and 182, 192^3 474 and 365,
// 240^3 734 and 667, 256^3 719 and 700; FP32 160^3 215 and 129, 224^3 435 and
// 293, 256^3 420 and 398; with kernels built for longer lines FP32 272^3 822
// and 975, 512x64x512 509 and 566.
constexpr int SINE_TILES = 8;

bool sine_kernels(const ppml_desc *d)
{
    for (int a = 0; a < 3; a++)
        if (grav_no(d->n[a]) > 16 * SINE_TILES) return false;
    return true;
}

// Whether they run in FP64: for FP64 states, and for FP32 states of a grid with
// an axis of at most SINE_SHORT cells.  In FP32 every pass rounds its sums of
// mirror cells, where the library path forms and rounds them once for all axes;
// on long axes the shorter sums of the products outweigh that, on short ones
// they do not.  Error of the FP32 potential against 64 bits over the library
// path's, max norm / rms, FP32 transforms: 6^3 1.40 / 1.22, 16^3 1.21 / 1.06, 32^3
// 1.21 / 1.13, 48x48x200 1.30 / 1.19, 48^3 1.02 / 0.96, 70^3 0.94 / 0.95, 100^3
// 0.97 / 0.96, 104^3 1.00 / 0.95, 128^3 0.78 / 0.80, 256^3 0.85 / 0.84; FP64
// transforms: 6^3 0.35 / 0.26, 32^3 0.12 / 0.15, 64^3 0.08 / 0.10.  The solve in us,
// library / FP32 / FP64 transforms: 24^3 88 / 45 / 46, 64^3 97 / 47 / 53, 48x200x48
// 109 / 77 / 105, 64x256x256 209 / 143 / 187, 24x256x256 169 / 133 / 167.
constexpr int SINE_SHORT = 64;

bool sine_fp64(const ppml_desc *d)
{
    return d->prec == PPML_FP64 || d->n[0] <= SINE_SHORT || d->n[1] <= SINE_SHORT || d->n[2] <= SINE_SHORT;
}

size_t sine_elem(const ppml_desc *d) { return sine_kernels(d) && sine_fp64(d) ? sizeof(double) : elem(d); }

size_t sine_table_bytes(const ppml_desc *d, int axis)
{
    const int n = d->n[axis];
    if (!sine_kernels(d)) return (size_t)n * n * elem(d);
    return sine_fp64(d) ? sine_table_count<double>(n) * sizeof(double) : sine_table_count<float>(n) * sizeof(float);
}

ScratchLayout layout(const ppml_desc *d)
{
    ScratchLayout L;
    L.half = 0;
    size_t sz = align_up((size_t)nfields(d) * (size_t)ncells(d) * elem(d));
    L.ctrl = sz;
    sz += CTRL_BYTES;
    L.maxima = sz;
    sz += maxima_bytes(ncells(d));
    L.totals = sz;
    sz += align_up(8 * sizeof(double));
    L.phi = L.wx = L.wy = L.sx = L.sy = L.sz = L.fx = L.fy = L.fz = L.gpart = L.gedge = 0;
    if (d->self_gravity) {
        const size_t e = elem(d);
        const size_t n0 = (size_t)d->n[0], n1 = (size_t)d->n[1], n2 = (size_t)d->n[2];
        L.phi = sz;
        sz += align_up((n0 + 2) * (n1 + 2) * (n2 + 2) * e);
        L.wx = sz;
        sz += align_up(n0 * n1 * n2 * sine_elem(d));
        L.wy = sz;
        if (!sine_kernels(d)) sz += align_up(n0 * n1 * n2 * e);  // the passes of ppml_sine.hpp run in place
        L.sx = sz;
        sz += align_up(sine_table_bytes(d, 0));
        L.sy = sz;
        sz += align_up(sine_table_bytes(d, 1));
        L.sz = sz;
        sz += align_up(sine_table_bytes(d, 2));
        L.fx = sz;
        sz += align_up(n0 * sizeof(double));
        L.fy = sz;
        sz += align_up(n1 * sizeof(double));
        L.fz = sz;
        sz += align_up(n2 * sizeof(double));
        L.gpart = sz;
        sz += align_up((size_t)grav_blocks(ncells(d)) * GRAV_MOM * sizeof(double));
        L.gedge = sz;
        sz += align_up((size_t)grav_edge_cells(d->n[0], d->n[1], d->n[2]) * sine_elem(d));
    }
    L.total = sz;
    return L;
}

}  // namespace

struct ppml_grid {
    ppml_desc d;
    GridParams gp;         // batch launches and the per-cell kernels
    GridParams gpE, gpL;   // solo launches of the two stage kernels (own z chunks)
    GridParams gpB;        // solo launches of the row kernels of small 3-D grids
    bool brick;            // the grid takes those
    int ltile;             // tile shape of the solo launches
    hipStream_t stream;
    int device;
    void *state;
    void *half;
    Ctrl *ctrl;
    double *totals;
    bool in_batch;         // admitted to a batch: stepped only by the batch
    hipStream_t bstream;   // that batch's stream (the batch kernels write the state there)
    bool has_state;
    std::vector<hipEvent_t> ev;  // 4 events per timed step
    long long timed;             // steps recorded since the last read
    // self-gravity (Sec. 2.5)
    rocblas_handle blas;
    void *phi, *wx, *wy, *sx, *sy, *sz, *gedge;
    double *fx, *fy, *fz, *gpart;
    double grav_coef;      // 4 pi G h^2
    double grav_norm;      // prod_a 2 / (n_a + 1)
    // a captured chunk of STEP_GRAPH steps, replayed by long ppml_step calls
    hipGraphExec_t sexec;
    bool graph_off;        // capture failed once: launch eagerly
};

namespace {

// Work groups of a stage launch for one grid: one per tile, in 2-D one per four
// strips (a wave each).
int work_groups(const GridParams &gp)
{
    constexpr int per = SHEET_THREADS / 64;
    const int t = gp.tiles[0] * gp.tiles[1] * gp.tiles[2];
    return gp.ndim == 2 ? (t + per - 1) / per : t;
}

// ... of a launch of the row kernels: one per four rows' strips.
int brick_groups(const GridParams &gp)
{
    constexpr int per = SHEET_THREADS / 64;
    return (int)(((long long)gp.tiles[0] * gp.n[1] * gp.n[2] + per - 1) / per);
}

template <typename T> void launch_speeds(ppml_grid *g)
{
    const T *U = (const T *)g->state;
    const int nb = (int)std::min<long long>(2048, (g->gp.ncell + SPEED_THREADS - 1) / SPEED_THREADS);
    switch (g->d.ndim) {
    case 1: k_speeds<T, 1><<<nb, SPEED_THREADS, 0, g->stream>>>(U, g->gp, g->ctrl); break;
    case 2: k_speeds<T, 2><<<nb, SPEED_THREADS, 0, g->stream>>>(U, g->gp, g->ctrl); break;
    default: k_speeds<T, 3><<<nb, SPEED_THREADS, 0, g->stream>>>(U, g->gp, g->ctrl); break;
    }
}

template <typename T, int NDIM> void launch_stages(ppml_grid *g, hipEvent_t *ev)
{
    const T *U = (const T *)g->state;
    T *Us = (T *)g->state;
    T *W = (T *)g->half;
    if constexpr (NDIM == 2) {
        if (ev) (void)hipEventRecord(ev[1], g->stream);
        with_rows<T>(g->gp.cz, [&](auto rows) {
            constexpr int R = decltype(rows)::value;
            k_euler_sheet<T, R><<<work_groups(g->gp), SHEET_THREADS, 0, g->stream>>>(U, W, g->gp, g->ctrl);
            if (ev) (void)hipEventRecord(ev[2], g->stream);
            k_lagr_sheet<T, R><<<work_groups(g->gp), SHEET_THREADS, 0, g->stream>>>(W, Us, g->gp, g->ctrl);
        });
        if (ev) (void)hipEventRecord(ev[3], g->stream);
    } else if (NDIM == 3 && g->brick) {
        const GridParams &gp = g->gpB;
        const int nb = brick_groups(gp);
        if (ev) (void)hipEventRecord(ev[1], g->stream);
        if (gp.potential == POT_HALO) k_euler_brick<T, 2><<<nb, SHEET_THREADS, 0, g->stream>>>(U, W, gp, g->ctrl);
        else if (gp.self_grav) k_euler_brick<T, 1><<<nb, SHEET_THREADS, 0, g->stream>>>(U, W, gp, g->ctrl);
        else k_euler_brick<T, 0><<<nb, SHEET_THREADS, 0, g->stream>>>(U, W, gp, g->ctrl);
        if (ev) (void)hipEventRecord(ev[2], g->stream);
        k_lagr_brick<T><<<nb, SHEET_THREADS, 0, g->stream>>>(W, Us, gp, g->ctrl);
        if (ev) (void)hipEventRecord(ev[3], g->stream);
    } else {
        with_tile<NDIM>(g->ltile, [&](auto tl) {
            using TL = decltype(tl);
            const GridParams &ge = g->gpE;
            const GridParams &gl = g->gpL;
            const int nbe = work_groups(ge);
            const int nbl = work_groups(gl);
            if (ev) (void)hipEventRecord(ev[1], g->stream);
            if constexpr (NDIM == 3) {
                if (ge.potential == POT_HALO)
                    k_euler<T, 3, TL::tx, TL::ty, 2><<<nbe, TL::nt, 0, g->stream>>>(U, W, ge, g->ctrl);
                else if (ge.self_grav)
                    k_euler<T, 3, TL::tx, TL::ty, 1><<<nbe, TL::nt, 0, g->stream>>>(U, W, ge, g->ctrl);
                else
                    k_euler<T, 3, TL::tx, TL::ty><<<nbe, TL::nt, 0, g->stream>>>(U, W, ge, g->ctrl);
            } else {
                k_euler<T, NDIM, TL::tx, TL::ty><<<nbe, TL::nt, 0, g->stream>>>(U, W, ge, g->ctrl);
            }
            if (ev) (void)hipEventRecord(ev[2], g->stream);
            k_lagr<T, NDIM, TL::tx, TL::ty, LG<T>::g><<<nbl, TL::nt, 0, g->stream>>>(W, Us, gl, g->ctrl);
            if (ev) (void)hipEventRecord(ev[3], g->stream);
        });
    }
}

// 1-D grids whose steps run in one kernel on one CU (ppml_line.hpp).  Its time
// follows the cells, that of the two stage launches is their dispatch; us per
// step, line kernel against stage kernels: FP64 64 cells 1.9 / 10.0, 512 3.7 /
// 11.7, 1024 5.4 / 12.2, 2048 9.8 / 12.4, 2500 12.4 / 12.5; FP32 64 1.4 / 8.1,
// 512 2.3 / 9.4, 2048 5.8 / 10.3, 3500 9.5 / 10.6, 4096 11.3 / 10.7.
template <typename T> constexpr long long line_cells() { return sizeof(T) == 8 ? 2304 : 3840; }
// A call's steps share one filling and emptying of the LDS, so calls of one to
// three steps take the kernel for shorter grids only: us per step, FP64 calls of
// 1 step 1800 cells 14.1 / 14.8, 2150 16.0 / 14.8, of 2 2150 13.2 / 13.8, 2304 14.6 /
// 14.1; FP32 of 1 2700 12.6 / 13.1, 3000 13.5 / 12.8, of 2 3300 11.7 / 12.2, 3600
// 12.7 / 12.2, of 3 3600 11.7 / 11.9, 3840 12.0 / 11.7.
template <typename T> constexpr long long line_cells(long long nsteps)
{
    if (nsteps == 1) return sizeof(T) == 8 ? 1856 : 2752;
    if (nsteps == 2) return sizeof(T) == 8 ? 2176 : 3392;
    if (nsteps == 3) return sizeof(T) == 8 ? 2304 : 3712;
    return line_cells<T>();
}

// (nsteps: of the call; 0: of calls of any length)
bool line_grid(const ppml_desc *d, long long nsteps = 0)
{
    return d->ndim == 1 && d->n[0] <= (d->prec == PPML_FP64 ? line_cells<double>(nsteps) : line_cells<float>(nsteps));
}

// Beside the launches of 2-D or 3-D grids the line kernel also takes longer
// 1-D grids, in memory instead of LDS: a second chain of launches slows the
// first (24 1-D and 24 2-D grids FP32, one of 3.9 k cells: 37 us per step with
// both chains, 28 with one).  Past a few thousand cells its time per step would
// pass that of a 2-D chain.
constexpr long long LINE_BATCH_CELLS = 4608;

// Threads of a line kernel's work groups for grids of up to n cells: a wave
// per segment up to LINE_THREADS.
int line_threads(long long n)
{
    return (int)std::min<long long>(LINE_THREADS, 64 * ((n + LINE_W - 1) / LINE_W));
}

// nsteps steps of a short 1-D grid; start: the run's parameters are these,
// otherwise those of the control block.
template <typename T> int launch_line(ppml_grid *g, long long nsteps, double dt_fixed, double t_stop, bool start)
{
    const long long n = g->gp.n[0];
    const size_t lds = line_lds<T>(n);
    if (lds > 65536)
        HIPCHK(hipFuncSetAttribute((const void *)k_line<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    for (long long s = 0; s < nsteps; s += LINE_STEPS) {
        const int m = (int)std::min<long long>(LINE_STEPS, nsteps - s);
        k_line<T><<<1, line_threads(n), lds, g->stream>>>((T *)g->state, g->gp, g->ctrl, start && s == 0 ? nsteps : -1,
                                                          dt_fixed, t_stop, m);
    }
    HIPCHK(hipGetLastError());
    return PPML_OK;
}

// GEMMs of the sine transforms (column-major view of the C-order arrays:
// a matrix with leading dimension n0 has the x index as its row).
rocblas_status gemm(rocblas_handle h, rocblas_operation ta, rocblas_operation tb, int m, int n, int k, const float *A,
                    int lda, long long sa, const float *B, int ldb, long long sb, float *C, int ldc, long long sc,
                    int batch)
{
    const float one = 1.0f, zero = 0.0f;
    if (batch == 1) return rocblas_sgemm(h, ta, tb, m, n, k, &one, A, lda, B, ldb, &zero, C, ldc);
    return rocblas_sgemm_strided_batched(h, ta, tb, m, n, k, &one, A, lda, sa, B, ldb, sb, &zero, C, ldc, sc, batch);
}

rocblas_status gemm(rocblas_handle h, rocblas_operation ta, rocblas_operation tb, int m, int n, int k,
                    const double *A, int lda, long long sa, const double *B, int ldb, long long sb, double *C, int ldc,
                    long long sc, int batch)
{
    const double one = 1.0, zero = 0.0;
    if (batch == 1) return rocblas_dgemm(h, ta, tb, m, n, k, &one, A, lda, B, ldb, &zero, C, ldc);
    return rocblas_dgemm_strided_batched(h, ta, tb, m, n, k, &one, A, lda, sa, B, ldb, sb, &zero, C, ldc, sc, batch);
}

// Sine transform of every line of one axis, on data in (sum | difference)
// slots along that axis: the odd modes are So times the sums, the even
// modes Se times the differences (forward); back, the sums are So^T times
// the odd modes and the differences Se^T times the even modes.  Column-major
// views of the C-order arrays: x as rows (C = op(S) A over the n1 n2
// columns), y per plane (C_k = A_k op(S)^T, a strided batch over the n2
// planes), z as columns (C = A op(S)^T over the n0 n1 rows).
template <typename T> int sine_transform(ppml_grid *g, int axis, bool inverse, const T *A, T *C)
{
    const int n[3] = {g->gp.n[0], g->gp.n[1], g->gp.n[2]};
    const int na = n[axis];
    const int no = grav_no(na), ne = grav_ne(na);
    const T *S = (const T *)(axis == 0 ? g->sx : axis == 1 ? g->sy : g->sz);
    const rocblas_operation N_ = rocblas_operation_none, T_ = rocblas_operation_transpose;
    const long long plane = (long long)n[0] * n[1];
    for (int half = 0; half < 2; half++) {
        const int m = half ? ne : no;             // slots of this half
        if (m == 0) continue;
        const T *Sh = S + (half ? (long long)no * no : 0);  // m x m, column major
        const long long off = half ? no : 0;      // first slot of the half
        rocblas_status st;
        if (axis == 0)
            st = gemm(g->blas, inverse ? T_ : N_, N_, m, n[1] * n[2], m, Sh, m, 0, A + off, n[0], 0, C + off, n[0], 0,
                      1);
        else if (axis == 1)
            st = gemm(g->blas, N_, inverse ? N_ : T_, n[0], m, m, A + off * n[0], n[0], plane, Sh, m, 0,
                      C + off * n[0], n[0], plane, n[2]);
        else
            st = gemm(g->blas, N_, inverse ? N_ : T_, (int)plane, m, m, A + off * plane, (int)plane, 0, Sh, m, 0,
                      C + off * plane, (int)plane, 0, 1);
        if (st != rocblas_status_success)
            return fail(PPML_EHIP, "rocBLAS GEMM of the sine transform: status %d", (int)st);
    }
    return PPML_OK;
}

constexpr int SINE_BLOCKS = 256;  // a block per CU

template <typename T, int MT, int KIND, typename ST>
int sine_launch(ppml_grid *g, const SineIn<T, KIND, ST> *src, SineOut<T, KIND, ST> *dst, const T *S, int nlines)
{
    using Shape = SineShape<T, MT, KIND>;
    constexpr int lds = Shape::CT * Shape::TILE;
    if (lds > 64 * 1024)
        HIPCHK(hipFuncSetAttribute((const void *)k_sine<T, MT, KIND, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    const int tiles = (nlines + 15) / 16;
    const int waves = std::max(1, std::min(Shape::WAVES, (tiles + SINE_BLOCKS - 1) / SINE_BLOCKS));
    const int blocks = std::min(SINE_BLOCKS, (tiles + waves - 1) / waves);
    const SineArgs args = {g->grav_coef, g->grav_norm};
    k_sine<T, MT, KIND, ST><<<blocks, 64 * waves, lds, g->stream>>>(src, dst, S, (const T *)g->gedge, g->fx, g->fy,
                                                                    g->fz, g->gp, args);
    return PPML_OK;
}

template <typename T, int KIND, typename ST>
int sine_pass(ppml_grid *g, const SineIn<T, KIND, ST> *src, SineOut<T, KIND, ST> *dst)
{
    constexpr int axis = KIND == SINE_Z ? 2 : KIND == SINE_Y_FWD || KIND == SINE_Y_INV ? 1 : 0;
    const int *n = g->gp.n;
    const T *S = (const T *)(axis == 0 ? g->sx : axis == 1 ? g->sy : g->sz);
    const int nl = axis == 0 ? n[1] * n[2] : axis == 1 ? n[0] * n[2] : n[0] * n[1];
    switch (sine_tiles(n[axis])) {
    case 1: return sine_launch<T, 1, KIND, ST>(g, src, dst, S, nl);
    case 2: return sine_launch<T, 2, KIND, ST>(g, src, dst, S, nl);
    case 3: return sine_launch<T, 3, KIND, ST>(g, src, dst, S, nl);
    case 4: return sine_launch<T, 4, KIND, ST>(g, src, dst, S, nl);
    case 5: return sine_launch<T, 5, KIND, ST>(g, src, dst, S, nl);
    case 6: return sine_launch<T, 6, KIND, ST>(g, src, dst, S, nl);
    case 7: return sine_launch<T, 7, KIND, ST>(g, src, dst, S, nl);
    case 8: return sine_launch<T, 8, KIND, ST>(g, src, dst, S, nl);
    }
    return fail(PPML_EINVAL, "sine transform of %d cells", n[axis]);
}

template <typename T> void sine_tables(ppml_grid *g)
{
    void *S[3] = {g->sx, g->sy, g->sz};
    double *f[3] = {g->fx, g->fy, g->fz};
    for (int a = 0; a < 3; a++) {
        const int n = g->gp.n[a];
        const long long m = std::max<long long>(sine_table_count<T>(n), n);
        k_sine_table<T><<<(unsigned)((m + 255) / 256), 256, 0, g->stream>>>((T *)S[a], f[a], n);
    }
}

// The potential of a state stored as ST by transforms in T.
template <typename T, typename ST> int sine_solve(ppml_grid *g)
{
    const GridParams &gp = g->gp;
    const ST *rho = (const ST *)g->state;
    ST *phi = (ST *)g->phi;
    T *E = (T *)g->gedge, *X = (T *)g->wx;
    const long long nedge = grav_edge_cells(gp.n[0], gp.n[1], gp.n[2]);
    k_grav_edge_terms<ST, T><<<(unsigned)((nedge + 255) / 256), 256, 0, g->stream>>>(phi, rho, g->grav_coef, gp, E);
    int rc;
    if ((rc = sine_pass<T, SINE_X_FWD, ST>(g, rho, X))) return rc;
    if ((rc = sine_pass<T, SINE_Y_FWD, T>(g, X, X))) return rc;
    if ((rc = sine_pass<T, SINE_Z, T>(g, X, X))) return rc;
    if ((rc = sine_pass<T, SINE_Y_INV, T>(g, X, X))) return rc;
    if ((rc = sine_pass<T, SINE_X_INV, ST>(g, X, phi))) return rc;
    HIPCHK(hipGetLastError());
    return PPML_OK;
}

// The self-gravity potential of the current state into g->phi (Sec. 2.5).
template <typename T> int launch_gravity(ppml_grid *g)
{
    const GridParams &gp = g->gp;
    const long long N = gp.ncell;
    const int n0 = gp.n[0], n1 = gp.n[1], n2 = gp.n[2];
    const T *rho = (const T *)g->state;
    T *phi = (T *)g->phi;
    T *X = (T *)g->wx;
    T *Y = (T *)g->wy;
    const int rows = n1 * n2;
    const int nb = grav_blocks(N);
    const int chunk = (rows + nb - 1) / nb;
    k_grav_moments_partial<T><<<nb, GRAV_THREADS, 0, g->stream>>>(rho, gp, chunk, g->gpart);
    k_grav_moments_final<<<1, GRAV_THREADS, 0, g->stream>>>(g->gpart, nb, g->ctrl);
    const long long nshell = (long long)(n0 + 2) * (n1 + 2) * (n2 + 2) - N;
    k_grav_shell<T><<<(unsigned)((nshell + 255) / 256), 256, 0, g->stream>>>(gp, g->ctrl, g->d.grav_G, phi);
    if (sine_kernels(&g->d)) return sine_fp64(&g->d) ? sine_solve<double, T>(g) : sine_solve<T, T>(g);
    // shell terms of the outer layer, then the right-hand side's sums and
    // differences into Y
    T *E = (T *)g->gedge;
    const long long nedge = grav_edge_cells(n0, n1, n2);
    k_grav_edge_terms<T, T><<<(unsigned)((nedge + 255) / 256), 256, 0, g->stream>>>(phi, nullptr, 0.0, gp, E);
    const long long nrep = (long long)grav_no(n0) * grav_no(n1) * grav_no(n2);
    const unsigned nbr = (unsigned)((nrep + 255) / 256);
    k_grav_butterfly<T><<<nbr, 256, 0, g->stream>>>(rho, E, g->grav_coef, Y, gp);
    HIPCHK(hipGetLastError());
    int rc;
    if ((rc = sine_transform<T>(g, 0, false, Y, X))) return rc;
    if ((rc = sine_transform<T>(g, 1, false, X, Y))) return rc;
    if ((rc = sine_transform<T>(g, 2, false, Y, X))) return rc;
    const dim3 ged((unsigned)((n0 + 255) / 256), (unsigned)std::min((rows + 3) / 4, 4096));
    k_grav_eigdiv<T><<<ged, 256, 0, g->stream>>>(X, g->fx, g->fy, g->fz, gp, g->grav_norm);
    HIPCHK(hipGetLastError());
    if ((rc = sine_transform<T>(g, 2, true, X, Y))) return rc;
    if ((rc = sine_transform<T>(g, 1, true, Y, X))) return rc;
    if ((rc = sine_transform<T>(g, 0, true, X, Y))) return rc;
    k_grav_unbutterfly<T><<<nbr, 256, 0, g->stream>>>(Y, phi, gp);
    HIPCHK(hipGetLastError());
    return PPML_OK;
}

template <typename T> int launch_step(ppml_grid *g, hipEvent_t *ev)
{
    // ev (may be NULL): events recorded before the gravity solve, before,
    // between and after the stage kernels
    if (ev) (void)hipEventRecord(ev[0], g->stream);
    if (g->gp.self_grav) {
        int rc = launch_gravity<T>(g);
        if (rc) return rc;
    }
    switch (g->d.ndim) {
    case 1: launch_stages<T, 1>(g, ev); break;
    case 2: launch_stages<T, 2>(g, ev); break;
    default: launch_stages<T, 3>(g, ev); break;
    }
    return PPML_OK;
}

// Totals of the state; partial: 48 bytes for each of totals_blocks.
template <typename T> void launch_totals(ppml_grid *g, double mean_cells, double *partial)
{
    const long long N = g->gp.ncell;
    int nb = totals_blocks(N);
    long long chunk = (N + nb - 1) / nb;
    k_totals_partial<T><<<nb, TOT_THREADS, 0, g->stream>>>((const T *)g->state, N, nfields(&g->d), chunk, partial);
    k_totals_final<<<1, TOT_THREADS, 0, g->stream>>>(partial, nb, nfields(&g->d), g->d.ndim, g->totals, g->ctrl,
                                                      mean_cells);
}

int check_err(ppml_grid *g)
{
    int err = 0;
    HIPCHK(hipMemcpyAsync(&err, &g->ctrl->err, sizeof(int), hipMemcpyDeviceToHost, g->stream));
    HIPCHK(hipStreamSynchronize(g->stream));
    if (err) return fail(PPML_ENONFINITE, "a step produced rho <= 0, eps <= 0 or a non-finite value");
    return PPML_OK;
}

int grid_ok(ppml_grid *g)
{
    if (!g) return fail(PPML_EINVAL, "grid is NULL");
    return PPML_OK;
}

// A grid in a batch is stepped on the batch's stream: calls that touch its
// state on the grid's own stream first wait for the batch's queued work.
int settle(ppml_grid *g)
{
    if (g->in_batch && g->bstream != g->stream) HIPCHK(hipStreamSynchronize(g->bstream));
    return PPML_OK;
}

// After the state is set: reset the control block, record the mean density
// (the given one, or the mean of the state when rho_mean0 <= 0), compute the
// CFL maxima of the state into slot 0.  Kernels only: nothing is copied from
// the host.
int finish_set_async(ppml_grid *g, double t, double rho_mean0)
{
    k_ctrl_reset<<<1, 2 * MSLOT_MAX, 0, g->stream>>>(g->ctrl, g->gp.mslots, t, rho_mean0);
    HIPCHK(hipGetLastError());
    // the partial sums go to the stage output's area (at least 256 bytes), which
    // holds nothing as long as the state is being set
    double *const partial = (double *)g->half;
    if (g->d.prec == PPML_FP64) {
        launch_totals<double>(g, rho_mean0 > 0.0 ? 0.0 : (double)g->gp.ncell, partial);
        launch_speeds<double>(g);
    } else {
        launch_totals<float>(g, rho_mean0 > 0.0 ? 0.0 : (double)g->gp.ncell, partial);
        launch_speeds<float>(g);
    }
    HIPCHK(hipGetLastError());
    g->has_state = true;
    return PPML_OK;
}

int finish_set(ppml_grid *g, double t, double rho_mean0)
{
    int rc = finish_set_async(g, t, rho_mean0);
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(g->stream));
    return PPML_OK;
}

// The transfers of ppml_transfer.hpp; their threads and buffers may not be had.
template <typename T>
int upload(ppml_grid *g, const double *const *src, int nsrc, T *dst, XferHold &hold, const char *what)
{
    hipError_t e;
    try {
        e = xfer_upload<T>(g->device, g->stream, src, nsrc, g->gp.ncell, dst, hold);
    } catch (const std::exception &) {
        return fail(PPML_ENOMEM, "%s: host allocation failed", what);
    }
    return e == hipSuccess ? PPML_OK : fail(PPML_EHIP, "%s: %s", what, hipGetErrorString(e));
}

template <typename T> int download(ppml_grid *g, const T *src, long long n, double *dst, const char *what)
{
    hipError_t e;
    try {
        e = xfer_download<T>(g->device, g->stream, src, n, dst);
    } catch (const std::exception &) {
        return fail(PPML_ENOMEM, "%s: host allocation failed", what);
    }
    return e == hipSuccess ? PPML_OK : fail(PPML_EHIP, "%s: %s", what, hipGetErrorString(e));
}

bool all_finite(const double *a, long long n, bool positive)
{
    try {
        return xfer_check(a, n, positive);
    } catch (const std::exception &) {
        // no memory for the threads' bookkeeping
    }
    for (long long i = 0; i < n; i++)
        if (!std::isfinite(a[i]) || (positive && !(a[i] > 0.0))) return false;
    return true;
}

// Number of z chunks of a 3-D stage launch.  A work group streams cz planes
// after `warm` planes of pipeline start-up (in units of a full plane); the
// launch runs in ceil(groups / slots) rounds of resident work groups, so the
// time is modelled as rounds * (cz + warm) and minimised over the chunk count.
int choose_chunks(long long tiles_xy, int nz, long long slots, double warm)
{
    if (slots < 1) slots = 1;
    int best = 1;
    double best_cost = 1e300;
    for (int c = 1; c <= nz; c++) {
        const int cz = (nz + c - 1) / c;
        if ((long long)(c - 1) * cz >= nz) continue;  // same chunks as a smaller count
        const long long groups = tiles_xy * c;
        if (groups > (1ll << 30)) break;
        const double rounds = (double)((groups + slots - 1) / slots);
        const double cost = rounds * (cz + warm);
        if (cost < best_cost * (1.0 - 1e-9)) {
            best_cost = cost;
            best = c;
        }
    }
    return best;
}

// (tile: as launched)
template <typename T> void stage_slots(int device, int tile, int xf, long long &slots_e, long long &slots_l)
{
    int cus = 0, be = 0, bl = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) cus = 0;
    with_tile<3>(tile, [&](auto tl) {
        using TL = decltype(tl);
        hipError_t e =
            xf == 2   ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&be, k_euler<T, 3, TL::tx, TL::ty, 2>, TL::nt, 0)
            : xf == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&be, k_euler<T, 3, TL::tx, TL::ty, 1>, TL::nt, 0)
                      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&be, k_euler<T, 3, TL::tx, TL::ty>, TL::nt, 0);
        if (e != hipSuccess) be = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&bl, k_lagr<T, 3, TL::tx, TL::ty, LG<T>::g>, TL::nt, 0) !=
            hipSuccess)
            bl = 0;
    });
    (void)hipGetLastError();
    if (cus < 1) cus = 256;
    slots_e = (long long)cus * (be > 0 ? be : 2);
    slots_l = (long long)cus * (bl > 0 ? bl : 2);
}

// Rows per wave of the 2-D grids that share a launch.  A row more costs a wave
// about what its first costs beyond the rows shared (1 + r, in rows); the 1024
// SIMDs work off the waves in turn, a wave alone on its SIMD taking 1.3 of its
// share.  us per step at 1, 2, 3, 8 rows, FP32: 256^2 11.9, 11.4, 12.7, 19.1;
// 371^2 15.4, 15.6, 14.3, 20.9; 768x700 32.3, 27.2, 28.6, 31.8; 1500^2 97, 78,
// 68, 65 (the tile kernels before: 13.9, 17.0, 31.2, 93); FP64 at 1, 2 rows:
// 256^2 16.6, 15.3; 1500^2 189, 147 (18.7, 216).
// (grid(i): the i-th; allocates nothing, as the allocation-free entry point
// comes through here)
template <typename F> int sheet_rows(int count, int prec, F &&grid)
{
    int best = 1;
    double best_t = 1e300;
    for (int r : SHEET_ROWS) {
        if (prec == PPML_FP64 && r > 2) break;
        double waves = 0.0;
        for (int i = 0; i < count; i++) {
            const GridParams &gp = grid(i);
            waves += (double)((gp.n[0] + SHEET_W - 1) / SHEET_W) * ((gp.n[1] + r - 1) / r);
        }
        const double t = (1.0 + r) * std::max(std::ceil(waves / 1024.0), 1.3);
        if (t < best_t) {
            best_t = t;
            best = r;
        }
    }
    return best;
}

void set_rows(GridParams &gp, int rows)
{
    gp.tiles[0] = (gp.n[0] + SHEET_W - 1) / SHEET_W;
    gp.tiles[1] = (gp.n[1] + rows - 1) / rows;
    gp.tiles[2] = 1;
    gp.cz = rows;
}

// Work-group tiling of a grid for tile shape v: x/y tiles, and a z chunk
// small enough that a 3-D grid alone gives the launch a few thousand work
// groups (batches then fit the chunks of their 3-D grids together).
void set_tiling(GridParams &gp, int ndim, int prec, int v)  // v: as launched
{
    if (ndim == 2) {
        set_rows(gp, sheet_rows(1, prec, [&](int) -> const GridParams & { return gp; }));
        return;
    }
    const int tx = TILE_X[ndim][v], ty = TILE_Y[ndim][v];
    gp.tiles[0] = (gp.n[0] + tx - 1) / tx;
    gp.tiles[1] = ndim >= 2 ? (gp.n[1] + ty - 1) / ty : 1;
    gp.tiles[2] = 1;
    gp.cz = 1;
    if (ndim == 3) {
        long long tiles = (long long)gp.tiles[0] * gp.tiles[1];
        int cz = gp.n[2];
        while (cz > 16 && tiles * ((gp.n[2] + cz - 1) / cz) < 2048) cz = (cz + 1) / 2;
        gp.cz = cz;
        gp.tiles[2] = (gp.n[2] + cz - 1) / cz;
    }
}

void set_chunks(GridParams &gp, int chunks)
{
    const int nz = gp.n[2];
    gp.cz = (nz + chunks - 1) / chunks;
    gp.tiles[2] = (nz + gp.cz - 1) / gp.cz;
}

// Z chunks shared by the 3-D grids of a batch: every work group of the launch
// streams at most cz planes after its start-up (`warm`, in plane units).  With
// the groups' work spread over the resident slots, the launch takes about
// max(sum of the groups' lengths / slots, the longest group); cz minimises
// that over all the batch's grids at once, where chunks chosen per grid as if
// it ran alone cut every grid into short chunks whose start-up dominates.
int batch_cz3(const std::vector<GridParams *> &gps, long long slots, double warm)
{
    int nzmax = 1;
    for (const GridParams *gp : gps) nzmax = gp->n[2] > nzmax ? gp->n[2] : nzmax;
    if (slots < 1) slots = 1;
    int best = nzmax;
    double best_t = 1e300;
    for (int c = 1; c <= nzmax; c++) {
        const int cz = (nzmax + c - 1) / c;
        if ((long long)(c - 1) * cz >= nzmax) continue;  // same cz as a smaller count
        double work = 0.0, longest = 0.0;
        for (const GridParams *gp : gps) {
            const int nz = gp->n[2];
            const int ch = (nz + cz - 1) / cz;
            const int czg = (nz + ch - 1) / ch;
            work += (double)gp->tiles[0] * gp->tiles[1] * ch * (czg + warm);
            longest = czg + warm > longest ? czg + warm : longest;
        }
        const double t = work / (double)slots > longest ? work / (double)slots : longest;
        if (t < best_t * (1.0 - 1e-9)) {
            best_t = t;
            best = cz;
        }
    }
    return best;
}

}  // namespace

extern "C" {

size_t ppml_state_bytes(const ppml_desc *d)
{
    if (validate(d) != PPML_OK) return 0;
    return (size_t)nfields(d) * (size_t)ncells(d) * elem(d);
}

size_t ppml_scratch_bytes(const ppml_desc *d)
{
    if (validate(d) != PPML_OK) return 0;
    return layout(d).total;
}

}  // extern "C"

namespace {

// Grid parameters, pointers into the scratch area and the inflow ghost states
// of a validated descriptor (everything of ppml_create but the self-gravity
// set-up and the z chunks).  Allocates nothing: g is the caller's object.
int init_grid(ppml_grid *g, const ppml_desc *d, void *state_dev, void *scratch_dev, void *hip_stream)
{
    g->d = *d;
    HIPCHK(hipGetDevice(&g->device));
    g->stream = (hipStream_t)hip_stream;
    g->state = state_dev;
    ScratchLayout L = layout(d);
    char *s = (char *)scratch_dev;
    g->half = s + L.half;
    g->ctrl = (Ctrl *)(s + L.ctrl);
    g->totals = (double *)(s + L.totals);
    GridParams &gp = g->gp;
    memset(&gp, 0, sizeof gp);
    gp.ndim = d->ndim;
    double hmin = 1e300;
    for (int a = 0; a < 3; a++) {
        gp.n[a] = (int)d->n[a];
        gp.lo[a] = d->lo[a];
        gp.h[a] = (d->hi[a] - d->lo[a]) / (double)d->n[a];
        gp.inv_h[a] = 1.0 / gp.h[a];
        gp.bc_lo[a] = a < d->ndim ? d->bc_lo[a] : PPML_PERIODIC;
        gp.bc_hi[a] = a < d->ndim ? d->bc_hi[a] : PPML_PERIODIC;
        if (a < d->ndim && gp.h[a] < hmin) hmin = gp.h[a];
    }
    gp.ncell = ncells(d);
    gp.mslots = maxima_slots(gp.ncell);
    gp.gamma = d->gamma;
    if (d->flags & PPML_FLAG_ISOTHERMAL) {
        gp.pa = d->iso_cs * d->iso_cs;
        gp.pb = 0.0;
        gp.gs = 1.0;
    } else {
        gp.pa = 0.0;
        gp.pb = d->gamma - 1.0;
        gp.gs = d->gamma;
    }
    gp.cfl_hmin = d->cfl * hmin;
    gp.vacuum_ratio = (d->flags & PPML_FLAG_ISOTHERMAL) ? 0.0 : d->vacuum_ratio;
    gp.potential = d->potential;
    gp.first_order = (d->flags & PPML_FLAG_FIRST_ORDER) ? 1 : 0;
    for (int i = 0; i < 8; i++) gp.pot[i] = d->pot[i];
    TileRule rule;
    rule.add(gp);
    g->ltile = d->ndim == 3 ? rule.tile(d->prec, d->tile) : d->tile;
    set_tiling(gp, d->ndim, d->prec, g->ltile);
    // conserved ghost states of inflow faces, converted in FP64 as the state
    // is, into the control block
    double tab[6][6];
    memset(tab, 0, sizeof tab);
    gp.any_inflow = 0;
    for (int a = 0; a < d->ndim; a++)
        for (int s = 0; s < 2; s++) {
            if ((s ? d->bc_hi[a] : d->bc_lo[a]) != PPML_INFLOW) continue;
            const double *st = d->inflow[2 * a + s];
            const double r = st[0];
            const double ux = st[1];
            const double uy = d->ndim >= 2 ? st[2] : 0.0;
            const double uz = d->ndim >= 3 ? st[3] : 0.0;
            const double e = st[4] / (d->gamma - 1.0);
            const double ke = 0.5 * r * (ux * ux + uy * uy + uz * uz);
            double *c = tab[2 * a + s];
            c[0] = r;
            c[1] = r * ux;
            c[2] = r * uy;
            c[3] = r * uz;
            c[4] = e + ke;
            c[5] = e;
            gp.any_inflow = 1;
        }
    if (gp.any_inflow) {
        InflowTable it;
        memcpy(it.v, tab, sizeof tab);
        k_set_inflow<<<1, 64, 0, g->stream>>>(g->ctrl, it);
        HIPCHK(hipGetLastError());
    }
    g->blas = nullptr;
    g->sexec = nullptr;
    g->graph_off = false;
    g->phi = g->wx = g->wy = g->sx = g->sy = g->sz = g->gedge = nullptr;
    g->fx = g->fy = g->fz = g->gpart = nullptr;
    g->has_state = false;
    g->in_batch = false;
    g->bstream = nullptr;
    g->timed = 0;
    return PPML_OK;
}

// Whether a 3-D grid alone takes the row kernels: up to four waves (row strips)
// per SIMD, the default tile shape (the others name the marching kernels' work
// groups) and no inflow face, whose ghost states the row kernels do not form.
// us per step, march / rows: FP32 24^3 30 / 20, 40x60x30 (1800 waves) 40 / 31,
// 58x27x148 (3996) 54 / 39, 64^3 (8192) 48 / 62, 100^3 (20000) 105 / 115; FP64
// 24^3 42 / 30, 40x60x30 56 / 45, 58x27x148 88 / 68, 64^3 71 / 114.
constexpr long long BRICK_WAVES = 4096;
// FP64 rows of up to eight cells (a launch of such strips takes 5 us longer than
// of wider ones, in both precisions) win over the march from some hundred on: us
// per step, march / rows: 5^3 33.2 / 36.6, 8^3 34.5 / 37.8, 8x16x16 35.1 / 36.8,
// 6x12x30 36.6 / 36.0, 4x32x32 42.7 / 34.7; 9^3 34.5 / 28.2.
constexpr long long BRICK_NARROW = 8, BRICK_NARROW_WAVES = 512;
bool brick_grid(const ppml_desc *d, const GridParams &gp)
{
    const long long waves = (d->n[0] + SHEET_W - 1) / SHEET_W * d->n[1] * d->n[2];
    if (d->ndim != 3 || d->tile != 0 || gp.any_inflow) return false;
    if (d->prec == PPML_FP64 && d->n[0] <= BRICK_NARROW && waves < BRICK_NARROW_WAVES) return false;
    return waves <= BRICK_WAVES;
}

// Z chunks of the solo stage launches, fitted to the resident work groups of
// each stage kernel (start-up cost: 3 z-only planes in the Eulerian kernel, 6
// in the Lagrangian kernel).  After the self-gravity set-up, which selects
// the Eulerian instantiation.
void init_chunks(ppml_grid *g)
{
    const GridParams &gp = g->gp;
    const ppml_desc *d = &g->d;
    g->gpE = gp;
    g->gpL = gp;
    g->gpB = gp;
    g->brick = brick_grid(d, gp);
    if (g->brick) {
        g->gpB.tiles[0] = (gp.n[0] + SHEET_W - 1) / SHEET_W;
        return;
    }
    if (d->ndim == 3) {
        long long se, sl;
        const int xf = gp.potential == POT_HALO ? 2 : (gp.self_grav ? 1 : 0);
        if (d->prec == PPML_FP64) stage_slots<double>(g->device, g->ltile, xf, se, sl);
        else stage_slots<float>(g->device, g->ltile, xf, se, sl);
        const long long txy = (long long)gp.tiles[0] * gp.tiles[1];
        set_chunks(g->gpE, choose_chunks(txy, gp.n[2], se, 1.5));
        set_chunks(g->gpL, choose_chunks(txy, gp.n[2], sl, 3.0));
    }
}

}  // namespace

extern "C" {

int ppml_create(const ppml_desc *d, void *state_dev, void *scratch_dev, void *hip_stream, ppml_grid **out)
{
    int rc = validate(d);
    if (rc != PPML_OK) return rc;
    if (!out) return fail(PPML_EINVAL, "out is NULL");
    if (!state_dev || !scratch_dev) return fail(PPML_EINVAL, "state and scratch pointers must be non-NULL");
    if (((uintptr_t)state_dev % ALIGN) || ((uintptr_t)scratch_dev % ALIGN))
        return fail(PPML_EINVAL, "device pointers must be %zu-byte aligned", ALIGN);
    ppml_grid *g = new (std::nothrow) ppml_grid();
    if (!g) return fail(PPML_ENOMEM, "host allocation failed");
    if ((rc = init_grid(g, d, state_dev, scratch_dev, hip_stream))) {
        delete g;
        return rc;
    }
    GridParams &gp = g->gp;
    const ScratchLayout L = layout(d);
    char *s = (char *)scratch_dev;
    if (d->self_gravity) {
        g->phi = s + L.phi;
        g->wx = s + L.wx;
        g->wy = s + L.wy;
        g->sx = s + L.sx;
        g->sy = s + L.sy;
        g->sz = s + L.sz;
        g->fx = (double *)(s + L.fx);
        g->fy = (double *)(s + L.fy);
        g->fz = (double *)(s + L.fz);
        g->gpart = (double *)(s + L.gpart);
        g->gedge = s + L.gedge;
        gp.self_grav = 1;
        gp.phi = g->phi;
        const double h = gp.h[0];
        g->grav_coef = 4.0 * M_PI * d->grav_G * h * h;
        g->grav_norm = (2.0 / (double)(gp.n[0] + 1)) * (2.0 / (double)(gp.n[1] + 1)) * (2.0 / (double)(gp.n[2] + 1));
        if (sine_kernels(d)) {
            if (sine_fp64(d)) sine_tables<double>(g);
            else sine_tables<float>(g);
        } else {
            if (rocblas_create_handle(&g->blas) != rocblas_status_success) {
                delete g;
                return fail(PPML_EHIP, "rocblas_create_handle failed");
            }
            if (rocblas_set_stream(g->blas, g->stream) != rocblas_status_success) {
                rocblas_destroy_handle(g->blas);
                delete g;
                return fail(PPML_EHIP, "rocblas_set_stream failed");
            }
            const long long nt = grav_table_count(gp.n[0]) + grav_table_count(gp.n[1]) + grav_table_count(gp.n[2]);
            const unsigned nbt = (unsigned)((nt + 255) / 256);
            if (d->prec == PPML_FP64)
                k_grav_tables<double><<<nbt, 256, 0, g->stream>>>((double *)g->sx, (double *)g->sy, (double *)g->sz,
                                                                   g->fx, g->fy, g->fz, gp.n[0], gp.n[1], gp.n[2]);
            else
                k_grav_tables<float><<<nbt, 256, 0, g->stream>>>((float *)g->sx, (float *)g->sy, (float *)g->sz, g->fx,
                                                                  g->fy, g->fz, gp.n[0], gp.n[1], gp.n[2]);
        }
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
        if (e != hipSuccess) {
            if (g->blas) rocblas_destroy_handle(g->blas);
            delete g;
            return fail(PPML_EHIP, "self-gravity tables: %s", hipGetErrorString(e));
        }
    }
    init_chunks(g);
    *out = g;
    return PPML_OK;
}

int ppml_set_primitive(ppml_grid *g, const double *rho, const double *vx, const double *vy, const double *vz,
                       const double *p)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    if (!rho || !p) return fail(PPML_EINVAL, "rho and p are required");
    const long long N = g->gp.ncell;
    if (!all_finite(rho, N, true)) return fail(PPML_EINVAL, "rho must be finite and > 0");
    if (!all_finite(p, N, true)) return fail(PPML_EINVAL, "p must be finite and > 0");
    const double *v[3] = {vx, vy, vz};
    for (int a = 0; a < g->d.ndim; a++)
        if (v[a] && !all_finite(v[a], N, false)) return fail(PPML_EINVAL, "velocity %d has non-finite values", a);
    double *prim = nullptr;
    HIPCHK(hipMallocAsync((void **)&prim, (size_t)5 * N * sizeof(double), g->stream));
    const double *src[5] = {rho, vx, vy, vz, p};
    XferHold hold;
    rc = upload<double>(g, src, 5, prim, hold, "copy of the primitives");
    hipError_t e = hipSuccess;
    if (rc == PPML_OK) {
        int nb = (int)std::min<long long>(4096, (N + 255) / 256);
        if (g->d.prec == PPML_FP64) k_prim_to_cons<double><<<nb, 256, 0, g->stream>>>(prim, (double *)g->state, g->gp);
        else k_prim_to_cons<float><<<nb, 256, 0, g->stream>>>(prim, (float *)g->state, g->gp);
        e = hipGetLastError();
    }
    (void)hipFreeAsync(prim, g->stream);
    if (rc) return rc;
    if (e != hipSuccess) return fail(PPML_EHIP, "prim_to_cons: %s", hipGetErrorString(e));
    return finish_set(g, 0.0, 0.0);
}

int ppml_set_conserved(ppml_grid *g, const double *const *f, double rho_mean0, double t)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    if (!f || !f[PPML_RHO] || !f[PPML_ETOT] || !f[PPML_EINT]) return fail(PPML_EINVAL, "rho, Et and e are required");
    const long long N = g->gp.ncell;
    const int nd = g->d.ndim;
    if (!all_finite(f[PPML_RHO], N, true)) return fail(PPML_EINVAL, "rho must be finite and > 0");
    if (!all_finite(f[PPML_EINT], N, true)) return fail(PPML_EINVAL, "rho*eps must be finite and > 0");
    if (!all_finite(f[PPML_ETOT], N, false)) return fail(PPML_EINVAL, "rho*E must be finite");
    if (!std::isfinite(t) || t < 0.0) return fail(PPML_EINVAL, "t must be finite and >= 0");
    // stored field s <- ppml_field
    const int nfs = nfields(&g->d);
    const double *src[6];
    for (int q = 0; q < nfs; q++) {
        const int fld = q == 0 ? PPML_RHO : (q <= nd ? q : (q == nd + 1 ? PPML_ETOT : PPML_EINT));
        src[q] = f[fld];
        if (q >= 1 && q <= nd && src[q] && !all_finite(src[q], N, false))
            return fail(PPML_EINVAL, "field %d has non-finite values", fld);
    }
    XferHold hold;
    rc = g->d.prec == PPML_FP64 ? upload<double>(g, src, nfs, (double *)g->state, hold, "set_conserved")
                                : upload<float>(g, src, nfs, (float *)g->state, hold, "set_conserved");
    if (rc) return rc;
    return finish_set(g, t, rho_mean0);
}

namespace {

// Steps per captured graph of a solo grid.  Every step reads its time step
// and run limits from the control block, so one graph of STEP_GRAPH steps
// serves any call; steps past the run's end are no-ops.
constexpr int STEP_GRAPH = 32;

// Capture STEP_GRAPH steps of the grid into g->sexec (once).  The launches
// are captured on a private non-blocking stream (the grid's own stream may be
// the null stream, which cannot be captured); the graph is then launched on
// the grid's stream, in order with the rest of its work.  False if capture
// fails; the caller then launches eagerly.
bool step_graph(ppml_grid *g)
{
    if (g->sexec) return true;
    if (g->graph_off) return false;
    g->graph_off = true;  // until the capture below succeeds
    // capture on the grid's device, whichever device is current
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != g->device && hipSetDevice(g->device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    hipStream_t cap = nullptr;
    if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        if (prev >= 0 && prev != g->device) (void)hipSetDevice(prev);
        return false;
    }
    hipGraph_t gr = nullptr;
    hipGraphExec_t ex = nullptr;
    bool ok = false;
    const hipStream_t own = g->stream;
    if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        g->stream = cap;
        int rc = PPML_OK;
        for (int s = 0; s < STEP_GRAPH && rc == PPML_OK; s++)
            rc = g->d.prec == PPML_FP64 ? launch_step<double>(g, nullptr) : launch_step<float>(g, nullptr);
        g->stream = own;
        const hipError_t e = hipStreamEndCapture(cap, &gr);
        ok = rc == PPML_OK && e == hipSuccess && gr && hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0) == hipSuccess;
    }
    if (gr) (void)hipGraphDestroy(gr);
    (void)hipStreamDestroy(cap);
    (void)hipGetLastError();
    if (prev >= 0 && prev != g->device) (void)hipSetDevice(prev);
    if (!ok) {
        if (ex) (void)hipGraphExecDestroy(ex);
        return false;
    }
    g->sexec = ex;
    g->graph_off = false;
    return true;
}

}  // namespace

int ppml_step(ppml_grid *g, int32_t nsteps, double dt_fixed, double t_stop)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if (nsteps < 0) return fail(PPML_EINVAL, "nsteps must be >= 0");
    if (!g->has_state) return fail(PPML_ESTATE, "state was never set");
    if (!std::isfinite(dt_fixed) || !std::isfinite(t_stop)) return fail(PPML_EINVAL, "dt_fixed and t_stop must be finite");
    if (nsteps == 0) return PPML_OK;
    if (g->in_batch) return fail(PPML_ESTATE, "grid is stepped by its batch");
    // per-step timing splits the step into its stage kernels
    const bool timing = (size_t)(4 * (g->timed + 1)) <= g->ev.size();
    const bool line = line_grid(&g->d, nsteps);
    if (line && !timing)
        return g->d.prec == PPML_FP64 ? launch_line<double>(g, nsteps, dt_fixed, t_stop, true)
                                      : launch_line<float>(g, nsteps, dt_fixed, t_stop, true);
    k_set_run<<<1, 1, 0, g->stream>>>(g->ctrl, dt_fixed, t_stop, (long long)nsteps);
    HIPCHK(hipGetLastError());  // before a capture attempt clears the last error
    // long calls replay the captured chunk (launch overhead once per
    // STEP_GRAPH steps); not while per-step timing is recorded, nor with
    // self-gravity (its library GEMMs, on long axes, stay outside captured
    // graphs)
    int s = 0;
    if (nsteps >= STEP_GRAPH && !timing && !g->gp.self_grav && step_graph(g)) {
        for (; s + STEP_GRAPH <= nsteps; s += STEP_GRAPH) HIPCHK(hipGraphLaunch(g->sexec, g->stream));
    }
    for (; s < nsteps; s++) {
        hipEvent_t *ev = nullptr;
        if ((size_t)(4 * (g->timed + 1)) <= g->ev.size()) ev = &g->ev[4 * g->timed];
        if (line && !ev)  // past the timed steps
            return g->d.prec == PPML_FP64 ? launch_line<double>(g, nsteps - s, 0.0, 0.0, false)
                                          : launch_line<float>(g, nsteps - s, 0.0, 0.0, false);
        rc = g->d.prec == PPML_FP64 ? launch_step<double>(g, ev) : launch_step<float>(g, ev);
        if (rc) return rc;
        if (ev) g->timed++;
    }
    HIPCHK(hipGetLastError());
    return PPML_OK;
}

}  // extern "C"

// Work area of ppml_step_noalloc: the Eulerian-stage output, the control block
// and the CFL maxima of one grid, one copy per GPU the library runs on,
// held until the process ends.  Host code never passes the array's name to a
// kernel or a copy (in host code it is only a stand-in for the device
// symbol): its device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[PPML_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int NOALLOC_MAX_DEV = 64;
std::mutex g_noalloc_mu;
void *g_noalloc_ptr[NOALLOC_MAX_DEV];

// Device address of the work area on the current device (looked up on the
// first call on that device, with the device current).
int noalloc_area(int device, void **out)
{
    if (device < 0 || device >= NOALLOC_MAX_DEV) return fail(PPML_EINVAL, "device %d out of range", device);
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(PPML_EHIP, "hipGetSymbolAddress of the work area: %s", hipGetErrorString(e));
        g_noalloc_ptr[device] = ptr;
    }
    *out = g_noalloc_ptr[device];
    return PPML_OK;
}

}  // namespace

extern "C" {

int ppml_step_noalloc(const ppml_desc *d, void *state_dev, double rho_mean0, double t0, int32_t nsteps,
                      double dt_fixed, double t_stop, void *hip_stream, double *t_out, int64_t *steps_out)
{
    int rc = validate(d);
    if (rc != PPML_OK) return rc;
    if (d->self_gravity) return fail(PPML_EINVAL, "self-gravity grids step through ppml_create / ppml_step");
    if (!state_dev) return fail(PPML_EINVAL, "state pointer must be non-NULL");
    if ((uintptr_t)state_dev % ALIGN) return fail(PPML_EINVAL, "the state pointer must be %zu-byte aligned", ALIGN);
    if (nsteps < 0) return fail(PPML_EINVAL, "nsteps must be >= 0");
    if (!std::isfinite(dt_fixed) || !std::isfinite(t_stop) || !std::isfinite(rho_mean0))
        return fail(PPML_EINVAL, "dt_fixed, t_stop and rho_mean0 must be finite");
    if (!std::isfinite(t0) || t0 < 0.0) return fail(PPML_EINVAL, "t0 must be finite and >= 0");
    const size_t need = layout(d).total;
    if (need > (size_t)PPML_NOALLOC_SCRATCH_BYTES)
        return fail(PPML_EINVAL, "the grid needs %zu bytes of work area; the fixed area holds %zu", need,
                    (size_t)PPML_NOALLOC_SCRATCH_BYTES);
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    void *area = nullptr;
    if ((rc = noalloc_area(dev, &area))) return rc;
    ppml_grid g{};  // on the stack: no host allocation
    if ((rc = init_grid(&g, d, state_dev, area, hip_stream))) return rc;
    init_chunks(&g);
    // every value of the work area that a step reads is written first: the
    // control block and the maxima slots by the reset, the mean density and the
    // partials by the kernels below, the stage output by the Eulerian kernel
    if ((rc = finish_set_async(&g, t0, rho_mean0))) return rc;
    if (nsteps > 0 && line_grid(d, nsteps)) {
        rc = d->prec == PPML_FP64 ? launch_line<double>(&g, nsteps, dt_fixed, t_stop, true)
                                  : launch_line<float>(&g, nsteps, dt_fixed, t_stop, true);
        if (rc) return rc;
    } else if (nsteps > 0) {
        k_set_run<<<1, 1, 0, g.stream>>>(g.ctrl, dt_fixed, t_stop, (long long)nsteps);
        HIPCHK(hipGetLastError());
        for (int s = 0; s < nsteps; s++) {
            rc = d->prec == PPML_FP64 ? launch_step<double>(&g, nullptr) : launch_step<float>(&g, nullptr);
            if (rc) return rc;
        }
    }
    HIPCHK(hipGetLastError());
    if (t_out || steps_out) {
        Ctrl c;
        HIPCHK(hipMemcpyAsync(&c, g.ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, g.stream));
        HIPCHK(hipStreamSynchronize(g.stream));
        if (t_out) *t_out = c.t;
        if (steps_out) *steps_out = c.steps;
        if (c.err) return fail(PPML_ENONFINITE, "a step produced rho <= 0, eps <= 0 or a non-finite value");
    }
    return PPML_OK;
}

int ppml_get_time(ppml_grid *g, double *t, double *dt_last, int64_t *steps)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    Ctrl c;
    HIPCHK(hipMemcpyAsync(&c, g->ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, g->stream));
    HIPCHK(hipStreamSynchronize(g->stream));
    if (t) *t = c.t;
    if (dt_last) *dt_last = c.dt_last;
    if (steps) *steps = c.steps;
    if (c.err) return fail(PPML_ENONFINITE, "a step produced rho <= 0, eps <= 0 or a non-finite value");
    return PPML_OK;
}

int ppml_max_speeds(ppml_grid *g, double *vmax, double *cmax)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    Ctrl c;
    k_fold_max<<<1, 64, 0, g->stream>>>(g->ctrl, g->gp.mslots);
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(&c, g->ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, g->stream));
    HIPCHK(hipStreamSynchronize(g->stream));
    double v, cs;
    unsigned long long vb = c.vmax_bits, cb = c.cmax_bits;
    memcpy(&v, &vb, sizeof v);
    memcpy(&cs, &cb, sizeof cs);
    if (vmax) *vmax = v;
    if (cmax) *cmax = cs;
    return PPML_OK;
}

int ppml_get_conserved(ppml_grid *g, int32_t field, double *host_out)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    if (!host_out) return fail(PPML_EINVAL, "host_out is NULL");
    const int nd = g->d.ndim;
    int s;
    switch (field) {
    case PPML_RHO: s = 0; break;
    case PPML_MX: s = 1; break;
    case PPML_MY: s = nd >= 2 ? 2 : -1; break;
    case PPML_MZ: s = nd >= 3 ? 3 : -1; break;
    case PPML_ETOT: s = nd + 1; break;
    case PPML_EINT: s = nd + 2; break;
    default: s = -1;
    }
    if (s < 0) return fail(PPML_EINVAL, "field %d is not stored for ndim=%d", field, nd);
    const long long N = g->gp.ncell;
    return g->d.prec == PPML_FP64 ? download<double>(g, (const double *)g->state + (size_t)s * N, N, host_out, "get_conserved")
                                  : download<float>(g, (const float *)g->state + (size_t)s * N, N, host_out, "get_conserved");
}

int ppml_totals(ppml_grid *g, double out[6])
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    if (!out) return fail(PPML_EINVAL, "out is NULL");
    if (!g->has_state) return fail(PPML_ESTATE, "state was never set");
    // (a buffer of its own: a read leaves the stage output alone, which another
    // thread's batch call may be using)
    double *partial = nullptr;
    HIPCHK(hipMallocAsync((void **)&partial, (size_t)totals_blocks(g->gp.ncell) * 6 * sizeof(double), g->stream));
    if (g->d.prec == PPML_FP64) launch_totals<double>(g, 0.0, partial);
    else launch_totals<float>(g, 0.0, partial);
    const hipError_t e = hipGetLastError();
    (void)hipFreeAsync(partial, g->stream);
    HIPCHK(e);
    HIPCHK(hipMemcpyAsync(out, g->totals, 6 * sizeof(double), hipMemcpyDeviceToHost, g->stream));
    HIPCHK(hipStreamSynchronize(g->stream));
    return PPML_OK;
}

int ppml_sync(ppml_grid *g)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if ((rc = settle(g))) return rc;
    return check_err(g);
}

int ppml_set_timing(ppml_grid *g, int32_t cap)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if (cap < 0 || cap > (1 << 20)) return fail(PPML_EINVAL, "timing capacity out of range");
    HIPCHK(hipStreamSynchronize(g->stream));
    for (hipEvent_t e : g->ev) (void)hipEventDestroy(e);
    g->ev.clear();
    g->timed = 0;
    for (int i = 0; i < 4 * cap; i++) {
        hipEvent_t e;
        HIPCHK(hipEventCreate(&e));
        g->ev.push_back(e);
    }
    return PPML_OK;
}

int ppml_get_timing_split(ppml_grid *g, double ms[3], int64_t *nsteps)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(g->stream));
    double acc[3] = {0.0, 0.0, 0.0};
    for (long long s = 0; s < g->timed; s++)
        for (int q = 0; q < 3; q++) {
            float a = 0.f;
            HIPCHK(hipEventElapsedTime(&a, g->ev[4 * s + q], g->ev[4 * s + q + 1]));
            acc[q] += a;
        }
    if (ms)
        for (int q = 0; q < 3; q++) ms[q] = acc[q];
    if (nsteps) *nsteps = g->timed;
    g->timed = 0;
    return PPML_OK;
}

int ppml_get_timing(ppml_grid *g, double *ms_euler, double *ms_lagr, int64_t *nsteps)
{
    double ms[3];
    int rc = ppml_get_timing_split(g, ms, nsteps);
    if (rc) return rc;
    if (ms_euler) *ms_euler = ms[1];
    if (ms_lagr) *ms_lagr = ms[2];
    return PPML_OK;
}

int ppml_get_potential(ppml_grid *g, double *host_out)
{
    int rc = grid_ok(g);
    if (rc) return rc;
    if (!host_out) return fail(PPML_EINVAL, "host_out is NULL");
    if (!g->gp.self_grav) return fail(PPML_EINVAL, "self-gravity is off for this grid");
    if (!g->has_state) return fail(PPML_ESTATE, "state was never set");
    if (g->in_batch) return fail(PPML_ESTATE, "grid is stepped by its batch");
    rc = g->d.prec == PPML_FP64 ? launch_gravity<double>(g) : launch_gravity<float>(g);
    if (rc) return rc;
    const long long np = (long long)(g->gp.n[0] + 2) * (g->gp.n[1] + 2) * (g->gp.n[2] + 2);
    return g->d.prec == PPML_FP64 ? download<double>(g, (const double *)g->phi, np, host_out, "get_potential")
                                  : download<float>(g, (const float *)g->phi, np, host_out, "get_potential");
}

int ppml_destroy(ppml_grid *g)
{
    if (!g) return fail(PPML_EINVAL, "grid is NULL");
    if (g->in_batch) return fail(PPML_ESTATE, "retire the grid from its batch first");
    (void)hipStreamSynchronize(g->stream);
    for (hipEvent_t e : g->ev) (void)hipEventDestroy(e);
    if (g->sexec) (void)hipGraphExecDestroy(g->sexec);
    if (g->blas) rocblas_destroy_handle(g->blas);
    delete g;
    return PPML_OK;
}

const char *ppml_strerror(int status)
{
    switch (status) {
    case PPML_OK: return "ok";
    case PPML_EINVAL: return "invalid argument";
    case PPML_ENOMEM: return "out of memory";
    case PPML_EHIP: return "HIP runtime error";
    case PPML_ENONFINITE: return "non-physical or non-finite state";
    case PPML_EBUDGET: return "memory budget exceeded";
    case PPML_ESTATE: return "invalid object state";
    default: return "unknown status";
    }
}

const char *ppml_last_error(void) { return g_err; }

int ppml_version(void) { return 100; }

int ppml_tile_count(int32_t ndim)
{
    if (ndim < 1 || ndim > 3) return fail(PPML_EINVAL, "ndim must be 1, 2 or 3 (got %d)", ndim);
    return NTILE[ndim];
}

int ppml_tile_shape(int32_t ndim, int32_t variant, int32_t *tx, int32_t *ty)
{
    if (ndim < 1 || ndim > 3) return fail(PPML_EINVAL, "ndim must be 1, 2 or 3 (got %d)", ndim);
    if (variant < 0 || variant >= NTILE[ndim]) return fail(PPML_EINVAL, "tile %d out of range", variant);
    if (tx) *tx = TILE_X[ndim][variant];
    if (ty) *ty = TILE_Y[ndim][variant];
    return PPML_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batches
// ---------------------------------------------------------------------------
struct ppml_batch {
    hipStream_t stream;
    int device;
    int capacity;
    size_t budget;   // 0: unlimited
    size_t in_use;   // state + scratch bytes of the admitted grids
    int prec;        // precision shared by all admitted grids (-1: none yet)
    std::vector<ppml_grid *> slots;
    BatchEntry *d_ents;   // device table, grouped by dimensionality
    int *d_steps;         // device per-entry step counts, then ...
    int *d_first;         // ... first work group of every entry in its launch
    BatchEntry *h_ents;   // pinned host copies
    int *h_steps;
    std::vector<int> entry_slot;
    int goff[4], gn[4], gtiles[4];  // grids stepped by the stage kernels, per dimensionality
    int rows2;            // rows per wave of the 2-D launches
    int few;              // steps of the calls the table is built for, 0: four and more
    bool few_matters;     // some grid takes the line kernel by the steps of a call
    int nline, nlds;      // 1-D grids stepped by the line kernel, first in the table; those of them in LDS
    long long line_nmax, lds_nmax;  // cells of the longest
    int tile[4], ltile[4];  // tile shape per dimensionality, as set and as launched
    bool dirty;
    long long version;
    hipGraph_t graph;
    hipGraphExec_t exec;
    int graph_nsteps;
    long long graph_version;
    // grids of different dimensionalities share nothing: their launch chains
    // run as parallel branches (streams forked from and joined to the batch
    // stream, default priority), so the 1-D launches overlap the 2-D and 3-D
    // ones instead of adding their time; side[0] runs the line kernel.
    hipStream_t side[4];
    hipEvent_t ev_fork, ev_join[4];
};

namespace {

size_t grid_bytes(const ppml_grid *g) { return ppml_state_bytes(&g->d) + ppml_scratch_bytes(&g->d); }

int batch_rebuild(ppml_batch *b)
{
    int n = 0;
    b->entry_slot.clear();
    bool beside = false;  // grids of more than one dimension share the batch
    TileRule rule;
    bool near = false;  // 1-D grids near the line kernel's limit
    for (const ppml_grid *g : b->slots) {
        near = near || (g && line_grid(&g->d) && !line_grid(&g->d, 1));
        beside = beside || (g && g->d.ndim > 1);
        if (g && g->d.ndim == 3) rule.add(g->gp);
    }
    for (int nd = 1; nd <= 3; nd++) b->ltile[nd] = nd == 3 ? rule.tile(b->prec, b->tile[3]) : b->tile[nd];
    b->few_matters = near && !beside;
    // kind: 0 stage kernels, 1 line kernel in LDS, 2 line kernel in memory
    auto kind_of = [&](const ppml_grid *g) {
        if (line_grid(&g->d, beside ? 0 : b->few)) return 1;
        return beside && g->d.ndim == 1 && g->d.n[0] <= LINE_BATCH_CELLS ? 2 : 0;
    };
    auto add = [&](int nd, int kind) {
        for (int s = 0; s < b->capacity; s++) {
            ppml_grid *g = b->slots[s];
            if (!g || g->d.ndim != nd || kind_of(g) != kind) continue;
            BatchEntry &e = b->h_ents[n];
            e.gp = g->gp;
            set_tiling(e.gp, nd, b->prec, b->ltile[nd]);
            e.state = g->state;
            e.half = g->half;
            e.ctrl = g->ctrl;
            e.tile0 = 0;
            e.pad = 0;
            b->entry_slot.push_back(s);
            n++;
        }
    };
    add(1, 1);
    b->nlds = n;
    b->lds_nmax = 0;
    for (int i = 0; i < n; i++) b->lds_nmax = std::max<long long>(b->lds_nmax, b->h_ents[i].gp.n[0]);
    add(1, 2);
    b->nline = n;
    b->line_nmax = 0;
    for (int i = 0; i < n; i++) b->line_nmax = std::max<long long>(b->line_nmax, b->h_ents[i].gp.n[0]);
    for (int nd = 1; nd <= 3; nd++) {
        b->goff[nd] = n;
        int tiles = 0;
        add(nd, 0);
        b->gn[nd] = n - b->goff[nd];
        if (nd == 2 && b->gn[2] > 0) {
            const BatchEntry *ents = b->h_ents + b->goff[2];
            b->rows2 = sheet_rows(b->gn[2], b->prec, [&](int i) -> const GridParams & { return ents[i].gp; });
            for (int i = b->goff[2]; i < n; i++) set_rows(b->h_ents[i].gp, b->rows2);
        }
        if (nd == 3 && b->gn[3] > 0) {
            // one chunk length for all 3-D grids, fitted to the Lagrangian
            // kernel's resident work groups (its start-up: 6 z-only planes,
            // about 3 full ones)
            std::vector<GridParams *> gps;
            for (int i = b->goff[3]; i < n; i++) gps.push_back(&b->h_ents[i].gp);
            long long se, sl;
            if (b->prec == PPML_FP64) stage_slots<double>(b->device, b->ltile[3], 0, se, sl);
            else stage_slots<float>(b->device, b->ltile[3], 0, se, sl);
            const int cz = batch_cz3(gps, sl, 3.0);
            for (GridParams *gp : gps) set_chunks(*gp, (gp->n[2] + cz - 1) / cz);
        }
        for (int i = b->goff[nd]; i < n; i++) {
            BatchEntry &e = b->h_ents[i];
            e.tile0 = tiles;
            tiles += work_groups(e.gp);
        }
        b->gtiles[nd] = tiles;
    }
    if (n > 0) {
        HIPCHK(hipMemcpyAsync(b->d_ents, b->h_ents, (size_t)n * sizeof(BatchEntry), hipMemcpyHostToDevice, b->stream));
        int *first = b->h_steps + b->capacity;
        for (int i = 0; i < n; i++) first[i] = b->h_ents[i].tile0;
        b->d_first = b->d_steps + b->capacity;
        HIPCHK(hipMemcpyAsync(b->d_first, first, (size_t)n * sizeof(int), hipMemcpyHostToDevice, b->stream));
        HIPCHK(hipStreamSynchronize(b->stream));
    }
    b->dirty = false;
    b->version++;
    return PPML_OK;
}

template <typename T, int NDIM> void batch_stage(ppml_batch *b, bool lagr, hipStream_t st)
{
    if (!b->gn[NDIM]) return;
    if constexpr (NDIM == 2) {
        const BatchEntry *e = b->d_ents + b->goff[2];
        const int *first = b->d_first + b->goff[2];
        with_rows<T>(b->rows2, [&](auto rows) {
            constexpr int R = decltype(rows)::value;
            if (lagr) k_lagr_sheet_batch<T, R><<<b->gtiles[2], SHEET_THREADS, 0, st>>>(e, first, b->gn[2]);
            else k_euler_sheet_batch<T, R><<<b->gtiles[2], SHEET_THREADS, 0, st>>>(e, first, b->gn[2]);
        });
    } else {
        with_tile<NDIM>(b->ltile[NDIM], [&](auto tl) {
            using TL = decltype(tl);
            const BatchEntry *e = b->d_ents + b->goff[NDIM];
            const int *first = b->d_first + b->goff[NDIM];
            if (lagr)
                k_lagr_batch<T, NDIM, TL::tx, TL::ty, LG<T>::g><<<b->gtiles[NDIM], TL::nt, 0, st>>>(e, first, b->gn[NDIM]);
            else
                k_euler_batch<T, NDIM, TL::tx, TL::ty><<<b->gtiles[NDIM], TL::nt, 0, st>>>(e, first, b->gn[NDIM]);
        });
    }
}

template <typename T, int NDIM> void batch_chain(ppml_batch *b, int nsteps, hipStream_t st)
{
    for (int s = 0; s < nsteps; s++) {
        batch_stage<T, NDIM>(b, false, st);
        batch_stage<T, NDIM>(b, true, st);
    }
}

// nsteps steps of the short 1-D grids.
template <typename T> int batch_lines(ppml_batch *b, int nsteps, hipStream_t st)
{
    const size_t lds = line_lds<T>(b->lds_nmax);
    if (lds > 65536)
        HIPCHK(hipFuncSetAttribute((const void *)k_line_batch<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    for (int s = 0; s < nsteps; s += LINE_STEPS)
        k_line_batch<T><<<b->nline, line_threads(b->line_nmax), lds, st>>>(
            b->d_ents, b->nlds, std::min(LINE_STEPS, nsteps - s));
    return PPML_OK;
}

// nsteps steps of every grid: one chain of stage launches per dimensionality
// present, and the line kernel; with more than one, each runs on a side stream
// forked from the batch stream and joined back to it.
template <typename T> int batch_enqueue(ppml_batch *b, int nsteps)
{
    int present = b->nline ? 1 : 0;
    for (int nd = 1; nd <= 3; nd++) present += b->gn[nd] ? 1 : 0;
    const bool fork = present > 1;
    if (fork) HIPCHK(hipEventRecord(b->ev_fork, b->stream));
    for (int nd = 0; nd <= 3; nd++) {
        if (!(nd == 0 ? b->nline : b->gn[nd])) continue;
        hipStream_t st = fork ? b->side[nd] : b->stream;
        if (fork) HIPCHK(hipStreamWaitEvent(st, b->ev_fork, 0));
        if (nd == 0) {
            const int rc = batch_lines<T>(b, nsteps, st);
            if (rc) return rc;
        } else if (nd == 1) batch_chain<T, 1>(b, nsteps, st);
        else if (nd == 2) batch_chain<T, 2>(b, nsteps, st);
        else batch_chain<T, 3>(b, nsteps, st);
        HIPCHK(hipGetLastError());
        if (fork) {
            HIPCHK(hipEventRecord(b->ev_join[nd], st));
            HIPCHK(hipStreamWaitEvent(b->stream, b->ev_join[nd], 0));
        }
    }
    return PPML_OK;
}

void batch_drop_graph(ppml_batch *b)
{
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
    b->graph_nsteps = -1;
}

}  // namespace

extern "C" {

int ppml_batch_create(int32_t capacity, size_t budget_bytes, void *hip_stream, ppml_batch **out)
{
    if (!out) return fail(PPML_EINVAL, "out is NULL");
    if (capacity < 1 || capacity > 65536) return fail(PPML_EINVAL, "capacity must be in [1, 65536]");
    int device = 0;
    HIPCHK(hipGetDevice(&device));
    ppml_batch *b = new (std::nothrow) ppml_batch();
    if (!b) return fail(PPML_ENOMEM, "host allocation failed");
    b->stream = (hipStream_t)hip_stream;
    b->device = device;
    b->capacity = capacity;
    b->budget = budget_bytes;
    b->in_use = 0;
    b->prec = -1;
    b->slots.assign(capacity, nullptr);
    b->d_ents = nullptr;
    b->d_steps = nullptr;
    b->h_ents = nullptr;
    b->h_steps = nullptr;
    b->dirty = true;
    b->nline = b->nlds = 0;
    b->few = 0;
    b->few_matters = false;
    b->line_nmax = b->lds_nmax = 0;
    b->rows2 = 1;
    b->d_first = nullptr;
    for (int nd = 0; nd < 4; nd++) b->tile[nd] = 0;
    b->version = 0;
    b->graph = nullptr;
    b->exec = nullptr;
    b->graph_nsteps = -1;
    b->graph_version = -1;
    for (int nd = 0; nd < 4; nd++) {
        b->side[nd] = nullptr;
        b->ev_join[nd] = nullptr;
    }
    b->ev_fork = nullptr;
    hipError_t e = hipMalloc(&b->d_ents, (size_t)capacity * sizeof(BatchEntry));
    if (e == hipSuccess) e = hipMalloc(&b->d_steps, (size_t)2 * capacity * sizeof(int));
    if (e == hipSuccess) e = hipEventCreateWithFlags(&b->ev_fork, hipEventDisableTiming);
    for (int nd = 0; nd <= 3 && e == hipSuccess; nd++) {
        e = hipStreamCreateWithFlags(&b->side[nd], hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&b->ev_join[nd], hipEventDisableTiming);
    }
    if (e == hipSuccess) e = hipHostMalloc(&b->h_ents, (size_t)capacity * sizeof(BatchEntry), hipHostMallocDefault);
    if (e == hipSuccess) e = hipHostMalloc(&b->h_steps, (size_t)2 * capacity * sizeof(int), hipHostMallocDefault);
    if (e != hipSuccess) {
        if (b->d_ents) (void)hipFree(b->d_ents);
        if (b->d_steps) (void)hipFree(b->d_steps);
        if (b->h_ents) (void)hipHostFree(b->h_ents);
        if (b->h_steps) (void)hipHostFree(b->h_steps);
        for (int nd = 0; nd <= 3; nd++) {
            if (b->side[nd]) (void)hipStreamDestroy(b->side[nd]);
            if (b->ev_join[nd]) (void)hipEventDestroy(b->ev_join[nd]);
        }
        if (b->ev_fork) (void)hipEventDestroy(b->ev_fork);
        delete b;
        return fail(PPML_ENOMEM, "batch tables: %s", hipGetErrorString(e));
    }
    *out = b;
    return PPML_OK;
}

int ppml_batch_admit(ppml_batch *b, ppml_grid *g, int32_t *slot)
{
    if (!b || !g) return fail(PPML_EINVAL, "batch and grid are required");
    if (g->in_batch) return fail(PPML_ESTATE, "grid already belongs to a batch");
    if (!g->has_state) return fail(PPML_ESTATE, "grid state was never set");
    if (g->device != b->device) return fail(PPML_EINVAL, "grid and batch live on different devices");
    if (b->prec >= 0 && g->d.prec != b->prec) return fail(PPML_EINVAL, "all grids of a batch share one precision");
    if (g->gp.self_grav || g->gp.potential == POT_HALO)
        return fail(PPML_EINVAL, "grids with self-gravity or the halo potential step alone, not in a batch");
    const size_t need = grid_bytes(g);
    if (b->budget > 0 && b->in_use + need > b->budget)
        return fail(PPML_EBUDGET, "admitting %zu bytes would exceed the budget (%zu of %zu in use)", need, b->in_use,
                    b->budget);
    int s = -1;
    for (int i = 0; i < b->capacity; i++)
        if (!b->slots[i]) {
            s = i;
            break;
        }
    if (s < 0) return fail(PPML_EBUDGET, "batch is full (%d grids)", b->capacity);
    HIPCHK(hipStreamSynchronize(b->stream));
    HIPCHK(hipStreamSynchronize(g->stream));
    b->slots[s] = g;
    b->in_use += need;
    b->prec = g->d.prec;
    g->in_batch = true;
    g->bstream = b->stream;
    b->dirty = true;
    if (slot) *slot = s;
    return PPML_OK;
}

int ppml_batch_retire(ppml_batch *b, int32_t slot)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    if (slot < 0 || slot >= b->capacity || !b->slots[slot]) return fail(PPML_EINVAL, "slot %d is not in use", slot);
    HIPCHK(hipStreamSynchronize(b->stream));
    ppml_grid *g = b->slots[slot];
    g->in_batch = false;
    b->in_use -= grid_bytes(g);
    b->slots[slot] = nullptr;
    b->dirty = true;
    bool any = false;
    for (ppml_grid *x : b->slots) any = any || x;
    if (!any) b->prec = -1;
    return PPML_OK;
}

int ppml_batch_step(ppml_batch *b, int32_t nsteps, const int32_t *steps_per_slot, double dt_fixed, double t_stop,
                    int32_t use_graph)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    if (nsteps < 0) return fail(PPML_EINVAL, "nsteps must be >= 0");
    if (!std::isfinite(dt_fixed) || !std::isfinite(t_stop)) return fail(PPML_EINVAL, "dt_fixed and t_stop must be finite");
    HIPCHK(hipStreamSynchronize(b->stream));  // staging buffers are free again
    const int few = nsteps > 0 && nsteps < 4 ? nsteps : 0;
    if (b->few_matters && nsteps > 0 && few != b->few) b->dirty = true;
    if (b->dirty) {
        b->few = few;
        int rc = batch_rebuild(b);
        if (rc) return rc;
    }
    const int n = (int)b->entry_slot.size();
    if (n == 0 || nsteps == 0) return PPML_OK;
    for (int i = 0; i < n; i++) {
        int s = b->entry_slot[i];
        int k = steps_per_slot ? steps_per_slot[s] : nsteps;
        if (k < 0 || k > nsteps) return fail(PPML_EINVAL, "steps of slot %d must lie in [0, nsteps]", s);
        b->h_steps[i] = k;
    }
    HIPCHK(hipMemcpyAsync(b->d_steps, b->h_steps, (size_t)n * sizeof(int), hipMemcpyHostToDevice, b->stream));
    k_batch_set_run<<<(n + 255) / 256, 256, 0, b->stream>>>(b->d_ents, n, b->d_steps, dt_fixed, t_stop);
    HIPCHK(hipGetLastError());
    const bool fp64 = b->prec == PPML_FP64;
    if (use_graph) {
        if (!b->exec || b->graph_version != b->version || b->graph_nsteps != nsteps) {
            batch_drop_graph(b);
            HIPCHK(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
            const int erc = fp64 ? batch_enqueue<double>(b, nsteps) : batch_enqueue<float>(b, nsteps);
            hipGraph_t gr = nullptr;
            const hipError_t ce = hipStreamEndCapture(b->stream, &gr);
            if (erc) {
                if (gr) (void)hipGraphDestroy(gr);
                return erc;
            }
            HIPCHK(ce);
            b->graph = gr;
            HIPCHK(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
            b->graph_nsteps = nsteps;
            b->graph_version = b->version;
        }
        HIPCHK(hipGraphLaunch(b->exec, b->stream));
    } else {
        const int erc = fp64 ? batch_enqueue<double>(b, nsteps) : batch_enqueue<float>(b, nsteps);
        if (erc) return erc;
    }
    return PPML_OK;
}

int ppml_batch_sync(ppml_batch *b)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    HIPCHK(hipStreamSynchronize(b->stream));
    for (int s = 0; s < b->capacity; s++) {
        ppml_grid *g = b->slots[s];
        if (!g) continue;
        int err = 0;
        HIPCHK(hipMemcpy(&err, &g->ctrl->err, sizeof(int), hipMemcpyDeviceToHost));
        if (err) return fail(PPML_ENONFINITE, "grid in slot %d produced a non-physical or non-finite value", s);
    }
    return PPML_OK;
}

int ppml_batch_info(ppml_batch *b, int32_t *count, size_t *bytes_in_use)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    int n = 0;
    for (ppml_grid *x : b->slots) n += x ? 1 : 0;
    if (count) *count = n;
    if (bytes_in_use) *bytes_in_use = b->in_use;
    return PPML_OK;
}

int ppml_batch_set_tile(ppml_batch *b, int32_t ndim, int32_t variant)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    if (ndim < 1 || ndim > 3) return fail(PPML_EINVAL, "ndim must be 1, 2 or 3 (got %d)", ndim);
    if (variant < 0 || variant >= NTILE[ndim]) return fail(PPML_EINVAL, "tile %d out of range", variant);
    for (ppml_grid *x : b->slots)
        if (x && x->d.ndim == ndim) return fail(PPML_ESTATE, "grids of ndim %d are admitted", ndim);
    b->tile[ndim] = variant;
    b->dirty = true;
    return PPML_OK;
}

int ppml_batch_destroy(ppml_batch *b)
{
    if (!b) return fail(PPML_EINVAL, "batch is NULL");
    (void)hipStreamSynchronize(b->stream);
    batch_drop_graph(b);
    for (ppml_grid *g : b->slots)
        if (g) g->in_batch = false;
    (void)hipFree(b->d_ents);
    (void)hipFree(b->d_steps);
    (void)hipHostFree(b->h_ents);
    (void)hipHostFree(b->h_steps);
    for (int nd = 0; nd <= 3; nd++) {
        (void)hipStreamDestroy(b->side[nd]);
        (void)hipEventDestroy(b->ev_join[nd]);
    }
    (void)hipEventDestroy(b->ev_fork);
    delete b;
    return PPML_OK;
}

}  // extern "C"
