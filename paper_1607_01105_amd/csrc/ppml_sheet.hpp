// ppml_sheet.hpp -- the two stage kernels of 2-D grids on gfx950: a wave per
// strip of a few rows, without LDS tiles or barriers.
//
// A wave owns up to SHEET_W = 58 columns of R rows, one lane per column and three
// halo lanes on each side.  It loads the R + 6 rows its update reads at once
// (one memory latency), takes the neighbours along x over DPP wave shifts and
// those along y from its own registers, and finishes its rows in straight-line
// code.  A row alone (R = 1) builds five slopes, four interface values and three
// profiles per field along y where R rows share them, so R follows the size of
// the launch: as many waves as the SIMDs need first, then more rows per wave
// (sheet_rows).  What bounds it: launch and memory latency on small grids, the
// vector instructions on large ones.
#pragma once

#include "ppml_line.hpp"

namespace ppml {

constexpr int SHEET_W = 64 - 2 * GH;
constexpr int SHEET_THREADS = 256;
// Strip and chunk of this wave; false past the last one.  Chunks run fastest,
// so that the waves of a work group, and neighbouring groups, share halo rows.
__device__ __forceinline__ bool sheet_strip(const GridParams &gp, int group, int &bx, int &by)
{
    const int t = group * (SHEET_THREADS / 64) + wave_id();
    bx = t / gp.tiles[1];
    by = t - bx * gp.tiles[1];
    return bx < gp.tiles[0];
}

// Columns per strip: the grid's, split evenly (a last strip of eight columns or
// fewer cost a whole launch 2 us, 64x64 FP32: 12.4 us per step instead of 9.4).
__device__ __forceinline__ int sheet_width(const GridParams &gp) { return (gp.n[0] + gp.tiles[0] - 1) / gp.tiles[0]; }

// Row loader: the boundary-mapped column of the lane and the ghost rules that
// stay the same along the march.
template <typename T> struct SheetColumn {
    const T *f[5];  // uniform
    int cx;         // mapped column
    int nx;
    bool flipx;
    int facex;      // inflow face of a ghost column, or -1
};

template <typename T> __device__ __forceinline__ SheetColumn<T> sheet_column(const GridParams &gp, const T *U, int c)
{
    SheetColumn<T> s;
#pragma unroll
    for (int q = 0; q < 5; q++) s.f[q] = U + (size_t)q * (size_t)gp.ncell;
    int fl;
    s.cx = map_index(c, gp.n[0], gp.bc_lo[0], gp.bc_hi[0], fl);
    s.nx = gp.n[0];
    s.flipx = fl != 0;
    s.facex = gp.any_inflow ? inflow_face(c, gp.n[0], gp.bc_lo[0], gp.bc_hi[0], 0) : -1;
    return s;
}

// Row j of the lane's column, as it is stored: the fields of the mask's low
// five bits, or, where `full`, of its next five.
template <typename T, int MASK>
__device__ __forceinline__ void sheet_load(const GridParams &gp, const SheetColumn<T> &s, int j, bool full, T (&v)[5])
{
    int fl;
    const int off = map_index(j, gp.n[1], gp.bc_lo[1], gp.bc_hi[1], fl) * s.nx + s.cx;
#pragma unroll
    for (int q = 0; q < 5; q++)
        v[q] = ((full ? MASK >> 5 : MASK) >> q) & 1 ? s.f[q][off] : T(0);
}

// ... and with the ghost rules applied: mirrored momenta, inflow states (a y
// face overrides x; after an x face only a y reflection applies).
template <typename T>
__device__ __forceinline__ void sheet_ghosts(const GridParams &gp, const Ctrl *ctrl, const SheetColumn<T> &s, int j, T (&v)[5])
{
    const bool flipy = (j < 0 && gp.bc_lo[1] == BC_REFLECT) || (j >= gp.n[1] && gp.bc_hi[1] == BC_REFLECT);
    if (s.flipx) v[1] = -v[1];
    if (flipy) v[2] = -v[2];
    if (gp.any_inflow) {
        const int fy = inflow_face(j, gp.n[1], gp.bc_lo[1], gp.bc_hi[1], 1);
        const int face = fy >= 0 ? fy : s.facex;
        if (face >= 0) {
#pragma unroll
            for (int q = 0; q < 5; q++) v[q] = inflow_value<T>(ctrl, face, inflow_component<2>(q));
            if (fy < 0 && flipy) v[2] = -v[2];
        }
    }
}

// Column i = 0 .. R + 5 (rows j0 - 3 .. j0 + R + 2) of a quantity: its profiles
// of the rows i = 2 .. R + 3 (pr[i - 2]).
template <int R, typename T>
__device__ __forceinline__ void sheet_profiles(int first_order, const T (&q)[R + 6], Profile<T> (&pr)[R + 2])
{
    T sl[R + 4], iv[R + 3];  // slopes of i = 1 .. R + 4, values between i + 1 and i + 2
#pragma unroll
    for (int i = 0; i < R + 4; i++) sl[i] = limited_slope(q[i], q[i + 1], q[i + 2]);
#pragma unroll
    for (int i = 0; i < R + 3; i++) iv[i] = interface_value(q[i + 1], q[i + 2], sl[i], sl[i + 1]);
#pragma unroll
    for (int i = 0; i < R + 2; i++) pr[i] = profile(first_order, q[i + 2], iv[i], iv[i + 1]);
}

// Eulerian stage (Sec. 2.1-2.2) of the wave's strip.
template <typename T, int R>
__device__ __forceinline__ void euler_sheet(const T *__restrict__ U, T *__restrict__ Wst, const GridParams &gp, Ctrl *ctrl,
                                            const int group, const bool lead)
{
    // the state's loads first: they do not wait for the control block's
    int bx, by;
    const bool strip = sheet_strip(gp, group, bx, by);
    const int ln = threadIdx.x & 63;
    const int width = sheet_width(gp);
    const int c = bx * width - GH + ln;
    const bool out = ln >= GH && ln < GH + width && c < gp.n[0];
    const SheetColumn<T> col = sheet_column(gp, U, c);
    const int j0 = by * R;
    T u[R + 6][5];
    if (strip) {
#pragma unroll
        for (int i = 0; i < R + 6; i++)
            sheet_load<T, 0x15 | (0x1F << 5)>(gp, col, j0 - GH + i, i >= GH && i < R + GH, u[i]);
    }
    const double tau_d = uniform(compute_tau(ctrl, gp));
    if (lead) publish_step(ctrl, gp, tau_d);
    if (!(tau_d > 0.0) || !strip) return;
    const T gam = uniform((T)gp.gs), gm1 = uniform((T)gp.pb), prho = uniform((T)gp.pa), tau = uniform((T)tau_d);
    const T hx = uniform((T)gp.h[0]), hy = uniform((T)gp.h[1]);
    const T ihx = uniform((T)gp.inv_h[0]), ihy = uniform((T)gp.inv_h[1]);
    const T tohx = uniform((T)(tau_d * gp.inv_h[0])), tohy = uniform((T)(tau_d * gp.inv_h[1]));
    (void)hx; (void)hy; (void)ihx; (void)ihy; (void)tohx; (void)tohy;
#pragma unroll
    for (int i = 0; i < R + 6; i++) sheet_ghosts(gp, ctrl, col, j0 - GH + i, u[i]);

    // y direction: Riemann problems at the faces below rows 0 .. R
    T v[R + 6], p[R + 6], s[R + 2];
    Profile<T> pv[R + 2], pp[R + 2];
    VP<T> y[R + 1];
#pragma unroll
    for (int i = 0; i < R + 6; i++) {
#ifdef PPML_EXACT
        v[i] = u[i][2] / u[i][0];
#else
        v[i] = u[i][2] * fast_rcp(u[i][0]);
#endif
        p[i] = prho * u[i][0] + gm1 * u[i][4];
        if (i >= 2 && i < R + 4) s[i - 2] = dsqrt(u[i][0]);
    }
    sheet_profiles<R>(gp.first_order, v, pv);
    sheet_profiles<R>(gp.first_order, p, pp);
#pragma unroll
    for (int i = 0; i <= R; i++)
        y[i] = riemann(gp.first_order, s[i], s[i + 1], u[i + 2][0] * s[i], u[i + 3][0] * s[i + 1], p[i + 2] * s[i],
                       p[i + 3] * s[i + 1], pv[i], pv[i + 1], pp[i], pp[i + 1], gam, tau, hy, tohy);
#pragma unroll
    for (int r = 0; r < R; r++) {
        // x direction of row r: the face between the previous lane's cell and this one
        const T(&w0)[5] = u[r + GH];
        const T rho = w0[0], pr = p[r + GH], sr = s[r + 1];
#ifdef PPML_EXACT
        const T vx = w0[1] / rho;
#else
        const T vx = w0[1] * fast_rcp(rho);
#endif
        const T r32 = rho * sr, ps = pr * sr;
        const Profile<T> xv = line_profile(gp.first_order, lane_prev(vx), vx, lane_next(vx));
        const Profile<T> xp = line_profile(gp.first_order, lane_prev(pr), pr, lane_next(pr));
        const VP<T> a = riemann(gp.first_order, lane_prev(sr), sr, lane_prev(r32), r32, lane_prev(ps), ps, lane_prev(xv), xv,
                                lane_prev(xp), xp, gam, tau, hx, tohx);
        const VP<T> b{lane_next(a.V), lane_next(a.P)};
        if (out && j0 + r < gp.n[1]) {
            const VP<T> &lo = y[r], &hi = y[r + 1];
            const T DPx = PPML_DIV(b.P - a.P, hx, ihx);
            T sPV = PPML_DIV(b.P * b.V - a.P * a.V, hx, ihx);
            T sV = PPML_DIV(b.V - a.V, hx, ihx);
            const T DPy = PPML_DIV(hi.P - lo.P, hy, ihy);
            sPV = sPV + PPML_DIV(hi.P * hi.V - lo.P * lo.V, hy, ihy);
            sV = sV + PPML_DIV(hi.V - lo.V, hy, ihy);
            const T e = w0[4];
            T w[5];
            w[0] = rho;
            w[1] = w0[1] - tau * DPx;
            w[2] = w0[2] - tau * DPy;
            w[3] = w0[3] - tau * sPV;
            w[4] = e - ((tau * gm1) * e) * sV;
            if (gp.potential != POT_NONE) {
                double g[3];
                potential_grad<0>(gp, c, j0 + r, 0, g);
                const double work = (double)w0[1] * g[0] + (double)w0[2] * g[1];
                const double tr = tau_d * (double)rho;
                w[1] = (T)((double)w[1] - tr * g[0]);
                w[2] = (T)((double)w[2] - tr * g[1]);
                w[3] = (T)((double)w[3] - tau_d * work);
            }
            const int o = (j0 + r) * gp.n[0] + c;
#pragma unroll
            for (int q = 0; q < 5; q++) (Wst + (size_t)q * (size_t)gp.ncell)[o] = w[q];
        }
    }
}

// Lagrangian stage (Sec. 2.3), energy correction and CFL maxima of the wave's
// strip.
template <typename T, int R>
__device__ __forceinline__ void lagr_sheet(const T *__restrict__ Wst, T *__restrict__ U, const GridParams &gp, Ctrl *ctrl,
                                           const int group, const bool lead, const int slot_i, T *red)
{
    constexpr int NF = 5;
    // the loads first, as in the Eulerian kernel
    int bx, by;
    const bool strip = sheet_strip(gp, group, bx, by);
    const int ln = threadIdx.x & 63;
    const int width = sheet_width(gp);
    const int c = bx * width - GH + ln;
    const bool out = ln >= GH && ln < GH + width && c < gp.n[0];
    const SheetColumn<T> col = sheet_column(gp, Wst, c);
    const int j0 = by * R;
    T w[R + 6][NF];
    if (strip) {
#pragma unroll
        for (int i = 0; i < R + 6; i++) sheet_load<T, 0x3FF>(gp, col, j0 - GH + i, true, w[i]);
    }
    const double tau_d = ctrl->tau;
    if (!(tau_d > 0.0)) return;
    const int sl = ctrl->slot_l;
    if (lead) advance_step(ctrl, tau_d, sl);
    T vmax = T(0), cmax = T(0);
    if (strip) {
        const T gam = uniform((T)gp.gs), gm1 = uniform((T)gp.pb), prho = uniform((T)gp.pa), tau = uniform((T)tau_d);
        const T hx = uniform((T)gp.h[0]), hy = uniform((T)gp.h[1]);
        const T tohx = uniform((T)(tau_d * gp.inv_h[0])), tohy = uniform((T)(tau_d * gp.inv_h[1]));
        (void)hx; (void)hy; (void)tohx; (void)tohy; (void)tau;
        const double thr = uniform(gp.vacuum_ratio * ctrl->rho_mean0);
#pragma unroll
        for (int i = 0; i < R + 6; i++) sheet_ghosts(gp, ctrl, col, j0 - GH + i, w[i]);

        // rows -1 .. R: v_x, transverse v_y, sqrt(rho)
        T ux[R + 2], vt[R + 2], s[R + 2];
#pragma unroll
        for (int i = 0; i < R + 2; i++) {
            const T(&q)[NF] = w[i + 2];
#ifdef PPML_EXACT
            ux[i] = q[1] / q[0];
            const T uy = q[2] / q[0];
#else
            const T ir = fast_rcp(q[0]);
            ux[i] = q[1] * ir;
            const T uy = q[2] * ir;
#endif
            vt[i] = tmpl3(lane_next(uy), lane_prev(uy), uy);
            s[i] = dsqrt(q[0]);
        }
        // velocities and flux weights of the faces: below rows 0 .. R along y;
        // along x a lane forms its cell's flux through its right face, used
        // where the flow there is to the right, and through its left face,
        // used where it is to the left
        T vy[R + 1], vx[R];
        bool up[R + 1], left[R];
#ifdef PPML_EXACT
        T zy[R + 1], zx[R], vr[R], zr[R];
#else
        FaceW<T> fy[R + 1], fw[R], fr[R];
#endif
#pragma unroll
        for (int i = 0; i <= R; i++) {
            vy[i] = interface_velocity(vt[i], s[i], vt[i + 1], s[i + 1]);
            up[i] = vy[i] >= T(0);
#ifdef PPML_EXACT
            zy[i] = dabs(vy[i]) * tau / hy;
#else
            fy[i] = face_weights(gp.first_order, up[i], vy[i] * tohy);
#endif
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            const T t = tmpl3(ux[r + 2], ux[r], ux[r + 1]);
            vx[r] = interface_velocity(lane_prev(t), lane_prev(s[r + 1]), t, s[r + 1]);
            left[r] = vx[r] >= T(0);
#ifdef PPML_EXACT
            zx[r] = dabs(vx[r]) * tau / hx;
            vr[r] = lane_next(vx[r]);
            zr[r] = lane_next(zx[r]);
#else
            fw[r] = face_weights(gp.first_order, left[r], vx[r] * tohx);
            fr[r] = FaceW<T>{lane_next(fw[r].vs), lane_next(fw[r].a), lane_next(fw[r].b)};
#endif
        }
        T fn[R][NF];
#pragma unroll
        for (int f = 0; f < NF; f++) {
            T q[R + 6], F[R + 1];
            Profile<T> pr[R + 2];
#pragma unroll
            for (int i = 0; i < R + 6; i++) q[i] = w[i][f];
            sheet_profiles<R>(gp.first_order, q, pr);
#pragma unroll
            for (int i = 0; i <= R; i++) {
                const Profile<T> &a = pr[i], &b = pr[i + 1];
#ifdef PPML_EXACT
                F[i] = upwind_flux(vy[i], zy[i], a, b);
#else
                F[i] = face_flux(fy[i], Profile<T>{up[i] ? a.dl : b.dl, up[i] ? a.dr : b.dr, up[i] ? a.c : b.c});
#endif
            }
#pragma unroll
            for (int r = 0; r < R; r++) {
                const T q0 = q[r + GH];
                const Profile<T> x = line_profile(gp.first_order, lane_prev(q0), q0, lane_next(q0));
#ifdef PPML_EXACT
                const T Fm = lane_prev(vr[r] * avg_left(x.L, x.R, x.Q6, zr[r]));
                const T Fl = vx[r] * avg_right(x.L, x.R, x.Q6, zx[r]);
                const T Fx = left[r] ? Fm : Fl;
                T a = (lane_next(Fx) - Fx) / hx;
                a = a + (F[r + 1] - F[r]) / hy;
                fn[r][f] = q0 - tau * a;
#else
                const T Fm = lane_prev(face_flux(fr[r], x));
                const T Fl = face_flux(fw[r], x);
                const T Fx = left[r] ? Fm : Fl;
                fn[r][f] = q0 - ((lane_next(Fx) - Fx) + (F[r + 1] - F[r]));
#endif
            }
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (!(out && j0 + r < gp.n[1])) continue;
            energy_correction<T, 2>(fn[r], thr);
            const int o = (j0 + r) * gp.n[0] + c;
#pragma unroll
            for (int f = 0; f < NF; f++) (U + (size_t)f * (size_t)gp.ncell)[o] = fn[r][f];
            T v, cs;
            cell_speeds<T, 2>(fn[r][0], fn[r][1], fn[r][2], T(0), fn[r][4], prho, gam, gm1, v, cs);
            if (bad_cell(fn[r][0], fn[r][3], fn[r][4], v, cs)) atomicOr(&ctrl->err, 1);
            vmax = vmax > v ? vmax : v;
            cmax = cmax > cs ? cmax : cs;
        }
    }
    publish_max<SHEET_THREADS>(ctrl, gp.mslots, sl ^ 1, slot_i, vmax, cmax, red);
}

// Work group of a solo launch, each XCD a contiguous range (see block_tile).
__device__ __forceinline__ int sheet_group(int groups)
{
    const int b = blockIdx.x, x = b & 7, q = groups >> 3, r = groups & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

template <typename T, int R>
__global__ __launch_bounds__(SHEET_THREADS) void k_euler_sheet(const T *__restrict__ U, T *__restrict__ Wst, GridParams gp,
                                                               Ctrl *ctrl)
{
    euler_sheet<T, R>(U, Wst, gp, ctrl, sheet_group((int)gridDim.x), blockIdx.x == 0);
}

// Two waves per SIMD (<= 256 registers, the accumulation registers included) for
// the FP64 kernels of several rows, which take twice that otherwise.
template <typename T, int R> constexpr int sheet_waves() { return sizeof(T) == 8 && R > 1 ? 2 : 1; }

template <typename T, int R>
__global__ __launch_bounds__(SHEET_THREADS) __attribute__((amdgpu_waves_per_eu(sheet_waves<T, R>()))) void k_lagr_sheet(const T *__restrict__ Wst, T *__restrict__ U, GridParams gp,
                                                              Ctrl *ctrl)
{
    __shared__ T red[2 * SHEET_THREADS / 64];
    lagr_sheet<T, R>(Wst, U, gp, ctrl, sheet_group((int)gridDim.x), blockIdx.x == 0 && threadIdx.x == 0,
                  (int)(blockIdx.x % gp.mslots), red);
}

template <typename T, int R>
__global__ __launch_bounds__(SHEET_THREADS) void k_euler_sheet_batch(const BatchEntry *__restrict__ ents,
                                                                     const int *__restrict__ first, int ne)
{
    // ahead of the waves of the line kernel that shares the chip (its grids'
    // steps are far shorter than this chain's)
    __builtin_amdgcn_s_setprio(2);
    const BatchEntry *e = ents + batch_entry(first, ne, blockIdx.x);
    const int L = blockIdx.x - e->tile0;
    euler_sheet<T, R>((const T *)e->state, (T *)e->half, e->gp, e->ctrl, L, L == 0);
}

template <typename T, int R>
__global__ __launch_bounds__(SHEET_THREADS) __attribute__((amdgpu_waves_per_eu(sheet_waves<T, R>()))) void k_lagr_sheet_batch(
    const BatchEntry *__restrict__ ents, const int *__restrict__ first, int ne)
{
    __shared__ T red[2 * SHEET_THREADS / 64];
    __builtin_amdgcn_s_setprio(2);
    const BatchEntry *e = ents + batch_entry(first, ne, blockIdx.x);
    const int L = blockIdx.x - e->tile0;
    lagr_sheet<T, R>((const T *)e->half, (T *)e->state, e->gp, e->ctrl, L, L == 0 && threadIdx.x == 0, L % e->gp.mslots, red);
}

}  // namespace ppml
