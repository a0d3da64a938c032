// ppml_brick.hpp -- the two stage kernels of small 3-D grids on gfx950: a wave
// per row, without LDS tiles, barriers or a march along z.
//
// The marching kernels (ppml_kernels.hpp) build each z parabola once, but a
// chunk of planes is a chain: six start-up planes and then every plane's
// phases, 2 to 3 us each, however few work groups there are.  Here a wave
// finishes up to SHEET_W columns of one row of one plane in straight-line code:
// it loads the row's neighbours in y and z at once, takes those in x over DPP
// wave shifts, and builds five slopes, four interface values and three profiles
// per field and axis along y and z where the march shares them: 1850 and 1010
// vector instructions per wave in the two FP32 stages, where the march issues
// 1230 and 540 per 64 cells at 100^3 (start-up included) but waits for its
// phases.  Used where the waves are few (brick_grid): what bounds it there is
// launch and memory latency.
#pragma once

#include "ppml_sheet.hpp"

namespace ppml {

// The lane's boundary-mapped column.
template <typename T> struct Brick {
    const T *U;     // field 0 (uniform)
    long long N;
    int cx;
    bool flipx;     // a mirrored ghost column
};

// A row of cells (uniform): its offset, and whether it is a mirrored ghost.
struct BrickRow {
    int off;
    bool flipy, flipz;
};

// Strip of this wave: width of the strips, first column - GH + lane, row, plane.
__device__ __forceinline__ bool brick_strip(const GridParams &gp, int group, int &width, int &c, int &j, int &k)
{
    const int t = __builtin_amdgcn_readfirstlane(group * (SHEET_THREADS / 64) + wave_id());
    const int r = t / gp.n[1], bx = r / gp.n[2];
    j = t - r * gp.n[1];
    k = r - bx * gp.n[2];
    width = sheet_width(gp);
    c = bx * width - GH + (int)(threadIdx.x & 63);
    return bx < gp.tiles[0];
}

template <typename T> __device__ __forceinline__ Brick<T> brick_column(const GridParams &gp, const T *U, int c)
{
    Brick<T> b;
    int fl;
    b.U = U;
    b.N = gp.ncell;
    b.cx = map_index(c, gp.n[0], gp.bc_lo[0], gp.bc_hi[0], fl);
    b.flipx = fl != 0;
    return b;
}

__device__ __forceinline__ BrickRow brick_row(const GridParams &gp, int j, int k)
{
    BrickRow r;
    int fy, fz;
    const int jj = map_index(j, gp.n[1], gp.bc_lo[1], gp.bc_hi[1], fy);
    const int kk = map_index(k, gp.n[2], gp.bc_lo[2], gp.bc_hi[2], fz);
    r.off = (kk * gp.n[1] + jj) * gp.n[0];
    r.flipy = fy != 0;
    r.flipz = fz != 0;
    return r;
}

// The rows i = 0 .. 6 (offsets -3 .. 3) of the cell's column along y and z.
struct BrickRows {
    BrickRow y[7], z[7];
};
__device__ __forceinline__ BrickRows brick_rows(const GridParams &gp, int j, int k)
{
    BrickRows r;
#pragma unroll
    for (int i = 0; i < 7; i++) {
        r.y[i] = brick_row(gp, j - GH + i, k);
        r.z[i] = brick_row(gp, j, k - GH + i);
    }
    return r;
}

// Field f of the lane's cell in a row (mirrored ghosts: the momentum normal to
// the wall negated).
template <typename T> __device__ __forceinline__ T brick_at(const Brick<T> &b, const BrickRow &r, int f)
{
    const T v = (b.U + (size_t)f * (size_t)b.N)[r.off + b.cx];
    const bool flip = f == 1 ? b.flipx : (f == 2 ? r.flipy : (f == 3 && r.flipz));
    return flip ? -v : v;
}

// Eulerian stage (Sec. 2.1-2.2).  XF as in euler_body.
template <typename T, int XF>
__device__ __forceinline__ void euler_brick(const T *__restrict__ U, T *__restrict__ Wst, const GridParams &gp, Ctrl *ctrl,
                                            const int group, const bool lead)
{
    int width, c, j, k;
    const bool strip = brick_strip(gp, group, width, c, j, k);
    const double tau_d = uniform(compute_tau(ctrl, gp));
    if (lead) publish_step(ctrl, gp, tau_d);
    if (!(tau_d > 0.0) || !strip) return;
    const T gam = uniform((T)gp.gs), gm1 = uniform((T)gp.pb), prho = uniform((T)gp.pa), tau = uniform((T)tau_d);
    const T h[3] = {uniform((T)gp.h[0]), uniform((T)gp.h[1]), uniform((T)gp.h[2])};
    const T ih[3] = {uniform((T)gp.inv_h[0]), uniform((T)gp.inv_h[1]), uniform((T)gp.inv_h[2])};
    const T toh[3] = {uniform((T)(tau_d * gp.inv_h[0])), uniform((T)(tau_d * gp.inv_h[1])),
                      uniform((T)(tau_d * gp.inv_h[2]))};
    (void)h; (void)ih; (void)toh;
    const int ln = threadIdx.x & 63;
    const bool out = ln >= GH && ln < GH + width && c < gp.n[0];
    const Brick<T> b = brick_column(gp, U, c);
    const BrickRows rows = brick_rows(gp, j, k);
    T u0[6];
#pragma unroll
    for (int f = 0; f < 6; f++) u0[f] = brick_at(b, rows.y[GH], f);

    // y and z: Riemann problems at the faces below and above the cell
    VP<T> lo[2], hi[2];
#pragma unroll
    for (int a = 1; a <= 2; a++) {
        T rho[7], v[7], p[7], s[3];
        Profile<T> pv[3], pp[3];
#pragma unroll
        for (int i = 0; i < 7; i++) {
            const BrickRow &r = a == 1 ? rows.y[i] : rows.z[i];
            rho[i] = i == GH ? u0[0] : brick_at(b, r, 0);
            const T m = i == GH ? u0[a + 1] : brick_at(b, r, a + 1);
            const T e = i == GH ? u0[5] : brick_at(b, r, 5);
#ifdef PPML_EXACT
            v[i] = m / rho[i];
#else
            v[i] = m * fast_rcp(rho[i]);
#endif
            p[i] = prho * rho[i] + gm1 * e;
            if (i >= 2 && i <= 4) s[i - 2] = dsqrt(rho[i]);
        }
        sheet_profiles<1>(gp.first_order, v, pv);
        sheet_profiles<1>(gp.first_order, p, pp);
        VP<T> y[2];
#pragma unroll
        for (int i = 0; i < 2; i++)
            y[i] = riemann(gp.first_order, s[i], s[i + 1], rho[i + 2] * s[i], rho[i + 3] * s[i + 1], p[i + 2] * s[i],
                           p[i + 3] * s[i + 1], pv[i], pv[i + 1], pp[i], pp[i + 1], gam, tau, h[a], toh[a]);
        lo[a - 1] = y[0];
        hi[a - 1] = y[1];
    }
    // x: the face between the previous lane's cell and this one
    const T rho = u0[0], e = u0[5];
#ifdef PPML_EXACT
    const T vx = u0[1] / rho;
#else
    const T vx = u0[1] * fast_rcp(rho);
#endif
    const T pr = prho * rho + gm1 * e;
    const T sr = dsqrt(rho), r32 = rho * sr, ps = pr * sr;
    const Profile<T> xv = line_profile(gp.first_order, lane_prev(vx), vx, lane_next(vx));
    const Profile<T> xp = line_profile(gp.first_order, lane_prev(pr), pr, lane_next(pr));
    const VP<T> xa = riemann(gp.first_order, lane_prev(sr), sr, lane_prev(r32), r32, lane_prev(ps), ps, lane_prev(xv), xv,
                             lane_prev(xp), xp, gam, tau, h[0], toh[0]);
    const VP<T> xb{lane_next(xa.V), lane_next(xa.P)};
    if (!out) return;
    const T DPx = PPML_DIV(xb.P - xa.P, h[0], ih[0]);
    T sPV = PPML_DIV(xb.P * xb.V - xa.P * xa.V, h[0], ih[0]);
    T sV = PPML_DIV(xb.V - xa.V, h[0], ih[0]);
    const T DPy = PPML_DIV(hi[0].P - lo[0].P, h[1], ih[1]);
    sPV = sPV + PPML_DIV(hi[0].P * hi[0].V - lo[0].P * lo[0].V, h[1], ih[1]);
    sV = sV + PPML_DIV(hi[0].V - lo[0].V, h[1], ih[1]);
    const T DPz = PPML_DIV(hi[1].P - lo[1].P, h[2], ih[2]);
    const T DPVz = PPML_DIV(hi[1].P * hi[1].V - lo[1].P * lo[1].V, h[2], ih[2]);
    const T DVz = PPML_DIV(hi[1].V - lo[1].V, h[2], ih[2]);
    sPV = sPV + DPVz;
    sV = sV + DVz;
    T w[6];
    w[0] = rho;
    w[1] = u0[1] - tau * DPx;
    w[2] = u0[2] - tau * DPy;
    w[3] = u0[3] - tau * DPz;
    w[4] = u0[4] - tau * sPV;
    w[5] = e - ((tau * gm1) * e) * sV;
    if (XF != 0 || gp.potential != POT_NONE) {
        double g[3];
        potential_grad<XF>(gp, c, j, k, g);
        if constexpr (XF != 0)
            if (gp.self_grav) self_gravity_grad<T>(gp, c, j, k, g);
        const double work = (double)u0[1] * g[0] + (double)u0[2] * g[1] + (double)u0[3] * g[2];
        const double tr = tau_d * (double)rho;
#pragma unroll
        for (int a = 0; a < 3; a++) w[1 + a] = (T)((double)w[1 + a] - tr * g[a]);
        w[4] = (T)((double)w[4] - tau_d * work);
    }
    const int o = rows.y[GH].off + c;
#pragma unroll
    for (int f = 0; f < 6; f++) (Wst + (size_t)f * (size_t)gp.ncell)[o] = w[f];
}

// Lagrangian stage (Sec. 2.3), energy correction and CFL maxima.
template <typename T>
__device__ __forceinline__ void lagr_brick(const T *__restrict__ Wst, T *__restrict__ U, const GridParams &gp, Ctrl *ctrl,
                                           const int group, const bool lead, const int slot_i, T *red)
{
    constexpr int NF = 6;
    const double tau_d = ctrl->tau;
    if (!(tau_d > 0.0)) return;
    const int sl = ctrl->slot_l;
    if (lead) advance_step(ctrl, tau_d, sl);
    T vmax = T(0), cmax = T(0);
    int width, c, j, k;
    if (brick_strip(gp, group, width, c, j, k)) {
        const T gam = uniform((T)gp.gs), gm1 = uniform((T)gp.pb), prho = uniform((T)gp.pa), tau = uniform((T)tau_d);
        const T h[3] = {uniform((T)gp.h[0]), uniform((T)gp.h[1]), uniform((T)gp.h[2])};
        const T toh[3] = {uniform((T)(tau_d * gp.inv_h[0])), uniform((T)(tau_d * gp.inv_h[1])),
                          uniform((T)(tau_d * gp.inv_h[2]))};
        (void)h; (void)toh; (void)tau;
        const double thr = uniform(gp.vacuum_ratio * ctrl->rho_mean0);
        const int ln = threadIdx.x & 63;
        const bool out = ln >= GH && ln < GH + width && c < gp.n[0];
        const Brick<T> b = brick_column(gp, Wst, c);
        const BrickRows rows = brick_rows(gp, j, k);

        // velocities of the nine rows around the cell's, [z][y], and sqrt(rho)
        // of the rows that share a face with it
        T ux[3][3], uy[3][3], uz[3][3], s0 = 0, sy[2], sz[2];
#pragma unroll
        for (int z = 0; z < 3; z++)
#pragma unroll
            for (int y = 0; y < 3; y++) {
                const BrickRow r = z == 1 ? rows.y[GH - 1 + y] : (y == 1 ? rows.z[GH - 1 + z] : brick_row(gp, j + y - 1, k + z - 1));
                const T rho = brick_at(b, r, 0);
                const T mx = brick_at(b, r, 1), my = brick_at(b, r, 2), mz = brick_at(b, r, 3);
#ifdef PPML_EXACT
                ux[z][y] = mx / rho;
                uy[z][y] = my / rho;
                uz[z][y] = mz / rho;
#else
                const T ir = fast_rcp(rho);
                ux[z][y] = mx * ir;
                uy[z][y] = my * ir;
                uz[z][y] = mz * ir;
#endif
                if (z == 1 && y == 1) s0 = dsqrt(rho);
                if (z == 1 && y != 1) sy[y / 2] = dsqrt(rho);
                if (z != 1 && y == 1) sz[z / 2] = dsqrt(rho);
            }
        // transverse velocities (Sec. 2.3) and the velocities of the faces: x
        // the one to the previous lane; y and z below and above the cell
        T v[5];  // x, y low, y high, z low, z high
        {
            const T t = tmpl9(ux[2][2], ux[0][2], ux[2][0], ux[0][0], ux[1][2], ux[1][0], ux[2][1], ux[0][1], ux[1][1]);
            v[0] = interface_velocity(lane_prev(t), lane_prev(s0), t, s0);
            T ty[3], tz[3];
#pragma unroll
            for (int y = 0; y < 3; y++)
                ty[y] = tmpl9(lane_next(uy[2][y]), lane_next(uy[0][y]), lane_prev(uy[2][y]), lane_prev(uy[0][y]),
                              lane_next(uy[1][y]), lane_prev(uy[1][y]), uy[2][y], uy[0][y], uy[1][y]);
#pragma unroll
            for (int z = 0; z < 3; z++)
                tz[z] = tmpl9(lane_next(uz[z][2]), lane_next(uz[z][0]), lane_prev(uz[z][2]), lane_prev(uz[z][0]),
                              lane_next(uz[z][1]), lane_prev(uz[z][1]), uz[z][2], uz[z][0], uz[z][1]);
            v[1] = interface_velocity(ty[0], sy[0], ty[1], s0);
            v[2] = interface_velocity(ty[1], s0, ty[2], sy[1]);
            v[3] = interface_velocity(tz[0], sz[0], tz[1], s0);
            v[4] = interface_velocity(tz[1], s0, tz[2], sz[1]);
        }
        bool up[5];
#ifdef PPML_EXACT
        T zc[5];
#else
        FaceW<T> fw[5];
#endif
#pragma unroll
        for (int q = 0; q < 5; q++) {
            constexpr int axis[5] = {0, 1, 1, 2, 2};
            up[q] = v[q] >= T(0);
#ifdef PPML_EXACT
            zc[q] = dabs(v[q]) * tau / h[axis[q]];
#else
            fw[q] = face_weights(gp.first_order, up[q], v[q] * toh[axis[q]]);
#endif
        }
        // x: a lane forms its cell's flux through its right face, used where the
        // flow there is to the right, and through its left face, used where it
        // is to the left
#ifdef PPML_EXACT
        const T vr = lane_next(v[0]), zr = lane_next(zc[0]);
#else
        const FaceW<T> fr{lane_next(fw[0].vs), lane_next(fw[0].a), lane_next(fw[0].b)};
#endif
        T fn[NF];
#pragma unroll
        for (int f = 0; f < NF; f++) {
            const T q0 = brick_at(b, rows.y[GH], f);
            T D[2];  // y, z flux differences
#pragma unroll
            for (int a = 0; a < 2; a++) {
                T q[7], F[2];
                Profile<T> pr[3];
#pragma unroll
                for (int i = 0; i < 7; i++)
                    q[i] = i == GH ? q0 : brick_at(b, a == 0 ? rows.y[i] : rows.z[i], f);
                sheet_profiles<1>(gp.first_order, q, pr);
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const Profile<T> &l = pr[i], &r = pr[i + 1];
                    const int w = 1 + 2 * a + i;
#ifdef PPML_EXACT
                    F[i] = upwind_flux(v[w], zc[w], l, r);
#else
                    F[i] = face_flux(fw[w], Profile<T>{up[w] ? l.dl : r.dl, up[w] ? l.dr : r.dr, up[w] ? l.c : r.c});
#endif
                }
#ifdef PPML_EXACT
                D[a] = (F[1] - F[0]) / h[1 + a];
#else
                D[a] = F[1] - F[0];
#endif
            }
            const Profile<T> x = line_profile(gp.first_order, lane_prev(q0), q0, lane_next(q0));
#ifdef PPML_EXACT
            const T Fm = lane_prev(vr * avg_left(x.L, x.R, x.Q6, zr));
            const T Fl = v[0] * avg_right(x.L, x.R, x.Q6, zc[0]);
            const T Fx = up[0] ? Fm : Fl;
            T acc = (lane_next(Fx) - Fx) / h[0];
            acc = acc + D[0];
            acc = acc + D[1];
            fn[f] = q0 - tau * acc;
#else
            const T Fm = lane_prev(face_flux(fr, x));
            const T Fl = face_flux(fw[0], x);
            const T Fx = up[0] ? Fm : Fl;
            T acc = lane_next(Fx) - Fx;
            acc = acc + D[0];
            acc = acc + D[1];
            fn[f] = q0 - acc;
#endif
        }
        if (out) {
            energy_correction<T, 3>(fn, thr);
            const int o = rows.y[GH].off + c;
#pragma unroll
            for (int f = 0; f < NF; f++) (U + (size_t)f * (size_t)gp.ncell)[o] = fn[f];
            T sv, sc;
            cell_speeds<T, 3>(fn[0], fn[1], fn[2], fn[3], fn[5], prho, gam, gm1, sv, sc);
            if (bad_cell(fn[0], fn[4], fn[5], sv, sc)) atomicOr(&ctrl->err, 1);
            vmax = sv;
            cmax = sc;
        }
    }
    publish_max<SHEET_THREADS>(ctrl, gp.mslots, sl ^ 1, slot_i, vmax, cmax, red);
}

template <typename T, int XF>
__global__ __launch_bounds__(SHEET_THREADS) void k_euler_brick(const T *__restrict__ U, T *__restrict__ Wst, GridParams gp,
                                                               Ctrl *ctrl)
{
    euler_brick<T, XF>(U, Wst, gp, ctrl, sheet_group((int)gridDim.x), blockIdx.x == 0);
}

// At least two waves per SIMD (<= 256 registers) in FP64.
template <typename T>
__global__ __launch_bounds__(SHEET_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_lagr_brick(
    const T *__restrict__ Wst, T *__restrict__ U, GridParams gp, Ctrl *ctrl)
{
    __shared__ T red[2 * SHEET_THREADS / 64];
    lagr_brick<T>(Wst, U, gp, ctrl, sheet_group((int)gridDim.x), blockIdx.x == 0 && threadIdx.x == 0,
                  (int)(blockIdx.x % gp.mslots), red);
}

}  // namespace ppml
