// ppml_line.hpp -- 1-D grids of up to a few thousand cells on gfx950: every
// step of a call in one kernel, one work group per grid.
//
// A 1-D step is two tiny launches otherwise, each of which waits out a
// dispatch and a chain of memory latencies: 11.6 us per step at 512 cells FP64,
// whatever the grid's size.  Here the state stays in LDS, in two buffers that
// alternate from step to step, and a step costs one barrier.  A wave advances
// segments of LINE_W = 52 cells, one lane per cell and six halo lanes on each
// side (three per stage), through both stages in registers; what a lane needs
// of its neighbours comes over DPP wave shifts, so neither stage goes through
// LDS or waits for other waves.  The halo lanes repeat their neighbours' work
// (64/52 of it), with the same operations on the same values.  The time is
// then the vector instructions of one CU: it grows with the cells, and long
// grids stay with the two stage kernels, which spread over the chip.
#pragma once

#include "ppml_kernels.hpp"

namespace ppml {

constexpr int LINE_HALO = 6;
constexpr int LINE_W = 64 - 2 * LINE_HALO;
constexpr int LINE_THREADS = 1024;
// steps one launch takes at most (a long call is split, so that other streams
// get the CU in between)
constexpr int LINE_STEPS = 1024;

// LDS of a grid of n cells: two buffers of four fields and the waves' maxima.
template <typename T> constexpr size_t line_lds(long long n)
{
    return ((size_t)8 * n + 2 * 2 * (LINE_THREADS / 64)) * sizeof(T);
}

// The value of the previous (next) lane of the wave, 0 in the first (last),
// whose results no lane uses.  Every lane must be active.
template <int CTRL_> __device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL_, 0xF, 0xF, true);
}
template <int CTRL_> __device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float, dpp_mov<CTRL_>(__builtin_bit_cast(int, v)));
}
template <int CTRL_> __device__ __forceinline__ double dpp_mov(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_mov<CTRL_>((int)(unsigned)b), hi = (unsigned)dpp_mov<CTRL_>((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <typename T> __device__ __forceinline__ T lane_prev(T v) { return dpp_mov<0x138>(v); }  // wave_shr:1
template <typename T> __device__ __forceinline__ T lane_next(T v) { return dpp_mov<0x130>(v); }  // wave_shl:1

template <typename T> __device__ __forceinline__ Profile<T> lane_prev(const Profile<T> &p)
{
#ifdef PPML_EXACT
    return Parab<T>{lane_prev(p.L), lane_prev(p.R), lane_prev(p.Q6)};
#else
    return Jumps<T>{lane_prev(p.dl), lane_prev(p.dr), lane_prev(p.c)};
#endif
}

// Profile of the lane's cell from its value and its neighbours' (Appendix).
template <typename T> __device__ __forceinline__ Profile<T> line_profile(int first_order, T qm, T q0, T qp)
{
    const T d = limited_slope(qm, q0, qp);
    const T il = interface_value(qm, q0, lane_prev(d), d);
    return profile(first_order, q0, il, lane_next(il));
}

// Maximum over each row of 16 lanes, in its last lane (values >= 0).
template <typename T> __device__ __forceinline__ T line_max16(T v)
{
    v = dmax(v, dpp_mov<0x111>(v));
    v = dmax(v, dpp_mov<0x112>(v));
    v = dmax(v, dpp_mov<0x114>(v));
    return dmax(v, dpp_mov<0x118>(v));
}
// Maxima of a and b over the wave: a's in lane 31, b's in lane 63 of the
// result.  The halves are exchanged first, so that both take one reduction.
__device__ __forceinline__ void swap_halves(unsigned &a, unsigned &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ float line_max2(float a, float b)
{
    unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    swap_halves(x, y);
    float v = line_max16(dmax(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y)));
    return dmax(v, dpp_mov<0x142>(v));
}
__device__ __forceinline__ double line_max2(double a, double b)
{
    unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32), yl = (unsigned)y, yh = (unsigned)(y >> 32);
    swap_halves(xl, yl);
    swap_halves(xh, yh);
    x = ((unsigned long long)xh << 32) | xl;
    y = ((unsigned long long)yh << 32) | yl;
    double v = line_max16(dmax(__builtin_bit_cast(double, x), __builtin_bit_cast(double, y)));
    return dmax(v, dpp_mov<0x142>(v));
}
__device__ __forceinline__ float read_lane(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double read_lane(double v, int l)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Up to nlaunch steps of one grid by the whole work group (LINE_THREADS
// threads at most).  run_steps >= 0 starts a run of that many steps with the
// given parameters; otherwise the control block holds the run.  LDS: the two
// buffers lie in LDS; otherwise they are the state U and the stage output W in
// memory (for grids that LDS does not hold).
template <typename T, bool LDS>
__device__ __forceinline__ void line_body(T *U, T *W, const GridParams &gp, Ctrl *ctrl, long long run_steps,
                                          double run_dt, double run_t_stop, int nlaunch, T *lds)
{
    constexpr int NF = 4;
    const int n = gp.n[0];
    const int nseg = (n + LINE_W - 1) / LINE_W;
    const int wv = wave_id(), ln = threadIdx.x & 63, nw = (int)blockDim.x >> 6;
    T *const red = lds + (LDS ? 2 * NF * n : 0);  // [2 parities][|v|, c][waves]

    const int set = ctrl->slot_cur;
    long long steps_left = run_steps >= 0 ? run_steps : ctrl->steps_left;
    const double dt_fixed = run_steps >= 0 ? run_dt : ctrl->dt_fixed;
    const double t_stop = run_steps >= 0 ? run_t_stop : ctrl->t_stop;
    double t = ctrl->t, dt_last = 0.0;
    const double thr = uniform(gp.vacuum_ratio * ctrl->rho_mean0);
    double vm, cm;
    {
        unsigned long long vb, cb;
        fold_max(ctrl, gp.mslots, set, vb, cb);
        vm = __longlong_as_double((long long)vb);
        cm = __longlong_as_double((long long)cb);
    }
    const T gam = uniform((T)gp.gs);
    const T gm1 = uniform((T)gp.pb);
    const T prho = uniform((T)gp.pa);
    const T hx = uniform((T)gp.h[0]), ihx = uniform((T)gp.inv_h[0]);
    (void)hx;
    (void)ihx;

    if constexpr (LDS)
        for (int i = threadIdx.x; i < NF * n; i += blockDim.x) lds[i] = U[i];
    __syncthreads();

    // source cell, momentum flip and inflow face of the lane's cell in a
    // segment; the segment a wave takes first is the same on every step
    auto source = [&](int c, int &flip, int &face) {
        face = inflow_face(c, n, gp.bc_lo[0], gp.bc_hi[0], 0);
        return map_index(c, n, gp.bc_lo[0], gp.bc_hi[0], flip);
    };
    auto interior = [&](int seg) { return seg > 0 && (seg + 1) * LINE_W + LINE_HALO <= n; };
    int flip0, face0;
    const int cs0 = source(wv * LINE_W - LINE_HALO + ln, flip0, face0);

    int taken = 0;
    bool bad = false;
    while (taken < nlaunch && steps_left > 0) {
        double tau_d = dt_fixed > 0.0 ? dt_fixed : gp.cfl_hmin / (vm + cm);
        if (t_stop > 0.0) {
            const double rem = t_stop - t;
            if (rem <= 0.0) tau_d = 0.0;
            else if (tau_d > rem) tau_d = rem;
        }
        tau_d = uniform(tau_d);
        if (!(tau_d > 0.0)) break;
        const T tau = uniform((T)tau_d);
        const T tohx = uniform((T)(tau_d * gp.inv_h[0]));
        (void)tohx;
        const T *src;
        T *dst;
        if constexpr (LDS) {
            src = lds + (taken & 1) * NF * n;
            dst = lds + ((taken & 1) ^ 1) * NF * n;
        } else {
            src = taken & 1 ? W : U;
            dst = taken & 1 ? U : W;
        }
        T vmax = T(0), cmax = T(0);
#pragma unroll 1
        for (int seg = wv; seg < nseg; seg += nw) {
            const int c = seg * LINE_W - LINE_HALO + ln;
            const bool edge = !interior(seg);  // (uniform) the segment has ghost lanes
            int cs = c, flip = 0, face = -1;
            if (seg == wv) {
                cs = cs0;
                flip = flip0;
                face = face0;
            } else if (edge) {
                cs = source(c, flip, face);
            }
            T rho = src[cs], mx = src[n + cs], Et = src[2 * n + cs], e = src[3 * n + cs];
            if (flip) mx = -mx;
            if (gp.any_inflow && face >= 0) {
                rho = inflow_value<T>(ctrl, face, 0);
                mx = inflow_value<T>(ctrl, face, 1);
                Et = inflow_value<T>(ctrl, face, 4);
                e = inflow_value<T>(ctrl, face, 5);
            }

            // ---- Eulerian stage (Sec. 2.1-2.2): the face between the
            // previous lane's cell and this one ----
#ifdef PPML_EXACT
            const T v = mx / rho;
#else
            const T ir = fast_rcp(rho);
            const T v = mx * ir;
#endif
            const T p = prho * rho + gm1 * e;
            const T s = dsqrt(rho), r32 = rho * s, ps = p * s;
            const T v_m = lane_prev(v), p_m = lane_prev(p), s_m = lane_prev(s);
            const Profile<T> pv = line_profile(gp.first_order, v_m, v, lane_next(v));
            const Profile<T> pp = line_profile(gp.first_order, p_m, p, lane_next(p));
            const VP<T> a = riemann(gp.first_order, s_m, s, lane_prev(r32), r32, lane_prev(ps), ps, lane_prev(pv), pv,
                                    lane_prev(pp), pp, gam, tau, hx, tohx);
            const VP<T> b{lane_next(a.V), lane_next(a.P)};
            const T DPx = PPML_DIV(b.P - a.P, hx, ihx);
            const T sPV = PPML_DIV(b.P * b.V - a.P * a.V, hx, ihx);
            const T sV = PPML_DIV(b.V - a.V, hx, ihx);
            T w[NF];
            w[0] = rho;
            w[1] = mx - tau * DPx;
            w[2] = Et - tau * sPV;
            w[3] = e - ((tau * gm1) * e) * sV;
            if (gp.potential != POT_NONE) {
                double g[3];
                potential_grad<0>(gp, cs, 0, 0, g);
                const double work = (double)mx * g[0];
                const double tr = tau_d * (double)rho;
                w[1] = (T)((double)w[1] - tr * g[0]);
                w[2] = (T)((double)w[2] - tau_d * work);
            }
            // ghosts of the stage's output: outflow and reflecting faces copy
            // the lanes of the cells they mirror (at most three cells inside,
            // so in this segment), inflow faces hold their state; periodic
            // ghosts have computed their cell's values
            if (edge && gp.bc_lo[0] != BC_PERIODIC) {
                const int l = ln + (cs - c);  // the lane of the mirrored cell
#pragma unroll
                for (int f = 1; f < NF; f++) w[f] = __shfl(w[f], l, 64);
                if (flip) w[1] = -w[1];
                if (gp.any_inflow && face >= 0) {
                    w[1] = inflow_value<T>(ctrl, face, 1);
                    w[2] = inflow_value<T>(ctrl, face, 4);
                    w[3] = inflow_value<T>(ctrl, face, 5);
                }
            }

            // ---- Lagrangian stage (Sec. 2.3): upwind fluxes through the face
            // between the previous lane's cell and this one ----
#ifdef PPML_EXACT
            const T u = w[1] / rho;
#else
            const T u = w[1] * ir;
#endif
            const T vh = interface_velocity(lane_prev(u), s_m, u, s);
            const bool left = vh >= T(0);
            // a lane forms its cell's flux through its right face, used where
            // the flow there is to the right, and through its left face, used
            // where it is to the left
            T fn[NF];
#ifdef PPML_EXACT
            const T vr = lane_next(vh);
            const T z = dabs(vh) * tau / hx, zr = lane_next(z);
#pragma unroll
            for (int f = 0; f < NF; f++) {
                const Parab<T> q = line_profile(gp.first_order, lane_prev(w[f]), w[f], lane_next(w[f]));
                const T Fr = vr * avg_left(q.L, q.R, q.Q6, zr), Fl = vh * avg_right(q.L, q.R, q.Q6, z);
                const T Fm = lane_prev(Fr);
                const T F = left ? Fm : Fl;
                fn[f] = w[f] - tau * ((lane_next(F) - F) / hx);
            }
#else
            const FaceW<T> fw = face_weights(gp.first_order, left, vh * tohx);
            const FaceW<T> fr{lane_next(fw.vs), lane_next(fw.a), lane_next(fw.b)};
#pragma unroll
            for (int f = 0; f < NF; f++) {
                const Jumps<T> q = line_profile(gp.first_order, lane_prev(w[f]), w[f], lane_next(w[f]));
                const T Fm = lane_prev(face_flux(fr, q));
                const T Fl = face_flux(fw, q);
                const T F = left ? Fm : Fl;
                fn[f] = w[f] - (lane_next(F) - F);
            }
#endif
            if (ln >= LINE_HALO && ln < LINE_HALO + LINE_W && c < n) {
                energy_correction<T, 1>(fn, thr);
                T sv, sc;
                cell_speeds<T, 1>(fn[0], fn[1], T(0), T(0), fn[3], prho, gam, gm1, sv, sc);
                bad = bad || bad_cell(fn[0], fn[2], fn[3], sv, sc);
                vmax = vmax > sv ? vmax : sv;
                cmax = cmax > sc ? cmax : sc;
#pragma unroll
                for (int f = 0; f < NF; f++) dst[f * n + c] = fn[f];
            }
        }
        T *const r = red + (taken & 1) * 2 * (LINE_THREADS / 64);
        const T mm = line_max2(vmax, cmax);
        if ((ln & 31) == 31) r[(ln >> 5) * (LINE_THREADS / 64) + wv] = mm;
        t = t + tau_d;
        dt_last = tau_d;
        steps_left--;
        taken++;
        __syncthreads();
        // |v| of the waves in the first row of 16 lanes, c in the second
        const T m = line_max16(r[(ln & 16) + ((ln & 15) < nw ? (ln & 15) : 0)]);
        vm = (double)read_lane(m, 15);
        cm = (double)read_lane(m, 31);
    }

    if (LDS ? taken > 0 : taken & 1) {
        const T *fin = LDS ? lds + (taken & 1) * NF * n : W;
        for (int i = threadIdx.x; i < NF * n; i += blockDim.x) U[i] = fin[i];
    }
    if (__any(bad) && ln == 0) atomicOr(&ctrl->err, 1);
    if (threadIdx.x == 0) {
        if (run_steps >= 0) {
            ctrl->dt_fixed = dt_fixed;
            ctrl->t_stop = t_stop;
        }
        ctrl->steps_left = steps_left;
        if (taken > 0) {
            ctrl->t = t;
            ctrl->dt_last = dt_last;
            ctrl->steps = ctrl->steps + taken;
        }
    }
    if (taken > 0 && (int)threadIdx.x < gp.mslots) {
        unsigned long long *p = max_slot(ctrl, gp.mslots, set, threadIdx.x);
        p[0] = threadIdx.x == 0 ? (unsigned long long)__double_as_longlong(vm) : 0ull;
        p[1] = threadIdx.x == 0 ? (unsigned long long)__double_as_longlong(cm) : 0ull;
    }
}

extern __shared__ __align__(16) unsigned char line_shared[];

template <typename T>
__global__ __launch_bounds__(LINE_THREADS) void k_line(T *U, GridParams gp, Ctrl *ctrl, long long run_steps,
                                                       double run_dt, double run_t_stop, int nlaunch)
{
    line_body<T, true>(U, nullptr, gp, ctrl, run_steps, run_dt, run_t_stop, nlaunch, reinterpret_cast<T *>(line_shared));
}

// The short 1-D grids of a batch, one work group each: the first nlds in LDS,
// the rest in memory.
template <typename T>
__global__ __launch_bounds__(LINE_THREADS) void k_line_batch(const BatchEntry *__restrict__ ents, int nlds, int nlaunch)
{
    const BatchEntry *e = ents + blockIdx.x;
    T *const lds = reinterpret_cast<T *>(line_shared);
    if ((int)blockIdx.x < nlds)
        line_body<T, true>((T *)e->state, nullptr, e->gp, e->ctrl, -1, 0.0, 0.0, nlaunch, lds);
    else
        line_body<T, false>((T *)e->state, (T *)e->half, e->gp, e->ctrl, -1, 0.0, 0.0, nlaunch, lds);
}

}  // namespace ppml
