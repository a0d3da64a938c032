// ppml_sine.hpp -- the sine transforms of the self-gravity potential
// (Sec. 2.5) on the matrix cores of gfx950, five passes over the grid.
//
//   x forward   density (+ shell terms) -> sums and differences -> modes
//   y forward   sums and differences -> modes, in place
//   z           forward, division by the eigenvalue, inverse, in place
//   y inverse   modes -> sums and differences -> cells, in place
//   x inverse   modes -> cells, into the interior of the padded potential
//
// A wave owns 16 lines of an axis of n cells.  It reads them once into
// registers as the right operand of the 16x16x4 matrix instruction (lane
// l = 16 q + c holds line c), the mirror cells b and n-1-b already added and
// subtracted: the odd modes are So times the sums, the even modes Se times
// the differences (half the products of the full matrix).  The matrices come
// through LDS, `ct` tiles of 16 rows at a time, shared by the block's waves.
// The order of the four k indices that a lane holds in a 16-deep block is
// that of the result registers (krow), so in the z pass the amplitudes leave
// the first product as the right operand of the second: scaled by the
// eigenvalue, they never leave the registers.
//
// The transforms of FP32 states run in FP64 where an axis is short (sine_fp64),
// from the stored density to the stored potential: the work array and the outer
// layer's list hold FP64 then.
//
// A line is read whole before any of it is written and no line belongs to
// two waves, so y and z run in place.
//
// Bound: the matrix rate and, beside it, the loads and stores at the ends of
// a block's life, which one block a CU cannot hide behind products (the
// matrix cores are busy for 63% of a y pass at 256^3 FP32).  A solve's passes
// against two half-size library products an axis and direction with kernels
// for the sums, the division and the differences between them (19 passes over
// the grid): 150^3 FP64 135 us against 318, 256^3 FP32 350 against 375 (the
// products alone 168 at the rate of a large FP32 product).  The x forward pass
// at 256^3 FP32 takes 63 us; with the shell terms added to every cell's
// density as it was loaded (registers for 8 waves a block instead of 16) 85.  Blocks of four
// waves with 64 KB of the table at a time took 79 us where a y pass at 256^3
// takes 57.
#pragma once

#include <type_traits>

#include "ppml_gravity.hpp"

namespace ppml {

// (named: in kernel signatures an unnamed one has other names on host and device)
enum SineKind : int { SINE_X_FWD, SINE_Y_FWD, SINE_Z, SINE_Y_INV, SINE_X_INV };

typedef float sine_f4 __attribute__((ext_vector_type(4)));
typedef double sine_d4 __attribute__((ext_vector_type(4)));
template <typename T> struct SineVec { using type = sine_f4; };
template <> struct SineVec<double> { using type = sine_d4; };

// D += A B: lane l gives A(l % 16, k) and B(k, l % 16) for k = l / 16 and
// receives column l % 16 of D, rows krow(l / 16, 0..3).
__device__ __forceinline__ sine_f4 sine_mma(float a, float b, sine_f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ sine_d4 sine_mma(double a, double b, sine_d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Row of a 16-row tile in register s of a lane of group q = l / 16.
template <typename T> __device__ __forceinline__ constexpr int krow(int q, int s)
{
    return sizeof(T) == 4 ? 4 * q + s : 4 * s + q;
}

// Leading dimension of the staged matrix rows (MT tiles of 16 entries): FP32
// rows are read 16 bytes a lane (an odd multiple of 16 bytes apart, so 16
// rows fall on 16 different groups of four banks), FP64 rows 8 bytes a lane.
template <typename T> __host__ __device__ constexpr int sine_ld(int mt)
{
    return sizeof(T) == 4 ? 16 * mt + 4 : 16 * mt + 2;
}

// Blocks of 16 of the longer (odd) half of an axis of n cells.
__host__ __device__ constexpr int sine_tiles(int n) { return (grav_no(n) + 15) / 16; }

// Table of an axis: tiles of 16 rows of the odd half, then of the even half
// (rows of sine_ld entries, zero beyond the half's extent), first with the
// modes as rows, then with the cells as rows.  A chunk of tiles is copied to
// LDS as it stands.
template <typename T> __host__ __device__ constexpr long long sine_table_count(int n)
{
    return 2ll * sine_tiles(n) * 2 * 16 * sine_ld<T>(sine_tiles(n));
}

template <typename T> __global__ void k_sine_table(T *__restrict__ S, double *__restrict__ f, int n)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int mt = sine_tiles(n), ld = sine_ld<T>(mt);
    if (t < n) {
        const double s = sin(M_PI * (double)grav_mode((int)t, n) / (2.0 * (double)(n + 1)));
        f[t] = 1.0 - 2.0 * s * s / 3.0;
    }
    if (t >= sine_table_count<T>(n)) return;
    const int col = (int)(t % ld);
    long long r = t / ld;
    const int row = (int)(r % 16);
    r /= 16;
    const int h = (int)(r % 2), tile = (int)(r / 2) % mt, form = (int)(r / 2) / mt;
    const int m = h ? grav_ne(n) : grav_no(n);
    const int a = form ? col : 16 * tile + row, b = form ? 16 * tile + row : col;
    T v = T(0);
    if (a < m && b < m) {
        const long long j = 2 * a + 1 + h, k = b + 1;
        v = (T)sinpi((double)((j * k) % (2ll * (n + 1))) / (double)(n + 1));
    }
    S[t] = v;
}

// Element types of a pass's source and destination.
template <typename T, int KIND, typename ST> using SineIn = std::conditional_t<KIND == SINE_X_FWD, ST, T>;
template <typename T, int KIND, typename ST> using SineOut = std::conditional_t<KIND == SINE_X_INV, ST, T>;

struct SineArgs {
    double coef, norm;  // right-hand side 4 pi G h^2, inverse transform's factor
};

// Launch shape: a block per CU, its LDS holding the whole table where that
// fits (all but FP64 lines of more than 192 cells), else an even share of
// it at a time; as many waves as their registers allow (a line's two halves
// take MT / 2 times the element's bytes a lane, in the z pass the results as
// much again).
constexpr int SINE_LDS = 160 * 1024;
template <typename T, int MT, int KIND> struct SineShape {
    static constexpr int TILE = 2 * 16 * sine_ld<T>(MT) * (int)sizeof(T);
    static constexpr int PARTS = (MT * TILE + SINE_LDS - 1) / SINE_LDS;
    static constexpr int CT = (MT + PARTS - 1) / PARTS;
    static constexpr int REGS = 2 * MT * (int)sizeof(T) * (KIND == SINE_Z ? 2 : 1);
    static constexpr int WAVES = REGS <= 64 ? 16 : REGS <= 160 ? 8 : 4;
};

// Four entries of the staged matrix row at `row`, columns 16 t + krow(q, 0..3).
__device__ __forceinline__ sine_f4 sine_row(const float *row, int t, int q)
{
    return *(const sine_f4 *)(row + 16 * t + 4 * q);
}
__device__ __forceinline__ sine_d4 sine_row(const double *row, int t, int q)
{
    sine_d4 a;
#pragma unroll
    for (int s = 0; s < 4; s++) a[s] = row[16 * t + 4 * s + q];
    return a;
}

// (ST: storage type of the density and the potential, T that of the transforms)
template <typename T, int MT, int KIND, typename ST>
__global__ __launch_bounds__((64 * SineShape<T, MT, KIND>::WAVES)) void k_sine(
    const SineIn<T, KIND, ST> *src, SineOut<T, KIND, ST> *dst, const T *__restrict__ S, const T *__restrict__ E,
    const double *__restrict__ fx, const double *__restrict__ fy, const double *__restrict__ fz, GridParams gp,
    SineArgs args)
{
    using V = typename SineVec<T>::type;
    using In = SineIn<T, KIND, ST>;
    using Out = SineOut<T, KIND, ST>;
    constexpr int LD = sine_ld<T>(MT);
    constexpr bool FWD = KIND <= SINE_Z, INV = KIND >= SINE_Z;
    constexpr int AXIS = KIND == SINE_Z ? 2 : KIND == SINE_Y_FWD || KIND == SINE_Y_INV ? 1 : 0;
    constexpr int CT = SineShape<T, MT, KIND>::CT;
    constexpr int HALF = 16 * LD;
    constexpr int TILE16 = SineShape<T, MT, KIND>::TILE / 16;  // 16-byte words of a tile
    constexpr int FULL = MT - 1;  // blocks of 16 that lie inside both halves
    constexpr int QMAX = krow<T>(3, 0);
    extern __shared__ double sine_lds[];
    const T *P = (const T *)sine_lds;  // [CT][half][16][LD]
    const int n0 = gp.n[0], n1 = gp.n[1], n2 = gp.n[2];
    const int n = gp.n[AXIS], no = grav_no(n), ne = grav_ne(n);
    const int nlines = AXIS == 0 ? n1 * n2 : AXIS == 1 ? n0 * n2 : n0 * n1;
    const int q = (threadIdx.x & 63) >> 4, c = threadIdx.x & 15;
    const int waves = blockDim.x >> 6;
    const uint4 *table = (const uint4 *)(S + (INV && !FWD ? sine_table_count<T>(n) / 2 : 0));
    // rows 16 t0 ... (modes: forward, z; cells: inverse) of both halves to LDS
    auto stage = [&](int t0, int tn) {
        const int words = tn * TILE16;
        for (int u = threadIdx.x & ~63; u < words; u += blockDim.x) {
            const int w = u + (threadIdx.x & 63);
            if (w < words)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(table + t0 * TILE16 + w),
                    (__attribute__((address_space(3))) void *)((uint4 *)sine_lds + u), 16, 0, 0);
        }
    };
    if (CT == MT) stage(0, MT);

    const int groups = (nlines + 16 * waves - 1) / (16 * waves);
    for (int grp = blockIdx.x; grp < groups; grp += gridDim.x) {
        // the offsets below depend on the stride and the group's first row,
        // laundered here: computed where they are used instead of ahead of
        // the loop, in registers that the lines need
        int st = AXIS == 0 ? 1 : AXIS == 1 ? n0 : n0 * n1;
        if (AXIS != 0) asm volatile("" : "+s"(st));
        int qk = krow<T>(q, 0);
        asm volatile("" : "+v"(qk));
        const int line = (grp * waves + (int)(threadIdx.x >> 6)) * 16 + c;
        const bool live = line < nlines;
        const int ln = live ? line : nlines - 1;
        // the line's place along the two other axes
        const int lb = ln / (AXIS == 0 ? n1 : n0), la = ln - lb * (AXIS == 0 ? n1 : n0);
        const int base = AXIS == 0 ? ln * n0 : AXIS == 1 ? lb * n0 * n1 + la : ln;
        const int out = KIND == SINE_X_INV ? (int)pad_index(gp, 0, la, lb) : base;
        // an element is a uniform pointer plus a lane's byte offset: that of
        // its group's first row (up), or of its last one counted backwards
        auto at = [](const In *p, unsigned off) { return *(const In *)((const char *)p + off); };
        auto put = [](Out *p, unsigned off, Out v) { *(Out *)((char *)p + off) = v; };
        const unsigned in_up = (unsigned)(base + qk * st) * (unsigned)sizeof(In);
        const unsigned in_dn = (unsigned)(base + (QMAX - qk) * st) * (unsigned)sizeof(In);
        const unsigned out_up = (unsigned)(out + qk * st) * (unsigned)sizeof(Out);

        // the lines: cells b and n-1-b (forward) or odd and even modes
        // (inverse); zero beyond the half's extent
        T xo[4 * MT], xe[4 * MT];
        double scale = 1.0, scale0 = 1.0;  // of the line's cells, of its two ends
        if constexpr (KIND == SINE_X_FWD) {
            // a line in the outer layer comes whole from the right-hand side
            // listed there, any other from the density but for its two ends
            const bool full = la == 0 || la == n1 - 1 || lb == 0 || lb == n2 - 1;
            const T *El = E + grav_edge_index(0, la, lb, n0, n1, n2);
            if constexpr (std::is_same_v<T, ST>) {
                const T *up = (full ? El : src + base) + qk;
                const T *dn = (full ? El : src + base) + (n - 1 - qk);
                if (!full) scale = args.coef;
                scale0 = q == 0 ? 1.0 : scale;
#pragma unroll
                for (int p = 0; p < 4 * MT; p++) {
                    const int u = 16 * (p >> 2) + krow<T>(0, p & 3);
                    const int ul = (p >> 2) < FULL || u + qk < no ? u : no - 1 - qk;
                    xo[p] = up[ul];
                    xe[p] = dn[-ul];
                }
            } else {
                // (a lambda above as well cost the pass 3 of 63 us at 256^3)
                auto load = [&](const auto *line) {
                    const auto *up = line + qk, *dn = line + (n - 1 - qk);
#pragma unroll
                    for (int p = 0; p < 4 * MT; p++) {
                        const int u = 16 * (p >> 2) + krow<T>(0, p & 3);
                        const int ul = (p >> 2) < FULL || u + qk < no ? u : no - 1 - qk;
                        xo[p] = up[ul];
                        xe[p] = dn[-ul];
                    }
                };
                if (!full) scale = args.coef;
                scale0 = q == 0 ? 1.0 : scale;
                if (full) load(El);
                else load(src + base);
            }
            if (!full && q == 0) xo[0] = El[0], xe[0] = El[n > 1];
        } else {
#pragma unroll
            for (int p = 0; p < 4 * MT; p++) {
                const int u = 16 * (p >> 2) + krow<T>(0, p & 3);  // row of group 0
                if ((p >> 2) < FULL) {
                    xo[p] = at(src + u * st, in_up);
                    xe[p] = FWD ? at(src + (n - 1 - u - QMAX) * st, in_dn) : at(src + (no + u) * st, in_up);
                } else {
                    const int b = u + qk;
                    const int bl = b < no ? b : no - 1, be = FWD ? n - 1 - bl : b < ne ? no + b : n - 1;
                    xo[p] = src[base + bl * st];
                    xe[p] = src[base + be * st];
                }
            }
        }
#pragma unroll
        for (int p = 0; p < 4 * MT; p++) {
            const int b = 16 * (p >> 2) + krow<T>(0, p & 3) + qk;
            const bool pair = (p >> 2) < FULL || b < ne, in = (p >> 2) < FULL || b < no;
            if constexpr (KIND == SINE_X_FWD) {
                const double lo = (p ? scale : scale0) * (double)xo[p], hi = (p ? scale : scale0) * (double)xe[p];
                xo[p] = in ? (T)(pair ? lo + hi : lo) : T(0);
                xe[p] = pair ? (T)(lo - hi) : T(0);
            } else {
                const T lo = xo[p], hi = xe[p];
                xo[p] = in ? (FWD && pair ? lo + hi : lo) : T(0);
                xe[p] = pair ? (FWD ? lo - hi : hi) : T(0);
            }
        }
        const double f2 = KIND == SINE_Z ? fx[la] * fy[lb] : 0.0;

        V yo[KIND == SINE_Z ? MT : 1], ye[KIND == SINE_Z ? MT : 1];
        if constexpr (KIND == SINE_Z) {
#pragma unroll
            for (int t = 0; t < MT; t++) yo[t] = V(0), ye[t] = V(0);
        }
        // cells b and n-1-b of block t from their sums and differences
        auto put_cells = [&](int t, const V &so, const V &de) {
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int u = 16 * t + krow<T>(0, r);
                const int b = u + qk;
                if (live && b < no) put(dst + u * st, out_up, (Out)(so[r] + de[r]));
                if (live && b < ne) dst[out + (n - 1 - b) * st] = (Out)(so[r] - de[r]);
            }
        };
        for (int t0 = 0; t0 < MT; t0 += CT) {
            const int tn = MT - t0 < CT ? MT - t0 : CT;
            if (CT < MT) {
                __syncthreads();
                stage(t0, tn);
            }
            if (CT < MT || grp == (int)blockIdx.x) {
                __builtin_amdgcn_s_waitcnt(0);  // this wave's copies to LDS
                __syncthreads();
            }
#pragma unroll 1
            for (int t = 0; t < tn; t++) {
                const T *ro = P + (32 * t + c) * LD, *re = ro + HALF;
                // two sums a half, over every other block of 16: independent
                // instructions in flight, shorter chains of roundings
                V d[2][2] = {{V(0), V(0)}, {V(0), V(0)}};
#pragma unroll
                for (int k = 0; k < MT; k++) {
                    const V ao = sine_row(ro, k, q), ae = sine_row(re, k, q);
#pragma unroll
                    for (int s = 0; s < 4; s++) {
                        d[0][k & 1] = sine_mma(ao[s], xo[4 * k + s], d[0][k & 1]);
                        d[1][k & 1] = sine_mma(ae[s], xe[4 * k + s], d[1][k & 1]);
                    }
                }
                const V so = d[0][0] + d[0][1], se = d[1][0] + d[1][1];
                const int row = 16 * (t0 + t);
                if constexpr (KIND == SINE_Z) {
                    V go, ge;
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int a = row + krow<T>(0, r) + qk;
                        go[r] = grav_amplitude<T>(so[r], f2, fz[a < no ? a : no - 1], args.norm);
                        ge[r] = grav_amplitude<T>(se[r], f2, fz[a < ne ? no + a : n - 1], args.norm);
                    }
#pragma unroll
                    for (int k = 0; k < MT; k++)
#pragma unroll
                        for (int s = 0; s < 4; s++) {
                            const int w = (32 * t + krow<T>(0, s) + qk) * LD + 16 * k + c;
                            yo[k] = sine_mma(P[w], go[s], yo[k]);
                            ye[k] = sine_mma(P[HALF + w], ge[s], ye[k]);
                        }
                } else if constexpr (INV) {
                    put_cells(t0 + t, so, se);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int u = row + krow<T>(0, r);
                        if (live && u + qk < no) put(dst + u * st, out_up, so[r]);
                        if (live && u + qk < ne) put(dst + (no + u) * st, out_up, se[r]);
                    }
                }
            }
        }
        if constexpr (KIND == SINE_Z) {
#pragma unroll
            for (int t = 0; t < MT; t++) put_cells(t, yo[t], ye[t]);
        }
    }
}

}  // namespace ppml
