// ws_device.hpp -- device-side data and helpers of the gfx950 time step.
//
// State is kept as eta = w - w_s (free surface), P, Q in FP32 structure-of-
// arrays fields of nyp rows x pitch floats (x fastest, rows padded to whole
// tiles).  Bathymetry is kept as the still-water depth at the corners,
// D = w_s - z (unclamped), so that every kernel works with depths measured
// from the still water level and a lake at rest is all zeros.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ws {

constexpr int TX = 64;        // solver tile width  (cells along x)
constexpr int TY = 16;        // solver tile height (cells along y) = column segment length
constexpr int MX = 16;        // row segment length (4 per solver tile row)
constexpr int NT = 256;       // threads per solver tile workgroup (4 wave64)
constexpr int NTB = 128;      // the same in the batch (2 wave64)
constexpr int SO = 62;        // stencil: output columns per 64-lane strip wave
constexpr int SY = 8;         // stencil: nominal rows streamed per strip wave (default)
constexpr int SWG = 4;        // stencil: strip waves per workgroup
constexpr int MAXC = 256;     // wave components per side
constexpr int TABW = 8;       // doubles per component: a, omega, kx, ky, cx, cy, phase, -
constexpr int NRED_MAX = 2048;  // reduced unknowns per row/column system

enum { BC_SOLID = 0, BC_SPONGE = 1, BC_WAVES = 2 };
enum { BSNQ = 0, NLSW = 1 };
enum { FRIC_NONE = 0, FRIC_QUAD = 1, FRIC_MANNING = 2 };

struct SideDev {
    int type, width, ncomp;
    float expo;         // sponge: exponent s of the damping factor gamma^s (1 = eq. 30)
    const double *tab;  // ncomp * TABW
};

struct Dom {
    int nx, ny, pitch, zpitch;
    int nu, nv;         // reduced unknowns of one row / one column system
    int model, friction;
    int gl;             // ghost-buffer positions per layer: max(nx, ny) + 4
    float dx, dy, rdx, rdy;
    float g, Bd, theta, eps, fcoef;
    const float *D;     // corner still-water depth, (ny+1) rows x zpitch
    const float *gh;    // wave-maker ghost values at the pass's time (see ghost_index)
    SideDev side[4];
};

// Wave-maker ghost values are precomputed per time level: [side][layer][pos][eta, P, Q],
// layer 0 next to the boundary, pos = along-side cell index + 2 (covers -2 .. n+1).
__device__ __forceinline__ size_t ghost_index(const Dom &d, int side, int layer, int pos) {
    return (((size_t)side * 2 + layer) * d.gl + pos) * 3;
}

__device__ __forceinline__ bool is_wall(const Dom &d, int s) { return d.side[s].type != BC_WAVES; }

// Side type by a run-time side index, as selects: keeps a Dom held in
// registers free of dynamic indexing.
__device__ __forceinline__ int side_type(const Dom &d, int s) {
    return s == 0 ? d.side[0].type : s == 1 ? d.side[1].type : s == 2 ? d.side[2].type : d.side[3].type;
}

// Corner index behind a side: mirrored across walls and sponges, held at the
// boundary value across wave makers; clamped into range for padding cells.
__device__ __forceinline__ int map_corner(int c, int n, bool lo_wall, bool hi_wall) {
    if (c < 0) c = lo_wall ? -c : 0;
    if (c > n) c = hi_wall ? 2 * n - c : n;
    return c < 0 ? 0 : (c > n ? n : c);
}

__device__ __forceinline__ float corner_D(const Dom &d, int ci, int cj) {
    int i = map_corner(ci, d.nx, is_wall(d, 0), is_wall(d, 1));
    int j = map_corner(cj, d.ny, is_wall(d, 2), is_wall(d, 3));
    return d.D[(size_t)j * d.zpitch + i];
}

// Wave-maker values at (x, y, t): sum of a sin(omega t + phi - kx x - ky y),
// discharges c cos(theta) eta, c sin(theta) eta per component.  The phase is
// formed and reduced to [-pi, pi] in double, the sine taken in single.
// Components first, first + stride, ... of the sum (one lane's share).
__device__ inline void wave_partial(const SideDev &s, double x, double y, double t, int first, int stride,
                                    float &se, float &sp, float &sq) {
    for (int m = first; m < s.ncomp; m += stride) {
        const double *c = s.tab + TABW * m;
        double ph = c[1] * t + c[6] - (c[2] * x + c[3] * y);
        ph -= 6.283185307179586 * rint(ph * 0.15915494309189535);
        const float v = (float)c[0] * sinf((float)ph);
        se += v;
        sp += (float)c[4] * v;
        sq += (float)c[5] * v;
    }
}

__device__ inline void wave_eval(const SideDev &s, double x, double y, double t, float &e,
                                 float &p, float &q) {
    float se = 0.f, sp = 0.f, sq = 0.f;
    for (int m = 0; m < s.ncomp; ++m) {
        const double *c = s.tab + TABW * m;
        double ph = c[1] * t + c[6] - (c[2] * x + c[3] * y);
        ph -= 6.283185307179586 * rint(ph * 0.15915494309189535);
        float v = (float)c[0] * sinf((float)ph);
        se += v;
        sp += (float)c[4] * v;
        sq += (float)c[5] * v;
    }
    e = se;
    p = sp;
    q = sq;
}

// Panel layout: eight columns side by side, row after row, then the next eight
// (float index of column i, row j of an ny-row field).  A workgroup that takes
// eight whole columns reads one contiguous run of memory.
__device__ __forceinline__ unsigned panel(int i, int j, int ny) {
    return ((unsigned)(i >> 3) * (unsigned)ny + (unsigned)j) * 8u + (unsigned)(i & 7);
}

// Value of cell (i, j), inside or in the two-cell ghost ring: reflected across
// every wall side first (normal discharge of that side changes sign), then, if
// still behind a wave-maker side, that maker's values at the reflected
// position (precomputed ghost buffer).  Cells further out (padding) are
// clamped into the domain.
__device__ inline void load_cell(const Dom &d, const float *__restrict__ E,
                                 const float *__restrict__ P, const float *__restrict__ Q, int i,
                                 int j, float &e, float &p, float &q) {
    float sp = 1.f, sq = 1.f;
    if (i < 0 && is_wall(d, 0)) { i = -1 - i; sp = -sp; }
    if (i >= d.nx && is_wall(d, 1)) { i = 2 * d.nx - 1 - i; sp = -sp; }
    if (j < 0 && is_wall(d, 2)) { j = -1 - j; sq = -sq; }
    if (j >= d.ny && is_wall(d, 3)) { j = 2 * d.ny - 1 - j; sq = -sq; }
    const bool in_i = i >= 0 && i < d.nx, in_j = j >= 0 && j < d.ny;
    int side = -1;
    if (!in_i) side = i < 0 ? 0 : 1;
    else if (!in_j) side = j < 0 ? 2 : 3;
    if (side >= 0 && side_type(d, side) == BC_WAVES) {
        int layer = side == 0 ? -1 - i : side == 1 ? i - d.nx : side == 2 ? -1 - j : j - d.ny;
        int pos = (side < 2 ? j : i) + 2;
        layer = layer < 0 ? 0 : (layer > 1 ? 1 : layer);
        pos = pos < 0 ? 0 : (pos >= d.gl ? d.gl - 1 : pos);
        const float *g = d.gh + ghost_index(d, side, layer, pos);
        e = g[0];
        p = g[1];
        q = g[2];
    } else {
        i = i < 0 ? 0 : (i >= d.nx ? d.nx - 1 : i);
        j = j < 0 ? 0 : (j >= d.ny ? d.ny - 1 : j);
        size_t k = (size_t)j * d.pitch + i;
        e = E[k];
        p = P[k];
        q = Q[k];
    }
    p *= sp;
    q *= sq;
}

// ---------------------------------------------------------------- KP07 parts
// minmod of three: the smallest if all are positive, the largest if all are
// negative, else 0 -- the median of (min, max, 0) (v_med3: three
// instructions with v_min3 and v_max3).
__device__ __forceinline__ float minmod3(float a, float b, float c) {
    const float mn = fminf(a, fminf(b, c)), mx = fmaxf(a, fmaxf(b, c));
    return __builtin_amdgcn_fmed3f(mn, mx, 0.f);
}

// Hardware reciprocal, reciprocal square root and square root (1 ulp); their
// arguments here are never denormal except sqrt of a vanishing depth.
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float frsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Lane shifts across the 64-lane wave (DPP wave_shr:1 / wave_shl:1): lane k
// takes lane k-1 (shr) or k+1 (shl); the lane without a source takes `old`.
__device__ __forceinline__ float shr1(float v, float old) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float shl1(float v, float old) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), 0x130, 0xf, 0xf, false));
}
// The same shifts where the edge lane's result is never used (it belongs to
// a halo lane): the vacated lane reads 0 (bound_ctrl), so the shift is one
// DPP move with no copy of an "old" value first.
__device__ __forceinline__ float shr1z(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float shl1z(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

struct F3 { float e, n, t; };  // surface, normal and tangential discharge at a face

// Reconstruction constants of the generalized minmod limiter with parameter
// theta: minmod(theta a, c/2, theta b) = theta minmod(a, c/(2 theta), b) for
// theta > 0, and the face values take half the slope, so the limiter runs on
// the plain differences with the central one scaled by kc = 1/(2 theta), and
// the face values add or subtract hth = theta/2 times its result (two
// multiplies fewer a variable).  thr: the depth eps^(1/4) from which eq. 14 is
// m / h (kept away from 0, where the reciprocal would be infinite).
struct Recon { float kc, hth, thr; };
__device__ __forceinline__ Recon recon_k(float th, float eps) {
    return {0.5f / th, 0.5f * th, fmaxf(fsqrt(fsqrt(eps)), 1e-9f)};
}

// All arithmetic from here to the face fluxes is written in explicit fused
// and separate operations with contraction off: the compiler's choice between
// the two may differ between kernel instances (strip heights, batch or
// single), which must give the same bits.

// Limited linear reconstruction of one variable of a cell along one
// direction: v its value, a and b its differences to the lower and upper
// neighbour (a row's b is the next row's a).
__device__ __forceinline__ void face_values(float v, float a, float b, Recon rk, float &lo, float &hi) {
#pragma clang fp contract(off)
    const float m = minmod3(a, rk.kc * (a + b), b);
    lo = fmaf(-rk.hth, m, v);
    hi = fmaf(rk.hth, m, v);
}

// Conservative positivity correction of a cell's two face surfaces against
// the depths of its faces (w < B  <=>  eta < -D).
__device__ __forceinline__ void keep_positive(float e0, float Dlo, float Dhi, float &lo, float &hi) {
#pragma clang fp contract(off)
    const bool fix_hi = hi < -Dhi, fix_lo = !fix_hi && lo < -Dlo;
    const float l = lo, h = hi;
    lo = fix_hi ? fmaf(2.f, e0, Dhi) : (fix_lo ? -Dlo : l);
    hi = fix_hi ? -Dhi : (fix_lo ? fmaf(2.f, e0, Dlo) : h);
}

// One side of a face: velocities, discharges, wave speed, momentum flux.
struct FaceSide { float u, v, n, t, c, F; };

// Central-upwind flux at a face in well-balanced ("pre-balanced") form.  With
// D_f the face still-water depth and h = eta + D_f, the pressure g h^2/2 is
// split into g eta (eta + 2 D_f)/2 + g D_f^2/2; the constant g D_f^2/2 passes
// through the central-upwind average unchanged and cancels exactly against
// the matching part of the bottom source, so it is dropped here and the
// source becomes g (D_hi - D_lo)/dx * eta_cell.  Where both sides are dry the
// face flux of the original form is zero, i.e. (0, -g D_f^2/2, 0) here.
// With the weight w = a+/(a+ - a-) the average (a+ X_L - a- X_R)/(a+ - a-) is
// X_R + w (X_L - X_R), and the diffusion's a+ a-/(a+ - a-) is w a-.
// wet (uniform over the wave): both sides of every lane's face are at least
// thr deep, where eq. 14 gives u = m / h, the discharges themselves, and no
// case of the general form below applies: 44 operations instead of about 85
// for most waves of most grids.  A lane's own result does not depend on which
// of the two forms its wave took.
// Returns (mass, normal momentum, tangential momentum).
__device__ __forceinline__ void cu_flux(bool wet, float g, float eps, float thr, float Df, const F3 &L, const F3 &R,
                                        float &H0, float &H1, float &H2) {
#pragma clang fp contract(off)
    const float hg = 0.5f * g, hL = L.e + Df, hR = R.e + Df;
    FaceSide l, r;
    float am, ap, inv;
    bool dry = false;
    if (wet) {
        auto side = [&](float h, const F3 &s) -> FaceSide {
            const float f = frcp(h), u = f * s.n;
            return {u, f * s.t, s.n, s.t, fsqrt(g * h), fmaf(hg * s.e, fmaf(2.f, Df, s.e), s.n * u)};
        };
        l = side(hL, L);
        r = side(hR, R);
        ap = fmaxf(fmaxf(l.u + l.c, r.u + r.c), 0.f);
        am = fminf(fminf(l.u - l.c, r.u - r.c), 0.f);
        inv = frcp(ap - am);
    } else {
        auto side = [&](float hraw, const F3 &s) -> FaceSide {
            const float h = fmaxf(hraw, 0.f), h2 = h * h, h4 = h2 * h2;
            const bool deep = h >= thr;
            // eq. (14): u = m * sqrt(2) h / sqrt(h^4 + max(h^4, eps))
            const float f = deep ? frcp(h) : 1.41421356237f * h * frsq(h4 + fmaxf(h4, eps));
            const float u = f * s.n, v = f * s.t, n = deep ? s.n : h * u, t = deep ? s.t : h * v;
            const float e = h > 0.f ? s.e : -Df;
            return {u, v, n, t, fsqrt(g * h), fmaf(hg * e, fmaf(2.f, Df, e), n * u)};
        };
        l = side(hL, L);
        r = side(hR, R);
        ap = fmaxf(fmaxf(l.u + l.c, r.u + r.c), 0.f);
        am = fminf(fminf(l.u - l.c, r.u - r.c), 0.f);
        dry = ap - am <= 1e-10f;
        inv = frcp(dry ? 1.f : ap - am);
    }
    const float w = ap * inv, k = w * am, dn = l.n - r.n, tR = r.n * r.v;
    H0 = fmaf(k, R.e - L.e, fmaf(w, dn, r.n));
    H1 = fmaf(-k, dn, fmaf(w, l.F - r.F, r.F));
    H2 = fmaf(-k, l.t - r.t, fmaf(w, fmaf(l.n, l.v, -tR), tR));
    if (!wet) {
        H0 = dry ? 0.f : H0;
        H1 = dry ? -hg * Df * Df : H1;
        H2 = dry ? 0.f : H2;
    }
}

// Row/column system coefficients of eq. 23 for one cell, from the cell's
// still-water depth d and the difference dd = d_{+1} - d_{-1} of its two
// neighbours along the direction (d_x = dd / (2 h)).  With the spacing h:
// alpha = (B + 1/3) d^2 / h^2 and beta = d d_x / (6 h) = d dd / (12 h^2), and
// A = beta - alpha, B = 1 + 2 alpha, C = -beta - alpha.  The constant
// factors come premultiplied: kal = (B + 1/3) / h^2, kbe = 1 / (12 h^2).
struct TriK { float kal, kbe; };
__device__ __forceinline__ TriK tri_k(float Bd, float rh) { return {(Bd + 1.f / 3.f) * rh * rh, rh * rh * (1.f / 12.f)}; }
__device__ __forceinline__ void tri_coef_bsnq(TriK k, float dep, float dd, float &A, float &B, float &C) {
    const float al = k.kal * (dep * dep);
    const float be = k.kbe * (dep * dd);
    A = be - al;
    B = 1.f + 2.f * al;
    C = -be - al;
}
__device__ __forceinline__ void tri_coef(const Dom &d, TriK k, float dep, float dd, float &A, float &B,
                                         float &C) {
    if (d.model == NLSW) {
        A = 0.f;
        B = 1.f;
        C = 0.f;
        return;
    }
    tri_coef_bsnq(k, dep, dd, A, B, C);
}

// Sponge layers (eq. 30): gamma = (1 + cos(pi (Ls - dist) / Ls)) / 2 within Ls
// of the side; a partially reflective layer damps by gamma^s (s = 1: the
// layer of eq. 30).  The factor of a cell is that of its column (west and
// east layers) times that of its row (south and north).  Contraction is off,
// so that every kernel rounds it alike.
__device__ inline float sponge_side(const SideDev &s, float dist, float Ls) {
#pragma clang fp contract(off)
    if (s.type != BC_SPONGE || dist >= Ls) return 1.f;
    const float gamma = 0.5f * (1.f + cospif((Ls - dist) / Ls));
    return s.expo == 1.f ? gamma : s.expo == 0.f ? 1.f : powf(gamma, s.expo);
}
__device__ inline float sponge_x(const Dom &d, int i) {
#pragma clang fp contract(off)
    return sponge_side(d.side[0], ((float)i + 0.5f) * d.dx, (float)d.side[0].width * d.dx) *
           sponge_side(d.side[1], ((float)(d.nx - i) - 0.5f) * d.dx, (float)d.side[1].width * d.dx);
}
__device__ inline float sponge_y(const Dom &d, int j) {
#pragma clang fp contract(off)
    return sponge_side(d.side[2], ((float)j + 0.5f) * d.dy, (float)d.side[2].width * d.dy) *
           sponge_side(d.side[3], ((float)(d.ny - j) - 0.5f) * d.dy, (float)d.side[3].width * d.dy);
}

}  // namespace ws
