// ws_solve.hpp -- the implicit solves of one pass in a single launch: every
// workgroup takes whole rows (eq. 21) or whole columns (eq. 22) from the
// increments to the new discharges, with nothing in memory in between.
//
// A lane owns one segment of FM cells in registers: coefficients of eq. 23
// from the cell depths, elimination of the segment's interior in favour of
// its first and last unknowns (the partition method, as seg_eliminate), one
// equation per segment for the last unknowns alone, parallel cyclic reduction
// of those equations across the lanes through LDS (one barrier a level, two
// buffers), back substitution, and the epilogue (P = P^n + dP, shoreline fix,
// sponge).  The elimination and its reciprocals are done once, not once in a
// reduction and again in an expansion, and the increments, the depth and the
// equations cross memory once: 10 words a cell (U*, V* increments, depth and
// surface twice, P^n, Q^n, P, Q) against 12.75 in three kernels, and one
// launch (4 to 5 us each at the smallest sizes) instead of three.
// Row workgroups read whole rows 16 bytes a lane and hand the cells to the
// owning lanes through LDS (segments padded to FMP floats: conflict-free
// 16-byte accesses); column workgroups read C consecutive columns of each
// row, C lanes a run, straight into the owning lanes' registers.
// us a pass's solves, summed kernel durations of a trace, three kernels
// (reduction, best PCR, expansion) / one: 128 x 64 cells 16.2 / 6.8, 1024 x 512
// 18.1 / 8.9, 1024 x 1024 23.7 / 12.9, 2048 x 1500 55.8 / 35.8 (events around a
// launch read 2 to 3 us more; the other figures in this file are such).  Bound
// by latency up to about a million cells (two trips to memory, the reduction's
// levels), above by the columns' 32-byte runs: a workgroup pulls whole 128-byte
// lines through its CU's 64 bytes a clock.
#pragma once
#include "ws_kernels.hpp"

namespace ws {

constexpr int FM = 16;    // cells a lane owns
constexpr int FMT = 32;   // the same in columns of more than FS_TALL cells
constexpr int FMP = 20;   // LDS stride of a row segment (floats)
// 128 segments x 8 columns: a workgroup's 1024 lanes.  Taking the tall form
// earlier costs a second launch and gains nothing: us at a line of 2048 / of
// 1024 cells: 2048 x 2048 49.2 / 50.1, 2048 x 1500 37.9 / 39.8, 1024 x 1100
// 18.2 / 29.3.
constexpr int FS_TALL = 2048;
__host__ __device__ constexpr int fs_m(int ny) { return ny > FS_TALL ? FMT : FM; }

// Threads of a workgroup (T, whole waves): 8 columns a run, at least one
// whole row, at least 256.  Runs of 16 columns (64 bytes) halve the lines a
// column workgroup shares with its neighbours, but also the workgroups: us a
// solve at 16 / 8 / 4 columns: 601 x 601 14.2 / 12.6 / 12.8, 1024 x 512 12.3 /
// 11.7 / 11.9, 1024 x 1024 20.0 / 17.3 / 18, 2048 x 1500 (8) 39.6 / (4) 41.
__host__ __device__ constexpr int fs_segs(int n, int M = FM) { return (n + M - 1) / M; }
inline int fs_threads(int nx, int ny) {
    const int need = 8 * fs_segs(ny, fs_m(ny)), m = need > fs_segs(nx) ? need : fs_segs(nx);
    return m <= 256 ? 256 : (m + 63) / 64 * 64;
}
// A tall grid of up to FS_NARROW columns of cells runs in one launch (k_solve_tall)
// of 4 columns a run: at 8 it gives too few workgroups, and its rows, in a
// launch of their own, are over in a moment.  us a step of the three kernels /
// rows and columns apart / one launch: 48 x 3000 cells 94 / 118 / 90, 48 x 4096
// 111 / 142 / 113, 256 x 2500 129 / 138 / 103, 512 x 3000 192 / 182 / 164; 700 x 2500
// (rows and columns apart / one launch) 186 / 189.
constexpr int FS_NARROW = 512;
inline bool fs_narrow(int nx, int ny) { return ny > FS_TALL && nx <= FS_NARROW; }
inline int fs_narrow_threads(int ny) { return (4 * fs_segs(ny, FMT) + 63) / 64 * 64; }
inline bool fs_fits(int nx, int ny) { return ny <= 2 * FS_TALL && fs_segs(nx) <= 1024; }
// Rows of a row workgroup, columns of a column workgroup (a power of two, 4 to
// 64), workgroups of each (rows padded to the 8 XCDs).
__host__ __device__ inline int fs_rows(int T, int nx) { return T / fs_segs(nx); }
__host__ __device__ inline int fs_cols(int T, int ny, int M) {
    const int c = T / fs_segs(ny, M);
    return c >= 64 ? 64 : c >= 32 ? 32 : c >= 16 ? 16 : c >= 8 ? 8 : 4;
}
__host__ __device__ inline int fs_row_groups(int T, int nx, int ny) {
    const int r = fs_rows(T, nx);
    return ((ny + r - 1) / r + 7) / 8 * 8;
}
__host__ __device__ inline int fs_col_groups(int T, int nx, int ny) {
    const int c = fs_cols(T, ny, fs_m(ny));
    return (nx + c - 1) / c;
}
constexpr size_t fs_lds(int T) { return (size_t)T * FMP * sizeof(float); }

// One segment of M cells: cells i0 .. i0 + M - 1 of a line of n cells, dep[k]
// the still-water depth of cell i0 + k - 1, r the right-hand sides.
// Coefficients of eq. 23, and the elimination of the interior, every row
// divided by its diagonal (three arrays, not four): afterwards x_k = r_k -
// a_k x_first - c_k x_last for 1 <= k <= M - 2; f: x_first = f.z - f.x x_{-1} -
// f.y x_last; l: l.x x_first + l.y x_last + l.z x_{+1} = l.w.  The line's
// ends fold as in seg_coefs (glo, ghi: the maker's discharge change, 0 behind
// a wall), by selects: a branch had the compiler copy all the arrays.  Cells
// past the end need not be identity rows, as no cell of the line refers to
// them, but finite ones: the callers give them a depth of zero or the ghost's.  Coefficients and forward elimination go cell by cell, with a
// scheduling fence every few, so that the depths die as the rows are born.
template <int M>
__device__ __forceinline__ void fs_eliminate(TriK tk, int i0, int n, bool lo_wall, bool hi_wall, float glo, float ghi,
                                             const float (&dep)[M + 2], float (&a)[M], float (&c)[M], float (&r)[M],
                                             float3 &f, float4 &l) {
#pragma clang fp contract(off)
    const int kl = n - 1 - i0;  // the line's last cell
    const float hw = hi_wall ? 1.f : 0.f;
    float b0 = 1.f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const float dc = dep[k + 1], dd = dep[k + 2] - dep[k];
        const float al = tk.kal * (dc * dc), be = tk.kbe * (dc * dd);
        float ak = be - al, bk = fmaf(2.f, al, 1.f), ck = -be - al;
        const float cw = k == kl ? ck : 0.f;
        bk = fmaf(-cw, hw, bk);
        r[k] = fmaf(-cw, ghi, r[k]);
        ck -= cw;
        if (k == 0) {
            const float aw = i0 == 0 ? ak : 0.f;
            b0 = lo_wall ? bk - aw : bk;
            r[0] = fmaf(-aw, glo, r[0]);
            a[0] = ak - aw;
            c[0] = ck;
        } else if (k == M - 1) {
            l = make_float4(-ak * a[k - 1], fmaf(-ak, c[k - 1], bk), ck, fmaf(-ak, r[k - 1], r[k]));
        } else if (k == 1) {
            const float ib = frcp(bk);
            a[1] = ak * ib;
            c[1] = ck * ib;
            r[1] = r[1] * ib;
        } else {
            const float ib = frcp(fmaf(-ak, c[k - 1], bk)), m = ak * ib;
            a[k] = -m * a[k - 1];
            c[k] = ck * ib;
            r[k] = fmaf(-m, r[k - 1], r[k] * ib);
        }
        if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = M - 3; k >= 1; --k) {
        a[k] = fmaf(-c[k], a[k + 1], a[k]);
        r[k] = fmaf(-c[k], r[k + 1], r[k]);
        c[k] = -c[k] * c[k + 1];
    }
    const float inv = frcp(fmaf(-c[0], a[1], b0));
    f = make_float3(a[0] * inv, -c[0] * c[1] * inv, fmaf(-c[0], r[1], r[0]) * inv);
    __builtin_amdgcn_sched_barrier(0);
}

// The segments' equations across the lanes of a workgroup: segment s of nseg
// of a line, its neighbours `str` threads away.  Returns x_first and x_last.
// buf: 6 T floats.  Every thread of the workgroup calls it (nseg is uniform).
__device__ __forceinline__ float2 fs_reduced(float3 f, float4 l, int s, int nseg, int str, float *buf) {
#pragma clang fp contract(off)
    const int t = threadIdx.x, T = blockDim.x;
    float *cur = buf, *nxt = buf + 3 * T;
    auto put = [&](float *p, float x, float y, float z) {
        p[t] = x;
        p[T + t] = y;
        p[2 * T + t] = z;
    };
    auto get = [&](const float *p, int s2, int t2) {  // zeros past the line's ends
        const bool in = s2 >= 0 && s2 < nseg;
        const int q = in ? t2 : t;
        return make_float3(in ? p[q] : 0.f, in ? p[T + q] : 0.f, in ? p[2 * T + q] : 0.f);
    };
    put(cur, f.x, f.y, f.z);
    __syncthreads();
    const float3 n = get(cur, s + 1, t + str);  // first unknown of the next segment
    // l.x x_first + l.y x + l.z x_next_first = l.w with both firsts replaced
    float d = frcp(fmaf(-l.x, f.y, fmaf(-l.z, n.x, l.y)));
    float ea = -l.x * f.x * d, ec = -l.z * n.y * d, er = fmaf(-l.x, f.z, fmaf(-l.z, n.z, l.w)) * d;
    for (int st = 1; st < nseg; st <<= 1) {
        float *p = cur;
        cur = nxt;
        nxt = p;
        put(cur, ea, ec, er);
        __syncthreads();
        const float3 m = get(cur, s - st, t - st * str), q = get(cur, s + st, t + st * str);
        d = frcp(fmaf(-ea, m.y, fmaf(-ec, q.x, 1.f)));
        er = fmaf(-ea, m.z, fmaf(-ec, q.z, er)) * d;
        ea = -ea * m.x * d;
        ec = -ec * q.y * d;
    }
    nxt[t] = er;
    __syncthreads();
    const float xm = s > 0 ? nxt[t - str] : 0.f;  // last unknown of the segment before
    return make_float2(fmaf(-f.x, xm, fmaf(-f.y, er, f.z)), er);
}

template <int M>
__device__ __forceinline__ void fs_back(const float (&a)[M], const float (&c)[M], float (&r)[M], float2 x) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 1; k <= M - 2; ++k) r[k] = fmaf(-a[k], x.x, fmaf(-c[k], x.y, r[k]));
    r[0] = x.x;
    r[M - 1] = x.y;
    __builtin_amdgcn_sched_barrier(0);
}

// Depth of the ghost cell behind a wave-maker side: the side's corners held.
__device__ __forceinline__ float held_depth(const float *D, size_t c0, size_t c1) {
    return fmaxf(0.25f * ((D[c0] + D[c0]) + (D[c1] + D[c1])), 0.f);
}

template <bool EARLY>
__device__ __forceinline__ void solve_rows(const SolveArgs &A, float *lds, int T, int g) {
#pragma clang fp contract(off)
    const Dom &d = A.d;
    const int nseg = fs_segs(d.nx), R = fs_rows(T, d.nx);
    const int t = threadIdx.x, row = t / nseg, s = t - row * nseg, j = g * R + row;
    const bool live = row < R && j < d.ny;
    const int jl = live ? j : 0;
    const size_t o = (size_t)jl * d.pitch, oz = (size_t)jl * d.zpitch;
    // coalesced: thread (row, s) moves 16 bytes at cells 4 (s + m nseg)
    float4 vr[4], vd[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int q = 4 * (s + m * nseg);
        vr[m] = live ? *reinterpret_cast<const float4 *>(A.rx + o + q) : make_float4(0.f, 0.f, 0.f, 0.f);
        vd[m] = live ? *reinterpret_cast<const float4 *>(A.Dc + panel(q, jl, d.ny)) : make_float4(0.f, 0.f, 0.f, 0.f);
        // padding past the row's end is never written: whatever it holds must not spread
        // (the depths' holds other data, old corners after a terrain edit, whose pivots
        // can vanish)
        const bool in0 = q < d.nx, in1 = q + 1 < d.nx, in2 = q + 2 < d.nx, in3 = q + 3 < d.nx;
        vr[m] = make_float4(in0 ? vr[m].x : 0.f, in1 ? vr[m].y : 0.f, in2 ? vr[m].z : 0.f, in3 ? vr[m].w : 0.f);
        vd[m] = make_float4(in0 ? vd[m].x : 0.f, in1 ? vd[m].y : 0.f, in2 ? vd[m].z : 0.f, in3 ? vd[m].w : 0.f);
    }
    const int i0 = s * FM;
    float glo = 0.f, ghi = 0.f, dlo = 0.f, dhi = 0.f;  // maker changes and ghost depths of the row's ends
    if (live && s == 0 && !is_wall(d, 0)) {
        glo = A.gh1[ghost_index(d, 0, 0, j + 2) + 1] - A.gh0[ghost_index(d, 0, 0, j + 2) + 1];
        dlo = held_depth(d.D, oz, oz + d.zpitch);
    }
    if (live && s == nseg - 1 && !is_wall(d, 1)) {
        ghi = A.gh1[ghost_index(d, 1, 0, j + 2) + 1] - A.gh0[ghost_index(d, 1, 0, j + 2) + 1];
        dhi = held_depth(d.D, oz + d.nx, oz + d.zpitch + d.nx);
    }
    float *mine = lds + (size_t)(row < R ? row * nseg : 0) * FMP;  // the row's segments
    auto put4 = [&](const float4 (&v)[4]) {
        if (row < R)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int q = s + m * nseg;
                *reinterpret_cast<float4 *>(mine + (q >> 2) * FMP + 4 * (q & 3)) = v[m];
            }
    };
    float dep[FM + 2], r[FM], a[FM], c[FM];
    put4(vd);
    __syncthreads();
    const float *seg = mine + (row < R ? s : 0) * FMP;
#pragma unroll
    for (int k = 0; k < FM; k += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(seg + k);
        dep[k + 1] = fmaxf(v.x, 0.f);
        dep[k + 2] = fmaxf(v.y, 0.f);
        dep[k + 3] = fmaxf(v.z, 0.f);
        dep[k + 4] = fmaxf(v.w, 0.f);
    }
    dep[0] = s > 0 && row < R ? fmaxf(seg[FM - 1 - FMP], 0.f) : is_wall(d, 0) ? dep[1] : dlo;
    dep[FM + 1] = s < nseg - 1 && row < R ? fmaxf(seg[FMP], 0.f) : 0.f;
    __syncthreads();
    put4(vr);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < FM; k += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(seg + k);
        r[k] = v.x;
        r[k + 1] = v.y;
        r[k + 2] = v.z;
        r[k + 3] = v.w;
    }
    {   // the ghost past the row's last cell: mirrored, or held behind a maker
        const int kl = d.nx - 1 - i0;
        const bool wall = is_wall(d, 1);
#pragma unroll
        for (int k = 0; k < FM; ++k) {
            const float gd = wall ? dep[k + 1] : dhi;
            dep[k + 2] = k == kl ? gd : dep[k + 2];
        }
    }
    __syncthreads();
    float3 f;
    float4 l;
    fs_eliminate<FM>(tri_k(d.Bd, d.rdx), i0, d.nx, is_wall(d, 0), is_wall(d, 1), glo, ghi, dep, a, c, r, f, l);
    float4 vp[4], ve[4];
    auto epilogue_loads = [&] {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int q = 4 * (s + m * nseg);
            vp[m] = live ? *reinterpret_cast<const float4 *>(A.pbase + o + q) : make_float4(0.f, 0.f, 0.f, 0.f);
            ve[m] = live ? *reinterpret_cast<const float4 *>(A.eraw + o + q) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    if (EARLY) epilogue_loads();
    const float2 x = fs_reduced(f, l, s, nseg, 1, lds);
    fs_back(a, c, r, x);
    __syncthreads();
    if (row < R)
#pragma unroll
        for (int k = 0; k < FM; k += 4)
            *reinterpret_cast<float4 *>(const_cast<float *>(seg) + k) = make_float4(r[k], r[k + 1], r[k + 2], r[k + 3]);
    if (!EARLY) epilogue_loads();
    const float *gx = A.Dc + (size_t)d.ny * d.zpitch;  // sponge factors of the columns
    const float gy = A.sponge && live ? A.Dc[panel(d.nx, jl, d.ny)] : 1.f;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int q = 4 * (s + m * nseg);
        vd[m] = live ? *reinterpret_cast<const float4 *>(A.Dc + panel(q, jl, d.ny)) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    int bad = 0;
    if (live)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int qs = s + m * nseg, i = 4 * qs;
            const float4 dx = *reinterpret_cast<const float4 *>(mine + (qs >> 2) * FMP + 4 * (qs & 3));
            float4 P = make_float4(vp[m].x + dx.x, vp[m].y + dx.y, vp[m].z + dx.z, vp[m].w + dx.w), e = ve[m];
            const float4 D = vd[m];
            const bool i1 = i + 1 < d.nx, i2 = i + 2 < d.nx, i3 = i + 3 < d.nx;
            P.x = shore(P.x, e.x, D.x, d.eps);
            P.y = shore(P.y, e.y, D.y, d.eps);
            P.z = shore(P.z, e.z, D.z, d.eps);
            P.w = shore(P.w, e.w, D.w, d.eps);
            if (A.sponge) {
                const float4 g4 = *reinterpret_cast<const float4 *>(gx + i);
                const float m0 = D.x > 0.f ? g4.x * gy : 1.f, m1 = D.y > 0.f ? g4.y * gy : 1.f;
                const float m2 = D.z > 0.f ? g4.z * gy : 1.f, m3 = D.w > 0.f ? g4.w * gy : 1.f;
                P = make_float4(P.x * m0, P.y * m1, P.z * m2, P.w * m3);
                e = make_float4(e.x * m0, e.y * m1, e.z * m2, e.w * m3);
            }
            bad |= i < d.nx && !(isfinite(P.x) && isfinite(e.x));
            bad |= i1 && !(isfinite(P.y) && isfinite(e.y));
            bad |= i2 && !(isfinite(P.z) && isfinite(e.z));
            bad |= i3 && !(isfinite(P.w) && isfinite(e.w));
            auto store = [&](float *p, float4 v) {
                if (i3) {
                    *reinterpret_cast<float4 *>(p + i) = v;
                } else {
                    if (i < d.nx) p[i] = v.x;
                    if (i1) p[i + 1] = v.y;
                    if (i2) p[i + 2] = v.z;
                }
            };
            store(A.pout + o, P);
            if (A.sponge) store(A.eta + o, e);
        }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(A.health, 1);
}

template <int M, bool EARLY>
__device__ __forceinline__ void solve_cols(const SolveArgs &A, float *lds, int T, int g) {
#pragma clang fp contract(off)
    const Dom &d = A.d;
    const int nseg = fs_segs(d.ny, M), C = fs_cols(T, d.ny, M);
    const int t = threadIdx.x, s = t / C, i = g * C + (t & (C - 1)), j0 = s * M;
    const bool live = s < nseg && i < d.nx;
    const int ic = live ? i : 0, jc = live ? j0 : 0, kl = d.ny - 1 - jc;  // kl: the column's last cell
    // one lane offset per layout and uniform row offsets (a lane offset per row
    // cost 34 registers); what lies past the column's end is other data of
    // the workspace, and replaced
    const unsigned pb = 4u * (unsigned)d.pitch;
    const auto br = bres(ldp(A.rx, A.fstride), A.fstride), bd = bres(A.Dc, 4u * (unsigned)d.zpitch * (unsigned)(d.ny + 1));
    const auto bq = bres(ldp(A.pbase, A.fstride), A.fstride), be = bres(A.eraw, A.fstride);
    const auto bo = bres(ldp(A.pout, A.fstride), A.fstride);
    const unsigned vo = (unsigned)jc * pb + 4u * (unsigned)ic, vp = 4u * panel(ic, jc, d.ny);
    float dep[M + 2], r[M], a[M], c[M];
#pragma unroll
    for (int k = 0; k < M; ++k) r[k] = bld(br, vo, k * pb);
    dep[0] = bld(bd, jc > 0 ? vp - 32u : vp, 0);
#pragma unroll
    for (int k = 0; k < M + 1; ++k) dep[k + 1] = bld(bd, vp + 32u * k, 0);
    float glo = 0.f, ghi = 0.f, dlo = 0.f, dhi = 0.f;
    const bool lo_wall = is_wall(d, 2), hi_wall = is_wall(d, 3);
    if (!lo_wall && live && s == 0) {
        glo = A.gh1[ghost_index(d, 2, 0, i + 2) + 2] - A.gh0[ghost_index(d, 2, 0, i + 2) + 2];
        dlo = 0.25f * ((d.D[i] + d.D[i + 1]) + (d.D[i] + d.D[i + 1]));
    }
    if (!hi_wall && live && kl < M) {
        ghi = A.gh1[ghost_index(d, 3, 0, i + 2) + 2] - A.gh0[ghost_index(d, 3, 0, i + 2) + 2];
        const float *Dn = d.D + (size_t)d.ny * d.zpitch;
        dhi = 0.25f * ((Dn[i] + Dn[i + 1]) + (Dn[i] + Dn[i + 1]));
    }
    dep[0] = jc > 0 || lo_wall ? dep[0] : dlo;  // walls: the first and last cells' own depths
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const float gd = hi_wall ? dep[k + 1] : dhi;
        dep[k + 2] = k < kl ? dep[k + 2] : gd;
        r[k] = k <= kl ? r[k] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < M + 2; ++k) dep[k] = fmaxf(dep[k], 0.f);
    float3 f;
    float4 l;
    fs_eliminate<M>(tri_k(d.Bd, d.rdy), jc, d.ny, lo_wall, hi_wall, glo, ghi, dep, a, c, r, f, l);
    // the epilogue goes EP rows at a time
    constexpr int EP = 16;
    float vq[EP], ve[EP], vd[EP];
    auto epilogue_loads = [&](int k0) {
#pragma unroll
        for (int k = 0; k < EP; ++k) {
            vq[k] = bld(bq, vo, (k0 + k) * pb);
            ve[k] = bld(be, vo, (k0 + k) * pb);
            vd[k] = bld(bd, vp + 32u * (k0 + k), 0);
        }
    };
    if (EARLY) epilogue_loads(0);
    const float2 x = fs_reduced(f, l, s, nseg, C, lds);
    if (!live) return;
    fs_back(a, c, r, x);
    const float gx = A.sponge ? A.Dc[(size_t)d.ny * d.zpitch + i] : 1.f;
    int bad = 0;
#pragma unroll
    for (int k0 = 0; k0 < M; k0 += EP) {
        if (!EARLY || k0 > 0) epilogue_loads(k0);
#pragma unroll
        for (int k = 0; k < EP; ++k) r[k0 + k] = shore(vq[k] + r[k0 + k], ve[k], vd[k], d.eps);
        if (A.sponge) {
            float gy[EP];
#pragma unroll
            for (int k = 0; k < EP; ++k)
                gy[k] = A.Dc[panel(d.nx, min(jc + k0 + k, d.ny - 1), d.ny)];
#pragma unroll
            for (int k = 0; k < EP; ++k) r[k0 + k] *= vd[k] > 0.f ? gx * gy[k] : 1.f;
        }
        // all values before the first store: left to itself the compiler moves
        // each row's loads and arithmetic under its store's condition, sixteen
        // round trips to memory in a row
#pragma unroll
        for (int k = 0; k < EP; ++k) asm volatile("" : "+v"(r[k0 + k]));
#pragma unroll
        for (int k = 0; k < EP; ++k)
            if (k0 + k <= kl) {
                bad |= !isfinite(r[k0 + k]);
                bst(bo, vo, (k0 + k) * pb, r[k0 + k]);
            }
    }
    // lanes that left are not in the vote; one lane of those here reports
    const unsigned long long v = __ballot(bad);
    if (v && (int)(threadIdx.x & 63) == __ffsll((long long)v) - 1) atomicOr(A.health, 1);
}

// Row workgroups first, then column workgroups.  Consecutive ones go to one
// XCD: neighbouring columns share 128-byte lines of the row-major fields,
// neighbouring rows those of the depth panels.
template <bool EARLY, bool TALL = false>
__device__ __forceinline__ void solve_body(const SolveArgs &A, float *lds, int b) {
    const int T = blockDim.x, nr = fs_row_groups(T, A.d.nx, A.d.ny), nc = fs_col_groups(T, A.d.nx, A.d.ny);
    if (b < nr) {
        const int g = xcd_order(b, nr);
        if (g * fs_rows(T, A.d.nx) < A.d.ny) solve_rows<EARLY>(A, lds, T, g);
    } else if (TALL && A.d.ny > FS_TALL) {
        solve_cols<FMT, EARLY>(A, lds, T, xcd_order(b - nr, nc));
    } else {
        solve_cols<FM, EARLY>(A, lds, T, xcd_order(b - nr, nc));
    }
}

// Up to FS_EARLY threads the registers suffice to have the epilogue's loads in
// flight across the reduction, which a small grid's few waves need: 128 x 64
// cells 10.5 -> 9.8 us, 1024 x 512 12.8 -> 12.3.  Larger workgroups load late.
constexpr int FS_EARLY = 512;
__global__ __launch_bounds__(FS_EARLY) __attribute__((amdgpu_waves_per_eu(4))) void k_solve(SolveArgs A) {
    extern __shared__ __align__(16) float fs_buf[];
    solve_body<true>(A, fs_buf, blockIdx.x);
}
__global__ __launch_bounds__(1024) void k_solve_big(SolveArgs A) {
    extern __shared__ __align__(16) float fs_buf[];
    solve_body<false>(A, fs_buf, blockIdx.x);
}
__global__ __launch_bounds__(FS_EARLY) void k_solve_tall(SolveArgs A) {
    extern __shared__ __align__(16) float fs_buf[];
    solve_body<true, true>(A, fs_buf, blockIdx.x);
}
// Wider grids, at 8 columns a run: columns of more than FS_TALL cells fill a
// CU's registers with one workgroup (128 a lane, 6 more spilled to 28 bytes of
// scratch), so the rows get a launch of their own, with small workgroups.
__global__ __launch_bounds__(1024) void k_solve_rows(SolveArgs A) {
    extern __shared__ __align__(16) float fs_buf[];
    solve_rows<false>(A, fs_buf, blockDim.x, xcd_order(blockIdx.x, gridDim.x));
}
__global__ __launch_bounds__(1024) void k_solve_cols(SolveArgs A) {
    extern __shared__ __align__(16) float fs_buf[];
    solve_cols<FMT, false>(A, fs_buf, blockDim.x, xcd_order(blockIdx.x, gridDim.x));
}

}  // namespace ws
