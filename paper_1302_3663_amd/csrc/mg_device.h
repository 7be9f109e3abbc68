// Device code shared by the multigrid translation units: the rows of the two
// operators, the taps of the transfers, and the passes of a V-cycle inside
// one workgroup.
//
// Multiply-adds are fused only inside one source expression, never across
// statements, so a row computes the same bits in every kernel that inlines
// it (the launched passes, the one-workgroup coarse cycle and the bricks).
#pragma once

#include "common.h"
#include "kernels.h"

#pragma clang fp contract(on)

namespace ibmg {

// ---------------------------------------------------------------------------
// rows of the two operators: (A x) at one unknown and the diagonal entry.
// Templated on the dimension D and (viscous) the component A so that every
// loop unrolls and all loads of a row issue together.
// ---------------------------------------------------------------------------
__device__ inline int self_sign(Ref r, long long c) { return (r.s != 0 && r.idx == c) ? r.s : 0; }

// the bi-th axis other than A
template <int A>
__device__ constexpr int other_axis(int bi) { return bi < A ? bi : bi + 1; }

template <typename T, int D>
__device__ inline void p_row_slow(const Grid &g, const T *__restrict__ x, const CoefP<T> &cf, T cvisc, int i, int j,
                                  int k, T &Ax, T &dg)
{
    const long long c = at(g, i, j, k);
    Ref rb[2 * D], rx[2 * D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        int qp[3] = {i, j, k}, qm[3] = {i, j, k};
        qp[a] += 1;
        qm[a] -= 1;
        rb[2 * a] = ref_at(g, face_mask(a), ROLE_C, qp[0], qp[1], qp[2]);
        rb[2 * a + 1] = ref_at(g, face_mask(a), ROLE_C, i, j, k);
        rx[2 * a] = ref_at(g, 0, ROLE_P, qp[0], qp[1], qp[2]);
        rx[2 * a + 1] = ref_at(g, 0, ROLE_P, qm[0], qm[1], qm[2]);
    }
    T bt[2 * D], xn[2 * D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        bt[2 * a] = ld(cf.beta[a], rb[2 * a]);
        bt[2 * a + 1] = ld(cf.beta[a], rb[2 * a + 1]);
        xn[2 * a] = ld(x, rx[2 * a]);
        xn[2 * a + 1] = ld(x, rx[2 * a + 1]);
    }
    const T xc = x[c];
    T acc = 0, d = 0;
#pragma unroll
    for (int t = 0; t < 2 * D; ++t) {
        acc += bt[t] * (xc - xn[t]);
        d += bt[t] * T(1 - self_sign(rx[t], c));
    }
    Ax = acc * cvisc;
    dg = d * cvisc;
}

// Constant viscosity, eq:NSdis1: the 2D + 1 point Laplacian of component A
// alone with unit coefficients (the viscosity is folded into cvisc), every
// neighbour resolved through the boundary rules.
template <typename T, int D, int A>
__device__ inline void u_row_slow_dec(const Grid &g, const T *__restrict__ ua, const T *__restrict__ rho, T mass,
                                      T cvisc, int i, int j, int k, T &Ax, T &dg)
{
    const long long f = at(g, i, j, k);
    const int ma = face_mask(A);
    Ref rp[D], rm[D];
#pragma unroll
    for (int b = 0; b < D; ++b) {
        int qp[3] = {i, j, k}, qm[3] = {i, j, k};
        qp[b] += 1;
        qm[b] -= 1;
        rp[b] = ref_at(g, ma, ROLE_V, qp[0], qp[1], qp[2]);
        rm[b] = ref_at(g, ma, ROLE_V, qm[0], qm[1], qm[2]);
    }
    const T xf = ua[f];
    T acc = 0, d = 0;
#pragma unroll
    for (int b = 0; b < D; ++b) {
        acc += (ld(ua, rp[b]) - xf) - (xf - ld(ua, rm[b]));
        d += T(1 - self_sign(rp[b], f)) + T(1 - self_sign(rm[b], f));
    }
    const T m = mass * rho[f];
    Ax = m * xf - cvisc * acc;
    dg = m + cvisc * d;
}

template <typename T, int D, int A>
__device__ inline void u_row_slow(const Grid &g, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc, int i, int j,
                                  int k, T &Ax, T &dg)
{
    if (cf.dec) {
        u_row_slow_dec<T, D, A>(g, x.c[A], cf.rho[A], mass, cvisc, i, j, k, Ax, dg);
        return;
    }
    const int q[3] = {i, j, k};
    const long long f = at(g, i, j, k);
    const int ma = face_mask(A);
    int qa_m[3] = {i, j, k}, qa_p[3] = {i, j, k};
    qa_m[A] -= 1;
    qa_p[A] += 1;
    // resolve every reference first (arithmetic only)
    const Ref rcp = ref_at(g, 0, ROLE_C, i, j, k);
    const Ref rcm = ref_at(g, 0, ROLE_C, qa_m[0], qa_m[1], qa_m[2]);
    const Ref rvp = ref_at(g, ma, ROLE_V, qa_p[0], qa_p[1], qa_p[2]);
    const Ref rvm = ref_at(g, ma, ROLE_V, qa_m[0], qa_m[1], qa_m[2]);
    Ref rmp[D - 1], rmm[D - 1], rap[D - 1], ram[D - 1], r0[D - 1], r1[D - 1], r2[D - 1], r3[D - 1];
#pragma unroll
    for (int bi = 0; bi < D - 1; ++bi) {
        const int B = other_axis<A>(bi);
        const int c = 3 - A - B;
        const int mb = face_mask(B), mem = edge_mask(D, c);
        int qb_p[3] = {q[0], q[1], q[2]}, qb_m[3] = {q[0], q[1], q[2]};
        qb_p[B] += 1;
        qb_m[B] -= 1;
        int qbp_am[3] = {qb_p[0], qb_p[1], qb_p[2]};
        qbp_am[A] -= 1;
        rmp[bi] = ref_at(g, mem, ROLE_C, qb_p[0], qb_p[1], qb_p[2]);
        rmm[bi] = ref_at(g, mem, ROLE_C, i, j, k);
        rap[bi] = ref_at(g, ma, ROLE_V, qb_p[0], qb_p[1], qb_p[2]);
        ram[bi] = ref_at(g, ma, ROLE_V, qb_m[0], qb_m[1], qb_m[2]);
        r0[bi] = ref_at(g, mb, ROLE_V, qb_p[0], qb_p[1], qb_p[2]);
        r1[bi] = ref_at(g, mb, ROLE_V, qbp_am[0], qbp_am[1], qbp_am[2]);
        r2[bi] = ref_at(g, mb, ROLE_V, i, j, k);
        r3[bi] = ref_at(g, mb, ROLE_V, qa_m[0], qa_m[1], qa_m[2]);
    }
    // then every load
    const T *__restrict__ ua = x.c[A];
    const T xf = ua[f];
    const T rho = cf.rho[A][f];
    const T cp = T(2) * ld(cf.muc, rcp), cm = T(2) * ld(cf.muc, rcm);
    const T vp = ld(ua, rvp), vm = ld(ua, rvm);
    T mp[D - 1], mm[D - 1], ap[D - 1], am[D - 1], b0[D - 1], b1[D - 1], b2[D - 1], b3[D - 1];
#pragma unroll
    for (int bi = 0; bi < D - 1; ++bi) {
        const int B = other_axis<A>(bi);
        const T *__restrict__ ub = x.c[B];
        const T *__restrict__ me = cf.mue[3 - A - B];
        mp[bi] = ld(me, rmp[bi]);
        mm[bi] = ld(me, rmm[bi]);
        ap[bi] = ld(ua, rap[bi]);
        am[bi] = ld(ua, ram[bi]);
        b0[bi] = ld(ub, r0[bi]);
        b1[bi] = ld(ub, r1[bi]);
        b2[bi] = ld(ub, r2[bi]);
        b3[bi] = ld(ub, r3[bi]);
    }
    T acc = cp * (vp - xf) - cm * (xf - vm);
    T d = cp * T(1 - self_sign(rvp, f)) + cm * T(1 - self_sign(rvm, f));
#pragma unroll
    for (int bi = 0; bi < D - 1; ++bi) {
        acc += mp[bi] * ((ap[bi] - xf) + (b0[bi] - b1[bi])) - mm[bi] * ((xf - am[bi]) + (b2[bi] - b3[bi]));
        d += mp[bi] * T(1 - self_sign(rap[bi], f)) + mm[bi] * T(1 - self_sign(ram[bi], f));
    }
    const T m = mass * rho;
    Ax = m * xf - cvisc * acc;
    dg = m + cvisc * d;
}

// Rows read through the ghost layer: every neighbour sits at a fixed
// offset.  Where the ghost across a boundary mirrors the point itself, the
// diagonal gains the reflection: coefficient x (1 - sign) instead of the
// coefficient alone.  The arithmetic of a row stands apart from its loads,
// so that every reader of the fields (uniform arrays, windows in LDS)
// computes the same bits.

// where a point lies along each axis: lo, hi: first or last cell position of
// an axis that does not wrap; walls: its ends are both walls
struct Edge {
    const Grid &g;
    int q[3];
    __device__ bool lo(int d) const { return g.bc[d] != AX_PERIODIC && q[d] == 0; }
    __device__ bool hi(int d) const { return g.bc[d] != AX_PERIODIC && q[d] == g.n[d] - 1; }
    __device__ bool walls(int d) const { return g.bc[d] == AX_WALLS; }
};

// pressure: xc the value at the cell, xn and bt its neighbours and the face
// coefficients towards them (per axis: above, below)
template <typename T, int D, typename E>
__device__ inline void p_row_math(const E &q, T xc, const T *xn, const T *bt, T cvisc, T &Ax, T &dg)
{
    T acc = 0, d = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        acc += bt[2 * a] * (xc - xn[2 * a]) + bt[2 * a + 1] * (xc - xn[2 * a + 1]);
        d += bt[2 * a] + bt[2 * a + 1];
        if (q.lo(a)) d -= bt[2 * a + 1];                                // even mirror
        if (q.hi(a)) d += q.walls(a) ? -bt[2 * a] : bt[2 * a];          // odd at the outflow
    }
    Ax = acc * cvisc;
    dg = d * cvisc;
}

// constant viscosity: component A alone, vp and vm its neighbours per axis
template <typename T, int D, int A, typename E>
__device__ inline void u_row_dec_math(const E &q, T xf, const T *vp, const T *vm, T r, T mass, T cvisc,
                                      T &Ax, T &dg)
{
    T acc = 0, d = T(2 * D);
#pragma unroll
    for (int b = 0; b < D; ++b) {
        acc += (vp[b] - xf) - (xf - vm[b]);
        if (b != A) {
            if (q.lo(b)) d += T(1);                                // odd mirror
            if (q.hi(b)) d += q.walls(b) ? T(1) : T(-1);           // even at the outflow
        }
    }
    const T m = mass * r;
    Ax = m * xf - cvisc * acc;
    dg = m + cvisc * d;
}

// What a coupled viscous row reads besides its own value, for component A:
// the cell viscosities above and below (cu, cl), the neighbours along A (vp,
// vm), and per other axis B the edge viscosities (mp, mm), the neighbours
// along B (ap, am) and the four u_B around the face.
template <typename T, int D>
struct URow {
    T cu, cl, vp, vm;
    T mp[D - 1], mm[D - 1], ap[D - 1], am[D - 1], b0[D - 1], b1[D - 1], b2[D - 1], b3[D - 1];
};

template <typename T, int D, int A, typename E>
__device__ inline void u_row_math(const E &q, T xf, const URow<T, D> &r, T rho, T mass, T cvisc, T &Ax,
                                  T &dg)
{
    const T cp = T(2) * r.cu, cm = T(2) * r.cl;
    T acc = cp * (r.vp - xf) - cm * (xf - r.vm);
    T d = cp + cm;
#pragma unroll
    for (int bi = 0; bi < D - 1; ++bi) {
        const int B = other_axis<A>(bi);
        acc += r.mp[bi] * ((r.ap[bi] - xf) + (r.b0[bi] - r.b1[bi])) - r.mm[bi] * ((xf - r.am[bi]) + (r.b2[bi] - r.b3[bi]));
        d += r.mp[bi] + r.mm[bi];
        if (q.lo(B)) d += r.mm[bi];                                // odd mirror
        if (q.hi(B)) d += q.walls(B) ? r.mp[bi] : -r.mp[bi];       // even at the outflow
    }
    const T m = mass * rho;
    Ax = m * xf - cvisc * acc;
    dg = m + cvisc * d;
}

template <typename T, int D>
__device__ inline void p_row(const Grid &g, const T *__restrict__ x, const CoefP<T> &cf, T cvisc, int i, int j, int k,
                             T &Ax, T &dg)
{
    const int c = (int)at(g, i, j, k);
    const int st[3] = {1, g.NX, (int)g.NXY};
    T xn[2 * D], bt[2 * D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        xn[2 * a] = x[c + st[a]];
        xn[2 * a + 1] = x[c - st[a]];
        bt[2 * a] = cf.beta[a][c + st[a]];
        bt[2 * a + 1] = cf.beta[a][c];
    }
    p_row_math<T, D>(Edge{g, {i, j, k}}, x[c], xn, bt, cvisc, Ax, dg);
}

// Constant viscosity through the ghost layer: component A alone, unit
// coefficients; a mirrored self-reference adds to the diagonal as in u_row.
// (r: the density at the face, read by the caller)
template <typename T, int D, int A>
__device__ inline void u_row_dec_r(const Grid &g, const T *__restrict__ ua, T r, T mass, T cvisc, int i, int j, int k,
                                   T &Ax, T &dg)
{
    const int f = (int)at(g, i, j, k);
    const int st[3] = {1, g.NX, (int)g.NXY};
    T vp[D], vm[D];
#pragma unroll
    for (int b = 0; b < D; ++b) {
        vp[b] = ua[f + st[b]];
        vm[b] = ua[f - st[b]];
    }
    u_row_dec_math<T, D, A>(Edge{g, {i, j, k}}, ua[f], vp, vm, r, mass, cvisc, Ax, dg);
}

template <typename T, int D, int A>
__device__ inline void u_row_dec(const Grid &g, const T *__restrict__ ua, const T *__restrict__ rho, T mass, T cvisc,
                                 int i, int j, int k, T &Ax, T &dg)
{
    u_row_dec_r<T, D, A>(g, ua, rho[at(g, i, j, k)], mass, cvisc, i, j, k, Ax, dg);
}

// u_a at the row's point and its axis neighbours, read from the uniform
// array at fixed offsets
template <typename T>
struct UaFlat {
    const T *__restrict__ p;
    int f;
    int st[3];
    __device__ T here() const { return p[f]; }
    __device__ T nb(int ax, int s) const { return p[f + s * st[ax]]; }
};

// The coupled viscous row (eq:NSdis1-1 with eq:divergencePartial) at uniform
// entry f, lattice position (i, j, k), with u_a read through `ua` (the
// uniform array, or a window of it) and every other field through f.  One
// body for every reader, so that all of them compute the same bits.
template <typename T, int D, int A, typename UA, typename XV>
__device__ inline void u_row_core(const Grid &g, const UA &ua, const XV &x, const CoefU<T> &cf, T rho, T mass, T cvisc,
                                  int f, int i, int j, int k, T &Ax, T &dg)
{
    const int st[3] = {1, g.NX, (int)g.NXY};
    const int sa = st[A];
    const T xf = ua.here();
    URow<T, D> r;
    r.cu = cf.muc[f];
    r.cl = cf.muc[f - sa];
    r.vp = ua.nb(A, 1);
    r.vm = ua.nb(A, -1);
#pragma unroll
    for (int bi = 0; bi < D - 1; ++bi) {
        const int B = other_axis<A>(bi);
        const int sb = st[B];
        const T *__restrict__ ub = x.c[B];
        const T *__restrict__ me = cf.mue[3 - A - B];
        r.mp[bi] = me[f + sb];
        r.mm[bi] = me[f];
        r.ap[bi] = ua.nb(B, 1);
        r.am[bi] = ua.nb(B, -1);
        r.b0[bi] = ub[f + sb];
        r.b1[bi] = ub[f + sb - sa];
        r.b2[bi] = ub[f];
        r.b3[bi] = ub[f - sa];
    }
    u_row_math<T, D, A>(Edge{g, {i, j, k}}, xf, r, rho, mass, cvisc, Ax, dg);
}

template <typename T, int D, int A>
__device__ inline void u_row(const Grid &g, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc, int i, int j,
                             int k, T &Ax, T &dg)
{
    const int f = (int)at(g, i, j, k);
    // read before the branch, which both forms take it in
    const T rho = cf.rho[A][f];
    if (cf.dec) {
        u_row_dec_r<T, D, A>(g, x.c[A], rho, mass, cvisc, i, j, k, Ax, dg);
        return;
    }
    const UaFlat<T> ua{x.c[A], f, {1, g.NX, (int)g.NXY}};
    u_row_core<T, D, A>(g, ua, x, cf, rho, mass, cvisc, f, i, j, k, Ax, dg);
}

// runtime-dimension entry points (coarsest dense assembly)
template <typename T>
__device__ inline void p_row_slow_any(const Grid &g, const T *x, const CoefP<T> &cf, T cvisc, int i, int j, int k, T &Ax,
                                      T &dg)
{
    if (g.D == 3) p_row_slow<T, 3>(g, x, cf, cvisc, i, j, k, Ax, dg);
    else p_row_slow<T, 2>(g, x, cf, cvisc, i, j, k, Ax, dg);
}

template <typename T>
__device__ inline void u_row_slow_any(const Grid &g, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc, int a,
                                      int i, int j, int k, T &Ax, T &dg)
{
    if (g.D == 3) {
        if (a == 0) u_row_slow<T, 3, 0>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
        else if (a == 1) u_row_slow<T, 3, 1>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
        else u_row_slow<T, 3, 2>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
    } else {
        if (a == 0) u_row_slow<T, 2, 0>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
        else u_row_slow<T, 2, 1>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
    }
}

// ---------------------------------------------------------------------------
// transfers
// ---------------------------------------------------------------------------
// Per-axis taps of a transfer, resolved through the boundary rules once per
// axis: index along the axis, sign, and weight (zero for a fixed face).
struct AxisTaps {
    int q[4];
    double w[4];
};

template <int NT>
__device__ inline void resolve_taps(const Grid &g, int d, int vert, int role, const int *raw, const double *wraw,
                                    AxisTaps &t)
{
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        int q = raw[a], s = 1;
        const bool live = resolve(g, d, vert, role, q, s);
        t.q[a] = live ? q : 0;
        t.w[a] = live ? (s > 0 ? wraw[a] : -wraw[a]) : 0.0;
    }
}

// The first step of full weighting: along x on one fine line src(i) around the
// coarse index I.  The bricks send these sums to the workgroups that weight
// the lines; the other passes take restrict_point, which adds in this order.
template <int VX, typename SRC>
__device__ inline double restrict_line(const Grid &gf, int role, int I, SRC src)
{
    constexpr int N0 = VX ? 3 : 4;
    AxisTaps t;
    int raw[4];
    double wr[4];
    rst_weights(VX, I, raw, wr);
    resolve_taps<N0>(gf, 0, VX, role, raw, wr, t);
    double v[N0], rs = 0.0;
#pragma unroll
    for (int a = 0; a < N0; ++a) v[a] = (double)src(t.q[a]);
#pragma unroll
    for (int a = 0; a < N0; ++a) rs += t.w[a] * v[a];
    return rs;
}

// both steps at once, every load before the first sum (the same sums)
template <typename T, int D, int VM>
__device__ inline double restrict_point(const Grid &gf, int role, const T *__restrict__ src, int I, int J, int K)
{
    constexpr int N0 = (VM & 1) ? 3 : 4;
    constexpr int N1 = (VM & 2) ? 3 : 4;
    constexpr int N2 = D == 3 ? ((VM & 4) ? 3 : 4) : 1;
    const int Q[3] = {I, J, K};
    AxisTaps t[3];
    int raw[4];
    double wr[4];
    rst_weights(VM & 1, Q[0], raw, wr);
    resolve_taps<N0>(gf, 0, VM & 1, role, raw, wr, t[0]);
    rst_weights((VM >> 1) & 1, Q[1], raw, wr);
    resolve_taps<N1>(gf, 1, (VM >> 1) & 1, role, raw, wr, t[1]);
    if (D == 3) {
        rst_weights((VM >> 2) & 1, Q[2], raw, wr);
        resolve_taps<N2>(gf, 2, (VM >> 2) & 1, role, raw, wr, t[2]);
    } else {
        t[2].q[0] = 0;
        t[2].w[0] = 1.0;
    }
    T v[N2][N1][N0];
#pragma unroll
    for (int c = 0; c < N2; ++c)
#pragma unroll
        for (int b = 0; b < N1; ++b)
#pragma unroll
            for (int a = 0; a < N0; ++a) v[c][b][a] = src[at(gf, t[0].q[a], t[1].q[b], t[2].q[c])];
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < N2; ++c)
#pragma unroll
        for (int b = 0; b < N1; ++b) {
            double rs = 0.0;
#pragma unroll
            for (int a = 0; a < N0; ++a) rs += t[0].w[a] * (double)v[c][b][a];
            s += t[1].w[b] * t[2].w[c] * rs;
        }
    return s;
}

// linear interpolation of the coarse values src at fine point (i, j, k)
template <typename T, int D, int VM>
__device__ inline double prolong_point(const Grid &gc, int role, const T *__restrict__ src, int i, int j, int k)
{
    constexpr int N2 = D == 3 ? 2 : 1;
    const int q[3] = {i, j, k};
    AxisTaps t[3];
    int raw[2];
    double wr[2];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int vert = (VM >> d) & 1;
        const int n = prl_weights(vert, q[d], raw, wr);
        if (n == 1) { raw[1] = raw[0]; wr[1] = 0.0; }
        resolve_taps<2>(gc, d, vert, role, raw, wr, t[d]);
    }
    if (D == 2) {
        t[2].q[0] = 0;
        t[2].w[0] = 1.0;
    }
    T v[N2][2][2];
#pragma unroll
    for (int c = 0; c < N2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) v[c][b][a] = src[at(gc, t[0].q[a], t[1].q[b], t[2].q[c])];
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < N2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) s += t[0].w[a] * t[1].w[b] * t[2].w[c] * (double)v[c][b][a];
    return s;
}

template <typename T, int D>
__device__ inline double restrict_any(int vm, const Grid &gf, int role, const T *src, int I, int J, int K)
{
    switch (vm) {
    case 0: return restrict_point<T, D, 0>(gf, role, src, I, J, K);
    case 1: return restrict_point<T, D, 1>(gf, role, src, I, J, K);
    case 2: return restrict_point<T, D, 2>(gf, role, src, I, J, K);
    case 3: return restrict_point<T, D, 3>(gf, role, src, I, J, K);
    case 4: return restrict_point<T, D, 4>(gf, role, src, I, J, K);
    case 5: return restrict_point<T, D, 5>(gf, role, src, I, J, K);
    case 6: return restrict_point<T, D, 6>(gf, role, src, I, J, K);
    default: return restrict_point<T, D, 7>(gf, role, src, I, J, K);
    }
}

template <typename T, int D>
__device__ inline double prolong_any(int vm, const Grid &gc, int role, const T *src, int i, int j, int k)
{
    switch (vm) {
    case 0: return prolong_point<T, D, 0>(gc, role, src, i, j, k);
    case 1: return prolong_point<T, D, 1>(gc, role, src, i, j, k);
    case 2: return prolong_point<T, D, 2>(gc, role, src, i, j, k);
    case 3: return prolong_point<T, D, 3>(gc, role, src, i, j, k);
    case 4: return prolong_point<T, D, 4>(gc, role, src, i, j, k);
    case 5: return prolong_point<T, D, 5>(gc, role, src, i, j, k);
    case 6: return prolong_point<T, D, 6>(gc, role, src, i, j, k);
    default: return prolong_point<T, D, 7>(gc, role, src, i, j, k);
    }
}

// ---------------------------------------------------------------------------
// the coarse part of a V-cycle in one workgroup
// ---------------------------------------------------------------------------
template <typename T>
__device__ inline CoefU<T> coef_u(const LevTab<T> &lt)
{
    CoefU<T> cf;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cf.rho[a] = lt.rho[a];
        cf.mue[a] = lt.mue[a];
    }
    cf.muc = lt.muc;
    cf.dec = lt.dec;
    return cf;
}

// A x and the diagonal of one row of the velocity (VEL) or pressure system
template <typename T, int D, int VEL, int A>
__device__ inline void wg_row(const LevTab<T> &lt, int i, int j, int k, T &Ax, T &dg)
{
    if (VEL) {
        const VelArr<T> x{{lt.xu[0], lt.xu[1], lt.xu[2]}};
        u_row<T, D, A>(lt.g, x, coef_u(lt), lt.mass, lt.cvu, i, j, k, Ax, dg);
    } else {
        const CoefP<T> cf{{lt.beta[0], lt.beta[1], lt.beta[2]}};
        p_row<T, D>(lt.g, lt.xp, cf, lt.cvp, i, j, k, Ax, dg);
    }
}

// ---- per-point bodies, shared by the one-workgroup cycle and the batched
// passes; the arithmetic is that of the launched kernels

// red-black Gauss-Seidel update of the t-th point of one colour
template <typename T, int D, int VEL, int A>
__device__ inline void sweep_at(const LevTab<T> &lt, const Box &box, int colour, int t)
{
    int i, j, k;
    if (!box_colour_pos(box, colour, t, i, j, k)) return;
    T *x = VEL ? lt.xu[A] : lt.xp;
    const T *b = VEL ? lt.bu[A] : lt.bp;
    const long long e = at(lt.g, i, j, k);
    const T be = b[e], xe = x[e];
    T Ax, dg;
    wg_row<T, D, VEL, A>(lt, i, j, k, Ax, dg);
    const T xn = xe + (be - Ax) / dg;
    x[e] = xn;
    write_images(lt.g, VEL ? face_mask(A) : 0, VEL ? ROLE_V : ROLE_P, x, i, j, k, xn);
}

// r = b - A x at the t-th unknown of the box (t in range); returns r
template <typename T, int D, int VEL, int A>
__device__ inline T resid_at(const LevTab<T> &lt, const Box &box, int t)
{
    int i, j, k;
    box_pos(box, t, i, j, k);
    const long long e = at(lt.g, i, j, k);
    const T be = (VEL ? lt.bu[A] : lt.bp)[e];
    T Ax, dg;
    wg_row<T, D, VEL, A>(lt, i, j, k, Ax, dg);
    const T rv = be - Ax;
    (VEL ? lt.ru[A] : lt.rp)[e] = rv;
    return rv;
}

// coarse right-hand side = restriction of the fine residual at the t-th
// coarse unknown; the coarse correction there is cleared with its images
template <typename T, int D, int VEL, int A>
__device__ inline void restrict_at(const LevTab<T> &lt, const LevTab<T> &lc, const Box &box, int t)
{
    const int vmask = VEL ? face_mask(A) : 0;
    const int role = VEL ? ROLE_V : ROLE_P;
    int I, J, K;
    box_pos(box, t, I, J, K);
    const long long e = at(lc.g, I, J, K);
    (VEL ? lc.bu[A] : lc.bp)[e] = (T)restrict_any<T, D>(vmask, lt.g, role, VEL ? lt.ru[A] : lt.rp, I, J, K);
    T *xc = VEL ? lc.xu[A] : lc.xp;
    xc[e] = T(0);
    write_images(lc.g, vmask, role, xc, I, J, K, T(0));
}

// fine x += prolongation of the coarse correction at the t-th fine unknown
template <typename T, int D, int VEL, int A>
__device__ inline void prolong_at(const LevTab<T> &lc, const LevTab<T> &lt, const Box &box, int t)
{
    const int vmask = VEL ? face_mask(A) : 0;
    const int role = VEL ? ROLE_V : ROLE_P;
    int i, j, k;
    box_pos(box, t, i, j, k);
    T *x = VEL ? lt.xu[A] : lt.xp;
    const long long e = at(lt.g, i, j, k);
    const T xe = x[e];
    const T v = xe + (T)prolong_any<T, D>(vmask, lc.g, role, VEL ? lc.xu[A] : lc.xp, i, j, k);
    x[e] = v;
    write_images(lt.g, vmask, role, x, i, j, k, v);
}

__device__ inline int colour_count(const Box &b) { return ((b.ext[0] + 1) >> 1) * b.ext[1] * b.ext[2]; }
__device__ inline int point_count(const Box &b) { return b.ext[0] * b.ext[1] * b.ext[2]; }

template <typename T, int D, int VEL, int A>
__device__ inline void wg_sweep_comp(const LevTab<T> &ltr)
{
    const LevTab<T> lt = ltr;
    const Grid &g = lt.g;
    const int vmask = VEL ? face_mask(A) : 0;
    const Box box = unk_box(g, vmask);
    const BoxDiv bd = lt.bd[VEL ? A : 3];
    const int n = ((box.ext[0] + 1) >> 1) * box.ext[1] * box.ext[2];
    T *x = VEL ? lt.xu[A] : lt.xp;
    const T *b = VEL ? lt.bu[A] : lt.bp;
    for (int colour = 0; colour < 2; ++colour) {
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            int i, j, k;
            if (!box_colour_pos(box, bd, colour, t, i, j, k)) continue;
            const long long e = at(g, i, j, k);
            const T be = b[e], xe = x[e];
            T Ax, dg;
            wg_row<T, D, VEL, A>(lt, i, j, k, Ax, dg);
            const T xn = xe + (be - Ax) / dg;
            x[e] = xn;
            write_images(g, vmask, VEL ? ROLE_V : ROLE_P, x, i, j, k, xn);
        }
        __syncthreads();
    }
}

template <typename T, int D, int VEL>
__device__ void wg_sweep(const LevTab<T> &lt)
{
    wg_sweep_comp<T, D, VEL, 0>(lt);
    if (VEL) {
        wg_sweep_comp<T, D, VEL, 1>(lt);
        if (D == 3) wg_sweep_comp<T, D, VEL, (D == 3 ? 2 : 1)>(lt);
    }
}

template <typename T, int D, int VEL, int A>
__device__ inline void wg_residual_comp(const LevTab<T> &ltr)
{
    const LevTab<T> lt = ltr;
    const Box box = unk_box(lt.g, VEL ? face_mask(A) : 0);
    const BoxDiv bd = lt.bd[VEL ? A : 3];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    T *r = VEL ? lt.ru[A] : lt.rp;
    const T *b = VEL ? lt.bu[A] : lt.bp;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        int i, j, k;
        box_pos(box, bd, t, i, j, k);
        const long long e = at(lt.g, i, j, k);
        const T be = b[e];
        T Ax, dg;
        wg_row<T, D, VEL, A>(lt, i, j, k, Ax, dg);
        r[e] = be - Ax;
    }
}

// coarse right-hand side = restriction of the fine residual, coarse
// correction cleared (with its images)
template <typename T, int D, int VEL, int A>
__device__ inline void wg_restrict_comp(const LevTab<T> &ltr, const LevTab<T> &lcr)
{
    const LevTab<T> lt = ltr, lc = lcr;
    const int vmask = VEL ? face_mask(A) : 0;
    const int role = VEL ? ROLE_V : ROLE_P;
    const Box box = unk_box(lc.g, vmask);
    const BoxDiv bd = lc.bd[VEL ? A : 3];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    const T *src = VEL ? lt.ru[A] : lt.rp;
    T *bc = VEL ? lc.bu[A] : lc.bp;
    T *xc = VEL ? lc.xu[A] : lc.xp;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        int I, J, K;
        box_pos(box, bd, t, I, J, K);
        const long long e = at(lc.g, I, J, K);
        bc[e] = (T)restrict_any<T, D>(vmask, lt.g, role, src, I, J, K);
        xc[e] = T(0);
        write_images(lc.g, vmask, role, xc, I, J, K, T(0));
    }
}

template <typename T, int D, int VEL, int A>
__device__ inline void wg_prolong_comp(const LevTab<T> &lcr, const LevTab<T> &ltr)
{
    const LevTab<T> lc = lcr, lt = ltr;
    const int vmask = VEL ? face_mask(A) : 0;
    const int role = VEL ? ROLE_V : ROLE_P;
    const Box box = unk_box(lt.g, vmask);
    const BoxDiv bd = lt.bd[VEL ? A : 3];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    const T *src = VEL ? lc.xu[A] : lc.xp;
    T *x = VEL ? lt.xu[A] : lt.xp;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        int i, j, k;
        box_pos(box, bd, t, i, j, k);
        const long long e = at(lt.g, i, j, k);
        const T xe = x[e];
        const T v = xe + (T)prolong_any<T, D>(vmask, lc.g, role, src, i, j, k);
        x[e] = v;
        write_images(lt.g, vmask, role, x, i, j, k, v);
    }
}

// columns of a tail matrix as stored: whole blocks of 16 bytes
__host__ __device__ inline int tail_ld(int n, int wsz) { return wsz == 4 ? (n + 3) & ~3 : (n + 1) & ~1; }

// Restriction of the fine residual onto the tail's unknowns, as a compact
// vector (bv[t]: the t-th unknown of the tail level); the same arithmetic as
// the restriction into the coarse level's b.
template <typename T, int D, int VEL>
__device__ inline void wg_restrict_tail(const LevTab<T> &ltr, const Grid &gc, const Tail &tail, T *bv)
{
    const LevTab<T> lt = ltr;
    const int role = VEL ? ROLE_V : ROLE_P;
    for (int t = threadIdx.x; t < tail.n; t += blockDim.x) {
        const int a = tail.comp[t];
        int I, J, K;
        decode(gc, tail.idx[t], I, J, K);
        const T *src = VEL ? (a == 0 ? lt.ru[0] : (a == 1 ? lt.ru[1] : lt.ru[2])) : lt.rp;
        bv[t] = (T)restrict_any<T, D>(VEL ? face_mask(a) : 0, lt.g, role, src, I, J, K);
    }
    for (int t = tail.n + threadIdx.x; t < tail_ld(tail.n, sizeof(T)); t += blockDim.x) bv[t] = T(0);
}

// x = Tm bv at the tail's unknowns, with the ghost images of x; the rest of
// x is zero already.  Tm is stored in blocks of W columns (W = 16 bytes over
// the element size): block q holds, row after row, the W entries of columns
// qW .. qW+W-1, so that the rows of a wave read contiguous memory per
// 16-byte load.
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
    using type = float4;
    static constexpr int n = 4;
};
template <>
struct Vec16<double> {
    using type = double2;
    static constexpr int n = 2;
};

// position of entry (row r, column j) of an n-row tail matrix
template <typename T>
__device__ inline long long tail_at(int n, int r, int j)
{
    constexpr int W = Vec16<T>::n;
    return (long long)(j / W) * ((long long)n * W) + (long long)r * W + (j % W);
}

// One row of Tm bv by the eight lanes u = 0 .. 7 of a row (neighbours in a
// wave): lane u takes the column blocks u, u + 8, ... in order, and the eight
// partial sums are added pairwise, so the order is the same in every kernel
// that uses it.  Columns past n (up to whole blocks) are zero in Tm, and bv
// holds zeros there.  Every lane of the wave must call it.
template <typename T>
__device__ inline T tail_row(const T *__restrict__ Tm, int n, int r, int u, const T *bv)
{
    using V = typename Vec16<T>::type;
    constexpr int W = Vec16<T>::n;
    const V *__restrict__ rv = reinterpret_cast<const V *>(Tm) + r;
    const int nq = tail_ld(n, sizeof(T)) / W;
    T sum = T(0);
#pragma unroll 4
    for (int q = u; q < nq; q += TAIL_LANES) {
        const V t = rv[(long long)q * n];
        const T *tt = reinterpret_cast<const T *>(&t);
#pragma unroll
        for (int w = 0; w < W; ++w) sum += tt[w] * bv[q * W + w];
    }
#pragma unroll
    for (int o = 1; o < TAIL_LANES; o <<= 1) sum += __shfl_xor(sum, o);
    return sum;
}

template <typename T, int D, int VEL>
__device__ inline void wg_apply_tail(const LevTab<T> &lcr, const Tail &tail, const T *bv)
{
    using V = typename Vec16<T>::type;
    constexpr int W = Vec16<T>::n;
    const LevTab<T> lc = lcr;
    const T *__restrict__ Tm = static_cast<const T *>(tail.Tm);
    const int n = tail.n;
    const int nq = tail_ld(n, sizeof(T)) / W;
    for (int r = threadIdx.x; r < n; r += blockDim.x) {
        // a thread a row: the lanes of a wave read contiguous memory (eight
        // lanes a row measured 42 -> 51 us for the whole cycle in 2D); the
        // eight partial sums of tail_row
        const V *__restrict__ rv = reinterpret_cast<const V *>(Tm) + r;
        T part[TAIL_LANES] = {};
        for (int q0 = 0; q0 < nq; q0 += TAIL_LANES) {
            V t[TAIL_LANES];
#pragma unroll
            for (int u = 0; u < TAIL_LANES; ++u)
                if (q0 + u < nq) t[u] = rv[(long long)(q0 + u) * n];
#pragma unroll
            for (int u = 0; u < TAIL_LANES; ++u) {
                if (q0 + u >= nq) continue;
                const T *tt = reinterpret_cast<const T *>(&t[u]);
#pragma unroll
                for (int w = 0; w < W; ++w) part[u] += tt[w] * bv[(q0 + u) * W + w];
            }
        }
#pragma unroll
        for (int o = 1; o < TAIL_LANES; o <<= 1)
#pragma unroll
            for (int u = 0; u < TAIL_LANES; u += 2 * o) part[u] += part[u + o];
        const T sum = part[0];
        const int a = tail.comp[r];
        T *x = VEL ? (a == 0 ? lc.xu[0] : (a == 1 ? lc.xu[1] : lc.xu[2])) : lc.xp;
        const long long e = tail.idx[r];
        x[e] = sum;
        int i, j, k;
        decode(lc.g, e, i, j, k);
        write_images(lc.g, VEL ? face_mask(a) : 0, VEL ? ROLE_V : ROLE_P, x, i, j, k, sum);
    }
}

// The part of a V-cycle from level l0 down to the coarsest level and back,
// in one workgroup: the same passes, in the same order, as the launched
// kernels, with a barrier where a launch boundary would be.  With a tail
// (tail.n > 0, tail.level = l0 + 1) the levels below l0 are the tail's
// matrix applied to the restricted residual (bv: shared scratch of
// TAIL_MAX values).
template <typename T, int D, int VEL>
__device__ __attribute__((always_inline)) inline void coarse_cycle(const LevTab<T> *__restrict__ tab, int l0, int L, int nu1,
                                                                  int nu2, int ndense,
                                    const long long *__restrict__ uidx, const int *__restrict__ ucomp,
                                    const double *__restrict__ M, const Tail &tail, T *bv)
{
    constexpr int A2 = D == 3 ? 2 : 1;
    const bool tailed = tail.n > 0;
    const int lb = tailed ? tail.level : L - 1;   // bottom of the recursion
    for (int l = l0; l < lb; ++l) {
        const LevTab<T> &lt = tab[l];
        for (int s = 0; s < nu1; ++s) wg_sweep<T, D, VEL>(lt);
        wg_residual_comp<T, D, VEL, 0>(lt);
        if (VEL) {
            wg_residual_comp<T, D, VEL, 1>(lt);
            if (D == 3) wg_residual_comp<T, D, VEL, A2>(lt);
        }
        __syncthreads();
        const LevTab<T> &lc = tab[l + 1];
        if (tailed && l + 1 == lb) {
            wg_restrict_tail<T, D, VEL>(lt, lc.g, tail, bv);
        } else {
            wg_restrict_comp<T, D, VEL, 0>(lt, lc);
            if (VEL) {
                wg_restrict_comp<T, D, VEL, 1>(lt, lc);
                if (D == 3) wg_restrict_comp<T, D, VEL, A2>(lt, lc);
            }
        }
        __syncthreads();
    }
    if (tailed) {
        wg_apply_tail<T, D, VEL>(tab[lb], tail, bv);
        __syncthreads();
    } else {
        const LevTab<T> lt = tab[L - 1];
        if (ndense > 0) {
            __shared__ double dv[64];
            const int r = threadIdx.x;
            if (r < ndense) {
                const int c = ucomp[r];
                const T *b = VEL ? (c == 0 ? lt.bu[0] : (c == 1 ? lt.bu[1] : lt.bu[2])) : lt.bp;
                dv[r] = (double)b[uidx[r]];
            }
            __syncthreads();
            if (r < ndense) {
                double sum = 0.0;
                for (int j = 0; j < ndense; ++j) sum += M[r * ndense + j] * dv[j];
                const int c = ucomp[r];
                T *x = VEL ? (c == 0 ? lt.xu[0] : (c == 1 ? lt.xu[1] : lt.xu[2])) : lt.xp;
                x[uidx[r]] = (T)sum;
                int i, jj, k;
                decode(lt.g, uidx[r], i, jj, k);
                write_images(lt.g, VEL ? face_mask(c) : 0, VEL ? ROLE_V : ROLE_P, x, i, jj, k, (T)sum);
            }
            __syncthreads();
        } else {
            for (int s = 0; s < nu1 + nu2; ++s) wg_sweep<T, D, VEL>(lt);
        }
    }
    for (int l = lb - 1; l >= l0; --l) {
        const LevTab<T> &lt = tab[l];
        const LevTab<T> &lc = tab[l + 1];
        wg_prolong_comp<T, D, VEL, 0>(lc, lt);
        if (VEL) {
            wg_prolong_comp<T, D, VEL, 1>(lc, lt);
            if (D == 3) wg_prolong_comp<T, D, VEL, A2>(lc, lt);
        }
        __syncthreads();
        for (int s = 0; s < nu2; ++s) wg_sweep<T, D, VEL>(lt);
    }
}

}  // namespace ibmg
