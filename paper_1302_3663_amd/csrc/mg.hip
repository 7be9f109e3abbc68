// Multigrid kernels for the pressure system A_p = -D(beta G) (eq:NSdis4,
// eq:divergenceGrad) and the viscous system
// A_u = (sigma rho / dt) I - Re^-1 D.(mu (D u + D u^T)) (eq:NSdis1-1,
// eq:divergencePartial) on the staggered grid: red-black Gauss-Seidel
// (component by component, red then black), residual with a fused squared
// norm, full-weighting restriction, linear prolongation, and the direct
// solve on the coarsest level (Sec. "Multigrid").
//
// Every kernel is templated on the arithmetic type T (double, or float for
// the inner cycles of the refined solver).  A point more than one cell away
// from every boundary reads its neighbours at fixed offsets; points near a
// boundary resolve each neighbour through the boundary rules of common.h.
//
// The rows, the transfers' taps and the passes of the one-workgroup cycle are
// in mg_device.h, shared with bricks.hip.
#include <algorithm>

#include <hip/hip_ext.h>

#include "common.h"
#include "kernels.h"
#include "mg_device.h"

#pragma clang fp contract(on)

namespace ibmg {

constexpr long long XCD_REMAP_MAX_NEL = 16ll << 20;

// ---------------------------------------------------------------------------
// Workgroups go to the chip's 8 XCDs in turn (workgroup b to XCD b mod 8),
// and each XCD has its own L2.  Renumbered so that the rows and planes that
// neighbouring points share stay in one L2 (a bijection of [0, gridDim.x)):
// remap < 0 gives each XCD one contiguous range of the index space, while
// remap > 0 deals out strips of so many workgroups, an eighth of a plane, so
// that an XCD keeps its strip from plane to plane.  0 keeps the hardware
// order.  Measured on the smoothers: ranges are 10% faster than the hardware
// order on arrays of 4.4 M entries and 5-7% slower on 34.5 M, where the planes
// a point reads no longer fit an XCD's L2; strips are 1-2% faster there.
// ---------------------------------------------------------------------------
__device__ inline unsigned xcd_block(int remap, unsigned b, unsigned nb)
{
    constexpr unsigned NXCD = 8;
    if (!remap) return b;
    if (remap > 0) {
        const unsigned n = (unsigned)remap, round = NXCD * n, r = b / round, t = b - r * round;
        return (r + 1) * round <= nb ? r * round + (t % NXCD) * n + t / NXCD : b;
    }
    const unsigned q = nb / NXCD, r = nb % NXCD, x = b % NXCD;
    return x * q + (x < r ? x : r) + b / NXCD;
}

__device__ inline unsigned xcd_block(int remap) { return xcd_block(remap, blockIdx.x, gridDim.x); }

__host__ __device__ static inline int xcd_remap(const Grid &g, const Box &box, long long blocks)
{
    const long long planes = g.D == 3 ? box.ext[2] : box.ext[1], n = (blocks / planes + 4) / 8;
    return g.nel <= XCD_REMAP_MAX_NEL ? -1 : (int)(n > 1 ? n : 1);
}

// ---------------------------------------------------------------------------
// smoothers: one colour of one component; the updated value is also written
// to its ghost images so that later passes read it at fixed offsets.  Each
// point reads its own x and b before its row, so that all of its loads are
// in flight together (read after the row, they cost a second round trip).
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(256) k_smooth_p(Grid g, Box box, const T *__restrict__ b, T *x, CoefP<T> cf, T cvisc,
                                                  int colour, int remap)
{
    int i, j, k;
    if (!box_colour_pos(box, colour, xcd_block(remap) * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long c = at(g, i, j, k);
    const T bc = b[c], xc = x[c];
    T Ax, dg;
    p_row<T, D>(g, x, cf, cvisc, i, j, k, Ax, dg);
    const T xn = xc + (bc - Ax) / dg;
    x[c] = xn;
    write_images(g, 0, ROLE_P, x, i, j, k, xn);
}

template <typename T, int D, int A>
__global__ void __launch_bounds__(256) k_smooth_u(Grid g, Box box, const T *__restrict__ b, VelArr<T> x, CoefU<T> cf,
                                                  T mass, T cvisc, int colour, int remap)
{
    int i, j, k;
    if (!box_colour_pos(box, colour, xcd_block(remap) * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long f = at(g, i, j, k);
    const T bf = b[f], xf = x.c[A][f];
    T Ax, dg;
    u_row<T, D, A>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
    const T xn = xf + (bf - Ax) / dg;
    x.c[A][f] = xn;
    write_images(g, face_mask(A), ROLE_V, x.c[A], i, j, k, xn);
}

// The same colour passes (3D), z-blocked: a workgroup owns a band of `rows`
// rows of one colour in each plane of a run of ZB_PLANES consecutive planes
// and walks those planes in order, so that the planes a point reads above
// and below were read by the same workgroup one step before (hits in its
// caches) rather than fetched again by other workgroups at other times.  The
// points of one colour are independent, so this order gives the same bits
// as the flat launch.
constexpr int ZB_PLANES = 16;

template <typename T>
__global__ void __launch_bounds__(256) k_smooth_p_zb(Grid g, Box box, const T *__restrict__ b, T *x, CoefP<T> cf,
                                                     T cvisc, int colour, int rows, int nbands)
{
    const int half = (box.ext[0] + 1) >> 1;
    const int j0 = (blockIdx.x % nbands) * rows, kz0 = (blockIdx.x / nbands) * ZB_PLANES;
    const int npts = half * min(rows, box.ext[1] - j0);
    const int kz1 = min(kz0 + ZB_PLANES, box.ext[2]);
    for (int kz = kz0; kz < kz1; ++kz) {
        const int k = box.lo[2] + kz;
        for (int t = threadIdx.x; t < npts; t += blockDim.x) {
            const int j = box.lo[1] + j0 + t / half;
            const int i = box.lo[0] + 2 * (t % half) + ((box.lo[0] + j + k + colour) & 1);
            if (i >= box.lo[0] + box.ext[0]) continue;
            const long long c = at(g, i, j, k);
            const T bc = b[c], xc = x[c];
            T Ax, dg;
            p_row<T, 3>(g, x, cf, cvisc, i, j, k, Ax, dg);
            const T xn = xc + (bc - Ax) / dg;
            x[c] = xn;
            write_images(g, 0, ROLE_P, x, i, j, k, xn);
        }
    }
}

template <typename T, int A>
__global__ void __launch_bounds__(256) k_smooth_u_zb(Grid g, Box box, const T *__restrict__ b, VelArr<T> x, CoefU<T> cf,
                                                     T mass, T cvisc, int colour, int rows, int nbands)
{
    const int half = (box.ext[0] + 1) >> 1;
    const int j0 = (blockIdx.x % nbands) * rows, kz0 = (blockIdx.x / nbands) * ZB_PLANES;
    const int npts = half * min(rows, box.ext[1] - j0);
    const int kz1 = min(kz0 + ZB_PLANES, box.ext[2]);
    for (int kz = kz0; kz < kz1; ++kz) {
        const int k = box.lo[2] + kz;
        for (int t = threadIdx.x; t < npts; t += blockDim.x) {
            const int j = box.lo[1] + j0 + t / half;
            const int i = box.lo[0] + 2 * (t % half) + ((box.lo[0] + j + k + colour) & 1);
            if (i >= box.lo[0] + box.ext[0]) continue;
            const long long f = at(g, i, j, k);
            const T bf = b[f], xf = x.c[A][f];
            T Ax, dg;
            u_row<T, 3, A>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
            const T xn = xf + (bf - Ax) / dg;
            x.c[A][f] = xn;
            write_images(g, face_mask(A), ROLE_V, x.c[A], i, j, k, xn);
        }
    }
}

// one colour of every component of the constant-viscosity system (eq:NSdis1)
// in one launch: the components do not couple, so this is the sweep of the
// components one after another.  blockIdx.y is the component.
template <typename T, int D>
__global__ void __launch_bounds__(256) k_smooth_u_dec(Grid g, VelBox boxes, VelArrC<T> b, VelArr<T> x, CoefU<T> cf,
                                                      T mass, T cvisc, int colour, int remap)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_colour_pos(boxes.b[a], colour, xcd_block(remap) * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long f = at(g, i, j, k);
    T *xa = x.c[a];
    const T bf = b.c[a][f], xf = xa[f];
    T Ax, dg;
    if (a == 0) u_row_dec<T, D, 0>(g, x.c[0], cf.rho[0], mass, cvisc, i, j, k, Ax, dg);
    else if (a == 1) u_row_dec<T, D, 1>(g, x.c[1], cf.rho[1], mass, cvisc, i, j, k, Ax, dg);
    else u_row_dec<T, D, (D == 3 ? 2 : 1)>(g, x.c[2], cf.rho[2], mass, cvisc, i, j, k, Ax, dg);
    const T xn = xf + (bf - Ax) / dg;
    xa[f] = xn;
    write_images(g, face_mask(a), ROLE_V, xa, i, j, k, xn);
}

// ---------------------------------------------------------------------------
// One full red-black sweep of one component in one launch.  Each workgroup
// owns a tile of the component's unknowns and stages a window of the tile
// plus two points on every side in LDS: the red points of the tile and of
// the ring around it are updated from the old black values, then the black
// points of the tile from those reds.  The red ring is computed again by
// the neighbouring tiles with the same arithmetic.  The result goes to a
// second buffer (x_out), so that no workgroup reads a value another one has
// already updated.  Along periodic axes the window holds the wrapped points
// themselves; along the other axes it holds the ghost images, which a red
// update refreshes inside the window.
// ---------------------------------------------------------------------------
template <typename T, int D>
struct RBTile {
    static constexpr int H = 2;
    static constexpr int TX = D == 3 ? 8 : 16, TY = D == 3 ? 8 : 16, TZ = D == 3 ? (sizeof(T) == 8 ? 4 : 8) : 1;
    static constexpr int WX = TX + 2 * H, WY = TY + 2 * H, WZ = D == 3 ? TZ + 2 * H : 1;
    static constexpr int W = WX * WY * WZ;
};

// write v (times the sign) to the ghost images of (i, j, k) along the
// non-periodic axes that fall inside the window [o, o + W)
template <typename T, int D>
__device__ inline void write_images_window(const Grid &g, int vmask, int role, T *x, int i, int j, int k, T v,
                                           const int o[3], const int w[3])
{
    const int q[3] = {i, j, k};
    AxisImages im[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        im[d] = d < D && g.bc[d] != AX_PERIODIC ? images_of(g, d, (vmask >> d) & 1, role, q[d])
                                               : AxisImages{{0, 0}, {0, 0}};
    if ((im[0].s[0] | im[0].s[1] | im[1].s[0] | im[1].s[1] | im[2].s[0] | im[2].s[1]) == 0) return;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (a == 0 && b == 0 && c == 0) continue;
                const int sa = a ? im[0].s[a - 1] : 1;
                const int sb = b ? im[1].s[b - 1] : 1;
                const int sc = c ? im[2].s[c - 1] : 1;
                if (sa == 0 || sb == 0 || sc == 0) continue;
                const int qa = a ? im[0].q[a - 1] : i;
                const int qb = b ? im[1].q[b - 1] : j;
                const int qc = c ? im[2].q[c - 1] : k;
                if (qa < o[0] || qa >= o[0] + w[0] || qb < o[1] || qb >= o[1] + w[1]) continue;
                if (D == 3 && (qc < o[2] || qc >= o[2] + w[2])) continue;
                x[at(g, qa, qb, qc)] = sa * sb * sc > 0 ? v : -v;
            }
}

template <typename T, int D, int VEL, int A>
__global__ void __launch_bounds__(256) k_smooth_rb(Grid g, Box box, VelArrC<T> xin, const T *__restrict__ b,
                                                   CoefU<T> cu, CoefP<T> cp, T mass, T cvisc, T *xout)
{
    using TL = RBTile<T, D>;
    constexpr int NARR = VEL ? 2 * D + 2 : D + 2;
    constexpr int BS = 256;
    __shared__ T w[NARR][TL::W];
    const int vmask = VEL ? face_mask(A) : 0;
    const int role = VEL ? ROLE_V : ROLE_P;
    // this workgroup's tile and window origin (extended lattice coordinates)
    const int ntx = (box.ext[0] + TL::TX - 1) / TL::TX, nty = (box.ext[1] + TL::TY - 1) / TL::TY;
    const int tid = blockIdx.x;
    const int t0 = tid % ntx, t1 = (tid / ntx) % nty, t2 = tid / (ntx * nty);
    const int lo[3] = {box.lo[0] + t0 * TL::TX, box.lo[1] + t1 * TL::TY, D == 3 ? box.lo[2] + t2 * TL::TZ : 0};
    const int o[3] = {lo[0] - TL::H, lo[1] - TL::H, D == 3 ? lo[2] - TL::H : 0};
    const int wd[3] = {TL::WX, TL::WY, TL::WZ};
    // the window as a grid: same axes and boundary kinds, window strides
    Grid gw = g;
    gw.NX = TL::WX;
    gw.NY = TL::WY;
    gw.NXY = (long long)TL::WX * TL::WY;
    const long long shift = at(gw, o[0], o[1], o[2]);
    // source arrays of the window, in the order of w
    const T *src[NARR];
    if (VEL) {
        src[0] = xin.c[A];
#pragma unroll
        for (int bi = 0; bi < D - 1; ++bi) {
            const int B = other_axis<A>(bi);
            src[1 + bi] = xin.c[B];
            src[D + 3 + bi] = cu.mue[3 - A - B];
        }
        src[D] = b;
        src[D + 1] = cu.rho[A];
        src[D + 2] = cu.muc;
    } else {
        src[0] = xin.c[0];
        src[1] = b;
#pragma unroll
        for (int a = 0; a < D; ++a) src[2 + a] = cp.beta[a];
    }
    // stage the window: every load issued before the first store
    constexpr int PER = (TL::W + BS - 1) / BS;
    int eidx[PER];
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const int sidx = threadIdx.x + it * BS;
        int q[3] = {o[0] + sidx % TL::WX, o[1] + (sidx / TL::WX) % TL::WY, D == 3 ? o[2] + sidx / (TL::WX * TL::WY) : 0};
        bool ok = sidx < TL::W;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (g.bc[d] == AX_PERIODIC) {
                if (q[d] < 0) q[d] += g.n[d];
                while (q[d] >= g.n[d]) q[d] -= g.n[d];
            } else if (q[d] < -1 || q[d] > g.n[d] + 1) {
                ok = false;
            }
        }
        eidx[it] = ok ? (int)at(g, q[0], q[1], q[2]) : -1;
    }
    T v[NARR][PER];
#pragma unroll
    for (int m = 0; m < NARR; ++m)
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const T x = src[m][eidx[it] >= 0 ? eidx[it] : 0];
            v[m][it] = eidx[it] >= 0 ? x : T(0);
        }
#pragma unroll
    for (int m = 0; m < NARR; ++m)
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const int sidx = threadIdx.x + it * BS;
            if (sidx < TL::W) w[m][sidx] = v[m][it];
        }
    __syncthreads();
    // window views shifted so that at(gw, i, j, k) indexes them
    VelArr<T> xw{{nullptr, nullptr, nullptr}};
    CoefU<T> cw = cu;
    CoefP<T> pw = cp;
    T *bw;
    if (VEL) {
        xw.c[A] = &w[0][0] - shift;
#pragma unroll
        for (int bi = 0; bi < D - 1; ++bi) {
            const int B = other_axis<A>(bi);
            xw.c[B] = &w[1 + bi][0] - shift;
            cw.mue[3 - A - B] = &w[D + 3 + bi][0] - shift;
        }
        bw = &w[D][0] - shift;
        cw.rho[A] = &w[D + 1][0] - shift;
        cw.muc = &w[D + 2][0] - shift;
    } else {
        xw.c[0] = &w[0][0] - shift;
        bw = &w[1][0] - shift;
#pragma unroll
        for (int a = 0; a < D; ++a) pw.beta[a] = &w[2 + a][0] - shift;
    }
    T *xa = xw.c[VEL ? A : 0];
    int ulo[3], uhi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) unk_range(g, d, (vmask >> d) & 1, ulo[d], uhi[d]);
    // red: the tile and the ring around it, enumerated by colour
    constexpr int RX = TL::TX + 2, RY = TL::TY + 2, RZ = D == 3 ? TL::TZ + 2 : 1, RH = RX / 2;
    for (int t = threadIdx.x; t < RH * RY * RZ; t += BS) {
        const int ih = t % RH, r = t / RH;
        const int q1 = lo[1] - 1 + r % RY, q2 = D == 3 ? lo[2] - 1 + r / RY : 0;
        const int q0 = lo[0] - 1 + 2 * ih + ((lo[0] - 1 + q1 + q2) & 1);
        const int qq[3] = {q0, q1, q2};
        bool unknown = true;
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (g.bc[d] != AX_PERIODIC && (qq[d] < ulo[d] || qq[d] > uhi[d])) unknown = false;
        if (!unknown) continue;
        T Ax, dg;
        if (VEL) u_row<T, D, A>(gw, xw, cw, mass, cvisc, q0, q1, q2, Ax, dg);
        else p_row<T, D>(gw, xa, pw, cvisc, q0, q1, q2, Ax, dg);
        const long long f = at(gw, q0, q1, q2);
        const T xn = xa[f] + (bw[f] - Ax) / dg;
        xa[f] = xn;
        write_images_window<T, D>(gw, vmask, role, xa, q0, q1, q2, xn, o, wd);
    }
    __syncthreads();
    // black: the tile, enumerated by colour
    constexpr int TH = TL::TX / 2;
    for (int t = threadIdx.x; t < TH * TL::TY * TL::TZ; t += BS) {
        const int ih = t % TH, r = t / TH;
        const int q1 = lo[1] + r % TL::TY, q2 = D == 3 ? lo[2] + r / TL::TY : 0;
        const int q0 = lo[0] + 2 * ih + ((lo[0] + q1 + q2 + 1) & 1);
        if (q0 >= box.lo[0] + box.ext[0] || q1 >= box.lo[1] + box.ext[1]) continue;
        if (D == 3 && q2 >= box.lo[2] + box.ext[2]) continue;
        T Ax, dg;
        if (VEL) u_row<T, D, A>(gw, xw, cw, mass, cvisc, q0, q1, q2, Ax, dg);
        else p_row<T, D>(gw, xa, pw, cvisc, q0, q1, q2, Ax, dg);
        const long long f = at(gw, q0, q1, q2);
        xa[f] = xa[f] + (bw[f] - Ax) / dg;
    }
    __syncthreads();
    // the tile's unknowns and their ghost images to the output buffer
    constexpr int TT = TL::TX * TL::TY * TL::TZ;
    for (int sidx = threadIdx.x; sidx < TT; sidx += BS) {
        const int q0 = lo[0] + sidx % TL::TX, q1 = lo[1] + (sidx / TL::TX) % TL::TY;
        const int q2 = D == 3 ? lo[2] + sidx / (TL::TX * TL::TY) : 0;
        if (q0 >= box.lo[0] + box.ext[0] || q1 >= box.lo[1] + box.ext[1]) continue;
        if (D == 3 && q2 >= box.lo[2] + box.ext[2]) continue;
        const T val = xa[at(gw, q0, q1, q2)];
        xout[at(g, q0, q1, q2)] = val;
        write_images(g, vmask, role, xout, q0, q1, q2, val);
    }
}

// ---------------------------------------------------------------------------
// One launch per red-black sweep of a velocity component (3D), marching
// along z.  A workgroup owns a tile of ZM_TX x ZM_TY points in each plane of
// a run [z0, z1) of planes and holds u_a of ZM_NS consecutive planes, the
// tile widened by ZM_H points on every side, in LDS.  Stepping p = z0 ..
// z1 - 1, it loads plane p + 3, updates the red points of plane p + 1 (the
// tile and a ring of one point around it), then the black points of plane p
// (the tile).  Ring points, and the red planes z0 - 1 and z1, belong to other
// workgroups: they are updated again here, from the same values with the
// same arithmetic, so that the black points at the tile's edge see the red
// values of after the pass.  Every red point thus reads the black values of
// before the sweep and every black point the red values of after it: the
// bits of the two colour passes.  The other fields are read from global
// memory, each point's once per sweep, so the sweep streams every array
// about once instead of once per colour.  Results go to a second buffer,
// since the window's halo must see values from before the sweep.
//
// Window planes: red at p + 1 reads p .. p + 2 and writes ghost images up to
// two planes away (the one past the outflow face); black at p reads
// p - 1 .. p + 1.  Six slots let the load of plane p + 4 overwrite p - 2
// while black p may still be reading p - 1, so a step needs two barriers.
// (Running red p + 1 and black p - 1 in one phase, one barrier a step, was
// slower.)
// ---------------------------------------------------------------------------
constexpr int ZM_TX = 64, ZM_TY = 8, ZM_H = 2, ZM_WX = ZM_TX + 2 * ZM_H, ZM_WY = ZM_TY + 2 * ZM_H;
constexpr int ZM_PS = ZM_WX * ZM_WY, ZM_NS = 6, ZM_BS = 256;

// u_a at a point of the window and along its axes: in-plane neighbours in the
// point's plane, z neighbours in the planes below and above
template <typename T>
struct UaWin {
    const T *w;
    int c;       // position in the plane
    int pl[3];   // offsets of the planes z - 1, z, z + 1
    __device__ T here() const { return w[pl[1] + c]; }
    __device__ T nb(int ax, int s) const
    {
        return ax == 2 ? w[pl[1 + s] + c] : w[pl[1] + c + (ax == 0 ? s : s * ZM_WX)];
    }
};

__device__ inline int zm_slot(int z) { return (((z % ZM_NS) + ZM_NS) % ZM_NS) * ZM_PS; }

template <typename T, int A>
__global__ void __launch_bounds__(ZM_BS) k_smooth_zm(Grid g, Box box, VelArrC<T> xin, const T *__restrict__ b,
                                                      CoefU<T> cf, T mass, T cvisc, T *xout, int cz, int remap)
{
    __shared__ T w[ZM_NS * ZM_PS];
    constexpr int vmask = 1 << A;
    const int ntx = (box.ext[0] + ZM_TX - 1) / ZM_TX, nty = (box.ext[1] + ZM_TY - 1) / ZM_TY;
    const int tid = (int)xcd_block(remap);
    const int t0 = tid % ntx, t1 = (tid / ntx) % nty, ch = tid / (ntx * nty);
    const int lo0 = box.lo[0] + t0 * ZM_TX, lo1 = box.lo[1] + t1 * ZM_TY;
    const int hx = min(lo0 + ZM_TX, box.lo[0] + box.ext[0]), hy = min(lo1 + ZM_TY, box.lo[1] + box.ext[1]);
    const int z0 = box.lo[2] + ch * cz, z1 = min(z0 + cz, box.lo[2] + box.ext[2]);
    const int o0 = lo0 - ZM_H, o1 = lo1 - ZM_H;
    int ulo[3], uhi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) unk_range(g, d, (vmask >> d) & 1, ulo[d], uhi[d]);
    const bool per[3] = {g.bc[0] == AX_PERIODIC, g.bc[1] == AX_PERIODIC, g.bc[2] == AX_PERIODIC};
    // a lattice coordinate along a periodic axis, brought into [0, n)
    auto wrap = [&](int d, int q) { return !per[d] ? q : (q < 0 ? q + g.n[d] : (q >= g.n[d] ? q - g.n[d] : q)); };
    // positions stored along a non-periodic axis: -1 .. n + 1
    auto stored = [&](int d, int q) { return per[d] || (q >= -1 && q <= g.n[d] + 1); };
    const T *__restrict__ xa = xin.c[A];

    auto load_plane = [&](int z) {
        T *dst = w + zm_slot(z);
        const int rz = wrap(2, z);
        const bool zok = stored(2, z);
        constexpr int PER = (ZM_PS + ZM_BS - 1) / ZM_BS;
        T v[PER];
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const int sidx = threadIdx.x + it * ZM_BS;
            const int qx = o0 + sidx % ZM_WX, qy = o1 + sidx / ZM_WX;
            const bool ok = sidx < ZM_PS && zok && stored(0, qx) && stored(1, qy);
            v[it] = ok ? xa[at(g, wrap(0, qx), wrap(1, qy), rz)] : T(0);
        }
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const int sidx = threadIdx.x + it * ZM_BS;
            if (sidx < ZM_PS) dst[sidx] = v[it];
        }
    };

    // the ghost images (non-periodic axes) of window point (x, y, z) that
    // fall inside the window's planes zl .. zh
    auto win_images = [&](int x, int y, int z, T v, int zl, int zh) {
        const int q[3] = {x, y, z};
        AxisImages im[3];
#pragma unroll
        for (int d = 0; d < 3; ++d)
            im[d] = per[d] ? AxisImages{{0, 0}, {0, 0}} : images_of(g, d, (vmask >> d) & 1, ROLE_V, q[d]);
        if ((im[0].s[0] | im[0].s[1] | im[1].s[0] | im[1].s[1] | im[2].s[0] | im[2].s[1]) == 0) return;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc)
#pragma unroll
            for (int bb = 0; bb < 3; ++bb)
#pragma unroll
                for (int aa = 0; aa < 3; ++aa) {
                    if (aa == 0 && bb == 0 && cc == 0) continue;
                    const int sa = aa ? im[0].s[aa - 1] : 1;
                    const int sb = bb ? im[1].s[bb - 1] : 1;
                    const int sc = cc ? im[2].s[cc - 1] : 1;
                    if (sa == 0 || sb == 0 || sc == 0) continue;
                    const int qa = aa ? im[0].q[aa - 1] : x;
                    const int qb = bb ? im[1].q[bb - 1] : y;
                    const int qc = cc ? im[2].q[cc - 1] : z;
                    if (qa < o0 || qa >= o0 + ZM_WX || qb < o1 || qb >= o1 + ZM_WY || qc < zl || qc > zh) continue;
                    w[zm_slot(qc) + (qb - o1) * ZM_WX + (qa - o0)] = sa * sb * sc > 0 ? v : -v;
                }
    };

    constexpr int RH = (ZM_TX + 2) / 2, RY = ZM_TY + 2, NRED = RH * RY;
    constexpr int BH = ZM_TX / 2, NBLACK = BH * ZM_TY;

    // the t-th red point of plane z in the tile and its ring; zl .. zh:
    // planes held
    auto red_point = [&](int z, int t, int zl, int zh) {
        const int ih = t % RH, r = t / RH;
        const int y = lo1 - 1 + r;
        const int x = lo0 - 1 + 2 * ih + ((lo0 - 1 + y + z) & 1);
        if (x > hx || y > hy) return;
        if (!per[0] && (x < ulo[0] || x > uhi[0])) return;
        if (!per[1] && (y < ulo[1] || y > uhi[1])) return;
        const int rx = wrap(0, x), ry = wrap(1, y), rz = wrap(2, z);
        const int f = (int)at(g, rx, ry, rz);
        const UaWin<T> ua{w, (y - o1) * ZM_WX + (x - o0), {zm_slot(z - 1), zm_slot(z), zm_slot(z + 1)}};
        const T rho = cf.rho[A][f];
        const T bf = b[f], xe = ua.here();
        T Ax, dg;
        u_row_core<T, 3, A>(g, ua, xin, cf, rho, mass, cvisc, f, rx, ry, rz, Ax, dg);
        const T xn = xe + (bf - Ax) / dg;
        w[ua.pl[1] + ua.c] = xn;
        win_images(x, y, z, xn, zl, zh);
        if (z >= z0 && z < z1 && x >= lo0 && x < hx && y >= lo1 && y < hy) {
            xout[f] = xn;
            write_images(g, vmask, ROLE_V, xout, x, y, z, xn);
        }
    };
    auto red_unknown_plane = [&](int z) { return per[2] || (z >= ulo[2] && z <= uhi[2]); };

    // the t-th black point of plane z (in [z0, z1)) in the tile
    auto black_point = [&](int z, int t) {
        const int ih = t % BH, r = t / BH;
        const int y = lo1 + r;
        const int x = lo0 + 2 * ih + ((lo0 + y + z + 1) & 1);
        if (x >= hx || y >= hy) return;
        const int f = (int)at(g, x, y, z);
        const UaWin<T> ua{w, (y - o1) * ZM_WX + (x - o0), {zm_slot(z - 1), zm_slot(z), zm_slot(z + 1)}};
        const T rho = cf.rho[A][f];
        const T bf = b[f], xe = ua.here();
        T Ax, dg;
        u_row_core<T, 3, A>(g, ua, xin, cf, rho, mass, cvisc, f, x, y, z, Ax, dg);
        const T xn = xe + (bf - Ax) / dg;
        xout[f] = xn;
        write_images(g, vmask, ROLE_V, xout, x, y, z, xn);
    };

    for (int z = z0 - 2; z <= z0 + 2; ++z) load_plane(z);
    __syncthreads();
    for (int t = threadIdx.x; t < 2 * NRED; t += ZM_BS) {
        const int z = t < NRED ? z0 - 1 : z0;
        if (red_unknown_plane(z)) red_point(z, t < NRED ? t : t - NRED, z0 - 2, z0 + 2);
    }
    __syncthreads();
    for (int p = z0; p < z1; ++p) {
        load_plane(p + 3);
        __syncthreads();
        if (red_unknown_plane(p + 1))
            for (int t = threadIdx.x; t < NRED; t += ZM_BS) red_point(p + 1, t, p, p + 3);
        __syncthreads();
        for (int t = threadIdx.x; t < NBLACK; t += ZM_BS) black_point(p, t);
    }
}


// ---------------------------------------------------------------------------
// block reduction of one double per thread into partial[slot] (fixed order)
// ---------------------------------------------------------------------------
__device__ inline void block_sum_store(double v, double *partial, long long slot)
{
    __shared__ double red[256];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[slot] = red[0];
}

// residual r = b - A x at every unknown (r may be null) and per-block
// partial sums of r^2 (partial may be null); grid-stride over the box
template <typename T, int D>
__global__ void __launch_bounds__(256) k_resid_p(Grid g, Box box, const T *__restrict__ b, const T *__restrict__ x,
                                                 CoefP<T> cf, T cvisc, T *r, double *partial)
{
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    double acc = 0.0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        int i, j, k;
        box_pos(box, t, i, j, k);
        const long long c = at(g, i, j, k);
        const T bc = b[c];
        T Ax, dg;
        p_row<T, D>(g, x, cf, cvisc, i, j, k, Ax, dg);
        const T rv = bc - Ax;
        if (r) r[c] = rv;
        acc += (double)rv * (double)rv;
    }
    if (partial) block_sum_store(acc, partial, blockIdx.x);
}

template <typename T, int D, int A>
__device__ inline T resid_u_at(const Grid &g, const VelArrC<T> &b, const VelArr<T> &x, const CoefU<T> &cf, T mass,
                               T cvisc, const VelArr<T> &r, int i, int j, int k)
{
    const long long f = at(g, i, j, k);
    const T bf = b.c[A][f];
    T Ax, dg;
    u_row<T, D, A>(g, x, cf, mass, cvisc, i, j, k, Ax, dg);
    const T rv = bf - Ax;
    if (r.c[A]) r.c[A][f] = rv;
    return rv;
}

// component blockIdx.y, as k_resid_p
template <typename T, int D>
__global__ void __launch_bounds__(256) k_resid_u(Grid g, VelBox boxes, VelArrC<T> b, VelArr<T> x, CoefU<T> cf, T mass,
                                                 T cvisc, VelArr<T> r, double *partial)
{
    constexpr int A2 = D == 3 ? 2 : 1;
    const int a = blockIdx.y;
    const Box box = boxes.b[a];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    double acc = 0.0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        int i, j, k;
        box_pos(box, t, i, j, k);
        T rv;
        if (a == 0) rv = resid_u_at<T, D, 0>(g, b, x, cf, mass, cvisc, r, i, j, k);
        else if (a == 1) rv = resid_u_at<T, D, 1>(g, b, x, cf, mass, cvisc, r, i, j, k);
        else rv = resid_u_at<T, D, A2>(g, b, x, cf, mass, cvisc, r, i, j, k);
        acc += (double)rv * (double)rv;
    }
    if (partial) block_sum_store(acc, partial, (long long)blockIdx.y * gridDim.x + blockIdx.x);
}

// From so many points a component on, the waves of one round of components
// fill the chip several times over; below, each component has its own.
constexpr long long RESID_ALL_MIN = 1ll << 20;

// How the rows of a level's velocity residual are dealt out: `all` holds the
// rows of every component, in `blocks` blocks of waves; with norms nb blocks
// take them in rounds, and a block's place in the partial sums is its number
// before the remapping.  The same for a solve alone and in a group, so that
// both add up a norm in the same order.
struct ResidRows {
    Box all;
    unsigned blocks, nb;
    int remap;
    bool large, norm;   // all components in turn; rows by waves with norms too
};
__host__ __device__ static inline ResidRows resid_rows(const Grid &g)
{
    ResidRows R;
    R.all = unk_box(g, face_mask(0));
    const bool rows = rows_by_waves(R.all);
    long long mx = 0;
    for (int a = 0; a < g.D; ++a) {
        const Box b = unk_box(g, face_mask(a));
        const long long n = (long long)b.ext[0] * b.ext[1] * b.ext[2];
        mx = n > mx ? n : mx;
        for (int d = 0; d < 3; ++d) {
            const int he = R.all.lo[d] + R.all.ext[d], hb = b.lo[d] + b.ext[d];
            R.all.lo[d] = b.lo[d] < R.all.lo[d] ? b.lo[d] : R.all.lo[d];
            R.all.ext[d] = (hb > he ? hb : he) - R.all.lo[d];
        }
    }
    R.large = mx >= RESID_ALL_MIN;
    R.norm = rows && R.large;
    R.blocks = row_blocks(R.all);
    R.nb = R.blocks < NORM_BLOCKS_MAX ? R.blocks : NORM_BLOCKS_MAX;
    R.remap = xcd_remap(g, R.all, R.blocks);
    return R;
}

// Components [a0, a1) of the residual at the points of block blk of the rows;
// NORM: their squares added to acc
template <typename T, int D, bool NORM>
__device__ inline void resid_u_block(const Grid &g, const Box &all, const VelBox &boxes, const VelArrC<T> &b,
                                     const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc, const VelArr<T> &r, int a0,
                                     int a1, unsigned blk, double acc[3])
{
    constexpr int A2 = D == 3 ? 2 : 1;
    int i, j, k;
    if (!row_pos(all, blk, i, j, k)) return;
    auto in = [&](const Box &q) {
        return i >= q.lo[0] && i < q.lo[0] + q.ext[0] && j >= q.lo[1] && j < q.lo[1] + q.ext[1] && k >= q.lo[2] &&
               k < q.lo[2] + q.ext[2];
    };
    auto add = [&](int a, T v) {
        if (NORM) acc[a] += (double)v * (double)v;
    };
    if (a0 == 0 && in(boxes.b[0])) add(0, resid_u_at<T, D, 0>(g, b, x, cf, mass, cvisc, r, i, j, k));
    if (a0 <= 1 && a1 > 1 && in(boxes.b[1])) add(1, resid_u_at<T, D, 1>(g, b, x, cf, mass, cvisc, r, i, j, k));
    if (D == 3 && a1 > 2 && in(boxes.b[2])) add(2, resid_u_at<T, D, A2>(g, b, x, cf, mass, cvisc, r, i, j, k));
}

// The residual, rows by waves: `ncomp` components from blockIdx.y on, in turn,
// so that what they share (the velocities, the viscosities) comes from the
// caches.  NORM: all components and their squared norms, rounds of gridDim.x
// blocks, partial sums per component and block.  Numbered through in a grid-stride loop over one component
// (k_resid_u), the divisions of the index and each component's own fetch of
// what they share bound it: 1110 us at 256 x 256 x 512 in FP32 against 725, in
// FP64 with norms 2080 against 1580; 98 against 61 at 128 x 128 x 256 in FP32.
template <typename T, int D, bool NORM>
__global__ void __launch_bounds__(256) k_resid_u_rows(Grid g, Box all, VelBox boxes, VelArrC<T> b, VelArr<T> x,
                                                      CoefU<T> cf, T mass, T cvisc, VelArr<T> r, int ncomp, int remap,
                                                      unsigned blocks, double *partial)
{
    const int a0 = NORM ? 0 : blockIdx.y, a1 = NORM ? D : a0 + ncomp;
    double acc[3] = {0.0, 0.0, 0.0};
    for (unsigned blk = xcd_block(remap); blk < blocks; blk += gridDim.x) {
        resid_u_block<T, D, NORM>(g, all, boxes, b, x, cf, mass, cvisc, r, a0, a1, blk, acc);
        if (!NORM) return;
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        block_sum_store(acc[a], partial, (long long)a * gridDim.x + blockIdx.x);
        __syncthreads();
    }
}

// sum of squares of a field over the unknowns of one or more lattices
template <typename T>
__global__ void __launch_bounds__(256) k_norm2(VelBox boxes, Grid g, VelArrC<T> v, double *partial)
{
    const int a = blockIdx.y;
    const Box box = boxes.b[a];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    double acc = 0.0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        int i, j, k;
        box_pos(box, t, i, j, k);
        const double w = (double)v.c[a][at(g, i, j, k)];
        acc += w * w;
    }
    block_sum_store(acc, partial, (long long)blockIdx.y * gridDim.x + blockIdx.x);
}

// one block: out[0] = sum of partial[0..n) in a fixed order
__global__ void __launch_bounds__(256) k_reduce_final(const double *__restrict__ partial, long long n, double *out)
{
    double acc = 0.0;
    for (long long t = threadIdx.x; t < n; t += blockDim.x) acc += partial[t];
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

// ---------------------------------------------------------------------------
// transfers
// ---------------------------------------------------------------------------
// coarse[c] = full-weighting restriction of fine[c] at every coarse unknown
// (or every stored coarse position for coefficients); zero_x[c], when set,
// is cleared at the same positions (the coarse correction starts at zero)
template <typename T, int D>
__global__ void __launch_bounds__(256) k_restrict(Grid gf, Grid gc, VelBox boxes, int masks, int role,
                                                  VelArrC<T> fine, VelArr<T> coarse, T scale, VelArr<T> zero_x)
{
    const int comp = blockIdx.y;
    const int vmask = (masks >> (4 * comp)) & 0xF;
    int I, J, K;
    if (!box_pos(boxes.b[comp], blockIdx.x * blockDim.x + threadIdx.x, I, J, K)) return;
    const double s = restrict_any<T, D>(vmask, gf, role, fine.c[comp], I, J, K);
    const long long e = at(gc, I, J, K);
    coarse.c[comp][e] = (T)(s * (double)scale);
    if (zero_x.c[comp]) {
        zero_x.c[comp][e] = T(0);
        write_images(gc, vmask, role, zero_x.c[comp], I, J, K, T(0));
    }
}

// fine[c] += linear interpolation of coarse[c] at every fine unknown
template <typename T, int D>
__global__ void __launch_bounds__(256) k_prolong_add(Grid gc, Grid gf, VelBox boxes, int masks, int role,
                                                     VelArrC<T> coarse, VelArr<T> fine)
{
    const int comp = blockIdx.y;
    const int vmask = (masks >> (4 * comp)) & 0xF;
    int i, j, k;
    if (!box_pos(boxes.b[comp], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long e = at(gf, i, j, k);
    const T xe = fine.c[comp][e];
    const T v = xe + (T)prolong_any<T, D>(vmask, gc, role, coarse.c[comp], i, j, k);
    fine.c[comp][e] = v;
    write_images(gf, vmask, role, fine.c[comp], i, j, k, v);
}

// The same interpolation for large boxes: a wave walks a row, so the taps
// along y and z are scalars and only boundary lanes look for ghost images.
// Numbered through, the points are bound by the instructions of their taps:
// 573 us at 256 x 256 x 512 in FP32 against 320 by rows, 80 against 58 at
// 128 x 128 x 256.  (The restriction by rows took the same time: 334 and 329.)

// a point that may have ghost images: within one of an end of its axis
__device__ inline bool near_end(const Grid &g, int d, int q) { return q <= 1 || q >= g.n[d] - 1; }

// the ghost images of point i of a row; `ends`: the row has some along y or z
template <typename T>
__device__ inline void row_images(const Grid &g, int vmask, int role, bool ends, T *x, int i, int j, int k, T v)
{
    if (ends) {
        write_images(g, vmask, role, x, i, j, k, v);
        return;
    }
    if (!near_end(g, 0, i)) return;
    const AxisImages im = images_of(g, 0, vmask & 1, role, i);
    if (im.s[0]) x[at(g, im.q[0], j, k)] = im.s[0] > 0 ? v : -v;
    if (im.s[1]) x[at(g, im.q[1], j, k)] = im.s[1] > 0 ? v : -v;
}

// The taps of the coarse iterate are read where they lie: the ghost positions
// hold what they stand for (every pass that writes an unknown writes its
// images) and the fixed faces hold zero.
template <typename T, int D, int VM>
__device__ inline void prolong_row(const Grid &gc, const Grid &gf, const Box &box, int role,
                                   const T *__restrict__ coarse, T *fine, int j, int k)
{
    int q1[2], q2[2], q0[2];
    double w1[2], w2[2], w0[2];
    if (prl_weights((VM >> 1) & 1, j, q1, w1) == 1) { q1[1] = q1[0]; w1[1] = 0.0; }
    q2[0] = 0;
    w2[0] = 1.0;
    if (D == 3 && prl_weights((VM >> 2) & 1, k, q2, w2) == 1) { q2[1] = q2[0]; w2[1] = 0.0; }
    const bool ends = near_end(gf, 1, j) || (D == 3 && near_end(gf, 2, k));
    const T *__restrict__ row[D == 3 ? 2 : 1][2];
#pragma unroll
    for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) row[c][b] = coarse + at(gc, 0, q1[b], q2[c]);
    T *const frow = fine + at(gf, 0, j, k);
#pragma unroll 1
    for (int i = box.lo[0] + (int)(threadIdx.x & 63); i < box.lo[0] + box.ext[0]; i += 64) {
        if (prl_weights(VM & 1, i, q0, w0) == 1) { q0[1] = q0[0]; w0[1] = 0.0; }
        const T xe = frow[i];
        T v[D == 3 ? 2 : 1][2][2];
#pragma unroll
        for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) v[c][b][a] = row[c][b][q0[a]];
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) s += w0[a] * w1[b] * w2[c] * (double)v[c][b][a];
        const T x = xe + (T)s;
        frow[i] = x;
        row_images(gf, VM, role, ends, fine, i, j, k, x);
    }
}

// this wave's row of the box; false: none
__device__ inline bool wave_row(const Box &box, int &j, int &k)
{
    const int row = (int)xcd_block(-1) * ROW_WAVES + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int kk = row / box.ext[1];
    j = __builtin_amdgcn_readfirstlane(box.lo[1] + (row - kk * box.ext[1]));
    k = __builtin_amdgcn_readfirstlane(box.lo[2] + kk);
    return kk < box.ext[2];
}

template <typename T, int D, bool VEL>
__global__ void __launch_bounds__(256) k_prolong_rows(Grid gc, Grid gf, VelBox boxes, int role, VelArrC<T> coarse,
                                                      VelArr<T> fine)
{
    const int a = VEL ? (int)blockIdx.y : 0;
    int j, k;
    if (!wave_row(boxes.b[a], j, k)) return;
    if (!VEL) prolong_row<T, D, 0>(gc, gf, boxes.b[0], role, coarse.c[0], fine.c[0], j, k);
    else if (a == 0) prolong_row<T, D, 1>(gc, gf, boxes.b[0], role, coarse.c[0], fine.c[0], j, k);
    else if (a == 1) prolong_row<T, D, 2>(gc, gf, boxes.b[1], role, coarse.c[1], fine.c[1], j, k);
    else if (D == 3) prolong_row<T, D, 4>(gc, gf, boxes.b[2], role, coarse.c[2], fine.c[2], j, k);
}

// ---------------------------------------------------------------------------
// coarsest level: dense inverse, assembled by applying the stencil to unit
// vectors, inverted by Gauss-Jordan with partial pivoting (one workgroup)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_dense_assemble(Grid g, int velocity, int n, const long long *__restrict__ uidx,
                                                        const int *__restrict__ ucomp, CoefP<double> cp,
                                                        CoefU<double> cu, double mass, double cvisc, double *tmp,
                                                        double *Aw)
{
    // block j: column j of A (row-major n x n) = A applied to the unit vector e_j
    const int j = blockIdx.x;
    const int nc = velocity ? g.D : 1;
    const long long nel = g.nel;
    double *base = tmp + (long long)j * nc * nel;
    VelArr<double> x{{base, nc > 1 ? base + nel : nullptr, nc > 2 ? base + 2 * nel : nullptr}};
    for (long long e = threadIdx.x; e < nc * nel; e += blockDim.x) base[e] = 0.0;
    __syncthreads();
    if (threadIdx.x == 0) x.c[velocity ? ucomp[j] : 0][uidx[j]] = 1.0;
    __syncthreads();
    for (int r = threadIdx.x; r < n; r += blockDim.x) {
        int i, jj, k;
        decode(g, uidx[r], i, jj, k);
        double Ax, dg;
        if (velocity) u_row_slow_any<double>(g, x, cu, mass, cvisc, ucomp[r], i, jj, k, Ax, dg);
        else p_row_slow_any<double>(g, x.c[0], cp, cvisc, i, jj, k, Ax, dg);
        Aw[r * n + j] = Ax;
    }
}

// Gauss-Jordan with partial pivoting on [A | I] held in LDS, one workgroup;
// singular (all-Neumann/periodic pressure): A + alpha 1 1^T, alpha = trace / n^2
__global__ void __launch_bounds__(1024) k_dense_gj(int n, int singular, const double *__restrict__ Aw, double *M)
{
    __shared__ double A[DENSE_LDS][DENSE_LDS + 1], B[DENSE_LDS][DENSE_LDS + 1];
    __shared__ double f[DENSE_LDS];
    __shared__ double tr;
    __shared__ int piv;
    const int t = threadIdx.x;
    for (int e = t; e < n * n; e += blockDim.x) {
        const int r = e / n, c = e % n;
        A[r][c] = Aw[e];
        B[r][c] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
    if (singular) {
        if (t == 0) {
            double s = 0.0;
            for (int i = 0; i < n; ++i) s += A[i][i];
            tr = s / ((double)n * (double)n);
        }
        __syncthreads();
        for (int e = t; e < n * n; e += blockDim.x) A[e / n][e % n] += tr;
        __syncthreads();
    }
    for (int k = 0; k < n; ++k) {
        if (t == 0) {
            int p = k;
            for (int i = k + 1; i < n; ++i)
                if (fabs(A[i][k]) > fabs(A[p][k])) p = i;
            piv = p;
        }
        __syncthreads();
        const int p = piv;
        if (p != k && t < n) {
            double v = A[k][t]; A[k][t] = A[p][t]; A[p][t] = v;
            v = B[k][t]; B[k][t] = B[p][t]; B[p][t] = v;
        }
        __syncthreads();
        const double pv = A[k][k];
        __syncthreads();
        if (t < n) {
            A[k][t] /= pv;
            B[k][t] /= pv;
        }
        __syncthreads();
        if (t < n) f[t] = A[t][k];
        __syncthreads();
        for (int e = t; e < n * n; e += blockDim.x) {
            const int r = e / n, c = e % n;
            if (r == k) continue;
            A[r][c] -= f[r] * A[k][c];
            B[r][c] -= f[r] * B[k][c];
        }
        __syncthreads();
    }
    for (int e = t; e < n * n; e += blockDim.x) M[e] = B[e / n][e % n];
}

// x = M b over the coarsest unknowns (M in FP64), ghost images updated
template <typename T>
__global__ void __launch_bounds__(64) k_dense_apply(Grid g, int velocity, int n, const long long *__restrict__ uidx,
                                                    const int *__restrict__ ucomp, const double *__restrict__ M,
                                                    VelArrC<T> b, VelArr<T> x)
{
    __shared__ double bv[64];
    const int r = threadIdx.x;
    if (r < n) bv[r] = (double)b.c[ucomp[r]][uidx[r]];
    __syncthreads();
    if (r < n) {
        double s = 0.0;
        for (int j = 0; j < n; ++j) s += M[r * n + j] * bv[j];
        const int c = ucomp[r];
        x.c[c][uidx[r]] = (T)s;
        int i, jj, k;
        decode(g, uidx[r], i, jj, k);
        write_images(g, velocity ? face_mask(c) : 0, velocity ? ROLE_V : ROLE_P, x.c[c], i, jj, k, (T)s);
    }
}

// ---------------------------------------------------------------------------
// element-wise helpers
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) k_fill(T *p, long long n, T v)
{
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
        p[t] = v;
}

// dst(unknowns) = (Td) src(unknowns)
template <typename Ts, typename Td>
__global__ void __launch_bounds__(256) k_cast_unknowns(Grid g, VelBox boxes, VelArrC<Ts> src, VelArr<Td> dst)
{
    const int a = blockIdx.y;
    int i, j, k;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (!box_pos(boxes.b[a], t, i, j, k)) return;
    const long long e = at(g, i, j, k);
    dst.c[a][e] = (Td)src.c[a][e];
}

// Start of the FP32 inner cycles of a refined iteration, one launch for
// what a cast and a clear per component would do: b32 = (float) r64 at the
// unknowns of each component and x32 = 0 over the whole array (ghosts and
// fixed faces included).  One thread per array entry.
__global__ void __launch_bounds__(256) k_inner_start(Grid g, VelBox boxes, VelArrC<double> r, VelArr<float> b32,
                                                     VelArr<float> x32)
{
    const int a = blockIdx.y;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= g.nel) return;
    x32.c[a][e] = 0.0f;
    int i, j, k;
    decode(g, e, i, j, k);
    const Box &b = boxes.b[a];
    if (i >= b.lo[0] && i < b.lo[0] + b.ext[0] && j >= b.lo[1] && j < b.lo[1] + b.ext[1] && k >= b.lo[2] &&
        k < b.lo[2] + b.ext[2])
        b32.c[a][e] = (float)r.c[a][e];
}

// x(unknowns) += (double) e(unknowns), ghost images of x updated (role:
// velocity components or pressure)
__global__ void __launch_bounds__(256) k_add_correction(Grid g, VelBox boxes, int velocity, VelArrC<float> e,
                                                        VelArr<double> x)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_pos(boxes.b[a], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long q = at(g, i, j, k);
    const double v = x.c[a][q] + (double)e.c[a][q];
    x.c[a][q] = v;
    write_images(g, velocity ? face_mask(a) : 0, velocity ? ROLE_V : ROLE_P, x.c[a], i, j, k, v);
}

// dst(unknowns) = src(unknowns) with the ghost images of dst written; fixed
// positions of dst are left as they are (zero in solver arrays)
template <typename T>
__global__ void __launch_bounds__(256) k_load_unknowns(Grid g, VelBox boxes, int velocity, VelArrC<T> src, VelArr<T> dst)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_pos(boxes.b[a], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    const long long q = at(g, i, j, k);
    const T v = src.c[a] ? src.c[a][q] : T(0);
    dst.c[a][q] = v;
    write_images(g, velocity ? face_mask(a) : 0, velocity ? ROLE_V : ROLE_P, dst.c[a], i, j, k, v);
}

// coefficient ghost layer: every stored position writes its even images
template <typename T>
__global__ void __launch_bounds__(256) k_coef_ghosts(Grid g, CoefSet<T> set)
{
    const int q = blockIdx.y;
    const int vmask = set.vmask[q];
    T *v = set.v[q];
    Box box{{0, 0, 0}, {1, 1, 1}};
    for (int d = 0; d < 3; ++d) box.ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    int i, j, k;
    if (!box_pos(box, blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    write_images(g, vmask, ROLE_C, v, i, j, k, v[at(g, i, j, k)]);
}

// ---------------------------------------------------------------------------
// V-cycle-preconditioned GCR on the finest level (FP64): operator apply,
// inner products over the unknowns, and the two updates.  The scalar
// coefficients stay on the device; every thread forms the same quotient.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) k_apply_u(Grid g, VelBox boxes, VelArr<double> z, CoefU<double> cf,
                                                 double mass, double cvisc, VelArr<double> q)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_pos(boxes.b[a], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    double Ax, dg;
    if (a == 0) u_row<double, D, 0>(g, z, cf, mass, cvisc, i, j, k, Ax, dg);
    else if (a == 1) u_row<double, D, 1>(g, z, cf, mass, cvisc, i, j, k, Ax, dg);
    else u_row<double, D, (D == 3 ? 2 : 1)>(g, z, cf, mass, cvisc, i, j, k, Ax, dg);
    q.c[a][at(g, i, j, k)] = Ax;
}

template <int D>
__global__ void __launch_bounds__(256) k_apply_p(Grid g, Box box, const double *z, CoefP<double> cf, double cvisc,
                                                 double *q)
{
    int i, j, k;
    if (!box_pos(box, blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    double Ax, dg;
    p_row<double, D>(g, z, cf, cvisc, i, j, k, Ax, dg);
    q[at(g, i, j, k)] = Ax;
}

// per-block sums of x . y over the unknowns of every component (blockIdx.y)
__global__ void __launch_bounds__(256) k_dot(VelBox boxes, Grid g, VelArrC<double> x, VelArrC<double> y,
                                             double *partial)
{
    const int a = blockIdx.y;
    const Box box = boxes.b[a];
    const int n = box.ext[0] * box.ext[1] * box.ext[2];
    double acc = 0.0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        int i, j, k;
        box_pos(box, t, i, j, k);
        const long long e = at(g, i, j, k);
        acc += x.c[a][e] * y.c[a][e];
    }
    block_sum_store(acc, partial, (long long)blockIdx.y * gridDim.x + blockIdx.x);
}

// q -= s qi and z -= s zi at the unknowns, s = num / den
__global__ void __launch_bounds__(256) k_gcr_axpy2(Grid g, VelBox boxes, const double *num, const double *den,
                                                   VelArrC<double> qi, VelArrC<double> zi, VelArr<double> q,
                                                   VelArr<double> z)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_pos(boxes.b[a], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    const double sc = num[0] / den[0];
    const long long e = at(g, i, j, k);
    q.c[a][e] -= sc * qi.c[a][e];
    z.c[a][e] -= sc * zi.c[a][e];
}

// x += s z at the unknowns (s = num / den), ghost images of x updated
__global__ void __launch_bounds__(256) k_gcr_update(Grid g, VelBox boxes, int velocity, const double *num,
                                                    const double *den, VelArrC<double> z, VelArr<double> x)
{
    const int a = blockIdx.y;
    int i, j, k;
    if (!box_pos(boxes.b[a], blockIdx.x * blockDim.x + threadIdx.x, i, j, k)) return;
    const double sc = num[0] / den[0];
    const long long e = at(g, i, j, k);
    const double v = x.c[a][e] + sc * z.c[a][e];
    x.c[a][e] = v;
    write_images(g, velocity ? face_mask(a) : 0, velocity ? ROLE_V : ROLE_P, x.c[a], i, j, k, v);
}

// ---------------------------------------------------------------------------
// the coarse part of a V-cycle in one workgroup (its passes: mg_device.h)
// ---------------------------------------------------------------------------
// an array of a staged level: its place in the arena, or (offset -1) the
// array where it already is
template <typename T>
__device__ inline T *arena_ptr(unsigned char *arena, int off, T *global)
{
    return off >= 0 ? reinterpret_cast<T *>(arena + off) : global;
}

// The workgroup's table of levels: the global tables, with the arrays of the
// levels from ls down that the plan places in the LDS arena rebased there.
// Staged coefficients are copied in.  Staged solver arrays are cleared,
// except on the start level l0, whose x and b carry the cycle's input.  Only
// levels ls .. lend - 1 are touched, and of them only the staged arrays.
template <typename T, int D, int VEL>
__device__ inline void stage_levels(const LevTab<T> *__restrict__ tab, int l0, int L, int ls, int lend,
                                    const LdsLevel *__restrict__ lev, unsigned char *arena, LevTab<T> *wt)
{
    for (int l = threadIdx.x; l < L; l += blockDim.x) {
        LevTab<T> t = tab[l];
        if (l >= ls) {
            const LdsLevel o = lev[l];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                t.xu[a] = arena_ptr<T>(arena, o.xu[a], t.xu[a]);
                t.bu[a] = arena_ptr<T>(arena, o.bu[a], t.bu[a]);
                t.ru[a] = arena_ptr<T>(arena, o.ru[a], t.ru[a]);
                t.rho[a] = arena_ptr<T>(arena, o.rho[a], const_cast<T *>(t.rho[a]));
                t.beta[a] = arena_ptr<T>(arena, o.beta[a], const_cast<T *>(t.beta[a]));
                t.mue[a] = arena_ptr<T>(arena, o.mue[a], const_cast<T *>(t.mue[a]));
            }
            t.xp = arena_ptr<T>(arena, o.xp, t.xp);
            t.bp = arena_ptr<T>(arena, o.bp, t.bp);
            t.rp = arena_ptr<T>(arena, o.rp, t.rp);
            t.muc = arena_ptr<T>(arena, o.muc, const_cast<T *>(t.muc));
        }
        wt[l] = t;
    }
    __syncthreads();
    for (int l = ls; l < lend; ++l) {
        const LevTab<T> src = tab[l];
        const LevTab<T> dst = wt[l];
        const bool start = l == l0;
        const int nel = (int)src.g.nel;
        // two elements per round, every load before any store, so that a
        // round costs one trip to global memory
        constexpr int U = 2;
        for (int e0 = threadIdx.x; e0 < nel; e0 += U * blockDim.x) {
            if (VEL) {
                T rh[U][3], xv[U][3], bv[U][3], mc[U], me[U][3];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * blockDim.x;
                    if (e >= nel) break;
#pragma unroll
                    for (int a = 0; a < D; ++a) {
                        if (dst.rho[a] != src.rho[a]) rh[u][a] = src.rho[a][e];
                        xv[u][a] = start ? src.xu[a][e] : T(0);
                        bv[u][a] = start ? src.bu[a][e] : T(0);
                    }
                    if (dst.muc != src.muc) mc[u] = src.muc[e];
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        if (dst.mue[a] && dst.mue[a] != src.mue[a]) me[u][a] = src.mue[a][e];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * blockDim.x;
                    if (e >= nel) break;
#pragma unroll
                    for (int a = 0; a < D; ++a) {
                        if (dst.rho[a] != src.rho[a]) const_cast<T *>(dst.rho[a])[e] = rh[u][a];
                        if (dst.xu[a] != src.xu[a]) dst.xu[a][e] = xv[u][a];
                        if (dst.bu[a] != src.bu[a]) dst.bu[a][e] = bv[u][a];
                        if (dst.ru[a] != src.ru[a]) dst.ru[a][e] = T(0);
                    }
                    if (dst.muc != src.muc) const_cast<T *>(dst.muc)[e] = mc[u];
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        if (dst.mue[a] && dst.mue[a] != src.mue[a]) const_cast<T *>(dst.mue[a])[e] = me[u][a];
                }
            } else {
                T bt[U][3], xv[U], bv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * blockDim.x;
                    if (e >= nel) break;
#pragma unroll
                    for (int a = 0; a < D; ++a)
                        if (dst.beta[a] != src.beta[a]) bt[u][a] = src.beta[a][e];
                    xv[u] = start ? src.xp[e] : T(0);
                    bv[u] = start ? src.bp[e] : T(0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * blockDim.x;
                    if (e >= nel) break;
#pragma unroll
                    for (int a = 0; a < D; ++a)
                        if (dst.beta[a] != src.beta[a]) const_cast<T *>(dst.beta[a])[e] = bt[u][a];
                    if (dst.xp != src.xp) dst.xp[e] = xv[u];
                    if (dst.bp != src.bp) dst.bp[e] = bv[u];
                    if (dst.rp != src.rp) dst.rp[e] = T(0);
                }
            }
        }
    }
    __syncthreads();
}

// a staged start level hands its iterate (with its ghost images) back
template <typename T, int D, int VEL>
__device__ inline void unstage_start(const LevTab<T> *__restrict__ tab, int l0, int ls, const LevTab<T> *wt)
{
    if (l0 < ls) return;
    __syncthreads();
    const LevTab<T> src = wt[l0];
    const LevTab<T> dst = tab[l0];
    const int nel = (int)dst.g.nel;
    for (int e = threadIdx.x; e < nel; e += blockDim.x) {
        if (VEL) {
#pragma unroll
            for (int a = 0; a < D; ++a) dst.xu[a][e] = src.xu[a][e];
        } else {
            dst.xp[e] = src.xp[e];
        }
    }
}

template <typename T, int D, int VEL>
__global__ void __launch_bounds__(wg_threads(D, VEL)) k_coarse_vcycle(const LevTab<T> *__restrict__ tab, int l0, int L, int nu1,
                                                               int nu2, int ndense, const long long *__restrict__ uidx,
                                                               const int *__restrict__ ucomp,
                                                               const double *__restrict__ M, LdsPlan plan, Tail tail)
{
    extern __shared__ __align__(16) unsigned char wg_arena[];
    __shared__ LevTab<T> wt[WG_MAXLEV];
    __shared__ T bv[TAIL_MAX];
    stage_levels<T, D, VEL>(tab, l0, L, plan.ls, tail.n > 0 ? tail.level + 1 : L, plan.lev, wg_arena, wt);
    coarse_cycle<T, D, VEL>(wt, l0, L, nu1, nu2, ndense, uidx, ucomp, M, tail, bv);
    unstage_start<T, D, VEL>(tab, l0, plan.ls, wt);
}

// Column j of a tail's matrix: the cycle from the tail's level down and back,
// on the unit right-hand side of its j-th unknown, every level staged in LDS
// (the plan stages all of them; no level is a start level, so every solver
// array begins at zero).
template <typename T, int D, int VEL>
__global__ void __launch_bounds__(wg_threads(D, VEL)) k_tail_columns(const LevTab<T> *__restrict__ tab, int L, int nu1,
                                                                    int nu2, int ndense,
                                                                    const long long *__restrict__ uidx,
                                                                    const int *__restrict__ ucomp,
                                                                    const double *__restrict__ M, LdsPlan plan,
                                                                    Tail tail)
{
    extern __shared__ __align__(16) unsigned char wg_arena[];
    __shared__ LevTab<T> wt[WG_MAXLEV];
    __shared__ T bv[1];
    const int lt = tail.level;
    const int j = blockIdx.x;
    stage_levels<T, D, VEL>(tab, -1, L, plan.ls, L, plan.lev, wg_arena, wt);
    if (threadIdx.x == 0) {
        const int a = tail.comp[j];
        T *b = VEL ? (a == 0 ? wt[lt].bu[0] : (a == 1 ? wt[lt].bu[1] : wt[lt].bu[2])) : wt[lt].bp;
        b[tail.idx[j]] = T(1);
    }
    __syncthreads();
    const Tail none{nullptr, nullptr, nullptr, 0, 0};
    coarse_cycle<T, D, VEL>(wt, lt, L, nu1, nu2, ndense, uidx, ucomp, M, none, bv);
    __syncthreads();
    T *Tm = const_cast<T *>(static_cast<const T *>(tail.Tm));
    for (int r = threadIdx.x; r < tail.n; r += blockDim.x) {
        const int a = tail.comp[r];
        const T *x = VEL ? (a == 0 ? wt[lt].xu[0] : (a == 1 ? wt[lt].xu[1] : wt[lt].xu[2])) : wt[lt].xp;
        Tm[tail_at<T>(tail.n, r, j)] = x[tail.idx[r]];
    }
}

// ---------------------------------------------------------------------------
// batched passes: one launch covers the same pass of several contexts.
// Block b of a launch works for the context described by ent[b]; a context
// whose flag is clear is skipped.  Each point is updated exactly as by the
// single-context kernels above.
// ---------------------------------------------------------------------------
template <typename T>
__device__ inline const LevTab<T> &tab_of(const void *p) { return *static_cast<const LevTab<T> *>(p); }

// A copy of the i-th level table at p, read through scalar loads.  The tables
// are written once when a context is created and every lane of a block reads
// the same one; through a generic pointer they would come in with vector
// loads, one more round trip that the row's own loads wait behind.
template <typename T>
__device__ inline LevTab<T> tab_copy(const void *p, int i = 0)
{
    constexpr int N = sizeof(LevTab<T>) / 4;
    static_assert(sizeof(LevTab<T>) % 4 == 0, "the table is read in 4-byte words");
    typedef const __attribute__((address_space(4))) unsigned int ConstWord;
    const ConstWord *w = (const ConstWord *)p + (long long)i * N;
    struct Words {
        unsigned int v[N];
    } r;
#pragma unroll
    for (int k = 0; k < N; ++k) r.v[k] = w[k];
    return __builtin_bit_cast(LevTab<T>, r);
}

template <typename T, int D, int VEL, int A>
__global__ void __launch_bounds__(256) k_bsweep(const BEntry *__restrict__ ent, const int *__restrict__ flags,
                                                int colour)
{
    const BEntry E = ent[blockIdx.x];
    const int on = flags[E.ctx];
    const LevTab<T> lt = tab_copy<T>(E.tab);
    if (!on) return;
    const Box box = unk_box(lt.g, VEL ? face_mask(A) : 0);
    sweep_at<T, D, VEL, A>(lt, box, colour, (int)(blockIdx.x - E.base) * blockDim.x + threadIdx.x);
}

// residual of every component (blockIdx.y) with a grid-stride loop over the
// context's nb blocks; with E.partial set, per-block sums of r^2 in the
// layout of the single-context residual kernels
template <typename T, int D, int VEL>
__global__ void __launch_bounds__(256) k_bresid(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    const int on = flags[E.ctx];
    const LevTab<T> lt = tab_copy<T>(E.tab);
    if (!on) return;
    const int a = blockIdx.y;
    const int lb = blockIdx.x - E.base;
    const Box box = unk_box(lt.g, VEL ? face_mask(a) : 0);
    const int n = point_count(box);
    double acc = 0.0;
    for (int t = lb * blockDim.x + threadIdx.x; t < n; t += E.nb * blockDim.x) {
        T rv;
        if (a == 0) rv = resid_at<T, D, VEL, 0>(lt, box, t);
        else if (a == 1) rv = resid_at<T, D, VEL, 1>(lt, box, t);
        else rv = resid_at<T, D, VEL, (D == 3 ? 2 : 1)>(lt, box, t);
        acc += (double)rv * (double)rv;
    }
    if (E.partial) block_sum_store(acc, E.partial, (long long)a * E.nb + lb);
}

// the velocity residual of large members with its norm, rows by waves: the
// blocks, rounds and sums of k_resid_u_rows
template <typename T, int D>
__global__ void __launch_bounds__(256) k_bresid_rows(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    const int on = flags[E.ctx];
    const LevTab<T> lt = tab_copy<T>(E.tab);
    if (!on) return;
    const unsigned lb = blockIdx.x - E.base;
    const ResidRows R = resid_rows(lt.g);
    VelBox boxes;
    for (int a = 0; a < D; ++a) boxes.b[a] = unk_box(lt.g, face_mask(a));
    const VelArr<T> x{{lt.xu[0], lt.xu[1], lt.xu[2]}}, r{{lt.ru[0], lt.ru[1], lt.ru[2]}};
    const VelArrC<T> b{{lt.bu[0], lt.bu[1], lt.bu[2]}};
    double acc[3] = {0.0, 0.0, 0.0};
    for (unsigned blk = xcd_block(R.remap, lb, R.nb); blk < R.blocks; blk += R.nb)
        resid_u_block<T, D, true>(lt.g, R.all, boxes, b, x, coef_u(lt), lt.mass, lt.cvu, r, 0, D, blk, acc);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        block_sum_store(acc[a], E.partial, (long long)a * R.nb + lb);
        __syncthreads();
    }
}

// one block per context: norms[ctx] = sum of its E.nb partial sums, in the
// order of the single-context final reduction
__global__ void __launch_bounds__(256) k_breduce(const BEntry *__restrict__ ent, const int *__restrict__ flags,
                                                 double *norms)
{
    const BEntry E = ent[blockIdx.x];
    if (!flags[E.ctx]) return;
    double acc = 0.0;
    for (long long t = threadIdx.x; t < E.nb; t += blockDim.x) acc += E.partial[t];
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) norms[E.ctx] = red[0];
}

// restriction to the next level (the context's table at l and l + 1)
template <typename T, int D, int VEL>
__global__ void __launch_bounds__(256) k_brestrict(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    if (!flags[E.ctx]) return;
    const LevTab<T> lt = tab_copy<T>(E.tab, 0);
    const LevTab<T> lc = tab_copy<T>(E.tab, 1);
    const int a = blockIdx.y;
    const Box box = unk_box(lc.g, VEL ? face_mask(a) : 0);
    const int t = (blockIdx.x - E.base) * blockDim.x + threadIdx.x;
    if (t >= point_count(box)) return;
    if (a == 0) restrict_at<T, D, VEL, 0>(lt, lc, box, t);
    else if (a == 1) restrict_at<T, D, VEL, 1>(lt, lc, box, t);
    else restrict_at<T, D, VEL, (D == 3 ? 2 : 1)>(lt, lc, box, t);
}

template <typename T, int D, int VEL>
__global__ void __launch_bounds__(256) k_bprolong(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    if (!flags[E.ctx]) return;
    const LevTab<T> lt = tab_copy<T>(E.tab, 0);
    const LevTab<T> lc = tab_copy<T>(E.tab, 1);
    const int a = blockIdx.y;
    const Box box = unk_box(lt.g, VEL ? face_mask(a) : 0);
    const int t = (blockIdx.x - E.base) * blockDim.x + threadIdx.x;
    if (t >= point_count(box)) return;
    if (a == 0) prolong_at<T, D, VEL, 0>(lc, lt, box, t);
    else if (a == 1) prolong_at<T, D, VEL, 1>(lc, lt, box, t);
    else prolong_at<T, D, VEL, (D == 3 ? 2 : 1)>(lc, lt, box, t);
}

// refined solver, start of an outer iteration: FP32 right-hand side = the
// FP64 residual at the unknowns, FP32 correction cleared (whole arrays)
template <int VEL>
__global__ void __launch_bounds__(256) k_bprep32(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    if (!flags[E.ctx]) return;
    const LevTab<double> &l64 = tab_of<double>(E.tab);
    const LevTab<float> &l32 = tab_of<float>(E.tab2);
    const int t = (blockIdx.x - E.base) * blockDim.x + threadIdx.x;
    const int ncomp = VEL ? l64.g.D : 1;
    for (int a = 0; a < ncomp; ++a) {
        float *x32 = VEL ? l32.xu[a] : l32.xp;
        if (t < l64.g.nel) x32[t] = 0.0f;
        const Box box = unk_box(l64.g, VEL ? face_mask(a) : 0);
        int i, j, k;
        if (t < point_count(box)) {
            box_pos(box, t, i, j, k);
            const long long e = at(l64.g, i, j, k);
            (VEL ? l32.bu[a] : l32.bp)[e] = (float)(VEL ? l64.ru[a] : l64.rp)[e];
        }
    }
}

// refined solver, end of an outer iteration: x += (double) e at the unknowns
template <int VEL>
__global__ void __launch_bounds__(256) k_badd(const BEntry *__restrict__ ent, const int *__restrict__ flags)
{
    const BEntry E = ent[blockIdx.x];
    if (!flags[E.ctx]) return;
    const LevTab<double> &l64 = tab_of<double>(E.tab);
    const LevTab<float> &l32 = tab_of<float>(E.tab2);
    const int a = blockIdx.y;
    const int vmask = VEL ? face_mask(a) : 0;
    const Box box = unk_box(l64.g, vmask);
    const int t = (blockIdx.x - E.base) * blockDim.x + threadIdx.x;
    if (t >= point_count(box)) return;
    int i, j, k;
    box_pos(box, t, i, j, k);
    const long long q = at(l64.g, i, j, k);
    double *x = VEL ? l64.xu[a] : l64.xp;
    const double v = x[q] + (double)(VEL ? l32.xu[a] : l32.xp)[q];
    x[q] = v;
    write_images(l64.g, vmask, VEL ? ROLE_V : ROLE_P, x, i, j, k, v);
}

// the coarse part of the V-cycle of every context, one workgroup each
template <typename T, int D, int VEL>
__global__ void __launch_bounds__(wg_threads(D, VEL)) k_bcoarse(const BCoarse *__restrict__ items, const int *__restrict__ flags,
                                                  int nu1, int nu2)
{
    const BCoarse I = items[blockIdx.x];
    if (!flags[I.ctx]) return;
    extern __shared__ __align__(16) unsigned char wg_arena[];
    __shared__ LevTab<T> wt[WG_MAXLEV];
    __shared__ T bv[TAIL_MAX];
    const LevTab<T> *tab = static_cast<const LevTab<T> *>(I.tab);
    stage_levels<T, D, VEL>(tab, I.l0, I.L, I.lds_from, I.tail.n > 0 ? I.tail.level + 1 : I.L, I.lds, wg_arena, wt);
    coarse_cycle<T, D, VEL>(wt, I.l0, I.L, nu1, nu2, I.ndense, I.uidx, I.ucomp, I.M, I.tail, bv);
    unstage_start<T, D, VEL>(tab, I.l0, I.lds_from, wt);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(long long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

// events armed for the next timed launch (set_launch_events): the kernel's
// own start and end are recorded into them by the dispatch
static thread_local hipEvent_t t_ev_start = nullptr, t_ev_stop = nullptr;

void set_launch_events(hipEvent_t start, hipEvent_t stop)
{
    t_ev_start = start;
    t_ev_stop = stop;
}

bool take_launch_events(hipEvent_t *start, hipEvent_t *stop)
{
    if (!t_ev_start) return false;
    *start = t_ev_start;
    *stop = t_ev_stop;
    t_ev_start = t_ev_stop = nullptr;
    return true;
}

static inline long long box_count(const Box &b) { return (long long)b.ext[0] * b.ext[1] * b.ext[2]; }

// rows per band of a z-blocked pass: about one point of the colour per
// thread in each plane, at least 4 rows
static inline int zb_rows(const Box &P) { return std::max(4, 256 / std::max(1, (P.ext[0] + 1) / 2)); }

template <typename T>
void launch_smooth_p(const Grid &g, const T *b, T *x, const CoefP<T> &cf, T cvisc, int colour, hipStream_t s, int zb)
{
    const Box P = unk_box(g, 0);
    const long long n = (long long)((P.ext[0] + 1) / 2) * P.ext[1] * P.ext[2];
    if (n <= 0) return;
    if (zb && g.D == 3) {
        const int rows = zb_rows(P), nbands = (P.ext[1] + rows - 1) / rows;
        const int nz = (P.ext[2] + ZB_PLANES - 1) / ZB_PLANES;
        launch_timed(k_smooth_p_zb<T>, dim3((unsigned)(nbands * nz)), dim3(256), s, g, P, b, x, cf, cvisc, colour, rows,
                     nbands);
        return;
    }
    const int remap = xcd_remap(g, P, blocks_for(n));
    if (g.D == 3)
        launch_timed(k_smooth_p<T, 3>, dim3(blocks_for(n)), dim3(256), s, g, P, b, x, cf, cvisc, colour, remap);
    else
        launch_timed(k_smooth_p<T, 2>, dim3(blocks_for(n)), dim3(256), s, g, P, b, x, cf, cvisc, colour, remap);
}

template <typename T>
void launch_smooth_u(const Grid &g, int a, const T *b, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc,
                     int colour, hipStream_t s, int zb)
{
    const Box P = unk_box(g, face_mask(a));
    const long long n = (long long)((P.ext[0] + 1) / 2) * P.ext[1] * P.ext[2];
    if (n <= 0) return;
    if (zb && g.D == 3) {
        const int rows = zb_rows(P), nbands = (P.ext[1] + rows - 1) / rows;
        const int nz = (P.ext[2] + ZB_PLANES - 1) / ZB_PLANES;
        const dim3 grid((unsigned)(nbands * nz)), blk(256);
        if (a == 0) launch_timed(k_smooth_u_zb<T, 0>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, rows, nbands);
        else if (a == 1) launch_timed(k_smooth_u_zb<T, 1>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, rows, nbands);
        else launch_timed(k_smooth_u_zb<T, 2>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, rows, nbands);
        return;
    }
    const dim3 grid(blocks_for(n)), blk(256);
    const int remap = xcd_remap(g, P, blocks_for(n));
    if (g.D == 3) {
        if (a == 0) launch_timed(k_smooth_u<T, 3, 0>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, remap);
        else if (a == 1) launch_timed(k_smooth_u<T, 3, 1>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, remap);
        else launch_timed(k_smooth_u<T, 3, 2>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, remap);
    } else {
        if (a == 0) launch_timed(k_smooth_u<T, 2, 0>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, remap);
        else launch_timed(k_smooth_u<T, 2, 1>, grid, blk, s, g, P, b, x, cf, mass, cvisc, colour, remap);
    }
}

template <typename T>
void launch_smooth_u_dec(const Grid &g, const VelArrC<T> &b, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc,
                         int colour, hipStream_t s)
{
    VelBox parts;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        parts.b[a] = a < g.D ? unk_box(g, face_mask(a)) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a >= g.D) continue;
        const Box &P = parts.b[a];
        const long long n = (long long)((P.ext[0] + 1) / 2) * P.ext[1] * P.ext[2];
        mx = n > mx ? n : mx;
    }
    if (mx <= 0) return;
    const dim3 grid(blocks_for(mx), g.D), blk(256);
    const int remap = xcd_remap(g, parts.b[0], blocks_for(mx));
    if (g.D == 3) launch_timed(k_smooth_u_dec<T, 3>, grid, blk, s, g, parts, b, x, cf, mass, cvisc, colour, remap);
    else launch_timed(k_smooth_u_dec<T, 2>, grid, blk, s, g, parts, b, x, cf, mass, cvisc, colour, remap);
}

template <typename T>
void launch_smooth_rb(const Grid &g, int vel, int a, const VelArrC<T> &xin, const T *b, const CoefU<T> &cu,
                      const CoefP<T> &cp, T mass, T cvisc, T *xout, hipStream_t s)
{
    const Box P = unk_box(g, vel ? face_mask(a) : 0);
    if (box_count(P) <= 0) return;
    const int D = g.D;
    const int TX = D == 3 ? 8 : 16, TY = D == 3 ? 8 : 16, TZ = D == 3 ? (sizeof(T) == 8 ? 4 : 8) : 1;
    const unsigned nt = (unsigned)(((P.ext[0] + TX - 1) / TX) * ((P.ext[1] + TY - 1) / TY) * ((P.ext[2] + TZ - 1) / TZ));
    const dim3 grid(nt), blk(256);
#define RB(DD, VV, AA) launch_timed(k_smooth_rb<T, DD, VV, AA>, grid, blk, s, g, P, xin, b, cu, cp, mass, cvisc, xout)
    if (D == 3) {
        if (!vel) RB(3, 0, 0);
        else if (a == 0) RB(3, 1, 0);
        else if (a == 1) RB(3, 1, 1);
        else RB(3, 1, 2);
    } else {
        if (!vel) RB(2, 0, 0);
        else if (a == 0) RB(2, 1, 0);
        else RB(2, 1, 1);
    }
#undef RB
}

// Runs of planes per workgroup for the z-marching sweep: about
// ZM_TARGET_BLOCKS workgroups, at least ZM_MIN_RUN planes each (each run also
// updates the red points of the two planes around it).
constexpr int ZM_TARGET_BLOCKS = 8192, ZM_MIN_RUN = 4;

int zm_run(const Box &P)
{
    const long long tiles = (long long)((P.ext[0] + ZM_TX - 1) / ZM_TX) * ((P.ext[1] + ZM_TY - 1) / ZM_TY);
    const long long want = std::max<long long>(1, (ZM_TARGET_BLOCKS + tiles - 1) / tiles);
    const int runs = (int)std::max<long long>(1, std::min<long long>(want, P.ext[2] / ZM_MIN_RUN));
    return (P.ext[2] + runs - 1) / runs;
}

bool zm_fits(const Grid &g)
{
    if (g.D != 3) return false;
    const int need[3] = {ZM_WX, ZM_WY, ZM_NS + 2};
    for (int d = 0; d < 3; ++d)
        if (g.bc[d] == AX_PERIODIC && (g.n[d] < need[d] || g.n[d] % 2)) return false;
    return true;
}

template <typename T>
void launch_smooth_zm(const Grid &g, int a, const VelArrC<T> &xin, const T *b, const CoefU<T> &cu, T mass, T cvisc,
                      T *xout, hipStream_t s)
{
    const Box P = unk_box(g, face_mask(a));
    if (box_count(P) <= 0) return;
    const int cz = zm_run(P);
    const long long nb = (long long)((P.ext[0] + ZM_TX - 1) / ZM_TX) * ((P.ext[1] + ZM_TY - 1) / ZM_TY) *
                         ((P.ext[2] + cz - 1) / cz);
    const dim3 grid((unsigned)nb), blk(ZM_BS);
    const int remap = -1;
#define ZM(AA) launch_timed(k_smooth_zm<T, AA>, grid, blk, s, g, P, xin, b, cu, mass, cvisc, xout, cz, remap)
    if (a == 0) ZM(0);
    else if (a == 1) ZM(1);
    else ZM(2);
#undef ZM
}

static inline unsigned stride_blocks(long long n)
{
    const unsigned b = blocks_for(n);
    const long long want = std::max<long long>(NORM_BLOCKS, (n + 256 * 16 - 1) / (256 * 16));
    const unsigned cap = (unsigned)std::min<long long>(want, NORM_BLOCKS_MAX);
    return b < cap ? (b ? b : 1) : cap;
}

template <typename T>
int launch_resid_p(const Grid &g, const T *b, const T *x, const CoefP<T> &cf, T cvisc, T *r, double *partial,
                   hipStream_t s)
{
    const Box P = unk_box(g, 0);
    const unsigned nb = stride_blocks(box_count(P));
    if (g.D == 3) launch_timed(k_resid_p<T, 3>, dim3(nb), dim3(256), s, g, P, b, x, cf, cvisc, r, partial);
    else launch_timed(k_resid_p<T, 2>, dim3(nb), dim3(256), s, g, P, b, x, cf, cvisc, r, partial);
    return (int)nb;
}

template <typename T>
int launch_resid_u(const Grid &g, const VelArrC<T> &b, const VelArr<T> &x, const CoefU<T> &cf, T mass, T cvisc,
                   const VelArr<T> &r, double *partial, hipStream_t s)
{
    VelBox parts;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        parts.b[a] = a < g.D ? unk_box(g, face_mask(a)) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < g.D && box_count(parts.b[a]) > mx) mx = box_count(parts.b[a]);
    }
    const ResidRows R = resid_rows(g);
    if (rows_by_waves(parts.b[0]) && (R.large || !partial)) {
        const unsigned nb = partial ? R.nb : R.blocks;
        const dim3 grid(nb, R.large ? 1 : g.D), blk(256);
        const int nc = R.large ? g.D : 1;
#define LAUNCH(DD, NN)                                                                                             \
    launch_timed(k_resid_u_rows<T, DD, NN>, grid, blk, s, g, R.all, parts, b, x, cf, mass, cvisc, r, nc, R.remap, \
                 R.blocks, partial)
        if (g.D == 3) {
            if (partial) LAUNCH(3, true);
            else LAUNCH(3, false);
        } else {
            if (partial) LAUNCH(2, true);
            else LAUNCH(2, false);
        }
#undef LAUNCH
        return (int)nb * g.D;
    }
    const unsigned nb = stride_blocks(mx);
    if (g.D == 3)
        launch_timed(k_resid_u<T, 3>, dim3(nb, 3), dim3(256), s, g, parts, b, x, cf, mass, cvisc, r, partial);
    else
        launch_timed(k_resid_u<T, 2>, dim3(nb, 2), dim3(256), s, g, parts, b, x, cf, mass, cvisc, r, partial);
    return (int)nb * g.D;
}

template <typename T>
int launch_norm2(const Grid &g, int ncomp, const int *vmasks, const VelArrC<T> &v, double *partial, hipStream_t s)
{
    VelBox boxes;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        boxes.b[a] = a < ncomp ? unk_box(g, vmasks[a]) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < ncomp && box_count(boxes.b[a]) > mx) mx = box_count(boxes.b[a]);
    }
    const unsigned nb = stride_blocks(mx);
    launch_timed(k_norm2<T>, dim3(nb, ncomp), dim3(256), s, boxes, g, v, partial);
    return (int)nb * ncomp;
}

void launch_reduce_final(const double *partial, long long n, double *out, hipStream_t s)
{
    launch_timed(k_reduce_final, dim3(1), dim3(256), s, partial, n, out);
}

static inline Box stored_box(const Grid &g, int vmask)
{
    Box b;
    for (int d = 0; d < 3; ++d) {
        b.lo[d] = 0;
        b.ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    }
    return b;
}

template <typename T>
void launch_restrict(const Grid &gf, const Grid &gc, int ncomp, const int *vmasks, int role, bool all_stored,
                     const VelArrC<T> &fine, const VelArr<T> &coarse, T scale, hipStream_t s,
                     const VelArr<T> *zero_x)
{
    VelBox parts;
    int masks = 0;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        if (a < ncomp) {
            parts.b[a] = all_stored ? stored_box(gc, vmasks[a]) : unk_box(gc, vmasks[a]);
            masks |= vmasks[a] << (4 * a);
            mx = box_count(parts.b[a]) > mx ? box_count(parts.b[a]) : mx;
        } else {
            parts.b[a] = parts.b[0];
        }
    }
    const VelArr<T> zx = zero_x ? *zero_x : VelArr<T>{{nullptr, nullptr, nullptr}};
    if (mx <= 0) return;
    if (gf.D == 3)
        launch_timed(k_restrict<T, 3>, dim3(blocks_for(mx), ncomp), dim3(256), s, gf, gc, parts, masks, role, fine,
                     coarse, scale, zx);
    else
        launch_timed(k_restrict<T, 2>, dim3(blocks_for(mx), ncomp), dim3(256), s, gf, gc, parts, masks, role, fine,
                     coarse, scale, zx);
}

// Interpolation by rows: of the pressure or of the velocity's components, from
// 2^21 points a component on (at 64 x 64 x 128 and 96 x 96 x 192 in FP64 both
// forms take the same time, 15.4 and 16.2 us), and rows that fill most of
// their waves
constexpr long long PROLONG_ROWS_MIN = 1ll << 21;

static bool prolong_by_rows(const VelBox &parts, int ncomp, int masks, int role, long long points)
{
    bool rows = (role == ROLE_P && masks == 0) || (role == ROLE_V && masks == (ncomp == 3 ? 0x421 : 0x21));
    for (int a = 0; a < ncomp; ++a) rows = rows && rows_by_waves(parts.b[a]);
    return rows && points >= PROLONG_ROWS_MIN;
}
static unsigned wave_row_blocks(const Box &b)
{
    return (unsigned)(((long long)b.ext[1] * b.ext[2] + ROW_WAVES - 1) / ROW_WAVES);
}

template <typename T>
void launch_prolong_add(const Grid &gc, const Grid &gf, int ncomp, const int *vmasks, int role,
                        const VelArrC<T> &coarse, const VelArr<T> &fine, hipStream_t s)
{
    VelBox parts;
    int masks = 0;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        if (a < ncomp) {
            parts.b[a] = unk_box(gf, vmasks[a]);
            masks |= vmasks[a] << (4 * a);
            mx = box_count(parts.b[a]) > mx ? box_count(parts.b[a]) : mx;
        } else {
            parts.b[a] = parts.b[0];
        }
    }
    if (mx <= 0) return;
    if (prolong_by_rows(parts, ncomp, masks, role, mx)) {
        unsigned nb = 1;
        for (int a = 0; a < ncomp; ++a) nb = std::max(nb, wave_row_blocks(parts.b[a]));
        const dim3 grid(nb, ncomp), blk(256);
#define LAUNCH(DD, VV) launch_timed(k_prolong_rows<T, DD, VV>, grid, blk, s, gc, gf, parts, role, coarse, fine)
        if (gf.D == 3) {
            if (masks) LAUNCH(3, true);
            else LAUNCH(3, false);
        } else {
            if (masks) LAUNCH(2, true);
            else LAUNCH(2, false);
        }
#undef LAUNCH
        return;
    }
    if (gf.D == 3)
        launch_timed(k_prolong_add<T, 3>, dim3(blocks_for(mx), ncomp), dim3(256), s, gc, gf, parts, masks, role,
                     coarse, fine);
    else
        launch_timed(k_prolong_add<T, 2>, dim3(blocks_for(mx), ncomp), dim3(256), s, gc, gf, parts, masks, role,
                     coarse, fine);
}

void launch_dense_inverse(const Grid &g, int velocity, int n, const long long *uidx, const int *ucomp,
                          const CoefP<double> &cp, const CoefU<double> &cu, double mass, double cvisc, double *tmp,
                          int singular, double *Aw, double *M, hipStream_t s)
{
    if (n <= 0 || n > DENSE_LDS) return;
    hipLaunchKernelGGL(k_dense_assemble, dim3(n), dim3(256), 0, s, g, velocity, n, uidx, ucomp, cp, cu, mass, cvisc,
                       tmp, Aw);
    hipLaunchKernelGGL(k_dense_gj, dim3(1), dim3(1024), 0, s, n, singular, Aw, M);
}

void launch_dense_gj(int n, int singular, const double *Aw, double *M, hipStream_t s)
{
    if (n <= 0 || n > DENSE_LDS) return;
    hipLaunchKernelGGL(k_dense_gj, dim3(1), dim3(1024), 0, s, n, singular, Aw, M);
}

template <typename T>
void launch_dense_apply(const Grid &g, int velocity, int n, const long long *uidx, const int *ucomp, const double *M,
                        const VelArrC<T> &b, const VelArr<T> &x, hipStream_t s)
{
    launch_timed(k_dense_apply<T>, dim3(1), dim3(64), s, g, velocity, n, uidx, ucomp, M, b, x);
}

template <typename T>
void launch_fill(T *p, long long n, T v, hipStream_t s)
{
    unsigned nb = blocks_for(n);
    if (nb > 2048) nb = 2048;
    if (nb == 0) nb = 1;
    launch_timed(k_fill<T>, dim3(nb), dim3(256), s, p, n, v);
}

template <typename Ts, typename Td>
void launch_cast_unknowns(const Grid &g, int ncomp, const int *vmasks, const VelArrC<Ts> &src, const VelArr<Td> &dst,
                          hipStream_t s)
{
    VelBox boxes;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        boxes.b[a] = a < ncomp ? unk_box(g, vmasks[a]) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < ncomp && box_count(boxes.b[a]) > mx) mx = box_count(boxes.b[a]);
    }
    launch_timed(k_cast_unknowns<Ts, Td>, dim3(blocks_for(mx), ncomp), dim3(256), s, g, boxes, src, dst);
}

void launch_inner_start(const Grid &g, int ncomp, const int *vmasks, const VelArrC<double> &r, const VelArr<float> &b32,
                        const VelArr<float> &x32, hipStream_t s)
{
    VelBox boxes;
    for (int a = 0; a < 3; ++a) boxes.b[a] = a < ncomp ? unk_box(g, vmasks[a]) : Box{{0, 0, 0}, {0, 0, 0}};
    launch_timed(k_inner_start, dim3(blocks_for(g.nel), ncomp), dim3(256), s, g, boxes, r, b32, x32);
}

void launch_add_correction(const Grid &g, int ncomp, const int *vmasks, const VelArrC<float> &e,
                           const VelArr<double> &x, hipStream_t s)
{
    const int velocity = vmasks[0] != 0 ? 1 : 0;
    VelBox boxes;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        boxes.b[a] = a < ncomp ? unk_box(g, vmasks[a]) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < ncomp && box_count(boxes.b[a]) > mx) mx = box_count(boxes.b[a]);
    }
    launch_timed(k_add_correction, dim3(blocks_for(mx), ncomp), dim3(256), s, g, boxes, velocity, e, x);
}

template <typename T>
void launch_load_unknowns(const Grid &g, int ncomp, const int *vmasks, const VelArrC<T> &src, const VelArr<T> &dst,
                          hipStream_t s)
{
    VelBox boxes;
    long long mx = 0;
    for (int a = 0; a < 3; ++a) {
        boxes.b[a] = a < ncomp ? unk_box(g, vmasks[a]) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < ncomp && box_count(boxes.b[a]) > mx) mx = box_count(boxes.b[a]);
    }
    const int velocity = vmasks[0] != 0 ? 1 : 0;
    launch_timed(k_load_unknowns<T>, dim3(blocks_for(mx), ncomp), dim3(256), s, g, boxes, velocity, src, dst);
}

template <typename T>
void launch_coef_ghosts(const Grid &g, const CoefSet<T> &set, hipStream_t s)
{
    long long mx = 0;
    for (int q = 0; q < set.n; ++q) mx = std::max(mx, box_count(stored_box(g, set.vmask[q])));
    if (set.n > 0 && mx > 0)
        hipLaunchKernelGGL(k_coef_ghosts<T>, dim3(blocks_for(mx), set.n), dim3(256), 0, s, g, set);
}

int wg_lds_budget()
{
    static int budget = -1;
    if (budget < 0) {
        int dev = 0, v = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) v = 65536;
        // the kernel's own shared data: the level table, the coarsest
        // right-hand side and the tail's right-hand side
        budget = v - (int)(WG_MAXLEV * sizeof(LevTab<double>)) - 1024 - (int)(TAIL_MAX * sizeof(double));
        if (budget < 0) budget = 0;
    }
    return budget;
}

// allow a dynamic arena above the default limit (once per kernel)
template <typename K>
static void allow_lds(K kernel, int bytes)
{
    static int allowed = 0;
    if (bytes > allowed) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                bytes) == hipSuccess)
            allowed = bytes;
    }
}

// raise the dynamic-LDS limit of every one-workgroup kernel to the full
// budget once, so that no launch needs the attribute call (which has no
// place inside a captured graph)
void wg_prepare()
{
    const int b = wg_lds_budget();
#define PREP(T, DD, VV)                              \
    do {                                             \
        allow_lds(k_coarse_vcycle<T, DD, VV>, b);    \
        allow_lds(k_bcoarse<T, DD, VV>, b);          \
        allow_lds(k_tail_columns<T, DD, VV>, b);     \
    } while (0)
    PREP(double, 2, 0); PREP(double, 2, 1); PREP(double, 3, 0); PREP(double, 3, 1);
    PREP(float, 2, 0); PREP(float, 2, 1); PREP(float, 3, 0); PREP(float, 3, 1);
#undef PREP
}

template <typename T>
void launch_coarse_vcycle(int D, const LevTab<T> *tab, int l0, int L, int vel, int nu1, int nu2, int ndense,
                          const long long *uidx, const int *ucomp, const double *M, const LdsPlan &plan,
                          const Tail &tail, hipStream_t s)
{
#define LAUNCH(DD, VV)                                                                                              \
    do {                                                                                                            \
        allow_lds(k_coarse_vcycle<T, DD, VV>, plan.bytes);                                                          \
        launch_timed_shm(k_coarse_vcycle<T, DD, VV>, dim3(1), dim3(wg_threads(DD, VV)), plan.bytes, s, tab, l0, L, \
                         nu1, nu2, ndense, uidx, ucomp, M, plan, tail);                                             \
    } while (0)
    if (D == 3) {
        if (vel) LAUNCH(3, 1);
        else LAUNCH(3, 0);
    } else {
        if (vel) LAUNCH(2, 1);
        else LAUNCH(2, 0);
    }
#undef LAUNCH
}
template void launch_coarse_vcycle<double>(int, const LevTab<double> *, int, int, int, int, int, int,
                                           const long long *, const int *, const double *, const LdsPlan &,
                                           const Tail &, hipStream_t);
template void launch_coarse_vcycle<float>(int, const LevTab<float> *, int, int, int, int, int, int,
                                          const long long *, const int *, const double *, const LdsPlan &,
                                          const Tail &, hipStream_t);

template <typename T>
void launch_tail_columns(int D, const LevTab<T> *tab, int L, int vel, int nu1, int nu2, int ndense,
                         const long long *uidx, const int *ucomp, const double *M, const LdsPlan &plan,
                         const Tail &tail, hipStream_t s)
{
    if (tail.n <= 0) return;
#define LAUNCH(DD, VV)                                                                                              \
    do {                                                                                                            \
        allow_lds(k_tail_columns<T, DD, VV>, plan.bytes);                                                           \
        hipLaunchKernelGGL((k_tail_columns<T, DD, VV>), dim3(tail.n), dim3(wg_threads(DD, VV)), plan.bytes, s, tab, \
                           L, nu1, nu2, ndense, uidx, ucomp, M, plan, tail);                                         \
    } while (0)
    if (D == 3) {
        if (vel) LAUNCH(3, 1);
        else LAUNCH(3, 0);
    } else {
        if (vel) LAUNCH(2, 1);
        else LAUNCH(2, 0);
    }
#undef LAUNCH
}
template void launch_tail_columns<double>(int, const LevTab<double> *, int, int, int, int, int, const long long *,
                                          const int *, const double *, const LdsPlan &, const Tail &, hipStream_t);
template void launch_tail_columns<float>(int, const LevTab<float> *, int, int, int, int, int, const long long *,
                                         const int *, const double *, const LdsPlan &, const Tail &, hipStream_t);

int norm_pass(const Grid &g, int vel) { return vel && resid_rows(g).norm ? BK_RESID_ROWS : BK_RESID; }

int batch_blocks(int kind, const Grid &g, const Grid &gc, int vel, int A)
{
    const int nc = vel ? g.D : 1;
    long long mx = 0;
    switch (kind) {
    case BK_SWEEP: {
        const Box b = unk_box(g, vel ? face_mask(A) : 0);
        return (int)blocks_for((long long)((b.ext[0] + 1) / 2) * b.ext[1] * b.ext[2]);
    }
    case BK_RESID:
        for (int a = 0; a < nc; ++a) mx = std::max(mx, box_count(unk_box(g, vel ? face_mask(a) : 0)));
        return (int)stride_blocks(mx);
    case BK_RESID_ROWS: return (int)resid_rows(g).nb;
    case BK_RESTRICT:
        for (int a = 0; a < nc; ++a) mx = std::max(mx, box_count(unk_box(gc, vel ? face_mask(a) : 0)));
        return (int)blocks_for(mx);
    case BK_PROLONG:
    case BK_ADD:
        for (int a = 0; a < nc; ++a) mx = std::max(mx, box_count(unk_box(g, vel ? face_mask(a) : 0)));
        return (int)blocks_for(mx);
    case BK_PREP: return (int)blocks_for(g.nel);
    }
    return 0;
}

template <typename T>
void launch_bpass(int kind, int D, int vel, int A, int colour, const BEntry *ent, unsigned nblocks, const int *flags,
                  hipStream_t s)
{
    if (nblocks == 0) return;
    const dim3 blk(256);
    const dim3 gc(nblocks, vel ? D : 1);
#define PASS3(K, ...)                                                                                               \
    do {                                                                                                            \
        if (vel) hipLaunchKernelGGL((K<T, 3, 1>), gc, blk, 0, s, ent, flags);                                       \
        else hipLaunchKernelGGL((K<T, 3, 0>), gc, blk, 0, s, ent, flags);                                           \
    } while (0)
#define PASS2(K)                                                                                                    \
    do {                                                                                                            \
        if (vel) hipLaunchKernelGGL((K<T, 2, 1>), gc, blk, 0, s, ent, flags);                                       \
        else hipLaunchKernelGGL((K<T, 2, 0>), gc, blk, 0, s, ent, flags);                                           \
    } while (0)
    switch (kind) {
    case BK_SWEEP: {
        const dim3 g1(nblocks);
        if (D == 3) {
            if (!vel) hipLaunchKernelGGL((k_bsweep<T, 3, 0, 0>), g1, blk, 0, s, ent, flags, colour);
            else if (A == 0) hipLaunchKernelGGL((k_bsweep<T, 3, 1, 0>), g1, blk, 0, s, ent, flags, colour);
            else if (A == 1) hipLaunchKernelGGL((k_bsweep<T, 3, 1, 1>), g1, blk, 0, s, ent, flags, colour);
            else hipLaunchKernelGGL((k_bsweep<T, 3, 1, 2>), g1, blk, 0, s, ent, flags, colour);
        } else {
            if (!vel) hipLaunchKernelGGL((k_bsweep<T, 2, 0, 0>), g1, blk, 0, s, ent, flags, colour);
            else if (A == 0) hipLaunchKernelGGL((k_bsweep<T, 2, 1, 0>), g1, blk, 0, s, ent, flags, colour);
            else hipLaunchKernelGGL((k_bsweep<T, 2, 1, 1>), g1, blk, 0, s, ent, flags, colour);
        }
        break;
    }
    case BK_RESID:
        if (D == 3) PASS3(k_bresid);
        else PASS2(k_bresid);
        break;
    case BK_RESID_ROWS:
        if (D == 3) hipLaunchKernelGGL((k_bresid_rows<T, 3>), dim3(nblocks), blk, 0, s, ent, flags);
        else hipLaunchKernelGGL((k_bresid_rows<T, 2>), dim3(nblocks), blk, 0, s, ent, flags);
        break;
    case BK_RESTRICT:
        if (D == 3) PASS3(k_brestrict);
        else PASS2(k_brestrict);
        break;
    case BK_PROLONG:
        if (D == 3) PASS3(k_bprolong);
        else PASS2(k_bprolong);
        break;
    case BK_PREP:
        if (vel) hipLaunchKernelGGL(k_bprep32<1>, dim3(nblocks), blk, 0, s, ent, flags);
        else hipLaunchKernelGGL(k_bprep32<0>, dim3(nblocks), blk, 0, s, ent, flags);
        break;
    case BK_ADD:
        if (vel) hipLaunchKernelGGL(k_badd<1>, gc, blk, 0, s, ent, flags);
        else hipLaunchKernelGGL(k_badd<0>, gc, blk, 0, s, ent, flags);
        break;
    }
#undef PASS3
#undef PASS2
}

void launch_breduce(const BEntry *ent, unsigned nitems, const int *flags, double *norms, hipStream_t s)
{
    if (nitems) hipLaunchKernelGGL(k_breduce, dim3(nitems), dim3(256), 0, s, ent, flags, norms);
}

template <typename T>
void launch_bcoarse(int D, int vel, const BCoarse *items, unsigned nitems, const int *flags, int nu1, int nu2,
                    int lds_bytes, hipStream_t s)
{
    if (nitems == 0) return;
    const dim3 g(nitems), b(wg_threads(D, vel));
#define LAUNCH(DD, VV)                                                                                              \
    do {                                                                                                            \
        allow_lds(k_bcoarse<T, DD, VV>, lds_bytes);                                                                 \
        hipLaunchKernelGGL((k_bcoarse<T, DD, VV>), g, b, lds_bytes, s, items, flags, nu1, nu2);                     \
    } while (0)
    if (D == 3) {
        if (vel) LAUNCH(3, 1);
        else LAUNCH(3, 0);
    } else {
        if (vel) LAUNCH(2, 1);
        else LAUNCH(2, 0);
    }
#undef LAUNCH
}
template void launch_bpass<double>(int, int, int, int, int, const BEntry *, unsigned, const int *, hipStream_t);
template void launch_bpass<float>(int, int, int, int, int, const BEntry *, unsigned, const int *, hipStream_t);
template void launch_bcoarse<double>(int, int, const BCoarse *, unsigned, const int *, int, int, int, hipStream_t);
template void launch_bcoarse<float>(int, int, const BCoarse *, unsigned, const int *, int, int, int, hipStream_t);

static VelBox unknown_boxes(const Grid &g, int velocity, long long &mx)
{
    VelBox boxes;
    mx = 0;
    const int nc = velocity ? g.D : 1;
    for (int a = 0; a < 3; ++a) {
        boxes.b[a] = a < nc ? unk_box(g, velocity ? face_mask(a) : 0) : Box{{0, 0, 0}, {0, 0, 0}};
        if (a < nc && box_count(boxes.b[a]) > mx) mx = box_count(boxes.b[a]);
    }
    return boxes;
}

void launch_apply(const Grid &g, int velocity, const VelArr<double> &z, const CoefP<double> &cp,
                  const CoefU<double> &cu, double mass, double cvisc, const VelArr<double> &q, hipStream_t s)
{
    long long mx;
    const VelBox boxes = unknown_boxes(g, velocity, mx);
    if (mx <= 0) return;
    if (velocity) {
        const dim3 grid(blocks_for(mx), g.D);
        if (g.D == 3) hipLaunchKernelGGL(k_apply_u<3>, grid, dim3(256), 0, s, g, boxes, z, cu, mass, cvisc, q);
        else hipLaunchKernelGGL(k_apply_u<2>, grid, dim3(256), 0, s, g, boxes, z, cu, mass, cvisc, q);
    } else {
        if (g.D == 3)
            hipLaunchKernelGGL(k_apply_p<3>, dim3(blocks_for(mx)), dim3(256), 0, s, g, boxes.b[0], z.c[0], cp, cvisc,
                               q.c[0]);
        else
            hipLaunchKernelGGL(k_apply_p<2>, dim3(blocks_for(mx)), dim3(256), 0, s, g, boxes.b[0], z.c[0], cp, cvisc,
                               q.c[0]);
    }
}

int launch_dot(const Grid &g, int velocity, const VelArrC<double> &x, const VelArrC<double> &y, double *partial,
               hipStream_t s)
{
    long long mx;
    const VelBox boxes = unknown_boxes(g, velocity, mx);
    const unsigned nb = stride_blocks(mx);
    const int nc = velocity ? g.D : 1;
    hipLaunchKernelGGL(k_dot, dim3(nb, nc), dim3(256), 0, s, boxes, g, x, y, partial);
    return (int)nb * nc;
}

void launch_gcr_axpy2(const Grid &g, int velocity, const double *num, const double *den, const VelArrC<double> &qi,
                      const VelArrC<double> &zi, const VelArr<double> &q, const VelArr<double> &z, hipStream_t s)
{
    long long mx;
    const VelBox boxes = unknown_boxes(g, velocity, mx);
    if (mx <= 0) return;
    hipLaunchKernelGGL(k_gcr_axpy2, dim3(blocks_for(mx), velocity ? g.D : 1), dim3(256), 0, s, g, boxes, num, den,
                       qi, zi, q, z);
}

void launch_gcr_update(const Grid &g, int velocity, const double *num, const double *den, const VelArrC<double> &z,
                       const VelArr<double> &x, hipStream_t s)
{
    long long mx;
    const VelBox boxes = unknown_boxes(g, velocity, mx);
    if (mx <= 0) return;
    hipLaunchKernelGGL(k_gcr_update, dim3(blocks_for(mx), velocity ? g.D : 1), dim3(256), 0, s, g, boxes, velocity,
                       num, den, z, x);
}

// explicit instantiations
#define INST(T)                                                                                                     \
    template void launch_smooth_p<T>(const Grid &, const T *, T *, const CoefP<T> &, T, int, hipStream_t, int);          \
    template void launch_smooth_u<T>(const Grid &, int, const T *, const VelArr<T> &, const CoefU<T> &, T, T, int,  \
                                     hipStream_t, int);                                                                  \
    template void launch_smooth_u_dec<T>(const Grid &, const VelArrC<T> &, const VelArr<T> &, const CoefU<T> &, T,  \
                                         T, int, hipStream_t);                                                      \
    template void launch_smooth_rb<T>(const Grid &, int, int, const VelArrC<T> &, const T *, const CoefU<T> &,      \
                                      const CoefP<T> &, T, T, T *, hipStream_t);                                    \
    template void launch_smooth_zm<T>(const Grid &, int, const VelArrC<T> &, const T *, const CoefU<T> &, T, T, T *, \
                                      hipStream_t);                                                                 \
    template int launch_resid_p<T>(const Grid &, const T *, const T *, const CoefP<T> &, T, T *, double *,          \
                                   hipStream_t);                                                                    \
    template int launch_resid_u<T>(const Grid &, const VelArrC<T> &, const VelArr<T> &, const CoefU<T> &, T, T,     \
                                   const VelArr<T> &, double *, hipStream_t);                                       \
    template int launch_norm2<T>(const Grid &, int, const int *, const VelArrC<T> &, double *, hipStream_t);        \
    template void launch_restrict<T>(const Grid &, const Grid &, int, const int *, int, bool, const VelArrC<T> &,   \
                                     const VelArr<T> &, T, hipStream_t, const VelArr<T> *);                         \
    template void launch_prolong_add<T>(const Grid &, const Grid &, int, const int *, int, const VelArrC<T> &,      \
                                        const VelArr<T> &, hipStream_t);                                            \
    template void launch_dense_apply<T>(const Grid &, int, int, const long long *, const int *, const double *,    \
                                        const VelArrC<T> &, const VelArr<T> &, hipStream_t);                        \
    template void launch_load_unknowns<T>(const Grid &, int, const int *, const VelArrC<T> &, const VelArr<T> &,    \
                                          hipStream_t);                                                             \
    template void launch_coef_ghosts<T>(const Grid &, const CoefSet<T> &, hipStream_t);                                       \
    template void launch_fill<T>(T *, long long, T, hipStream_t);
INST(double)
INST(float)
#undef INST
template void launch_cast_unknowns<double, float>(const Grid &, int, const int *, const VelArrC<double> &,
                                                  const VelArr<float> &, hipStream_t);
template void launch_cast_unknowns<float, double>(const Grid &, int, const int *, const VelArrC<float> &,
                                                  const VelArr<double> &, hipStream_t);
template void launch_cast_unknowns<double, double>(const Grid &, int, const int *, const VelArrC<double> &,
                                                   const VelArr<double> &, hipStream_t);
template void launch_fill<int>(int *, long long, int, hipStream_t);
template void launch_fill<unsigned char>(unsigned char *, long long, unsigned char, hipStream_t);

}  // namespace ibmg
