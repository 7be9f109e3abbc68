// The latency-bound levels of a V-cycle in one launch.
//
// On levels up to about 64 x 64 x 128 a launched colour pass takes 4-6 us of
// which the arithmetic is well under one: the rest is the launch, the first
// loads after the caches were invalidated at the kernel boundary, and the
// drain.  A grid-wide barrier inside one kernel costs as much (3-17 us
// for 64-256 workgroups, measured), but a pass only needs the values of its
// neighbours: here each workgroup keeps a brick of every level (a box of
// whole lines along x, widened by one point) in LDS, and after each colour
// pass exchanges the box's surface with the workgroups around it through
// mailboxes.  Such an exchange takes 1.2 us whatever the number of
// workgroups (measured), so a pass costs about 2 us.
//
// Mailboxes.  A level's mailbox has one entry per point of the level's
// uniform array: the value together with the number of the exchange that
// wrote it, in 8-byte words stored and loaded whole (relaxed, agent scope),
// so a word carries its own validity and no fence or flag is needed.  A
// reader polls the entry of each point it needs until the number is the one
// it waits for.  Entries are not overwritten before they have been read: a
// point's entry in mx is written once per sweep, and its owner cannot be a
// whole sweep (two exchanges for the pressure, six for the velocity) ahead of
// a neighbour, since it needs the neighbour's values of the passes between;
// mb carries residuals, prolonged iterates and final iterates of a level
// visit, any two of which are separated by exchanges that depend on the
// readers of the first.  The right-hand side of the tail's level is read whole
// by every workgroup with rows of the tail's matrix, while a poster waits only
// for the rows that it needs itself.  So it may be a cycle ahead of a reader,
// but not two: no row is posted before every workgroup of that level has
// posted its part of the same cycle, each after it has read the cycle before.
// That mailbox has two copies, used in turn.
//
// All workgroups must be on the chip at once.  Each first counts itself in;
// if the last has not arrived within a time limit (workgroups of another
// stream holding the chip), one of them runs the cycle alone on the global
// arrays, by the passes of the one-workgroup cycle, and the others leave: the
// same bits, later.  So every wait ends.
//
// The arithmetic is that of the launched passes (mg_device.h): same bits.
#include <type_traits>

#include "bricks.h"
#include "common.h"
#include "kernels.h"
#include "mg_device.h"

#pragma clang fp contract(on)

namespace ibmg {

// everything inlines into the kernel, so that a brick's description stays in
// scalar registers
#define BRICK_FN __device__ __attribute__((always_inline)) inline

typedef unsigned long long u64;
// polls before a workgroup gives up on a value (seconds; only a lost
// neighbour could cause it).  From then on NaN takes the place of what it hands
// on from level to level and of its result, and it counts itself in
// BrickCtl::lost, which the host turns into an error.
constexpr int BRICK_POLLS = 1 << 21;

template <typename T>
constexpr int MW = brick_mail_words(sizeof(T));

template <typename T>
BRICK_FN void post(u64 *p, T v, unsigned ep)
{
    const u64 tag = (u64)ep << 32;
    if (sizeof(T) == 4) {
        __hip_atomic_store(p, tag | __float_as_uint((float)v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        const u64 b = (u64)__double_as_longlong((double)v);
        __hip_atomic_store(p, tag | (b & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 1, tag | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// entries at words w[u] of a mailbox, those of bits `need`: every load of a
// round in flight together
template <typename T, int N>
BRICK_FN void collect(const u64 *box, const unsigned (&w)[N], unsigned need, unsigned ep, T (&v)[N], int *dead)
{
    u64 x[N][MW<T>];
    int left = *(volatile int *)dead ? 1 : BRICK_POLLS;
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (N > 1 && !(need >> u & 1)) continue;
            const u64 *p = reinterpret_cast<const u64 *>(reinterpret_cast<const char *>(box) + w[u] * 8u);
#pragma unroll
            for (int q = 0; q < MW<T>; ++q)
                x[u][q] = __hip_atomic_load(p + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int q = 0; q < MW<T>; ++q)
                if (N == 1 || (need >> u & 1)) ok = ok && (unsigned)(x[u][q] >> 32) == ep;
        if (ok) break;
        if (--left <= 0) {
            *(volatile int *)dead = 1;
            break;
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (sizeof(T) == 4) v[u] = (T)__uint_as_float((unsigned)x[u][0]);
        else v[u] = (T)__longlong_as_double((long long)((x[u][0] & 0xffffffffull) | (x[u][MW<T> - 1] << 32)));
    }
}

// whether this workgroup has given up on a value
BRICK_FN bool gave_up(const int *dead) { return *(const volatile int *)dead != 0; }

// words of a read-only table through scalar loads (every lane reads the same)
template <typename S>
BRICK_FN S cload(const S *p)
{
    return *(const __attribute__((address_space(4))) S *)p;
}

// a scalar kept in its register (the compiler would load it again at each use)
template <typename S>
BRICK_FN S pin(S x)
{
    asm volatile("" : "+s"(x));
    return x;
}

BRICK_FN BrickPass load_pass(const BrickPass *p)
{
    constexpr int N = sizeof(BrickPass) / 4;
    struct Words {
        unsigned v[N];
    } r;
#pragma unroll
    for (int k = 0; k < N; ++k) r.v[k] = cload(reinterpret_cast<const unsigned *>(p) + k);
    return __builtin_bit_cast(BrickPass, r);
}

// q / d, exact for q d < 2^32 (r = 2^32 / d rounded up)
BRICK_FN unsigned recip(unsigned d) { return 0xffffffffu / d + 1u; }
BRICK_FN int fast_div(int q, int d, unsigned r) { return d == 1 ? q : (int)__umulhi((unsigned)q, r); }

// the parts of a grid that the passes use
template <typename T>
BRICK_FN Grid load_grid(const LevTab<T> *t, int D)
{
    Grid g;
    g.D = D;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        g.n[d] = cload(&t->g.n[d]);
        g.bc[d] = cload(&t->g.bc[d]);
    }
    g.NX = g.n[0] + 3;
    g.NY = g.n[1] + 3;
    g.NXY = (long long)g.NX * g.NY;
    g.nel = 0;
    g.h = 0.0;
    return g;
}

// this workgroup's box of a level: lines [ya, yb) x [za, zb) along x (2D: z
// is one plane)
struct Lines {
    int ya, yb, za, zb;
};

template <int D>
BRICK_FN Lines own_lines(const Grid &g, const BrickLev *b, int wg)
{
    const int sy = cload(&b->sy), cy = cload(&b->cy);
    const int s2 = wg / sy, s1 = wg - s2 * sy;
    Lines x;
    // the position past the last cell holds unknowns only on an outflow axis
    x.ya = s1 * cy;
    x.yb = min(x.ya + cy, g.n[1]);
    if (s1 == sy - 1 && g.bc[1] == AX_INOUT) x.yb = g.n[1] + 1;
    x.za = 0;
    x.zb = 1;
    if (D == 3) {
        const int cz = cload(&b->cz);
        x.za = s2 * cz;
        x.zb = min(x.za + cz, g.n[2]);
        if (s2 == cload(&b->sz) - 1 && g.bc[2] == AX_INOUT) x.zb = g.n[2] + 1;
    }
    return x;
}

BRICK_FN bool has_box(const BrickLev *b, int wg) { return wg < cload(&b->sy) * cload(&b->sz); }

// whether line (cj, ck) holds unknowns of component a, bit a
template <int D, int VEL>
BRICK_FN unsigned line_comps(const Grid &g, int cj, int ck)
{
    unsigned m = 0;
#pragma unroll
    for (int a = 0; a < (VEL ? D : 1); ++a) {
        int lo1, hi1, lo2, hi2;
        unk_range(g, 1, VEL && a == 1, lo1, hi1);
        unk_range(g, 2, VEL && a == 2, lo2, hi2);
        if (cj >= lo1 && cj <= hi1 && ck >= lo2 && ck <= hi2) m |= 1u << a;
    }
    return m;
}

// A point's bits: it is an unknown; it lies on the surface of the box; it has
// a ghost image in the window below or above along x, y, z.
constexpr unsigned PT_UNKNOWN = 1, PT_SURF = 2;
constexpr int PT_IMG = 2;   // first of the six image bits (2 d + side)
constexpr unsigned PT_IMG_X = 3u << 2, PT_IMG_YZ = 15u << 4;

// A thread's slot: two neighbouring x positions of a line, one of each colour.
// f, e: the first one's entry in the level's arrays and in a window.  m: the
// bits above of the line, per component (8 bits each, those of x left out); x:
// per colour and kind of lattice along x (cells, faces) three bits: unknown,
// image below, image above; then the parity of the line.
struct Slot {
    int f, e;
    unsigned m, x;
    // of the two, the position of a colour
    BRICK_FN int step(int colour) const { return (int)((x >> 12 ^ (unsigned)colour) & 1u); }
};

// This workgroup's brick of one level.
template <typename T, int D, int VEL>
struct Brick {
    static constexpr int NC = VEL ? D : 1;
    Grid g;
    Lines x;
    int wy;
    unsigned char *w0;   // windows
    char *base;
    unsigned stride;
    u64 *mx0, *mb0;
    const BrickLev *b;
    int hx, no, nr;      // slots per line, own slots, slots around the box
    unsigned rhx, rly;

    BRICK_FN Brick(const LevTab<T> *tab, const BrickPlan *plan, int l, int wg, unsigned char *arena)
        : g(load_grid(tab + l, D)), b(&plan->lev[l])
    {
        x = own_lines<D>(g, b, wg);
        wy = cload(&b->wy);
        w0 = arena + cload(&b->lds);
        base = pin(reinterpret_cast<char *>(cload(&tab[l].xp)));
        stride = cload(&b->stride);
        mx0 = pin(cload(&b->mx));
        mb0 = pin(cload(&b->mb));
        hx = ((g.bc[0] == AX_INOUT ? g.n[0] : g.n[0] - 1) + 2) >> 1;
        rhx = recip((unsigned)hx);
        rly = recip((unsigned)(x.yb - x.ya));
        no = (x.yb - x.ya) * (x.zb - x.za) * hx;
        nr = (D == 3 ? 2 * (x.yb - x.ya + 2) + 2 * (x.zb - x.za) : 2) * hx;
    }
    // an entry of the level's arrays at a byte offset; of a window
    BRICK_FN T &arr(unsigned bytes) const { return *reinterpret_cast<T *>(base + bytes); }
    BRICK_FN T &win(int bytes) const { return *reinterpret_cast<T *>(w0 + bytes); }
    BRICK_FN int line_entry(int j, int k) const
    {
        return ((D == 3 ? k - x.za + 1 : 0) * wy + (j - x.ya + 1)) * g.NX + 1;
    }
    BRICK_FN void own_line(int line, int &j, int &k) const
    {
        const int ly = x.yb - x.ya, kk = D == 3 ? fast_div(line, ly, rly) : 0;
        j = x.ya + line - kk * ly;
        k = x.za + kk;
    }
    // the slot ih of the line held at raw position (j, k) of the window
    BRICK_FN Slot slot_on(int j, int k, int ih) const
    {
        int cj = j, ck = k;
        if (g.bc[1] == AX_PERIODIC) cj = j < 0 ? j + g.n[1] : (j >= g.n[1] ? j - g.n[1] : j);
        if (D == 3 && g.bc[2] == AX_PERIODIC) ck = k < 0 ? k + g.n[2] : (k >= g.n[2] ? k - g.n[2] : k);
        Slot s;
        s.m = 0;
        if (cj < 0 || cj > g.n[1] || ck < 0 || ck > g.n[2]) cj = ck = -9;   // beyond the domain: no unknowns
        const int par = (cj + ck) & 1;
        s.f = (int)at(g, 2 * ih, cj, ck);
        s.e = line_entry(j, k) + 2 * ih;
        s.x = (unsigned)par << 12;
        const unsigned comps = line_comps<D, VEL>(g, cj, ck);
        const bool surf = j == x.ya || j == x.yb - 1 || (D == 3 && (k == x.za || k == x.zb - 1));
        const int role = VEL ? ROLE_V : ROLE_P;
        // image bits along y and z by kind of lattice.  A line past the end of
        // a periodic axis (a neighbour's, held where the stencil looks for
        // it) has no image along it.
        unsigned im[2] = {0, 0};
#pragma unroll
        for (int d = 1; d < D; ++d) {
            const int q = d == 1 ? j : k, n = g.n[d], lo = (d == 1 ? x.ya : x.za) - 1, hi = d == 1 ? x.yb : x.zb;
            if (q < 0 || q > n || (q > 0 && q < n - 1) || (g.bc[d] == AX_PERIODIC && q == n)) continue;
#pragma unroll
            for (int vert = 0; vert < 2; ++vert) {
                const AxisImages m = images_of(g, d, vert, role, q);
                if (m.s[0] && m.q[0] >= lo && m.q[0] <= hi) im[vert] |= 1u << (PT_IMG + 2 * d);
                if (m.s[1] && m.q[1] >= lo && m.q[1] <= hi) im[vert] |= 2u << (PT_IMG + 2 * d);
            }
        }
        constexpr unsigned MY = 3u << (PT_IMG + 2), MZ = 3u << (PT_IMG + 4);
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            unsigned w = (surf ? PT_SURF : 0u) | PT_UNKNOWN;
            w |= (VEL && a == 1 ? im[1] : im[0]) & MY;
            w |= (VEL && a == 2 ? im[1] : im[0]) & MZ;
            if (comps >> a & 1) s.m |= w << (8 * a);
        }
#pragma unroll
        for (int colour = 0; colour < 2; ++colour) {
            const int i = 2 * ih + (par ^ colour);
#pragma unroll
            for (int vert = 0; vert < (VEL ? 2 : 1); ++vert) {
                int lo, hi;
                unk_range(g, 0, vert, lo, hi);
                unsigned w = i >= lo && i <= hi ? 1u : 0u;
                if (i == 0 || i == g.n[0] - 1) {
                    const AxisImages m = images_of(g, 0, vert, role, i);
                    w |= (m.s[0] ? 2u : 0u) | (m.s[1] ? 4u : 0u);
                }
                s.x |= w << (3 * (2 * colour + vert));
            }
        }
        return s;
    }
    BRICK_FN Slot own(int q) const
    {
        const int line = fast_div(q < no ? q : 0, hx, rhx);
        int j, k;
        own_line(line, j, k);
        Slot s = slot_on(j, k, q < no ? q - line * hx : 0);
        if (q >= no) s.m = 0;
        return s;
    }
    // the q-th slot on the lines of the window around the box
    BRICK_FN Slot ring(int q) const
    {
        const int r = fast_div(q < nr ? q : 0, hx, rhx), ly = x.yb - x.ya + 2;
        int j, k = 0;
        if (D == 3) {
            if (r < 2 * ly) {
                k = r < ly ? x.za - 1 : x.zb;
                j = x.ya - 1 + (r < ly ? r : r - ly);
            } else {
                const int s = r - 2 * ly;
                k = x.za + (s >> 1);
                j = s & 1 ? x.yb : x.ya - 1;
            }
        } else {
            j = r ? x.yb : x.ya - 1;
        }
        Slot s = slot_on(j, k, q < nr ? q - r * hx : 0);
        if (q >= nr) s.m = 0;
        return s;
    }
};

// the bits of a slot's point of component a (P: its pass) and one colour; 0:
// no unknown
BRICK_FN unsigned point_bits(const Slot &s, const BrickPass &P, int a, int colour)
{
    const unsigned x = s.x >> (3 * (2 * colour + P.face_x));
    const unsigned w = (s.m >> (8 * a) & 0xffu) | ((x & 6u) << 1);
    return (x & 1u) && (w & PT_UNKNOWN) ? w : 0u;
}

// value v of a component into the window at byte e, with its ghost images
template <typename T, int D, int VEL>
BRICK_FN void place(const Brick<T, D, VEL> &B, const BrickPass &P, unsigned w, int e, T v)
{
    e += P.win[0];
    B.win(e) = v;
    int ox = 0;
    T vx = v;
    if (w & PT_IMG_X) {
        const bool lo = w & (1u << PT_IMG);
        ox = lo ? P.img[0][0] : P.img[0][1];
        vx = (P.odd >> (lo ? 0 : 1) & 1) ? -v : v;
        B.win(e + ox) = vx;
    }
    if (!(w & PT_IMG_YZ)) return;
    const bool ylo = w & (1u << (PT_IMG + 2)), yhi = w & (2u << (PT_IMG + 2));
    const bool ny = (P.odd >> (ylo ? 2 : 3) & 1) != 0;
    const int oy = ylo ? P.img[1][0] : P.img[1][1];
    if (ylo || yhi) {
        B.win(e + oy) = ny ? -v : v;
        if (ox) B.win(e + oy + ox) = ny ? -vx : vx;
    }
    if (D == 3) {
        const bool zlo = w & (1u << (PT_IMG + 4)), zhi = w & (2u << (PT_IMG + 4));
        if (!(zlo || zhi)) return;
        const bool nz = (P.odd >> (zlo ? 4 : 5) & 1) != 0;
        const int oz = zlo ? P.img[2][0] : P.img[2][1];
        B.win(e + oz) = nz ? -v : v;
        if (ox) B.win(e + oz + ox) = nz ? -vx : vx;
        if (ylo || yhi) {
            B.win(e + oz + oy) = ny != nz ? -v : v;
            if (ox) B.win(e + oz + oy + ox) = ny != nz ? -vx : vx;
        }
    }
}

// a point as its row sees the boundaries: its image bits along the axes that
// do not wrap (which == 1, 2: the other axes; the pressure: axis number)
struct PointEdge {
    unsigned w;
    const BrickPass &P;
    BRICK_FN bool lo(int n) const { return (w & (unsigned)P.edge) >> P.axis[n] & 1u; }
    BRICK_FN bool hi(int n) const { return (w & (unsigned)P.edge) >> P.axis[n] & 2u; }
    BRICK_FN bool walls(int n) const { return P.walls >> n & 1; }
};
// the same by axis for constant viscosity, where the own axis never counts
struct PointEdgeDec {
    unsigned w;
    const BrickPass &P;
    BRICK_FN bool lo(int d) const { return PT_IMG + 2 * d != P.axis[0] && ((w & (unsigned)P.edge) >> (PT_IMG + 2 * d) & 1u); }
    BRICK_FN bool hi(int d) const { return PT_IMG + 2 * d != P.axis[0] && ((w & (unsigned)P.edge) >> (PT_IMG + 2 * d) & 2u); }
    BRICK_FN bool walls(int d) const
    {
        return P.walls >> (PT_IMG + 2 * d == P.axis[1] ? 1 : 2) & 1;
    }
};

// what a point's update reads besides the iterate
template <typename T, int D, int VEL>
struct PointCoef {
    T b, rho, cu, cl, mp[D - 1], mm[D - 1];   // viscous row
    T bt[2 * D];                              // pressure row
};

template <typename T, int D, int VEL>
BRICK_FN PointCoef<T, D, VEL> point_coef(const Brick<T, D, VEL> &B, const BrickPass &P, bool dec, int f)
{
    PointCoef<T, D, VEL> c;
    const unsigned o = (unsigned)f * (unsigned)sizeof(T);
    c.b = B.arr(o + P.coef[0]);
    if (VEL) {
        c.rho = B.arr(o + P.coef[1]);
        if (!dec) {
            c.cu = B.arr(o + P.coef[2]);
            c.cl = B.arr(o + P.coef[3]);
#pragma unroll
            for (int n = 0; n < D - 1; ++n) {
                c.mp[n] = B.arr(o + P.coef[4 + 2 * n]);
                c.mm[n] = B.arr(o + P.coef[5 + 2 * n]);
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < 2 * D; ++q) c.bt[q] = B.arr(o + P.coef[2 + q]);
    }
    return c;
}

// A x and the diagonal of a component's row at window byte e, the iterate
// read from the windows
template <typename T, int D, int VEL>
BRICK_FN void brick_row(const Brick<T, D, VEL> &B, const BrickPass &P, bool dec, T mass, T cv,
                        const PointCoef<T, D, VEL> &c, unsigned w, int e, T &x, T &Ax, T &dg)
{
    const int ea = e + P.win[0];
    x = B.win(ea);
    if (VEL) {
        if (dec) {
            const int st[3] = {(int)sizeof(T), B.g.NX * (int)sizeof(T), B.wy * B.g.NX * (int)sizeof(T)};
            T vp[D], vm[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                vp[d] = B.win(ea + st[d]);
                vm[d] = B.win(ea - st[d]);
            }
            u_row_dec_math<T, D, -1>(PointEdgeDec{w, P}, x, vp, vm, c.rho, mass, cv, Ax, dg);
            return;
        }
        URow<T, D> r;
        r.cu = c.cu;
        r.cl = c.cl;
        r.vp = B.win(ea + P.step[0]);
        r.vm = B.win(ea - P.step[0]);
#pragma unroll
        for (int n = 0; n < D - 1; ++n) {
            const int s = P.step[1 + n], eb = e + P.win[1 + n];
            r.mp[n] = c.mp[n];
            r.mm[n] = c.mm[n];
            r.ap[n] = B.win(ea + s);
            r.am[n] = B.win(ea - s);
            r.b0[n] = B.win(eb + s);
            r.b1[n] = B.win(eb + s - P.step[0]);
            r.b2[n] = B.win(eb);
            r.b3[n] = B.win(eb - P.step[0]);
        }
        u_row_math<T, D, 0>(PointEdge{w, P}, x, r, c.rho, mass, cv, Ax, dg);
    } else {
        T xn[2 * D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            xn[2 * d] = B.win(ea + P.step[d]);
            xn[2 * d + 1] = B.win(ea - P.step[d]);
        }
        p_row_math<T, D>(PointEdge{w, P}, x, xn, c.bt, cv, Ax, dg);
    }
}

// a thread's slots of a brick
struct SlotSet {
    Slot own[BRICK_SLOTS], ring[BRICK_SLOTS];
};

// the points of one component and colour on the lines around the box, from
// the mailboxes (box) into the window
template <typename T, int D, int VEL>
BRICK_FN void fetch_points(const Brick<T, D, VEL> &B, const SlotSet &S, u64 *box, int a, int colour, unsigned ep,
                           int *dead)
{
    const BrickPass P = load_pass(&B.b->pass[a]);
    unsigned w[BRICK_SLOTS], at_[BRICK_SLOTS], need = 0;
    T v[BRICK_SLOTS];
#pragma unroll
    for (int u = 0; u < BRICK_SLOTS; ++u) {
        w[u] = u * BRICK_THREADS < B.nr ? point_bits(S.ring[u], P, a, colour) : 0u;
        at_[u] = P.mail + (unsigned)(S.ring[u].f + S.ring[u].step(colour)) * MW<T>;
        need |= (w[u] ? 1u : 0u) << u;
    }
    if (!need) return;
    collect<T, BRICK_SLOTS>(box, at_, need, ep, v, dead);
#pragma unroll
    for (int u = 0; u < BRICK_SLOTS; ++u)
        if (w[u]) place<T, D, VEL>(B, P, w[u], (S.ring[u].e + S.ring[u].step(colour)) * (int)sizeof(T), v[u]);
}

// what the next pass must first fetch: nothing, the points of the last pass
// (component and colour, from mx), or all of them (from mb)
struct Pending {
    int kind;        // PEND_NONE, PEND_PASS, PEND_ALL
    int a, colour;
    unsigned ep;
};
constexpr int PEND_NONE = 0, PEND_PASS = 1, PEND_ALL = 2;

template <typename T, int D, int VEL>
BRICK_FN void fetch(const Brick<T, D, VEL> &B, const SlotSet &S, const Pending &pd, int *dead)
{
    if (pd.kind == PEND_NONE) return;
    const bool all = pd.kind == PEND_ALL;
    const int first = all ? 0 : 2 * pd.a + pd.colour, last = all ? 2 * B.NC : first + 1;
#pragma unroll 1
    for (int ac = first; ac < last; ++ac)
        fetch_points<T, D, VEL>(B, S, all ? B.mb0 : B.mx0, ac >> 1, ac & 1, pd.ep, dead);
}

// Every own position of components [c0, c0 + nc), dealt out to the threads:
// body(component, line, j, k, i) for the unknowns.
template <typename T, int D, int VEL, typename F>
BRICK_FN void each_own(const Brick<T, D, VEL> &B, int c0, int nc, F body)
{
    const int xw = 2 * B.hx, one = 2 * B.no;
    const unsigned rxw = recip((unsigned)xw);
#pragma unroll 1
    for (int q = threadIdx.x; q < nc * one; q += BRICK_THREADS) {
        const int s = (q >= one) + (q >= 2 * one), r = q - s * one, a = c0 + s;
        const int line = fast_div(r, xw, rxw), i = r - line * xw;
        int j, k, lo, hi;
        B.own_line(line, j, k);
        unk_range(B.g, 0, VEL && a == 0, lo, hi);
        if ((line_comps<D, VEL>(B.g, j, k) >> a & 1) && i >= lo && i <= hi) body(a, s, line, j, k, i);
    }
}

// word of the x sum I of line (j, k): two words each, on the line's entries
template <typename T>
BRICK_FN unsigned sum_word(const Grid &g, int j, int k, int I)
{
    return (unsigned)at(g, -1, j, k) * MW<T> + 2u * (unsigned)I;
}

// The x sums of the residual's lines (first step of the restriction) of
// components [c0, c0 + nc), one per coarse position, into mb as doubles.  buf:
// the residual, lines of NX entries from position 0.
template <typename T, int D, int VEL>
BRICK_FN void post_sums(const Brick<T, D, VEL> &B, const T *buf, int c0, int nc, unsigned ep)
{
    const int lines = (B.x.yb - B.x.ya) * (B.x.zb - B.x.za), NX = B.g.NX, nc0 = B.g.n[0] >> 1;
    const int xw = nc0 + 1, one = lines * xw;
    const unsigned rxw = recip((unsigned)xw);
    const int role = VEL ? ROLE_V : ROLE_P;
    Grid gc = B.g;
    gc.n[0] = nc0;
#pragma unroll 1
    for (int q = threadIdx.x; q < nc * one; q += BRICK_THREADS) {
        const int s = (q >= one) + (q >= 2 * one), r = q - s * one, a = c0 + s;
        const int line = fast_div(r, xw, rxw), I = r - line * xw;
        int j, k, lo, hi;
        B.own_line(line, j, k);
        unk_range(gc, 0, VEL && a == 0, lo, hi);
        if (!(line_comps<D, VEL>(B.g, j, k) >> a & 1) || I < lo || I > hi) continue;
        const T *src = buf + (s * lines + line) * NX;
        const double v = VEL && a == 0 ? restrict_line<1>(B.g, role, I, [&](int i) { return src[i]; })
                                       : restrict_line<0>(B.g, role, I, [&](int i) { return src[i]; });
        post<double>(B.mb0 + (B.b->pass[a].mail + sum_word<T>(B.g, j, k, I)), v, ep);
    }
}

// Where a window of lines [y0, y0 + ny) x [z0, z0 + nz) of a level (grid g, its
// mailboxes' components ms words apart) comes from, W values a line: its x
// sums (SUMS: positions 0 .. W - 1, two words each) or its iterate (positions
// -1 .. W - 2).  A line or position beyond the boundary holds what it stands
// for, zero where nothing is known, so that the transfers read it like any
// other.
template <typename T, int D, int VEL, bool SUMS>
BRICK_FN void window_sources(const Grid &g, unsigned ms, int y0, int ny, int z0, int nz, int W, unsigned *from)
{
    constexpr int NC = VEL ? D : 1;
    const int lines = ny * nz, role = VEL ? ROLE_V : ROLE_P;
    Grid gx = g;
    if (SUMS) gx.n[0] = W - 1;
    for (int q = threadIdx.x; q < NC * lines * W; q += blockDim.x) {
        const int a = q / (lines * W), line = q / W - a * lines, c = q - (q / W) * W;
        int i = SUMS ? c : c - 1, j = y0 + line % ny, k = D == 3 ? z0 + line / ny : 0, sg = 1, lo, hi;
        bool ok = j >= -2 && j <= g.n[1] + 2 && resolve(g, 1, VEL && a == 1, role, j, sg);
        if (D == 3) ok = ok && k >= -2 && k <= g.n[2] + 2 && resolve(g, 2, VEL && a == 2, role, k, sg);
        ok = ok && (line_comps<D, VEL>(g, j, k) >> a & 1);
        if (!SUMS) ok = ok && i <= g.n[0] + 1 && resolve(g, 0, VEL && a == 0, role, i, sg);
        unk_range(gx, 0, VEL && a == 0, lo, hi);
        ok = ok && i >= lo && i <= hi;
        const unsigned w = ok ? (unsigned)a * ms + (SUMS ? sum_word<T>(g, j, k, i) : (unsigned)at(g, i, j, k) * MW<T>) : 0u;
        from[q] = ok ? w | (sg < 0 ? BRICK_NEG : 0u) : BRICK_ZERO;
    }
}

// n entries into LDS from the mailboxes box, as the table says
template <typename V>
BRICK_FN void fetch_window(const unsigned *from, int n, u64 *box, unsigned ep, V *dst, int *dead)
{
    constexpr int N = sizeof(V) == 4 ? 8 : 4;
#pragma unroll 1
    for (int q0 = threadIdx.x; q0 < n; q0 += N * BRICK_THREADS) {
        unsigned f[N], w[N], need = 0;
        V v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) f[u] = q0 + u * BRICK_THREADS < n ? from[q0 + u * BRICK_THREADS] : BRICK_ZERO;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            need |= (f[u] & BRICK_ZERO ? 0u : 1u) << u;
            w[u] = f[u] & (BRICK_NEG - 1);
        }
        if (need) collect<V, N>(box, w, need, ep, v, dead);
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (q0 + u * BRICK_THREADS < n)
                dst[q0 + u * BRICK_THREADS] = f[u] & BRICK_ZERO ? V(0) : (f[u] & BRICK_NEG ? -v[u] : v[u]);
    }
}

// the window of level l + 1's iterate around the box x of level l
struct WindowAt {
    int y0, ny, z0, nz;
};
template <int D>
BRICK_FN WindowAt iterate_window(const Lines &x)
{
    WindowAt w;
    w.y0 = (x.ya >> 1) - 1;
    w.ny = ((x.yb - 1) >> 1) + 2 - w.y0;
    w.z0 = D == 3 ? (x.za >> 1) - 1 : 0;
    w.nz = D == 3 ? ((x.zb - 1) >> 1) + 2 - w.z0 : 1;
    return w;
}
// the window of level l - 1's x sums around the box x of level l
template <int D>
BRICK_FN WindowAt sums_window(const Lines &x)
{
    WindowAt w;
    w.y0 = 2 * x.ya - 1;
    w.ny = 2 * (x.yb - x.ya) + 2;
    w.z0 = D == 3 ? 2 * x.za - 1 : 0;
    w.nz = D == 3 ? 2 * (x.zb - x.za) + 2 : 1;
    return w;
}

// the tables of level l for workgroup blockIdx.x, once per context: working
// the same out on every visit of a level took 30 % of a V-cycle of 48 x 48 x 96
template <typename T, int D, int VEL>
__global__ void __launch_bounds__(BRICK_THREADS) k_brick_tables(const LevTab<T> *__restrict__ tab,
                                                                const BrickPlan *__restrict__ plan, int l, int lm,
                                                                int lc)
{
    const int wg = blockIdx.x;
    const BrickLev *b = &plan->lev[l];
    if (!has_box(b, wg)) return;
    const Brick<T, D, VEL> B(tab, plan, l, wg, nullptr);
    if (l <= lc) {
        Slot *s = static_cast<Slot *>(b->slots) + (size_t)wg * (b->os + b->rs) * BRICK_THREADS;
        for (int u = 0; u < b->os; ++u)
            s[u * BRICK_THREADS + threadIdx.x] = B.own((int)threadIdx.x + u * BRICK_THREADS);
        for (int u = 0; u < b->rs; ++u)
            s[(b->os + u) * BRICK_THREADS + threadIdx.x] = B.ring((int)threadIdx.x + u * BRICK_THREADS);
        const Grid gc = load_grid(tab + l + 1, D);
        const WindowAt w = iterate_window<D>(B.x);
        window_sources<T, D, VEL, false>(gc, (unsigned)tab[l + 1].g.nel * MW<T>, w.y0, w.ny, w.z0, w.nz, gc.NX,
                                         b->from_x + (size_t)wg * b->nx);
    }
    if (l > lm) {
        const Grid gf = load_grid(tab + l - 1, D);
        const WindowAt w = sums_window<D>(B.x);
        window_sources<T, D, VEL, true>(gf, (unsigned)tab[l - 1].g.nel * MW<T>, w.y0, w.ny, w.z0, w.nz, B.g.n[0] + 1,
                                        b->from_s + (size_t)wg * b->ns);
    }
}

// Second step of the restriction: components [c0, c0 + nc) of the coarse
// right-hand side at the own points of the coarse brick C, from the x sums of
// the lines around them in `buf`: into C's global b, or (last: C is the
// tail's level) into its mx, `copy` words on.
template <typename T, int D, int VEL>
BRICK_FN void brick_restrict(const Brick<T, D, VEL> &C, const double *buf, int c0, int nc, const WindowAt &wa, int W,
                             bool last, unsigned copy, unsigned ep, const int *dead)
{
    const bool lost = gave_up(dead);
    each_own<T, D, VEL>(C, c0, nc, [&](int a, int s, int, int J, int K, int I) {
        // three lines per axis of faces, four per axis of cells (the fourth
        // weight of faces is zero and its line read again)
        const int v1 = VEL && a == 1, v2 = VEL && a == 2;
        int r1[4], r2[4];
        double w1[4] = {0.0, 0.0, 0.0, 0.0}, w2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            r1[q] = 2 * J - 1 + (v1 && q == 3 ? 0 : q);
            r2[q] = 2 * K - 1 + (v2 && q == 3 ? 0 : q);
            w1[q] = v1 ? (q == 1 ? 0.5 : 0.25) : (q == 1 || q == 2 ? 0.375 : 0.125);
            w2[q] = v2 ? (q == 1 ? 0.5 : 0.25) : (q == 1 || q == 2 ? 0.375 : 0.125);
        }
        const double *src = buf + s * wa.ny * wa.nz * W + I;
        double sum = 0.0;
        if (D == 2) {
            r2[0] = 0;
            w2[0] = 1.0;
        }
#pragma unroll
        for (int c = 0; c < (D == 3 ? 4 : 1); ++c) {
            double v[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = src[((r2[c] - wa.z0) * wa.ny + r1[b] - wa.y0) * W];
            if (c == 3 && v2) continue;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (b == 3 && v1) continue;
                sum += w1[b] * w2[c] * v[b];
            }
        }
        if (lost) sum = __builtin_nan("");
        const int e = (int)at(C.g, I, J, K);
        const BrickPass *P = &C.b->pass[a];
        if (last) post<T>(C.mx0 + (P->mail + copy + (unsigned)e * MW<T>), (T)sum, ep);
        else C.arr((unsigned)e * (unsigned)sizeof(T) + P->coef[0]) = (T)sum;
    });
}

// Every own point of components [c0, c0 + nc) in whole waves of one component
// and colour: body(component, its pass, colour, q, slot, bits) for slot q's
// point (bits 0: no unknown).
template <typename T, int D, int VEL, typename F>
BRICK_FN void each_point(const Brick<T, D, VEL> &B, const Slot *own, int c0, int nc, F body)
{
    const int chunks = (B.no + 63) >> 6, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#pragma unroll 1
    for (int it = wave; it < 2 * nc * chunks; it += BRICK_THREADS / 64) {
        const int ac = it / chunks, a = c0 + (ac >> 1), colour = ac & 1;
        const int q = (it - ac * chunks) * 64 + ((int)threadIdx.x & 63);
        if (q >= B.no) continue;
        const Slot s = own[q];
        const BrickPass P = load_pass(&B.b->pass[a]);
        body(a, P, colour, q, s, point_bits(s, P, a, colour));
    }
}

// x += P e at the own points, e the coarse iterate in `buf` (a window of W
// values a line, from position -1)
template <typename T, int D, int VEL>
BRICK_FN void brick_prolong(const Brick<T, D, VEL> &B, const Slot *own, const T *buf, const WindowAt &wa, int W,
                            unsigned ep)
{
    each_point<T, D, VEL>(B, own, 0, B.NC, [&](int a, const BrickPass &P, int colour, int q0, const Slot &s, unsigned wb) {
        if (!wb) return;
        const T *src = buf + a * wa.ny * wa.nz * W + 1;
        const int line = fast_div(q0, B.hx, B.rhx);
        int q[3];
        B.own_line(line, q[1], q[2]);
        q[0] = 2 * (q0 - line * B.hx) + s.step(colour);
        int r[3][2];
        double w[3][2];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            // faces: the coarse face itself, or the mean of the two around
            // it; cells: 3/4 and 1/4
            const bool vert = VEL && d == a, odd = q[d] & 1;
            r[d][0] = q[d] >> 1;
            r[d][1] = r[d][0] + (odd ? 1 : (vert ? 0 : -1));
            w[d][0] = vert ? (odd ? 0.5 : 1.0) : 0.75;
            w[d][1] = vert ? (odd ? 0.5 : 0.0) : 0.25;
        }
        if (D == 2) {
            r[2][0] = 0;
            w[2][0] = 1.0;
        }
        T v[D == 3 ? 2 : 1][2][2];
#pragma unroll
        for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int x = 0; x < 2; ++x) v[c][b][x] = src[((r[2][c] - wa.z0) * wa.ny + r[1][b] - wa.y0) * W + r[0][x]];
        double sum = 0.0;
#pragma unroll
        for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int x = 0; x < 2; ++x) sum += w[0][x] * w[1][b] * w[2][c] * (double)v[c][b][x];
        const int o = s.step(colour), e = (s.e + o) * (int)sizeof(T);
        const T xn = B.win(e + P.win[0]) + (T)sum;
        if (wb & PT_SURF) post<T>(B.mb0 + (P.mail + (unsigned)(s.f + o) * MW<T>), xn, ep);
        place<T, D, VEL>(B, P, wb, e, xn);
    });
}

// the own iterate into mb (final: into the global arrays, with its ghost
// images there)
template <typename T, int D, int VEL>
BRICK_FN void brick_out(const Brick<T, D, VEL> &B, bool final, unsigned ep, const int *dead)
{
    const bool lost = gave_up(dead);
    each_own<T, D, VEL>(B, 0, B.NC, [&](int a, int, int, int j, int k, int i) {
        const BrickPass *P = &B.b->pass[a];
        const T v = lost ? (T)__builtin_nan("") : B.win((B.line_entry(j, k) + i) * (int)sizeof(T) + P->win[0]);
        const unsigned e = (unsigned)at(B.g, i, j, k);
        if (!final) {
            post<T>(B.mb0 + (P->mail + e * MW<T>), v, ep);
        } else {
            T *xg = &B.arr((unsigned)(VEL ? 3 + 5 * a : 0) * B.stride);
            xg[e] = v;
            write_images(B.g, VEL ? 1 << a : 0, VEL ? ROLE_V : ROLE_P, xg, i, j, k, v);
        }
    });
}

template <typename T, int D, int VEL>
__global__ void __launch_bounds__(BRICK_THREADS) k_bricks(const LevTab<T> *__restrict__ tab,
                                                          const BrickPlan *__restrict__ plan, int ncyc, int xzero,
                                                          BrickCtl *ctl)
{
    using BR = Brick<T, D, VEL>;
    extern __shared__ __align__(16) unsigned char arena[];
    __shared__ T bv[TAIL_MAX];
    __shared__ int s_state, s_dead;
    constexpr int NC = VEL ? D : 1;
    const int N = gridDim.x;
    // neighbouring bricks on one XCD: workgroup b runs on XCD b mod 8
    const int wg = N % 8 == 0 ? (int)(blockIdx.x % 8) * (N / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    int *dead = &s_dead;
    const int lm = cload(&plan->lm), lc = cload(&plan->lc);

    unsigned ep = __builtin_amdgcn_readfirstlane(
        (int)__hip_atomic_load(&ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (threadIdx.x == 0) {
        s_dead = 0;
        const unsigned ticket = __hip_atomic_fetch_add(&ctl->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned st = 0;
        if (ticket == (unsigned)N - 1) {
            if (__hip_atomic_compare_exchange_strong(&ctl->state, &st, (unsigned)BRICK_GO, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                st = BRICK_GO;
        } else {
            const long long t0 = wall_clock64(), limit = ctl->limit;
            while ((st = __hip_atomic_load(&ctl->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
                if (wall_clock64() - t0 >= limit) {
                    const unsigned mine = (unsigned)(BRICK_SOLO + wg);
                    if (__hip_atomic_compare_exchange_strong(&ctl->state, &st, mine, __ATOMIC_RELAXED,
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                        st = mine;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        s_state = (int)st;
    }
    // meanwhile the other waves bring the first level's windows in
    if (has_box(&plan->lev[lm], wg)) {
        const BR B(tab, plan, lm, wg, arena);
        const int n = cload(&B.b->wn), NX = B.g.NX;
        for (int e = threadIdx.x; e < n; e += BRICK_THREADS) {
            // the window is a box of the uniform array, whose ghosts hold
            // their images (past the array: nothing is read)
            const int line = e / NX, kk = line / B.wy, jj = line - kk * B.wy;
            const int row = B.x.ya + jj, pl = D == 3 ? B.x.za + kk : 0;
            const bool in = !xzero && row < B.g.NY && (D != 3 || pl < B.g.n[2] + 3);
            const unsigned f = ((unsigned)pl * B.g.NY + row) * NX + (e - line * NX);
#pragma unroll
            for (int a = 0; a < NC; ++a)
                B.win((a * n + e) * (int)sizeof(T)) =
                    in ? B.arr(f * (unsigned)sizeof(T) + (unsigned)(VEL ? 3 + 5 * a : 0) * B.stride) : T(0);
        }
    }
    __syncthreads();
    if (s_state != BRICK_GO) {
        if (s_state == BRICK_SOLO + wg) {
            for (int c = 0; c < ncyc; ++c) {
                coarse_cycle<T, D, VEL>(tab, lm, plan->L, plan->nu1, plan->nu2, 0, nullptr, nullptr, nullptr,
                                        plan->tail, bv);
                __syncthreads();
            }
            if (threadIdx.x == 0) atomicAdd(&ctl->solo_runs, 1);
        }
    } else {
        const int nl = lc - lm + 1;
        Pending carry{PEND_NONE, 0, 0, 0};
        unsigned copy = 0;   // words to the cycle's copy of the tail level's mx
#pragma unroll 1
        for (int v = 0; v < 2 * nl * ncyc; ++v) {
            const int vv = v % (2 * nl);
            const bool down = vv < nl;
            const int l = down ? lm + vv : lc - (vv - nl);
            const bool act = has_box(&plan->lev[l], wg), last = l == lc;
            const BR B(tab, plan, l, wg, arena);
            unsigned char *const below = arena + cload(&plan->lev[l + 1].lds);
            const T mass = VEL ? cload(&tab[l].mass) : T(0), cv = VEL ? cload(&tab[l].cvu) : cload(&tab[l].cvp);
            const bool dec = VEL && cload(&tab[l].dec) != 0;
            const int os = cload(&B.b->os);
            const Slot *const own = static_cast<const Slot *>(cload(&B.b->slots)) +
                                    (size_t)wg * (os + cload(&B.b->rs)) * BRICK_THREADS;
            SlotSet S;
            if (act)
#pragma unroll
                for (int u = 0; u < BRICK_SLOTS; ++u) {
                    if (u * BRICK_THREADS < B.no) S.own[u] = own[u * BRICK_THREADS + threadIdx.x];
                    if (u * BRICK_THREADS < B.nr) S.ring[u] = own[(os + u) * BRICK_THREADS + threadIdx.x];
                }
            Pending pd = down && l == lm ? carry : Pending{PEND_NONE, 0, 0, 0};
            if (!down) {
                // the coarse correction, from the mailboxes of level l + 1
                if (act) {
                    const WindowAt wa = iterate_window<D>(B.x);
                    const int W = (B.g.n[0] >> 1) + 3;
                    T *buf = reinterpret_cast<T *>(below);
                    fetch_window<T>(cload(&B.b->from_x) + (size_t)wg * cload(&B.b->nx), NC * wa.ny * wa.nz * W,
                                    cload(&plan->lev[l + 1].mb), ep, buf, dead);
                    __syncthreads();
                    brick_prolong<T, D, VEL>(B, own, buf, wa, W, ep + 1);
                    pd = Pending{PEND_ALL, 0, 0, ep + 1};
                }
                ++ep;
            }
            // the sweeps: every component, red then black.  The coefficients
            // of a thread's points are loaded before it waits for the
            // neighbours' values.
            const int np = 2 * NC * (down ? cload(&plan->nu1) : cload(&plan->nu2));
            if (act) {
                int a = 0, colour = 0;
#pragma unroll 1
                for (int pass = 0; pass < np; ++pass) {
                    const BrickPass P = load_pass(&B.b->pass[a]);
                    PointCoef<T, D, VEL> c[BRICK_SLOTS];
                    unsigned w[BRICK_SLOTS];
#pragma unroll
                    for (int u = 0; u < BRICK_SLOTS; ++u) {
                        w[u] = 0;
                        if (u * BRICK_THREADS >= B.no) continue;
                        w[u] = point_bits(S.own[u], P, a, colour);
                        if (w[u]) c[u] = point_coef<T, D, VEL>(B, P, dec, S.own[u].f + S.own[u].step(colour));
                    }
                    fetch<T, D, VEL>(B, S, pd, dead);
                    __syncthreads();
                    const unsigned e1 = ep + 1 + (unsigned)pass;
#pragma unroll
                    for (int u = 0; u < BRICK_SLOTS; ++u)
                        if (w[u]) {
                            const int e = (S.own[u].e + S.own[u].step(colour)) * (int)sizeof(T);
                            T xe, Ax, dg;
                            brick_row<T, D, VEL>(B, P, dec, mass, cv, c[u], w[u], e, xe, Ax, dg);
                            const T xn = xe + (c[u].b - Ax) / dg;
                            if (w[u] & PT_SURF)
                                post<T>(B.mx0 + (P.mail + (unsigned)(S.own[u].f + S.own[u].step(colour)) * MW<T>), xn, e1);
                            place<T, D, VEL>(B, P, w[u], e, xn);
                        }
                    pd = Pending{PEND_PASS, a, colour, e1};
                    colour ^= 1;
                    if (!colour) a = a + 1 == NC ? 0 : a + 1;
                }
            }
            ep += (unsigned)np;
            if (!down) {
                const bool end = v == 2 * nl * ncyc - 1;
                if (l == lm && !end) {
                    carry = pd;
                    continue;
                }
                ++ep;
                if (act) {
                    __syncthreads();
                    brick_out<T, D, VEL>(B, end, ep, dead);
                    __syncthreads();
                }
                continue;
            }
            // the coarse right-hand side, all components at once or, where
            // the LDS does not hold that, one by one
            ++ep;
            const bool coarse = has_box(&plan->lev[l + 1], wg);
            const int gs = cload(&plan->lev[l].gs);
            if (act) {
                fetch<T, D, VEL>(B, S, pd, dead);
                __syncthreads();
            }
#pragma unroll 1
            for (int c0 = 0; c0 < NC; c0 += gs) {
                if (act) {
                    T *buf = reinterpret_cast<T *>(below);
                    const int lines = (B.x.yb - B.x.ya) * (B.x.zb - B.x.za);
                    each_point<T, D, VEL>(B, own, c0, gs, [&](int a, const BrickPass &P, int colour, int q, const Slot &s,
                                                              unsigned w) {
                        const int line = fast_div(q, B.hx, B.rhx), o = s.step(colour);
                        T r = T(0);   // a fixed face's is read with weight zero
                        if (w) {
                            const PointCoef<T, D, VEL> c = point_coef<T, D, VEL>(B, P, dec, s.f + o);
                            T xe, Ax, dg;
                            brick_row<T, D, VEL>(B, P, dec, mass, cv, c, w, (s.e + o) * (int)sizeof(T), xe, Ax, dg);
                            r = c.b - Ax;
                        }
                        buf[((a - c0) * lines + line) * B.g.NX + 2 * (q - line * B.hx) + o] = r;
                    });
                    __syncthreads();
                    post_sums<T, D, VEL>(B, buf, c0, gs, ep);
                }
                __syncthreads();
                if (!coarse) continue;
                const BR C(tab, plan, l + 1, wg, arena);
                const WindowAt wa = sums_window<D>(C.x);
                const int W = C.g.n[0] + 1, one = wa.ny * wa.nz * W;
                double *buf = reinterpret_cast<double *>(below);
                fetch_window<double>(cload(&C.b->from_s) + (size_t)wg * cload(&C.b->ns) + c0 * one, gs * one, B.mb0, ep,
                                     buf, dead);
                __syncthreads();
                brick_restrict<T, D, VEL>(C, buf, c0, gs, wa, W, last, copy, ep + 1, dead);
                __syncthreads();
            }
            if (coarse && !last) {
                // the coarse correction starts at zero
                const int n = NC * cload(&plan->lev[l + 1].wn);
                T *w = reinterpret_cast<T *>(below);
                for (int e = threadIdx.x; e < n; e += BRICK_THREADS) w[e] = T(0);
                __syncthreads();
            }
            if (!last) continue;
            const Tail &tail = plan->tail;
            const int n = cload(&tail.n);
            const unsigned ms = (unsigned)cload(&tab[l + 1].g.nel) * MW<T>;
            if (coarse && brick_has_rows(wg, n)) {
                // the tail: rows dealt out to the workgroups of its level
                const BrickLev *cb = &plan->lev[l + 1];
                u64 *const mx = cload(&cb->mx), *const mb = cload(&cb->mb);
                const int *const comp = cload(&tail.comp);
                const long long *const idx = cload(&tail.idx);
                for (int t = threadIdx.x; t < tail_ld(n, sizeof(T)); t += BRICK_THREADS) {
                    T val[1] = {T(0)};
                    if (t < n) {
                        const unsigned at_[1] = {copy + comp[t] * ms + (unsigned)idx[t] * MW<T>};
                        collect<T, 1>(mx, at_, 1u, ep + 1, val, dead);
                        if (gave_up(dead)) val[0] = (T)__builtin_nan("");   // a term of every row
                    }
                    bv[t] = val[0];
                }
                __syncthreads();
                const int nact = cload(&cb->sy) * cload(&cb->sz), per = BRICK_TAIL_ROWS;
                const T *Tm = static_cast<const T *>(cload(&tail.Tm));
                for (int r0 = wg * per; r0 < n; r0 += nact * per) {
                    const int r = r0 + threadIdx.x / TAIL_LANES, u = threadIdx.x % TAIL_LANES;
                    const T sum = tail_row<T>(Tm, n, r < n ? r : n - 1, u, bv);
                    if (r < n && u == 0) post<T>(mb + (comp[r] * ms + (unsigned)idx[r] * MW<T>), sum, ep + 2);
                }
            }
            copy = copy ? 0u : NC * ms;
            ep += 2;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_dead) atomicAdd(&ctl->lost, 1);
        const unsigned d = __hip_atomic_fetch_add(&ctl->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (d == (unsigned)N - 1) {
            __hip_atomic_store(&ctl->epoch, ep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->state, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <typename T, int D, int VEL>
static int resident(int bytes)
{
    int dev = 0, cus = 0, per = 0;
    // the limit is the kernel's, for every context of the process: always the
    // whole budget, never this plan's bytes, which may be fewer than another's
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(k_bricks<T, D, VEL>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, BRICK_LDS_BUDGET) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_bricks<T, D, VEL>, BRICK_THREADS, bytes) != hipSuccess) {
        (void)hipGetLastError();   // the levels are launched pass by pass instead
        return 0;
    }
    return cus * per;
}

template <typename T>
int bricks_resident(int D, int vel, int lds_bytes)
{
    if (D == 3) return vel ? resident<T, 3, 1>(lds_bytes) : resident<T, 3, 0>(lds_bytes);
    return vel ? resident<T, 2, 1>(lds_bytes) : resident<T, 2, 0>(lds_bytes);
}

template <typename T>
void launch_bricks(int D, int vel, const LevTab<T> *tab, const BrickPlan *plan_dev, const BrickPlan &plan, int ncyc,
                   int xzero, BrickCtl *ctl, hipStream_t s)
{
#define LAUNCH(DD, VV)                                                                                          \
    launch_timed_shm(k_bricks<T, DD, VV>, dim3(plan.nwg), dim3(BRICK_THREADS), plan.lds_bytes, s, tab, plan_dev, \
                     ncyc, xzero, ctl)
    if (D == 3) {
        if (vel) LAUNCH(3, 1);
        else LAUNCH(3, 0);
    } else {
        if (vel) LAUNCH(2, 1);
        else LAUNCH(2, 0);
    }
#undef LAUNCH
}

template <typename T>
void launch_brick_tables(int D, int vel, const LevTab<T> *tab, const BrickPlan *plan_dev, const BrickPlan &plan,
                         hipStream_t s)
{
    for (int l = plan.lm; l <= plan.lc + 1; ++l) {
        const dim3 g((unsigned)(plan.lev[l].sy * plan.lev[l].sz)), b(BRICK_THREADS);
#define LAUNCH(DD, VV) hipLaunchKernelGGL((k_brick_tables<T, DD, VV>), g, b, 0, s, tab, plan_dev, l, plan.lm, plan.lc)
        if (D == 3) {
            if (vel) LAUNCH(3, 1);
            else LAUNCH(3, 0);
        } else {
            if (vel) LAUNCH(2, 1);
            else LAUNCH(2, 0);
        }
#undef LAUNCH
    }
}

#define INST(T)                                                                                                     \
    template void launch_brick_tables<T>(int, int, const LevTab<T> *, const BrickPlan *, const BrickPlan &, hipStream_t); \
    template int bricks_resident<T>(int, int, int);                                                                 \
    template void launch_bricks<T>(int, int, const LevTab<T> *, const BrickPlan *, const BrickPlan &, int, int, BrickCtl *, \
                                   hipStream_t);
INST(double)
INST(float)
#undef INST

}  // namespace ibmg
