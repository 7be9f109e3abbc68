// Host check (built by tests/test_brick_order_cpu.py): no entry of the
// bricks' mailboxes is written again before all its readers have read it.
//
// The plan of a problem is the library's own (plan_bricks).  Every workgroup's
// posts and reads of a launch of several V-cycles are walked line by line in
// program order, with a vector clock per workgroup: what it knows to be done,
// through the values that it has waited for.  Whoever overwrites a line must
// know of every read of what it overwrites.  A read of a value that nobody
// posted is reported too.
#include <cstdio>
#include <unordered_map>

#include "api.hip"

namespace {

struct Rules {
    int copies;        // of the tail level's right-hand side
    bool rows_only;    // only workgroups with rows of the tail's matrix read it
};

struct Post {
    unsigned ep;
    int wg, pos;
};
struct Entry {
    std::vector<Post> posts;
    std::vector<std::vector<std::pair<int, int>>> readers;   // per post: workgroup, position
};

struct Walk {
    const ibb_ctx *c;
    const BrickPlan &P;
    const bool vel;
    const Rules R;
    const int D, NC, N, nt;
    int pos = 0;
    long long reads = 0, lost = 0, unordered = 0;
    std::unordered_map<unsigned long long, Entry> box;
    std::vector<std::vector<int>> clock;                 // per workgroup
    std::vector<std::vector<std::vector<int>>> at_pos;   // clocks after the reads of a position
    std::vector<std::vector<unsigned long long>> tail_rows;   // per workgroup: keys of its rows
    std::unordered_map<unsigned long long, std::vector<unsigned long long>> tail_line;   // rows on a line

    Walk(const ibb_ctx *cc, const BrickPlan &p, bool v, Rules r)
        : c(cc), P(p), vel(v), R(r), D(cc->d.dim), NC(v ? cc->d.dim : 1), N(p.nwg), nt(cc->tail[v ? 1 : 0].n)
    {
        clock.assign(N, std::vector<int>(N, -1));
        tail_rows.resize(N);
        const int l = P.lc + 1, nact = P.lev[l].sy * P.lev[l].sz;
        std::vector<long long> idx;
        std::vector<int> cmp;
        level_unknowns(const_cast<ibb_ctx *>(c), l, vel, idx, cmp);
        for (int row = 0; row < nt; ++row) {
            int i, j, k;
            decode(c->lv[l].g, idx[row], i, j, k);
            const unsigned long long key = (3ull << 60) | (unsigned)row;
            tail_rows[(row / BRICK_TAIL_ROWS) % nact].push_back(key);
            tail_line[line(cmp[row], j, k)].push_back(key);
        }
    }
    static unsigned long long line(int a, int j, int k) { return ((unsigned long long)a << 40) | (unsigned)(j << 16) | (unsigned)k; }
    // kind 0: mx of a colour, 1: mb, 2: the tail's right-hand side in copy q
    static unsigned long long key(int kind, int l, int a, int q, int j, int k)
    {
        return ((unsigned long long)kind << 60) | ((unsigned long long)l << 52) | ((unsigned long long)q << 48) | line(a, j, k);
    }
    const Grid &grid(int l) const { return c->lv[l].g; }
    bool has(int l, int wg) const { return wg < P.lev[l].sy * P.lev[l].sz; }
    struct Box {
        int ya, yb, za, zb;
    };
    Box own(int l, int wg) const
    {
        const Grid &g = grid(l);
        const BrickLev &b = P.lev[l];
        const int s2 = wg / b.sy, s1 = wg % b.sy;
        Box x{s1 * b.cy, std::min((s1 + 1) * b.cy, g.n[1]), 0, 1};
        if (s1 == b.sy - 1 && g.bc[1] == AX_INOUT) x.yb = g.n[1] + 1;
        if (D == 3) {
            x.za = s2 * b.cz;
            x.zb = std::min((s2 + 1) * b.cz, g.n[2]);
            if (s2 == b.sz - 1 && g.bc[2] == AX_INOUT) x.zb = g.n[2] + 1;
        }
        return x;
    }
    bool holds(const Grid &g, int a, int j, int k) const
    {
        int lo1, hi1, lo2, hi2;
        unk_range(g, 1, vel && a == 1, lo1, hi1);
        unk_range(g, 2, vel && a == 2, lo2, hi2);
        return j >= lo1 && j <= hi1 && k >= lo2 && k <= hi2;
    }
    // the lines of the window around the box: f(canonical j, k)
    template <typename F>
    void ring(int l, int wg, F f) const
    {
        const Grid &g = grid(l);
        const Box x = own(l, wg);
        for (int k = D == 3 ? x.za - 1 : 0; k <= (D == 3 ? x.zb : 0); ++k)
            for (int j = x.ya - 1; j <= x.yb; ++j) {
                if (j >= x.ya && j < x.yb && (D == 2 || (k >= x.za && k < x.zb))) continue;
                int cj = j, ck = k;
                if (g.bc[1] == AX_PERIODIC) cj = (j + g.n[1]) % g.n[1];
                if (D == 3 && g.bc[2] == AX_PERIODIC) ck = (k + g.n[2]) % g.n[2];
                if (cj >= 0 && cj <= g.n[1] && ck >= 0 && ck <= g.n[2]) f(cj, ck);
            }
    }
    template <typename F>
    void lines(int l, int wg, bool surface, F f) const
    {
        const Box x = own(l, wg);
        for (int k = x.za; k < x.zb; ++k)
            for (int j = x.ya; j < x.yb; ++j)
                if (!surface || j == x.ya || j == x.yb - 1 || (D == 3 && (k == x.za || k == x.zb - 1))) f(j, k);
    }
    // the lines that stand behind a window of level l: f(component, j, k)
    template <typename F>
    void window(int l, int y0, int ny, int z0, int nz, F f) const
    {
        const Grid &g = grid(l);
        for (int a = 0; a < NC; ++a)
            for (int kk = z0; kk < z0 + nz; ++kk)
                for (int jj = y0; jj < y0 + ny; ++jj) {
                    int j = jj, k = kk, s = 1;
                    bool ok = j >= -2 && j <= g.n[1] + 2 && resolve(g, 1, vel && a == 1, vel ? ROLE_V : ROLE_P, j, s);
                    if (D == 3) ok = ok && k >= -2 && k <= g.n[2] + 2 && resolve(g, 2, vel && a == 2, vel ? ROLE_V : ROLE_P, k, s);
                    if (ok && holds(g, a, j, k)) f(a, j, k);
                }
    }

    void read(int wg, unsigned long long k, unsigned ep)
    {
        ++reads;
        Entry &e = box[k];
        for (size_t q = e.posts.size(); q-- > 0;) {
            const Post &p = e.posts[q];
            if (p.ep != ep) continue;
            if (p.pos >= pos && p.wg != wg) break;   // not yet posted here
            const std::vector<int> &src = at_pos[p.pos][p.wg];
            for (int w = 0; w < N; ++w) clock[wg][w] = std::max(clock[wg][w], src[w]);
            e.readers[q].push_back({wg, pos});
            return;
        }
        ++lost;
    }
    std::vector<std::pair<unsigned long long, Post>> fresh;
    void post(int wg, unsigned long long k, unsigned ep) { fresh.push_back({k, {ep, wg, pos}}); }
    // every workgroup has done its reads of this position, then its posts
    void next()
    {
        for (int w = 0; w < N; ++w) clock[w][w] = pos;
        at_pos.push_back(clock);
        for (auto &f : fresh) {
            Entry &e = box[f.first];
            e.posts.push_back(f.second);
            e.readers.emplace_back();
        }
        fresh.clear();
        ++pos;
    }
    // whoever posts over a value knows of all its readers
    void check()
    {
        for (auto &it : box) {
            Entry &e = it.second;
            for (size_t q = 0; q + 1 < e.posts.size(); ++q) {
                const Post &n = e.posts[q + 1];
                for (auto &r : e.readers[q])
                    if (r.first != n.wg && at_pos[n.pos][n.wg][r.first] < r.second) ++unordered;
            }
        }
    }

    struct Pending {
        int kind = 0, a = 0, colour = 0;   // 1: the last pass, 2: all
        unsigned ep = 0;
    };
    void fetch(int l, int wg, const Pending &pd)
    {
        if (!pd.kind) return;
        ring(l, wg, [&](int j, int k) {
            for (int a = 0; a < NC; ++a) {
                if (!holds(grid(l), a, j, k)) continue;
                if (pd.kind == 2) read(wg, key(1, l, a, 0, j, k), pd.ep);
                else if (pd.a == a) read(wg, key(0, l, a, pd.colour, j, k), pd.ep);
            }
        });
    }
    void post_lines(int l, int wg, bool surface, unsigned ep)
    {
        lines(l, wg, surface, [&](int j, int k) {
            for (int a = 0; a < NC; ++a)
                if (holds(grid(l), a, j, k)) post(wg, key(1, l, a, 0, j, k), ep);
        });
    }

    void run(int ncyc)
    {
        const int lm = P.lm, lc = P.lc, nl = lc - lm + 1;
        unsigned ep = 0;
        Pending carry;
        for (int v = 0; v < 2 * nl * ncyc; ++v) {
            const int vv = v % (2 * nl), copy = v / (2 * nl) % R.copies;
            const bool down = vv < nl;
            const int l = down ? lm + vv : lc - (vv - nl);
            Pending pd = down && l == lm ? carry : Pending{};
            if (!down) {
                for (int w = 0; w < N; ++w) {
                    if (!has(l, w)) continue;
                    const Box x = own(l, w);
                    const int y0 = (x.ya >> 1) - 1, z0 = D == 3 ? (x.za >> 1) - 1 : 0;
                    window(l + 1, y0, ((x.yb - 1) >> 1) + 2 - y0, z0, D == 3 ? ((x.zb - 1) >> 1) + 2 - z0 : 1,
                           [&](int a, int j, int k) {
                               if (l == lc)
                                   for (unsigned long long r : tail_line[line(a, j, k)]) read(w, r, ep);
                               else read(w, key(1, l + 1, a, 0, j, k), ep);
                           });
                    post_lines(l, w, true, ep + 1);
                }
                next();
                pd.kind = 2;
                pd.ep = ++ep;
            }
            const int np = 2 * NC * (down ? c->d.nu1 : c->d.nu2);
            for (int pass = 0; pass < np; ++pass) {
                const int a = pass / 2 % NC, colour = pass & 1;
                const unsigned e1 = ep + 1 + (unsigned)pass;
                for (int w = 0; w < N; ++w) {
                    if (!has(l, w)) continue;
                    fetch(l, w, pd);
                    lines(l, w, true, [&](int j, int k) {
                        if (holds(grid(l), a, j, k)) post(w, key(0, l, a, colour, j, k), e1);
                    });
                }
                next();
                pd.kind = 1;
                pd.a = a;
                pd.colour = colour;
                pd.ep = e1;
            }
            ep += (unsigned)np;
            if (!down) {
                const bool end = v == 2 * nl * ncyc - 1;
                if (l == lm && !end) {
                    carry = pd;
                    continue;
                }
                ++ep;
                if (!end)
                    for (int w = 0; w < N; ++w)
                        if (has(l, w)) post_lines(l, w, false, ep);
                next();
                continue;
            }
            ++ep;
            const bool last = l == lc;
            for (int w = 0; w < N; ++w)
                if (has(l, w)) fetch(l, w, pd);
            next();
            const int gs = P.lev[l].gs;
            for (int c0 = 0; c0 < NC; c0 += gs) {
                auto in = [&](int a) { return a >= c0 && a < c0 + gs; };
                for (int w = 0; w < N; ++w)
                    if (has(l, w))
                        lines(l, w, false, [&](int j, int k) {
                            for (int a = 0; a < NC; ++a)
                                if (in(a) && holds(grid(l), a, j, k)) post(w, key(1, l, a, 0, j, k), ep);
                        });
                next();
                for (int w = 0; w < N; ++w) {
                    if (!has(l + 1, w)) continue;
                    const Box x = own(l + 1, w);
                    window(l, 2 * x.ya - 1, 2 * (x.yb - x.ya) + 2, D == 3 ? 2 * x.za - 1 : 0,
                           D == 3 ? 2 * (x.zb - x.za) + 2 : 1, [&](int a, int j, int k) {
                               if (in(a)) read(w, key(1, l, a, 0, j, k), ep);
                           });
                    if (last)
                        lines(l + 1, w, false, [&](int j, int k) {
                            for (int a = 0; a < NC; ++a)
                                if (in(a) && holds(grid(l + 1), a, j, k)) post(w, key(2, l + 1, a, copy, j, k), ep + 1);
                        });
                }
                next();
            }
            if (!last) continue;
            const Grid &gt = grid(l + 1);
            for (int w = 0; w < N; ++w) {
                if (!has(l + 1, w) || (R.rows_only && !brick_has_rows(w, nt))) continue;
                for (int a = 0; a < NC; ++a)
                    for (int k = 0; k <= gt.n[2]; ++k)
                        for (int j = 0; j <= gt.n[1]; ++j)
                            if (holds(gt, a, j, k)) read(w, key(2, l + 1, a, copy, j, k), ep + 1);
                for (unsigned long long r : tail_rows[w]) post(w, r, ep + 2);
            }
            next();
            ep += 2;
        }
        check();
    }
};

// cycles a launch: enough for each copy to be written twice
constexpr int CYCLES = 2 * BRICK_TAIL_COPIES + 1;

}  // namespace

int main()
{
    const int grids[][4] = {{2, 16, 16, 0},   {2, 24, 24, 0},   {2, 32, 16, 0},   {2, 32, 32, 0},   {2, 64, 16, 0},
                            {2, 64, 32, 0},   {2, 128, 64, 0},  {2, 48, 16, 2},   {2, 40, 96, 1},   {3, 8, 8, 8},
                            {3, 8, 8, 16},    {3, 16, 16, 16},  {3, 16, 16, 32},  {3, 24, 24, 40},  {3, 32, 16, 32},
                            {3, 32, 32, 32},  {3, 32, 32, 64},  {3, 48, 48, 96},  {3, 64, 64, 128}};
    const int sweeps[][2] = {{2, 2}, {1, 1}, {1, 3}, {3, 1}};
    long long plans = 0, reads = 0, bad = 0, before = 0;
    for (auto &gr : grids)
        for (auto &nu : sweeps)
            for (int prec = 0; prec < 2; ++prec)
                for (int bc = 0; bc < (gr[0] == 3 ? 2 : 1); ++bc) {
                    const bool big = gr[0] == 3 && (long long)gr[1] * gr[2] * gr[3] > 40000;
                    if (big && (nu[0] != 2 || bc)) continue;   // the largest take a while
                    ibb_desc d{};
                    d.dim = gr[0];
                    for (int a = 0; a < 3; ++a) d.n[a] = a < d.dim ? gr[1 + a] : 1;
                    // tubes (open along z) or periodic along x and z; channels by the fourth number: periodic along x
                    // between walls, walls all round, or open along x
                    d.axis_bc[0] = d.dim == 3 ? (bc ? AX_PERIODIC : AX_WALLS) : gr[3];
                    d.axis_bc[1] = AX_WALLS;
                    d.axis_bc[2] = bc ? AX_PERIODIC : AX_INOUT;
                    d.h = 1.0 / d.n[0];
                    d.dt = d.sigma = d.eps = d.rho0 = d.mu_out = d.mu_max = 1.0;
                    d.omega = d.h;
                    d.nu1 = nu[0];
                    d.nu2 = nu[1];
                    d.max_cycles = 10;
                    d.rtol = 1e-8;
                    d.precision = prec ? IBB_FP32_REFINED : IBB_FP64;
                    d.inner_cycles = CYCLES;
                    if (check_desc(&d)) {
                        printf("bad descriptor\n");
                        return 1;
                    }
                    ibb_ctx c;
                    setup_shapes(&c, &d, 1, 1);
                    for (int vel = 0; vel < 2; ++vel) {
                        BrickPlan P;
                        if (!plan_bricks(&c, vel == 1, P)) continue;
                        ++plans;
                        Walk w(&c, P, vel == 1, Rules{BRICK_TAIL_COPIES, true});
                        w.run(CYCLES);
                        reads += w.reads;
                        // one copy that every workgroup of the tail's level reads
                        long long one = 0;
                        if (!big) {
                            Walk q(&c, P, vel == 1, Rules{1, false});
                            q.run(CYCLES);
                            one = q.unordered;
                        }
                        before += one > 0;
                        if (w.unordered || w.lost)
                            printf("%dD %dx%dx%d V(%d,%d) %s %s levels %d-%d, %d workgroups, tail %d: %lld reads out "
                                   "of order, %lld never posted\n",
                                   d.dim, d.n[0], d.n[1], d.n[2], nu[0], nu[1], prec ? "FP32" : "FP64",
                                   vel ? "velocity" : "pressure", P.lm, P.lc, P.nwg, w.nt, w.unordered, w.lost);
                        bad += w.unordered + w.lost;
                    }
                }
    printf("%lld plans, %lld reads, %lld mismatches; one copy for all: %lld plans out of order\n", plans, reads, bad,
           before);
    // a walk that could not find the unordered reads of one copy would prove nothing
    return bad != 0 || before == 0;
}
