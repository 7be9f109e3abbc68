// Immersed-boundary kernels: node binning, the spread of force and density
// to the faces (eq:discrForceCouple, eq:discrDensCouple) and of the
// viscosity maximum to cells and edges (eq:ViscExp), the interpolation of
// face velocities to nodes (eq:discrVelCouple), the Euler move of the
// nodes, and the spring breakage and force passes (eq:springF and the
// breakage rule of the "Elastic Forces" section).
//
// The spread runs as a gather: each lattice point visits the nodes of the
// bins around it, in ascending node order within a bin, so the result does
// not depend on thread timing and no atomics touch the fields.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ibmg {

// lattices of so many points and fewer are spread with a wave a point
constexpr long long SPREAD_WAVE_MAX_POINTS = 65536;

static inline unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

__device__ inline double domain_len(const Grid &g, int d) { return g.n[d] * g.h; }

// nearest periodic image of a separation along axis d
__device__ inline double min_image(const Grid &g, int d, double v)
{
    if (g.bc[d] != AX_PERIODIC) return v;
    const double L = domain_len(g, d);
    return v - L * floor(v / L + 0.5);
}

// ---------------------------------------------------------------------------
// counting sort with a deterministic order inside each bucket
// ---------------------------------------------------------------------------
__global__ void k_count_keys(const int *__restrict__ keys, int n, int *count)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) atomicAdd(&count[keys[t]], 1);
}

// exclusive scan of count[0..nb) into start[0..nb] in three passes over
// tiles of SCAN_TILE buckets: tile sums, a scan of the tile sums, and a
// scan inside every tile offset by its tile's start
constexpr int SCAN_TILE = 1024;

// inclusive scan of one int per thread across a 1024-thread block
__device__ inline int block_incl_scan(int v, int *buf)
{
    const int t = threadIdx.x;
    buf[t] = v;
    __syncthreads();
    for (int off = 1; off < SCAN_TILE; off <<= 1) {
        const int w = t >= off ? buf[t - off] : 0;
        __syncthreads();
        buf[t] += w;
        __syncthreads();
    }
    const int r = buf[t];
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(1024) k_scan_tiles(const int *__restrict__ count, int nb, int *tsum)
{
    __shared__ int buf[SCAN_TILE];
    const int i = blockIdx.x * SCAN_TILE + threadIdx.x;
    const int r = block_incl_scan(i < nb ? count[i] : 0, buf);
    if (threadIdx.x == SCAN_TILE - 1) tsum[blockIdx.x] = r;
}

// one block: tsum[0..nt) -> exclusive prefix in place; start[nb] = total
__global__ void __launch_bounds__(1024) k_scan_tsum(int *tsum, int nt, int *start, int nb)
{
    __shared__ int buf[SCAN_TILE];
    int carry = 0;
    for (int base = 0; base < nt; base += SCAN_TILE) {
        const int i = base + threadIdx.x;
        const int v = i < nt ? tsum[i] : 0;
        const int r = block_incl_scan(v, buf);
        if (i < nt) tsum[i] = carry + r - v;
        carry += buf[SCAN_TILE - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) start[nb] = carry;
}

__global__ void __launch_bounds__(1024) k_scan_apply(const int *__restrict__ count, int nb, const int *__restrict__ tsum,
                                                     int *start)
{
    __shared__ int buf[SCAN_TILE];
    const int i = blockIdx.x * SCAN_TILE + threadIdx.x;
    const int v = i < nb ? count[i] : 0;
    const int r = block_incl_scan(v, buf);
    if (i < nb) start[i] = tsum[blockIdx.x] + r - v;
}

int scan_scratch_ints(long long nb) { return (int)((nb + SCAN_TILE - 1) / SCAN_TILE) + 2; }

__global__ void k_scatter_keys(const int *__restrict__ keys, int n, const int *__restrict__ start, int *cursor, int *ids)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int k = keys[t];
    const int pos = start[k] + atomicAdd(&cursor[k], 1);
    ids[pos] = t;
}

// order each bucket by id modulo `mod` (mod = 0: by id).  A one-wavefront
// workgroup takes `per` neighbouring buckets at a time: its lanes look up
// their lengths together, and each bucket of two and more is loaded into LDS
// and every entry written to its rank, the number of entries with a smaller
// key (keys within a bucket are distinct).  A bucket longer than the LDS tile
// is ordered by the first lane, by insertion.  Most of the bins of a domain
// are empty: looked up one after the other, 2 M of them took 95 us, and take 28 so.
constexpr int RANK_TILE = 1024;
constexpr int RANK_GRID = 8192, RANK_PER = 16;

__global__ void __launch_bounds__(64) k_sort_buckets(const int *__restrict__ start, int nb, int *ids, int mod, int per)
{
    __shared__ int tile[RANK_TILE];
    for (long long b0 = (long long)blockIdx.x * per; b0 < nb; b0 += (long long)gridDim.x * per) {
        const int own = (int)b0 + (int)threadIdx.x;
        int first = 0, len = 0;
        if ((int)threadIdx.x < per && own < nb) {
            first = start[own];
            len = start[own + 1] - first;
        }
        unsigned long long mask = __ballot(len > 1);
        while (mask) {
            const int l = __builtin_ctzll(mask);
            mask &= mask - 1;
            const int lo = __builtin_amdgcn_readlane(first, l), n = __builtin_amdgcn_readlane(len, l), hi = lo + n;
            if (n <= RANK_TILE) {
                for (int q = threadIdx.x; q < n; q += blockDim.x) tile[q] = ids[lo + q];
                __syncthreads();
                for (int q = threadIdx.x; q < n; q += blockDim.x) {
                    const int v = tile[q];
                    const int kv = mod ? v % mod : v;
                    int rank = 0;
                    for (int r = 0; r < n; ++r) {
                        const int w = tile[r];
                        rank += (mod ? w % mod : w) < kv;
                    }
                    ids[lo + rank] = v;
                }
                __syncthreads();
            } else if (threadIdx.x == 0) {
                for (int i = lo + 1; i < hi; ++i) {
                    const int v = ids[i];
                    const int kv = mod ? v % mod : v;
                    int j = i - 1;
                    while (j >= lo && (mod ? ids[j] % mod : ids[j]) > kv) {
                        ids[j + 1] = ids[j];
                        --j;
                    }
                    ids[j + 1] = v;
                }
            }
        }
    }
}

void launch_bucket_sort(const int *keys, int n, int nbuckets, int *count, int *start, int *ids, int mod,
                        int *scan_tmp, hipStream_t s)
{
    launch_fill<int>(count, nbuckets, 0, s);
    if (n > 0) hipLaunchKernelGGL(k_count_keys, dim3(nblk(n)), dim3(256), 0, s, keys, n, count);
    const int nt = (nbuckets + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL(k_scan_tiles, dim3(nt), dim3(SCAN_TILE), 0, s, count, nbuckets, scan_tmp);
    hipLaunchKernelGGL(k_scan_tsum, dim3(1), dim3(SCAN_TILE), 0, s, scan_tmp, nt, start, nbuckets);
    hipLaunchKernelGGL(k_scan_apply, dim3(nt), dim3(SCAN_TILE), 0, s, count, nbuckets, scan_tmp, start);
    launch_fill<int>(count, nbuckets, 0, s);
    if (n > 0) hipLaunchKernelGGL(k_scatter_keys, dim3(nblk(n)), dim3(256), 0, s, keys, n, start, count, ids);
    // buckets beyond the first RANK_GRID share workgroups, up to RANK_PER each
    const int per = std::max(1, std::min(RANK_PER, nbuckets / RANK_GRID));
    const long long ng = std::min<long long>(std::max(1, (nbuckets + per - 1) / per), RANK_GRID * 16);
    launch_timed(k_sort_buckets, dim3((unsigned)ng), dim3(64), s, start, nbuckets, ids, mod, per);
}

// ---------------------------------------------------------------------------
// bins: cell size at least twice the delta width along each axis, so every
// node within the support of a point lies in the point's bin or a neighbour
// ---------------------------------------------------------------------------
__device__ inline int bin_coord(const Bins &bins, int d, double x)
{
    int b = (int)floor(x / bins.bs[d]);
    return b < 0 ? 0 : (b >= bins.nb[d] ? bins.nb[d] - 1 : b);
}

__global__ void k_bin_of(Grid g, Bins bins, const double *__restrict__ X, long long stride, int eta)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= eta) return;
    int b[3] = {0, 0, 0};
    for (int d = 0; d < g.D; ++d) {
        double x = X[d * stride + s];
        if (g.bc[d] == AX_PERIODIC) {
            const double L = domain_len(g, d);
            x -= L * floor(x / L);
        }
        b[d] = bin_coord(bins, d, x);
    }
    bins.bin_of[s] = (b[2] * bins.nb[1] + b[1]) * bins.nb[0] + b[0];
}

// Bins are at least the delta width w wide (bins_for_width), so the nodes
// within a point's support lie in its own bin or the BIN_REACH bins on
// either side.
constexpr int BIN_REACH = 2, BIN_SPAN = 2 * BIN_REACH + 1;

// distinct bins along axis d where the points of bin b look for nodes, in
// increasing offset from b - BIN_REACH (wrapped on a periodic axis; every
// bin, in order, when a periodic axis has no more than 2 BIN_REACH)
__device__ inline int bin_candidates(const Grid &g, const Bins &bins, int d, int b, int lst[BIN_SPAN])
{
    if (d >= g.D) {
        lst[0] = 0;
        return 1;
    }
    const int nb = bins.nb[d];
    if (g.bc[d] == AX_PERIODIC && nb <= 2 * BIN_REACH) {
        for (int t = 0; t < nb; ++t) lst[t] = t;
        return nb;
    }
    int c = 0;
    for (int o = -BIN_REACH; o <= BIN_REACH; ++o) {
        int t = b + o;
        if (g.bc[d] == AX_PERIODIC) t = (t + nb) % nb;
        else if (t < 0 || t >= nb) continue;
        lst[c++] = t;
    }
    return c;
}

// The candidate bins along x as at most two runs of consecutive bins (a
// wrap splits them): each run's nodes are one range of the sorted ids, in
// bin order and ascending within a bin, as bin by bin.
struct XRuns {
    int lo[2], hi[2];
    int n;
};

__device__ inline XRuns x_runs(const int lst[BIN_SPAN], int cnt)
{
    XRuns r;
    r.n = 1;
    r.lo[0] = r.hi[0] = lst[0];
    r.lo[1] = r.hi[1] = 0;
    for (int e = 1; e < cnt; ++e) {
        if (lst[e] == r.hi[r.n - 1] + 1) {
            r.hi[r.n - 1] = lst[e];
        } else {
            r.lo[r.n] = r.hi[r.n] = lst[e];
            ++r.n;
        }
    }
    return r;
}

// near[bin]: does any bin where the bin's points look hold a node?  Marked from
// the occupied bins into cleared flags: asked bin by bin, 2 M bins took 90 us,
// so with 40000 nodes 14 and 5 for the clearing.
__global__ void __launch_bounds__(256) k_bin_near(Grid g, Bins bins, int eta)
{
    // a thread a node and (y, z) offset; the first node of a bin marks for it
    constexpr int ROWS = BIN_SPAN * BIN_SPAN;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)eta * ROWS) return;
    const int p = (int)(t / ROWS), o = (int)(t - (long long)p * ROWS);
    const int bin = bins.bin_of[bins.sorted[p]];
    if (bins.start[bin] != p) return;
    const int b[3] = {bin % bins.nb[0], (bin / bins.nb[0]) % bins.nb[1], bin / (bins.nb[0] * bins.nb[1])};
    // the e-th bin along axis d that looks at bin b: the relation of
    // bin_candidates goes both ways
    auto looks = [&](int d, int e) -> int {
        if (d >= g.D) return e == 0 ? 0 : -1;
        const int nb = bins.nb[d];
        const bool per = g.bc[d] == AX_PERIODIC;
        if (per && nb <= 2 * BIN_REACH) return e < nb ? e : -1;
        const int q = b[d] + e - BIN_REACH;
        if (per) return q < 0 ? q + nb : (q >= nb ? q - nb : q);
        return q >= 0 && q < nb ? q : -1;
    };
    const int y = looks(1, o % BIN_SPAN), z = looks(2, o / BIN_SPAN);
    if (y < 0 || z < 0) return;
    unsigned char *row = bins.near + (z * bins.nb[1] + y) * bins.nb[0];
#pragma unroll
    for (int e = 0; e < BIN_SPAN; ++e) {
        const int x = looks(0, e);
        if (x >= 0) row[x] = 1;
    }
}

void launch_bin_nodes(const Grid &g, const Bins &bins, const double *X, long long stride, int eta, int *scan_tmp,
                      hipStream_t s)
{
    if (eta > 0) hipLaunchKernelGGL(k_bin_of, dim3(nblk(eta)), dim3(256), 0, s, g, bins, X, stride, eta);
    launch_bucket_sort(bins.bin_of, eta, bins.nbins, bins.count, bins.start, bins.sorted, 0, scan_tmp, s);
    if (bins.near) {
        launch_fill<unsigned char>(bins.near, bins.nbins, 0, s);
        if (eta > 0)
            hipLaunchKernelGGL(k_bin_near, dim3(nblk((long long)eta * BIN_SPAN * BIN_SPAN)), dim3(256), 0, s, g, bins,
                               eta);
    }
}

// the bins where a point looks for nodes, along each axis, and its own bin
struct BinNbr {
    int cnt[3];
    int lst[3][BIN_SPAN];
    int own;
};

__device__ inline BinNbr bin_neighbours(const Grid &g, const Bins &bins, const double x[3])
{
    BinNbr r;
    int b[3];
    for (int d = 0; d < 3; ++d) {
        b[d] = 0;
        if (d < g.D) {
            double xx = x[d];
            if (g.bc[d] == AX_PERIODIC) {
                const double L = domain_len(g, d);
                xx -= L * floor(xx / L);
            }
            b[d] = bin_coord(bins, d, xx);
        }
        r.cnt[d] = bin_candidates(g, bins, d, b[d], r.lst[d]);
    }
    r.own = (b[2] * bins.nb[1] + b[1]) * bins.nb[0] + b[0];
    return r;
}

// no node where the point looks: every sum over candidates is empty
__device__ inline bool nothing_near(const Bins &bins, const BinNbr &nbr)
{
    return bins.near && !bins.near[nbr.own];
}

// delta~(x - X_s, w) = w^-D prod_d phi((x_d - X_d) / w), zero outside the support
__device__ inline double delta_w(const Grid &g, int kernel, double inv_w, double scale, const double x[3],
                                 const double *__restrict__ X, long long stride, int s)
{
    double w = scale;
    for (int d = 0; d < g.D; ++d) {
        const double r = min_image(g, d, x[d] - X[d * stride + s]) * inv_w;
        if (!(fabs(r) < 2.0)) return 0.0;
        w *= phi_eval(kernel, r);
    }
    return w;
}

__device__ inline void lattice_coord(const Grid &g, int vmask, int i, int j, int k, double x[3])
{
    const int q[3] = {i, j, k};
    for (int d = 0; d < 3; ++d) x[d] = ((vmask >> d) & 1) ? q[d] * g.h : (q[d] + 0.5) * g.h;
}

// ---------------------------------------------------------------------------
// Spread through a table of factors.  A node's delta is a product of one
// factor per axis, and the (4 w / h)^D lattice points in its support share
// them: a gather that works out each factor where it is used is bound by its
// cosines, three in FP64 for every pair of point and node.  So the factors are
// worked out once a node and lattice index (k_node_table), by the expressions
// of delta_w, and the gathers multiply them in its order: the same bits.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_node_table(Grid g, int kernel, Bins bins, const double *__restrict__ X,
                                                    const double *__restrict__ F, long long stride, int eta,
                                                    double width, NodeTab tab)
{
    // a lattice point's coordinate is rounded before a node's is taken off, as
    // where points work out their own
#pragma clang fp contract(off)
    // a thread a node, lattice kind and axis
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int runs = 2 * g.D;
    if (t >= (long long)eta * runs) return;
    const int p = (int)(t / runs), q = (int)(t - (long long)p * runs), v = q / g.D, d = q - v * g.D;
    const int s = bins.sorted[p], n = g.n[d];
    double *rec = tab.rec + (long long)p * tab.record;
    const double Xd = X[d * stride + s], inv_w = 1.0 / width;
    double c = Xd;
    if (g.bc[d] == AX_PERIODIC) c -= domain_len(g, d) * floor(c / domain_len(g, d));
    // one index below the support; a node far outside reaches nothing
    const double lo = floor((c - 2.0 * width) / g.h - (v ? 0.0 : 0.5));
    const bool reach = lo > -1e9 && lo < 1e9;
    const int base = reach ? (int)lo : -(1 << 30);
    reinterpret_cast<int *>(rec)[v * 4 + d] = base;
    if (v == 0 && F) rec[4 + d] = F[d * stride + s];
    double *f = rec + 8 + (v * g.D + d) * tab.nt;
    for (int e = 0; e < tab.nt; ++e) {
        int i = base + e;
        if (g.bc[d] == AX_PERIODIC) i = i < 0 ? i + n : (i >= n ? i - n : i);
        const double x = v ? i * g.h : (i + 0.5) * g.h;
        const double r = min_image(g, d, x - Xd) * inv_w;
        f[e] = reach && fabs(r) < 2.0 ? phi_eval(kernel, r) : 0.0;
    }
}

// A wave takes a box of 8 x 4 x 2 lattice points (8 x 8 in two dimensions) and
// walks the nodes of all bins that any of them looks at, in the order of
// bin_candidates, so that ranges, indices and records are scalar and the lanes
// read the same few lines of a record's factors; nodes that reach none of the
// points are passed over.  With a point to itself a lane walked fewer nodes,
// but each lane its own: a load touched some 25 lines, and that bound the
// gather.  256 x 256 x 512 points, 150000 nodes, width 2.6 h: 3.3-4.4 ms a
// lattice with the factors worked out for every pair, 2.1-3.4 through the
// table with a point a lane, 1.2-1.4 so; 128 x 128 x 256 points, 40000 nodes,
// width 1.3 h: 361-534, 171-286 and 120-133 us.
template <int D>
struct BoxGather {
    static constexpr int BX = 8, BY = D == 3 ? 4 : 8, BZ = D == 3 ? 2 : 1;
    const int *start;
    const double *rec;
    int q[3], n[3], off[3], head[3], record, nt;
    int nb[3], qlo[3], qhi[3], first[3], cnt[3], lo[2], hi[2], runs;
    bool near;

    // this wave's box and lane's point; false: no box
    __device__ bool place(const Grid &g, int vmask, int i0, int j0, int k0, int &i, int &j, int &k)
    {
        const int lane = threadIdx.x & 63;
        i = i0 + (lane & 7);
        j = j0 + (lane >> 3) % BY;
        k = k0 + (lane >> 3) / BY;
        const int o[3] = {i0, j0, k0}, e[3] = {BX, BY, BZ};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            qlo[d] = o[d];
            qhi[d] = min(o[d] + e[d], stored_extent(g, d, (vmask >> d) & 1)) - 1;
        }
        q[0] = i;
        q[1] = j;
        q[2] = k;
        return i <= qhi[0] && j <= qhi[1] && k <= qhi[2];
    }
    __device__ void bins_of(const Grid &g, const Bins &bins, const NodeTab &tab, int vmask, bool live)
    {
        start = bins.start;
        rec = tab.rec;
        record = tab.record;
        nt = tab.nt;
        int own = 0;
        double x[3], xl[3], xh[3];
        lattice_coord(g, vmask, q[0], q[1], q[2], x);
        lattice_coord(g, vmask, qlo[0], qlo[1], qlo[2], xl);
        lattice_coord(g, vmask, qhi[0], qhi[1], qhi[2], xh);
#pragma unroll
        for (int d = D - 1; d >= 0; --d) {
            const int v = (vmask >> d) & 1;
            const bool per = g.bc[d] == AX_PERIODIC;
            nb[d] = bins.nb[d];
            n[d] = per ? g.n[d] : 0;
            head[d] = v * 4 + d;
            off[d] = 8 + (v * D + d) * nt;
            own = own * nb[d] + bin_coord(bins, d, x[d]);
            const int b0 = __builtin_amdgcn_readfirstlane(bin_coord(bins, d, xl[d])) - BIN_REACH;
            const int b1 = __builtin_amdgcn_readfirstlane(bin_coord(bins, d, xh[d])) + BIN_REACH;
            if (per && b1 - b0 + 1 >= nb[d]) {
                first[d] = 0;
                cnt[d] = nb[d];
            } else if (per) {
                first[d] = b0 < 0 ? b0 + nb[d] : b0;
                cnt[d] = b1 - b0 + 1;
            } else {
                first[d] = max(b0, 0);
                cnt[d] = min(b1, nb[d] - 1) - first[d] + 1;
            }
        }
        if (D == 2) {
            first[2] = 0;
            cnt[2] = 1;
        }
        // along x the bins are one run, or two where they wrap
        const int last = first[0] + cnt[0] - 1;
        runs = last >= nb[0] ? 2 : 1;
        lo[0] = first[0];
        hi[0] = min(last, nb[0] - 1);
        lo[1] = 0;
        hi[1] = last - nb[0];
        near = __any(live && !(bins.near && !bins.near[own]));
    }
    // take(weight, record) for every node that reaches this lane's point.
    // Lanes look up the rows' ranges, then nodes, 64 at a time; the factors of
    // eight nodes are in flight together.
    template <typename F>
    __device__ void each(double scale, F take) const
    {
        constexpr int U = 8;
        const int lane = threadIdx.x & 63, total = cnt[2] * cnt[1] * runs;
        for (int t0 = 0; t0 < total; t0 += 64) {
            int p0 = 0, len = 0;
            if (t0 + lane < total) {
                const int t = (t0 + lane) / runs, r = (t0 + lane) - t * runs, c = t / cnt[1], b = t - c * cnt[1];
                int y = first[1] + b, z = D == 3 ? first[2] + c : 0;
                if (y >= nb[1]) y -= nb[1];
                if (D == 3 && z >= nb[2]) z -= nb[2];
                const int row = (z * nb[1] + y) * nb[0];
                p0 = start[row + (r ? lo[1] : lo[0])];
                len = start[row + (r ? hi[1] : hi[0]) + 1] - p0;
            }
            int sum = len;   // over the rows up to this one
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int s = __shfl_up(sum, o);
                sum += lane >= o ? s : 0;
            }
            const int all = __builtin_amdgcn_readlane(sum, 63);
            const int shift = p0 - (sum - len);   // place of a node less its number here
            for (int base = 0; base < all; base += 64) {
                const int num = base + lane;
                int row = 0;   // first row whose sum exceeds num
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) row += __shfl(sum, row + o - 1) <= num ? o : 0;
                const int at_row = __shfl(shift, row & 63), p = num < all ? num + at_row : 0;
                const int *__restrict__ hdr = reinterpret_cast<const int *>(rec + (long long)p * record);
                int h[D];
                bool reach = num < all;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    h[d] = hdr[head[d]];
                    reach = reach && (n[d] || (h[d] <= qhi[d] && h[d] + nt > qlo[d]));
                }
                unsigned long long mask = __ballot(reach);
                while (mask) {
                    const double *at[U];
                    double f[U][D];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        bool in = mask != 0;
                        const int l = in ? __builtin_ctzll(mask) : 0;
                        mask &= mask - 1;   // 0 stays 0
                        at[u] = rec + (long long)__builtin_amdgcn_readlane(p, l) * record;
                        int e[D];
#pragma unroll
                        for (int d = 0; d < D; ++d) {
                            e[d] = q[d] - __builtin_amdgcn_readlane(h[d], l);
                            if (n[d]) e[d] = e[d] < 0 ? e[d] + n[d] : (e[d] >= n[d] ? e[d] - n[d] : e[d]);
                            in = in && (unsigned)e[d] < (unsigned)nt;
                        }
#pragma unroll
                        for (int d = 0; d < D; ++d) f[u][d] = at[u][off[d] + (in ? e[d] : 0)];
                        f[u][0] = in ? f[u][0] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        double w = scale;
#pragma unroll
                        for (int d = 0; d < D; ++d) w *= f[u][d];
                        if (w != 0.0) take(w, at[u]);
                    }
                }
            }
        }
    }
};

// Whether boxes of E points along periodic axis d may look at all its bins and
// a point at some only.  Their walk would start at the axis' first bin and the
// point's own before its wrap, and add up the nodes in another order.
static bool walk_wraps(const Grid &g, const Bins &bins, int d, int E)
{
    return g.bc[d] == AX_PERIODIC && bins.nb[d] > 2 * BIN_REACH &&
           (E - 1) * g.h / bins.bs[d] + 2.0 + 2 * BIN_REACH >= bins.nb[d];
}

NodeTab node_table(const Grid &g, const Bins &bins, double width, int eta, double *at, long long room)
{
    NodeTab t{nullptr, 0, 0};
    long long points = 1;
    for (int d = 0; d < g.D; ++d) points *= stored_extent(g, d, 1);
    const double nt = ceil(4.0 * width / g.h) + 2.0;
    if (eta <= 0 || points <= SPREAD_WAVE_MAX_POINTS || nt > 64.0) return t;
    // an index of a short periodic axis could lie in a run twice
    for (int d = 0; d < g.D; ++d)
        if (g.bc[d] == AX_PERIODIC && nt > g.n[d]) return t;
    const int E[3] = {BoxGather<3>::BX, g.D == 3 ? BoxGather<3>::BY : BoxGather<2>::BY, BoxGather<3>::BZ};
    for (int d = 0; d < g.D; ++d)
        if (walk_wraps(g, bins, d, E[d])) return t;
    t.nt = (int)nt;
    t.record = 8 + 2 * g.D * t.nt;
    if ((long long)eta * t.record <= room) t.rec = at;
    return t;
}

// this wave's box of a lattice: four along x to a workgroup
template <int D>
__device__ inline bool wave_box(const Grid &g, int vmask, BoxGather<D> &nodes, int &i, int &j, int &k)
{
    using B = BoxGather<D>;
    const int ny = (stored_extent(g, 1, (vmask >> 1) & 1) + B::BY - 1) / B::BY;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nx = (stored_extent(g, 0, vmask & 1) + 4 * B::BX - 1) / (4 * B::BX);
    const int t = blockIdx.x / nx, z = t / ny;
    const int i0 = ((blockIdx.x - t * nx) * 4 + wave) * B::BX, j0 = (t - z * ny) * B::BY, k0 = z * B::BZ;
    return nodes.place(g, vmask, i0, j0, k0, i, j, k);
}
template <int D>
static unsigned wave_boxes(const Grid &g, int vmask)
{
    using B = BoxGather<D>;
    const long long nx = (stored_extent(g, 0, vmask & 1) + 4 * B::BX - 1) / (4 * B::BX);
    const long long ny = (stored_extent(g, 1, (vmask >> 1) & 1) + B::BY - 1) / B::BY;
    return (unsigned)(nx * ny * ((stored_extent(g, 2, (vmask >> 2) & 1) + B::BZ - 1) / B::BZ));
}

template <int D>
__global__ void __launch_bounds__(256) k_spread_face_t(Grid g, Phys ph, Bins bins, NodeTab tab, int has_f, int a,
                                                       double width, double *f_out, double *rho_out)
{
    const int vmask = face_mask(a);
    int i, j, k;
    BoxGather<D> nodes;
    const bool live = wave_box<D>(g, vmask, nodes, i, j, k);
    if (!__any(live)) return;
    double scale = 1.0;
    for (int d = 0; d < D; ++d) scale /= width;
    double accf = 0.0, accw = 0.0;
    nodes.bins_of(g, bins, tab, vmask, live);
    if (nodes.near)
        nodes.each(scale, [&](double w, const double *r) {
            if (has_f) accf += r[4 + a] * w;
            accw += w;
        });
    if (!live) return;
    const long long u = at(g, i, j, k);
    if (f_out) f_out[u] = accf;
    if (rho_out) rho_out[u] = ph.rho0 + ph.rho_b * ph.d0_pow_d * accw;
}

template <int D>
__global__ void __launch_bounds__(256) k_spread_visc_t(Grid g, Phys ph, Bins bins, NodeTab tab, int vmask,
                                                       double *mu_out)
{
    int i, j, k;
    BoxGather<D> nodes;
    const bool live = wave_box<D>(g, vmask, nodes, i, j, k);
    if (!__any(live)) return;
    const double width = ph.omega;
    double scale = 1.0, vol = 1.0;
    for (int d = 0; d < D; ++d) {
        scale /= width;
        vol *= 2.0 * width;
    }
    const double dmu = ph.mu_max - ph.mu_out;
    double best = ph.mu_out, wmax = 0.0;
    nodes.bins_of(g, bins, tab, vmask, live);
    if (dmu > 0.0 && nodes.near)
        nodes.each(scale, [&](double w, const double *) { wmax = w > wmax ? w : wmax; });
    if (wmax > 0.0) {
        const double cand = vol * dmu * wmax + ph.mu_out;
        best = cand > best ? cand : best;
    }
    if (live) mu_out[at(g, i, j, k)] = best;
}

void launch_node_table(const Grid &g, int kernel, const Bins &bins, const double *X, const double *F, long long stride,
                       int eta, double width, const NodeTab &tab, hipStream_t s)
{
    if (!tab.rec) return;
    launch_timed(k_node_table, dim3(nblk((long long)eta * 2 * g.D)), dim3(256), s, g, kernel, bins, X, F, stride, eta,
                 width, tab);
}

// f_a(x) = sum_s F_a(s) delta~ and rho_a(x) = rho0 + rho_b d0^D sum_s delta~
// at every closed-domain a-face
__global__ void __launch_bounds__(256) k_spread_face(Grid g, Phys ph, Bins bins, const double *__restrict__ X,
                                                     const double *__restrict__ F, long long stride, int a,
                                                     double width, double *f_out, double *rho_out)
{
    const int vmask = face_mask(a);
    int ext[3];
    for (int d = 0; d < 3; ++d) ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)ext[0] * ext[1] * ext[2]) return;
    const int i = (int)(t % ext[0]);
    t /= ext[0];
    const int j = (int)(t % ext[1]);
    const int k = (int)(t / ext[1]);
    double x[3];
    lattice_coord(g, vmask, i, j, k, x);
    const double inv_w = 1.0 / width;
    double scale = 1.0;
    for (int d = 0; d < g.D; ++d) scale /= width;
    const BinNbr nbr = bin_neighbours(g, bins, x);
    double accf = 0.0, accw = 0.0;
    const int nz = nothing_near(bins, nbr) ? 0 : nbr.cnt[2];
    const XRuns xr = x_runs(nbr.lst[0], nbr.cnt[0]);
    for (int c = 0; c < nz; ++c)
        for (int b = 0; b < nbr.cnt[1]; ++b)
            for (int rq = 0; rq < xr.n; ++rq) {
                const int row = (nbr.lst[2][c] * bins.nb[1] + nbr.lst[1][b]) * bins.nb[0];
                const int p1 = bins.start[row + xr.hi[rq] + 1];
                for (int p = bins.start[row + xr.lo[rq]]; p < p1; ++p) {
                    const int s = bins.sorted[p];
                    const double w = delta_w(g, ph.kernel, inv_w, scale, x, X, stride, s);
                    if (w == 0.0) continue;
                    if (F) accf += F[a * stride + s] * w;
                    accw += w;
                }
            }
    const long long u = at(g, i, j, k);
    if (f_out) f_out[u] = accf;
    if (rho_out) rho_out[u] = ph.rho0 + ph.rho_b * ph.d0_pow_d * accw;
}

// The same gather with one wave per lattice point, for lattices too small
// to fill the chip with one point per thread while a point may see
// thousands of nodes (small grids, dense biofilms).  The 64 lanes evaluate
// the weights of 64 consecutive candidates at once; the sums then take them
// in candidate order, through the same expressions as k_spread_face, so
// the result is the same bits.
__global__ void __launch_bounds__(256) k_spread_face_w(Grid g, Phys ph, Bins bins, const double *__restrict__ X,
                                                       const double *__restrict__ F, long long stride, int a,
                                                       double width, double *f_out, double *rho_out)
{
    const int vmask = face_mask(a);
    const int lane = threadIdx.x & 63;
    int ext[3];
    for (int d = 0; d < 3; ++d) ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    long long t = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= (long long)ext[0] * ext[1] * ext[2]) return;   // the whole wave
    const int i = (int)(t % ext[0]);
    t /= ext[0];
    const int j = (int)(t % ext[1]);
    const int k = (int)(t / ext[1]);
    double x[3];
    lattice_coord(g, vmask, i, j, k, x);
    const double inv_w = 1.0 / width;
    double scale = 1.0;
    for (int d = 0; d < g.D; ++d) scale /= width;
    const BinNbr nbr = bin_neighbours(g, bins, x);
    double accf = 0.0, accw = 0.0;
    const int nz = nothing_near(bins, nbr) ? 0 : nbr.cnt[2];
    const XRuns xr = x_runs(nbr.lst[0], nbr.cnt[0]);
    for (int c = 0; c < nz; ++c)
        for (int b = 0; b < nbr.cnt[1]; ++b)
            for (int rq = 0; rq < xr.n; ++rq) {
                const int row = (nbr.lst[2][c] * bins.nb[1] + nbr.lst[1][b]) * bins.nb[0];
                const int p1 = bins.start[row + xr.hi[rq] + 1];
                for (int base = bins.start[row + xr.lo[rq]]; base < p1; base += 64) {
                    const int p = base + lane;
                    double w = 0.0, fv = 0.0;
                    if (p < p1) {
                        const int s = bins.sorted[p];
                        w = delta_w(g, ph.kernel, inv_w, scale, x, X, stride, s);
                        if (F) fv = F[a * stride + s];
                    }
                    const int cnt = p1 - base < 64 ? p1 - base : 64;
                    for (int q = 0; q < cnt; ++q) {
                        const double wq = __shfl(w, q);
                        const double fq = __shfl(fv, q);
                        if (wq == 0.0) continue;
                        if (F) accf += fq * wq;
                        accw += wq;
                    }
                }
            }
    if (lane == 0) {
        const long long u = at(g, i, j, k);
        if (f_out) f_out[u] = accf;
        if (rho_out) rho_out[u] = ph.rho0 + ph.rho_b * ph.d0_pow_d * accw;
    }
}

void launch_spread_face(const Grid &g, const Phys &ph, const Bins &bins, const NodeTab &tab, const double *X,
                        const double *F, long long stride, int a, double width, double *f_out, double *rho_out,
                        hipStream_t s)
{
    long long n = 1;
    for (int d = 0; d < 3; ++d) n *= stored_extent(g, d, d == a);
    if (n <= SPREAD_WAVE_MAX_POINTS)
        launch_timed(k_spread_face_w, dim3((unsigned)((n + 3) / 4)), dim3(256), s, g, ph, bins, X, F, stride, a,
                     width, f_out, rho_out);
    else if (tab.rec && g.D == 3)
        launch_timed(k_spread_face_t<3>, dim3(wave_boxes<3>(g, face_mask(a))), dim3(256), s, g, ph, bins, tab, F ? 1 : 0, a, width, f_out,
                     rho_out);
    else if (tab.rec)
        launch_timed(k_spread_face_t<2>, dim3(wave_boxes<2>(g, face_mask(a))), dim3(256), s, g, ph, bins, tab, F ? 1 : 0, a, width, f_out,
                     rho_out);
    else
        launch_timed(k_spread_face, dim3(nblk(n)), dim3(256), s, g, ph, bins, X, F, stride, a, width, f_out,
                     rho_out);
}

// mu(x) = max over nodes of (2 omega)^D (mu_max - mu_out) delta~ + mu_out,
// mu_out where no node reaches
__global__ void __launch_bounds__(256) k_spread_visc(Grid g, Phys ph, Bins bins, const double *__restrict__ X,
                                                     long long stride, int vmask, double *mu_out)
{
    int ext[3];
    for (int d = 0; d < 3; ++d) ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)ext[0] * ext[1] * ext[2]) return;
    const int i = (int)(t % ext[0]);
    t /= ext[0];
    const int j = (int)(t % ext[1]);
    const int k = (int)(t / ext[1]);
    double x[3];
    lattice_coord(g, vmask, i, j, k, x);
    const double width = ph.omega;
    const double inv_w = 1.0 / width;
    double scale = 1.0, vol = 1.0;
    for (int d = 0; d < g.D; ++d) {
        scale /= width;
        vol *= 2.0 * width;
    }
    const double dmu = ph.mu_max - ph.mu_out;
    double best = ph.mu_out;
    if (dmu > 0.0) {
        const BinNbr nbr = bin_neighbours(g, bins, x);
        double wmax = 0.0;
        const int nz = nothing_near(bins, nbr) ? 0 : nbr.cnt[2];
        const XRuns xr = x_runs(nbr.lst[0], nbr.cnt[0]);
        for (int c = 0; c < nz; ++c)
            for (int b = 0; b < nbr.cnt[1]; ++b)
                for (int rq = 0; rq < xr.n; ++rq) {
                    const int row = (nbr.lst[2][c] * bins.nb[1] + nbr.lst[1][b]) * bins.nb[0];
                    const int p1 = bins.start[row + xr.hi[rq] + 1];
                    for (int p = bins.start[row + xr.lo[rq]]; p < p1; ++p) {
                        const double w = delta_w(g, ph.kernel, inv_w, scale, x, X, stride, bins.sorted[p]);
                        wmax = w > wmax ? w : wmax;
                    }
                }
        if (wmax > 0.0) {
            const double cand = vol * dmu * wmax + ph.mu_out;
            best = cand > best ? cand : best;
        }
    }
    mu_out[at(g, i, j, k)] = best;
}

// k_spread_visc with one wave per lattice point (see k_spread_face_w); the
// largest weight does not depend on the order the candidates are taken in
__global__ void __launch_bounds__(256) k_spread_visc_w(Grid g, Phys ph, Bins bins, const double *__restrict__ X,
                                                       long long stride, int vmask, double *mu_out)
{
    const int lane = threadIdx.x & 63;
    int ext[3];
    for (int d = 0; d < 3; ++d) ext[d] = stored_extent(g, d, (vmask >> d) & 1);
    long long t = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= (long long)ext[0] * ext[1] * ext[2]) return;   // the whole wave
    const int i = (int)(t % ext[0]);
    t /= ext[0];
    const int j = (int)(t % ext[1]);
    const int k = (int)(t / ext[1]);
    double x[3];
    lattice_coord(g, vmask, i, j, k, x);
    const double width = ph.omega;
    const double inv_w = 1.0 / width;
    double scale = 1.0, vol = 1.0;
    for (int d = 0; d < g.D; ++d) {
        scale /= width;
        vol *= 2.0 * width;
    }
    const double dmu = ph.mu_max - ph.mu_out;
    double best = ph.mu_out;
    if (dmu > 0.0) {
        const BinNbr nbr = bin_neighbours(g, bins, x);
        double wmax = 0.0;
        const int nz = nothing_near(bins, nbr) ? 0 : nbr.cnt[2];
        const XRuns xr = x_runs(nbr.lst[0], nbr.cnt[0]);
        for (int c = 0; c < nz; ++c)
            for (int b = 0; b < nbr.cnt[1]; ++b)
                for (int rq = 0; rq < xr.n; ++rq) {
                    const int row = (nbr.lst[2][c] * bins.nb[1] + nbr.lst[1][b]) * bins.nb[0];
                    const int p1 = bins.start[row + xr.hi[rq] + 1];
                    for (int p = bins.start[row + xr.lo[rq]] + lane; p < p1; p += 64) {
                        const double w = delta_w(g, ph.kernel, inv_w, scale, x, X, stride, bins.sorted[p]);
                        wmax = w > wmax ? w : wmax;
                    }
                }
        for (int o = 32; o > 0; o >>= 1) {
            const double v = __shfl_xor(wmax, o);
            wmax = v > wmax ? v : wmax;
        }
        if (wmax > 0.0) {
            const double cand = vol * dmu * wmax + ph.mu_out;
            best = cand > best ? cand : best;
        }
    }
    if (lane == 0) mu_out[at(g, i, j, k)] = best;
}

void launch_spread_visc(const Grid &g, const Phys &ph, const Bins &bins, const NodeTab &tab, const double *X,
                        long long stride, int vmask, double *mu_out, hipStream_t s)
{
    long long n = 1;
    for (int d = 0; d < 3; ++d) n *= stored_extent(g, d, (vmask >> d) & 1);
    if (n <= SPREAD_WAVE_MAX_POINTS)
        launch_timed(k_spread_visc_w, dim3((unsigned)((n + 3) / 4)), dim3(256), s, g, ph, bins, X, stride, vmask,
                     mu_out);
    else if (tab.rec && g.D == 3)
        launch_timed(k_spread_visc_t<3>, dim3(wave_boxes<3>(g, vmask)), dim3(256), s, g, ph, bins, tab, vmask, mu_out);
    else if (tab.rec)
        launch_timed(k_spread_visc_t<2>, dim3(wave_boxes<2>(g, vmask)), dim3(256), s, g, ph, bins, tab, vmask, mu_out);
    else
        launch_timed(k_spread_visc, dim3(nblk(n)), dim3(256), s, g, ph, bins, X, stride, vmask, mu_out);
}

// ---------------------------------------------------------------------------
// interpolation U_a(s) = sum_x u_a(x) delta~(x - X_s, w) h^D over the
// closed-domain a-faces (fixed faces contribute the values they hold)
// ---------------------------------------------------------------------------
//
// One workgroup per (node, component): each thread takes lattice points of
// the support box, the partial sums are combined in a fixed tree order.
constexpr int INTERP_BLOCK = 128;

__global__ void __launch_bounds__(INTERP_BLOCK) k_interp(Grid g, int kernel, double width, VelArrC<double> u,
                                                         const double *__restrict__ X, long long xstride, int eta,
                                                         double *U, long long ustride)
{
    const int s = blockIdx.x;
    const int a = blockIdx.y;
    if (s >= eta) return;
    const double inv_w = 1.0 / width;
    double scale = 1.0, hD = 1.0;
    for (int d = 0; d < g.D; ++d) {
        scale /= width;
        hD *= g.h;
    }
    double Xs[3] = {0.0, 0.0, 0.0};
    for (int d = 0; d < g.D; ++d) Xs[d] = X[d * xstride + s];
    const int vmask = face_mask(a);
    int qlo[3], ext[3];
    for (int d = 0; d < 3; ++d) {
        if (d >= g.D) { qlo[d] = 0; ext[d] = 1; continue; }
        const double off = ((vmask >> d) & 1) ? 0.0 : 0.5;
        qlo[d] = (int)floor((Xs[d] - 2.0 * width) / g.h - off);
        ext[d] = (int)ceil((Xs[d] + 2.0 * width) / g.h - off) - qlo[d] + 1;
    }
    const int ntap = ext[0] * ext[1] * ext[2];
    double acc = 0.0;
    for (int t = threadIdx.x; t < ntap; t += blockDim.x) {
        const int q[3] = {qlo[0] + t % ext[0], qlo[1] + (t / ext[0]) % ext[1], qlo[2] + t / (ext[0] * ext[1])};
        int qs[3] = {0, 0, 0};
        double w = scale;
        bool keep = true;
        for (int d = 0; d < g.D; ++d) {
            const int vert = (vmask >> d) & 1;
            const double xc = vert ? q[d] * g.h : (q[d] + 0.5) * g.h;
            const double r = (xc - Xs[d]) * inv_w;
            if (!(fabs(r) < 2.0)) { keep = false; break; }
            int tq = q[d];
            const int se = stored_extent(g, d, vert);
            if (g.bc[d] == AX_PERIODIC) tq = ((tq % g.n[d]) + g.n[d]) % g.n[d];
            else if (tq < 0 || tq >= se) { keep = false; break; }
            qs[d] = tq;
            w *= phi_eval(kernel, r);
        }
        if (keep) acc += u.c[a][at(g, qs[0], qs[1], qs[2])] * w;
    }
    __shared__ double red[INTERP_BLOCK];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = INTERP_BLOCK / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) U[a * ustride + s] = red[0] * hD;
}

// The same sum with a wave to a node and component, when the support spans at
// most INTERP_SPAN lattice indices along each axis: lane l works out the
// factor and the array index of one lattice index of one axis, and the taps
// take theirs from the lanes, in place of three cosines a tap and eight
// barriers a node.  A lane holds the two partial sums that two threads of the
// block hold, and they are added in the block's order: the same bits.
// Measured with 40000 nodes in 128 x 128 x 256: 353 us by blocks, 116 by waves.
constexpr int INTERP_SPAN = 16;

__global__ void __launch_bounds__(256) k_interp_w(Grid g, int kernel, double width, VelArrC<double> u,
                                                  const double *__restrict__ X, long long xstride, int eta, double *U,
                                                  long long ustride)
{
    const int a = blockIdx.y, s = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (s >= eta) return;   // the whole wave
    const int lane = threadIdx.x & 63;
    const double inv_w = 1.0 / width;
    double scale = 1.0, hD = 1.0;
    for (int d = 0; d < g.D; ++d) {
        scale /= width;
        hD *= g.h;
    }
    const int vmask = face_mask(a);
    int qlo[3], ext[3];
    double Xs[3] = {0.0, 0.0, 0.0};
    for (int d = 0; d < 3; ++d) {
        qlo[d] = 0;
        ext[d] = 1;
        if (d >= g.D) continue;
        Xs[d] = X[d * xstride + s];
        const double off = ((vmask >> d) & 1) ? 0.0 : 0.5;
        qlo[d] = (int)floor((Xs[d] - 2.0 * width) / g.h - off);
        ext[d] = (int)ceil((Xs[d] + 2.0 * width) / g.h - off) - qlo[d] + 1;
    }
    // lane l: lattice index l % INTERP_SPAN of axis l / INTERP_SPAN
    const int d0 = lane / INTERP_SPAN;
    double f = 0.0;
    int at0 = -1;   // index into the array, -1: not a tap
    if (d0 < g.D) {
        const int vert = (vmask >> d0) & 1;
        const int q = (d0 == 0 ? qlo[0] : (d0 == 1 ? qlo[1] : qlo[2])) + lane % INTERP_SPAN;
        double xc;
        {
#pragma clang fp contract(off)
            xc = vert ? q * g.h : (q + 0.5) * g.h;
        }
        const double r = (xc - (d0 == 0 ? Xs[0] : (d0 == 1 ? Xs[1] : Xs[2]))) * inv_w;
        if (fabs(r) < 2.0) {
            const int n = g.n[d0];
            const bool per = g.bc[d0] == AX_PERIODIC;
            const int tq = per ? ((q % n) + n) % n : q;
            if (per || (tq >= 0 && tq < stored_extent(g, d0, vert))) {
                at0 = tq;
                f = phi_eval(kernel, r);
            }
        }
    } else if (d0 == 2) {
        at0 = 0;   // two dimensions: no third axis
        f = 1.0;
    }
    const int exy = ext[0] * ext[1], ntap = exy * ext[2];
    double acc[2] = {0.0, 0.0};
    for (int t0 = 0; t0 < ntap; t0 += 128)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int t = t0 + 64 * e + lane;
            const int tz = t / exy, txy = t - tz * exy, ty = txy / ext[0], tx = txy - ty * ext[0];
            const bool in = t < ntap;
            const int lx = in ? tx : 0, ly = INTERP_SPAN + (in ? ty : 0), lz = 2 * INTERP_SPAN + (in ? tz : 0);
            const int ix = __shfl(at0, lx), iy = __shfl(at0, ly), iz = __shfl(at0, lz);
            const double fx = __shfl(f, lx), fy = __shfl(f, ly), fz = __shfl(f, lz);
            if (in && ix >= 0 && iy >= 0 && iz >= 0) {
                double w = scale * fx;
                w *= fy;
                if (g.D == 3) w *= fz;
                acc[e] += u.c[a][at(g, ix, iy, iz)] * w;
            }
        }
    double sum = acc[0] + acc[1];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o);
    if (lane == 0) U[a * ustride + s] = sum * hD;
}

void launch_interp(const Grid &g, int kernel, double width, const VelArrC<double> &u, const double *X,
                   long long xstride, int eta, double *U, long long ustride, hipStream_t s)
{
    if (eta <= 0) return;
    if (4.0 * width / g.h + 3.0 <= INTERP_SPAN) {
        launch_timed(k_interp_w, dim3((eta + 3) / 4, g.D), dim3(256), s, g, kernel, width, u, X, xstride, eta, U,
                     ustride);
        return;
    }
    launch_timed(k_interp, dim3(eta, g.D), dim3(INTERP_BLOCK), s, g, kernel, width, u, X, xstride, eta, U,
                       ustride);
}

// X += c U, periodic axes wrapped back into [0, L)
__global__ void k_euler(Grid g, double c, const double *__restrict__ U, double *X, long long stride, int eta)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= eta) return;
    for (int d = 0; d < g.D; ++d) {
        double x = X[d * stride + s] + c * U[d * stride + s];
        if (g.bc[d] == AX_PERIODIC) {
            const double L = domain_len(g, d);
            x -= L * floor(x / L);
        }
        X[d * stride + s] = x;
    }
}

void launch_euler(const Grid &g, double c, const double *U, double *X, long long stride, int eta, hipStream_t s)
{
    if (eta > 0) hipLaunchKernelGGL(k_euler, dim3(nblk(eta)), dim3(256), 0, s, g, c, U, X, stride, eta);
}

// ---------------------------------------------------------------------------
// springs
// ---------------------------------------------------------------------------
// separation X_j - X_i (nearest periodic image), each operation rounded on
// its own so that the breakage decision is reproducible
__device__ inline void separation_rn(const Grid &g, const double *__restrict__ X, long long stride, int i, int j,
                                     double v[3])
{
    for (int d = 0; d < 3; ++d) {
        v[d] = 0.0;
        if (d >= g.D) continue;
        double x = __dsub_rn(X[d * stride + j], X[d * stride + i]);
        if (g.bc[d] == AX_PERIODIC) {
            const double L = domain_len(g, d);
            x = __dsub_rn(x, __dmul_rn(L, floor(__dadd_rn(__ddiv_rn(x, L), 0.5))));
        }
        v[d] = x;
    }
}

__device__ inline double len2_rn(const double v[3])
{
    return __dadd_rn(__dadd_rn(__dmul_rn(v[0], v[0]), __dmul_rn(v[1], v[1])), __dmul_rn(v[2], v[2]));
}

__global__ void k_spring_break(Grid g, double ratio, const double *__restrict__ X, long long stride,
                               const int *__restrict__ ij, int m, const double *__restrict__ rest,
                               unsigned char *alive, int *n_broken)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m || !alive[e]) return;
    double v[3];
    separation_rn(g, X, stride, ij[e], ij[m + e], v);
    const double lim = __dmul_rn(ratio, rest[e]);
    if (len2_rn(v) > __dmul_rn(lim, lim)) {
        alive[e] = 0;
        atomicAdd(n_broken, 1);
    }
}

void launch_spring_break(const Grid &g, double ratio, const double *X, long long stride, const int *ij, int m,
                         const double *rest, unsigned char *alive, int *n_broken, hipStream_t s)
{
    if (m > 0)
        hipLaunchKernelGGL(k_spring_break, dim3(nblk(m)), dim3(256), 0, s, g, ratio, X, stride, ij, m, rest, alive,
                           n_broken);
}

// F_s = sum over surviving springs at s, in ascending spring order, of
// K (l - r) d / l with d = X_j - X_i (added at i, subtracted at j)
__global__ void __launch_bounds__(256) k_spring_force(Grid g, const double *__restrict__ X, long long stride, int eta,
                                                      const int *__restrict__ ij, int m,
                                                      const double *__restrict__ rest, const double *__restrict__ K,
                                                      const unsigned char *__restrict__ alive,
                                                      const int *__restrict__ inc_start,
                                                      const int *__restrict__ inc_list, double *F)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= eta) return;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int p = inc_start[s]; p < inc_start[s + 1]; ++p) {
        const int entry = inc_list[p];
        const int e = entry >= m ? entry - m : entry;
        if (!alive[e]) continue;
        const int i = ij[e], j = ij[m + e];
        double v[3];
        separation_rn(g, X, stride, i, j, v);
        const double l = sqrt(len2_rn(v));
        if (l == 0.0) continue;
        const double T = K[e] * (l - rest[e]);
        const double sg = (s == i) ? 1.0 : -1.0;
        for (int d = 0; d < g.D; ++d) acc[d] += sg * (T * v[d] / l);
    }
    for (int d = 0; d < g.D; ++d) F[d * stride + s] = acc[d];
}

void launch_spring_force(const Grid &g, const double *X, long long stride, int eta, const int *ij, int m,
                         const double *rest, const double *K, const unsigned char *alive, const int *inc_start,
                         const int *inc_list, double *F, hipStream_t s)
{
    if (eta > 0)
        launch_timed(k_spring_force, dim3(nblk(eta)), dim3(256), s, g, X, stride, eta, ij, m, rest, K, alive,
                           inc_start, inc_list, F);
}

// incidence keys: entry e -> node i of spring e, entry m + e -> node j
__global__ void k_incidence_keys(const int *__restrict__ ij, int m, int *keys)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 2 * m) keys[t] = ij[t];
}

void launch_incidence_keys(const int *ij, int m, int *keys, hipStream_t s)
{
    if (m > 0) hipLaunchKernelGGL(k_incidence_keys, dim3(nblk(2LL * m)), dim3(256), 0, s, ij, m, keys);
}

__global__ void k_count_alive(const unsigned char *__restrict__ alive, int m, int *out)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < m && alive[e]) atomicAdd(out, 1);
}

void launch_count_alive(const unsigned char *alive, int m, int *out, hipStream_t s)
{
    launch_fill<int>(out, 1, 0, s);
    if (m > 0) hipLaunchKernelGGL(k_count_alive, dim3(nblk(m)), dim3(256), 0, s, alive, m, out);
}

// ---------------------------------------------------------------------------
// detached fragments: connected components of the alive springs, each
// labelled by its smallest node id.  Labels only decrease and always name a
// node of the same component, so the fixed point does not depend on the
// order of the atomic updates: every component ends with one root, which is
// its smallest id.
// ---------------------------------------------------------------------------
__global__ void k_frag_anchor(Grid g, const double *__restrict__ X, long long stride, int eta, int axis, double dist,
                              unsigned char *anchored)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < eta) anchored[s] = X[axis * stride + s] < dist ? 1 : 0;
}

__global__ void k_frag_init(int *label, int eta)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < eta) label[s] = s;
}

// hook: for an alive spring whose ends carry different labels, point the
// larger label at the smaller one
__global__ void k_frag_hook(const int *__restrict__ ij, int m, const unsigned char *__restrict__ alive, int *label,
                            int *changed)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m || !alive[e]) return;
    const int a = label[ij[e]], b = label[ij[m + e]];
    if (a == b) return;
    const int hi = a > b ? a : b, lo = a > b ? b : a;
    if (atomicMin(&label[hi], lo) > lo) *changed = 1;
}

// shortcut: every node points straight at the end of its label chain
__global__ void k_frag_jump(int *label, int eta, int *changed)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= eta) return;
    const int l0 = label[s];
    int l = l0;
    while (true) {
        const int n = label[l];
        if (n == l) break;
        l = n;
    }
    if (l != l0) {
        label[s] = l;
        *changed = 1;
    }
}

__global__ void k_frag_mark(const int *__restrict__ label, const unsigned char *__restrict__ anchored, int eta,
                            int *root_anchored)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < eta && anchored[s]) root_anchored[label[s]] = 1;
}

// counts[0] += fragments, counts[1] += detached fragments
__global__ void k_frag_count(const int *__restrict__ label, const int *__restrict__ root_anchored, int eta,
                             int *counts)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= eta || label[s] != s) return;
    atomicAdd(&counts[0], 1);
    if (!root_anchored[s]) atomicAdd(&counts[1], 1);
}

void launch_frag_anchor(const Grid &g, const double *X, long long stride, int eta, int axis, double dist,
                        unsigned char *anchored, hipStream_t s)
{
    if (eta > 0)
        hipLaunchKernelGGL(k_frag_anchor, dim3(nblk(eta)), dim3(256), 0, s, g, X, stride, eta, axis, dist, anchored);
}

void launch_frag_init(int *label, int eta, hipStream_t s)
{
    if (eta > 0) hipLaunchKernelGGL(k_frag_init, dim3(nblk(eta)), dim3(256), 0, s, label, eta);
}

void launch_frag_round(const int *ij, int m, const unsigned char *alive, int *label, int eta, int *changed,
                       hipStream_t s)
{
    launch_fill<int>(changed, 1, 0, s);
    if (m > 0) hipLaunchKernelGGL(k_frag_hook, dim3(nblk(m)), dim3(256), 0, s, ij, m, alive, label, changed);
    if (eta > 0) hipLaunchKernelGGL(k_frag_jump, dim3(nblk(eta)), dim3(256), 0, s, label, eta, changed);
}

void launch_frag_count(const int *label, const unsigned char *anchored, int eta, int *root_anchored, int *counts,
                       hipStream_t s)
{
    launch_fill<int>(counts, 2, 0, s);
    if (eta <= 0) return;
    launch_fill<int>(root_anchored, eta, 0, s);
    hipLaunchKernelGGL(k_frag_mark, dim3(nblk(eta)), dim3(256), 0, s, label, anchored, eta, root_anchored);
    hipLaunchKernelGGL(k_frag_count, dim3(nblk(eta)), dim3(256), 0, s, label, root_anchored, eta, counts);
}

}  // namespace ibmg
