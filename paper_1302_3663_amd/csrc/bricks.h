// The levels of a V-cycle that are bound by latency, in one launch of many
// workgroups ("bricks"): plan, control block and launcher (kernel:
// bricks.hip).
#pragma once

#include "kernels.h"

namespace ibmg {

// threads of a brick workgroup; slots (pairs of neighbouring points along x,
// one of each colour) of a box, and of the lines around it, per thread
constexpr int BRICK_THREADS = 512;
constexpr int BRICK_SLOTS = 3;
// workgroups at most (one per CU of the chip)
constexpr int BRICK_MAX_WG = 256;
// LDS of a workgroup at most: the CU's, less the kernel's own shared data
constexpr int BRICK_LDS_BUDGET = 163840 - (int)(TAIL_MAX * sizeof(double)) - 256;
// The tail level's right-hand side goes to every workgroup with rows of the
// tail's matrix: BRICK_TAIL_ROWS at a time, dealt out in turn to those with a
// box on that level.  The others do not read it.  Its mailbox has two copies,
// used in turn by the cycles of a launch.
constexpr int BRICK_TAIL_ROWS = BRICK_THREADS / TAIL_LANES;
constexpr int BRICK_TAIL_COPIES = 2;
__host__ __device__ constexpr bool brick_has_rows(int wg, int n) { return wg * BRICK_TAIL_ROWS < n; }

// What a pass over one component of a level (velocity component, or the
// pressure) is made of, as uniform offsets: so one piece of code serves every
// component.  Axes: the component's own one first, then the others in order
// (pressure: x, y, z).
struct BrickPass {
    int win[3];          // bytes from the level's windows to this component's and the others'
    int step[3];         // bytes in a window from a line's point to the next along those axes
    unsigned coef[8];    // bytes from the level's arrays to: b, rho, and the viscous row's cell and edge
                         // viscosities (cu, cl, then mp, mm per other axis) or (from 2) the pressure row's
                         // face coefficients (above, below per axis)
    int img[3][2];       // bytes from a point to its ghost image below and above, per axis x, y, z
    int odd;             // bit 2 d + side: that image has the opposite sign
    int edge;            // the image bits (IMG) that also change the diagonal: axes that do not wrap
    int axis[3];         // the axes: bit position of their image bits
    int walls;           // bit n: the n-th axis has walls at both ends
    unsigned mail;       // words from a level's mailboxes to this component's
    int face_x;          // 1: faces along x
};

// One level cut into bricks: boxes of cy x cz lines along x (2D: cy rows,
// cz = 1), sy x sz of them, each in a window one line wider on every side, of
// wy lines a plane (the largest box's) and wn entries per component, at byte
// lds of the workgroup's LDS.  mx, mb: mailboxes, one uniform array of entries
// (brick_mail_words 8-byte words each) per component (the tail level's mx:
// BRICK_TAIL_COPIES of them).  The level's arrays lie
// `stride` bytes apart, in the order xp, bp, rp; then per component xu, bu,
// ru, rho, beta; muc; the edge viscosities.
struct BrickLev {
    int cy, cz, sy, sz;
    int lds, wn, wy;
    int gs;              // components restricted at once to the next level
    unsigned stride;
    int os, rs;          // own and ring slots a thread
    int nx, ns;          // entries of from_x, from_s a workgroup
    unsigned long long *mx, *mb;
    // made once per context (launch_brick_tables).  slots: per workgroup os,
    // then rs, times BRICK_THREADS slots of 16 bytes.  from_x: where the
    // entries of the window of level + 1's iterate come from that the
    // workgroup interpolates to this level; from_s: those of the window of
    // x sums of level - 1's residual that it restricts to this one.
    void *slots;
    unsigned *from_x, *from_s;
    BrickPass pass[3];
};
// entries of from_x and from_s: word of the mailboxes, opposite sign, zero
constexpr unsigned BRICK_NEG = 1u << 30, BRICK_ZERO = 1u << 31;

struct BrickPlan {
    int lm, lc;          // first and last level in bricks; level lc + 1 is the tail's
    int nwg, lds_bytes;
    int nu1, nu2;        // sweeps before and after the coarse correction
    Tail tail;
    int L, pad;          // for a cycle on one workgroup
    BrickLev lev[WG_MAXLEV];   // lev[lc + 1]: boxes of the tail level's restriction
};

// Control block of one system's launches (device memory, zero at first).
// arrive counts the workgroups that have started; state is 0 until the last
// of them sets GO, or one that waited longer than `limit` ticks of the
// 100 MHz clock takes the whole cycle upon itself (its number + BRICK_SOLO);
// the last one out clears them.  epoch numbers the exchanges.
constexpr int BRICK_GO = 1, BRICK_SOLO = 16;
struct BrickCtl {
    unsigned arrive, state, done, epoch;
    long long limit;
    int solo_runs;    // launches that ran on one workgroup
    int lost;         // workgroups that gave up waiting for a value: such results are worthless
};

// When a context launches bricks again after a launch that ran on one
// workgroup.  Something else held the chip then: a kernel of another stream,
// once, or another process, all the time.  So the context rests for the
// remainder of the solve and the next one; each further such launch doubles
// the rest, up to BRICK_REST_MAX solves, and each solve between that ran
// without one halves it.
constexpr int BRICK_REST_MAX = 256;
struct BrickRest {
    int left = 0, next = 1;   // solves still to rest for, with the present one; length of the next rest
    int seen = 0;             // launches on one workgroup so far
    bool resting() const { return left > 0; }
    void solve_begins()
    {
        if (left > 0) --left;
        else if (next > 1) next /= 2;
    }
    void saw(int solo_runs)
    {
        if (solo_runs == seen) return;
        seen = solo_runs;
        left = next + 1;
        next = next < BRICK_REST_MAX / 2 ? 2 * next : BRICK_REST_MAX;
    }
};

__host__ __device__ constexpr int brick_mail_words(int wsz) { return wsz / 4; }

// ncyc V-cycles from level plan.lm down to the tail and back, on the level's
// global x and b (xzero: x is zero at the start and need not be read);
// plan_dev is the device copy of plan
template <typename T>
void launch_bricks(int D, int vel, const LevTab<T> *tab, const BrickPlan *plan_dev, const BrickPlan &plan, int ncyc,
                   int xzero, BrickCtl *ctl, hipStream_t s);
// the tables of every level of a plan (its device copy complete but for them)
template <typename T>
void launch_brick_tables(int D, int vel, const LevTab<T> *tab, const BrickPlan *plan_dev, const BrickPlan &plan,
                         hipStream_t s);
// how many workgroups with lds_bytes of LDS can be on the current device at
// once
template <typename T>
int bricks_resident(int D, int vel, int lds_bytes);

}  // namespace ibmg
