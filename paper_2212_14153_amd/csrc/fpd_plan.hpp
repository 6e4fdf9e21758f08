// fpd_plan.hpp -- the nodes around a fiber that the steps of a pass update.
//
// Integer arithmetic only, compiled for the device and (tests/plan) for the host: every index
// that the patch and bead kernels form on a patch buffer follows from the functions here.
#pragma once

#include "fpd_device.hpp"

namespace fpd {

// Whether a bead of support box s at step t of a pass is near enough to its box when the plan was
// made (b: x0, x1, y0, y1; x1 < x0: none): its supports in the steps left then stay inside the
// partition.  Such a box and its ring of one node lie inside the columns that step t updates
// (the partition grown by kPassSteps - t), so the bead kernel pulls from nothing else; a bead
// that has gone further is not pulled at all.
template <class P> __host__ __device__ inline bool bead_in_plan(P b, const BeadSpan& s, int t) {
    const int left = kPassSteps - t, k = kPassMargin - (left > 1 ? left : 1);
    return b[1] >= b[0] && s.x0 >= b[0] - k && s.x1 <= b[1] + k && s.y0 >= b[2] - k &&
           s.y1 <= b[3] + k;
}

// Size of a patch's buffers: one fiber of n beads stretched by half in any orientation, its
// supports and the margins around them.
__host__ __device__ inline void plan_caps(int n, double l0, double rc, int nx, int ny, int& w,
                                          int& h) {
    const double span = ceil(1.5 * (n - 1) * l0 + 2.0 * rc + 4.0);
    constexpr int grow = 2 * (kPassMargin + kPassSteps - 1);
    w = (int)fmin(span + grow + 3 * kPassAlign, (double)nx);
    h = (int)fmin(span + grow, (double)ny);
}

// LDS of make_plan: the beads' boxes, and the partition's columns on a run of patch rows with
// the kPassSteps - 1 rows on either side that the first step's growth looks at.
constexpr int kPlanRun = 512;
struct PlanLds {
    int bound[4];
    int box[kMaxBeads][4];  // x0, x1, y0, y1; x1 < x0: none
    int lo[kPlanRun + 2 * (kPassSteps - 1)], hi[kPlanRun + 2 * (kPassSteps - 1)];
    int tiles;
};

// The threads of a block that make a plan.
struct PlanBlock {
    __device__ int tid() const { return threadIdx.x; }
    __device__ int threads() const { return blockDim.x; }
    __device__ void sync() const { __syncthreads(); }
    __device__ void low(int* p, int v) const { atomicMin(p, v); }
    __device__ void high(int* p, int v) const { atomicMax(p, v); }
    __device__ int add(int* p, int v) const { return atomicAdd(p, v); }
};

// The plan of unit u for a pass, from the current positions R of its beads (every thread of one
// block B).  A row's columns are the hull of the grown boxes that meet it, so a fiber at an angle
// does not take its whole rectangle.  Returns (to every thread) whether the fiber has outgrown
// the unit's buffers: its plan is then empty, no bead in it.
template <class B>
__host__ __device__ inline bool make_plan(const B& blk, const Lattice& L, double rc,
                                          const double (*R)[2], const PatchUnit& u, int* plan,
                                          PlanLds& sm) {
    const int tid = blk.tid(), nt = blk.threads();
    const int nx = L.nx, ny = L.ny;
    const bool per = L.periodic != 0;
    constexpr int M = kPassMargin, E = kPassSteps - 1, P = kPassAlign - 1;
    for (int i = tid; i < 4; i += nt) sm.bound[i] = i & 1 ? -0x3fffffff : 0x3fffffff;
    if (tid == 0) sm.tiles = 0;
    blk.sync();
    for (int i = tid; i < u.n; i += nt) {
        const double Rx = R[u.first + i][0], Ry = R[u.first + i][1];
        BeadSpan s{0, -1, 0, -1};
        if (bead_sane(Rx, Ry)) {
            s = bead_span(Rx, Ry, rc);
            blk.low(&sm.bound[0], s.x0);
            blk.high(&sm.bound[1], s.x1);
            blk.low(&sm.bound[2], s.y0);
            blk.high(&sm.bound[3], s.y1);
        }
        const int o[4] = {s.x0, s.x1, s.y0, s.y1};
        for (int k = 0; k < 4; ++k) {
            sm.box[i][k] = o[k];
            plan[kPlanBoxes + 4 * i + k] = o[k];
        }
    }
    blk.sync();
    // the patch rectangle: first column bx and row by (unwrapped), W x H nodes; a side that
    // would span the lattice is the lattice (allx, ally)
    const bool none = sm.bound[0] > sm.bound[1];
    const long long bw = (long long)sm.bound[1] - sm.bound[0] + 1 + 2 * (M + E + P);
    const long long bh = (long long)sm.bound[3] - sm.bound[2] + 1 + 2 * (M + E);
    int bx = sm.bound[0] - M - E - P;
    int X0 = none ? 0 : imod(bx, nx);
    const int lead = X0 % kPassAlign;
    X0 -= lead;
    bx -= lead;
    const bool allx = bw + lead >= nx;
    int W = allx ? nx : (int)bw + lead;
    if (allx) X0 = bx = 0;
    int by = sm.bound[2] - M - E;
    const bool ally = per && bh >= ny;
    int H;
    if (ally) {
        by = 0;
        H = ny;
    } else if (!per) {
        const long long top = by + bh < ny ? by + bh : ny;
        by = by > 0 ? by : 0;
        H = top > by ? (int)(top - by) : 0;
    } else {
        H = (int)bh;
    }
    if (none) W = H = 0;
    const bool outgrown = W > u.cap_w || H > u.cap_h;
    if (outgrown) {
        W = H = 0;
        for (int i = tid; i < u.n; i += nt) plan[kPlanBoxes + 4 * i + 1] = plan[kPlanBoxes + 4 * i] - 1;
    }
    if (tid == 0) {
        plan[0] = X0;
        plan[1] = W;
        plan[2] = none ? 0 : (per ? imod(by, ny) : by);
        plan[3] = H;
    }
    // rows of a grown box in the rectangle, at most
    const int tall = (int)fmin(ceil(2.0 * rc) + 4 + 2 * M, (double)H);
    int* tiles = plan + plan_tiles_at(u.cap_h);
    for (int r0 = 0; r0 < H; r0 += kPlanRun) {
        const int run = H - r0 < kPlanRun ? H - r0 : kPlanRun, span = run + 2 * E;
        blk.sync();
        for (int i = tid; i < span; i += nt) {
            sm.lo[i] = 0x3fffffff;
            sm.hi[i] = -0x3fffffff;
        }
        blk.sync();
        // rows r0 - E .. r0 + run + E - 1 of the partition
        for (int k = tid; k < u.n * tall; k += nt) {
            const int i = k / tall, j = k - i * tall;
            const int* o = sm.box[i];
            const int top = o[2] - M - by, r = (ally || top > 0 ? top : 0) + j;
            if (o[1] < o[0] || r > o[3] + M - by) continue;
            int c0 = o[0] - M - bx, c1 = o[1] + M + 1 - bx;
            if (allx) {
                const int w = c1 - c0;
                c0 = imod(c0, nx);
                c1 = c0 + w;
            }
            c0 = c0 / kPassAlign * kPassAlign;  // (c0 >= 0); the march masks whole lanes
            c1 = (c1 + P) / kPassAlign * kPassAlign;
            if (allx && c1 > nx) {
                c0 = 0;
                c1 = nx;
            }
            for (int q = ally ? imod(r, ny) - ny : r; q < r0 + run + E; q += ny) {
                if (q >= r0 - E && (ally || (q >= 0 && q < H))) {
                    blk.low(&sm.lo[q - r0 + E], c0);
                    blk.high(&sm.hi[q - r0 + E], c1);
                }
                if (!ally) break;
            }
        }
        blk.sync();
        // each step's columns: m rows and columns more on either side, m = kPassSteps - t
        int2* rows = (int2*)(plan + kPlanRows);
        for (int i = tid; i < run; i += nt) {
            int l = sm.lo[i + E], h = sm.hi[i + E];
            for (int m = 0; m < kPassSteps; ++m) {
                if (m > 0) {
                    l = min(l, min(sm.lo[i + E - m], sm.lo[i + E + m]));
                    h = max(h, max(sm.hi[i + E - m], sm.hi[i + E + m]));
                }
                int cl = l - m, ch = h + m;
                if (allx && l < h && (cl < 0 || ch > nx)) {
                    cl = 0;
                    ch = nx;
                }
                cl = max(cl, 0);
                ch = min(ch, W);
                rows[(kPassSteps - 1 - m) * u.cap_h + r0 + i] = l < h && cl < ch ? int2{cl, ch}
                                                                                : int2{0, 0};
            }
        }
        // the tiles of the first step (kPlanRun is a multiple of a tile's rows)
        for (int ty = tid; ty < (run + u.tile_h - 1) / u.tile_h; ty += nt) {
            int l = 0x3fffffff, h = -0x3fffffff;
            for (int i = ty * u.tile_h; i < min((ty + 1) * u.tile_h, run) + 2 * E; ++i) {
                l = min(l, sm.lo[i]);
                h = max(h, sm.hi[i]);
            }
            if (l >= h) continue;
            l -= E;
            h += E;
            if (allx && (l < 0 || h > nx)) {
                l = 0;
                h = nx;
            }
            l = max(l, 0);
            h = min(h, W);
            if (l >= h) continue;
            const int t0 = l / kPatchX, t1 = (h - 1) / kPatchX;
            const int at = blk.add(&sm.tiles, t1 - t0 + 1);
            for (int tx = t0; tx <= t1; ++tx)
                tiles[at + tx - t0] = ((r0 / u.tile_h + ty) << 16) | tx;
        }
    }
    blk.sync();
    if (tid == 0) plan[4] = sm.tiles;
    return outgrown;
}
static_assert(kPlanRun % (4 * kPatchY) == 0, "a run of plan rows is whole tiles");

}  // namespace fpd
