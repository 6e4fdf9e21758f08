// The index arithmetic of a pass on the host: plans (make_plan) of random fibers on random lattices,
// and every index that the patch and bead kernels form with them, against the sets of nodes that
// they stand for.  Prints what was covered; the first fault ends the run with status 1.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "fpd_plan.hpp"

using namespace fpd;

namespace {

struct OneThread {  // a block of one thread
    int tid() const { return 0; }
    int threads() const { return 1; }
    void sync() const {}
    void low(int* p, int v) const { if (v < *p) *p = v; }
    void high(int* p, int v) const { if (v > *p) *p = v; }
    int add(int* p, int v) const { const int o = *p; *p += v; return o; }
};

long g_case = 0;
#define NEED(cond, ...)                                             \
    do {                                                            \
        if (!(cond)) {                                              \
            std::printf("case %ld: %s: ", g_case, #cond);           \
            std::printf(__VA_ARGS__);                               \
            std::printf("\n");                                      \
            std::exit(1);                                           \
        }                                                           \
    } while (0)

struct Cover { long plans, outgrown, allx, ally, tall, wrapx, wrapy, inside, left, left_patch; };

struct Check {
    Lattice L{};
    PatchUnit u{};
    std::vector<double> R;
    double rc = 0.0;
    std::vector<int> plan;
    std::vector<char> set[kPassSteps + 1];
    int W = 0, H = 0;

    const double (*pos() const)[2] { return (const double(*)[2])R.data() + u.first; }
    bool per() const { return L.periodic != 0; }
    // whether node (x, y) of the lattice is one that step t updates, by the kernels' indices
    bool in(int t, int x, int y) const {
        const int c = view_index(x, plan[0], L.nx), r = view_index(y, plan[2], L.ny);
        return c >= 0 && c < W && r >= 0 && r < H && set[t][(size_t)r * W + c];
    }
    // the nodes that (x, y) is pulled from: all in step t's set?  (a row behind a wall is the
    // node's own)
    bool ring(int t, int x, int y) const {
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                int yy = y + dy;
                if (yy < 0 || yy >= L.ny) {
                    if (!per()) continue;
                    yy = imod(yy, L.ny);
                }
                if (!in(t, imod(x + dx, L.nx), yy)) return false;
            }
        return true;
    }
    bool ring_in_patch(int x, int y) const {
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                int yy = y + dy;
                if (yy < 0 || yy >= L.ny) {
                    if (!per()) continue;
                    yy = imod(yy, L.ny);
                }
                if (view_index(imod(x + dx, L.nx), plan[0], L.nx) >= W ||
                    view_index(yy, plan[2], L.ny) >= H)
                    return false;
            }
        return true;
    }

    void make(Cover& cov) {
        const int len = plan_ints(u.cap_w, u.cap_h);
        plan.assign((size_t)len + 64, 0x5a5a5a5a);
        PlanLds sm;
        const bool outgrown = make_plan(OneThread(), L, rc, pos() - u.first, u, plan.data(), sm);
        for (int i = 0; i < 64; ++i) NEED(plan[len + i] == 0x5a5a5a5a, "plan written past its end");
        W = plan[1];
        H = plan[3];
        ++cov.plans;
        if (outgrown) {
            ++cov.outgrown;
            NEED(W == 0 && H == 0 && plan[4] == 0, "an outgrown plan holds nodes");
            for (int i = 0; i < u.n; ++i)
                NEED(!bead_in_plan(&plan[kPlanBoxes + 4 * i],
                                   bead_span(pos()[i][0], pos()[i][1], rc), 1),
                     "bead %d in an outgrown plan", i);
            return;
        }
        NEED(W >= 0 && W <= u.cap_w && W <= L.nx && H >= 0 && H <= u.cap_h && H <= L.ny, "%d x %d",
             W, H);
        NEED(W == 0 || (plan[0] >= 0 && plan[0] < L.nx), "first column %d", plan[0]);
        NEED(H == 0 || (plan[2] >= 0 && plan[2] < L.ny && (per() || plan[2] + H <= L.ny)),
             "first row %d", plan[2]);
        if (W == L.nx) ++cov.allx;
        if (per() && H == L.ny) ++cov.ally;
        if (H > kPlanRun) ++cov.tall;
        if (W < L.nx && plan[0] + W > L.nx) ++cov.wrapx;
        if (per() && H < L.ny && plan[2] + H > L.ny) ++cov.wrapy;
        for (int t = 1; t <= kPassSteps; ++t) {
            set[t].assign((size_t)W * H, 0);
            for (int r = 0; r < H; ++r) {
                const int* c = &plan[kPlanRows + 2 * ((t - 1) * u.cap_h + r)];
                NEED(c[0] >= 0 && c[0] <= c[1] && c[1] <= W, "step %d row %d: [%d, %d)", t, r,
                     c[0], c[1]);
                for (int k = c[0]; k < c[1]; ++k) set[t][(size_t)r * W + k] = 1;
            }
        }
        steps();
        partition();
        tiles();
    }
    // each step pulls only what the step before updated, in the patch
    void steps() {
        for (int t = 2; t <= kPassSteps; ++t)
            for (int r = 0; r < H; ++r)
                for (int c = 0; c < W; ++c)
                    if (set[t][(size_t)r * W + c]) {
                        const int y = plan[2] + r;
                        NEED(ring(t - 1, (plan[0] + c) % L.nx, y >= L.ny ? y - L.ny : y),
                             "step %d pulls row %d column %d from outside", t, r, c);
                    }
    }
    // the last step's set holds every grown box, in whole lanes of the march
    void partition() {
        for (int i = 0; i < u.n; ++i) {
            if (!bead_sane(pos()[i][0], pos()[i][1])) continue;
            const BeadSpan s = bead_span(pos()[i][0], pos()[i][1], rc);
            const int ylo = per() ? s.y0 - kPassMargin : std::max(s.y0 - kPassMargin, 0);
            const int yhi = std::min(s.y1 + kPassMargin, ylo + L.ny - 1);
            const int xhi = std::min(s.x1 + kPassMargin, s.x0 - kPassMargin + L.nx - 1);
            for (int y = ylo; y <= yhi; ++y) {
                if (!per() && y >= L.ny) continue;
                for (int x = s.x0 - kPassMargin; x <= xhi; ++x)
                    NEED(in(kPassSteps, imod(x, L.nx), per() ? imod(y, L.ny) : y),
                         "bead %d: node %d, %d not in the partition", i, x, y);
            }
        }
        if (L.nx % 2 == 0)
            for (int r = 0; r < H; ++r)
                for (int c = 0; c < W; ++c) {
                    const int x = (plan[0] + c) % L.nx;
                    const int d = view_index(x ^ 1, plan[0], L.nx);
                    NEED(set[kPassSteps][(size_t)r * W + c] ==
                             (d < W ? set[kPassSteps][(size_t)r * W + d] : 0),
                         "row %d column %d: half a lane", r, c);
                }
    }
    // every node of the first step in exactly one tile of the list
    void tiles() {
        const int tx = (W + kPatchX - 1) / kPatchX, ty = (H + u.tile_h - 1) / u.tile_h;
        std::vector<char> seen((size_t)tx * ty + 1, 0);
        const int* list = &plan[plan_tiles_at(u.cap_h)];
        NEED(plan[4] >= 0 && plan[4] <= tx * ty, "%d tiles", plan[4]);
        for (int i = 0; i < plan[4]; ++i) {
            const int x = list[i] & 0xffff, y = list[i] >> 16;
            NEED(x < tx && y < ty && !seen[(size_t)y * tx + x], "tile %d, %d", x, y);
            seen[(size_t)y * tx + x] = 1;
        }
        for (int r = 0; r < H; ++r)
            for (int c = 0; c < W; ++c)
                if (set[1][(size_t)r * W + c])
                    NEED(seen[(size_t)(r / u.tile_h) * tx + c / kPatchX], "row %d column %d", r, c);
    }
    // bead i anywhere at step t: if the bead kernel pulls for it, then from step t's set
    void bead(int i, double Rx, double Ry, int t, Cover& cov) {
        int i0, w, j0, j1;
        bead_box(Rx, Ry, rc, L.nx, L.ny, per(), i0, w, j0, j1);
        if (w <= 0 || j1 < j0) return;
        const bool pulled = bead_in_plan(&plan[kPlanBoxes + 4 * i], bead_span(Rx, Ry, rc), t);
        bool patch = true;
        for (int j = j0; j <= j1; ++j)
            for (int c = 0; c < w; ++c) {
                const int x = imod(i0 + c, L.nx), y = j >= L.ny ? j - L.ny : j;
                if (pulled)
                    NEED(ring(t, x, y), "step %d: bead %d at %g, %g pulls %d, %d from outside", t,
                         i, Rx, Ry, x, y);
                else if (patch)
                    patch = ring_in_patch(x, y);
            }
        if (pulled) {
            ++cov.inside;
        } else {
            ++cov.left;
            if (!patch) ++cov.left_patch;  // would have been read past the patch
        }
    }
};

}  // namespace

int main(int argc, char** argv) {
    const long cases = argc > 1 ? std::atol(argv[1]) : 400;
    std::mt19937_64 gen(20221214);
    auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(gen); };
    auto num = [&](int a, int b) { return std::uniform_int_distribution<int>(a, b)(gen); };
    Cover cov{};
    for (g_case = 0; g_case < cases; ++g_case) {
        Check k;
        k.L.nx = num(0, 1) ? num(8, 120) : num(120, 420);
        k.L.ny = num(0, 5) == 0 ? num(530, 1150) : num(6, 260);
        k.L.periodic = num(0, 1);
        k.u.n = num(1, 9);
        k.u.first = num(0, 3);
        k.u.tile_h = kPatchY << num(0, 1);
        k.rc = uni(1.0, 9.0);
        if (k.L.nx * k.L.ny < 15000 && num(0, 7) == 0)  // (up to the lattice and far past it)
            k.rc = std::exp(uni(2.0, 16.0));
        const bool tall = k.L.ny > 520 && num(0, 2) > 0;
        const double l0 = tall ? 1.02 * k.L.ny / k.u.n : uni(1.0, 12.0);
        plan_caps(k.u.n, l0, k.rc, k.L.nx, k.L.ny, k.u.cap_w, k.u.cap_h);
        const double th = tall ? uni(1.4, 1.7) : uni(0.0, 6.3);
        const double stretch = num(0, 3) ? uni(0.6, 1.3) : uni(1.0, 4.0), bend = uni(-0.5, 0.5);
        // the first bead anywhere, also some periods away; now and then near a wall or an edge
        double x = uni(-2.0, 3.0) * k.L.nx, y = uni(0.0, 1.0) * k.L.ny;
        if (tall) y = uni(-0.05, 0.1) * k.L.ny;
        if (k.L.periodic) y += num(-1, 1) * k.L.ny;
        k.R.assign(2 * (size_t)kMaxBeads, 0.0);
        for (int i = 0; i < k.u.n; ++i) {
            k.R[2 * (k.u.first + i)] = x;
            k.R[2 * (k.u.first + i) + 1] = y;
            x += stretch * l0 * std::cos(th + bend * i);
            y += stretch * l0 * std::sin(th + bend * i);
        }
        if (num(0, 19) == 0) k.R[2 * (k.u.first + num(0, k.u.n - 1))] = NAN;
        if (num(0, 19) == 0) k.R[2 * (k.u.first + num(0, k.u.n - 1)) + 1] = uni(-2e9, 2e9);
        k.make(cov);
        if (!k.W || !k.H) continue;
        for (int i = 0; i < k.u.n; ++i)
            for (int m = 0; m < 6; ++m) {
                const double d = m == 0 ? 0.0 : m < 4 ? 6.5 : 2.0 * k.L.ny;
                const double Rx = k.pos()[i][0] + uni(-d, d), Ry = k.pos()[i][1] + uni(-d, d);
                for (int t = 1; t <= kPassSteps; ++t) k.bead(i, Rx, Ry, t, cov);
            }
    }
    std::printf("plans %ld outgrown %ld allx %ld ally %ld tall %ld wrapx %ld wrapy %ld inside %ld "
                "left %ld left_patch %ld\n",
                cov.plans, cov.outgrown, cov.allx, cov.ally, cov.tall, cov.wrapx, cov.wrapy,
                cov.inside, cov.left, cov.left_patch);
    return 0;
}
