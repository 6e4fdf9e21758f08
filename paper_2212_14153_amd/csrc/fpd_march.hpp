// fpd_march.hpp -- several fluid time steps in one pass over HBM (gfx950).
//
// One step reads and writes every population once, 18 values per node, and on a large lattice
// HBM bounds it (0.8 of the peak).  Away from the fiber nothing but the nodes themselves enters
// several consecutive steps, so a march does NT of them per visit: a wave takes a strip of
// columns and walks up a run of rows with NT pipeline stages, stage t one row behind stage
// t - 1, each row's populations handed on in registers.  The x neighbours of a
// lane's columns come from the next lane by whole-wave DPP moves, so there is no LDS and no
// barrier; the outermost columns of a wave lose one valid column per step and its run of rows
// one row per step on either side, which neighbouring waves recompute.  Intermediate rows are
// kept in the storage format, so the result has the bits of NT single steps.
//
// What bounds it, from counters at 8192 x 2048 (us of a march of four steps / its HBM bytes at
// the 6.65 TB/s of a copy / its vector instructions at 4, in float64 4.5, cycles each on 1024 SIMDs):
// float32 258 / 231 (1.54 GB) / 193, float64 527 / 451 (3.00 GB) / 256: HBM, which the overlapping
// columns and rows make read 1.5 times; float16 249 / 128 (0.85 GB) / 206, bfloat16 244 / 128 /
// 206: vector issue.  Instructions per node and step, recomputed ones included: 113 in
// float32 (94 without), 133 (113) in float64, 121 in the two-byte formats.  Whole run with the
// 40-bead fiber, per step: float32 195 -> 67 us, float64 385 -> 134, bfloat16 107 -> 60.
#pragma once

#include "fpd_device.hpp"

namespace fpd {

// Whole-wave moves by one lane; a lane without a source (the wave's first, resp. last)
// receives zero.  bound_ctrl lets the compiler fold the move into the instruction that uses
// it.
__device__ inline uint32_t lane_below(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xf, 0xf, true);
}
__device__ inline uint32_t lane_above(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xf, 0xf, true);
}
__device__ inline float lane_below(float v) { return __uint_as_float(lane_below(__float_as_uint(v))); }
__device__ inline float lane_above(float v) { return __uint_as_float(lane_above(__float_as_uint(v))); }
__device__ inline double lane_below(double v) {
    return __hiloint2double((int)lane_below((uint32_t)__double2hiint(v)),
                            (int)lane_below((uint32_t)__double2loint(v)));
}
__device__ inline double lane_above(double v) {
    return __hiloint2double((int)lane_above((uint32_t)__double2hiint(v)),
                            (int)lane_above((uint32_t)__double2loint(v)));
}

// ------------------------------------------------------------ buffer accesses -------
// One lattice row (its nine direction rows) as a buffer resource: an access past its end
// reads zero and writes nothing, so a lane is switched off by its offset, without a branch.
constexpr int kRowFlags = 0x00027000;      // raw buffer, 32-bit data format
constexpr unsigned kLaneOff = 0x80000000u; // beyond any row (rows stay below 2^31 bytes)

__device__ inline __amdgpu_buffer_rsrc_t row_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, kRowFlags);
}

constexpr int kStoreNt = 2;               // non-temporal

template <int W>
__device__ inline void row_load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff,
                                uint32_t (&w)[W]) {
    if constexpr (W == 1) {
        w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
    } else if constexpr (W == 2) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
        w[0] = x[0];
        w[1] = x[1];
    } else {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
        w[0] = x[0];
        w[1] = x[1];
        w[2] = x[2];
        w[3] = x[3];
    }
}
template <int W>
__device__ inline void row_store(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff,
                                 const uint32_t (&w)[W]) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    if constexpr (W == 1)
        __builtin_amdgcn_raw_buffer_store_b32(w[0], r, voff, soff, kStoreNt);
    else if constexpr (W == 2)
        __builtin_amdgcn_raw_buffer_store_b64(u2{w[0], w[1]}, r, voff, soff, kStoreNt);
    else
        __builtin_amdgcn_raw_buffer_store_b128(u4{w[0], w[1], w[2], w[3]}, r, voff, soff, kStoreNt);
}

// ------------------------------------------------------------ values of one lane ----
// C neighbouring nodes of one direction row as a lane holds them, in the storage format
// (W words).  pulled<SX>: the values one node left (SX = 1) or right (SX = -1) of each,
// i.e. a register of the lane or, at its edge, of the neighbouring lane.
template <int ST, int C> struct LaneRow {
    using Cd = Codec<ST>;
    using S = typename Cd::store_t;
    using T = typename Cd::T;
    static constexpr int W = C * (int)sizeof(S) / 4;
    static constexpr bool kPacked = sizeof(S) == 2;
    uint32_t w[W];
    __device__ inline T get(int i) const {
        if constexpr (sizeof(S) == 8)
            return __hiloint2double((int)w[2 * i + 1], (int)w[2 * i]);
        else if constexpr (sizeof(S) == 4)
            return __uint_as_float(w[i]);
        else
            return Cd::from_bits_scaled((w[i >> 1] >> (16 * (i & 1))) & 0xffffu);
    }
    template <int SX> __device__ inline void pulled(T (&o)[C]) const {
        if constexpr (SX == 0) {
#pragma unroll
            for (int i = 0; i < C; ++i) o[i] = get(i);
        } else if constexpr (SX == 1) {
            if constexpr (kPacked)
                o[0] = Cd::from_bits_scaled(lane_below(w[W - 1]) >> 16);
            else
                o[0] = lane_below(get(C - 1));
#pragma unroll
            for (int i = 1; i < C; ++i) o[i] = get(i - 1);
        } else {
            if constexpr (kPacked)
                o[C - 1] = Cd::from_bits_scaled(lane_above(w[0]) & 0xffffu);
            else
                o[C - 1] = lane_above(get(0));
#pragma unroll
            for (int i = 0; i + 1 < C; ++i) o[i] = get(i + 1);
        }
    }
    __device__ inline void set(const T (&t)[C]) {
        if constexpr (kPacked) {
#pragma unroll
            for (int i = 0; i < C; i += 2) w[i >> 1] = Cd::pack2_scaled(t[i], t[i + 1]);
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i) {
                if constexpr (sizeof(S) == 8) {
                    w[2 * i] = (uint32_t)__double2loint(t[i]);
                    w[2 * i + 1] = (uint32_t)__double2hiint(t[i]);
                } else {
                    w[i] = __float_as_uint(t[i]);
                }
            }
        }
    }
};

// Lanes on each side of a wave whose columns are not valid after NT steps.
constexpr int march_halo_lanes(int nt, int c) { return (nt + c - 1) / c; }

// What a march needs of one lattice.
struct MarchArgs {
    const void* src;
    void* dst;
    Lattice L;
    double u6, s_nu, s_q, s_e, s_eps, gx, gy;
    const PatchUnit* units;     // whose partitions (in plan `slot`) are not stored
    int n_units, slot;
    int strips, seg_rows;       // tiles: strips of columns, runs of rows
};

template <int ST, int NT, int C, int OL, int BC, bool FORCE>
struct March {
    using Row = LaneRow<ST, C>;
    using Cd = Codec<ST>;
    using T = typename Cd::T;
    using S = typename Cd::store_t;
    static constexpr int HL = (64 - OL) / 2;
    static_assert(HL >= march_halo_lanes(NT, C), "columns past the halo are not valid");
    static constexpr bool per = BC == 1;
    static constexpr bool kScaled = ST == FPD_F16DEV;

    // a stage boundary: directions 0, 1, 3 of the row being completed, and 2, 5, 6 of that
    // row and of the row below it, in two slots that change roles every row
    struct Held { Row mid[3], up[2][3]; };

    const char* src;
    char* dst;
    int nx, ny, y0, y1, lo1, hi1;
    unsigned rowb, planeb;              // bytes of a lattice row and of a direction row
    unsigned ld, st;                    // lane offsets of loads and stores
    int x0;                             // the lane's first column, before the wrap
    const PatchUnit* units;
    int slot;
    unsigned long long near;            // units whose patch rectangle meets the wave's tile
    T u6, s_nu, s_q, s_e, s_eps, Fx, Fy;
    Held h[NT > 1 ? NT - 1 : 1];
    Row q[2][9];

    __device__ inline int lo(int t) const { const int r = y0 - (NT - t); return per || r > 0 ? r : 0; }
    __device__ inline int hi(int t) const { const int r = y1 + (NT - t); return per || r < ny ? r : ny; }
    __device__ inline const char* row(int y) const { return src + (long long)y * rowb; }
    // Lane offset of the stores of row r: off for the columns that some fiber's partition
    // holds on that row (whole lanes; few waves have a fiber near, the others branch past).
    __device__ inline unsigned store_offset(int r) const {
        unsigned off = st;
        for (unsigned long long m = near; m != 0ull; m &= m - 1ull) {
            const PatchUnit u = load_unit(units, __builtin_ctzll(m));
            PlanPtr plan = unit_plan(u, slot);
            int d = r - plan[2];
            if (per && d < 0) d += ny;
            if ((unsigned)d >= (unsigned)plan[3]) continue;
            const int2 c = plan_row(u, plan, kPassSteps, d);
            int cl = x0 - plan[0];
            if (cl < 0) cl += nx;
            if (cl >= c.x && cl < c.y) off = kLaneOff;
        }
        return off;
    }
    // The units (bits) whose patch rectangle meets the wave's tile: lane i looks at unit i.
    // whole: the pass is a whole one (PatchUnit), in which the march does nothing.
    __device__ inline unsigned long long units_near(int n, int c0, int cols, bool& whole) const {
        const int lane = (int)threadIdx.x & 63;
        bool hit = false, all = false;
        if (lane < n) {
            const PatchUnit u = units[lane];
            const int* plan = u.plan + slot * u.plan_len;
            const int w = plan[1], h = plan[3], p0 = plan[2];
            all = plan[kPlanWhole] != 0;
            hit = w > 0 && h > 0 && cols_overlap(c0 % nx, min(cols, nx), plan[0], w, nx) &&
                  (per ? cols_overlap(y0, y1 - y0, p0, h, ny) : (y0 < p0 + h && p0 < y1));
        }
        whole = __ballot(all) != 0ull;
        return __ballot(hit);
    }
    __device__ inline int wrap(int y) const {
        if (per) {
            while (y < 0) y += ny;
            while (y >= ny) y -= ny;
        }
        return y;
    }
    // The nine direction rows that row y of the first stage pulls from, unshifted; a row
    // behind a wall is replaced by the reflected directions of the row itself.
    template <bool FAST> __device__ inline void fetch(int y, Row (&f)[9]) {
        const bool bot = !FAST && !per && y == 0, top = !FAST && !per && y == ny - 1;
        const int ym = FAST ? y - 1 : bot ? y : wrap(y - 1);
        const int yp = FAST ? y + 1 : top ? y : wrap(y + 1);
        const auto r0 = row_rsrc(row(FAST ? y : wrap(y)), rowb);
        const auto rm = row_rsrc(row(ym), rowb), rp = row_rsrc(row(yp), rowb);
        row_load(r0, ld, 0, f[0].w);
        row_load(r0, ld, planeb, f[1].w);
        row_load(r0, ld, 3 * planeb, f[3].w);
        row_load(rm, ld, (bot ? 4 : 2) * planeb, f[2].w);
        row_load(rm, ld, (bot ? 7 : 5) * planeb, f[5].w);
        row_load(rm, ld, (bot ? 8 : 6) * planeb, f[6].w);
        row_load(rp, ld, (top ? 2 : 4) * planeb, f[4].w);
        row_load(rp, ld, (top ? 5 : 7) * planeb, f[7].w);
        row_load(rp, ld, (top ? 6 : 8) * planeb, f[8].w);
    }
    // Pull, collide and encode one row: 0, 1, 3 from m, 2, 5, 6 from d, 4, 7, 8 from u.
    // bot, top: d, u hold the row's own reflected directions.
    __device__ inline void advance(const Row& m0, const Row& m1, const Row& m3, const Row& d2,
                                   const Row& d5, const Row& d6, const Row& u4, const Row& u7,
                                   const Row& u8, bool bot, bool top, Row (&p)[9]) {
        T g[9][C];
        m0.template pulled<0>(g[0]);
        m1.template pulled<1>(g[1]);
        m3.template pulled<-1>(g[3]);
        d2.template pulled<0>(g[2]);
        u4.template pulled<0>(g[4]);
        if (!bot) {
            d5.template pulled<1>(g[5]);
            d6.template pulled<-1>(g[6]);
        } else {
            d5.template pulled<0>(g[5]);
            d6.template pulled<0>(g[6]);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                g[5][i] -= u6;
                g[6][i] += u6;
            }
        }
        if (!top) {
            u7.template pulled<-1>(g[7]);
            u8.template pulled<1>(g[8]);
        } else {
            u7.template pulled<0>(g[7]);
            u8.template pulled<0>(g[8]);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                g[7][i] -= u6;
                g[8][i] += u6;
            }
        }
        T z[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            T n[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) n[k] = g[k][i];
            if constexpr (kScaled)
                z[i] = mrt_collide_scaled_open<T, FORCE>(n, Fx, Fy, s_nu, s_q, s_e, s_eps);
            else
                mrt_collide<T, FORCE>(n, Fx, Fy, s_nu, s_q, s_e, s_eps);
#pragma unroll
            for (int k = 0; k < 9; ++k) g[k][i] = n[k];
        }
        if constexpr (kScaled) {
#pragma unroll
            for (int i = 0; i < C; i += 2)
                p[0].w[i >> 1] = narrow_fma4(z[i], g[0][i], z[i + 1], g[0][i + 1]);
        } else {
            p[0].set(g[0]);
        }
#pragma unroll
        for (int k = 1; k < 9; ++k) p[k].set(g[k]);
    }
    // Row i of the first stage and, behind it, row i - (t - 1) of stage t; PH alternates
    // from row to row.  FAST: every stage has a row, none at a wall, and row i + 1 follows.
    template <bool FAST, int PH> __device__ inline void row_step(int i) {
        // (found before the row's work: few values are live here)
        unsigned off = st;
        if (near) off = store_offset(i - (NT - 1));
        Row p[9];
        if (FAST || i < hi1) {
            if (FAST || i + 1 < hi1) fetch<FAST>(i + 1, q[1 - PH]);
            Row(&c)[9] = q[PH];
            advance(c[0], c[1], c[3], c[2], c[5], c[6], c[4], c[7], c[8], !FAST && !per && i == 0,
                    !FAST && !per && i == ny - 1, p);
        }
#pragma unroll
        for (int t = 2; t <= NT; ++t) {
            Held& H = h[t - 2];
            Row(&up)[3] = H.up[PH];
            Row(&dn)[3] = H.up[1 - PH];
            const int r = i - (t - 1);
            Row n[9];
            if (FAST) {
                advance(H.mid[0], H.mid[1], H.mid[2], dn[0], dn[1], dn[2], p[4], p[7], p[8],
                        false, false, n);
            } else if (r >= lo(t) && r < hi(t)) {
                const bool top = !per && r == ny - 1;
                advance(H.mid[0], H.mid[1], H.mid[2], dn[0], dn[1], dn[2], top ? up[0] : p[4],
                        top ? up[1] : p[7], top ? up[2] : p[8], !per && r == 0, top, n);
            }
            if (!FAST && !per && r + 1 == 0) {  // stage t - 1 has just finished row 0
                up[0] = p[4];
                up[1] = p[7];
                up[2] = p[8];
            }
            dn[0] = p[2];
            dn[1] = p[5];
            dn[2] = p[6];
            H.mid[0] = p[0];
            H.mid[1] = p[1];
            H.mid[2] = p[3];
#pragma unroll
            for (int k = 0; k < 9; ++k) p[k] = n[k];
        }
        const int r = i - (NT - 1);
        if (FAST || (r >= y0 && r < y1)) {
            const auto o = row_rsrc(dst + (long long)r * rowb, rowb);
#pragma unroll
            for (int k = 0; k < 9; ++k) row_store(o, off, k * planeb, p[k].w);
        }
    }
    __device__ inline void run(const MarchArgs& a, int strip, int ya, int yb) {
        nx = a.L.nx;
        ny = a.L.ny;
        y0 = ya;
        y1 = yb;
        rowb = (unsigned)(a.L.stride * (int)sizeof(S));
        planeb = (unsigned)(a.L.plane * (int)sizeof(S));
        src = (const char*)a.src;
        dst = (char*)a.dst;
        const int lane = (int)threadIdx.x & 63;
        x0 = (strip * OL + lane - HL) * C;
        int xw = x0 % nx;
        if (xw < 0) xw += nx;
        ld = (unsigned)(xw * (int)sizeof(S));
        st = lane >= HL && lane < HL + OL && x0 < nx ? (unsigned)(x0 * (int)sizeof(S)) : kLaneOff;
        units = a.units;
        slot = a.slot;
        bool whole = false;
        near = a.n_units > 0 ? units_near(a.n_units, strip * OL * C, OL * C, whole) : 0ull;
        u6 = kScaled ? (T)(a.u6 * 16384.0) : (T)a.u6;
        s_nu = (T)a.s_nu;
        s_q = (T)a.s_q;
        s_e = (T)a.s_e;
        s_eps = (T)a.s_eps;
        Fx = (T)a.gx;
        Fy = (T)a.gy;
#pragma unroll
        for (int s = 0; s < NT - 1; ++s)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                h[s].mid[k] = Row{};
                h[s].up[0][k] = Row{};
                h[s].up[1][k] = Row{};
            }
        lo1 = lo(1);
        hi1 = hi(1);
        const int end = y1 + NT - 1;
        const int f0 = max(y0 + NT, 1);
        const int f1 = min(hi1, ny - 1) - 3;   // last pair start: i + 3 < hi1, row i + 3 exists
        fetch<false>(lo1, q[0]);
        if (whole) return;   // (behind the loads, which need not wait for it)
        int i = lo1;
        while (i < end) {
            row_step<false, 0>(i);
            row_step<false, 1>(i + 1);
            i += 2;
            if (i >= f0 && i < f1) {
                __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): nothing in flight at the loop's head
                do {
                    row_step<true, 0>(i);
                    row_step<true, 1>(i + 1);
                    i += 2;
                } while (i < f1);
            }
        }
    }
};

}  // namespace fpd
