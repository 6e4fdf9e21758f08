// fpd_march.hip -- the fluid part of a pass: kPassSteps time steps of every node outside the
// pass's partition in one kernel.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fpd_march.hpp"

namespace fpd {

template <int ST, int C, int OL, int BC, bool FORCE>
__global__ void __launch_bounds__(64) march_kernel(MarchArgs a) {
    const int strip = (int)blockIdx.x % a.strips, seg = (int)blockIdx.x / a.strips;
    const int y0 = seg * a.seg_rows, y1 = min(y0 + a.seg_rows, a.L.ny);
    March<ST, kPassSteps, C, OL, BC, FORCE> m;
    m.run(a, strip, y0, y1);
}

__host__ __device__ static inline MarchArgs march_args(const StepArgs& a,
                                                       const PatchUnit* units, int n_units,
                                                       int slot, int strips, int seg_rows) {
    MarchArgs m;
    m.src = a.src;
    m.dst = a.dst;
    m.L = a.L;
    m.u6 = a.u6;
    m.s_nu = a.s_nu_f;
    m.s_q = a.s_q_f;
    m.s_e = a.s_e;
    m.s_eps = a.s_eps;
    m.gx = a.gx;
    m.gy = a.gy;
    m.units = units;
    m.n_units = n_units;
    m.slot = slot;
    m.strips = strips;
    m.seg_rows = seg_rows;
    return m;
}

// One wave per (simulation, tile) item of a batch's marches of one kind.
template <int ST, int C, int OL, int BC, bool FORCE>
__global__ void __launch_bounds__(64) batch_march_kernel(BatchArgs b, int first) {
    const ItemRef e = item_ref(b.march_items, first + (int)blockIdx.x);
    if (first + (int)blockIdx.x >= b.counts[4] || e.sim < 0) return;
    const StepArgs s = load_args(b.args, 2 * e.sim + b.gpar);
    const PassSim p = load_pass(b.pass, e.sim);
    const MarchArgs a = march_args(s, p.units, p.n_units, b.gpar, p.strips, p.seg_rows);
    const int strip = e.local % a.strips, seg = e.local / a.strips;
    const int y0 = seg * a.seg_rows, y1 = min(y0 + a.seg_rows, a.L.ny);
    March<ST, kPassSteps, C, OL, BC, FORCE> m;
    m.run(a, strip, y0, y1);
}

// Waves of a march: two per SIMD of the device (1024 SIMDs), all resident at once, so none
// waits for another and the registers left take the patch and bead kernels beside them.
// Measured at 8192 x 2048 with the fiber (1024 / 1536 / 2048 / 3072 / 6144 waves): 65.3 /
// 76.8 / 66.1 / 71.7 / 74.7 us per step in float32, 188.9 / 171.8 / 138.9 / 145.6 / 151.6 in
// float64, 65.8 / 71.2 / 60.2 / 72.3 / 67.4 in bfloat16 deviations.  A wave recomputes up to
// kPassSteps - 1 rows on either side of its own, so small lattices take fewer, taller runs.
constexpr int kMarchWaves = 2048;
// Many fibers: their patch and bead blocks are everywhere, and the waves beside them end late.  A
// third wave per SIMD, in shorter runs of rows, evens that out.  8192 x 2048 with 25 fibers,
// 2048 / 3072 / 4096 waves, us per step: float32 97.7 / 86.5 / 87.6, float64 185 / 156 / 162,
// float16 94.9 / 73.8 / 77.3, bfloat16 91.0 / 74.2 / 76.3; 14 fibers, 2048 / 3072: float32
// 88.4 / 74.6, float64 176 / 160, float16 66.6 / 64.8; 8 fibers: 68.6 / 70.0, 170 / 157,
// 63.2 / 61.3, and 4096 x 1500 with 8: 31.1 / 39.2, 61.2 / 67.9, 30.0 / 31.3.
constexpr int kMarchWavesMany = 3072;
constexpr int kMarchManyUnits = 12;
constexpr int kMarchMinRows = 16;

template <int ST, int C, int OL>
static hipError_t launch_march_t(const StepArgs& a, const PassArgs& q, hipStream_t st,
                                 hipEvent_t t0, hipEvent_t t1) {
    const int strips = (a.L.nx + OL * C - 1) / (OL * C);
    const int waves = q.n_units >= kMarchManyUnits ? kMarchWavesMany : kMarchWaves;
    const int runs = std::max(1, std::min(waves / strips, a.L.ny / kMarchMinRows));
    const MarchArgs m = march_args(a, q.units, q.n_units, q.slot, strips,
                                   (a.L.ny + runs - 1) / runs);
    const int segs = (a.L.ny + m.seg_rows - 1) / m.seg_rows;
    const bool force = a.gx != 0.0 || a.gy != 0.0, per = a.L.periodic != 0;
    void (*k)(MarchArgs) = nullptr;
    if (per)
        k = force ? march_kernel<ST, C, OL, 1, true> : march_kernel<ST, C, OL, 1, false>;
    else
        k = force ? march_kernel<ST, C, OL, 0, true> : march_kernel<ST, C, OL, 0, false>;
    return launch_k(k, dim3((unsigned)strips * segs), dim3(64), st, t0, t1, m);
}

bool march_ok(int storage, const Lattice& L) {
    const long long elem = storage == FPD_F64 ? 8 : storage == FPD_F32 ? 4 : 2;
    if ((long long)L.stride * elem >= 0x7fffffffLL) return false;  // a row is one buffer resource
    return storage == FPD_F64 || storage == FPD_F32 || L.nx % 2 == 0;
}

// Columns a lane holds (C) and lanes of a wave that store (OL).  A row of a wave is stored
// in runs of OL * C values: multiples of 64 bytes (448 in float32 and float64) were 12 %
// faster at 8192 x 2048 than 480 bytes, whose ends are written as 32-byte halves of a line
// (float32, one wave per strip: 65.3 against 73.6 us per step); the two-byte formats lose more
// to idle lanes than to the ends (240 bytes 56.7, 224 bytes 62.1).  Two columns of
// float32 and of the two-byte formats, or one of float64, fit three waves per SIMD.
// Four columns of float32 (320 registers, one wave per SIMD) took 67.0, four of float16 65.1.
hipError_t launch_march(int storage, const StepArgs& a, const PassArgs& q, hipStream_t st,
                        hipEvent_t t0, hipEvent_t t1) {
    switch (storage) {
        case FPD_F64: return launch_march_t<FPD_F64, 1, 56>(a, q, st, t0, t1);
        case FPD_F32:
            return a.L.nx % 2 == 0 ? launch_march_t<FPD_F32, 2, 56>(a, q, st, t0, t1)
                                   : launch_march_t<FPD_F32, 1, 56>(a, q, st, t0, t1);
        case FPD_F16DEV: return launch_march_t<FPD_F16DEV, 2, 60>(a, q, st, t0, t1);
        case FPD_BF16DEV: return launch_march_t<FPD_BF16DEV, 2, 60>(a, q, st, t0, t1);
    }
    return hipErrorInvalidValue;
}

int march_kind(int storage, const Lattice& L, bool force) {
    return (force ? kMarchForce : 0) | (L.periodic ? kMarchPeriodic : 0) |
           (storage == FPD_F32 && L.nx % 2 ? kMarchNarrow : 0);
}

int march_cols(int storage, const Lattice& L) {
    if (storage == FPD_F64) return 56;
    if (storage == FPD_F32) return L.nx % 2 ? 56 : 112;
    return 120;
}

template <int ST, int C, int OL>
static hipError_t launch_batch_march_t(const BatchArgs& b, int kind, int first, int n,
                                       hipStream_t st) {
    void (*k)(BatchArgs, int) = nullptr;
    switch (kind & (kMarchForce | kMarchPeriodic)) {
        case 0: k = batch_march_kernel<ST, C, OL, 0, false>; break;
        case kMarchForce: k = batch_march_kernel<ST, C, OL, 0, true>; break;
        case kMarchPeriodic: k = batch_march_kernel<ST, C, OL, 1, false>; break;
        default: k = batch_march_kernel<ST, C, OL, 1, true>; break;
    }
    hipLaunchKernelGGL(k, dim3(n), dim3(64), 0, st, b, first);
    return hipGetLastError();
}

hipError_t launch_batch_march(int storage, const BatchArgs& b, const int kind_count[kMarchKinds],
                              hipStream_t st) {
    int first = 0;
    for (int kind = 0; kind < kMarchKinds; ++kind) {
        const int n = kind_count[kind];
        if (n <= 0) continue;
        hipError_t e = hipErrorInvalidValue;
        switch (storage) {
            case FPD_F64: e = launch_batch_march_t<FPD_F64, 1, 56>(b, kind, first, n, st); break;
            case FPD_F32:
                e = kind & kMarchNarrow ? launch_batch_march_t<FPD_F32, 1, 56>(b, kind, first, n, st)
                                        : launch_batch_march_t<FPD_F32, 2, 56>(b, kind, first, n, st);
                break;
            case FPD_F16DEV: e = launch_batch_march_t<FPD_F16DEV, 2, 60>(b, kind, first, n, st); break;
            case FPD_BF16DEV: e = launch_batch_march_t<FPD_BF16DEV, 2, 60>(b, kind, first, n, st); break;
        }
        if (e != hipSuccess) return e;
        first += n;
    }
    return hipSuccess;
}

}  // namespace fpd
