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

// Waves of a march: two per SIMD of the device (1024 SIMDs), all resident at once, so none
// waits for another and the registers left take the patch and bead kernels beside them.
// Measured at 8192 x 2048 with the fiber (1024 / 1536 / 2048 / 3072 / 6144 waves): 65.3 /
// 76.8 / 66.1 / 71.7 / 74.7 us per step in float32, 188.9 / 171.8 / 138.9 / 145.6 / 151.6 in
// float64, 65.8 / 71.2 / 60.2 / 72.3 / 67.4 in bfloat16 deviations.  A wave recomputes up to
// kPassSteps - 1 rows on either side of its own, so small lattices take fewer, taller runs.
constexpr int kMarchWaves = 2048;
constexpr int kMarchMinRows = 16;

template <int ST, int C, int OL>
static hipError_t launch_march_t(const StepArgs& a, const int* part, hipStream_t st) {
    MarchArgs m{};
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
    m.part = part;
    m.strips = (a.L.nx + OL * C - 1) / (OL * C);
    const int segs = std::max(1, std::min(kMarchWaves / m.strips, a.L.ny / kMarchMinRows));
    m.seg_rows = (a.L.ny + segs - 1) / segs;
    m.segs = (a.L.ny + m.seg_rows - 1) / m.seg_rows;
    const bool force = a.gx != 0.0 || a.gy != 0.0, per = a.L.periodic != 0;
    void (*k)(MarchArgs) = nullptr;
    if (per)
        k = force ? march_kernel<ST, C, OL, 1, true> : march_kernel<ST, C, OL, 1, false>;
    else
        k = force ? march_kernel<ST, C, OL, 0, true> : march_kernel<ST, C, OL, 0, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)m.strips * m.segs), dim3(64), 0, st, m);
    return hipGetLastError();
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
hipError_t launch_march(int storage, const StepArgs& a, const int* part, hipStream_t st) {
    switch (storage) {
        case FPD_F64: return launch_march_t<FPD_F64, 1, 56>(a, part, st);
        case FPD_F32:
            return a.L.nx % 2 == 0 ? launch_march_t<FPD_F32, 2, 56>(a, part, st)
                                   : launch_march_t<FPD_F32, 1, 56>(a, part, st);
        case FPD_F16DEV: return launch_march_t<FPD_F16DEV, 2, 60>(a, part, st);
        case FPD_BF16DEV: return launch_march_t<FPD_BF16DEV, 2, 60>(a, part, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace fpd
