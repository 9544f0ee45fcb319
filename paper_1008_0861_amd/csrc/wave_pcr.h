// The in-wave part of the interface reduction: cyclic tridiagonal systems
// with unit diagonal, Ra X_{j-s} + X_j + Rc X_{j+s} = Rd, one row per lane,
// reduced by parallel cyclic reduction (each step doubles the stride s).
//
// Lane order.  A 64-row system sits on the wave with row j in lane
// (j & 3) * 16 + (j >> 2): after the strides 1 and 2 it has split into four
// independent 16-row systems, each in one DPP row of 16 lanes, whose
// strides 1, 2, 4, 8 are row rotations (register moves; a ds_bpermute
// exchange of the six values costs about 330 cycles of latency per step in
// FP32 and twice the LDS instructions in FP64).
//
// Early end.  The couplings square with every step (they decay like
// rho^(cells between the unknowns)), so at the step sizes in use most of
// the later steps add nothing: once every |Ra|, |Rc| of the wave is below
// eps^2 a further step changes no X by more than eps^2 max|X|.  The test
// also asks for a finite right-hand side: a NaN or infinity takes all steps
// and spreads over the whole line, as it does without the test.  The first
// steps (which never suffice) run without a test.
#pragma once

#include "asd_device.h"

namespace asd {

// (one comparison: a NaN coupling and, through Rd * 0, a non-finite
// right-hand side fail it)
template <typename T>
__device__ __forceinline__ bool pcr_done(T Ra, T Rc, T Rd) {
    constexpr T tol = sizeof(T) == 4 ? T(0x1p-48) : T(0x1p-106);
    const bool small = fma(Rd, T(0), fabs(Ra) + fabs(Rc)) < tol;
    return __builtin_amdgcn_ballot_w64(small) == __builtin_amdgcn_ballot_w64(true);
}

// One step: rows m and p are the partners at -s and +s.
template <typename T>
__device__ __forceinline__ void pcr_combine(T& Ra, T& Rc, T& Rd, T am, T cm, T dm, T ap, T cp, T dp) {
    const T ib = fast_rcp<T>(T(1) - Ra * cm - Rc * ap);
    const T na = -Ra * am, nc = -Rc * cp, nd = Rd - Ra * dm - Rc * dp;
    Ra = na * ib;
    Rc = nc * ib;
    Rd = nd * ib;
}
template <typename T>
__device__ __forceinline__ void pcr_shfl_step(T& Ra, T& Rc, T& Rd, int lm, int lp) {
    const T am = __shfl(Ra, lm, 64), cm = __shfl(Rc, lm, 64), dm = __shfl(Rd, lm, 64);
    const T ap = __shfl(Ra, lp, 64), cp = __shfl(Rc, lp, 64), dp = __shfl(Rd, lp, 64);
    pcr_combine<T>(Ra, Rc, Rd, am, cm, dm, ap, cp, dp);
}

// lane i takes v of lane i - S (mod 16) of its row of 16 lanes
template <int S, typename T>
__device__ __forceinline__ T row_from(T v) {
    return dpp_mov<0x120 + S, 0xf>(v, v);
}
template <int S, typename T>
__device__ __forceinline__ void pcr_row_step(T& Ra, T& Rc, T& Rd) {
    const T am = row_from<S>(Ra), cm = row_from<S>(Rc), dm = row_from<S>(Rd);
    const T ap = row_from<16 - S>(Ra), cp = row_from<16 - S>(Rc), dp = row_from<16 - S>(Rd);
    pcr_combine<T>(Ra, Rc, Rd, am, cm, dm, ap, cp, dp);
}

// Row j of a 64-row system <-> its lane.
__device__ __forceinline__ int row_of_lane(int lane) { return ((lane & 15) << 2) | (lane >> 4); }
__device__ __forceinline__ int lane_of_row(int j) { return ((j & 3) << 4) | ((j >> 2) & 15); }

// One 64-row system per wave in that lane order (j = row_of_lane(lane)).
template <typename T>
__device__ __forceinline__ void pcr_wave64(int j, T& Ra, T& Rc, T& Rd) {
    pcr_shfl_step<T>(Ra, Rc, Rd, lane_of_row(j - 1), lane_of_row(j + 1));
    pcr_shfl_step<T>(Ra, Rc, Rd, lane_of_row(j - 2), lane_of_row(j + 2));
    if (pcr_done<T>(Ra, Rc, Rd)) return;
    pcr_row_step<1>(Ra, Rc, Rd);
    if (pcr_done<T>(Ra, Rc, Rd)) return;
    pcr_row_step<2>(Ra, Rc, Rd);
    if (pcr_done<T>(Ra, Rc, Rd)) return;
    pcr_row_step<4>(Ra, Rc, Rd);
    if (pcr_done<T>(Ra, Rc, Rd)) return;
    pcr_row_step<8>(Ra, Rc, Rd);
}

// nl rows (a power of two, at most LPL) in the first lanes of each group of
// LPL lanes (a line's), row j in lane j of the group; the lanes after them
// combine rows too, unused.  Every lane must call it.  (No early end here: in
// this rolled loop the tests cost 129^2 FP64 with walls at ncfl 1000, where they
// never hold, 4.7 %, and gained ragged FP32 lines at ncfl 10 nothing.  A whole
// wave per line needs no group base: with one in a register the FP64 sweep of 8
// cells per lane with walls takes 129 of them, one more than four waves per SIMD
// leave it.)
template <typename T, int LPL>
__device__ __forceinline__ void pcr_lanes(int lane, int nl, T& Ra, T& Rc, T& Rd) {
    const int base = LPL == 64 ? 0 : lane & ~(LPL - 1);
    for (int s = 1; s < nl; s <<= 1)
        pcr_shfl_step<T>(Ra, Rc, Rd, base | ((lane - s) & (nl - 1)), base | ((lane + s) & (nl - 1)));
}

}  // namespace asd
