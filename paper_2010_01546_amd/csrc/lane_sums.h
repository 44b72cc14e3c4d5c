// Sums of float64 values over the lanes of a wavefront on the vector pipe alone.  Several values at a time: each fold adds the halves
// of two of them into one register, so that N values take about N additions instead of 6 N.
#pragma once
#include "fw_internal.h"

namespace fw {

// x' + y' of the pair after lanes 32..63 of x changed places with lanes 0..31 of y: lanes below 32 hold the sum of x's halves, the others y's
__device__ __forceinline__ double fold32(double x, double y) {
    union { double d; unsigned i[2]; } a, b;
    a.d = x; b.d = y;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(a.i[k], b.i[k], false, false);
        a.i[k] = r[0]; b.i[k] = r[1];
    }
    return a.d + b.d;
}
// the same for the odd rows of 16 lanes of x and the even ones of y
__device__ __forceinline__ double fold16(double x, double y) {
    union { double d; unsigned i[2]; } a, b;
    a.d = x; b.d = y;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane16_swap(a.i[k], b.i[k], false, false);
        a.i[k] = r[0]; b.i[k] = r[1];
    }
    return a.d + b.d;
}
// sum over the 16 lanes of a row, in every one of them
__device__ __forceinline__ double sum16(double v) {
    union { double d; int i[2]; } a, b;
    a.d = v;
#define FW_SUM16(c) b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], c, 0xf, 0xf, true); b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], c, 0xf, 0xf, true); a.d += b.d
    FW_SUM16(0xB1);      // lanes 1,0,3,2
    FW_SUM16(0x4E);      // lanes 2,3,0,1
    FW_SUM16(0x141);     // half of 16 mirrored
    FW_SUM16(0x140);     // 16 mirrored
#undef FW_SUM16
    return a.d;
}

}  // namespace fw
