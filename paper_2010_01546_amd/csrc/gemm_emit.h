#pragma once
#include "fw_internal.h"

namespace fw {

// What the float32 kernels do with a finished element (row, col) of G Q, value v:
//   taps == 1: element index row * M + col.  taps > 1 (per-tap form): the product ran on rows (s, tap) of the permuted
//   gradient, and the element belongs at [s][col][tap] of an [S, M, taps] array (the layout of a convolution weight).
//   out (float32, or bfloat16 bits when out_bf16): the transformed gradient, written when non-null.
//   W (and V): the update  d = v + wd W;  V = momentum V + d (if V);  W -= lr (V or d)   (eq. (vtWrn_SGD)).
__device__ __forceinline__ void emit(const GemmEpilogue& e, int row, int col, int M, float v) {
    size_t idx;
    if (e.taps > 1) {
        const int s = row / e.taps, t = row - s * e.taps;
        idx = ((size_t)s * M + col) * e.taps + t;
    } else {
        idx = (size_t)row * M + col;
    }
    if (e.out) {
        if (e.out_bf16) reinterpret_cast<unsigned short*>(e.out)[idx] = f32_to_bf16_rne(v);
        else reinterpret_cast<float*>(e.out)[idx] = v;
    }
    if (e.W) {
        const float w = e.W[idx];
        float d = v + e.wd * w;
        if (e.V) {
            d = e.momentum * e.V[idx] + d;
            e.V[idx] = d;
        }
        e.W[idx] = w - e.lr * d;
    }
}

}  // namespace fw
