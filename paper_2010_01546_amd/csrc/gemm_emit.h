#pragma once
#include "fw_internal.h"

namespace fw {

// What the float32 kernels do with a finished element (row, col) of G Q, value v:
//   taps == 1: element index row * M + col.  taps > 1 (per-tap form): the product ran on rows (s, tap) of the permuted
//   gradient, and the element belongs at [s][col][tap] of an [S, M, taps] array (the layout of a convolution weight).
//   out (float32, or bfloat16 bits when out_bf16): the transformed gradient, written when non-null.
//   W (and V): the update  d = v + wd W;  V = momentum V + d (if V);  W -= lr (V or d)   (eq. (vtWrn_SGD)).
__device__ __forceinline__ size_t emit_index(const GemmEpilogue& e, int row, int col, int M) {
    if (e.taps <= 1) return (size_t)row * M + col;
    const int s = row / e.taps, t = row - s * e.taps;
    return ((size_t)s * M + col) * e.taps + t;
}
__device__ __forceinline__ void emit(const GemmEpilogue& e, int row, int col, int M, float v) {
    const size_t idx = emit_index(e, row, col, M);
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

// The update of N elements of a lane, element i at (row_of(i), col) where row_of(i) < S, no lane's row above that of a later lane: the old
// values of W and V are all asked for before the first new one is stored (a load behind a store waits for it, a round trip per
// element: 16 elements a lane, 767 x 68 bfloat16 gradient, 14.7 us one by one).
template <int N, class RowOf, class Values>
__device__ __forceinline__ void emit_update(const GemmEpilogue& e, const RowOf& row_of, int col, int S, int M, const Values& v) {
    float w[N], u[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int row = row_of(i);
        w[i] = u[i] = 0.f;
        if (__builtin_amdgcn_readfirstlane(row) >= S) continue;      // rows ascend with the lane
        const size_t idx = emit_index(e, row < S ? row : 0, col, M);
        w[i] = e.W[idx];
        if (e.V) u[i] = e.V[idx];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int row = row_of(i);
        if (row >= S) continue;
        const size_t idx = emit_index(e, row, col, M);
        float d = v[i] + e.wd * w[i];
        if (e.V) {
            d = e.momentum * u[i] + d;
            e.V[idx] = d;
        }
        e.W[idx] = w[i] - e.lr * d;
    }
}

}  // namespace fw
