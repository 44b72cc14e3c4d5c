// Recursive condition-number reduction (Sec. 4) for gfx950: one step is a chain of bandwidth-bound passes over
// M x M float32 matrices.
//
//   estimate (Sec. 4.2):  m' = argmax xi   ->  c = Phi_y Phi_y e_m'  ->  coherence set, weights w  ->
//                         v~ = Phi_y w  ->  v = v~/|v~|   [optional refinements v <- Phi_y v / |Phi_y v|]
//   step (Sec. 4.1):      u = Phi_y v, lambda_e = v^T u, g_e, a_e;  t = T^T v;  p = Phi_x t = Psi^T v (only if gamma < 1)
//   The small reductions in between (arg-max, size of the set, |v~|) are done by every workgroup of the pass that
//   needs them, for itself, from vectors of M entries, so that a step is six launches, four of which touch M x M data:
//   c | v~ | u and the partial products of t and p | t, p and the scalars | update | squared row norms.
//   p = Phi_x T^T v is taken as Psi^T v (Psi = T Phi_x is part of the state): all three products of the third launch
//   then need nothing but v, and no pass has to wait for t.
//   update, one fused pass over pairs of mirrored 32x32 tiles:
//       T'     = gamma (T + a v t^T) + (1-gamma) I                                               eq. (vT_rec)
//       Q'     = gamma^2 (Q + a(a+2) t t^T) + (1-gamma)^2 I
//                + gamma(1-gamma) (a (v t^T + t v^T) + T + T^T)                                  eq. (vQ_rec)
//       Qs'    = beta Qs + (1-beta) Q'                                                           eq. (vQs)
//       Phi_y' = gamma^2 (Phi_y + a (v u^T + u v^T) + a^2 lambda_e v v^T)
//                + gamma(1-gamma) (Psi + Psi^T + a (v p^T + p v^T)) + (1-gamma)^2 Phi_x          (= T' Phi_x T'^T)
//       Psi'   = gamma (Psi + a v p^T) + (1-gamma) Phi_x                                         (= T' Phi_x)
//     and the squared row norms of Phi_y' for the next step's arg-max.
// t = T^T v (the transposed reading of eq. (vtve)) is what makes T' equal gamma T~ T + (1-gamma) I.
// Matrix-vector products use one wavefront per row with a 64-lane shuffle reduction.
#include "fw_internal.h"
#include <mutex>

// Scratch of the allocation-free variant of the step (fw_cond_reduce_step_static): the workspace of one step for
// M <= 4608, held by every GPU the library runs on until the process ends.  In host code this name is only a handle
// for hipGetSymbolAddress; the address kernels are given comes from static_scratch() below.
static __device__ __align__(256) unsigned char scratch[6u << 20];

namespace fw {
namespace {

struct Scal {
    int m_prime, set_size, flags;
    float xi_mp, lambda_e, a_e, vnorm;
};

constexpr int TILE = 32;
constexpr int VM_ROWS_MIN = 16;  // fewest rows a workgroup takes in the T^T v partial products

struct WsLayout {
    size_t c, w, vt, v, u, t, p, tpart, ppart, xpart, scal, total;
    int Mp, nrb, vm_rows, nt;
};
inline WsLayout ws_layout(int M) {
    WsLayout L;
    L.Mp = (M + 63) / 64 * 64;
    // rows per workgroup of the T^T v pass: about 1024 workgroups in all, a multiple of 16 rows, at least 16
    {
        const long long colblocks = (M + 255) / 256;
        long long rows = ((long long)M * colblocks + 1023) / 1024;
        rows = (rows + VM_ROWS_MIN - 1) / VM_ROWS_MIN * VM_ROWS_MIN;
        L.vm_rows = (int)rows;
    }
    L.nrb = (M + L.vm_rows - 1) / L.vm_rows;
    L.nt = (M + TILE - 1) / TILE;
    size_t o = 0;
    auto take = [&](size_t floats) { size_t at = o; o += align_up(floats * sizeof(float), 256); return at; };
    L.c = take(L.Mp); L.w = take(L.Mp); L.vt = take(L.Mp); L.v = take(L.Mp); L.u = take(L.Mp); L.t = take(L.Mp); L.p = take(L.Mp);
    L.tpart = take((size_t)L.nrb * L.Mp);
    L.ppart = take((size_t)L.nrb * L.Mp);
    L.xpart = take((size_t)L.nt * L.Mp);
    L.scal = take(64);
    L.total = o;
    return L;
}

// sum over the wavefront, the same value in every lane, on the vector pipe alone (no LDS permutes: a tenth of their latency)
__device__ __forceinline__ float wave_sum_dpp(float v) {
#define FW_DPP_ADD(ctrl) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true))
    FW_DPP_ADD(0xB1);     // lanes 1,0,3,2
    FW_DPP_ADD(0x4E);     // lanes 2,3,0,1
    FW_DPP_ADD(0x141);    // half of 16 mirrored
    FW_DPP_ADD(0x140);    // 16 mirrored: every lane has the sum of its 16
#undef FW_DPP_ADD
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ float wave_max_dpp(float v) {
#define FW_DPP_MAX(ctrl) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true)))
    FW_DPP_MAX(0xB1); FW_DPP_MAX(0x4E); FW_DPP_MAX(0x141); FW_DPP_MAX(0x140);     // the moves of wave_sum_dpp
#undef FW_DPP_MAX
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

__device__ __forceinline__ int wave_min_dpp(int v) {
#define FW_DPP_MIN(ctrl) v = min(v, __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, true))
    FW_DPP_MIN(0xB1); FW_DPP_MIN(0x4E); FW_DPP_MIN(0x141); FW_DPP_MIN(0x140);
#undef FW_DPP_MIN
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// sum over the workgroup, the same value in every thread
__device__ __forceinline__ float block_sum(float v, float* red) {
    v = wave_sum_dpp(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
    return t;
}

// m' = argmax_m xi2[m], lowest index on ties (eq. (mt)), computed by a whole workgroup of 256 threads; every
// workgroup that calls it gets the same answer
__device__ __forceinline__ void block_argmax(const float* __restrict__ xi2, int M, float* bv, int* bi, float* best_out, int* idx_out) {
    float best = -1.f;
    int idx = 0x7fffffff;
    // ascending scan per thread with a strict comparison keeps the lowest index; four 16-byte loads in flight
    if ((M & 3) == 0) {
        const float4* x4 = reinterpret_cast<const float4*>(xi2);
        const int n4 = M >> 2, nt = blockDim.x;
        for (int k = threadIdx.x; k < n4; k += 4 * nt) {
            float4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = (k + j * nt < n4) ? x4[k + j * nt] : make_float4(-1.f, -1.f, -1.f, -1.f);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = 4 * (k + j * nt);
                if (q[j].x > best) { best = q[j].x; idx = m; }
                if (q[j].y > best) { best = q[j].y; idx = m + 1; }
                if (q[j].z > best) { best = q[j].z; idx = m + 2; }
                if (q[j].w > best) { best = q[j].w; idx = m + 3; }
            }
        }
    } else {
        for (int m = threadIdx.x; m < M; m += blockDim.x) {
            const float v = xi2[m];
            if (v > best) { best = v; idx = m; }
        }
    }
    const float top = wave_max_dpp(best);
    idx = wave_min_dpp(best == top ? idx : 0x7fffffff);
    best = top;
    if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = idx; }
    __syncthreads();
    best = bv[0]; idx = bi[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i)
        if (bv[i] > best || (bv[i] == best && bi[i] < idx)) { best = bv[i]; idx = bi[i]; }
    if (idx < 0 || idx >= M) idx = 0;  // every norm was NaN: keep the index in range
    *best_out = best; *idx_out = idx;
}

// dot product of a row of P with x (global memory or LDS), one wavefront per row, four 16-byte loads of the row in flight
__device__ __forceinline__ float row_dot(const float* __restrict__ row, const float* __restrict__ x, int M, int lane) {
    float acc = 0.f;
    if ((M & 3) == 0) {
        const float4* r4 = reinterpret_cast<const float4*>(row);
        const float4* x4 = reinterpret_cast<const float4*>(x);
        const int n4 = M >> 2;
        int k = lane;
        for (; k + 192 < n4; k += 256) {
            float4 a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { a[j] = r4[k + 64 * j]; b[j] = x4[k + 64 * j]; }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc += a[j].x * b[j].x + a[j].y * b[j].y + a[j].z * b[j].z + a[j].w * b[j].w;
        }
        for (; k < n4; k += 64) {
            const float4 a = r4[k], b = x4[k];
            acc += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
        }
    } else {
        for (int k = lane; k < M; k += 64) acc += row[k] * x[k];
    }
    return wave_sum_dpp(acc);
}

// The first four 16-byte loads of a row, issued before a workgroup's preparation (arg-max, weights, norm) so that the
// memory pipe is already busy while the small reductions run; row_dot_pref consumes them and continues like row_dot.
struct RowPref { float4 a[4]; };
__device__ __forceinline__ void row_prefetch(const float* __restrict__ row, int M, int lane, RowPref& p) {
    if ((M & 3) != 0) return;
    const float4* r4 = reinterpret_cast<const float4*>(row);
    const int n4 = M >> 2;
#pragma unroll
    for (int j = 0; j < 4; ++j) p.a[j] = r4[lane + 64 * j < n4 ? lane + 64 * j : 0];
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(p.a[j].x), "+v"(p.a[j].y), "+v"(p.a[j].z), "+v"(p.a[j].w));   // issued here, not later
}
__device__ __forceinline__ float row_dot_pref(const float* __restrict__ row, const float* __restrict__ x, int M, int lane, const RowPref& p) {
    if ((M & 3) != 0) return row_dot(row, x, M, lane);
    const float4* r4 = reinterpret_cast<const float4*>(row);
    const float4* x4 = reinterpret_cast<const float4*>(x);
    const int n4 = M >> 2;
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (lane + 64 * j < n4) {
            const float4 a = p.a[j], b = x4[lane + 64 * j];
            acc += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
        }
    int k = lane + 256;
    for (; k + 192 < n4; k += 256) {
        float4 a[4], b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { a[j] = r4[k + 64 * j]; b[j] = x4[k + 64 * j]; }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += a[j].x * b[j].x + a[j].y * b[j].y + a[j].z * b[j].z + a[j].w * b[j].w;
    }
    for (; k < n4; k += 64) {
        const float4 a = r4[k], b = x4[k];
        acc += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
    }
    return wave_sum_dpp(acc);
}

// c = Phi_y (Phi_y e_m') (eq. (vc)) with the arg-max of eq. (mt) found by every workgroup for itself; four rows per
// workgroup, one wavefront each.  Workgroup 0 records m' and xi_m'.
__global__ __launch_bounds__(256) void matvec_c_kernel(const float* __restrict__ P, const float* __restrict__ xi2, int M,
                                                       Scal* __restrict__ sc, float* __restrict__ c) {
    __shared__ float bv[4];
    __shared__ int bi[4];
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    RowPref pre;
    row_prefetch(P + (size_t)(r < M ? r : 0) * M, M, lane, pre);
    float best; int mp;
    block_argmax(xi2, M, bv, bi, &best, &mp);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->m_prime = mp;
        sc->xi_mp = sqrtf(fmaxf(best, 0.f));
        sc->flags = 0;
    }
    if (r >= M) return;
    const float acc = row_dot_pref(P + (size_t)r * M, P + (size_t)mp * M, M, lane, pre);
    if (lane == 0) c[r] = acc;
}

// v~ = Phi_y w (first line of eq. (tve)) with the coherence set and the alignment weights w_m = 1/(|set| c_m) on the
// set, 0 elsewhere (rule after eq. (vc)) formed on the fly: every workgroup counts the set for itself.
__global__ __launch_bounds__(256) void matvec_vt_kernel(const float* __restrict__ P, const float* __restrict__ c,
                                                        const float* __restrict__ xi2, int M, float c_rel, float c_abs,
                                                        Scal* __restrict__ sc, float* __restrict__ vt) {
    extern __shared__ __attribute__((aligned(16))) float wl[];   // M weights
    __shared__ float red[4];
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    RowPref pre;
    row_prefetch(P + (size_t)(r < M ? r : 0) * M, M, lane, pre);
    const float xi_mp = sc->xi_mp;
    // first pass: c_m on the set and 0 elsewhere into LDS, and the size of the set
    float cnt = 0.f;
    auto weight = [&](float cm, float x2) {
        const float thr = fmaxf(c_rel * xi_mp * sqrtf(fmaxf(x2, 0.f)), c_abs);
        const bool in = fabsf(cm) >= thr;
        cnt += in ? 1.f : 0.f;
        return in ? cm : 0.f;
    };
    if ((M & 3) == 0) {
        const float4* c4 = reinterpret_cast<const float4*>(c);
        const float4* x4 = reinterpret_cast<const float4*>(xi2);
        float4* w4 = reinterpret_cast<float4*>(wl);
        const int n4 = M >> 2, nt = blockDim.x;
        for (int k = threadIdx.x; k < n4; k += 2 * nt) {
            const bool two = k + nt < n4;
            const float4 ca = c4[k], xa = x4[k];
            const float4 cb = two ? c4[k + nt] : ca, xb = two ? x4[k + nt] : xa;
            w4[k] = make_float4(weight(ca.x, xa.x), weight(ca.y, xa.y), weight(ca.z, xa.z), weight(ca.w, xa.w));
            if (two) w4[k + nt] = make_float4(weight(cb.x, xb.x), weight(cb.y, xb.y), weight(cb.z, xb.z), weight(cb.w, xb.w));
        }
    } else {
        for (int m = threadIdx.x; m < M; m += blockDim.x) wl[m] = weight(c[m], xi2[m]);
    }
    const float total = block_sum(cnt, red);   // has the barriers that publish wl
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->set_size = (int)total;
        if (total == 0.f) sc->flags |= 1;
    }
    // second pass over LDS: w_m = 1/(|set| c_m) on the set
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
        const float cm = wl[m];
        wl[m] = cm != 0.f ? 1.f / (total * cm) : 0.f;
    }
    __syncthreads();
    if (r >= M) return;
    const float acc = row_dot_pref(P + (size_t)r * M, wl, M, lane, pre);
    if (lane == 0) vt[r] = acc;
}

// |v~| by a whole workgroup (the same value in every workgroup) and the factor that normalises it (second line of
// eq. (tve)); an empty set gives v = 0
__device__ __forceinline__ float block_inv_norm(const float* __restrict__ vt, int M, const Scal* __restrict__ sc, float* red, float* nrm_out) {
    float ss = 0.f;
    if ((M & 3) == 0) {
        const float4* v4 = reinterpret_cast<const float4*>(vt);
        const int n4 = M >> 2, nt = blockDim.x;
        for (int k = threadIdx.x; k < n4; k += 4 * nt) {
            float4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = (k + j * nt < n4) ? v4[k + j * nt] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int j = 0; j < 4; ++j) ss += q[j].x * q[j].x + q[j].y * q[j].y + q[j].z * q[j].z + q[j].w * q[j].w;
        }
    } else {
        for (int m = threadIdx.x; m < M; m += blockDim.x) ss += vt[m] * vt[m];
    }
    const float nrm = sqrtf(block_sum(ss, red));
    *nrm_out = nrm;
    return (nrm > 0.f && (sc->flags & 1) == 0) ? 1.f / nrm : 0.f;
}

// One refinement v <- Phi_y v / |Phi_y v| in unnormalised form: out = Phi_y (v~ / |v~|)
__global__ __launch_bounds__(256) void matvec_refine_kernel(const float* __restrict__ P, const float* __restrict__ vt, int M,
                                                            const Scal* __restrict__ sc, float* __restrict__ out) {
    __shared__ float red[4];
    float nrm;
    const float inv = block_inv_norm(vt, M, sc, red, &nrm);
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    const float acc = row_dot(P + (size_t)r * M, vt, M, lane) * inv;
    if (lane == 0) out[r] = acc;
}

// v = v~/|v~|, u = Phi_y v (workgroups below nmv: four rows each) and the partial products of t = T^T v and, with leak,
// p = Psi^T v over bands of vm_rows rows, tpart[band][j] = sum_{i in band} T[i][j] v[i] (the other workgroups: first
// those of T, then those of Psi), in one launch.
__global__ __launch_bounds__(256) void matvec_u_vecmat_kernel(const float* __restrict__ P, const float* __restrict__ T,
                                                              const float* __restrict__ Psi,
                                                              const float* __restrict__ vt, int M, int Mp, int vm_rows, int nmv, int nvm,
                                                              Scal* __restrict__ sc, float* __restrict__ v, float* __restrict__ u,
                                                              float* __restrict__ tpart, float* __restrict__ ppart) {
    __shared__ float red[4];
    float nrm;
    RowPref pre;
    const int ur = blockIdx.x * 4 + (threadIdx.x >> 6);
    if ((int)blockIdx.x < nmv) row_prefetch(P + (size_t)(ur < M ? ur : 0) * M, M, threadIdx.x & 63, pre);
    const float inv = block_inv_norm(vt, M, sc, red, &nrm);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->vnorm = nrm;
        if (!(nrm == nrm) || nrm > 3.0e38f) sc->flags |= 4;
    }
    if ((int)blockIdx.x < nmv) {
        const int lane = threadIdx.x & 63;
        const int r = ur;
        if (r >= M) return;
        const float acc = row_dot_pref(P + (size_t)r * M, vt, M, lane, pre) * inv;
        if (lane == 0) { u[r] = acc; v[r] = vt[r] * inv; }
        return;
    }
    const int ncol = (M + 255) / 256;
    int b = (int)blockIdx.x - nmv;
    if (b >= nvm) {        // the second set of bands multiplies Psi
        b -= nvm;
        T = Psi;
        tpart = ppart;
    }
    const int j = (b % ncol) * 256 + threadIdx.x;
    const int band = b / ncol;
    const int i0 = band * vm_rows;
    const int i1 = min(M, i0 + vm_rows);
    if (j >= M) return;
    float acc = 0.f;
    int i = i0;
    for (; i + 8 <= i1; i += 8) {
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = T[(size_t)(i + q) * M + j];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += x[q] * vt[i + q];
    }
    for (; i < i1; ++i) acc += T[(size_t)i * M + j] * vt[i];
    tpart[(size_t)band * Mp + j] = acc * inv;
}

// out[m] = sum over b < nparts of part[b][m]: 16 entries per workgroup, the parts dealt to sixteen groups of threads
// (eight loads in flight each) in a fixed order and combined through LDS
__device__ __forceinline__ void partial_sum_block(const float* __restrict__ part, int nparts, int M, int Mp, int blk, float* __restrict__ out,
                                                  float (*red)[16]) {
    const int e = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int m = blk * 16 + e;
    float acc = 0.f;
    if (m < M) {
        int b = grp;
        for (; b + 7 * 16 < nparts; b += 8 * 16) {
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = part[(size_t)(b + 16 * q) * Mp + m];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc += x[q];
        }
        for (; b < nparts; b += 16) acc += part[(size_t)b * Mp + m];
    }
    red[grp][e] = acc;
    __syncthreads();
    if (grp == 0 && m < M) {
        float t = 0.f;
#pragma unroll
        for (int g = 0; g < 16; ++g) t += red[g][e];
        out[m] = t;
    }
}

// squared row norms of the new Phi_y from the partial sums of the update pass
__global__ __launch_bounds__(256) void partial_sum_kernel(const float* __restrict__ part, int nparts, int M, int Mp, float* __restrict__ out) {
    __shared__ float red[16][16];
    partial_sum_block(part, nparts, M, Mp, blockIdx.x, out, red);
}

// lambda_e = v^T u (eq. (lambda)), g_e, a_e (eqs. (ge), (xi)), the guard and, where `record`, the diagnostics, by a whole workgroup: the
// same in every workgroup that calls it
__device__ __forceinline__ void step_scalars(const float* __restrict__ v, const float* __restrict__ u, int M, float* red,
                                             const float* __restrict__ lambda_bar, const fw_cond_params& prm, Scal* __restrict__ sc,
                                             fw_cond_info* __restrict__ info, bool record, float* a_out, float* lam_out) {
    float dot = 0.f;
    for (int m = threadIdx.x; m < M; m += blockDim.x) dot += v[m] * u[m];
    const float lam_e = block_sum(dot, red);
    int flags = sc->flags;
    float g_e = 1.f, a_e = 0.f;
    int applied = 0;
    if ((flags & 1) == 0) {
        g_e = prm.delta * (*lambda_bar) / fmaxf(lam_e, prm.eps);
        if (prm.guard && g_e >= 1.f) flags |= 2;
        else if (!(g_e == g_e) || g_e > 3.0e38f) flags |= 4;
        else { a_e = sqrtf(g_e) - 1.f; applied = 1; }
    }
    const float lam = (flags & 1) ? 0.f : lam_e;
    if (a_out) { *a_out = a_e; *lam_out = lam; }
    if (!record || threadIdx.x != 0) return;
    if (!a_out) { sc->lambda_e = lam; sc->a_e = a_e; }          // for the launch that follows
    if (info) {
        info->lambda_e = lam; info->g_e = g_e; info->a_e = a_e; info->v_norm = sc->vnorm;
        info->m_prime = sc->m_prime; info->set_size = sc->set_size; info->applied = applied; info->flags = flags;
    }
}

// t = T^T v (workgroups below nred) and p = Psi^T v (the next nred, with leak) from their partial products, and in the
// last workgroup lambda_e = v^T u (eq. (lambda)), g_e, a_e (eqs. (ge), (xi)), the guard and the diagnostics
__global__ __launch_bounds__(256) void t_reduce_scalars_kernel(const float* __restrict__ tpart, const float* __restrict__ ppart,
                                                               int nparts, int M, int Mp, int nred, int last,
                                                               float* __restrict__ t, float* __restrict__ pv, const float* __restrict__ v,
                                                               const float* __restrict__ u, const float* __restrict__ lambda_bar,
                                                               fw_cond_params prm, Scal* __restrict__ sc, fw_cond_info* __restrict__ info) {
    __shared__ float red[16][16];
    if ((int)blockIdx.x < nred) {
        partial_sum_block(tpart, nparts, M, Mp, blockIdx.x, t, red);
        return;
    }
    if ((int)blockIdx.x < last) {
        partial_sum_block(ppart, nparts, M, Mp, blockIdx.x - nred, pv, red);
        return;
    }
    step_scalars(v, u, M, &red[0][0], lambda_bar, prm, sc, info, true, nullptr, nullptr);
}

// Fused update over the pair of mirrored tiles (I,J) and (J,I), I >= J, one workgroup per pair (pairs enumerated along a
// one-dimensional grid).  Q, Qs, Phi_y and Phi_x are symmetric and kept exactly so: only their tile (I,J) is read, the
// mirrored position takes its old values from that tile transposed through LDS, so the pass reads 4 of the 16 M^2 words
// of a step only half (9 M^2 words move instead of 11).  T and Psi are not symmetric: both of their tiles are read, each
// position needs its own element and, for the terms T + T^T and Psi + Psi^T, the other tile's transposed one.
// FUSED: t and p are the partial products tpart and ppart still ([nparts][Mp]); a workgroup adds up the 64 entries its tiles need and
// works out the scalars for itself, all behind its own loads, which saves t_reduce_scalars_kernel.
template <bool FUSED>
__global__ __launch_bounds__(256) void update_kernel(fw_cond_state s, const float* __restrict__ v, const float* __restrict__ u,
                                                     const float* __restrict__ t, const float* __restrict__ p, Scal* __restrict__ sc,
                                                     fw_cond_params prm, int nparts, fw_cond_info* __restrict__ info, int Mp,
                                                     float* __restrict__ xpart) {
    const float gamma = prm.gamma, beta = prm.beta;
    // pair index -> (I, J), I >= J: I (I + 1) / 2 + J
    int I = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
    while ((I + 1) * (I + 2) / 2 <= (int)blockIdx.x) ++I;
    while (I * (I + 1) / 2 > (int)blockIdx.x) --I;
    const int J = (int)blockIdx.x - I * (I + 1) / 2;
    const int M = s.M;
    const bool leak = gamma < 1.f;
    // four LDS tiles, used twice: first for the transposed elements of T and Psi, then for those of the symmetric
    // matrices (a workgroup's LDS decides how many of them a compute unit holds, and with them the loads in flight)
    __shared__ float L0[TILE][TILE + 1], L1[TILE][TILE + 1], L2[TILE][TILE + 1], L3[TILE][TILE + 1];
    __shared__ float tp[2][64], tsum[FUSED ? 2 : 1][4][64], red[4];     // t, p of the rows of blocks I (0 .. 31) and J (32 .. 63)
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const float g1 = 1.f - gamma, g2 = gamma * gamma, gg1 = gamma * g1, g1sq = g1 * g1, b1 = 1.f - beta;

    // Everything this workgroup reads is asked for before anything is stored (the state pointers may not be told apart
    // by the compiler, so a load behind a store would wait for it: a chain of round trips that dominates small M).
    const int npos = (I == J) ? 1 : 2;
    float Qv[4], Yv[4], Sv[4], Xv[4], Tv[2][4], Pv[2][4], Tt[2][4], Pt[2][4];
    {
        const int j = J * TILE + tx;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = I * TILE + ty + 8 * r;
            const bool ok = i < M && j < M;
            const size_t e = ok ? (size_t)i * M + j : 0;
            Qv[r] = s.Q[e]; Yv[r] = s.Phi_y[e]; Sv[r] = s.Qs[e];
            Xv[r] = leak ? s.Phi_x[e] : 0.f;
        }
    }
#pragma unroll
    for (int pos = 0; pos < 2; ++pos) {
        const int rowblk = pos == 0 ? I : J, colblk = pos == 0 ? J : I;
        const int j = colblk * TILE + tx;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = rowblk * TILE + ty + 8 * r;
            const bool ok = pos < npos && i < M && j < M;
            const size_t e = ok ? (size_t)i * M + j : 0;
            Tv[pos][r] = s.T[e];
            Pv[pos][r] = leak ? s.Psi[e] : 0.f;
            Tt[pos][r] = 0.f; Pt[pos][r] = 0.f;
            if (!ok) { Tv[pos][r] = 0.f; Pv[pos][r] = 0.f; }
        }
    }
    float a, lam;
    if constexpr (FUSED) {
        const int e = threadIdx.x & 63, grp = threadIdx.x >> 6;
        const int m = (e < 32 ? I : J) * TILE + (e & 31);
        float st = 0.f, sp = 0.f;
        if (m < M)
            for (int b0 = grp; b0 < nparts; b0 += 16) {
                float xt[4], xp[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t at = (size_t)(b0 + 4 * q < nparts ? b0 + 4 * q : b0) * Mp + m;
                    xt[q] = t[at];
                    xp[q] = leak ? p[at] : 0.f;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (b0 + 4 * q < nparts) { st += xt[q]; sp += xp[q]; }
            }
        tsum[0][grp][e] = st; tsum[FUSED ? 1 : 0][grp][e] = sp;
        step_scalars(v, u, M, red, s.lambda_bar, prm, sc, info, blockIdx.x == 0, &a, &lam);     // has the barriers that publish tsum
        if (threadIdx.x < 128) {
            const int k = threadIdx.x >> 6;
            tp[k][e] = (tsum[k][0][e] + tsum[k][1][e]) + (tsum[k][2][e] + tsum[k][3][e]);
        }
    } else {
        a = sc->a_e; lam = sc->lambda_e;
        if (threadIdx.x < 64) {
            const int m = (threadIdx.x < 32 ? I : J) * TILE + (threadIdx.x & 31);
            tp[0][threadIdx.x] = m < M ? t[m] : 0.f;
            tp[1][threadIdx.x] = leak && m < M ? p[m] : 0.f;
        }
    }
    __syncthreads();
    const float aa2 = a * (a + 2.f), a2lam = a * a * lam;
    if (leak) {
        // transposed elements of T and Psi: position a reads tile b transposed and the other way round (the diagonal
        // tile reads itself)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int yy = ty + 8 * r;
            L0[yy][tx] = Tv[0][r]; L1[yy][tx] = Pv[0][r];
            if (npos == 2) { L2[yy][tx] = Tv[1][r]; L3[yy][tx] = Pv[1][r]; }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int yy = ty + 8 * r;
            if (npos == 2) { Tt[0][r] = L2[tx][yy]; Pt[0][r] = L3[tx][yy]; Tt[1][r] = L0[tx][yy]; Pt[1][r] = L1[tx][yy]; }
            else { Tt[0][r] = L0[tx][yy]; Pt[0][r] = L1[tx][yy]; }
        }
    }
    if (npos == 2) {
        // old values of the symmetric matrices at the mirrored position: the tile (I,J), read transposed where used
        if (leak) __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int yy = ty + 8 * r;
            L0[yy][tx] = Qv[r]; L1[yy][tx] = Yv[r]; L2[yy][tx] = Sv[r]; L3[yy][tx] = Xv[r];
        }
        __syncthreads();
    }

#pragma unroll
    for (int pos = 0; pos < 2; ++pos) {
        if (pos >= npos) break;
        const int rowblk = pos == 0 ? I : J, colblk = pos == 0 ? J : I;
        const int j = colblk * TILE + tx;
        const int ro = 32 * pos, co = 32 - ro;                 // where the row block's and the column block's entries lie in tp
        const float vj = j < M ? v[j] : 0.f, uj = j < M ? u[j] : 0.f, tj = tp[0][co + tx], pj = tp[1][co + tx];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int yy = ty + 8 * r;
            const int i = rowblk * TILE + yy;
            float sq = 0.f;
            if (i < M && j < M) {
                const size_t e = (size_t)i * M + j;
                const float vi = v[i], ui = u[i], ti = tp[0][ro + yy];
                const float dij = (i == j) ? 1.f : 0.f;
                const float Told = Tv[pos][r];
                const float Qold = pos == 0 ? Qv[r] : L0[tx][yy], Yold = pos == 0 ? Yv[r] : L1[tx][yy];
                const float Sold = pos == 0 ? Sv[r] : L2[tx][yy];
                const float Tn = gamma * (Told + a * vi * tj) + g1 * dij;
                float Qn = g2 * (Qold + aa2 * (ti * tj)) + g1sq * dij;
                float Yn = g2 * (Yold + a * (vi * uj + ui * vj) + a2lam * (vi * vj));
                if (leak) {
                    const float Psiold = Pv[pos][r], phix = pos == 0 ? Xv[r] : L3[tx][yy], pi = tp[1][ro + yy];
                    Qn += gg1 * (a * (vi * tj + ti * vj) + Told + Tt[pos][r]);
                    Yn += gg1 * (Psiold + Pt[pos][r] + a * (vi * pj + pi * vj)) + g1sq * phix;
                    s.Psi[e] = gamma * (Psiold + a * vi * pj) + g1 * phix;
                }
                s.T[e] = Tn;
                s.Q[e] = Qn;
                s.Qs[e] = beta * Sold + b1 * Qn;
                s.Phi_y[e] = Yn;
                sq = Yn * Yn;
            }
            // sum over the 32 lanes that share row i
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
            if (tx == 0 && i < M) xpart[(size_t)colblk * Mp + i] = sq;
        }
    }
}

// Up to here the sums ride along with the loads of the update; beyond it every workgroup's share of them costs more than the launch.  A
// step, fused / not: 72 features 21.2 / 22.7 us, 288 23.1 / 24.4, 576 26.2 / 27.1, 800 30.2 / 30.3, 1152 34.7 / 34.4, 1800 68 / 60.
constexpr int UPDATE_FUSED_MAX_M = 640;

// ---- the whole step in one launch, for few features
// Up to 64 features the six launches of the general form do next to nothing each: their time is the time between
// launches (about 4.4 us apiece).  Here one workgroup of 1024 threads brings all six matrices to LDS, their loads in
// flight together, and does the step from there.  The chain of five products runs in single wavefronts with a matrix in the
// registers of each, two barriers in all; the update is spread over all 16: a wavefront owns the rows wave, wave + 16, ..., a lane is a
// column.  64 features: 24 us with six launches, 13 us with every product spread over 16 wavefronts and 15 barriers, 10.5 us like this.
// The line lies where six matrices fill the LDS: with one matrix at a time in LDS and the others read behind one another
// from memory, one compute unit needed 77 us at 147 features against 31 us of the six launches.
constexpr int COND_SMALL_MAX_M = 64;

__global__ __launch_bounds__(1024) void cond_small_kernel(fw_cond_state s, fw_cond_params prm, fw_cond_info* __restrict__ info) {
    constexpr int PER = COND_SMALL_MAX_M / 16;
    constexpr int MAT = COND_SMALL_MAX_M * (COND_SMALL_MAX_M + 1);
    __shared__ float Py[MAT], Tm[MAT], Qm[MAT], Sm[MAT], Pm[MAT], Xm[MAT];
    __shared__ float x0[64], v[64], u[64], t[64], p[64];
    __shared__ float out_a, out_lam;
    __shared__ Scal sc;
    const int M = s.M, ld = M | 1;      // odd row pitch: rows and columns are both read without conflicts
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool leak = prm.gamma < 1.f;
    // element k of this thread: row wave + 16 k, column lane
#define FW_EACH(k, i, j)                                                                    \
    _Pragma("unroll") for (int k = 0; k < PER; ++k)                                         \
        if (const int i = wave + 16 * k, j = lane; i < M && j < M)
    auto load = [&](const float* __restrict__ src, float (&x)[PER]) {
        FW_EACH(k, i, j) x[k] = src[i * M + j];
    };
    auto put = [&](float* dst, const float (&x)[PER]) {
        FW_EACH(k, i, j) dst[i * ld + j] = x[k];
    };
    const float x2_raw = (wave == 0 && lane < M) ? s.xi2[lane] : -1.f, lambda_bar = *s.lambda_bar;
    const float x2 = x2_raw > -1.f ? x2_raw : -1.f;
    {
        float x[PER], y0[PER], y1[PER], y2[PER], y3[PER], y4[PER];
        load(s.Phi_y, x); load(s.T, y0); load(s.Q, y1); load(s.Qs, y2);
        if (leak) { load(s.Psi, y3); load(s.Phi_x, y4); }
        put(Py, x); put(Tm, y0); put(Qm, y1); put(Sm, y2);
        if (leak) { put(Pm, y3); put(Xm, y4); }
    }
    __syncthreads();

    // The chain of products: a wavefront holds a whole matrix, a column per lane, and takes the entries of x from its own lanes, so a
    // product needs no barrier.  Wavefront 0 has Phi_y and goes from the arg-max to v and u alone; 1 and 2 have T and Psi.
    if (wave < 3) {
        float col[COND_SMALL_MAX_M];
        {
            const float* src = wave == 0 ? Py : wave == 1 ? Tm : Pm;
            const bool mine = lane < M && (wave < 2 || leak);
#pragma unroll
            for (int i = 0; i < COND_SMALL_MAX_M; ++i) col[i] = (mine && i < M) ? src[i * ld + lane] : 0.f;
        }
        // column `lane` of the matrix times x (zero in the lanes from M on)
        auto product = [&](float x) {
            float y0 = 0.f, y1 = 0.f, y2 = 0.f, y3 = 0.f;
#pragma unroll
            for (int i = 0; i < COND_SMALL_MAX_M; i += 4) {
                auto at = [&](int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k)); };
                y0 += col[i] * at(i); y1 += col[i + 1] * at(i + 1); y2 += col[i + 2] * at(i + 2); y3 += col[i + 3] * at(i + 3);
            }
            return (y0 + y1) + (y2 + y3);
        };
        if (wave == 0) {
            // m', eq. (mt): norms that are NaN do not count, the lowest index on ties
            const float best = wave_max_dpp(x2);
            const unsigned long long ties = __ballot(lane < M && x2 == best);
            const int mp = ties ? __ffsll((long long)ties) - 1 : 0;
            const float xi_mp = sqrtf(fmaxf(best, 0.f));
            const float c = product(lane < M ? Py[mp * ld + lane] : 0.f);                                  // eq. (vc)
            // coherence set and weights (rule after eq. (vc))
            const bool in = lane < M && fabsf(c) >= fmaxf(prm.c_rel * xi_mp * sqrtf(fmaxf(x2, 0.f)), prm.c_abs);
            const int total = __popcll(__ballot(in));
            int flags = total == 0 ? 1 : 0;
            float cur = product(in && c != 0.f ? 1.f / ((float)total * c) : 0.f);                          // v~, first line of eq. (tve)
            float nrm, inv;
            for (int it = 0;; ++it) {
                nrm = sqrtf(wave_sum_dpp(cur * cur));
                inv = (nrm > 0.f && (flags & 1) == 0) ? 1.f / nrm : 0.f;
                if (it == prm.n_power_iters) break;
                cur = product(cur) * inv;                                                                  // refinement
            }
            if (!(nrm == nrm) || nrm > 3.0e38f) flags |= 4;
            x0[lane] = cur; v[lane] = cur * inv;
            if (lane == 0) { sc.vnorm = nrm; sc.m_prime = mp; sc.set_size = total; sc.flags = flags; sc.lambda_e = inv; }
        }
        __syncthreads();
        const float cur = x0[lane], inv = sc.lambda_e;
        const float y = product(cur) * inv;                     // u = Phi_y v, t = T^T v, p = Psi^T v
        (wave == 0 ? u : wave == 1 ? t : p)[lane] = y;
        if (wave == 0) {
            const float lam_e = wave_sum_dpp(cur * inv * y);                                               // eq. (lambda)
            int flags = sc.flags, applied = 0;
            float g_e = 1.f, a = 0.f;
            if ((flags & 1) == 0) {                             // eqs. (ge), (xi) and the guard
                g_e = prm.delta * lambda_bar / fmaxf(lam_e, prm.eps);
                if (prm.guard && g_e >= 1.f) flags |= 2;
                else if (!(g_e == g_e) || g_e > 3.0e38f) flags |= 4;
                else { a = sqrtf(g_e) - 1.f; applied = 1; }
            }
            const float lam = (flags & 1) ? 0.f : lam_e;
            if (lane == 0) {
                out_a = a; out_lam = lam;
                if (info) {
                    info->lambda_e = lam; info->g_e = g_e; info->a_e = a; info->v_norm = sc.vnorm;
                    info->m_prime = sc.m_prime; info->set_size = sc.set_size; info->applied = applied; info->flags = flags;
                }
            }
        }
    } else {
        __syncthreads();
    }
    __syncthreads();
    const float a = out_a, lam = out_lam;

    // update: the formulas of update_kernel.  Old values of a symmetric matrix come from its lower triangle (hi, lo), and the
    // terms of a symmetric result are taken in that order, so both positions get the same value.
    const float gamma = prm.gamma, beta = prm.beta;
    const float g1 = 1.f - gamma, g2 = gamma * gamma, gg1 = gamma * g1, g1sq = g1 * g1, b1 = 1.f - beta;
    const float aa2 = a * (a + 2.f), a2lam = a * a * lam;
    float ynew[PER];
    FW_EACH(k, i, j) {
        const int hi = max(i, j), lo = min(i, j), e = i * ld + j, eh = hi * ld + lo, el = lo * ld + hi;
        const bool diag = i == j;
        float qn = g2 * (Qm[eh] + aa2 * (t[i] * t[j])) + (diag ? g1sq : 0.f);
        float y = g2 * (Py[eh] + a * (v[hi] * u[lo] + u[hi] * v[lo]) + a2lam * (v[i] * v[j]));
        if (leak) {
            qn += gg1 * (a * (v[hi] * t[lo] + t[hi] * v[lo]) + Tm[eh] + Tm[el]);
            y += gg1 * (Pm[eh] + Pm[el] + a * (v[hi] * p[lo] + p[hi] * v[lo])) + g1sq * Xm[eh];
            s.Psi[i * M + j] = gamma * (Pm[e] + a * v[i] * p[j]) + g1 * Xm[eh];
        }
        s.T[i * M + j] = gamma * (Tm[e] + a * v[i] * t[j]) + (diag ? g1 : 0.f);
        s.Q[i * M + j] = qn;
        s.Qs[i * M + j] = beta * Sm[eh] + b1 * qn;
        s.Phi_y[i * M + j] = y;
        ynew[k] = y;
    }
    // squared row norms of the new Phi_y: a row belongs to one wavefront
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = wave + 16 * k;
        if (i >= M) break;
        const float q = wave_sum_dpp(lane < M ? ynew[k] * ynew[k] : 0.f);
        if (lane == 0) s.xi2[i] = q;
    }
#undef FW_EACH
}

__global__ __launch_bounds__(256) void state_init_kernel(fw_cond_state s) {
    const int M = s.M;
    const size_t n = (size_t)M * M;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
        const int i = (int)(e / M), j = (int)(e - (size_t)i * M);
        const float d = i == j ? 1.f : 0.f;
        const float ph = s.Phi_x[e];
        s.T[e] = d; s.Q[e] = d; s.Qs[e] = d;
        s.Phi_y[e] = ph;
        if (s.Psi) s.Psi[e] = ph;
    }
}

// Lower triangle -> full symmetric matrix, and the squared row norms of the result, in one pass over pairs of 64 x 64 tiles
// (I, J), I >= J (M a multiple of 4): the tile (I,J) is read once with 16-byte loads, written transposed as (J,I) through
// LDS, and leaves two sets of partial sums of squares: over its columns for the rows of block I, over its rows for the
// rows of block J (the mirrored tile's rows).  xpart[colblock][row], summed by partial_sum_kernel.
// With nks > 0 the lower triangle is the sum of the runs part[nks][M][M], added in order, and is written as well.
__global__ __launch_bounds__(256) void mirror_rownorm_kernel(float* __restrict__ P, int M, int Mp, float* __restrict__ xpart,
                                                             const float* __restrict__ part, int nks) {
    __shared__ float t[64][65];
    int I = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
    while ((I + 1) * (I + 2) / 2 <= (int)blockIdx.x) ++I;
    while (I * (I + 1) / 2 > (int)blockIdx.x) --I;
    const int J = (int)blockIdx.x - I * (I + 1) / 2;
    const int q = threadIdx.x & 15, r0 = threadIdx.x >> 4;     // 16 threads along a row (4 floats each), 16 rows per pass
    const int j = J * 64 + 4 * q;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int rr = r0 + 16 * pass, i = I * 64 + rr;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < M && j < M) {
            const size_t e = (size_t)i * M + j;
            if (nks > 0) {
                v = *reinterpret_cast<const float4*>(part + e);
                for (int z = 1; z < nks; ++z) {
                    const float4 w = *reinterpret_cast<const float4*>(part + (size_t)z * M * M + e);
                    v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
                }
                if (I != J) *reinterpret_cast<float4*>(P + e) = v;
            } else {
                v = *reinterpret_cast<const float4*>(P + e);
            }
            if (I == J) {            // diagonal tile: what lies above the diagonal is taken from below it, after the barrier
                if (j > i) v.x = 0.f;
                if (j + 1 > i) v.y = 0.f;
                if (j + 2 > i) v.z = 0.f;
                if (j + 3 > i) v.w = 0.f;
            }
        }
        t[rr][4 * q] = v.x; t[rr][4 * q + 1] = v.y; t[rr][4 * q + 2] = v.z; t[rr][4 * q + 3] = v.w;
    }
    __syncthreads();
    if (I == J) {
        // complete the tile in LDS (upper = lower transposed), write it back whole, one set of row sums
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int rr = r0 + 16 * pass, i = I * 64 + rr;
            float x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) { const int cc = 4 * q + k; x[k] = cc > rr ? t[cc][rr] : t[rr][cc]; }
            float sq = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
            if (i < M && j < M) *reinterpret_cast<float4*>(P + (size_t)i * M + j) = make_float4(x[0], x[1], x[2], x[3]);
            else sq = 0.f;
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
            if (q == 0 && i < M) xpart[(size_t)J * Mp + i] = sq;
        }
        return;
    }
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int rr = r0 + 16 * pass;
        // row sums of the tile as read (rows of block I, column block J)
        const int i = I * 64 + rr;
        float sq = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) { const float x = t[rr][4 * q + k]; sq += x * x; }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
        if (q == 0 && i < M) xpart[(size_t)J * Mp + i] = sq;
        // the mirrored tile: row rr of (J, I) is column rr of (I, J)
        const int im = J * 64 + rr, jm = I * 64 + 4 * q;
        float x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = t[4 * q + k][rr];
        float sm = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
        if (im < M && jm < M) *reinterpret_cast<float4*>(P + (size_t)im * M + jm) = make_float4(x[0], x[1], x[2], x[3]);
        else sm = 0.f;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) sm += __shfl_xor(sm, o, 64);
        if (q == 0 && im < M) xpart[(size_t)I * Mp + im] = sm;
    }
}

__global__ __launch_bounds__(256) void rownorm2_kernel(const float* __restrict__ P, int M, float* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    float acc = 0.f;
    for (int k = lane; k < M; k += 64) { const float x = P[(size_t)r * M + k]; acc += x * x; }
    acc = wave_sum(acc);
    if (lane == 0) out[r] = acc;
}

// Mirror image of the lower triangle and squared row norms in one launch, without scratch: a workgroup owns 16 rows.  Their
// part up to the diagonal is read along the rows, one wavefront per row; what lies beyond is the part of their 16 columns below
// the diagonal, read in runs of 64 bytes, turned in LDS and written along the rows.  Only elements on or below the
// diagonal are read and only elements above it are written, so workgroups do not meet.
// Bound by two or three rounds of dependent loads up to about 1000 features.  The refresh in its float32 form, against a launch
// each for mirror and norms: 15.3 us -> 12.7 us at 256 features, 20.2 -> 18.1 at 512, 65.8 -> 61.9 at 1152, 279 -> 272 at 1800.
constexpr int MIRROR_NORM_MAX_M = 2048;
__global__ __launch_bounds__(1024) void mirror_norm_rows_kernel(float* __restrict__ P, int M, float* __restrict__ out) {
    constexpr int NT = 8, LD = 68;                 // tiles of 64 columns per round; pitch that spreads the stores over the banks
    __shared__ float t[NT][16 * LD];
    __shared__ float red[16][17], row_sum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * 16;
    const int ci = i0 + (tid & 15), cj = tid >> 4; // reading: column ci, rows cj, cj + 64, ...
    const int wi = i0 + wave;                      // row part and writing: row wi
    float below = 0.f;
    for (int jb = i0; jb < M; jb += 64 * NT) {
        float v[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int j = jb + 64 * q + cj;
            v[q] = P[j < M && j > ci ? (size_t)j * M + ci : 0];
        }
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int j = jb + 64 * q + cj;
            if (!(j < M && j > ci)) v[q] = 0.f;
            t[q][(tid & 15) * LD + cj] = v[q];
        }
        below += ((v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3])) + ((v[4] * v[4] + v[5] * v[5]) + (v[6] * v[6] + v[7] * v[7]));
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int j = jb + 64 * q + lane;
            if (wi < M && j < M && j > wi) P[(size_t)wi * M + j] = t[q][wave * LD + lane];
        }
        __syncthreads();
    }
    float upto = 0.f;
    if (wi < M)
        for (int k = lane; k <= wi; k += 64 * 8) {
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = P[k + 64 * q <= wi ? (size_t)wi * M + k + 64 * q : 0];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = k + 64 * q <= wi ? x[q] * x[q] : 0.f;
            upto += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        }
    upto = wave_sum(upto);
    below += __shfl_xor(below, 16, 64);
    below += __shfl_xor(below, 32, 64);
    if (lane < 16) red[wave][lane] = below;
    if (lane == 0) row_sum[wave] = upto;
    __syncthreads();
    if (tid < 16 && i0 + tid < M) {
        double s = (double)row_sum[tid];
#pragma unroll
        for (int w = 0; w < 16; ++w) s += (double)red[w][tid];
        out[i0 + tid] = (float)s;
    }
}

// ---- the refresh in one launch, for few features
// Two products, the mirror image and the row norms are four launches that do little work each.  The strip of 16 rows of
// Phi_y needs only the same strip of Psi, so a workgroup forms its strip of Psi, keeps it in LDS and multiplies on: one
// wavefront per tile of 16 columns, v_mfma_f32_16x16x4_f32, operands straight from L2 (16 bytes per lane and load).  The
// matrix is written from its lower triangle (an element below the diagonal also goes to the mirrored position); the row norms are taken
// from the strip as computed, whose part above the diagonal differs from the stored one by rounding only.
// Only M / 16 compute units work, at 4 M^2 words each, so the form ends early.  Measured, this form against the four
// launches: 7.0 / 15.6 us at 64 features, 10.2 / 15.6 at 128, 16.5 / 15.4 at 160; with rows that are not 16-byte aligned
// (single loads) 11.0 / 14.9 at 75 and 26.9 / 18.5 at 147.
constexpr int REFRESH_ROWS_MAX_M = 128, REFRESH_ROWS_MAX_M_UNALIGNED = 80;
// Four accumulators, added pairwise: a single float32 chain over the whole contraction index had 1.2 times (up to 1.8 times) the
// error of the general form, whose wavefronts take a quarter of it each.
template <bool V4>
__device__ __forceinline__ floatx4 refresh_tile(const float* a_row, const float* __restrict__ b_row, int K, int kq) {
    constexpr int U = 4;
    floatx4 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 16 * U) {
        float a[U][4], b[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 16 * u + 4 * kq;
            if (V4) {
                const float4 y = *reinterpret_cast<const float4*>(b_row + (k < K ? k : 0));
                const float4 x = *reinterpret_cast<const float4*>(a_row + (k < K ? k : 0));
                a[u][0] = x.x; a[u][1] = x.y; a[u][2] = x.z; a[u][3] = x.w;
                b[u][0] = y.x; b[u][1] = y.y; b[u][2] = y.z; b[u][3] = y.w;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) { a[u][q] = a_row[k + q < K ? k + q : 0]; b[u][q] = b_row[k + q < K ? k + q : 0]; }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 16 * u + 4 * kq;
            // beyond the end both factors are zero (a value of entry 0 may be infinite)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool ok = k + q < K;
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? a[u][q] : 0.f, ok ? b[u][q] : 0.f, acc[q], 0, 0, 0);
            }
        }
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
template <bool V4>
__global__ __launch_bounds__(512) void refresh_rows_kernel(const float* __restrict__ T, const float* __restrict__ Phi_x, int M,
                                                            float* __restrict__ Psi, float* __restrict__ Phi_y, float* __restrict__ xi2) {
    constexpr int PITCH = REFRESH_ROWS_MAX_M + 4;      // 16 rows of one column group fall into distinct banks
    __shared__ __attribute__((aligned(16))) float Ps[16][PITCH];
    __shared__ float red[8][16];
    const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
    const int tile = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ntiles = blockDim.x >> 6;
    const int row0 = blockIdx.x * 16, col = tile * 16 + r;
    const float* Trow = T + (size_t)min(row0 + r, M - 1) * M;    // rows past the end feed results that are not stored
    const size_t coff = (size_t)min(col, M - 1) * M;
    floatx4 acc = refresh_tile<V4>(Trow, Phi_x + coff, M, kq);     // Phi_x is symmetric: its rows stand for its columns
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = row0 + 4 * kq + i;
        Ps[4 * kq + i][col] = acc[i];
        if (row < M && col < M) Psi[(size_t)row * M + col] = acc[i];
    }
    __syncthreads();
    acc = refresh_tile<V4>(Ps[r], T + coff, M, kq);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = row0 + 4 * kq + i;
        const float y = acc[i];
        if (row < M && col <= row) {
            Phi_y[(size_t)row * M + col] = y;
            if (col < row) Phi_y[(size_t)col * M + row] = y;
        }
        float q = col < M ? y * y : 0.f;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
        if (r == 0) red[tile][4 * kq + i] = q;
    }
    __syncthreads();
    if (threadIdx.x < 16 && row0 + (int)threadIdx.x < M) {
        double q = 0.0;
        for (int k = 0; k < ntiles; ++k) q += (double)red[k][threadIdx.x];
        xi2[row0 + threadIdx.x] = (float)q;
    }
}

}  // namespace

size_t cond_workspace_bytes(int M) { return ws_layout(M).total; }

fw_status cond_state_init(const fw_cond_state* s, hipStream_t st) {
    const size_t n = (size_t)s->M * s->M;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(state_init_kernel, dim3(blocks), dim3(256), 0, st, *s);
    FW_LAUNCH_CHECK();
    hipLaunchKernelGGL(rownorm2_kernel, dim3((s->M + 3) / 4), dim3(256), 0, st, s->Phi_x, s->M, s->xi2);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// Workspace of the refresh: room for Psi when the state has none, then the packed hi / lo planes of T, Phi_x and Psi.
static size_t refresh_xpart_bytes(int M) {
    const size_t nt = (size_t)(M + 63) / 64, Mp = (size_t)(M + 63) / 64 * 64;
    return align_up(nt * Mp * sizeof(float), 256);
}
static size_t refresh_split_bytes(int M) {
    return align_up((size_t)M * M * sizeof(float), 256) + 3 * gemm_split_packed_bytes(M, M) + refresh_xpart_bytes(M);
}
// Few 256-wide tiles leave compute units idle: the products then cut their contraction index into runs, which the passes behind
// them (packing of Psi, mirror image of Phi_y) add up on the way.  What the runs fill is also what the sums of the next batch use on
// a second stream, and beyond the lines below writing and reading them costs more than it saves.  Whole steps (12544 rows), us on one
// stream | with the next sums on a second one, without runs / in the product for Psi alone / for Phi_y alone / in both:
//   1584  339 / 326 / 316 / 301 | 266 / 275 / 260 / 249        2304  472 / 482 / 457 / 463 | 382 / 422 / 395 / 408
//   2016  417 / 402 / 394 / 376 | 325 / 353 / 331 / 323        2592  630 / 642 / 615 / 624 | 569 / 586 / 556 / 571
//   2052  470 / 465 / 443 / 438 | 374 / 379 / 380 / 379        2736  696 / 707 / 693 / 695 | 630 / 648 / 630 / 645
//   2160  473 / 480 / 448 / 450 | 383 / 427 / 388 / 399        3312  818 / 816 / 829 / 828 | 792 / 792 / 803 / 803
constexpr int REFRESH_RUNS_MAX_M = 2100, REFRESH_LOWER_RUNS_MAX_M = 2700;
static int refresh_runs(int M, int lower) {
    if (M < FW_REFRESH_SPLIT_MIN_M || (M & 3) != 0 || M > (lower ? REFRESH_LOWER_RUNS_MAX_M : REFRESH_RUNS_MAX_M)) return 1;
    return gemm_split_caller_runs(M, M, M, lower);
}
static size_t refresh_runs_bytes(int M) {
    const int a = refresh_runs(M, 0), b = refresh_runs(M, 1), n = a > b ? a : b;
    return n > 1 ? align_up((size_t)n * M * M * sizeof(float), 256) : 0;
}
size_t cond_refresh_workspace_bytes(int M) { return refresh_split_bytes(M) + refresh_runs_bytes(M); }

static bool refresh_in_rows(int M) { return M <= ((M & 3) == 0 ? REFRESH_ROWS_MAX_M : REFRESH_ROWS_MAX_M_UNALIGNED); }

bool cond_refresh_plan(int M, size_t ws_bytes, fw_refresh_plan* plan) {
    if (M <= 0 || M > 16384) return false;
    plan->split = (ws_bytes >= refresh_split_bytes(M) && M >= FW_REFRESH_SPLIT_MIN_M) ? 1 : 0;
    const bool runs = refresh_runs_bytes(M) > 0 && ws_bytes >= cond_refresh_workspace_bytes(M);
    if (plan->split) plan->mfma_flops_issued = gemm_split_flops_issued(M, M, M, 0, false, runs && refresh_runs(M, 0) > 1) +
                                               gemm_split_flops_issued(M, M, M, 1, false, runs && refresh_runs(M, 1) > 1);
    else if (refresh_in_rows(M)) {       // two products of every 16 x 16 tile, the contraction index in rounds of 64
        const double nt = (M + 15) / 16;
        plan->mfma_flops_issued = 2.0 * nt * nt * 2.0 * 256.0 * ((M + 63) / 64 * 64);
    } else plan->mfma_flops_issued = grad_gemm_f32_flops_issued(M, M, false) + grad_gemm_f32_flops_issued(M, M, true);
    return true;
}

// New block, new Phi_x: Psi = T Phi_x and Phi_y = T Phi_x T^T = Psi T^T by two M x M x M products, Phi_y made exactly
// symmetric from its lower triangle, and the squared row norms for the arg-max.  Few features: all of it in one launch
// (refresh_rows_kernel).  Otherwise both products have the form A B^T with
// row-major operands: Phi_x is symmetric (its rows stand for its columns), and T is exactly the factor wanted.
// With the full workspace the operands are split into bfloat16 hi + lo planes and multiplied on the bfloat16 matrix
// cores (three products per term, float32 accumulation: see gemm_split.hip); without it (allowed when the state carries
// Psi) the products run in plain float32 on the matrix cores.  Only the lower triangle of Phi_y is computed either way.
fw_status cond_state_refresh(const fw_cond_state* s, void* ws, size_t ws_bytes, hipStream_t st) {
    const int M = s->M;
    const size_t psi_bytes = align_up((size_t)M * M * sizeof(float), 256);
    char* base = reinterpret_cast<char*>(ws);
    float* Psi = s->Psi ? s->Psi : reinterpret_cast<float*>(base);
    if (refresh_in_rows(M)) {
        const dim3 grid((M + 15) / 16), blk(64 * ((M + 15) / 16));
        if ((M & 3) == 0) hipLaunchKernelGGL(refresh_rows_kernel<true>, grid, blk, 0, st, s->T, s->Phi_x, M, Psi, s->Phi_y, s->xi2);
        else hipLaunchKernelGGL(refresh_rows_kernel<false>, grid, blk, 0, st, s->T, s->Phi_x, M, Psi, s->Phi_y, s->xi2);
        FW_LAUNCH_CHECK();
        return FW_OK;
    }
    fw_status rc;
    // Below about 1500 features the float32 kernel is as fast (too few 256-wide tiles for 256 compute units, and the
    // three packing passes cost as much as a product); FW_REFRESH_SPLIT_MIN_M is where the split form starts.
    if (ws && ws_bytes >= refresh_split_bytes(M) && M >= FW_REFRESH_SPLIT_MIN_M) {
        const size_t pb = gemm_split_packed_bytes(M, M);
        void* Tp = base + psi_bytes;
        void* Xp = base + psi_bytes + pb;
        void* Pp = base + psi_bytes + 2 * pb;
        if ((rc = gemm_split_pack(s->T, M, M, Tp, st)) != FW_OK) return rc;
        if ((rc = gemm_split_pack(s->Phi_x, M, M, Xp, st)) != FW_OK) return rc;
        float* part = refresh_runs_bytes(M) > 0 && ws_bytes >= cond_refresh_workspace_bytes(M)
                          ? reinterpret_cast<float*>(base + refresh_split_bytes(M)) : nullptr;
        int runs = 1;
        if (part && refresh_runs(M, 0) > 1) {
            if ((rc = gemm_split_run(Tp, Xp, M, M, M, 0, part, st, part, &runs, true)) != FW_OK) return rc;
            if ((rc = gemm_split_sum_pack(part, runs, M, M, Psi, Pp, st)) != FW_OK) return rc;
        } else {
            if ((rc = gemm_split_run(Tp, Xp, M, M, M, 0, Psi, st)) != FW_OK) return rc;
            if ((rc = gemm_split_pack(Psi, M, M, Pp, st)) != FW_OK) return rc;
        }
        int lower_runs = 0;
        if (part && refresh_runs(M, 1) > 1) {
            if ((rc = gemm_split_run(Pp, Tp, M, M, M, 1, part, st, part, &lower_runs, true)) != FW_OK) return rc;
        } else {
            if ((rc = gemm_split_run(Pp, Tp, M, M, M, 1, s->Phi_y, st)) != FW_OK) return rc;
        }
        if ((M & 3) == 0) {
            // mirror and squared row norms in one pass
            float* xpart = reinterpret_cast<float*>(base + psi_bytes + 3 * pb);
            const int nt = (M + 63) / 64, Mp = nt * 64;
            hipLaunchKernelGGL(mirror_rownorm_kernel, dim3(nt * (nt + 1) / 2), dim3(256), 0, st, s->Phi_y, M, Mp, xpart, part, lower_runs);
            hipLaunchKernelGGL(partial_sum_kernel, dim3((M + 15) / 16), dim3(256), 0, st, xpart, nt, M, Mp, s->xi2);
            FW_LAUNCH_CHECK();
            return FW_OK;
        }
    } else {
        rc = grad_gemm(s->T, FW_F32, M, M, s->Phi_x, Psi, st);
        if (rc != FW_OK) return rc;
        // of the symmetric product only the strips that touch the lower triangle
        GemmEpilogue lower_half = {};
        lower_half.out = s->Phi_y; lower_half.taps = 1;
        rc = grad_gemm_f32(Psi, M, M, s->T, lower_half, st, nullptr, true);
        if (rc != FW_OK) return rc;
    }
    if (M <= MIRROR_NORM_MAX_M) {
        hipLaunchKernelGGL(mirror_norm_rows_kernel, dim3((M + 15) / 16), dim3(1024), 0, st, s->Phi_y, M, s->xi2);
        FW_LAUNCH_CHECK();
        return FW_OK;
    }
    rc = symmetrize_from_lower(s->Phi_y, M, st);
    if (rc != FW_OK) return rc;
    hipLaunchKernelGGL(rownorm2_kernel, dim3((M + 3) / 4), dim3(256), 0, st, s->Phi_y, M, s->xi2);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// Device address of `scratch` on the current device, looked up once per device (every GPU holds its own copy of the
// array at its own address).
fw_status cond_static_scratch(void** ptr, size_t* bytes) {
    constexpr int kMaxDevices = 64;
    static void* table[kMaxDevices] = {};
    static std::mutex mu;
    int dev = -1;
    FW_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return FW_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!table[dev]) {
        void* p = nullptr;
        FW_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return FW_ERR_HIP;
        table[dev] = p;
    }
    *ptr = table[dev];
    *bytes = sizeof(scratch);
    return FW_OK;
}

fw_status cond_reduce_step(const fw_cond_state* s, const fw_cond_params* p, fw_cond_info* info, void* ws, hipStream_t st) {
    const int M = s->M;
    if (M <= COND_SMALL_MAX_M) {
        hipLaunchKernelGGL(cond_small_kernel, dim3(1), dim3(1024), 0, st, *s, *p, info);
        FW_LAUNCH_CHECK();
        return FW_OK;
    }
    const WsLayout L = ws_layout(M);
    char* base = reinterpret_cast<char*>(ws);
    float* c = reinterpret_cast<float*>(base + L.c);
    float* w = reinterpret_cast<float*>(base + L.w);
    float* vt = reinterpret_cast<float*>(base + L.vt);
    float* v = reinterpret_cast<float*>(base + L.v);
    float* u = reinterpret_cast<float*>(base + L.u);
    float* t = reinterpret_cast<float*>(base + L.t);
    float* pv = reinterpret_cast<float*>(base + L.p);
    float* tpart = reinterpret_cast<float*>(base + L.tpart);
    float* ppart = reinterpret_cast<float*>(base + L.ppart);
    float* xpart = reinterpret_cast<float*>(base + L.xpart);
    Scal* sc = reinterpret_cast<Scal*>(base + L.scal);
    const dim3 mv_grid((M + 3) / 4), mv_blk(256);

    const int nmv = (M + 3) / 4, ncol = (M + 255) / 256, nred = (M + 15) / 16;
    hipLaunchKernelGGL(matvec_c_kernel, mv_grid, mv_blk, 0, st, s->Phi_y, s->xi2, M, sc, c);
    hipLaunchKernelGGL(matvec_vt_kernel, mv_grid, mv_blk, (size_t)L.Mp * sizeof(float), st, s->Phi_y, c, s->xi2, M, p->c_rel, p->c_abs, sc, vt);
    float* cur = vt;
    float* other = w;   // scratch vector for the optional refinements
    for (int it = 0; it < p->n_power_iters; ++it) {
        hipLaunchKernelGGL(matvec_refine_kernel, mv_grid, mv_blk, 0, st, s->Phi_y, cur, M, sc, other);
        float* tmp = cur; cur = other; other = tmp;
    }
    const bool leak = p->gamma < 1.f;
    const int nvm = ncol * L.nrb, last = nred * (leak ? 2 : 1);
    hipLaunchKernelGGL(matvec_u_vecmat_kernel, dim3(nmv + nvm * (leak ? 2 : 1)), mv_blk, 0, st, s->Phi_y, s->T, s->Psi, cur, M, L.Mp,
                       L.vm_rows, nmv, nvm, sc, v, u, tpart, ppart);
    const dim3 pairs(L.nt * (L.nt + 1) / 2);
    if (M <= UPDATE_FUSED_MAX_M) {
        hipLaunchKernelGGL(update_kernel<true>, pairs, dim3(256), 0, st, *s, v, u, tpart, ppart, sc, *p, L.nrb, info, L.Mp, xpart);
    } else {
        hipLaunchKernelGGL(t_reduce_scalars_kernel, dim3(last + 1), mv_blk, 0, st, tpart, ppart, L.nrb, M, L.Mp, nred, last, t, pv, v, u,
                           s->lambda_bar, *p, sc, info);
        hipLaunchKernelGGL(update_kernel<false>, pairs, dim3(256), 0, st, *s, v, u, t, pv, sc, *p, 0, info, L.Mp, xpart);
    }
    hipLaunchKernelGGL(partial_sum_kernel, dim3(nred), dim3(256), 0, st, xpart, L.nt, M, L.Mp, s->xi2);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

}  // namespace fw
