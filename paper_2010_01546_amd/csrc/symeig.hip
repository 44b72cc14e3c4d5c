// Eigenvectors of a real symmetric matrix in float64 for gfx950: A = Q T Q^T with T tridiagonal (Householder reflections),
// T = S Lambda S^T by divide and conquer, eigenvectors (Q S)^T, one per ROW.  Used by fw_whiten_evd (evd.hip).
//
// Reduction.  Row c = M-1, M-2, ... is eliminated against the leading c x c block, so that the active block always starts
// at the (aligned) origin.  One launch per step does everything that step needs: the rank-2 update that the PREVIOUS step
// left pending, the new reflector, and the product p = A v with it, in a single pass over the active block:
//     w = tau (p_prev - tau/2 (p_prev . v_prev) v_prev),   A <- A - v_prev w^T - w v_prev^T,   p = A v
// The vectors w, x (the row to eliminate) and v are worked out by every workgroup for itself (M entries each, two sums over
// the workgroup), so a step has no second launch and no grid-wide barrier; a thread owns fixed columns and keeps its entries
// of v_prev, w and v in registers while the rows of the workgroup stream past.  The whole matrix is stored (both triangles)
// so that rows are contiguous.  Bound: the launch and the two dependent sums (3.4 to 5.7 us a step) up to about 1000 rows, from
// there on the traffic of 16 M^3/3 bytes (7.3 us a step at 1025 to 1536 rows, 10.2 up to 2048, 14.6 up to 2560).  The last 128 rows are finished by one workgroup with the block in its registers.
// From 129 rows on, and for the last 2560 of more, tri_rows_kernel does all of it in one launch (see there); the steps are for what lies
// beyond and for a device that does not hold its workgroups at a time.
//
// Divide and conquer (J. J. M. Cuppen 1981).  T is torn at equidistant places into leaves of at most 16 rows (Jacobi, one
// wavefront each); a merge of two neighbours is a rank-one update D + rho z z^T.  Deflation as in the paper by Gu and
// Eisenstat (1995): entries with a negligible component of z, and one of two (nearly) equal entries after a plane
// rotation.  The secular equation is solved in coordinates relative to the nearest pole by rational interpolation of its two
// halves (Bunch, Nielsen, Sorensen 1978) inside a bracket, z is recomputed from the computed roots (Gu and Eisenstat), which
// makes the vectors orthogonal to working precision whatever the clustering, and the product with the children's vectors runs
// on the float64 matrix cores, over entries grouped by the child whose columns they reach (J. D. Rutter 1994).  All merges of a level
// share their launches; sizes after deflation stay on the device.
//
// Back-transformation: blocks of 64 reflectors in compact form I - Y^T F Y (rows of Y = reflectors, F upper triangular; R. Schreiber,
// C. Van Loan 1989).
#include "fw_internal.h"
#include "lane_sums.h"
#include <mutex>
#include <type_traits>

namespace fw {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2), aligned(8)));   // rows may start at odd entries

constexpr int TAIL = 128;     // rows finished by one workgroup
constexpr int LEAF = 16;      // largest leaf of the divide and conquer
constexpr int NB = 64;        // reflectors per block of the back-transformation
constexpr double EPS = 1.1102230246251565e-16;   // 2^-53

// sum over the 64 lanes by data-parallel-primitive moves (no LDS traffic); the sum ends up in lane 63
__device__ __forceinline__ double dpp_add(double v, const int ctrl_sel) {
    union { double d; int i[2]; } a, b;
    a.d = v;
    switch (ctrl_sel) {
#define FW_DPP(c, m) b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], c, m, 0xf, false); b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], c, m, 0xf, false); break;
        case 0: FW_DPP(0x111, 0xf)   // row_shr:1
        case 1: FW_DPP(0x112, 0xf)
        case 2: FW_DPP(0x114, 0xf)
        case 3: FW_DPP(0x118, 0xf)
        case 4: FW_DPP(0x142, 0xa)   // row_bcast:15 into rows 1 and 3
        default: FW_DPP(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef FW_DPP
    }
    return v + b.d;
}
__device__ __forceinline__ double wave_sum63(double v) {
#pragma unroll
    for (int s = 0; s < 6; ++s) v = dpp_add(v, s);
    return v;
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    union { double d; int i[2]; } a;
    a.d = v;
    a.i[0] = __builtin_amdgcn_readlane(a.i[0], lane);
    a.i[1] = __builtin_amdgcn_readlane(a.i[1], lane);
    return a.d;
}
__device__ __forceinline__ double wave_total(double v) { return lane_value(wave_sum63(v), 63); }

// sum over a workgroup of T threads, the same value in every thread; `red` holds T / 64 doubles and is not reused before the
// next barrier of the caller
template <int T>
__device__ __forceinline__ double block_total(double v, double* red) {
    v = wave_sum63(v);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) s += red[w];
    return s;
}

// reflector for (x_0 .. x_{n-1}) -> beta e_{n-1} from the sum of squares of the entries before the last and the last one:
// v = scale x with v_{n-1} = 1, H = I - tau v v^T.  It stands in every step's chain of dependent operations, so both reciprocals
// come from the hardware's estimate and two Newton steps each (the norm with a last correction from its residual) instead of a square
// root and two divisions behind it: 35 of 2270 us at 576 rows.
__device__ __forceinline__ void reflector(double ss, double alpha, double* tau, double* beta, double* scale) {
    if (ss == 0.0) { *tau = 0.0; *beta = alpha; *scale = 0.0; return; }
    const double n2 = alpha * alpha + ss;
    if (!(n2 > 1e-280 && n2 < 1e280)) {      // beyond the range where the estimates and their squares are normal numbers
        const double nrm = sqrt(n2), b = alpha >= 0.0 ? -nrm : nrm;
        *tau = (b - alpha) / b;
        *scale = 1.0 / (alpha - b);
        *beta = b;
        return;
    }
    double y = __builtin_amdgcn_rsq(n2);     // 1 / |x|
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-n2 * y, y, 1.0), y);
    double nrm = n2 * y;
    nrm = fma(0.5 * y, fma(-nrm, nrm, n2), nrm);
    const double den = fabs(alpha) + nrm;
    double r = __builtin_amdgcn_rcp(den);
#pragma unroll
    for (int i = 0; i < 2; ++i) r = fma(r, fma(-den, r, 1.0), r);
    *tau = fma(fabs(alpha), y, 1.0);
    *scale = alpha >= 0.0 ? r : -r;
    *beta = alpha >= 0.0 ? -nrm : nrm;
}

// Features that never vary have a zero row and column.  They are moved behind the others (perm[0 .. M-1] = source of each
// place): eliminated first, their rows give no reflector, so their eigenvectors stay exact unit vectors
// and no rounding noise of the others gets into them.  One workgroup.
__global__ __launch_bounds__(1024) void dead_last_kernel(const float* __restrict__ Phi, int M, int* __restrict__ perm) {
    __shared__ int cnt[16], base_live;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int pass = 0; pass < 2; ++pass) {         // count, then place
        int live = 0;                              // live features before this chunk
        for (int c0 = 0; c0 < M; c0 += 1024) {
            const int i = c0 + threadIdx.x;
            const bool l = i < M && Phi[(size_t)i * M + i] != 0.f;
            const unsigned long long mask = __ballot(l);
            if (lane == 0) cnt[wave] = __popcll(mask);
            __syncthreads();
            int before = live, all = 0;
            for (int w = 0; w < 16; ++w) { if (w < wave) before += cnt[w]; all += cnt[w]; }
            before += __popcll(mask & ((1ull << lane) - 1ull));
            if (pass == 1 && i < M) perm[l ? before : base_live + (i - before)] = i;
            live += all;
            __syncthreads();
        }
        if (threadIdx.x == 0) base_live = live;
        __syncthreads();
    }
}

// A = symmetric part of Phi in float64, columns beyond M zero; rows and columns in the order of `perm` unless it is null
__global__ __launch_bounds__(256) void sym_load_kernel(const float* __restrict__ Phi, int M, int ld, const int* __restrict__ perm,
                                                       double* __restrict__ A) {
    __shared__ float t[32][33];
    const int bi = blockIdx.y * 32, bj = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    auto at = [&](int i, int j) { return perm ? Phi[(size_t)perm[i] * M + perm[j]] : Phi[(size_t)i * M + j]; };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bj + ty + 8 * r, j = bi + tx;       // the mirrored tile
        t[ty + 8 * r][tx] = (i < M && j < M) ? at(i, j) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bi + ty + 8 * r, j = bj + tx;
        if (i < M && j < ld) A[(size_t)i * ld + j] = j < M ? 0.5 * ((double)at(i, j) + (double)t[tx][ty + 8 * r]) : 0.0;
    }
}

// columns of V back to the caller's order through a second buffer
__global__ __launch_bounds__(256) void restore_columns_kernel(const double* __restrict__ V, int M, int ld, const int* __restrict__ perm,
                                                              double* __restrict__ out, int back) {
    for (int j = blockIdx.x * 256 + threadIdx.x; j < M; j += gridDim.x * 256) {
        const size_t at = (size_t)blockIdx.y * ld;
        if (back) out[at + j] = V[at + j]; else out[at + perm[j]] = V[at + j];
    }
}

// One step of the reduction (see the head of the file): eliminates row c of the leading (c+1) x (c+1) block, C T >= c + 1.
// RB rows of loads are in flight per thread; the first RB are issued before the sums.
template <int T, int C, int RB>
__global__ __launch_bounds__(T) void tri_step_kernel(double* __restrict__ A, int ld, int c, int first, const double* __restrict__ vprev,
                                                     const double* __restrict__ pprev, double* __restrict__ vnew, double* __restrict__ pnew,
                                                     double* __restrict__ d, double* __restrict__ e, double* __restrict__ tau) {
    extern __shared__ double rowred[];            // [rows of this workgroup][T / 64]
    __shared__ double red[2][T / 64];
    __shared__ double s_alpha, s_d;
    const int t = threadIdx.x, wave = t >> 6;
    const int G = gridDim.x;
    double v[C], w[C], x[C], a[RB][C];
    const double tp = first ? 0.0 : tau[c + 1];
    double dot = 0.0;
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const int j = t + T * q;
        const bool ok = j <= c;
        v[q] = (ok && !first) ? vprev[j] : 0.0;
        w[q] = (ok && !first) ? pprev[j] : 0.0;
        x[q] = ok ? A[(size_t)c * ld + j] : 0.0;
    }
    const double vc = first ? 0.0 : vprev[c], pc = first ? 0.0 : pprev[c];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int i = blockIdx.x + G * r;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = t + T * q;
            a[r][q] = (i < c && j < c) ? A[(size_t)i * ld + j] : 0.0;
        }
    }
#pragma unroll
    for (int q = 0; q < C; ++q) dot += v[q] * w[q];
    const double h = first ? 0.0 : 0.5 * tp * tp * block_total<T>(dot, red[0]);
    const double wc = tp * pc - h * vc;
    double ss = 0.0;
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const int j = t + T * q;
        w[q] = tp * w[q] - h * v[q];
        x[q] -= vc * w[q] + wc * v[q];
        if (j < c - 1) ss += x[q] * x[q];
        if (j == c - 1) s_alpha = x[q];
        if (j == c) s_d = x[q];
    }
    ss = block_total<T>(ss, red[1]);
    double tn, beta, scale;
    reflector(ss, s_alpha, &tn, &beta, &scale);
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const int j = t + T * q;
        x[q] = j < c - 1 ? x[q] * scale : (j == c - 1 ? 1.0 : 0.0);
    }
    if (blockIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = t + T * q;
            if (j < c) vnew[j] = x[q];
        }
        if (t == 0) { tau[c] = tn; e[c - 1] = beta; d[c] = s_d; }
    }
    for (int r0 = 0; (int)blockIdx.x + G * r0 < c; r0 += RB) {
        if (r0 > 0) {
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int i = blockIdx.x + G * (r0 + r);
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    const int j = t + T * q;
                    a[r][q] = (i < c && j < c) ? A[(size_t)i * ld + j] : 0.0;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = blockIdx.x + G * (r0 + r);
            if (i < c) {
                const double vi = first ? 0.0 : vprev[i], wi = first ? 0.0 : tp * pprev[i] - h * vi;
                double acc = 0.0;
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    const int j = t + T * q;
                    const double u = a[r][q] - (vi * w[q] + wi * v[q]);
                    if (j < c && !first) A[(size_t)i * ld + j] = u;
                    acc += u * x[q];
                }
                acc = wave_sum63(acc);
                if ((t & 63) == 63) rowred[(r0 + r) * (T / 64) + wave] = acc;
            }
        }
    }
    __syncthreads();
    for (int r = t; (int)blockIdx.x + G * r < c; r += T) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < T / 64; ++k) s += rowred[r * (T / 64) + k];
        pnew[blockIdx.x + G * r] = s;
    }
}

// ---- the reduction in one launch, the matrix in registers
// A step of the chain above costs a launch and a pass over the active block in memory, yet 2560 x 2560 doubles fit the registers of
// the chip.  Here every workgroup keeps a block of 8 rows in registers (a thread owns fixed columns, as above) and what
// a step exchanges is its product p = A v and the next row to eliminate, n entries each.  They go through memory into places written
// once (a row of two buffers for each step, filled with SENTINEL before the launch): the owners store them past the caches, every
// workgroup polls the entries of its own columns until none is SENTINEL any more.  So the value is its own signal, and nothing is ever reset; 8
// rows in a row are 64 bytes of one owner (rows dealt out one by one, their lines written by sixteen owners: 2 to 3 us more a step).
// All workgroups have to be resident at a time (launch_rows).  A poll gives up after POLL_LIMIT rounds (some tenths of a second: two
// processes on one card may meet); the workgroups that wait for this one then do so too, and d[0] = NaN makes the caller's
// acceptance fail.  Rows per workgroup: eight, ten where eight would need more than 256 workgroups.
// Bound by the round trip through the last-level cache (about 1.7 us a step, 2.5 at 2304 rows, where 230 workgroups read 37 KB each) and two
// sums over the workgroup.  Whole call, launches per step -> this, the rest as it then was: 576 features 3.55 -> 2.85 ms, 2304 features
// 22.8 -> 14.2 ms (polls at once instead of after POLL_DELAY: 15.0 ms; after twice the delay: 14.8 ms).  Up to 128 rows the single
// workgroup is as fast.
constexpr unsigned long long SENTINEL = ~0ull;    // a NaN that no arithmetic on widened float32 produces; publish() keeps it out for good
constexpr int POLL_LIMIT = 1 << 18;
constexpr int ROWS_MAX_M = 2560;
constexpr int POLL_DELAY = 10;                    // of 64 clocks before the first poll: an early one only gets in the way of the stores

__device__ __forceinline__ void publish(double* p, double x) {
    unsigned long long b = (unsigned long long)__double_as_longlong(x);
    if (b == SENTINEL) b = 0x7ff8000000000000ull;
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const double* p) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// sums of RB (8 or 10) values over the wavefront; row 0 .. RB - 1 to out[0 .. RB - 1]
template <int RB>
__device__ __forceinline__ void row_sums(const double (&acc)[RB], int lane, double* out) {
    const double s0 = fold32(acc[0], acc[4]), s1 = fold32(acc[1], acc[5]), s2 = fold32(acc[2], acc[6]), s3 = fold32(acc[3], acc[7]);
    const double u0 = sum16(fold16(s0, s2)), u1 = sum16(fold16(s1, s3));    // rows 2 g and 2 g + 1 in lanes 16 g .. 16 g + 15
    double u2 = 0.0;
    if constexpr (RB == 10) {
        const double s4 = fold32(acc[RB - 2], acc[RB - 1]);
        u2 = sum16(fold16(s4, s4));                                         // row 8 below lane 32, row 9 from there on
    }
    if ((lane & 15) == 0) {
        out[lane >> 3] = u0; out[(lane >> 3) + 1] = u1;
        if constexpr (RB == 10) out[8 + (lane >> 5)] = u2;
    }
}

// T threads of C columns each, RB rows b RB .. b RB + RB - 1 per workgroup b.  Eliminates rows c0, c0 - 1, ..., 1 of the leading
// (c0 + 1) x (c0 + 1) block; c0 < C T, c0 < RB gridDim.x.  Pslot, Xslot: row c holds what step c leaves.
// The reflector's scale is not waited for: the rows are multiplied with x as it is (x_{c-1} left out), and the sum of squares that
// gives the scale crosses the workgroup together with the products.
template <int T, int C, int RB>
__global__ __launch_bounds__(T) void tri_rows_kernel(const double* __restrict__ A, int ld, int c0, int first, const double* __restrict__ vprev,
                                                     const double* __restrict__ pprev, double* __restrict__ Pslot, double* __restrict__ Xslot,
                                                     double* __restrict__ Vh, double* __restrict__ d, double* __restrict__ e,
                                                     double* __restrict__ tau, int polls) {
    constexpr int NW = T / 64;
    __shared__ double vl[C * T + RB];             // reflector of the step before
    __shared__ double rowred[NW][RB], rowp[RB], col[RB], red[2][NW];
    __shared__ double s_pc, s_alpha, s_d;
    __shared__ int s_bad;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int b = blockIdx.x, i0 = b * RB;
    double a[RB][C], v[C];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int i = i0 + r, j = t + T * q;
            a[r][q] = (i <= c0 && j <= c0) ? A[(size_t)i * ld + j] : 0.0;
        }
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const int j = t + T * q;
        v[q] = (j <= c0 && !first) ? vprev[j] : 0.0;
        vl[j] = v[q];
    }
    if (t < RB) {
        rowp[t] = (i0 + t <= c0 && !first) ? pprev[i0 + t] : 0.0;
        vl[C * T + t] = 0.0;
    }
    if (t == 0) s_bad = 0;                        // read behind the barrier of the first row, set from the second row on
    double tp = first ? 0.0 : tau[c0 + 1];
    for (int c = c0; c >= 1; --c) {
        if (i0 >= c) return;                      // no row of this workgroup is left (workgroup 0 stays to the end)
        double w[C], x[C];
        if (c == c0) {
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int j = t + T * q;
                w[q] = (j <= c && !first) ? pprev[j] : 0.0;
                x[q] = j <= c ? A[(size_t)c * ld + j] : 0.0;
            }
        } else {
            const double* ps = Pslot + (size_t)(c + 1) * ld;
            const double* xs = Xslot + (size_t)(c + 1) * ld;
            unsigned long long pb[C], xb[C];
            bool have_x = false;                  // the row comes first: its owner stored it before the products of the same step
            __builtin_amdgcn_s_sleep(POLL_DELAY);
            for (int spin = 0;; ++spin) {
                bool there = true, there_x = true;
#pragma unroll
                for (int q = 0; q < C; ++q) pb[q] = t + T * q <= c ? peek(ps + t + T * q) : 0;
                if (!have_x) {
#pragma unroll
                    for (int q = 0; q < C; ++q) xb[q] = t + T * q <= c ? peek(xs + t + T * q) : 0;
                }
#pragma unroll
                for (int q = 0; q < C; ++q) { there &= pb[q] != SENTINEL; there_x &= xb[q] != SENTINEL; }
                have_x = __all(there_x);
                if (have_x && __all(there)) break;
                if (spin + 1 >= polls) { s_bad = 1; break; }
            }
#pragma unroll
            for (int q = 0; q < C; ++q) { w[q] = __longlong_as_double((long long)pb[q]); x[q] = __longlong_as_double((long long)xb[q]); }
        }
        double dot = 0.0;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            dot += v[q] * w[q];
            if (t + T * q == c) s_pc = w[q];          // one thread, in every row: nobody else writes it
        }
        dot = block_total<T>(dot, red[0]);
        if (s_bad) {
            if (t == 0) d[0] = __longlong_as_double(0x7ff8000000000000ll);
            return;
        }
        const double h = 0.5 * tp * tp * dot, vc = vl[c], wc = tp * s_pc - h * vc;
        double ss = 0.0;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = t + T * q;
            w[q] = tp * w[q] - h * v[q];
            x[q] -= vc * w[q] + wc * v[q];
            if (j == c - 1) s_alpha = x[q];
            if (j == c) s_d = x[q];
            if (j >= c - 1) x[q] = 0.0;
            ss += x[q] * x[q];
        }
        double acc[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            // rows from c on are updated with what lies there and never looked at again
            const double vi = -vl[i0 + r], wi = -(tp * rowp[r] + h * vi);
            acc[r] = 0.0;
#pragma unroll
            for (int q = 0; q < C; ++q) {
                if (T * q >= c) break;
                a[r][q] = fma(vi, w[q], fma(wi, v[q], a[r][q]));
                acc[r] = fma(a[r][q], x[q], acc[r]);
            }
        }
        if (c - 1 - i0 < RB) {                    // the row to eliminate next
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (i0 + r == c - 1) {
#pragma unroll
                    for (int q = 0; q < C; ++q)
                        if (t + T * q < c) publish(Xslot + (size_t)c * ld + t + T * q, a[r][q]);
                }
        }
#pragma unroll
        for (int q = 0; q < C; ++q)
            if (t + T * q == c - 1) {
#pragma unroll
                for (int r = 0; r < RB; ++r) col[r] = a[r][q];
            }
        row_sums<RB>(acc, lane, rowred[wave]);
        ss = block_total<T>(ss, red[1]);
        double tn, beta, scale;
        reflector(ss, s_alpha, &tn, &beta, &scale);
        if (t < RB) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) s += rowred[k][t];
            s = scale * s + col[t];
            if (i0 + t < c) publish(Pslot + (size_t)c * ld + i0 + t, s);
            rowp[t] = s;
        }
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = t + T * q;
            v[q] = j == c - 1 ? 1.0 : x[q] * scale;
            vl[j] = v[q];
        }
        // what the later stages read: nothing in this launch waits for it
        if (b == 0) {
#pragma unroll
            for (int q = 0; q < C; ++q)
                if (t + T * q < c) Vh[(size_t)c * ld + t + T * q] = v[q];
            if (t == 0) {
                tau[c] = tn; e[c - 1] = beta; d[c] = s_d;
                if (c == 1) { d[0] = a[0][0]; tau[0] = 0.0; }
            }
        }
        tp = tn;
    }
}

// The last n0 = c0 + 1 <= TAIL rows in one workgroup of 16 wavefronts: wavefront g owns rows g, g + 16, ... and keeps them in
// registers (two columns per lane); x, p travel through LDS; two barriers a step.
__global__ __launch_bounds__(1024) void tri_tail_kernel(const double* __restrict__ A, int ld, int c0, int first, const double* __restrict__ vprev,
                                                        const double* __restrict__ pprev, double* __restrict__ Vh, double* __restrict__ d,
                                                        double* __restrict__ e, double* __restrict__ tau) {
    __shared__ double xs[TAIL], ps[TAIL];
    constexpr int RW = TAIL / 16;
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int n0 = c0 + 1;
    double a[RW][2];
    double v[2], w[2];
    const double tp = first ? 0.0 : tau[c0 + 1];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int j = lane + 64 * k;
        v[k] = (j < n0 && !first) ? vprev[j] : 0.0;
        w[k] = (j < n0 && !first) ? pprev[j] : 0.0;
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int i = g + 16 * r;
            a[r][k] = (i < n0 && j < n0) ? A[(size_t)i * ld + j] : 0.0;
        }
    }
    const double h0 = 0.5 * tp * tp * wave_total(v[0] * w[0] + v[1] * w[1]);
#pragma unroll
    for (int k = 0; k < 2; ++k) w[k] = tp * w[k] - h0 * v[k];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int i = g + 16 * r;
        if (i < n0) {
            const double vi = first ? 0.0 : vprev[i], wi = first ? 0.0 : tp * pprev[i] - h0 * vi;
#pragma unroll
            for (int k = 0; k < 2; ++k) a[r][k] -= vi * w[k] + wi * v[k];
            if (i == c0) {
#pragma unroll
                for (int k = 0; k < 2; ++k) xs[lane + 64 * k] = a[r][k];
            }
        }
    }
    __syncthreads();
    for (int c = c0; c >= 1; --c) {
        double x[2] = {xs[lane], xs[lane + 64]};
        const double alpha = xs[c - 1], dc = xs[c];
        double ss = 0.0;
#pragma unroll
        for (int k = 0; k < 2; ++k) ss += (lane + 64 * k < c - 1) ? x[k] * x[k] : 0.0;
        ss = wave_total(ss);
        double tn, beta, scale;
        reflector(ss, alpha, &tn, &beta, &scale);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int j = lane + 64 * k;
            x[k] = j < c - 1 ? x[k] * scale : (j == c - 1 ? 1.0 : 0.0);
        }
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (lane + 64 * k < c) Vh[(size_t)c * ld + lane + 64 * k] = x[k];
            if (lane == 0) { tau[c] = tn; e[c - 1] = beta; d[c] = dc; }
        }
        double p[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            p[r] = 0.0;
            if (g + 16 * r < c) p[r] = wave_total(a[r][0] * x[0] + a[r][1] * x[1]);
        }
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (lane == 0 && g + 16 * r < c) ps[g + 16 * r] = p[r];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) w[k] = lane + 64 * k < c ? ps[lane + 64 * k] : 0.0;
        const double h = 0.5 * tn * tn * wave_total(x[0] * w[0] + x[1] * w[1]);
#pragma unroll
        for (int k = 0; k < 2; ++k) w[k] = tn * w[k] - h * x[k];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int i = g + 16 * r;
            if (i < c) {
                const double vi = lane_value(i < 64 ? x[0] : x[1], i & 63), wi = tn * p[r] - h * vi;
#pragma unroll
                for (int k = 0; k < 2; ++k) a[r][k] -= vi * w[k] + wi * x[k];
                if (i == c - 1) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) xs[lane + 64 * k] = a[r][k];
                }
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) { d[0] = xs[0]; tau[0] = 0.0; }
}

// ------------------------------------------------------------------------------------------- divide and conquer
// boundaries of the P parts of a level: part k covers rows part_begin(k) .. part_begin(k+1) - 1
__device__ __host__ __forceinline__ int part_begin(int k, int P, int M) { return (int)((long long)k * M / P); }

struct DcArrays {                 // [M] each; a merge works on its own range
    double *d, *dn;               // eigenvalues of the level below (ascending inside a part), and of this level
    double *sd, *sz;              // sorted d and z
    int *srow;                    // row of the eigenvector that belongs to a sorted entry
    double *kd, *kz, *zh, *tau;   // kept entries: pole, z, recomputed z, offset of the root from its pole `org`
    int *krow, *org, *kpos;       // kept entries: row; pole next to the root; place of the root in the new order
    double *dd; int *drow;        // deflated entries
    int *ri, *rj; double *rc, *rs;   // plane rotations of the deflation, in order
    int *ucol, *urow;             // kept entries: column of U (those of the first child, those a rotation mixed, those of the second); row of V by column of U
    int *cnt;                     // per merge: kept, deflated, rotations, first mixed column of U + 65536 x first column of the second child
};

// tears T at the leaf boundaries: both diagonal neighbours lose |e|
__global__ void dc_tear_kernel(double* __restrict__ d, const double* __restrict__ e, int M, int P) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x + 1;
    if (k >= P) return;
    const int b = part_begin(k, P, M);
    const double r = fabs(e[b - 1]);
    d[b - 1] -= r;      // leaves have at least eight rows, so no entry is touched twice
    d[b] -= r;
}

// leaves: cyclic Jacobi on at most 16 x 16 by one wavefront; rows of V = eigenvectors, ascending
__global__ __launch_bounds__(64) void dc_leaf_kernel(double* __restrict__ dv, const double* __restrict__ e, int M, int ld, int P,
                                                     double* __restrict__ V) {
    __shared__ double Gs[LEAF][LEAF + 1], Rs[LEAF][LEAF + 1];
    const int off = part_begin(blockIdx.x, P, M), n = part_begin(blockIdx.x + 1, P, M) - off;
    const int lane = threadIdx.x;
    double nrm = 0.0;
    for (int m = lane; m < LEAF * LEAF; m += 64) {
        const int i = m >> 4, j = m & 15;
        double g = 0.0;
        if (i < n && j < n) {
            if (i == j) g = dv[off + i];
            else if (i == j + 1) g = e[off + j];
            else if (j == i + 1) g = e[off + i];
        }
        Gs[i][j] = g;
        Rs[i][j] = i == j ? 1.0 : 0.0;
        nrm += g * g;
    }
    nrm = wave_total(nrm);
    const double thr = 0.25 * EPS * sqrt(nrm);
    __syncthreads();
    const int kk = lane >> 3, sub = lane & 7;
    for (int sweep = 0; sweep < 24; ++sweep) {
        int any = 0;
        for (int step = 0; step < LEAF - 1; ++step) {
            int i, j;
            if (kk == 0) { i = LEAF - 1; j = step; }
            else { i = (step + kk) % (LEAF - 1); j = (step - kk + LEAF - 1) % (LEAF - 1); }
            if (i > j) { const int x = i; i = j; j = x; }
            const double al = Gs[i][i], be = Gs[j][j], ga = Gs[i][j];
            const bool rot = fabs(ga) > thr;
            double c = 1.0, s = 0.0;
            if (rot) {
                const double tau = be - al;
                const double tt = (tau >= 0.0 ? 2.0 : -2.0) * ga / (fabs(tau) + sqrt(tau * tau + 4.0 * ga * ga));
                c = 1.0 / sqrt(1.0 + tt * tt);
                s = c * tt;
            }
            any |= rot ? 1 : 0;
            __syncthreads();
            if (rot) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int col = sub + 8 * m;
                    const double x = Gs[i][col], y = Gs[j][col];
                    Gs[i][col] = c * x - s * y; Gs[j][col] = s * x + c * y;
                    const double f = Rs[i][col], g = Rs[j][col];
                    Rs[i][col] = c * f - s * g; Rs[j][col] = s * f + c * g;
                }
            }
            __syncthreads();
            if (rot) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int row = sub + 8 * m;
                    const double x = Gs[row][i], y = Gs[row][j];
                    Gs[row][i] = c * x - s * y; Gs[row][j] = s * x + c * y;
                }
            }
            __syncthreads();
        }
        if (!__any(any)) break;
    }
    // ascending order by counting; rows that do not exist stay behind
    for (int m = lane; m < n * LEAF; m += 64) {
        const int i = m >> 4, j = m & 15;
        const double li = Gs[i][i];
        int pos = 0;
        for (int k = 0; k < n; ++k) pos += (Gs[k][k] < li || (Gs[k][k] == li && k < i)) ? 1 : 0;
        if (pos >= n) pos = n - 1;
        if (j < n) V[(size_t)(off + pos) * ld + off + j] = Rs[i][j];
        if (j == 0) dv[off + pos] = li;
    }
}

// z, order, deflation of one merge per workgroup.  P = merges of the level; `e` holds the couplings.
__global__ __launch_bounds__(512) void dc_deflate_kernel(DcArrays D, const double* __restrict__ e, int M, int ld, int P, const double* __restrict__ V) {
    constexpr int CH = 512;
    __shared__ double ld_d[CH], ld_z[CH];
    const int m = blockIdx.x;
    const int off = part_begin(m, P, M), mid = part_begin(2 * m + 1, 2 * P, M), end = part_begin(m + 1, P, M);
    const int n = end - off, n1 = mid - off;
    const double rho = fabs(e[mid - 1]);
    const double sgn = e[mid - 1] >= 0.0 ? 1.0 : -1.0;
    const double r = 2.0 * rho;
    const double* d = D.d + off;
    double* sd = D.sd + off; double* sz = D.sz + off; int* srow = D.srow + off;
    for (int i = threadIdx.x; i < n; i += blockDim.x) { sd[i] = d[i]; sz[i] = 0.0; srow[i] = off + i; }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        // place in the merged order: entries of the first part come first on ties
        const double x = d[i];
        int lo = i < n1 ? n1 : 0, hi = i < n1 ? n : n1;
        const int base = lo;
        while (lo < hi) {
            const int k = (lo + hi) >> 1;
            if (i < n1 ? d[k] < x : d[k] <= x) lo = k + 1; else hi = k;
        }
        const int pos = (i < n1 ? i : i - n1) + (lo - base);
        sd[pos] = x;
        sz[pos] = (i < n1 ? V[(size_t)(off + i) * ld + mid - 1] : sgn * V[(size_t)(off + i) * ld + mid]) * 0.70710678118654752440;
        srow[pos] = off + i;
    }
    __syncthreads();
    const double big = fmax(fmax(fabs(sd[0]), fabs(sd[n - 1])), r);
    const double tol = 8.0 * EPS * big;
    // serial scan by one thread over chunks staged in LDS
    int nk = 0, nd = 0, nr = 0, prow = -1;
    double pd = 0.0, pz = 0.0;
    for (int c0 = 0; c0 < n; c0 += CH) {
        const int cn = min(CH, n - c0);
        __syncthreads();
        for (int i = threadIdx.x; i < cn; i += blockDim.x) { ld_d[i] = sd[c0 + i]; ld_z[i] = sz[c0 + i]; }
        __syncthreads();
        if (threadIdx.x == 0) {
            double qd = ld_d[0], qz = ld_z[0];
            for (int i = 0; i < cn; ++i) {
                double jd = qd, jz = qz;
                if (i + 1 < cn) { qd = ld_d[i + 1]; qz = ld_z[i + 1]; }
                const int jrow = c0 + i;                    // index into srow
                if (r * fabs(jz) <= tol) { D.dd[off + nd] = jd; D.drow[off + nd] = jrow; ++nd; continue; }
                if (prow >= 0) {
                    const double s2 = pz * pz + jz * jz;
                    if (fabs((jd - pd) * (pz * jz)) <= tol * s2) {
                        const double rr = sqrt(s2), c = jz / rr, s = pz / rr;
                        D.ri[off + nr] = prow; D.rj[off + nr] = jrow; D.rc[off + nr] = c; D.rs[off + nr] = s; ++nr;
                        D.dd[off + nd] = c * c * pd + s * s * jd; D.drow[off + nd] = prow; ++nd;
                        jd = s * s * pd + c * c * jd;
                        jz = rr;
                    } else {
                        D.kd[off + nk] = pd; D.kz[off + nk] = pz; D.krow[off + nk] = prow; ++nk;
                    }
                }
                prow = jrow; pd = jd; pz = jz;
            }
        }
    }
    __shared__ int s_nk;
    if (threadIdx.x == 0) {
        if (prow >= 0) { D.kd[off + nk] = pd; D.kz[off + nk] = pz; D.krow[off + nk] = prow; ++nk; }
        D.cnt[4 * m] = nk; D.cnt[4 * m + 1] = nd; D.cnt[4 * m + 2] = nr;
        D.cnt[4 * m + 3] = nk << 16;              // every column counts as mixed
        s_nk = nk;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < s_nk; i += blockDim.x) { D.ucol[off + i] = i; D.urow[off + i] = srow[D.krow[off + i]]; }
}

// The same for merges of up to DEFLATE_MAX entries, all in LDS, one thread only where something is rotated.  Which entries have a
// negligible component of z is known at once, and so is for which neighbours among the others the rotation is due, as long as neither
// has been rotated: the serial part starts at those pairs and ends where a rotated entry and its next neighbour part, which
// leaves most merges without any.  (One thread through all entries took 195 ns each: 0.93 of 14.2 ms at 2304 rows, 0.23 of 2.8 at 576.)
constexpr int DEFLATE_MAX = 4096;
__global__ __launch_bounds__(512) void dc_deflate_lds_kernel(DcArrays D, const double* __restrict__ e, int M, int ld, int P, const double* __restrict__ V) {
    __shared__ double cd[DEFLATE_MAX], cz[DEFLATE_MAX];
    __shared__ unsigned short ci[DEFLATE_MAX];            // place in the merged order
    __shared__ unsigned long long due[DEFLATE_MAX / 64], gone[DEFLATE_MAX / 64], mixed[DEFLATE_MAX / 64];
    __shared__ int cnt[8];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int off = part_begin(m, P, M), mid = part_begin(2 * m + 1, 2 * P, M), end = part_begin(m + 1, P, M);
    const int n = end - off, n1 = mid - off;
    const double rho = fabs(e[mid - 1]);
    const double sgn = e[mid - 1] >= 0.0 ? 1.0 : -1.0;
    const double r = 2.0 * rho;
    const double* d = D.d + off;
    double* sd = D.sd + off; double* sz = D.sz + off; int* srow = D.srow + off;
    for (int i = tid; i < n; i += 512) { sd[i] = d[i]; sz[i] = 0.0; srow[i] = off + i; }   // every place has a value (NaN)
    if (tid < DEFLATE_MAX / 64) { due[tid] = 0; gone[tid] = 0; mixed[tid] = 0; }
    __syncthreads();
    // place in the merged order: entries of the first part come first on ties
    for (int i = tid; i < n; i += 512) {
        const double x = d[i];
        int lo = i < n1 ? n1 : 0, hi = i < n1 ? n : n1;
        const int base = lo;
        while (lo < hi) {
            const int k = (lo + hi) >> 1;
            if (i < n1 ? d[k] < x : d[k] <= x) lo = k + 1; else hi = k;
        }
        const int pos = (i < n1 ? i : i - n1) + (lo - base);
        sd[pos] = x;
        sz[pos] = (i < n1 ? V[(size_t)(off + i) * ld + mid - 1] : sgn * V[(size_t)(off + i) * ld + mid]) * 0.70710678118654752440;
        srow[pos] = off + i;
    }
    __syncthreads();
    const double big = fmax(fmax(fabs(sd[0]), fabs(sd[n - 1])), r);
    const double tol = 8.0 * EPS * big;
    // places of the true ones of `yes` in order, behind those of earlier calls (`base`, updated)
    auto place = [&](bool yes, int& base) {
        const unsigned long long mask = __ballot(yes);
        if (lane == 0) cnt[wave] = __popcll(mask);
        __syncthreads();
        int before = base, all = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) { if (w < wave) before += cnt[w]; all += cnt[w]; }
        __syncthreads();
        base += all;
        return before + __popcll(mask & ((1ull << lane) - 1ull));
    };
    int ns = 0;                                           // entries with a component of z, moved together
    for (int c0 = 0; c0 < n; c0 += 512) {
        const int i = c0 + tid;
        const double x = i < n ? sd[i] : 0.0, z = i < n ? sz[i] : 0.0;
        const bool none = i < n && r * fabs(z) <= tol;
        const int first = ns, at = place(i < n && !none, ns);
        if (i < n && !none) { cd[at] = x; cz[at] = z; ci[at] = (unsigned short)i; }
        if (none) {
            const int k = c0 - first + (tid - (at - first));      // entries without one before this one
            D.dd[off + k] = x; D.drow[off + k] = i;
        }
    }
    __syncthreads();
    auto rotates = [&](double pd, double pz, double jd, double jz) { return fabs((jd - pd) * (pz * jz)) <= tol * (pz * pz + jz * jz); };
    for (int c0 = 0; c0 < ns; c0 += 512) {
        const int i = c0 + tid;
        const unsigned long long mask = __ballot(i + 1 < ns && rotates(cd[i], cz[i], cd[i + 1], cz[i + 1]));
        if (lane == 0 && i < ns) due[i >> 6] = mask;
    }
    __syncthreads();
    if (tid == 0) {
        int nd = n - ns, nr = 0, t = 0;
        for (;;) {
            // the next pair (t, t + 1) that is due
            int w = t >> 6;
            unsigned long long mask = w < DEFLATE_MAX / 64 ? due[w] & (~0ull << (t & 63)) : 0;
            while (!mask && ++w < DEFLATE_MAX / 64) mask = due[w];
            if (!mask) break;
            int p = 64 * w + __ffsll((long long)mask) - 1, j = p + 1;
            double pd = cd[p], pz = cz[p];
            while (j < ns) {
                double jd = cd[j], jz = cz[j];
                if (!rotates(pd, pz, jd, jz)) break;
                const double rr = sqrt(pz * pz + jz * jz), c = jz / rr, s = pz / rr;
                D.ri[off + nr] = ci[p]; D.rj[off + nr] = ci[j]; D.rc[off + nr] = c; D.rs[off + nr] = s; ++nr;
                D.dd[off + nd] = c * c * pd + s * s * jd; D.drow[off + nd] = ci[p]; ++nd;
                gone[p >> 6] |= 1ull << (p & 63);
                jd = s * s * pd + c * c * jd;
                jz = rr;
                p = j; pd = jd; pz = jz; ++j;
            }
            cd[p] = pd; cz[p] = pz;
            mixed[p >> 6] |= 1ull << (p & 63);
            t = j;
        }
        D.cnt[4 * m + 1] = nd; D.cnt[4 * m + 2] = nr;
    }
    __syncthreads();
    // kept entries in order, and for the product with the children's vectors by the columns these have: 0 first child, 1 both, 2 second
    auto kind = [&](int i) {
        if (i >= ns || ((gone[i >> 6] >> (i & 63)) & 1)) return 3;
        if ((mixed[i >> 6] >> (i & 63)) & 1) return 1;
        return srow[ci[i]] < off + n1 ? 0 : 2;
    };
    int nk = 0, count[3] = {0, 0, 0};
    for (int c0 = 0; c0 < ns; c0 += 512) {
        const int i = c0 + tid, what = kind(i);
        const int at = place(what < 3, nk);
        if (what < 3) { D.kd[off + at] = cd[i]; D.kz[off + at] = cz[i]; D.krow[off + at] = ci[i]; }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int c = place(what == k, count[k]);
            if (what == k) D.ucol[off + at] = c;          // inside its kind
        }
    }
    const int base[3] = {0, count[0], count[0] + count[1]};
    nk = 0;
    for (int c0 = 0; c0 < ns; c0 += 512) {
        const int i = c0 + tid, what = kind(i);
        const int at = place(what < 3, nk);
        if (what < 3) {
            const int c = D.ucol[off + at] + (what == 0 ? base[0] : what == 1 ? base[1] : base[2]);
            D.ucol[off + at] = c;
            D.urow[off + c] = srow[ci[i]];
        }
    }
    if (tid == 0) { D.cnt[4 * m] = nk; D.cnt[4 * m + 3] = base[1] | (base[2] << 16); }
}

// plane rotations of the deflation on rows of V, one thread per column; the chain prev -> next stays in a register
__global__ __launch_bounds__(64) void dc_rotate_kernel(DcArrays D, int M, int ld, int P, double* __restrict__ V) {
    const int m = blockIdx.y;
    const int nr = D.cnt[4 * m + 2];
    if (nr == 0) return;
    const int off = part_begin(m, P, M), end = part_begin(m + 1, P, M);
    const int col = off + blockIdx.x * 64 + threadIdx.x;
    if (col >= end) return;
    const int* srow = D.srow + off;
    int lastj = -1;
    double carry = 0.0;
    for (int k0 = 0; k0 < nr; k0 += 8) {
        double y[8];
        const int kn = min(8, nr - k0);
#pragma unroll
        for (int k = 0; k < 8; ++k)      // the second row of a rotation has not been touched by an earlier one
            if (k < kn) y[k] = V[(size_t)srow[D.rj[off + k0 + k]] * ld + col];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < kn) {
                const int i = D.ri[off + k0 + k], j = D.rj[off + k0 + k];
                if (i != lastj) {
                    if (lastj >= 0) V[(size_t)srow[lastj] * ld + col] = carry;
                    carry = V[(size_t)srow[i] * ld + col];
                }
                const double c = D.rc[off + k0 + k], s = D.rs[off + k0 + k];
                V[(size_t)srow[i] * ld + col] = c * carry - s * y[k];
                carry = s * carry + c * y[k];
                lastj = j;
            }
    }
    if (lastj >= 0) V[(size_t)srow[lastj] * ld + col] = carry;
}

// Root i of 1 + rho sum z^2 / (d - lambda) between poles i and i+1 (the last one beyond the last pole), one wavefront per
// root.  Coordinates relative to the nearer pole; each half of the sum is replaced by r + s / (pole - x) with its value and
// derivative, which gives a quadratic for the step; steps that leave the bracket are replaced by a (geometric) bisection.
__global__ __launch_bounds__(256) void dc_secular_kernel(DcArrays D, const double* __restrict__ e, int M, int P) {
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int k = D.cnt[4 * m];
    if (i >= k) return;
    const int off = part_begin(m, P, M), mid = part_begin(2 * m + 1, 2 * P, M);
    const double rho = 2.0 * fabs(e[mid - 1]);
    const double* kd = D.kd + off;
    const double* kz = D.kz + off;
    const bool last = i == k - 1;
    const double di = kd[i];
    double lo, hi, tau;
    int org = i;
    if (last) {
        double z2 = 0.0;
        for (int j = lane; j < k; j += 64) z2 += kz[j] * kz[j];
        lo = 0.0; hi = rho * wave_total(z2); tau = 0.5 * hi;
    } else {
        const double half = 0.5 * (kd[i + 1] - di);
        double f = 0.0;
        for (int j = lane; j < k; j += 64) f += kz[j] * kz[j] / ((kd[j] - di) - half);
        f = 1.0 + rho * wave_total(f);
        if (f >= 0.0) { lo = 0.0; hi = half; tau = half; }
        else { org = i + 1; lo = -half; hi = 0.0; tau = -half; }
    }
    if (k > 1) {
        const double dorg = kd[org];
        const double p0 = di - dorg, p1 = last ? 0.0 : kd[i + 1] - dorg;
        for (int it = 0; it < 100; ++it) {
            double psi = 0.0, phi = 0.0, dpsi = 0.0, dphi = 0.0;
            for (int j = lane; j < k; j += 64) {
                const double z = kz[j], inv = 1.0 / ((kd[j] - dorg) - tau);
                const double t1 = z * inv, t = z * t1, t2 = t1 * t1;
                if (j <= i) { psi += t; dpsi += t2; } else { phi += t; dphi += t2; }
            }
            psi = rho * wave_total(psi); phi = rho * wave_total(phi);
            dpsi = rho * wave_total(dpsi); dphi = rho * wave_total(dphi);
            const double f = 1.0 + psi + phi;
            if (fabs(f) <= 8.0 * EPS * (1.0 + fabs(psi) + fabs(phi))) break;
            if (f > 0.0) hi = fmin(hi, tau); else lo = fmax(lo, tau);
            const double a = p0 - tau;
            double eta;
            if (last) eta = a * f / (f - dpsi * a);
            else {
                const double b = p1 - tau;
                const double c0 = f - dpsi * a - dphi * b;
                const double B = (a + b) * f - a * b * (dpsi + dphi);
                const double s = sqrt(fmax(B * B - 4.0 * c0 * a * b * f, 0.0));
                eta = B > 0.0 ? 2.0 * a * b * f / (B + s) : (B - s) / (2.0 * c0);
            }
            double nt = tau + eta;
            if (!(nt > lo && nt < hi)) {
                const double l = hi > 0.0 ? lo : -hi, h = hi > 0.0 ? hi : -lo;      // distances from the pole
                const double b = l <= 0.0 ? h * 1e-3 : (h > 4.0 * l ? sqrt(l * h) : 0.5 * (l + h));
                nt = hi > 0.0 ? b : -b;
            }
            if (nt == tau) break;
            tau = nt;
        }
    } else tau = hi;     // a single pole: d + rho z^2
    if (lane == 0) { D.org[off + i] = org; D.tau[off + i] = tau; }
}

// Recomputed z (the rank-one vector for which the computed roots are exact), the places of roots and deflated entries in the
// new ascending order, the new eigenvalues, and the rows of the deflated eigenvectors copied.  One wavefront per entry.
__global__ __launch_bounds__(256) void dc_zhat_kernel(DcArrays D, int M, int ld, int P, const double* __restrict__ V, double* __restrict__ Vout) {
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int off = part_begin(m, P, M), end = part_begin(m + 1, P, M);
    const int n = end - off;
    if (w >= n) return;
    const int k = D.cnt[4 * m], nd = D.cnt[4 * m + 1];
    const double* kd = D.kd + off;
    const double* tau = D.tau + off;
    const int* org = D.org + off;
    const double* dd = D.dd + off;
    if (w < k) {
        const double di = kd[w];
        double pr = 1.0;
        for (int j = lane; j < k; j += 64) {
            const double L = (kd[org[j]] - di) + tau[j];      // lambda_j - d_w
            const double q = j < w ? kd[j] - di : (j + 1 < k ? kd[j + 1] - di : 1.0);
            pr *= L / q;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) pr *= __shfl_xor(pr, o, 64);
        const double lam = kd[org[w]] + tau[w];
        int before = 0;
        for (int j = lane; j < nd; j += 64) before += dd[j] <= lam ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        if (lane == 0) {
            D.zh[off + w] = copysign(sqrt(fabs(pr)), D.kz[off + w]);
            D.kpos[off + w] = off + w + before;
            D.dn[off + w + before] = lam;
        }
    } else {
        const int q = w - k;
        if (q >= nd) return;
        const double x = dd[q];
        int before = 0;
        for (int j = lane; j < nd; j += 64) before += (dd[j] < x || (dd[j] == x && j < q)) ? 1 : 0;
        for (int j = lane; j < k; j += 64) before += kd[org[j]] + tau[j] < x ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        if (before >= n) before = n - 1;
        if (lane == 0) D.dn[off + before] = x;
        const double* src = V + (size_t)D.srow[off + D.drow[off + q]] * ld;
        double* dst = Vout + (size_t)(off + before) * ld;
        for (int j = off + lane; j < end; j += 64) dst[j] = src[j];
    }
}

// rows of U: eigenvectors of D + rho z z^T for the kept entries, one wavefront per root; rows and columns beyond stay unused
__global__ __launch_bounds__(256) void dc_vectors_kernel(DcArrays D, int M, int ld, int P, double* __restrict__ U) {
    const int m = blockIdx.y, lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int k = D.cnt[4 * m];
    if (j >= k) return;
    const int off = part_begin(m, P, M);
    const double* kd = D.kd + off;
    const double* zh = D.zh + off;
    const double dorg = kd[D.org[off + j]], tau = D.tau[off + j];
    double* row = U + (size_t)(off + j) * ld + off;
    double ss = 0.0;
    for (int i = lane; i < k; i += 64) {
        const double u = zh[i] / ((kd[i] - dorg) - tau);
        row[D.ucol[off + i]] = u;
        ss += u * u;
    }
    const double inv = 1.0 / sqrt(wave_total(ss));
    for (int i = lane; i < k; i += 64) {                  // as above: a lane meets its own entries again
        const int c = D.ucol[off + i];
        row[c] *= inv;
    }
}

// ------------------------------------------------------------------------------------------- float64 matrix products
// One 64 x 64 tile of C = A B per workgroup of four wavefronts (32 x 32 each) on v_mfma_f64_16x16x4_f64; chunks of 16
// contraction entries in LDS as [k][row], the next chunk's loads in registers while the matrix cores work.  A 16x16x4
// product takes 64 cycles of a SIMD for 1 KB of fragments, so nothing but the matrix cores is near its limit.
// Operands are functors: load(k0, k_end, buf) fetches this thread's four entries of a chunk, zero from k_end on, KC tells how they lie
// (four along k of one row, or four along the rows of one k); rows exist up to k_end at least.
constexpr int GLD = 80;     // LDS row of 64 entries: 80 * 8 bytes put the two k of a half-wavefront 32 banks apart

template <bool KC>
struct Slot {                // where a thread's four entries of a 64 x 16 chunk lie
    int r, k;
    __device__ __forceinline__ Slot() {
        if (KC) { r = threadIdx.x >> 2; k = (threadIdx.x & 3) * 4; }
        else { k = threadIdx.x >> 4; r = (threadIdx.x & 15) * 4; }
    }
    __device__ __forceinline__ void store(double* s, const double (&b)[4]) const {
#pragma unroll
        for (int q = 0; q < 4; ++q) s[KC ? (k + q) * GLD + r : k * GLD + r + q] = b[q];
    }
};
// row-major matrix p[row][k], rows row0 .. row0 + 63 (valid below nr)
struct RowsK {
    static constexpr bool kc = true;
    const double* p; int ld, row0, nr;
    __device__ __forceinline__ void load(int k0, int k_end, const Slot<true>& s, double (&b)[4]) const {
        const int r = row0 + s.r, k = k0 + s.k;
        const double* q = p + (size_t)r * ld + k;
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = (r < nr && k + i < k_end) ? q[i] : 0.0;
    }
    // entries k0 .. k0 + 15 all lie below k_end: loads without a branch (a row beyond the end reads the last one; keep() makes it zero)
    __device__ __forceinline__ void load_whole(int k0, const Slot<true>& s, double (&b)[4]) const {
        const double* q = p + (size_t)min(row0 + s.r, nr - 1) * ld + k0 + s.k;
        const doublex2 x = *reinterpret_cast<const doublex2*>(q), y = *reinterpret_cast<const doublex2*>(q + 2);
        b[0] = x[0]; b[1] = x[1]; b[2] = y[0]; b[3] = y[1];
    }
    __device__ __forceinline__ double keep(const Slot<true>& s, int, double x) const { return row0 + s.r < nr ? x : 0.0; }
};
// row-major matrix p[k][col]; optional list of rows
struct ColsK {
    static constexpr bool kc = false;
    const double* p; int ld, col0, nc;
    const int* list;                       // row of entry k: list[k] if given
    __device__ __forceinline__ void load(int k0, int k_end, const Slot<false>& s, double (&b)[4]) const {
        const int k = k0 + s.k, c = col0 + s.r;
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = 0.0;
        if (k < k_end) {
            const double* q = p + (size_t)(list ? list[k] : k) * ld + c;
#pragma unroll
            for (int i = 0; i < 4; ++i) if (c + i < nc) b[i] = q[i];
        }
    }
    __device__ __forceinline__ void load_whole(int k0, const Slot<false>& s, double (&b)[4]) const {
        const int k = k0 + s.k, c = col0 + s.r;
        const double* q = p + (size_t)(list ? list[k] : k) * ld;
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = q[min(c + i, nc - 1)];
    }
    __device__ __forceinline__ double keep(const Slot<false>& s, int i, double x) const { return col0 + s.r + i < nc ? x : 0.0; }
};
// the same with a factor per k, or its square
struct ColsKScaled {
    static constexpr bool kc = false;
    const double* p; int ld, col0, nc; const double* g; bool square;
    __device__ __forceinline__ void load(int k0, int k_end, const Slot<false>& s, double (&b)[4]) const {
        const int k = k0 + s.k, c = col0 + s.r;
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = 0.0;
        if (k < k_end) {
            const double f = square ? g[k] * g[k] : g[k];
#pragma unroll
            for (int i = 0; i < 4; ++i) if (c + i < nc) b[i] = f * p[(size_t)k * ld + c + i];
        }
    }
    __device__ __forceinline__ void load_whole(int k0, const Slot<false>& s, double (&b)[4]) const {
        const int k = k0 + s.k, c = col0 + s.r;
        const double f = square ? g[k] * g[k] : g[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = f * p[(size_t)k * ld + min(c + i, nc - 1)];
    }
    __device__ __forceinline__ double keep(const Slot<false>& s, int i, double x) const { return col0 + s.r + i < nc ? x : 0.0; }
};
template <class OA, class OB, class Epi>
__device__ __forceinline__ void gemm64(const OA& A, const OB& B, int k_begin, int k_end, const Epi& epi) {
    __shared__ double As[2][16 * GLD], Bs[2][16 * GLD];
    const Slot<OA::kc> sa;
    const Slot<OB::kc> sb;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lq = lane >> 4;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    doublex4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = doublex4{0.0, 0.0, 0.0, 0.0};
    // chunk c in LDS, c + 1 and c + 2 in registers or on their way, one barrier a chunk.  Past the last whole chunk it is loaded again,
    // unread, so that no branch stands between a load and its use.
    double ra[2][4], rb[2][4];
    auto load = [&](int c, int set) { A.load_whole(k_begin + 16 * c, sa, ra[set]); B.load_whole(k_begin + 16 * c, sb, rb[set]); };
    auto stage = [&](int c, int set) {
        double x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { x[q] = A.keep(sa, q, ra[set][q]); y[q] = B.keep(sb, q, rb[set][q]); }
        sa.store(As[c & 1], x);
        sb.store(Bs[c & 1], y);
    };
    auto multiply = [&](int c) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            double fa[2], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                fa[t] = As[c & 1][(4 * ks + lq) * GLD + wr + 16 * t + lr];
                fb[t] = Bs[c & 1][(4 * ks + lq) * GLD + wc + 16 * t + lr];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
    };
    auto barrier = [] {
        FW_WAIT_LGKM0();
        __builtin_amdgcn_s_barrier();
        FW_COMPILER_FENCE();
    };
    const int len = k_end - k_begin, nfull = len > 0 ? len / 16 : 0;
    if (nfull > 0) {
        const int last = nfull - 1;
        load(0, 0);
        load(min(1, last), 1);
        stage(0, 0);
        load(min(2, last), 0);
        barrier();
        int c = 0;
        for (; c + 1 < nfull; c += 2) {
            stage(c + 1, 1);
            load(min(c + 3, last), 1);
            multiply(c);
            barrier();
            stage(c + 2, 0);
            load(min(c + 4, last), 0);
            multiply(c + 1);
            barrier();
        }
        if (c < nfull) { multiply(c); barrier(); }
    }
    if (nfull * 16 < len) {
        A.load(k_begin + 16 * nfull, k_end, sa, ra[0]);
        B.load(k_begin + 16 * nfull, k_end, sb, rb[0]);
        sa.store(As[0], ra[0]);
        sb.store(Bs[0], rb[0]);
        barrier();
        multiply(0);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) epi(wr + 16 * a + 4 * v + lq, wc + 16 * b + lr, acc[a][b][v]);
}

// new eigenvectors of a merge: U (kept x kept) times the kept rows of V; row j of the product goes to place kpos[j]
__global__ __launch_bounds__(256) void dc_product_kernel(DcArrays D, int M, int ld, int P, const double* __restrict__ U, const double* __restrict__ V,
                                                         double* __restrict__ Vout) {
    const int m = blockIdx.z;
    const int k = D.cnt[4 * m];
    const int row0 = blockIdx.y * 64;
    if (row0 >= k) return;
    const int off = part_begin(m, P, M), n = part_begin(m + 1, P, M) - off;
    const int col0 = blockIdx.x * 64;
    if (col0 >= n) return;
    // a child's vectors have nothing in the columns of the other: only the entries that reach into this tile's columns are summed over
    const int n1 = part_begin(2 * m + 1, 2 * P, M) - off, b1 = D.cnt[4 * m + 3] & 0xffff, b2 = D.cnt[4 * m + 3] >> 16;
    const int kb = col0 >= n1 ? b1 : 0, ke = col0 + 64 <= n1 ? b2 : k;
    const RowsK A = {U + (size_t)off * ld + off, ld, row0, k};
    const ColsK B = {V + off, ld, col0, n, D.urow + off};
    const int* kpos = D.kpos + off;
    gemm64(A, B, kb, ke, [&](int r, int c, double x) {
        if (row0 + r < k && col0 + c < n) Vout[(size_t)kpos[row0 + r] * ld + off + col0 + c] = x;
    });
}

// gram[block][slice] = Y Y^T of a block of reflectors (rows c0 .. c0 + 63 of Y) over a slice of the columns
constexpr int WY_SLICES = 4;
__global__ __launch_bounds__(256) void wy_gram_kernel(const double* __restrict__ Y, int ld, int M, double* __restrict__ gram) {
    const int c0 = blockIdx.x * NB, kmax = min(c0 + NB, M);
    const int ks = ((kmax + WY_SLICES - 1) / WY_SLICES + 15) / 16 * 16;
    const int kb = min(kmax, (int)blockIdx.y * ks), ke = min(kmax, kb + ks);
    double* dst = gram + ((size_t)blockIdx.x * WY_SLICES + blockIdx.y) * NB * NB;
    const RowsK A = {Y, ld, c0, M};
    gemm64(A, A, kb, ke, [&](int r, int c, double x) { dst[r * NB + c] = x; });
}
// F of a block: H_c0 H_c0+1 ... = I - Y^T F Y, upper triangular, F[:k][k] = -tau_k F[:k][:k] (Y y_k), F[k][k] = tau_k.  A row of F needs
// nothing of the other rows: one lane each, no barrier in the recurrence.
__global__ __launch_bounds__(256) void wy_factor_kernel(const double* __restrict__ gram, int M, const double* __restrict__ tau, double* __restrict__ F) {
    __shared__ double Gm[NB][NB + 2], Ft[NB][NB];        // Ft[column][row]
    const int c0 = blockIdx.x * NB;
    const double* src = gram + (size_t)blockIdx.x * WY_SLICES * NB * NB;
    for (int e = threadIdx.x; e < NB * NB; e += 256) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < WY_SLICES; ++k) s += src[(size_t)k * NB * NB + e];
        Gm[e & 63][e >> 6] = s;                          // symmetric; [column][row] so that a column of it lies along a row here
        Ft[e >> 6][e & 63] = 0.0;
    }
    __syncthreads();
    if (threadIdx.x < NB) {
        const int i = threadIdx.x;
        const double ti = c0 + i < M ? tau[c0 + i] : 0.0;
        for (int k = 0; k < NB; ++k) {
            const double tk = lane_value(ti, k);
            double s0 = 0.0, s1 = 0.0;
            int q = 0;
            for (; q + 8 <= k; q += 8) {
#pragma unroll
                for (int u = 0; u < 8; u += 2) { s0 += Ft[q + u][i] * Gm[k][q + u]; s1 += Ft[q + u + 1][i] * Gm[k][q + u + 1]; }
            }
            for (; q < k; ++q) s0 += Ft[q][i] * Gm[k][q];
            Ft[k][i] = i < k ? -tk * (s0 + s1) : i == k ? tk : 0.0;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NB * NB; e += 256) F[(size_t)blockIdx.x * NB * NB + e] = Ft[e & 63][e >> 6];
}
// Z = F Y, all blocks: the reflections are then V -= (V Y^T) Z
__global__ __launch_bounds__(256) void wy_form_kernel(const double* __restrict__ F, const double* __restrict__ Y, int ld, int M, double* __restrict__ Z) {
    const int c0 = blockIdx.y * NB, nb = min(NB, M - c0), kmax = c0 + nb;
    const int col0 = blockIdx.x * 64;
    if (col0 >= kmax) return;
    const RowsK A = {F + (size_t)blockIdx.y * NB * NB, NB, 0, NB};
    const ColsK B = {Y + (size_t)c0 * ld, ld, col0, kmax, nullptr};
    gemm64(A, B, 0, nb, [&](int r, int c, double x) {
        if (r < nb && col0 + c < kmax) Z[(size_t)(c0 + r) * ld + col0 + c] = x;
    });
}

// part[slice] = V Y^T restricted to a slice of the contraction index
__global__ __launch_bounds__(256) void wy_project_kernel(const double* __restrict__ V, const double* __restrict__ Y, int ld, int M, int c0,
                                                         int kmax, int kslice, double* __restrict__ part) {
    const int row0 = blockIdx.x * 64;
    const int kb = blockIdx.y * kslice, ke = min(kmax, kb + kslice);
    const RowsK A = {V, ld, row0, M};
    const RowsK B = {Y, ld, c0, M};
    double* dst = part + (size_t)blockIdx.y * M * NB;
    gemm64(A, B, kb, ke, [&](int r, int c, double x) {
        if (row0 + r < M) dst[(size_t)(row0 + r) * NB + c] = x;
    });
}
// out = sum of the slices
__global__ __launch_bounds__(256) void wy_sum_kernel(const double* __restrict__ part, int slices, int n, double* __restrict__ out) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    double x[8], s = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = k < slices ? part[(size_t)k * n + e] : 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += x[k];
    out[e] = s;
}
// V -= G Z, Z the rows of a block
__global__ __launch_bounds__(256) void wy_update_kernel(const double* __restrict__ Gm, const double* __restrict__ Y, int ld, int M, int c0,
                                                        int kmax, double* __restrict__ V) {
    const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
    const RowsK A = {Gm, NB, row0, M};
    const int nb = min(NB, M - c0);
    const ColsK B = {Y + (size_t)c0 * ld, ld, col0, kmax, nullptr};
    gemm64(A, B, 0, nb, [&](int r, int c, double x) {
        if (row0 + r < M && col0 + c < kmax) V[(size_t)(row0 + r) * ld + col0 + c] -= x;
    });
}

// All blocks of reflectors on 16 rows of V in one launch: V -= (V Y^T) Z, block after block.  The rows stay in registers as the transposed
// accumulators of v_mfma_f64_16x16x4_f64 -- a lane holds row lr, columns 16 tile + 4 lq .. + 3 -- which is at once the layout of
// the second operand of Y V^T and of the result of Z^T P^T: nothing of V moves between the blocks, and no workgroup waits for another.  Eight
// wavefronts share the column tiles (tile = wavefront + 8 slot); Y and Z come from the caches, the next tile's on their way while this one's are
// multiplied; the eight shares of P = V Y^T are added through LDS.  NS: slots per wavefront.
// Bound: the matrix cores of M / 16 compute units, and the reads of Y and Z by each of them.
constexpr int STRIP_MAX_M = 2560;
// f(0), f(1), .. f(N - 1) with compile-time constants
template <int N, class F>
__device__ __forceinline__ void each(const F& f) {
    if constexpr (N > 0) {
        each<N - 1>(f);
        f(std::integral_constant<int, N - 1>());
    }
}
template <int NS>
__global__ __launch_bounds__(512) void wy_strip_kernel(const double* __restrict__ Y, const double* __restrict__ Z, int ld, int M, double* __restrict__ V) {
    __shared__ double part[8][16][64], sum[16][64];
    const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = blockIdx.x * 16 + lr;
    const int zc = 4 * (lr & 3) + (lr >> 2);        // column of a tile that row lr of the result of Z^T P^T stands for
    double* vrow = V + (size_t)min(row, M - 1) * ld + 4 * lq;
    doublex4 acc[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int tl = wave + 8 * i;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][v] = 16 * tl < ld ? vrow[16 * tl + v] : 0.0;
    }
    for (int c0 = 0; c0 < M; c0 += NB) {
        const int nb = min(NB, M - c0), ntl = (c0 + nb + 15) / 16;
        const int act = wave < ntl ? (ntl - wave + 7) / 8 : 0;      // slots of this wavefront that hold columns below c0 + nb
        // P^T = Y V^T, 32 of the 64 reflectors at a time
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            doublex4 pt[2] = {doublex4{0.0, 0.0, 0.0, 0.0}, doublex4{0.0, 0.0, 0.0, 0.0}};
            const double* y0 = Y + (size_t)min(c0 + 32 * hf + lr, M - 1) * ld + 4 * lq;
            const double* y1 = Y + (size_t)min(c0 + 32 * hf + 16 + lr, M - 1) * ld + 4 * lq;
            doublex2 ya[2][4];
            auto load = [&](int i, doublex2 (&b)[4]) {
                const int at = 16 * min(wave + 8 * i, ntl - 1);
                b[0] = *reinterpret_cast<const doublex2*>(y0 + at); b[1] = *reinterpret_cast<const doublex2*>(y0 + at + 2);
                b[2] = *reinterpret_cast<const doublex2*>(y1 + at); b[3] = *reinterpret_cast<const doublex2*>(y1 + at + 2);
            };
            load(0, ya[0]);
            each<NS>([&](auto slot) {
                constexpr int i = decltype(slot)::value;
                if (i >= act) return;
                load(i + 1, ya[(i + 1) & 1]);
                const doublex2 (&b)[4] = ya[i & 1];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    pt[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[v >> 1][v & 1], acc[i][v], pt[0], 0, 0, 0);
                    pt[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[2 + (v >> 1)][v & 1], acc[i][v], pt[1], 0, 0, 0);
                }
            });
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) part[wave][8 * hf + 4 * m + v][lane] = pt[m][v];     // reflector 32 hf + 16 m + 4 v + lq
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int s = 2 * wave + k;
            double x = 0.0;
#pragma unroll
            for (int w = 0; w < 8; ++w) x += part[w][s][lane];
            sum[s][lane] = 4 * s + lq < nb ? -x : 0.0;              // reflector 4 s + lq
        }
        __syncthreads();
        // V^T -= Z^T P^T, 32 reflectors at a time
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            double p[8], za[2][8];
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = sum[8 * hf + k][lane];
            const double* zr[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) zr[k] = Z + (size_t)min(c0 + 32 * hf + 4 * k + lq, M - 1) * ld + zc;
            auto load = [&](int i, double (&b)[8]) {
                const int at = 16 * min(wave + 8 * i, ntl - 1);
#pragma unroll
                for (int k = 0; k < 8; ++k) b[k] = zr[k][at];
            };
            load(0, za[0]);
            each<NS>([&](auto slot) {
                constexpr int i = decltype(slot)::value;
                if (i >= act) return;
                load(i + 1, za[(i + 1) & 1]);
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(za[i & 1][k], p[k], acc[i], 0, 0, 0);
            });
        }
    }
    if (row >= M) return;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int tl = wave + 8 * i;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (16 * tl + 4 * lq + v < M) vrow[16 * tl + v] = acc[i][v];
    }
}

// ------------------------------------------------------------------------------------------- acceptance, T and Q
// W = V Phi
__global__ __launch_bounds__(256) void image_kernel(const double* __restrict__ V, const double* __restrict__ Phi, int ld, int M,
                                                    double* __restrict__ W) {
    const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
    const RowsK A = {V, ld, row0, M};
    const ColsK B = {Phi, ld, col0, M, nullptr};
    gemm64(A, B, 0, M, [&](int r, int c, double x) {
        if (row0 + r < M && col0 + c < M) W[(size_t)(row0 + r) * ld + col0 + c] = x;
    });
}
// scale of row i: sqrt(sum_k v_ik^2 |Phi_kk|); scale[M] = max(floor_abs, floor_rel trace(Phi))
__global__ __launch_bounds__(256) void row_scale_kernel(const double* __restrict__ V, const float* __restrict__ Phi, int ld, int M,
                                                        double floor_abs, double floor_rel, double* __restrict__ scale, int* __restrict__ flag) {
    const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x < 2) flag[threadIdx.x] = 0;
    if (r >= M) return;
    double s = 0.0, tr = 0.0;
    for (int j = lane; j < M; j += 64) {
        const double v = V[(size_t)r * ld + j], ph = Phi[(size_t)j * M + j];
        s += v * v * fabs(ph);
        tr += ph;
    }
    s = wave_total(s);
    tr = wave_total(tr);
    if (lane == 0) {
        scale[r] = sqrt(s);
        if (r == 0) scale[M] = fmax(floor_abs, floor_rel * tr);
    }
}
// On the tiles that touch the lower triangle: S = W V^T (blockIdx.z = 0), its diagonal is lambda, any off-diagonal entry above
// max(thr scale_i scale_j, scale_M) raises flag[0]; V V^T (blockIdx.z = 1, up to ORTH_FULL_MAX_M rows), any entry further than thr
// from the identity raises flag[1].  The first alone would pass two equal rows, or a zero one, among the vectors that Phi takes to
// (nearly) zero.  NaN raises.
__global__ __launch_bounds__(256) void residual_kernel(const double* __restrict__ W, const double* __restrict__ V, int ld, int M, double thr,
                                                       const double* __restrict__ scale, double* __restrict__ lam, int* __restrict__ flag) {
    const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
    if (col0 > row0) return;
    const bool image = blockIdx.z == 0;
    const RowsK A = {image ? W : V, ld, row0, M};
    const RowsK B = {V, ld, col0, M};
    const double floor = scale[M];
    int bad = 0;
    gemm64(A, B, 0, M, [&](int r, int c, double x) {
        const int i = row0 + r, j = col0 + c;
        if (i < M && j < M) {
            if (!image) { if (!(fabs(x - (i == j ? 1.0 : 0.0)) <= thr)) bad = 1; }
            else if (i == j) lam[i] = x;
            else if (!(fabs(x) <= fmax(thr * scale[i] * scale[j], floor))) bad = 1;
        }
    });
    if (__any(bad) && (threadIdx.x & 63) == 0) flag[blockIdx.z] = 1;
}
// The same look at V V^T for more rows, where the whole product took 0.38 ms of 23 at M = 2304 (this way 0.05): V (V^T x) = x for eight
// vectors of pseudo-random entries (R. Freivalds 1979).  A row of V V^T - I with an entry above the bound goes unseen
// only if its products with all eight cancel.
constexpr int ORTH_FULL_MAX_M = 1024;
constexpr int OV = 8, ORS = 64;        // vectors; rows per slice of V^T x
// entry of vector k at row r: +-[0.5, 1), from the bits of an integer hash
__device__ __forceinline__ double orth_entry(int r, int k) {
    unsigned h = (unsigned)r * 2654435761u ^ ((unsigned)k + 1u) * 2246822519u;
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13; h *= 3266489917u; h ^= h >> 16;
    const double m = 0.5 + (double)(h >> 1) * (1.0 / 4294967296.0);
    return (h & 1u) ? -m : m;
}
// part[slice][k][column] = sum over the slice's rows of V[row][column] x_k(row)
__global__ __launch_bounds__(256) void orth_back_kernel(const double* __restrict__ V, int ld, int M, double* __restrict__ part) {
    __shared__ double xs[ORS][OV];
    const int r0 = blockIdx.y * ORS, rn = min(ORS, M - r0), col = blockIdx.x * 256 + threadIdx.x;
    for (int e = threadIdx.x; e < ORS * OV; e += 256) xs[e / OV][e % OV] = e / OV < rn ? orth_entry(r0 + e / OV, e % OV) : 0.0;
    __syncthreads();
    if (col >= M) return;
    double acc[OV];
#pragma unroll
    for (int k = 0; k < OV; ++k) acc[k] = 0.0;
    for (int r = 0; r < rn; r += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = V[(size_t)(r0 + min(r + u, rn - 1)) * ld + col];    // past the end x is zero
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < OV; ++k) acc[k] += v[u] * xs[r + u][k];
    }
#pragma unroll
    for (int k = 0; k < OV; ++k) part[((size_t)blockIdx.y * OV + k) * M + col] = acc[k];
}
__global__ __launch_bounds__(256) void orth_sum_kernel(const double* __restrict__ part, int slices, int M, double* __restrict__ z) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= OV * M) return;
    double s = 0.0;
    for (int k = 0; k < slices; ++k) s += part[(size_t)k * OV * M + e];
    z[e] = s;
}
// rows of V times z against x, four rows per wavefront
__global__ __launch_bounds__(256) void orth_test_kernel(const double* __restrict__ V, int ld, int M, const double* __restrict__ z, double thr,
                                                        int* __restrict__ flag) {
    const int lane = threadIdx.x & 63, r0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4;
    if (r0 >= M) return;
    double acc[4][OV];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < OV; ++k) acc[i][k] = 0.0;
    for (int c = lane; c < M; c += 64) {
        double v[4], zz[OV];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = V[(size_t)min(r0 + i, M - 1) * ld + c];
#pragma unroll
        for (int k = 0; k < OV; ++k) zz[k] = z[(size_t)k * M + c];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < OV; ++k) acc[i][k] += v[i] * zz[k];
    }
    int bad = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < OV; ++k) {
            const double y = wave_total(acc[i][k]);
            if (r0 + i < M && !(fabs(y - orth_entry(r0 + i, k)) <= thr)) bad = 1;
        }
    if (bad && lane == 0) *flag = 1;
}
// The same scale for V = I, flag[0] cleared, flag[1] = is some diagonal entry zero: one workgroup
__global__ __launch_bounds__(1024) void diagonal_scale_kernel(const float* __restrict__ Phi, int M, double floor_abs, double floor_rel,
                                                              double* __restrict__ scale, int* __restrict__ flag) {
    __shared__ double red[16];
    __shared__ int zeros;
    if (threadIdx.x == 0) zeros = 0;
    __syncthreads();
    double tr = 0.0;
    bool zero = false;
    for (int i = threadIdx.x; i < M; i += 1024) {
        const double d = Phi[(size_t)i * M + i];
        scale[i] = sqrt(fabs(d));
        tr += d;
        zero |= d == 0.0;
    }
    if (zero) zeros = 1;
    tr = block_total<1024>(tr, red);      // its barrier also publishes `zeros`
    if (threadIdx.x == 0) { scale[M] = fmax(floor_abs, floor_rel * tr); flag[0] = 0; flag[1] = zeros; }
}
// Does V = I pass the test of residual_kernel?  Both triangles against the bound, which their mean then meets as well.
__global__ __launch_bounds__(256) void nearly_diagonal_kernel(const float* __restrict__ Phi, int M, double thr, const double* __restrict__ scale,
                                                              int* __restrict__ flag) {
    const double floor = scale[M];
    int bad = 0;
    for (int i = blockIdx.x; i < M; i += gridDim.x) {
        const double si = thr * scale[i];
        for (int j = threadIdx.x; j < M; j += 256)
            if (j != i && !(fabs((double)Phi[(size_t)i * M + j]) <= fmax(si * scale[j], floor))) bad = 1;
        if (__any(bad)) break;
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) *flag = 1;
}
// T = V^T diag(g) V (z = 0) and Q = V^T diag(g^2) V (z = 1) as float32: lower tiles, mirrored on the way out
__global__ __launch_bounds__(256) void spectral_product_kernel(const double* __restrict__ V, int ld, int M, const double* __restrict__ g,
                                                               float* __restrict__ o0, float* __restrict__ o1) {
    const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
    if (col0 > row0) return;
    float* out = blockIdx.z == 0 ? o0 : o1;
    const ColsKScaled A = {V, ld, row0, M, g, blockIdx.z == 1};
    const ColsK B = {V, ld, col0, M, nullptr};
    gemm64(A, B, 0, M, [&](int r, int c, double x) {
        const int i = row0 + r, j = col0 + c;
        if (i < M && j <= i) {
            out[(size_t)i * M + j] = (float)x;
            if (j < i) out[(size_t)j * M + i] = (float)x;
        }
    });
}

// three matrices, one per blockIdx.y: zero, and a bit pattern in the other two
__global__ __launch_bounds__(256) void fill64_kernel(double* __restrict__ p0, double* __restrict__ p1, double* __restrict__ p2, size_t n,
                                                     unsigned long long bits) {
    double* p = blockIdx.y == 0 ? p0 : blockIdx.y == 1 ? p1 : p2;
    const double x = blockIdx.y == 0 ? 0.0 : __longlong_as_double((long long)bits);
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) p[e] = x;
}
__global__ __launch_bounds__(256) void start_over_kernel(const double* __restrict__ copy, int ld, size_t n, double* __restrict__ V,
                                                         double* __restrict__ W) {
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
        W[e] = copy[e];
        V[e] = e % ld == e / ld ? 1.0 : 0.0;
    }
}
inline int grid_for(size_t n) {
    const size_t b = (n + 255) / 256;
    return (int)(b > 4096 ? 4096 : b);
}

template <int T, int C, int RB>
void launch_step(double* A, int ld, int c, int first, const double* vp, const double* pp, double* vn, double* pn, double* d, double* e,
                 double* tau, int G, hipStream_t st) {
    const int rows = (c + G - 1) / G;
    hipLaunchKernelGGL((tri_step_kernel<T, C, RB>), dim3(G), dim3(T), (size_t)(rows + RB) * (T / 64) * sizeof(double), st, A, ld, c, first, vp, pp,
                       vn, pn, d, e, tau);
}

// workgroups and threads of a step with c rows left
void step(double* A, int ld, int c, int first, const double* vp, const double* pp, double* vn, double* pn, double* d, double* e, double* tau,
          hipStream_t st) {
#define FW_STEP(T, C, RB, G) launch_step<T, C, RB>(A, ld, c, first, vp, pp, vn, pn, d, e, tau, G, st)
    const int n = c + 1;
    const int few = c < 256 ? c : 256;
    if (n <= 256) FW_STEP(256, 1, 1, few);
    else if (n <= 512) FW_STEP(256, 2, 2, 256);
    else if (n <= 768) FW_STEP(256, 3, 3, 256);
    else if (n <= 1024) FW_STEP(256, 4, 4, 256);
    else if (n <= 1536) FW_STEP(512, 3, 3, 256);
    else if (n <= 2048) FW_STEP(512, 4, 4, 256);
    else if (n <= 2560) FW_STEP(512, 5, 5, 256);
    else if (n <= 3072) FW_STEP(512, 6, 4, 256);
    else if (n <= 4096) FW_STEP(512, 8, 4, 256);
    else if (n <= 5120) FW_STEP(1024, 5, 4, 256);
    else if (n <= 8192) FW_STEP(1024, 8, 2, 256);
    else FW_STEP(1024, 16, 1, 256);
#undef FW_STEP
}

// Workgroups that wait for each other have to be resident together.  The launch is an ordinary one behind two checks: the device
// holds all of them at a time, and the stream may use all of its compute units.  Two such launches at a time, from two streams
// or threads, could each hold a part of the chip, so every one waits on its stream for the one before on that device.
// hipLaunchCooperativeKernel does this as well, but its first call adds a hardware queue to the process, and streams that ran side by
// side before share one from then on: the largest benchmark configuration on two streams, after decompositions of the two smaller
// ones, 1.44 ms without it, 1.69 ms with it, 1.41 ms like this (the decompositions themselves take as long either way).
struct RowsTurn {
    std::mutex lock;
    hipEvent_t done = nullptr;      // behind the latest launch; lives as long as the process
};
constexpr int MAX_DEVICES = 64;
RowsTurn rows_turns[MAX_DEVICES];
bool rows_fit(const void* kernel, int threads, unsigned workgroups, int dev, hipStream_t st) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(st, 32, mask) != hipSuccess) return false;
    int usable = 0;
    for (uint32_t word : mask) usable += __builtin_popcount(word);
    return usable >= cus && (long long)per_cu * cus >= (long long)workgroups;
}
// The reduction of the leading (c + 1) x (c + 1) block in one launch; false: not possible (too many rows, or the device does not hold
// the workgroups at a time), nothing was launched.
template <int T, int C, int RB>
bool launch_rows(const double* A, int ld, int c, int first, const double* vp, const double* pp, double* Pslot, double* Xslot, double* Y, double* d,
                 double* e, double* tau, int polls, hipStream_t st) {
    const void* kernel = reinterpret_cast<const void*>(tri_rows_kernel<T, C, RB>);
    const unsigned workgroups = c / RB + 1;
    int dev = -1;
    bool launched = false;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < MAX_DEVICES && rows_fit(kernel, T, workgroups, dev, st)) {
        RowsTurn& turn = rows_turns[dev];
        const std::lock_guard<std::mutex> hold(turn.lock);
        const bool have = turn.done || hipEventCreateWithFlags(&turn.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
        if (have && (hipEventQuery(turn.done) == hipSuccess || hipStreamWaitEvent(st, turn.done, 0) == hipSuccess)) {
            void* args[] = {&A, &ld, &c, &first, &vp, &pp, &Pslot, &Xslot, &Y, &d, &e, &tau, &polls};
            launched = hipLaunchKernel(kernel, dim3(workgroups), dim3(T), args, 0, st) == hipSuccess;
            if (launched && hipEventRecord(turn.done, st) != hipSuccess) (void)hipStreamSynchronize(st);
        }
    }
    (void)hipGetLastError();
    return launched;
}
// Threads and columns per thread: few columns shorten the chain of a step, many wavefronts lengthen its sums.  Whole calls, us: 512 features
// 1811 (256 threads of two 1833), 520 features 1929 (320 of two 1961), 576 features 2096 (320 of two 2117; in an earlier tree 2178, 256 of
// three 2274), 640 features 2261 (320 of two 2283), 768 features 2873 (256 of three 2977, 768 of one 2921), 1024 features 3770 (1024 of one 4179),
// 1536 features 6261 (768 of two 6519), 2048 features 9285 (1024 of two 10466).
bool rows(const double* A, int ld, int c, int first, const double* vp, const double* pp, double* Pslot, double* Xslot, double* Y, double* d,
          double* e, double* tau, int polls, hipStream_t st) {
    const int n = c + 1;
#define FW_ROWS(T, C, RB) return launch_rows<T, C, RB>(A, ld, c, first, vp, pp, Pslot, Xslot, Y, d, e, tau, polls, st)
    if (n <= 256) FW_ROWS(256, 1, 8);
    if (n <= 512) FW_ROWS(512, 1, 8);
    if (n <= 640) FW_ROWS(640, 1, 8);
    if (n <= 768) FW_ROWS(384, 2, 8);
    if (n <= 1024) FW_ROWS(512, 2, 8);
    if (n <= 1536) FW_ROWS(512, 3, 8);
    if (n <= 2048) FW_ROWS(512, 4, 8);
    if (n <= ROWS_MAX_M) FW_ROWS(512, 5, 10);
#undef FW_ROWS
    return false;
}

struct SmallWs { size_t d, e, tau, p0, p1, dn, sd, sz, kd, kz, zh, rtau, dd, rc, rs, scale, F, ints, flag, total; };
inline SmallWs small_layout(int M) {
    SmallWs L;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += align_up(bytes, 256); return at; };
    const size_t v = (size_t)(M + 64) * sizeof(double);
    L.d = take(v); L.e = take(v); L.tau = take(v); L.p0 = take(v); L.p1 = take(v); L.dn = take(v); L.sd = take(v); L.sz = take(v); L.kd = take(v);
    L.kz = take(v); L.zh = take(v); L.rtau = take(v); L.dd = take(v); L.rc = take(v); L.rs = take(v); L.scale = take(v);
    L.F = take((size_t)((M + NB - 1) / NB) * NB * NB * sizeof(double));
    L.ints = take((size_t)(M + 64) * 11 * sizeof(int));
    L.flag = take(256);
    L.total = o;
    return L;
}

}  // namespace

int sym_eig_ld(int M) { return (M + 15) / 16 * 16; }
size_t sym_eig_small_bytes(int M) { return small_layout(M).total; }
// doubles the first matrix buffer must hold besides the matrix: products of reflectors and projections of the back-transformation
size_t sym_eig_matrix_doubles(int M) {
    const size_t a = (size_t)M * sym_eig_ld(M), b = (size_t)M * NB * 9, c = (size_t)((M + NB - 1) / NB) * WY_SLICES * NB * NB;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// Eigenvectors of the symmetric part of Phi as rows, ascending eigenvalues.  dead: some diagonal entry is zero.  buf[0..3]: four matrices of
// sym_eig_matrix_doubles(M); on return *V and *free_buf name the buffer with the eigenvectors and one that is free.
fw_status sym_eig(const float* Phi, int M, bool dead, double* const buf[4], void* small, double** V, double** free_buf, hipStream_t st, EvdRun* run) {
    const int ld = sym_eig_ld(M);
    const SmallWs L = small_layout(M);
    char* sb = reinterpret_cast<char*>(small);
    auto dbl = [&](size_t at) { return reinterpret_cast<double*>(sb + at); };
    double *A = buf[0], *Y = buf[1], *Va = buf[2], *Vb = buf[3];
    double *d = dbl(L.d), *e = dbl(L.e), *tau = dbl(L.tau), *p[2] = {dbl(L.p0), dbl(L.p1)};
    int* perm = reinterpret_cast<int*>(sb + L.ints) + 8 * ((size_t)M + 64);
    const size_t nn = (size_t)M * ld;
    if (dead) hipLaunchKernelGGL(dead_last_kernel, dim3(1), dim3(1024), 0, st, Phi, M, perm);
    hipLaunchKernelGGL(sym_load_kernel, dim3((ld + 31) / 32, (M + 31) / 32), dim3(256), 0, st, Phi, M, ld, dead ? perm : nullptr, A);
    int c = M - 1, first = 1, cur = 0;
    auto vp = [&] { return Y + (size_t)(c + 1 < M ? c + 1 : c) * ld; };
    auto one_step = [&] {
        step(A, ld, c, first, vp(), p[cur ^ 1], Y + (size_t)c * ld, p[cur], d, e, tau, st);
        --c; first = 0; cur ^= 1;
    };
    hipLaunchKernelGGL(fill64_kernel, dim3(grid_for(nn), 3), dim3(256), 0, st, Y, Va, Vb, nn, M > TAIL ? SENTINEL : 0ull);
    bool reduced = false;
    if (M > TAIL) {
        while (c >= ROWS_MAX_M) one_step();
        FW_LAUNCH_CHECK();                // launch_rows clears the error of its own checks, and would clear one of these launches
        if (!(run && run->by_rows))
            reduced = rows(A, ld, c, first, vp(), p[cur ^ 1], Va, Vb, Y, d, e, tau, run && run->polls > 0 ? run->polls : POLL_LIMIT, st);
        if (run) run->one_launch = reduced ? 1 : 0;
        if (!reduced)
            while (c >= TAIL) one_step();
    }
    if (!reduced) hipLaunchKernelGGL(tri_tail_kernel, dim3(1), dim3(1024), 0, st, A, ld, c, first, vp(), p[cur ^ 1], Y, d, e, tau);
    if (M > TAIL) hipLaunchKernelGGL(fill64_kernel, dim3(grid_for(nn), 2), dim3(256), 0, st, Va, Vb, Vb, nn, 0ull);
    FW_LAUNCH_CHECK();

    int leaves = 1;
    while ((M + leaves - 1) / leaves > LEAF) leaves *= 2;
    DcArrays D;
    D.d = d; D.dn = dbl(L.dn); D.sd = dbl(L.sd); D.sz = dbl(L.sz); D.kd = dbl(L.kd); D.kz = dbl(L.kz); D.zh = dbl(L.zh); D.tau = dbl(L.rtau);
    D.dd = dbl(L.dd); D.rc = dbl(L.rc); D.rs = dbl(L.rs);
    int* ib = reinterpret_cast<int*>(sb + L.ints);
    const size_t mi = (size_t)M + 64;
    D.srow = ib; D.krow = ib + mi; D.org = ib + 2 * mi; D.kpos = ib + 3 * mi; D.drow = ib + 4 * mi; D.ri = ib + 5 * mi; D.rj = ib + 6 * mi;
    D.ucol = ib + 9 * mi; D.urow = ib + 10 * mi;
    D.cnt = ib + 7 * mi;         // four per merge; a level has at most M / 16 of them
    if (leaves > 1) hipLaunchKernelGGL(dc_tear_kernel, dim3((leaves + 255) / 256), dim3(256), 0, st, d, e, M, leaves);
    hipLaunchKernelGGL(dc_leaf_kernel, dim3(leaves), dim3(64), 0, st, d, e, M, ld, leaves, Va);
    for (int P = leaves / 2; P >= 1; P /= 2) {
        const int nmax = (M + P - 1) / P + 1;
        const dim3 waves((nmax + 3) / 4, P);
        if (nmax <= DEFLATE_MAX) hipLaunchKernelGGL(dc_deflate_lds_kernel, dim3(P), dim3(512), 0, st, D, e, M, ld, P, Va);
        else hipLaunchKernelGGL(dc_deflate_kernel, dim3(P), dim3(512), 0, st, D, e, M, ld, P, Va);
        hipLaunchKernelGGL(dc_rotate_kernel, dim3((nmax + 63) / 64, P), dim3(64), 0, st, D, M, ld, P, Va);
        hipLaunchKernelGGL(dc_secular_kernel, waves, dim3(256), 0, st, D, e, M, P);
        hipLaunchKernelGGL(dc_zhat_kernel, waves, dim3(256), 0, st, D, M, ld, P, Va, Vb);
        hipLaunchKernelGGL(dc_vectors_kernel, waves, dim3(256), 0, st, D, M, ld, P, A);
        hipLaunchKernelGGL(dc_product_kernel, dim3((nmax + 63) / 64, (nmax + 63) / 64, P), dim3(256), 0, st, D, M, ld, P, A, Va, Vb);
        double* x = Va; Va = Vb; Vb = x;
        double* y = D.d; D.d = D.dn; D.dn = y;
    }
    FW_LAUNCH_CHECK();

    // back-transformation: blocks of reflectors in ascending order
    const int nblk = (M + NB - 1) / NB, rt = (M + 63) / 64;
    double* F = dbl(L.F);
    double* Z = Vb;                                       // free until the end
    hipLaunchKernelGGL(wy_gram_kernel, dim3(nblk, WY_SLICES), dim3(256), 0, st, Y, ld, M, A);
    hipLaunchKernelGGL(wy_factor_kernel, dim3(nblk), dim3(256), 0, st, A, M, tau, F);
    hipLaunchKernelGGL(wy_form_kernel, dim3((M + 63) / 64, nblk), dim3(256), 0, st, F, Y, ld, M, Z);
    if (M <= STRIP_MAX_M) {
        const int slots = ((M + 15) / 16 + 7) / 8;
#define FW_STRIPS(NS) hipLaunchKernelGGL(wy_strip_kernel<NS>, dim3((M + 15) / 16), dim3(512), 0, st, Y, Z, ld, M, Va)
        if (slots <= 2) FW_STRIPS(2);
        else if (slots <= 5) FW_STRIPS(5);
        else if (slots <= 10) FW_STRIPS(10);
        else if (slots <= 15) FW_STRIPS(15);
        else FW_STRIPS(20);
#undef FW_STRIPS
    } else {
        double* part = A;
        double* G = A + (size_t)8 * M * NB;
        for (int b = 0; b < nblk; ++b) {
            const int c0 = b * NB, kmax = c0 + NB < M ? c0 + NB : M;
            int slices = 256 / rt;
            if (slices > 8) slices = 8;
            if (slices < 1) slices = 1;
            while (slices > 1 && kmax / slices < 64) --slices;
            const int kslice = ((kmax + slices - 1) / slices + 15) / 16 * 16;
            slices = (kmax + kslice - 1) / kslice;
            hipLaunchKernelGGL(wy_project_kernel, dim3(rt, slices), dim3(256), 0, st, Va, Y, ld, M, c0, kmax, kslice, part);
            if (slices > 1) hipLaunchKernelGGL(wy_sum_kernel, dim3((M * NB + 255) / 256), dim3(256), 0, st, part, slices, M * NB, G);
            hipLaunchKernelGGL(wy_update_kernel, dim3((kmax + 63) / 64, rt), dim3(256), 0, st, slices > 1 ? G : part, Z, ld, M, c0, kmax, Va);
        }
    }
    if (dead) {
        hipLaunchKernelGGL(restore_columns_kernel, dim3((M + 1023) / 1024, M), dim3(256), 0, st, Va, M, ld, perm, Vb, 0);
        hipLaunchKernelGGL(restore_columns_kernel, dim3((M + 1023) / 1024, M), dim3(256), 0, st, Vb, M, ld, perm, Va, 1);
    }
    FW_LAUNCH_CHECK();
    *V = Va; *free_buf = Vb;
    return FW_OK;
}

// W = V Phi, lambda_i = w_i . v_i, and on the device flag[0] != 0 if some |v_i Phi v_j^T|, i != j, exceeds both thr scale_i scale_j
// and max(floor_abs, floor_rel trace(Phi)), flag[1] != 0 if some entry of V V^T is further than thr from the identity.
// `copy`: one more matrix buffer, which gets the symmetric part of Phi in float64; `scratch`: another one
fw_status sym_eig_check(const float* Phi, int M, const double* V, double* W, double* copy, double* scratch, void* small, double thr, double floor_abs,
                        double floor_rel, double* lam, int* flag, hipStream_t st) {
    const int ld = sym_eig_ld(M), nt = (M + 63) / 64;
    double* scale = reinterpret_cast<double*>(reinterpret_cast<char*>(small) + small_layout(M).scale);
    hipLaunchKernelGGL(row_scale_kernel, dim3((M + 3) / 4), dim3(256), 0, st, V, Phi, ld, M, floor_abs, floor_rel, scale,
                       flag);
    hipLaunchKernelGGL(sym_load_kernel, dim3((ld + 31) / 32, (M + 31) / 32), dim3(256), 0, st, Phi, M, ld, nullptr, copy);
    hipLaunchKernelGGL(image_kernel, dim3(nt, nt), dim3(256), 0, st, V, copy, ld, M, W);
    hipLaunchKernelGGL(residual_kernel, dim3(nt, nt, M <= ORTH_FULL_MAX_M ? 2 : 1), dim3(256), 0, st, W, V, ld, M, thr, scale, lam, flag);
    if (M > ORTH_FULL_MAX_M) {
        const int slices = (M + ORS - 1) / ORS;
        double* z = scratch + (size_t)slices * OV * M;
        hipLaunchKernelGGL(orth_back_kernel, dim3((M + 255) / 256, slices), dim3(256), 0, st, V, ld, M, scratch);
        hipLaunchKernelGGL(orth_sum_kernel, dim3((OV * M + 255) / 256), dim3(256), 0, st, scratch, slices, M, z);
        hipLaunchKernelGGL(orth_test_kernel, dim3((M + 15) / 16), dim3(256), 0, st, V, ld, M, z, thr, flag + 1);
    }
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// on the device flag[0] != 0 unless V = I passes the test of sym_eig_check, flag[1] != 0 if some diagonal entry is zero
fw_status sym_eig_check_identity(const float* Phi, int M, void* small, double thr, double floor_abs, double floor_rel, int* flag,
                                 hipStream_t st) {
    double* scale = reinterpret_cast<double*>(reinterpret_cast<char*>(small) + small_layout(M).scale);
    hipLaunchKernelGGL(diagonal_scale_kernel, dim3(1), dim3(1024), 0, st, Phi, M, floor_abs, floor_rel, scale, flag);
    hipLaunchKernelGGL(nearly_diagonal_kernel, dim3(M < 1024 ? M : 1024), dim3(256), 0, st, Phi, M, thr, scale, flag);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// the symmetric part of Phi in float64
fw_status sym_eig_load(const float* Phi, int M, double* copy, hipStream_t st) {
    const int ld = sym_eig_ld(M);
    hipLaunchKernelGGL(sym_load_kernel, dim3((ld + 31) / 32, (M + 31) / 32), dim3(256), 0, st, Phi, M, ld, nullptr, copy);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// V = I and W = the symmetric part of Phi that sym_eig_check or sym_eig_load left in `copy`
fw_status sym_eig_start_over(const double* copy, int M, double* V, double* W, hipStream_t st) {
    const size_t nn = (size_t)M * sym_eig_ld(M);
    hipLaunchKernelGGL(start_over_kernel, dim3(grid_for(nn)), dim3(256), 0, st, copy, sym_eig_ld(M), nn, V, W);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

fw_status sym_eig_spectral_products(const double* V, int M, const double* root_g, float* T, float* Q, hipStream_t st) {
    const int nt = (M + 63) / 64;
    hipLaunchKernelGGL(spectral_product_kernel, dim3(nt, nt, 2), dim3(256), 0, st, V, sym_eig_ld(M), M, root_g, T, Q);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

}  // namespace fw
