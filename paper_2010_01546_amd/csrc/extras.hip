// Companions of the hot path: bias compensation when the tracked mean moves (Sec. 3.1, eq. (vtb_corr)) and the two
// monitoring figures of Sec. 6, whiteness rho (eq. (rho)) and normalised rank kappa (Sec. 3.2, eq. (hMs)).
#include "fw_internal.h"
#include "lane_sums.h"

namespace fw {
namespace {

// b[s] += scale * sum_{c,t} W[s][c][t] (mu_new[c] - mu_old[c]); one wavefront per output feature s, float64 sum.
// Sign: the layer output sum W~ (x - mu) + b must not change when mu moves, which needs the NEW mean minus the OLD one
// (the printed equation has them the other way round, against the relation it is derived from).
__global__ __launch_bounds__(256) void bias_compensate_kernel(float* __restrict__ b, const float* __restrict__ W, int S, int M, int taps,
                                                              const float* __restrict__ mu_old, const float* __restrict__ mu_new,
                                                              float scale) {
    const int lane = threadIdx.x & 63;
    const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (s >= S) return;
    const size_t n = (size_t)M * taps;
    const float* w = W + (size_t)s * n;
    double acc = 0.0;
    for (size_t e = lane; e < n; e += 64) {
        const int c = (int)(e / taps);
        acc += (double)w[e] * ((double)mu_new[c] - (double)mu_old[c]);
    }
    acc = wave_sum(acc);
    if (lane == 0) b[s] = (float)((double)b[s] + (double)scale * acc);
}

__global__ __launch_bounds__(256) void diag_extract_kernel(const float* __restrict__ P, int M, float* __restrict__ d) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m < M) d[m] = P[(size_t)m * M + m];
}

// rowsum[r] = (1 / d[r]) sum_c P[r][c]^2 / d[c]; one wavefront per row, 16-byte loads when the rows allow them
__global__ __launch_bounds__(256) void whiteness_rows_kernel(const float* __restrict__ P, const float* __restrict__ d, int M,
                                                             double* __restrict__ rowsum) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    const float* row = P + (size_t)r * M;
    double acc = 0.0;
    if ((M & 3) == 0) {
        const float4* row4 = reinterpret_cast<const float4*>(row);
        const float4* d4 = reinterpret_cast<const float4*>(d);
        const int n4 = M >> 2;
        int c = lane;
        for (; c + 64 < n4; c += 128) {
            const float4 p0 = row4[c], p1 = row4[c + 64], q0 = d4[c], q1 = d4[c + 64];
            acc += (double)(p0.x * p0.x / q0.x + p0.y * p0.y / q0.y) + (double)(p0.z * p0.z / q0.z + p0.w * p0.w / q0.w);
            acc += (double)(p1.x * p1.x / q1.x + p1.y * p1.y / q1.y) + (double)(p1.z * p1.z / q1.z + p1.w * p1.w / q1.w);
        }
        for (; c < n4; c += 64) {
            const float4 p0 = row4[c], q0 = d4[c];
            acc += (double)(p0.x * p0.x / q0.x + p0.y * p0.y / q0.y) + (double)(p0.z * p0.z / q0.z + p0.w * p0.w / q0.w);
        }
    } else {
        for (int c = lane; c < M; c += 64) {
            const float p = row[c];
            acc += (double)(p * p / d[c]);
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) rowsum[r] = acc / (double)d[r];
}

__device__ __forceinline__ double block_sum_1024(double v, double* red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i];
    return t;
}

// out[0] = rho = M / sum of the row sums (when rowsum is given);
// out[1] = kappa = Ms_hat / M, out[2] = Ms_hat = exp(-sum lb log lb), lb = max(lambda, 0) / sum, 0 log 0 = 0 (when
// lambda is given; the exponential of the spectral entropy is the reading of eq. (hMs) that has the two stated extremes)
__global__ __launch_bounds__(1024) void diagnostics_final_kernel(const double* __restrict__ rowsum, const float* __restrict__ lambda,
                                                                 int M, float* __restrict__ out) {
    __shared__ double red[16];
    if (rowsum) {
        double v = 0.0;
        for (int k = threadIdx.x; k < M; k += 1024) v += rowsum[k];
        const double tot = block_sum_1024(v, red);
        if (threadIdx.x == 0) out[0] = (float)((double)M / tot);
    }
    if (lambda) {
        double v = 0.0;
        for (int k = threadIdx.x; k < M; k += 1024) v += fmax((double)lambda[k], 0.0);
        const double tot = block_sum_1024(v, red);
        double ent = 0.0;
        for (int k = threadIdx.x; k < M; k += 1024) {
            const double lb = tot > 0.0 ? fmax((double)lambda[k], 0.0) / tot : 0.0;
            if (lb > 0.0) ent -= lb * log(lb);
        }
        ent = block_sum_1024(ent, red);
        if (threadIdx.x == 0) {
            const double ms = tot > 0.0 ? exp(ent) : 1.0;
            out[1] = (float)(ms / (double)M);
            out[2] = (float)ms;
        }
    }
}

// ---- condition-number probe: extreme Ritz values of Phi_y on a Krylov space of dimension <= 32 (Sec. 4: the condition
// number of Phi_y is what the recursion reduces).  Lanczos with full re-orthogonalisation, vectors and sums in float64
// (the matrix is read as float32, once per step: that read is the cost), no host synchronisation: a breakdown (the next
// image already lies in the space built so far) is recorded in `st` on the device and the remaining launches return at once.
struct ProbeState { int steps, done; double prev_beta; };
constexpr int PROBE_MAX_K = 32;
// above this the orthogonalisation of a step runs on many workgroups (a thread of the single one would need more registers than it has)
constexpr int PROBE_SPREAD_MIN_M = 2048;

// q_0 = b0 / |b0| (b0 = all ones when absent)
__global__ __launch_bounds__(1024) void probe_init_kernel(const float* __restrict__ b0, int M, double* __restrict__ q0, ProbeState* __restrict__ st) {
    __shared__ double red[16];
    double ss = 0.0;
    for (int m = threadIdx.x; m < M; m += 1024) { const double x = b0 ? (double)b0[m] : 1.0; ss += x * x; }
    const double nrm = sqrt(block_sum_1024(ss, red));
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (int m = threadIdx.x; m < M; m += 1024) q0[m] = (b0 ? (double)b0[m] : 1.0) * inv;
    if (threadIdx.x == 0) { st->steps = 0; st->done = nrm > 0.0 ? 0 : 1; st->prev_beta = 0.0; }
}

// w = A q, one wavefront per row, float64 accumulation
__global__ __launch_bounds__(256) void probe_matvec_kernel(const float* __restrict__ A, const double* __restrict__ q, int M,
                                                           double* __restrict__ w, const ProbeState* __restrict__ st) {
    if (st->done) return;
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    const float* row = A + (size_t)r * M;
    double acc = 0.0;
    if ((M & 3) == 0) {
        const float4* r4 = reinterpret_cast<const float4*>(row);
        const int n4 = M >> 2;
        int c = lane;
        for (; c + 192 < n4; c += 256) {
            float4 a[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = r4[c + 64 * j];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double* qq = q + 4 * (c + 64 * j);
                acc += (double)a[j].x * qq[0] + (double)a[j].y * qq[1] + (double)a[j].z * qq[2] + (double)a[j].w * qq[3];
            }
        }
        for (; c < n4; c += 64) {
            const float4 a = r4[c];
            const double* qq = q + 4 * c;
            acc += (double)a.x * qq[0] + (double)a.y * qq[1] + (double)a.z * qq[2] + (double)a.w * qq[3];
        }
    } else {
        int c = lane;
        for (; c + 448 < M; c += 512) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = row[c + 64 * u];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += (double)a[u] * q[c + 64 * u];
        }
        for (; c < M; c += 64) acc += (double)row[c] * q[c];
    }
    acc = wave_sum(acc);
    if (lane == 0) w[r] = acc;
}

// Step j of the recurrence, one workgroup: alpha_j = q_j . w, w made orthogonal to q_0 .. q_j (twice, all coefficients of
// a pass taken from the same w), beta_j = |w|, q_(j+1) = w / beta_j -- or the breakdown flag when nothing is left of w.
// A thread owns E entries and keeps them, and those of the up to NB > j basis vectors, in registers: one round of loads, all in flight
// together.  The coefficients of a pass are summed over the wavefront NB at a time, cross the workgroup through LDS and are added
// by every wavefront for itself in the order of the wavefronts, so a pass has one barrier.
// M = 525: 4.6 us a step with up to 8 vectors, 6.1 us with up to 16 (the basis read again for every product and subtraction, three barriers
// a pass: 10.3 us).
// H = 2: more vectors than registers, in two halves that take turns (four more rounds of loads from L2).  A step with 17 to 32 vectors, its
// product included: 27 us at 1025 and 28 at 2048 features; spread over several workgroups in four launches 34 and 35; with the
// basis read again for every product 25 and 38.
template <int E, int NB, int H>
__global__ __launch_bounds__(1024) void probe_orth_kernel(int j, int M, size_t ld, double* __restrict__ Qb, const double* __restrict__ w,
                                                          double* __restrict__ alpha, double* __restrict__ beta, double breakdown,
                                                          ProbeState* __restrict__ st) {
    __shared__ double part[3][16][H * NB + 1];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    double x[E], q[NB][E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = t + 1024 * e < M ? w[t + 1024 * e] : 0.0;
    // vectors h NB .. h NB + NB - 1.  One of several parts is read anew every time and behind the uses of the part before; masks would not
    // fit the scalar registers, so entries from M on repeat the last one (x is zero there) and vectors beyond j repeat it (their
    // coefficients are set to zero).
    auto load = [&](int h) {
        if constexpr (H == 1) {
#pragma unroll
            for (int e = 0; e < E; ++e)
#pragma unroll
                for (int i = 0; i < NB; ++i) q[i][e] = (i <= j && t + 1024 * e < M) ? Qb[(size_t)i * ld + t + 1024 * e] : 0.0;
        } else {
            const double* src = Qb;
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+s"(src));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const double* row = src + (size_t)min(h * NB + i, j) * ld;
#pragma unroll
                for (int e = 0; e < E; ++e) q[i][e] = row[min(t + 1024 * e, M - 1)];
            }
        }
    };
    load(0);
    if (st->done) return;
    // NB values per lane -> their sums over the wavefront in part[..][wave][0 .. NB - 1]
    auto sums_to = [&](const double (&v)[NB], double* out) {
        double h[NB / 2];
#pragma unroll
        for (int i = 0; i < NB / 2; ++i) h[i] = fold32(v[i], v[i + NB / 2]);
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
            const double s = sum16(fold16(h[i], h[i + NB / 4]));     // value i + g NB / 4 in lanes 16 g .. 16 g + 15
            if ((lane & 15) == 0) out[i + (lane >> 4) * (NB / 4)] = s;
        }
    };
    auto square = [&] {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) s += x[e] * x[e];
        return sum16(fold16(fold32(s, s), fold32(s, s)));            // over the wavefront, in every lane
    };
    double n0 = 0.0, al = 0.0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            if (h > 0) load(h);
            double v[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                v[i] = 0.0;
#pragma unroll
                for (int e = 0; e < E; ++e) v[i] += q[i][e] * x[e];
            }
            sums_to(v, part[pass][wave] + h * NB);
        }
        if (pass == 0) {
            const double s = square();
            if (lane == 0) part[0][wave][H * NB] = s;
        }
        __syncthreads();
        // coefficient `lane` (and behind the last one the square of the first pass)
        double c = 0.0;
        if (lane < H * NB + (pass == 0 ? 1 : 0)) {
#pragma unroll
            for (int g = 0; g < 16; ++g) c += part[pass][g][lane];
            if (H > 1 && lane > j && lane < H * NB) c = 0.0;
        }
        auto from_lane = [&](int i) {
            const long long b = __double_as_longlong(c);
            const unsigned lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), i), hi = __builtin_amdgcn_readlane((int)(b >> 32), i);
            return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        };
        if (pass == 0) { n0 = sqrt(from_lane(H * NB)); al = from_lane(j); }
#pragma unroll
        for (int h = H - 1; h >= 0; --h) {            // the half at hand first
            if (h < H - 1) load(h);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const double ci = from_lane(h * NB + i);
#pragma unroll
                for (int e = 0; e < E; ++e) x[e] -= ci * q[i][e];
            }
        }
        if constexpr (H > 1) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (t + 1024 * e >= M) x[e] = 0.0;
        }
    }
    const double s = square();
    if (lane == 0) part[2][wave][0] = s;
    __syncthreads();
    double s1 = 0.0;
#pragma unroll
    for (int g = 0; g < 16; ++g) s1 += part[2][g][0];
    const double nw = sqrt(s1);
    const bool stop = !(nw > breakdown * n0);
    if (!stop) {
        const double inv = 1.0 / nw;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int m = t + 1024 * e;
            if (m < M) Qb[(size_t)(j + 1) * ld + m] = x[e] * inv;
        }
    }
    if (t == 0) {
        alpha[j] = al;
        beta[j] = nw;
        st->steps = j + 1;
        if (stop) st->done = 1;
    }
}

// The same step for many features, spread over ceil(M / 256) workgroups (thread t of workgroup b owns entry 256 b + t of
// w) in four launches, because every reduction over all of w needs the workgroups to meet:
//   phase 1  partial coefficients q_i . w of the first pass and the partial |w|^2
//   phase 2  coefficients summed over the workgroups in a fixed order, w made orthogonal once, partial coefficients of the
//            second pass (alpha_j = the first pass's coefficient of q_j)
//   phase 3  second pass applied, partial |w|^2
//   phase 4  beta_j = |w|, q_(j+1) = w / beta_j, or the breakdown flag
// part: [2][nb][PROBE_MAX_K + 1] coefficients, then [2][nb] squared norms.
constexpr int PROBE_WG = 256;
__device__ __forceinline__ double block_sum_256(double v, double* red4) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = v;
    __syncthreads();
    return red4[0] + red4[1] + red4[2] + red4[3];
}
template <int PHASE>
__global__ __launch_bounds__(PROBE_WG) void probe_orth_phase_kernel(int j, int M, size_t ld, double* __restrict__ Qb, double* __restrict__ w,
                                                                    double* __restrict__ part, double* __restrict__ alpha,
                                                                    double* __restrict__ beta, double breakdown, ProbeState* __restrict__ st) {
    constexpr int KP = PROBE_MAX_K + 1;
    __shared__ double red4[4];
    __shared__ double wpart[4][KP];
    __shared__ double coef[KP];
    if (st->done) return;
    const int nb = gridDim.x, blk = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blk * PROBE_WG + threadIdx.x;
    const bool ok = m < M;
    double* cpart = part;                              // [2][nb][KP]
    double* npart = part + (size_t)2 * nb * KP;        // [2][nb]
    double wm = ok ? w[m] : 0.0;
    if (PHASE == 2 || PHASE == 3) {
        // coefficients of the pass before: every workgroup adds the partial results in the same order
        // (lane i of wavefront g takes the workgroups g, g + 4, ... of coefficient i; the four sums are added in order)
        const double* src = cpart + (size_t)(PHASE - 2) * nb * KP;
        {
            double c = 0.0;
            if (lane <= j) {
#pragma unroll 4
                for (int b = wave; b < nb; b += 4) c += src[(size_t)b * KP + lane];
            }
            if (lane < KP) wpart[wave][lane] = c;
        }
        __syncthreads();
        if ((int)threadIdx.x <= j) {
            const double c = wpart[0][threadIdx.x] + wpart[1][threadIdx.x] + wpart[2][threadIdx.x] + wpart[3][threadIdx.x];
            coef[threadIdx.x] = c;
            if (PHASE == 2 && blk == 0 && (int)threadIdx.x == j) alpha[j] = c;
        }
        __syncthreads();
        for (int i = 0; i <= j; ++i) wm -= coef[i] * (ok ? Qb[(size_t)i * ld + m] : 0.0);
        if (ok) w[m] = wm;
    }
    if (PHASE == 1 || PHASE == 2) {
        double* dst = cpart + ((size_t)(PHASE - 1) * nb + blk) * KP;
        for (int i = 0; i <= j; ++i) {
            double d = ok ? Qb[(size_t)i * ld + m] * wm : 0.0;
            d = wave_sum(d);
            if (lane == 0) wpart[wave][i] = d;
        }
        __syncthreads();
        if ((int)threadIdx.x <= j) dst[threadIdx.x] = wpart[0][threadIdx.x] + wpart[1][threadIdx.x] + wpart[2][threadIdx.x] + wpart[3][threadIdx.x];
    }
    if (PHASE == 1 || PHASE == 3) {
        const double s = block_sum_256(wm * wm, red4);
        if (threadIdx.x == 0) npart[(size_t)(PHASE == 1 ? 0 : 1) * nb + blk] = s;
    }
    if (PHASE == 4) {
        // at most 64 workgroups (M <= 16384): one partial norm per lane of the first wavefront, butterfly sum (fixed order)
        double s0 = ((int)threadIdx.x < nb) ? npart[threadIdx.x] : 0.0;
        double s1 = ((int)threadIdx.x < nb) ? npart[(size_t)nb + threadIdx.x] : 0.0;
        s0 = wave_sum(s0); s1 = wave_sum(s1);
        if (threadIdx.x == 0) { red4[0] = s0; red4[1] = s1; }
        __syncthreads();
        const double n0 = sqrt(red4[0]), nw = sqrt(red4[1]);
        const bool stop = !(nw > breakdown * n0);
        if (!stop && ok) Qb[(size_t)(j + 1) * ld + m] = wm / nw;
        // beta and the state are written by one thread of this last launch of the step.  A workgroup of this launch that
        // starts after the flag was raised returns at once; it would have written nothing (no q_(j+1) after a breakdown).
        if (blk == nb - 1 && threadIdx.x == 0) {
            beta[j] = nw;
            st->steps = j + 1;
            if (stop) st->done = 1;
        }
    }
}

// extreme eigenvalues of the symmetric tridiagonal matrix (alpha_0..alpha_(n-1); beta_0..beta_(n-2)) by bisection on the
// number of eigenvalues below x (sign changes of the pivots of T - x I)
__device__ int tridiag_count_below(const double* a, const double* b, int n, double x) {
    int cnt = 0;
    double d = 1.0;
    for (int i = 0; i < n; ++i) {
        const double off = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
        d = a[i] - x - (i > 0 ? off / d : 0.0);
        if (d == 0.0) d = -1e-300;
        if (d < 0.0) ++cnt;
    }
    return cnt;
}

// One workgroup, PROBE_CUTS / 64 wavefronts per eigenvalue; every round cuts the bracket of its eigenvalue into PROBE_CUTS + 1 parts, one
// trial point per thread.  The rounds follow one another and each is one serial chain of n float64 divisions, so the two
// eigenvalues run side by side; more points a round would save rounds, but the divisions of the wavefronts of a SIMD queue up.
// 129^11 = 2^77 of the bracket: a smallest eigenvalue far below the resolution of the largest is still told from zero.
// n = 16: 17.5 us (7 rounds of 512 points each, 2^63 of the bracket: 24.2 us; one wavefront for both, 24 rounds: 37 us).
constexpr int PROBE_CUTS = 128, PROBE_ROUNDS = 11;
__global__ __launch_bounds__(2 * PROBE_CUTS) void probe_final_kernel(const double* __restrict__ alpha, const double* __restrict__ beta,
                                                           const ProbeState* __restrict__ st, float* __restrict__ out) {
    __shared__ double al[PROBE_MAX_K], be[PROBE_MAX_K];
    __shared__ int first_s[2][2][PROBE_CUTS / 64];
    __shared__ double res[2];
    const int n = st->steps;
    if (n <= 0) { if (threadIdx.x < 4) out[threadIdx.x] = 0.f; return; }
    if ((int)threadIdx.x < n) { al[threadIdx.x] = alpha[threadIdx.x]; be[threadIdx.x] = beta[threadIdx.x]; }
    __syncthreads();
    double lo = al[0], hi = al[0];
    for (int i = 0; i < n; ++i) {
        const double r = (i > 0 ? fabs(be[i - 1]) : 0.0) + (i + 1 < n ? fabs(be[i]) : 0.0);
        lo = fmin(lo, al[i] - r);
        hi = fmax(hi, al[i] + r);
    }
    // largest: the smallest x with count_below(x) = n;  smallest: the smallest x with count_below(x) >= 1.
    // count_below grows with x, so the threads that reach the count form a suffix: the bracket becomes the part between
    // the last thread that does not and the first that does.
    constexpr int NW = PROBE_CUTS / 64;
    const int which = threadIdx.x / PROBE_CUTS, t = threadIdx.x % PROBE_CUTS, lane = t & 63;
    const int need = which == 0 ? n : 1;
    double a = lo, b = hi;
    for (int it = 0; it < PROBE_ROUNDS; ++it) {
        const double h = (b - a) / (double)(PROBE_CUTS + 1);
        const double x = a + h * (double)(t + 1);
        const bool ok = tridiag_count_below(al, be, n, x) >= need;
        const unsigned long long mask = __ballot(ok);
        // the first trial point of this wavefront that reaches the count, PROBE_CUTS when none does
        int* fs = first_s[which][it & 1];
        if (lane == 0) fs[t >> 6] = mask ? (t & ~63) + __ffsll((long long)mask) - 1 : PROBE_CUTS;
        __syncthreads();
        int first = PROBE_CUTS;
#pragma unroll
        for (int g = 0; g < NW; ++g) first = min(first, fs[g]);
        const double na = a + h * (double)first, nb = first < PROBE_CUTS ? a + h * (double)(first + 1) : b;
        a = na; b = nb;
    }
    if (t == 0) res[which] = 0.5 * (a + b);
    __syncthreads();
    if (threadIdx.x == 0) {
        const double lmax = res[0], lmin = res[1];
        out[0] = (float)lmax;
        out[1] = (float)lmin;
        out[2] = lmin > 0.0 ? (float)(lmax / lmin) : __builtin_inff();
        out[3] = (float)n;
    }
}

}  // namespace

namespace {
struct ProbeWs { size_t Q, w, alpha, beta, st, part, total, ld; };
ProbeWs probe_layout(int M, int k) {
    ProbeWs L;
    L.ld = align_up((size_t)M, 32);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes, 256); return at; };
    L.Q = take((size_t)(k + 1) * L.ld * sizeof(double));
    L.w = take(L.ld * sizeof(double));
    L.alpha = take(PROBE_MAX_K * sizeof(double));
    L.beta = take(PROBE_MAX_K * sizeof(double));
    L.st = take(sizeof(ProbeState));
    const size_t nb = ((size_t)M + PROBE_WG - 1) / PROBE_WG;
    L.part = take((2 * nb * (PROBE_MAX_K + 1) + 2 * nb) * sizeof(double));
    L.total = o;
    return L;
}
}  // namespace

size_t cond_probe_workspace_bytes(int M, int k) { return probe_layout(M, k < 1 ? 1 : (k > PROBE_MAX_K ? PROBE_MAX_K : k)).total; }

fw_status cond_probe(const float* Phi_y, int M, const float* b0, int k, float* out, void* ws, hipStream_t st) {
    const ProbeWs L = probe_layout(M, k);
    char* base = reinterpret_cast<char*>(ws);
    double* Qb = reinterpret_cast<double*>(base + L.Q);
    double* w = reinterpret_cast<double*>(base + L.w);
    double* alpha = reinterpret_cast<double*>(base + L.alpha);
    double* beta = reinterpret_cast<double*>(base + L.beta);
    ProbeState* ps = reinterpret_cast<ProbeState*>(base + L.st);
    double* part = reinterpret_cast<double*>(base + L.part);
    hipLaunchKernelGGL(probe_init_kernel, dim3(1), dim3(1024), 0, st, b0, M, Qb, ps);
    for (int j = 0; j < k; ++j) {
        hipLaunchKernelGGL(probe_matvec_kernel, dim3((M + 3) / 4), dim3(256), 0, st, Phi_y, Qb + (size_t)j * L.ld, M, w, ps);
        if (M > PROBE_SPREAD_MIN_M) {
            // many features: the step spread over ceil(M / 256) workgroups, four launches
            const dim3 g((M + PROBE_WG - 1) / PROBE_WG), blk(PROBE_WG);
            hipLaunchKernelGGL(probe_orth_phase_kernel<1>, g, blk, 0, st, j, M, L.ld, Qb, w, part, alpha, beta, 1e-7, ps);
            hipLaunchKernelGGL(probe_orth_phase_kernel<2>, g, blk, 0, st, j, M, L.ld, Qb, w, part, alpha, beta, 1e-7, ps);
            hipLaunchKernelGGL(probe_orth_phase_kernel<3>, g, blk, 0, st, j, M, L.ld, Qb, w, part, alpha, beta, 1e-7, ps);
            hipLaunchKernelGGL(probe_orth_phase_kernel<4>, g, blk, 0, st, j, M, L.ld, Qb, w, part, alpha, beta, 1e-7, ps);
        }
#define FW_PROBE_ORTH(E, NB, H) hipLaunchKernelGGL((probe_orth_kernel<E, NB, H>), dim3(1), dim3(1024), 0, st, j, M, L.ld, Qb, w, alpha, beta, 1e-7, ps)
        else if (M > 1024) {
            if (j < 8) FW_PROBE_ORTH(2, 8, 1);
            else if (j < 16) FW_PROBE_ORTH(2, 16, 1);
            else FW_PROBE_ORTH(2, 16, 2);
        }
        else if (j < 8) FW_PROBE_ORTH(1, 8, 1);
        else if (j < 16) FW_PROBE_ORTH(1, 16, 1);
        else FW_PROBE_ORTH(1, 32, 1);
#undef FW_PROBE_ORTH
    }
    hipLaunchKernelGGL(probe_final_kernel, dim3(1), dim3(2 * PROBE_CUTS), 0, st, alpha, beta, ps, out);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// ---- measurement helper: what the bfloat16 matrix cores sustain when every compute unit does nothing but dense
// v_mfma_f32_32x32x16_bf16 (the ceiling under the chip's power limit, against which the product kernels are read).
// A wavefront holds four A and four B fragments in registers (pseudo-random bfloat16 values in [-2, 2), or zeros) and
// runs `iters` rounds of the 16 products a_i b_j on 16 independent accumulators; the accumulators are added into `sink`
// at the end so that nothing is optimised away.
namespace {
constexpr int RATE_WGS = 1024;
__global__ __launch_bounds__(256) void mfma_rate_kernel(int zero_operands, int iters, float* __restrict__ sink) {
    bf16x8 a[4], b[4];
    unsigned h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
    for (int f = 0; f < 8; ++f) {
        unsigned short v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            h ^= h << 13; h ^= h >> 17; h ^= h << 5;
            // sign, exponent 126..128 (values in [0.5, 4)), 7 mantissa bits
            v[i] = zero_operands ? (unsigned short)0 : (unsigned short)(((h >> 3) & 0x8000u) | ((126u + (h >> 20) % 3u) << 7) | (h & 0x7Fu));
        }
        union { unsigned short u[8]; bf16x8 x; } cv;
#pragma unroll
        for (int i = 0; i < 8; ++i) cv.u[i] = v[i];
        if (f < 4) a[f] = cv.x; else b[f - 4] = cv.x;
    }
    floatx16 acc[16];
#pragma unroll
    for (int t = 0; t < 16; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t >> 2], b[t & 3], acc[t], 0, 0, 0);
    }
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 16; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += acc[t][i];
    if (sum == 123.456f) sink[0] = sum;     // never true for these operands: keeps the products alive without a store per lane
}
}  // namespace

fw_status mfma_rate_probe(int zero_operands, int iters, float* sink, double* flops, hipStream_t st) {
    hipLaunchKernelGGL(mfma_rate_kernel, dim3(RATE_WGS), dim3(256), 0, st, zero_operands, iters, sink);
    FW_LAUNCH_CHECK();
    if (flops) *flops = (double)RATE_WGS * 4.0 * (double)iters * 16.0 * 2.0 * 32.0 * 32.0 * 16.0;
    return FW_OK;
}

fw_status bias_compensate(float* b, const float* W, int S, int M, int taps, const float* mu_old, const float* mu_new, float scale,
                          hipStream_t st) {
    hipLaunchKernelGGL(bias_compensate_kernel, dim3((S + 3) / 4), dim3(256), 0, st, b, W, S, M, taps, mu_old, mu_new, scale);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

size_t diagnostics_workspace_bytes(int M) { return align_up((size_t)M * sizeof(float), 256) + align_up((size_t)M * sizeof(double), 256); }

fw_status diagnostics(const float* Phi_y, const float* lambda, int M, float* out, void* ws, hipStream_t st) {
    double* rowsum = nullptr;
    if (Phi_y) {
        float* d = reinterpret_cast<float*>(ws);
        rowsum = reinterpret_cast<double*>(reinterpret_cast<char*>(ws) + align_up((size_t)M * sizeof(float), 256));
        hipLaunchKernelGGL(diag_extract_kernel, dim3((M + 255) / 256), dim3(256), 0, st, Phi_y, M, d);
        hipLaunchKernelGGL(whiteness_rows_kernel, dim3((M + 3) / 4), dim3(256), 0, st, Phi_y, d, M, rowsum);
        FW_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(diagnostics_final_kernel, dim3(1), dim3(1024), 0, st, rowsum, lambda, M, out);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

}  // namespace fw
