// EVD / ZCA whitening matrix (Sec. 2, eqs. (vPhix_evd), (vT_EVD), (vg); Sec. 3.2, eqs. (hMs), (g_mod)) for gfx950.
//
// Phi_x = V^T Lambda V with the eigenvectors as rows of V, in float64 inside the workspace (small eigenvalues carry the
// largest gains): reduction to tridiagonal form, divide and conquer, back-transformation (symeig.hip).  The result is then
// CHECKED against Phi_x itself: W = V Phi_x, and every off-diagonal entry of W V^T must lie below kAccept sqrt(D_i D_j), D_i
// = sum_k v_ik^2 Phi_kk, i.e. a thousandth of what the storage of Phi_x as float32 leaves undetermined in that entry, or
// below kAcceptClamp times the eigenvalue at which the gains are clamped; and V V^T must agree with the identity to kAccept
// (rows that Phi_x takes to zero carry the largest gain and are seen by nothing else; by eight products with vectors where M
// is large).  Where V fails that, it is given up for V = I.  Where neither of the first two holds (diagonals graded over
// many decades above the clamp), or where the caller asks for a rotation threshold of its own (tol > 0), a one-sided Jacobi
// iteration goes on from there: orthogonal transformations are applied to the rows of W = V Phi_x and of V until the rows of
// W are mutually orthogonal; then W = Lambda V and lambda_k = w_k . v_k.  The iteration is blocked: rows are cut into blocks
// of 32, a round of the round-robin schedule takes disjoint pairs of blocks, and for every pair (64 rows) three kernels run:
// the 64x64 Gram matrix of the rows (partial sums over column slices), its diagonalisation by a cyclic two-sided Jacobi
// iteration in LDS, which yields the 64x64 rotation that makes the 64 rows orthogonal to each other, and the application of
// that rotation to the rows of W and V.  T = V^T diag(sqrt g) V and Q = V^T diag(g) V: in float64, or for many features as
// split products on the bfloat16 matrix cores (gemm_split.hip).
//
// Why not Jacobi alone: from V = I it needs 13 to 19 sweeps that each stream W and V once per round.  One call took
// 31 ms at M = 576, 175 ms at 2304 and 0.86 s at 4608; this way 3.6, 22.7 and 121 ms.
#include "fw_internal.h"

namespace fw {
namespace {

constexpr int JB = 32;        // rows per block
constexpr int JP = 2 * JB;    // rows per pair of blocks
constexpr int JSW = 512;      // columns per slice of the Gram kernel
constexpr double kAccept = 1.0 / (1ull << 34);   // 2^-10 of the float32 rounding 2^-24
constexpr double kAcceptClamp = 1.0 / (1ull << 30);

struct EvdWs {
    size_t mat[4], small, lam, gq, gh, tot, cnt, total;
    int nblk, nblk_even, npairs, nslices;
};
// T and Q from the scaled eigenvectors: from FW_REFRESH_SPLIT_MIN_M features on as split products on the bfloat16 matrix
// cores, below that in float64.  Measured at M = 2304 for T and Q together: split 0.20 ms, float64 0.32 ms; at M = 576 one
// float64 launch takes 20 us where two float32 covariance products with their reduction and mirror passes took 60.
inline bool evd_products_split(int M) { return M >= FW_REFRESH_SPLIT_MIN_M; }
inline EvdWs evd_layout(int M) {
    EvdWs L;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes, 256); return at; };
    L.nblk = (M + JB - 1) / JB;
    L.nblk_even = (L.nblk + 1) & ~1;
    L.npairs = L.nblk_even / 2;
    L.nslices = (M + JSW - 1) / JSW;
    // Four float64 matrices: [0] Phi while it is reduced, then vectors of the merges, projections, a copy of Phi, partial Gram
    // matrices; [1] reflectors, then rotations, packed planes and the scaled eigenvectors; [2], [3] eigenvectors and their
    // image V Phi.
    size_t m = sym_eig_matrix_doubles(M);
    const size_t g = (size_t)L.npairs * L.nslices * JP * JP;
    if (g > m) m = g;
    m *= sizeof(double);
    const size_t products = evd_products_split(M) ? gemm_split_packed_bytes(M, M) + (size_t)M * M * sizeof(float) : 0;
    for (int k = 0; k < 4; ++k) L.mat[k] = take(k == 1 && products > m ? products : m);
    L.small = take(sym_eig_small_bytes(M));
    L.lam = take((size_t)M * sizeof(double));
    L.gq = take((size_t)M * sizeof(double));
    L.gh = take((size_t)M * sizeof(double));
    L.tot = take(256);
    L.cnt = take(256);
    L.total = o;
    return L;
}

// One round of the round-robin ordering over n (even) players; pair k of round r.
__device__ __forceinline__ void rr_pair(int n, int r, int k, int* a, int* b) {
    const int m = n - 1;
    if (k == 0) { *a = m; *b = r; }
    else { *a = (r + k) % m; *b = (r - k + m) % m; }
}

// global row of member k (0..63) of the block pair (p, q); -1 if it does not exist
__device__ __forceinline__ int pair_row(int p, int q, int nblk, int M, int k) {
    const int blk = k < JB ? p : q;
    const int r = blk * JB + (k & (JB - 1));
    return (blk < nblk && r < M) ? r : -1;
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Partial Gram matrices: Gpart[pair][slice] = R_slice R_slice^T for the 64 rows R of the pair restricted to a slice of
// JSW columns, on v_mfma_f64_16x16x4_f64 (operand lane l: row l % 16, contraction entry l / 16; result register v of
// lane l: row 4 v + l / 16, column l % 16).  Chunks of 32 columns are staged in LDS; the four wavefronts take
// different 4-column steps of a chunk and each of them updates the ten 16x16 tiles of the lower triangle, both
// operands of a tile being fragments of the same staged rows; the four partial results are summed through LDS in
// wavefront order.
__global__ __launch_bounds__(256) void gram_kernel(const double* __restrict__ W, int ld, int M, int nblk, int nblk_even, int round,
                                                   int nslices, double* __restrict__ Gpart) {
    __shared__ double Xs[JP][33];
    __shared__ double red[40][64];
    int a, b;
    rr_pair(nblk_even, round, blockIdx.y, &a, &b);
    const int p = min(a, b), q = max(a, b);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lq = lane >> 4;
    doublex4 acc[10];
#pragma unroll
    for (int t = 0; t < 10; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
    const int c_begin = blockIdx.x * JSW, c_end = min(M, c_begin + JSW);
    // this thread's eight entries of a chunk: row (tid + 256 m) / 32, column (tid + 256 m) % 32; fetched one chunk ahead
    int grow[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) grow[m] = pair_row(p, q, nblk, M, (threadIdx.x + 256 * m) >> 5);
    const int cc = threadIdx.x & 31;
    double nxt[8];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int m = 0; m < 8; ++m) nxt[m] = (grow[m] >= 0 && c0 + cc < c_end) ? W[(size_t)grow[m] * ld + c0 + cc] : 0.0;
    };
    fetch(c_begin);
    for (int c0 = c_begin; c0 < c_end; c0 += 32) {
#pragma unroll
        for (int m = 0; m < 8; ++m) Xs[(threadIdx.x + 256 * m) >> 5][cc] = nxt[m];
        __syncthreads();
        if (c0 + 32 < c_end) fetch(c0 + 32);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ks = wave + 4 * h;
            double f[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) f[t] = Xs[16 * t + lr][4 * ks + lq];
            int n = 0;
#pragma unroll
            for (int ta = 0; ta < 4; ++ta)
#pragma unroll
                for (int tb = 0; tb <= ta; ++tb, ++n) acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[ta], f[tb], acc[n], 0, 0, 0);
        }
        __syncthreads();
    }
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int t = 0; t < 10; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double* slot = &red[t * 4 + v][lane];
                    *slot = w == 0 ? acc[t][v] : *slot + acc[t][v];
                }
        }
        __syncthreads();
    }
    double* dst = Gpart + ((size_t)blockIdx.y * nslices + blockIdx.x) * (JP * JP);
    for (int e = threadIdx.x; e < 40 * 64; e += 256) {
        const int tv = e >> 6, l = e & 63;
        const int t = tv >> 2, v = tv & 3;
        int ta = 0, base = 0;
        while (base + ta + 1 <= t) { base += ta + 1; ++ta; }   // tile t = ta (ta + 1) / 2 + tb
        const int tb = t - base;
        const int i = 16 * ta + 4 * v + (l >> 4), j = 16 * tb + (l & 15);
        const double g = red[tv][l];
        dst[i * JP + j] = g;
        dst[j * JP + i] = g;
    }
}

// Diagonalisation of the 64x64 Gram matrix of a pair: cyclic Jacobi with 32 disjoint index pairs per step (32 threads
// per index pair: half a wavefront).  The accumulated rotation R (new rows = R old rows, R G R^T diagonal) goes to Rot[pair];
// flags[pair] = 1 if any rotation was applied, and the counter gets the number applied in the first inner sweep.
__global__ __launch_bounds__(1024) void pair_evd_kernel(const double* __restrict__ Gpart, int nslices, double tol, int inner_sweeps,
                                                       double* __restrict__ Rot,
                                                       int* __restrict__ flags, int* __restrict__ counter) {
    __shared__ double Gs[JP][JP + 1], Rs[JP][JP + 1];
    __shared__ int n_rot, n_first;
    const int tid = threadIdx.x;
    const int kk = tid >> 5, sub = tid & 31;
    for (int e = tid; e < JP * JP; e += 1024) {
        const double* src = Gpart + (size_t)blockIdx.x * nslices * (JP * JP) + e;
        double g = 0.0;
        for (int sl = 0; sl < nslices; ++sl) g += src[(size_t)sl * (JP * JP)];
        Gs[e >> 6][e & 63] = g;
        Rs[e >> 6][e & 63] = (e >> 6) == (e & 63) ? 1.0 : 0.0;
    }
    if (tid == 0) { n_rot = 0; n_first = 0; }
    __syncthreads();
    int total = 0;
    for (int sweep = 0; sweep < inner_sweeps; ++sweep) {
        for (int step = 0; step < JP - 1; ++step) {
            int i, j;
            rr_pair(JP, step, kk, &i, &j);
            if (i > j) { const int t = i; i = j; j = t; }
            // every thread of the index pair works out the rotation for itself: the 32 of them sit in one wavefront,
            // so all of them have read the three entries before any of them rewrites rows i and j
            const double al = Gs[i][i], be = Gs[j][j], ga = Gs[i][j];
            double c = 1.0, s = 0.0;
            if (fabs(ga) > tol * sqrt(fabs(al * be)) && ga != 0.0) {
                const double tau = be - al;
                const double tt = (tau >= 0.0 ? 2.0 : -2.0) * ga / (fabs(tau) + sqrt(tau * tau + 4.0 * ga * ga));
                c = rsqrt(1.0 + tt * tt);
                s = c * tt;
                if (sub == 0) atomicAdd(&n_rot, 1);
            }
            if (s != 0.0) {   // rows i, j of G and of R
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int col = sub + 32 * m;
                    const double x = Gs[i][col], y = Gs[j][col];
                    Gs[i][col] = c * x - s * y; Gs[j][col] = s * x + c * y;
                    const double e = Rs[i][col], f = Rs[j][col];
                    Rs[i][col] = c * e - s * f; Rs[j][col] = s * e + c * f;
                }
            }
            __syncthreads();
            if (s != 0.0) {   // columns i, j of G
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int row = sub + 32 * m;
                    const double x = Gs[row][i], y = Gs[row][j];
                    Gs[row][i] = c * x - s * y; Gs[row][j] = s * x + c * y;
                }
            }
            __syncthreads();
        }
        const int r = n_rot;      // every thread reads the same value: the last barrier of the step loop has passed
        __syncthreads();
        if (tid == 0) { if (sweep == 0) n_first = r; n_rot = 0; }
        __syncthreads();
        total += r;
        if (r == 0) break;
    }
    if (total > 0)
        for (int e = tid; e < JP * JP; e += 1024) Rot[(size_t)blockIdx.x * (JP * JP) + e] = Rs[e >> 6][e & 63];
    if (tid == 0) {
        flags[blockIdx.x] = total > 0 ? 1 : 0;
        if (n_first > 0) atomicAdd(counter, n_first);
    }
}

// rows of the pair <- R rows, for W (blockIdx.z = 0) and V (1), on v_mfma_f64_16x16x4_f64: a wavefront keeps all
// fragments of R in registers and takes groups of 16 columns; the 64 x 16 block of a group is read into registers
// before any of it is written back.
__global__ __launch_bounds__(256) void rotate_rows_kernel(double* __restrict__ W, double* __restrict__ V, int ld, int M, int nblk,
                                                          int nblk_even, int round, const double* __restrict__ Rot,
                                                          const int* __restrict__ flags) {
    __shared__ double Rs[JP][JP + 1];
    if (flags[blockIdx.y] == 0) return;
    int a, b;
    rr_pair(nblk_even, round, blockIdx.y, &a, &b);
    const int p = min(a, b), q = max(a, b);
    for (int e = threadIdx.x; e < JP * JP; e += 256) Rs[e >> 6][e & 63] = Rot[(size_t)blockIdx.y * (JP * JP) + e];
    __syncthreads();
    double* Mat = blockIdx.z == 0 ? W : V;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lq = lane >> 4;
    double ra[4][16];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) ra[t][ks] = Rs[16 * t + lr][4 * ks + lq];
    int rowk[16];   // global rows of this lane's contraction entries 4 ks + lq
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) rowk[ks] = pair_row(p, q, nblk, M, 4 * ks + lq);
    for (int gi = 0; gi < 8; ++gi) {
        const int col0 = blockIdx.x * 512 + (wave * 8 + gi) * 16;
        if (col0 >= M) break;
        const int col = col0 + lr;
        const bool cok = col < M;
        double xb[16];
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) xb[ks] = (rowk[ks] >= 0 && cok) ? Mat[(size_t)rowk[ks] * ld + col] : 0.0;
        doublex4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[t][ks], xb[ks], acc[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gr = pair_row(p, q, nblk, M, 16 * t + 4 * v + lq);
                if (gr >= 0 && cok) Mat[(size_t)gr * ld + col] = acc[t][v];
            }
    }
}

__global__ void zero_int_kernel(int* p) { *p = 0; }

// lambda_k = w_k . v_k (signed), one wavefront per row
__global__ __launch_bounds__(256) void eig_kernel(const double* __restrict__ W, const double* __restrict__ V, int ld, int M,
                                                  double* __restrict__ lam) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= M) return;
    double acc = 0.0;
    for (int j = lane; j < M; j += 64) acc += W[(size_t)r * ld + j] * V[(size_t)r * ld + j];
    acc = wave_sum(acc);
    if (lane == 0) lam[r] = acc;
}

// tot[0] = sum of the positive eigenvalues, tot[1] = Ms_hat = exp(-sum lb log lb), lb = lambda / tot[0] (exponential of the
// spectral entropy; reading of eq. (hMs)).  One workgroup.
__global__ __launch_bounds__(1024) void spectrum_kernel(const double* __restrict__ lam, int M, double* __restrict__ tot_out) {
    __shared__ double red[16];
    __shared__ double s_tot;
    double tot = 0.0;
    for (int k = threadIdx.x; k < M; k += 1024) tot += fmax(lam[k], 0.0);
    tot = wave_sum(tot);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tot;
    __syncthreads();
    if (threadIdx.x == 0) { double t = 0; for (int i = 0; i < 16; ++i) t += red[i]; s_tot = t; }
    __syncthreads();
    tot = s_tot;
    double ent = 0.0;
    for (int k = threadIdx.x; k < M; k += 1024) {
        const double lb = tot > 0.0 ? fmax(lam[k], 0.0) / tot : 0.0;
        if (lb > 0.0) ent -= lb * log(lb);
    }
    ent = wave_sum(ent);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ent;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0;
        for (int i = 0; i < 16; ++i) t += red[i];
        tot_out[0] = tot;
        tot_out[1] = tot > 0.0 ? exp(t) : 1.0;
    }
}

// Sorted eigenvalues (decreasing) and gain roots, one wavefront per eigenvalue: its sorted position is the number of
// eigenvalues ahead of it (M comparisons; 336 us at M = 2304 when a single workgroup did all of them, 10 us like this).
//  mode 0: g = 1/max(lambda, eps)                                          eq. (vg)
//  mode 1: g = min(1/(M lb), g_max) for sorted position < round(Ms_hat), 1 otherwise   eq. (g_mod)
__global__ __launch_bounds__(256) void gains_kernel(const double* __restrict__ lam, int M, const double* __restrict__ tot_in, float eps,
                                                    float g_max, int mode, float* __restrict__ lam_sorted, double* __restrict__ gq,
                                                    double* __restrict__ gh) {
    const int lane = threadIdx.x & 63, k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= M) return;
    const double lk = lam[k];
    int pos = 0;
    for (int j = lane; j < M; j += 64) {
        const double lj = lam[j];
        pos += (lj > lk || (lj == lk && j < k)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pos += __shfl_xor(pos, o, 64);
    if (lane != 0) return;
    lam_sorted[pos] = (float)lk;
    const double tot = tot_in[0];
    int rank_sig = M;
    if (mode == 1) {
        double r = floor(tot_in[1] + 0.5);
        if (r < 1.0) r = 1.0;
        if (r > (double)M) r = (double)M;
        rank_sig = (int)r;
    }
    double g;
    if (mode == 0) g = 1.0 / fmax(lk, (double)eps);
    else if (pos >= rank_sig) g = 1.0;
    else if (lk <= 0.0 || tot <= 0.0) g = (double)g_max;
    else g = fmin(tot / ((double)M * lk), (double)g_max);
    gh[k] = sqrt(g);
    gq[k] = sqrt(gh[k]);
}

// X[k][j] = scale[k] * V[k][j] as float32
__global__ __launch_bounds__(256) void scale_rows_kernel(const double* __restrict__ V, const double* __restrict__ scale, int ld, int M,
                                                         float* __restrict__ X) {
    const double f = scale[blockIdx.y];
    for (int j = blockIdx.x * 256 + threadIdx.x; j < M; j += gridDim.x * 256)
        X[(size_t)blockIdx.y * M + j] = (float)(f * V[(size_t)blockIdx.y * ld + j]);
}

__global__ __launch_bounds__(256) void ema_kernel(float* __restrict__ Qs, const float* __restrict__ Q, size_t n, float beta) {
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256)
        Qs[e] = beta * Qs[e] + (1.f - beta) * Q[e];
}

inline int grid_for(size_t n) {
    size_t b = (n + 255) / 256;
    return (int)(b > 8192 ? 8192 : b);
}

}  // namespace

// lambda (already in `lam`) -> sorted eigenvalues, gains, T and Q
static fw_status evd_outputs(const double* V, int M, const fw_evd_params* p, double* lam, double* gq, double* gh, double* tot, float* X,
                             void* planes, float* T, float* Q, float* lambda, hipStream_t st) {
    const int ld = sym_eig_ld(M);
    hipLaunchKernelGGL(spectrum_kernel, dim3(1), dim3(1024), 0, st, lam, M, tot);
    hipLaunchKernelGGL(gains_kernel, dim3((M + 3) / 4), dim3(256), 0, st, lam, M, tot, p->eps, p->g_max, p->gain_mode, lambda, gq, gh);
    FW_LAUNCH_CHECK();
    if (!evd_products_split(M)) return sym_eig_spectral_products(V, M, gh, T, Q, st);
    for (int which = 0; which < 2; ++which) {
        float* out = which == 0 ? T : Q;
        hipLaunchKernelGGL(scale_rows_kernel, dim3((M + 1023) / 1024, M), dim3(256), 0, st, V, which == 0 ? gq : gh, ld, M, X);
        FW_LAUNCH_CHECK();
        // X^T X = (X^T)(X^T)^T: the columns of X as hi + lo planes are both operands; lower triangle only
        fw_status rc = gemm_split_pack_transposed(X, M, M, planes, st);
        if (rc != FW_OK) return rc;
        rc = gemm_split_run(planes, planes, M, M, M, 1, out, st);
        if (rc != FW_OK) return rc;
        rc = symmetrize_from_lower(out, M, st);
        if (rc != FW_OK) return rc;
    }
    return FW_OK;
}

size_t evd_workspace_bytes(int M) { return evd_layout(M).total; }

fw_status whiten_evd(const float* Phi_x, int M, const fw_evd_params* p, float* T, float* Q, float* Qs, float* lambda, void* ws,
                     size_t ws_bytes, hipStream_t st, EvdRun* run) {
    const EvdWs L = evd_layout(M);
    if (ws_bytes < L.total) return FW_ERR_WORKSPACE;
    char* base = reinterpret_cast<char*>(ws);
    double* mat[4];
    for (int k = 0; k < 4; ++k) mat[k] = reinterpret_cast<double*>(base + L.mat[k]);
    double* lam = reinterpret_cast<double*>(base + L.lam);
    double* gq = reinterpret_cast<double*>(base + L.gq);
    double* gh = reinterpret_cast<double*>(base + L.gh);
    double* tot = reinterpret_cast<double*>(base + L.tot);
    int* cnt = reinterpret_cast<int*>(base + L.cnt);
    const int ld = sym_eig_ld(M);
    const double tol = p->tol > 0.f ? (double)p->tol : 1e-12;
    const int max_sweeps = p->max_sweeps > 0 ? p->max_sweeps : 30;

    double *V = mat[2], *W = mat[3];
    // eigenvalues below the clamp all have the clamp's gain: entries far below it cannot move a gain
    const double floor_abs = p->gain_mode == 0 ? kAcceptClamp * (double)p->eps : 0.0;
    const double floor_rel = p->gain_mode == 1 ? kAcceptClamp / ((double)M * (double)p->g_max) : 0.0;
    // A Phi_x that is diagonal already (features whitened before, a fresh state) needs no decomposition: 1.6 ms -> 0.1 ms at M = 300.
    // The look costs two launches and a wait, about 20 us; knowing that no feature is dead saves three launches again.
    int verdict[2] = {1, 1};
    fw_status rc = sym_eig_check_identity(Phi_x, M, base + L.small, kAccept, floor_abs, floor_rel, cnt, st);
    if (rc != FW_OK) return rc;
    FW_HIP_TRY(hipMemcpyAsync(verdict, cnt, sizeof(verdict), hipMemcpyDeviceToHost, st));
    FW_HIP_TRY(hipStreamSynchronize(st));
    const bool diagonal = verdict[0] == 0;
    if (run) { run->one_launch = 0; run->diagonal = diagonal ? 1 : 0; run->sweeps = 0; }
    if (diagonal) {
        rc = sym_eig_load(Phi_x, M, mat[0], st);
        if (rc != FW_OK) return rc;
        rc = sym_eig_start_over(mat[0], M, V, W, st);
        if (rc != FW_OK) return rc;
        hipLaunchKernelGGL(eig_kernel, dim3((M + 3) / 4), dim3(256), 0, st, W, V, ld, M, lam);
        FW_LAUNCH_CHECK();
    } else {
        rc = sym_eig(Phi_x, M, verdict[1] != 0, mat, base + L.small, &V, &W, st, run);
        if (rc != FW_OK) return rc;
        rc = sym_eig_check(Phi_x, M, V, W, mat[0], mat[1], base + L.small, kAccept, floor_abs, floor_rel, lam, cnt, st);
        if (rc != FW_OK) return rc;
    }
    // the outputs are issued before the host looks at the verdict, so that the GPU does not wait for it; they leave mat[0], the
    // copy of Phi, alone (T or Q may lie where Phi_x was)
    float* X = reinterpret_cast<float*>(reinterpret_cast<char*>(mat[1]) + (evd_products_split(M) ? gemm_split_packed_bytes(M, M) : 0));
    rc = evd_outputs(V, M, p, lam, gq, gh, tot, X, mat[1], T, Q, lambda, st);
    if (rc != FW_OK) return rc;
    if (diagonal) verdict[1] = 0;
    else {
        FW_HIP_TRY(hipMemcpyAsync(verdict, cnt, sizeof(verdict), hipMemcpyDeviceToHost, st));
        FW_HIP_TRY(hipStreamSynchronize(st));
    }
    bool converged = verdict[0] == 0 && verdict[1] == 0 && !(p->tol > 0.f);
    if (!converged) {
        // rotations keep V as orthogonal as it is, so one that is not (a Phi_x with NaN or infinite entries leaves none) is
        // given up: sweeps from V = I
        if (verdict[1] != 0) {
            rc = sym_eig_start_over(mat[0], M, V, W, st);
            if (rc != FW_OK) return rc;
        }
        double* Gpart = mat[0];
        double* Rot = mat[1];
        int* flags = reinterpret_cast<int*>(base + L.small);
        const int ncolblk = (M + 511) / 512;
        const int inner = 1;   // inner sweeps per visit of a pair: one was the fastest overall (more inner sweeps, fewer outer ones)
        for (int sweep = 0; sweep < max_sweeps && !converged; ++sweep) {
            hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, st, cnt);
            for (int r = 0; r < L.nblk_even - 1; ++r) {
                hipLaunchKernelGGL(gram_kernel, dim3(L.nslices, L.npairs), dim3(256), 0, st, W, ld, M, L.nblk, L.nblk_even, r, L.nslices, Gpart);
                hipLaunchKernelGGL(pair_evd_kernel, dim3(L.npairs), dim3(1024), 0, st, Gpart, L.nslices, tol, inner, Rot, flags, cnt);
                hipLaunchKernelGGL(rotate_rows_kernel, dim3(ncolblk, L.npairs, 2), dim3(256), 0, st, W, V, ld, M, L.nblk, L.nblk_even, r, Rot,
                                   flags);
            }
            FW_LAUNCH_CHECK();
            int rotations = -1;
            FW_HIP_TRY(hipMemcpyAsync(&rotations, cnt, sizeof(int), hipMemcpyDeviceToHost, st));
            FW_HIP_TRY(hipStreamSynchronize(st));
            converged = rotations == 0;
            if (run) ++run->sweeps;
        }
        hipLaunchKernelGGL(eig_kernel, dim3((M + 3) / 4), dim3(256), 0, st, W, V, ld, M, lam);
        FW_LAUNCH_CHECK();
        rc = evd_outputs(V, M, p, lam, gq, gh, tot, X, mat[1], T, Q, lambda, st);
        if (rc != FW_OK) return rc;
    }
    if (Qs) {
        const size_t n = (size_t)M * M;
        hipLaunchKernelGGL(ema_kernel, dim3(grid_for(n)), dim3(256), 0, st, Qs, Q, n, p->beta);
        FW_LAUNCH_CHECK();
    }
    return converged ? FW_OK : FW_ERR_NOT_CONVERGED;
}

}  // namespace fw
