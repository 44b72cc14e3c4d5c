// Float32 products on the bfloat16 matrix cores:  C = A B^T  for row-major float32 (or bfloat16) A [S, K] and float32 B [N, K].
//
// A float32 number is x = h + 2^-16 (m + l) with three bfloat16 numbers h = bf16(x), m = bf16(2^16 (x - h)), l = bf16(2^16 (x - h) - m),
// each difference exact (splitting into three bfloat16 numbers: G. Henry, P. T. P. Tang, A. Heinecke 2019).  bfloat16 has the
// exponents of float32 but ends 16 bits earlier, at 2^-133: without the factor the last part of a number below 2^-110 is lost (4e-6 of
// it at 2^-116, 1e-3 at 2^-124), with it all 24 bits are kept down to the smallest one.
// Of the nine products of two such sums the six above 2^-24 are taken, h h, h m, m h, m m, h l, l h, on v_mfma_f32_32x32x16_bf16
// (sixteen times the rate of the float32 instruction).  A bfloat16 gradient is its own h: three products.  Products with the same
// factor share accumulators, one set for each half of a chunk, so that a rounding of a partial sum of the large products h h
// happens K / 32 times in a chain and the five small ones do not add to it.
//
// Infinite entries, and those above 2^112, have no such sum, and sums of products above that overflow with it: the result is infinite or
// NaN then.  A wavefront that sees such a result multiplies its 32 x 32 results once more in float32, so that they are what the
// float32 instruction gives.
//
// The operands are read as they lie in memory and split on the way into LDS: no packing pass and no workspace.
#include "fw_internal.h"
#include "gemm_emit.h"

namespace fw {
namespace {

constexpr int KC = 32;            // contraction entries per chunk

constexpr int TR = 64, TC = 64;   // output tile of a workgroup
constexpr int NT = 512;           // eight wavefronts: 2 x 2 of 32 x 32 results, twice, each set with a half of every chunk
constexpr int PITCH = TR + TC + 4;    // 16-byte units per group of 8 entries: the four groups of a row fall into different banks
constexpr int STAGE = 3 * 4 * PITCH;  // [plane][group of 8 entries][row: A's, then B's]

struct Raw { float4 a, b; };

__device__ __forceinline__ void split8(const float (&x)[8], uint4& h, uint4& m, uint4& l) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    unsigned hp[4], mp[4], lp[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float x0 = x[2 * k], x1 = x[2 * k + 1];
        union { bf2 v; unsigned u; } p;
        p.v[0] = (__bf16)x0; p.v[1] = (__bf16)x1;
        hp[k] = p.u;
        const float r0 = fmaf(-65536.f, __uint_as_float(p.u << 16), 65536.f * x0), r1 = fmaf(-65536.f, __uint_as_float(p.u & 0xffff0000u), 65536.f * x1);
        p.v[0] = (__bf16)r0; p.v[1] = (__bf16)r1;
        mp[k] = p.u;
        const float s0 = r0 - __uint_as_float(p.u << 16), s1 = r1 - __uint_as_float(p.u & 0xffff0000u);
        p.v[0] = (__bf16)s0; p.v[1] = (__bf16)s1;
        lp[k] = p.u;
    }
    h = make_uint4(hp[0], hp[1], hp[2], hp[3]);
    m = make_uint4(mp[0], mp[1], mp[2], mp[3]);
    l = make_uint4(lp[0], lp[1], lp[2], lp[3]);
}

// lower: of a square result the tiles that touch the lower triangle
template <bool ABF16>
__global__ __launch_bounds__(NT) void gemm_planes_kernel(const void* __restrict__ Av, const float* __restrict__ B, GemmEpilogue Out, int S, int N,
                                                         int K, int lower, int tiles) {
    __shared__ uint4 lds[2][STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    // consecutive workgroups go to the 8 XCDs in turn: each gets a contiguous run of tiles, whose rows of A its L2 then holds
    const int per_xcd = (tiles + 7) / 8;
    const int tile = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (tile >= tiles || ((int)blockIdx.x >> 3) >= per_xcd) return;
    int I, J;
    if (lower) {
        I = (int)((sqrtf(8.f * (float)tile + 1.f) - 1.f) * 0.5f);
        while ((I + 1) * (I + 2) / 2 <= tile) ++I;
        while (I * (I + 1) / 2 > tile) --I;
        J = tile - I * (I + 1) / 2;
    } else {
        const int ncb = (N + TC - 1) / TC;
        I = tile / ncb;
        J = tile - I * ncb;
    }
    const int row0 = I * TR, col0 = J * TC;
    const int part = wave >> 2, wr = (wave >> 1) & 1, wc = wave & 1;
    const int nfull = K / KC;

    // a thread brings 8 entries of one staged row per chunk.  Rows past the end are clamped: they only feed results that are not stored.
    const int kg = tid & 3, rr = tid >> 2;
    const bool is_a = rr < TR;                        // the same for a whole wavefront
    const size_t off = (size_t)(is_a ? min(row0 + rr, S - 1) : min(col0 + rr - TR, N - 1)) * K + 8 * kg;
    const float* src32 = (is_a ? reinterpret_cast<const float*>(Av) : B) + off;
    const unsigned short* src16 = reinterpret_cast<const unsigned short*>(Av) + off;
    Raw raw[2];
    auto load = [&](int c, Raw& r) {                  // of a whole chunk; rows need not be 16-byte aligned
        if (ABF16 && is_a) {
            __builtin_memcpy(&r.a, src16 + (size_t)c * KC, 16);
        } else {
            __builtin_memcpy(&r.a, src32 + (size_t)c * KC, 16);
            __builtin_memcpy(&r.b, src32 + (size_t)c * KC + 4, 16);
        }
    };
    auto load_ragged = [&](Raw& r) {                  // the last chunk, zero beyond the end
        const int left = K - nfull * KC - 8 * kg;
        const size_t at = (size_t)nfull * KC;
        float x[8];
        if (ABF16 && is_a) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                x[k] = __uint_as_float((2 * k < left ? (unsigned)src16[at + 2 * k] : 0u) | (2 * k + 1 < left ? (unsigned)src16[at + 2 * k + 1] << 16 : 0u));
#pragma unroll
            for (int k = 4; k < 8; ++k) x[k] = 0.f;
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = k < left ? src32[at + k] : 0.f;
        }
        r.a = make_float4(x[0], x[1], x[2], x[3]);
        r.b = make_float4(x[4], x[5], x[6], x[7]);
    };
    auto stage = [&](int c, const Raw& r) {
        uint4* at = lds[c & 1] + kg * PITCH + rr;
        if (ABF16 && is_a) {
            *reinterpret_cast<float4*>(at) = r.a;
            return;
        }
        const float x[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
        uint4 h, m, l;
        split8(x, h, m, l);
        at[0] = h;
        at[4 * PITCH] = m;
        at[8 * PITCH] = l;
    };

    floatx16 big, small, mm;                          // results times 1, 2^16, 2^32
#pragma unroll
    for (int i = 0; i < 16; ++i) big[i] = small[i] = mm[i] = 0.f;
    auto multiply = [&](int c) {
        const uint4* at = lds[c & 1] + (2 * part + half) * PITCH + l32;
        auto a = [&](int pl) { return *reinterpret_cast<const bf16x8*>(at + pl * 4 * PITCH + 32 * wr); };
        auto b = [&](int pl) { return *reinterpret_cast<const bf16x8*>(at + pl * 4 * PITCH + TR + 32 * wc); };
        const bf16x8 ah = a(0), bh = b(0), bm = b(1), bl = b(2);
        big = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, big, 0, 0, 0);
        if constexpr (!ABF16) {
            const bf16x8 am = a(1), al = a(2);
            small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, small, 0, 0, 0);
            mm = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bm, mm, 0, 0, 0);
            small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh, small, 0, 0, 0);
        }
        small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, small, 0, 0, 0);
        small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bm, small, 0, 0, 0);
    };
    auto barrier = [] {
        FW_WAIT_LGKM0();
        __builtin_amdgcn_s_barrier();
        FW_COMPILER_FENCE();
    };

    if (nfull > 0) {
        // chunk c in LDS, c + 1 and c + 2 in registers or on their way; one barrier per chunk: the buffer that chunk c + 1 goes to was
        // read before the barrier that ended chunk c - 1.  Past the end the last chunk is loaded and staged again, unread, so that
        // no branch stands between a load and its use (the compiler would wait for all loads there).
        const int last = nfull - 1;
        load(0, raw[0]);
        load(min(1, last), raw[1]);
        stage(0, raw[0]);
        load(min(2, last), raw[0]);
        barrier();
        auto turn = [&](int c, Raw& next) {
            stage(c + 1, next);
            load(min(c + 3, last), next);
            multiply(c);
            barrier();
        };
        int c = 0;
        for (; c + 1 < nfull; c += 2) {
            turn(c, raw[1]);
            turn(c + 1, raw[0]);
        }
        if (c < nfull) turn(c, raw[1]);
    }
    if (nfull * KC < K) {
        load_ragged(raw[0]);
        stage(nfull, raw[0]);
        barrier();
        multiply(nfull);
        barrier();
    }

#pragma unroll
    for (int i = 0; i < 16; ++i) big[i] += 0x1p-16f * (ABF16 ? small[i] : small[i] + 0x1p-16f * mm[i]);
    float* red = reinterpret_cast<float*>(lds);       // the two sets' halves of the sum: [wavefront of the set][register][lane]
    static_assert(TR * TC * 4 <= (int)sizeof(lds), "room for the partial tile");
    if (part == 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[((wave & 3) * 16 + i) * 64 + lane] = big[i];
    }
    __syncthreads();
    if (part == 1) return;
    const int col = col0 + 32 * wc + l32;
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        big[i] += red[((wave & 3) * 16 + i) * 64 + lane];
        finite &= fabsf(big[i]) <= 3.402823466e38f;
    }
    if (__any(!finite)) {
        const size_t arow = (size_t)min(row0 + 32 * wr + l32, S - 1) * K;
        const float* a32 = reinterpret_cast<const float*>(Av) + arow;
        const unsigned short* a16 = reinterpret_cast<const unsigned short*>(Av) + arow;
        const float* b32 = B + (size_t)min(col, N - 1) * K;
#pragma unroll
        for (int i = 0; i < 16; ++i) big[i] = 0.f;
        for (int k0 = 0; k0 < K; k0 += 2) {           // lanes below 32 have entry k0, the others k0 + 1
            const int k = k0 + half;
            const float x = k < K ? (ABF16 ? bf16_to_f32(a16[k]) : a32[k]) : 0.f, y = k < K ? b32[k] : 0.f;
            big = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, big, 0, 0, 0);
        }
    }
    const auto row_of = [&](int i) { return row0 + 32 * wr + 8 * (i >> 2) + 4 * half + (i & 3); };
    if (Out.W && !Out.out) {
        if (col < N) emit_update<16>(Out, row_of, col, S, N, big);
        return;
    }
    const bool plain = Out.out && !Out.out_bf16 && Out.taps == 1 && !Out.W;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = row_of(i);
        if (row < S && col < N) {
            if (plain) reinterpret_cast<float*>(Out.out)[(size_t)row * N + col] = big[i];
            else emit(Out, row, col, N, big[i]);
        }
    }
}

inline long long tiles_of(int S, int N, bool lower) {
    const long long tr = (S + TR - 1) / TR, tc = (N + TC - 1) / TC;
    return lower ? tr * (tr + 1) / 2 : tr * tc;
}

}  // namespace

// C = A B^T, A [S, K] float32 (or bfloat16 bits), B [N, K] float32; lower: S == N and only the lower triangle is wanted
fw_status gemm_planes(const void* A, bool a_bf16, int S, int N, int K, const float* B, const GemmEpilogue& e, bool lower, hipStream_t st) {
    const long long tiles = tiles_of(S, N, lower);
    if (tiles > (1 << 30)) return FW_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)((tiles + 7) / 8 * 8));
    if (a_bf16) hipLaunchKernelGGL(gemm_planes_kernel<true>, grid, dim3(NT), 0, st, A, B, e, S, N, K, lower ? 1 : 0, (int)tiles);
    else hipLaunchKernelGGL(gemm_planes_kernel<false>, grid, dim3(NT), 0, st, A, B, e, S, N, K, lower ? 1 : 0, (int)tiles);
    FW_LAUNCH_CHECK();
    return FW_OK;
}

// the float32 products it stands for (each is six bfloat16 ones), whole tiles and chunks
double gemm_planes_flops(int S, int N, int K, bool lower) {
    return 2.0 * (double)tiles_of(S, N, lower) * TR * TC * ((K + KC - 1) / KC * KC);
}

}  // namespace fw
