// Float32 GEMM on the matrix cores: out[M][N] = a[M][K] * w[N][K]^T and the same epilogues as the bf16 GEMMs
// (the projections of a float32 model, Sec. 3).  Any M and N, K a multiple of 4.
//
// MFMA used: v_mfma_f32_16x16x4_f32.  For D[16x16] += A[16x4] * B[4x16] lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and holds D[4*(l/16) + v][l%16] in accumulator register v (0..3).  Both operands use the same
// permutation of K, so a lane reads 16 bytes of its row (elements 16b + 4*(l/16) .. + 3) for four MFMAs.
//
// A wave owns T x T MFMA tiles; the four waves of a workgroup stand SP x SP over the output (SP = 1 or 2) or, where
// SP = 1, divide K among them and add up through LDS.  Operands go straight to registers, the next 16 * KB elements of K
// on their way while the present ones are multiplied.
//
// Every tile adds up in the same order, so that a row's result does not depend on the rows beside it (a float32 model's
// tokens have the same KV whatever step they are computed in, although M picks the tile): K in four quarters of whole
// blocks of 32, a sum for each, and the four added in turn.  Waves that divide K hold one sum each; the waves of the
// 128 x 128 tile form them one after another.
//
// What bounds it: for the products of a small model's chunk the number of waves and the latency of a walk along K,
// so the tile shrinks until the grid fills the chip and K is divided (256 rows of the tiny model, us a launch:
// 256 -> 768 18 -> 7, 256 -> 688 twice with SwiGLU 35 -> 9.5, 688 -> 256 48 -> 5); for large products the float32
// matrix rate, fed from L2 through tiles of 64 x 64 per wave (1024 x 4096 x 4096: 492 -> 323 us, 106 TFLOP/s, both
// against the 64 x 64 tiles on the vector ALUs of the generic kernel).
//
// NORM: `a` is the residual stream in front of an RMSNorm.  A row's norm is a factor of all its products, so the tile
// multiplies x by the gain as it reads it, adds up the squares beside the products (the same quarters of K, added in the
// same order in every tile) and scales its results by the row's factor at the end: no normed copy of the activations, and no
// launch of 3 us before the product (256 rows of the tiny model, two layers: 131 -> 126 us).  Every tile does this again for its
// rows, so it is for products that take less than such a launch more by it (gemm_f32_norms_input), on tiles whose waves divide K.
#include "kernels.hpp"

namespace cake {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Does the tile keep its finished sums in LDS?  128 x 128 with SwiGLU: two times 64 x 64 sums and the operands fill a
// wave's registers (1024 x 4096 x 4096: spilled 1742 us, in LDS 600).
constexpr bool f32_lds_total(int t, int sp, int epi) { return sp == 2 && epi == EPI_SWIGLU && t == 4; }

template <int T, int SP, int EPI, bool NORM>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(const float* __restrict__ a, const float* __restrict__ w, const float* __restrict__ w2, float* __restrict__ out,
                int M, int N, int K, int tiles_m, const float* __restrict__ gain, float eps) {
    constexpr int KW = SP == 1 ? 4 : 1;              // waves that divide K
    constexpr int NM = EPI == EPI_SWIGLU ? 2 : 1;    // weight matrices
    constexpr int KB = NM * T > 4 ? 1 : 2;           // 16-deep blocks per trip (one where 64 x 64 twice fill the registers)
    constexpr int BT = 16 * T * SP;                  // rows and columns of the workgroup's tile
    constexpr bool LDS_TOTAL = f32_lds_total(T, SP, EPI);
    static_assert(!NORM || KW > 1, "a row's squares are added up through LDS");
    __shared__ float4 parts[KW > 1 ? (KW - 1) * NM * T * T * 64 : 1];
    __shared__ float squares[NORM ? 64 * T : 1];   // of a row in a quarter of K
    extern __shared__ __attribute__((aligned(16))) float4 total_lds[];   // LDS_TOTAL: [NM][T][T][256]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const int kw = SP == 1 ? wave : 0, wm = SP == 1 ? 0 : wave >> 1, wn = SP == 1 ? 0 : wave & 1;
    const int m0 = (blockIdx.x % tiles_m) * BT + wm * 16 * T, n0 = (blockIdx.x / tiles_m) * BT + wn * 16 * T;

    const float *ap[T], *wp[NM][T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        ap[i] = a + size_t(min(m0 + 16 * i + l16, M - 1)) * K + 4 * lq;
        wp[0][i] = w + size_t(min(n0 + 16 * i + l16, N - 1)) * K + 4 * lq;
        if constexpr (NM == 2) wp[1][i] = w2 + size_t(min(n0 + 16 * i + l16, N - 1)) * K + 4 * lq;
    }
    auto ld = [&](const float* p, int k) { return k + 4 * lq < K ? *(const float4*)(p + k) : make_float4(0.f, 0.f, 0.f, 0.f); };
    auto load = [&](float4 (&av)[T][KB], float4 (&wv)[NM][T][KB], float4 (&gv)[KB], int k0) {
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            if constexpr (NORM) gv[b] = ld(gain + 4 * lq, k0 + 16 * b);
#pragma unroll
            for (int i = 0; i < T; ++i) av[i][b] = ld(ap[i], k0 + 16 * b);
#pragma unroll
            for (int n = 0; n < NM; ++n)
#pragma unroll
                for (int j = 0; j < T; ++j) wv[n][j][b] = ld(wp[n][j], k0 + 16 * b);
        }
    };
    f32x4 acc[NM][T][T];
#pragma unroll
    for (int n = 0; n < NM; ++n)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) acc[n][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float sq[T];   // NORM: squares of this lane's elements of row l16 of row tile i, of a quarter of K
#pragma unroll
    for (int i = 0; i < T; ++i) sq[i] = 0.f;
    auto mul = [&](float4 (&av)[T][KB], const float4 (&wv)[NM][T][KB], const float4 (&gv)[KB]) {
        if constexpr (NORM) {
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    float4& x = av[i][b];
                    sq[i] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
                    x.x *= gv[b].x; x.y *= gv[b].y; x.z *= gv[b].z; x.w *= gv[b].w;
                }
        }
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int n = 0; n < NM; ++n)
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            acc[n][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(((const float*)&av[i][b])[e], ((const float*)&wv[n][j][b])[e],
                                                                                acc[n][i][j], 0, 0, 0);
    };
    float4 av[2][T][KB], wv[2][NM][T][KB], gv[2][KB];
    f32x4 total[NM][T][T];   // KW = 1: the finished sums (in LDS where the registers do not hold them as well)
    const int quarter = (K + 127) / 128 * 32;
    auto sum_of = [&](int p) {   // quarter p of K into acc
        constexpr int STEP = 16 * KB;
        const int k_end = min((p + 1) * quarter, K);
        int k = p * quarter;
        if (k < k_end) load(av[0], wv[0], gv[0], k);
        for (; k < k_end; k += 2 * STEP) {   // two trips unrolled, so that the two register sets alternate without copies
            if (k + STEP < k_end) load(av[1], wv[1], gv[1], k + STEP);
            mul(av[0], wv[0], gv[0]);
            if (k + STEP >= k_end) break;
            if (k + 2 * STEP < k_end) load(av[0], wv[0], gv[0], k + 2 * STEP);
            mul(av[1], wv[1], gv[1]);
        }
        if constexpr (NORM) {   // the four lanes of a row
#pragma unroll
            for (int i = 0; i < T; ++i) {
                sq[i] += __shfl_xor(sq[i], 16, 64);
                sq[i] += __shfl_xor(sq[i], 32, 64);
            }
        }
    };
    if constexpr (KW > 1) {
        sum_of(kw);
    } else {
#pragma unroll 1
        for (int p = 0; p < 4; ++p) {
            sum_of(p);
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) {
                        f32x4& a = acc[m][i][j];
                        if constexpr (LDS_TOTAL) {
                            float4& t = total_lds[((m * T + i) * T + j) * 256 + threadIdx.x];
                            if (p > 0) a += f32x4{t.x, t.y, t.z, t.w};
                            if (p < 3) t = make_float4(a[0], a[1], a[2], a[3]);
                        } else {
                            if (p > 0) a += total[m][i][j];
                            if (p < 3) total[m][i][j] = a;
                        }
                        if (p < 3) a = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
        }
    }
    if constexpr (KW > 1) {   // waves 1 .. 3 hand their sums to wave 0, which adds them in that order
        if (wave > 0) {
#pragma unroll
            for (int n = 0; n < NM; ++n)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) {
                        const f32x4 v = acc[n][i][j];
                        parts[(((wave - 1) * NM + n) * T * T + i * T + j) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
                    }
        }
        if constexpr (NORM) {
            if (lq == 0) {
#pragma unroll
                for (int i = 0; i < T; ++i) squares[wave * 16 * T + 16 * i + l16] = sq[i];
            }
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int p = 0; p < KW - 1; ++p)
#pragma unroll
            for (int n = 0; n < NM; ++n)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) {
                        const float4 v = parts[((p * NM + n) * T * T + i * T + j) * 64 + lane];
                        acc[n][i][j][0] += v.x; acc[n][i][j][1] += v.y; acc[n][i][j][2] += v.z; acc[n][i][j][3] += v.w;
                    }
    }
    float factor[T];   // NORM: of row l16 of row tile i
    if constexpr (NORM) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int t = 16 * i + l16;
            const float s = squares[t] + squares[16 * T + t] + squares[32 * T + t] + squares[48 * T + t];
            factor[i] = 1.0f / sqrtf(s / float(K) + eps);
        }
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = m0 + 16 * i + 4 * lq + v;
            const float r = NORM ? __shfl(factor[i], 4 * lq + v, 64) : 1.f;
            if (row >= M) continue;
#pragma unroll
            for (int j = 0; j < T; ++j) {
                const int col = n0 + 16 * j + l16;
                if (col >= N) continue;
                float* o = out + size_t(row) * N + col;
                const float x = NORM ? acc[0][i][j][v] * r : acc[0][i][j][v];
                if constexpr (EPI == EPI_STORE_F32) *o = x;
                else if constexpr (EPI == EPI_RESIDUAL_F32) *o += x;
                else *o = x / (1.0f + expf(-x)) * (NORM ? acc[1][i][j][v] * r : acc[1][i][j][v]);
            }
        }
}

template <int T, int SP, int EPI, bool NORM>
static hipError_t launch_t(const float* a, const float* w, const float* w2, float* out, int M, int N, int K, const GemvNorm& nm,
                           hipStream_t st) {
    constexpr int BT = 16 * T * SP;
    const int tiles_m = (M + BT - 1) / BT, tiles_n = (N + BT - 1) / BT;
    constexpr int LDS = f32_lds_total(T, SP, EPI) ? 2 * T * T * 256 * int(sizeof(float4)) : 0;
    if (LDS > 0) {
        static bool attr_set = false;   // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)gemm_f32_kernel<T, SP, EPI, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((gemm_f32_kernel<T, SP, EPI, NORM>), dim3(tiles_m * tiles_n), dim3(256), LDS, st, a, w, w2, out, M, N, K, tiles_m,
                       nm.gain, nm.eps);
    return hipGetLastError();
}

static long f32_tiles(int t, int M, int N) { return long((M + t - 1) / t) * ((N + t - 1) / t); }

// The largest tile whose grid still gives most CUs a workgroup: 128 x 128 (64 x 64 per wave); 64 x 64, 32 x 32 or
// 16 x 16 with the waves dividing K.  (512 x 4096 x 1024: 58 us on 64 x 64 tiles, 78 on 32 x 32, 72 generic.)
// Where K is short, a tile's life is latency and 16 x 16 tiles in threes on a CU hide each other's (us, 16 and 32 square: 192
// tiles of 32, K 256 5.0 and 5.3, with norm and SwiGLU 7.8 and 9.0; K 688 7.6 and 8.0, 13.7 and 16.0; 256 tiles, K 256 6.0 and 5.4,
// K 688 9.2 and 8.1; 192 tiles, K 1536 18.7 and 16.0).
template <int EPI, bool NORM>
static hipError_t launch_epi(const float* a, const float* w, const float* w2, float* out, int M, int N, int K, const GemvNorm& nm,
                             hipStream_t st) {
    auto tiles = [&](int t) { return f32_tiles(t, M, N); };
    if (tiles(128) >= 192) {
        if constexpr (NORM) return hipErrorInvalidValue;
        else return launch_t<4, 2, EPI, NORM>(a, w, w2, out, M, N, K, nm, st);
    }
    if (tiles(64) >= 160) return launch_t<4, 1, EPI, NORM>(a, w, w2, out, M, N, K, nm, st);
    if (tiles(32) >= (K <= 1024 ? 224 : 160)) return launch_t<2, 1, EPI, NORM>(a, w, w2, out, M, N, K, nm, st);
    return launch_t<1, 1, EPI, NORM>(a, w, w2, out, M, N, K, nm, st);
}

// Whether the products of a context whose chunks have up to max_rows rows norm their input themselves: by the context and not
// by the chunk, so that a token's bits do not depend on its step.  The norm's launch takes 6.5 to 8 us of a chunk; in
// front of a plain product the squares and gains cost 10 % of it, more than that from about 3.5 GFLOP on, in front of SwiGLU next to
// nothing on tiles of 64 and 4 to 6 % on tiles of 128.  us, norm apart and inside: QKV 500 rows of 1024 -> 1536 40 and 35, 256
// of 2048 -> 3072 60 and 58, 64 of 4096 -> 6144 82 and 81, 500 of 1536 -> 2304 (3.5 GFLOP) 86 and 86, 500 of 2048 -> 3072
// 106 and 109, 137 of 4096 -> 6144 182 and 193, 1024 of 4096 -> 6144 637 and 680; gate/up 64 rows of 1024 -> 2 x 2816 28 and
// 25, 1024 of them 186 and 178, 256 of 4096 -> 2 x 11008 553 and 547, on 128: 1024 of 1536 -> 2 x 4096 249 and 256, 1024
// of 4096 -> 2 x 11008 1781 and 1845.
bool gemm_f32_norms_input(int epi, int max_rows, int N, int K) {
    return f32_tiles(128, max_rows, N) < 192 && (epi == EPI_SWIGLU || 2.0 * max_rows * N * K < 3.5e9);
}

hipError_t launch_gemm_f32(int epi, const float* a, const float* w, const float* w2, float* out, int M, int N, int K, hipStream_t st,
                           const GemvNorm& nm) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K <= 0 || (K & 3) || (nm.gain && epi == EPI_RESIDUAL_F32)) return hipErrorInvalidValue;
    if (epi == EPI_STORE_F32)
        return nm.gain ? launch_epi<EPI_STORE_F32, true>(a, w, w2, out, M, N, K, nm, st) : launch_epi<EPI_STORE_F32, false>(a, w, w2, out, M, N, K, nm, st);
    if (epi == EPI_RESIDUAL_F32) return launch_epi<EPI_RESIDUAL_F32, false>(a, w, w2, out, M, N, K, nm, st);
    if (epi == EPI_SWIGLU)
        return nm.gain ? launch_epi<EPI_SWIGLU, true>(a, w, w2, out, M, N, K, nm, st) : launch_epi<EPI_SWIGLU, false>(a, w, w2, out, M, N, K, nm, st);
    return hipErrorInvalidValue;
}

}  // namespace cake
