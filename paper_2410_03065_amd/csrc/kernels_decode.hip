// Kernels of the first-token step: one token (the prompt's last) goes through the decoder against
// the complete KV cache, then final norm, LM head and argmax.  With one row of activations every
// projection is a matrix-vector product that streams its weights once, and attention streams the
// layer's K and V once: the whole step is bound by HBM bandwidth, so these kernels are built
// around wide coalesced loads and plain fp32 vector arithmetic (no MFMA: there is no reuse).
//
// The paper counts the time to first token up to "the generation of the first token" (Sec. 5.1,
// Metrics); the prefill it describes (Sec. 3) ends with that token's logits.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace cake {

namespace {

__device__ __forceinline__ float wsum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wmax(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Sum over aligned groups of W lanes (W = 8, 16 or 32), result in every lane of the group.  The
// steps inside a row of 16 lanes are DPP moves fused into the add (no LDS traffic): swap
// neighbours, swap pairs, mirror the half row, mirror the row.
template <int W>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(W == 8 || W == 16 || W == 32, "group width");
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));  // row_half_mirror
    if (W >= 16) v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));  // row_mirror
    if (W >= 32) v += __shfl_xor(v, 16, 64);
    return v;
}

// Four floats from a caller's array that is aligned to its elements only, as norm gains may be (one 16-byte load all the
// same: the hardware asks for 4-byte alignment).
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));

// 16 bytes of T -> floats
template <typename T> struct Ld16;
template <> struct Ld16<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ uint4 raw(const float* p) { return *(const uint4*)p; }
    static __device__ __forceinline__ void unpack(const uint4& v, float* o) {
        o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ void load(const float* p, float* o) { unpack(raw(p), o); }
};
template <> struct Ld16<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ uint4 raw(const bf16_t* p) { return *(const uint4*)p; }
    static __device__ __forceinline__ void unpack(const uint4& v, float* o) {
        const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = __uint_as_float(w[i] << 16);
            o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ void load(const bf16_t* p, float* o) { unpack(raw(p), o); }
};

}  // namespace

// ------------------------------------------------------------------ matrix-vector product
// out[n] (op)= sum_k h[k] * w[n][k], where h is x itself or its RMSNorm (NORM: h = x / sqrt(mean(x^2) + eps) * gain).
// MODE 0: store; 1: add into out (residual stream); 2: silu(h.w[n]) * (h.w2[n]); 3: store with the rotary embedding of
// the token applied, rows 2i and 2i+1 of a head being a pair.
//
// One wave takes RB consecutive rows, 16-byte loads, 1 KB of a row per wave-instruction.  The weights are read once
// from HBM and bound the kernel: U pieces of every row are loaded before the first is used.  The norm needs no pass of
// its own: the squares are summed beside the products, the sums scaled at the end; and a wave holds both rows of a
// rotary pair.  Where x is normed and long enough to be worth a barrier, the workgroup stages x times the gain in LDS
// behind the first weight loads (STAGED: 2048 to 16K elements), otherwise every wave reads both from the caches.
// The logits may go to pinned memory as well, from the waves that form them, while the others still stream: a copy by the
// arg max afterwards took 9 us more for 128 256 values and 3 for 32 000.
// One row per wave (two for a rotary pair; four where there are 16K rows and more).  us for the Llama3-8B shape: W_q
// with norm and rotation 9.8 (norm 4.3, product 7.7 and rotation 4.5 as three launches), gate/up with norm 42 (4.3 and
// 41), LM head 171 (4.3 and 182); two rows per wave took 23.1 instead of 22.7 for the down product, and a second set of
// loads in flight 26.
template <typename T, int MODE, int RB, bool NORM, bool STAGED>
__global__ void __launch_bounds__(256) gemv_kernel(const float* __restrict__ x, const float* __restrict__ gain, float eps,
                                                   const T* __restrict__ w, const T* __restrict__ w2, float* __restrict__ out, int N,
                                                   int K, const double2* __restrict__ cs, int head_dim, float* __restrict__ host) {
    constexpr int E = Ld16<T>::N, NM = MODE == 2 ? 2 : 1;
    constexpr int U = RB * NM >= 4 ? 2 : 4, PIECE = 64 * E;   // pieces in flight per row
    extern __shared__ __attribute__((aligned(16))) float xs[];
    __shared__ float ss_part[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = (blockIdx.x * 4 + wave) * RB;
    const T* wr[NM][RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        wr[0][r] = w + size_t(min(row0 + r, N - 1)) * K;
        if constexpr (NM == 2) wr[1][r] = w2 + size_t(min(row0 + r, N - 1)) * K;
    }
    struct Set { uint4 raw[U][NM][RB]; };
    // whole sets in one go, the last one piece by piece (wave-uniform choices)
    auto load_piece = [&](Set& st, int u, int k) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int r = 0; r < RB; ++r) st.raw[u][m][r] = Ld16<T>::raw(wr[m][r] + k);
    };
    auto load = [&](Set& st, int k0) {
        if (k0 + U * PIECE <= K) {
#pragma unroll
            for (int u = 0; u < U; ++u) load_piece(st, u, k0 + u * PIECE + lane * E);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * PIECE + lane * E;
                if (k0 + (u + 1) * PIECE <= K) load_piece(st, u, k);   // without a test per lane
                else if (k < K) load_piece(st, u, k);
            }
        }
    };
    float acc[NM][RB] = {}, ss = 0.f;
    auto multiply_piece = [&](const Set& st, int u, int k) {
        float xf[E];
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            const float4 xv = STAGED ? *(const float4*)(xs + k + e) : *(const float4*)(x + k + e);
            xf[e] = xv.x; xf[e + 1] = xv.y; xf[e + 2] = xv.z; xf[e + 3] = xv.w;
            if constexpr (NORM && !STAGED) {
                const float4_any gv = *(const float4_any*)(gain + k + e);
#pragma unroll
                for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(xf[e + i], xf[e + i], ss);
                xf[e] *= gv.x; xf[e + 1] *= gv.y; xf[e + 2] *= gv.z; xf[e + 3] *= gv.w;
            }
        }
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                float wf[E];
                Ld16<T>::unpack(st.raw[u][m][r], wf);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[m][r] = __builtin_fmaf(wf[e], xf[e], acc[m][r]);
            }
    };
    auto multiply = [&](const Set& st, int k0) {
        if (k0 + U * PIECE <= K) {
#pragma unroll
            for (int u = 0; u < U; ++u) multiply_piece(st, u, k0 + u * PIECE + lane * E);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * PIECE + lane * E;
                if (k0 + (u + 1) * PIECE <= K) multiply_piece(st, u, k);
                else if (k < K) multiply_piece(st, u, k);
            }
        }
    };
    Set set;
    load(set, 0);
    if constexpr (STAGED) {
        for (int k = threadIdx.x * 4; k < K; k += 1024) {
            float4 v = *(const float4*)(x + k);
            if constexpr (NORM) {
                const float4_any g = *(const float4_any*)(gain + k);
                ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                v.x *= g.x; v.y *= g.y; v.z *= g.z; v.w *= g.w;
            }
            *(float4*)(xs + k) = v;
        }
        if constexpr (NORM) {
            ss = wsum(ss);
            if (lane == 0) ss_part[wave] = ss;
        }
        __syncthreads();
        if constexpr (NORM) ss = ss_part[0] + ss_part[1] + ss_part[2] + ss_part[3];
    }
    if (row0 >= N) return;
    for (int k0 = 0; k0 < K; k0 += U * PIECE) {
        multiply(set, k0);
        load(set, k0 + U * PIECE);
    }
    float norm = 1.0f;
    if constexpr (NORM) norm = 1.0f / sqrtf((STAGED ? ss : wsum(ss)) / float(K) + eps);
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[m][r] = wsum(acc[m][r]) * norm;
    if (lane != 0) return;
    if constexpr (MODE == 0 && RB == 4)
        if (host && row0 + RB <= N) *(float4*)(host + row0) = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int row = row0 + r;
        if (row >= N) break;
        if constexpr (MODE == 0) {
            out[row] = acc[0][r];
            if (host && (RB != 4 || row0 + RB > N)) host[row] = acc[0][r];
        } else if constexpr (MODE == 1) out[row] += acc[0][r];
        else if constexpr (MODE == 2) out[row] = acc[0][r] / (1.0f + __expf(-acc[0][r])) * acc[1][r];
        else if ((r & 1) == 0) {   // N and the head dimension are even
            const double2 c = cs[(row % head_dim) / 2];
            out[row] = float(acc[0][r] * c.x - acc[0][r + 1] * c.y);
            out[row + 1] = float(acc[0][r] * c.y + acc[0][r + 1] * c.x);
        }
    }
}

template <typename T, int MODE, bool NORM>
static hipError_t gemv_launch(const GemvNorm& nm, const float* x, const void* w, const void* w2, float* out, int N, int K,
                              const double* cs, int head_dim, float* host, hipStream_t st) {
    constexpr int RB_MIN = MODE == 3 ? 2 : 1;
#define CAKE_GEMV(RB, STAGED, LDS)                                                                                        \
    hipLaunchKernelGGL((gemv_kernel<T, MODE, RB, NORM, STAGED>), dim3((N + 4 * RB - 1) / (4 * RB)), dim3(256), LDS, st, x, \
                       nm.gain, nm.eps, (const T*)w, (const T*)w2, out, N, K, (const double2*)cs, head_dim, host)
    const size_t lds = size_t(K) * sizeof(float);
    if constexpr (NORM) {
        if (K >= 2048 && lds <= 65000) {
            if (N >= 16384 && MODE == 0) CAKE_GEMV(4, true, lds);
            else CAKE_GEMV(RB_MIN, true, lds);
            return hipGetLastError();
        }
    }
    if (N >= 16384 && MODE == 0) CAKE_GEMV(4, false, 0);
    else CAKE_GEMV(RB_MIN, false, 0);
#undef CAKE_GEMV
    return hipGetLastError();
}

hipError_t launch_gemv(int dtype, int mode, const GemvNorm& nm, const float* x, const void* w, const void* w2, float* out, int N,
                       int K, hipStream_t st, const double* cs, int head_dim, float* host) {
    if (N <= 0) return hipSuccess;
    if (K % (dtype == 0 ? 4 : 8) || mode < 0 || mode > 3 || (mode == 3 && (!cs || !nm.gain)) || (mode == 1 && nm.gain) || (host && (mode != 0 || (uintptr_t(host) & 15)))) return hipErrorInvalidValue;
#define CAKE_GEMV(MODE, NORM)                                                                              \
    return dtype == 0 ? gemv_launch<float, MODE, NORM>(nm, x, w, w2, out, N, K, cs, head_dim, host, st)          \
                      : gemv_launch<bf16_t, MODE, NORM>(nm, x, w, w2, out, N, K, cs, head_dim, host, st)
    if (mode == 1) CAKE_GEMV(1, false);
    if (mode == 3) CAKE_GEMV(3, true);
    if (!nm.gain) return hipErrorInvalidValue;   // the step's other products all follow a norm
    if (mode == 2) CAKE_GEMV(2, true);
    CAKE_GEMV(0, true);
#undef CAKE_GEMV
}

// ------------------------------------------------------------------ what every layer of the step starts from
// x = the token's embedding row (grid.x - 1 workgroups of 1024 elements), and the rotary pairs' (cos, sin) of its
// position in double precision like the prefill's table (the last workgroup).
template <typename T>
__global__ void __launch_bounds__(256) token_begin_kernel(const T* __restrict__ table, int id, float* __restrict__ x, int d,
                                                          double2* __restrict__ cs, int half, int pos, double log2_theta) {
    if (blockIdx.x == gridDim.x - 1) {
        for (int pair = threadIdx.x; pair < half; pair += 256) {
            const double inv_freq = exp2(-(double(pair) / double(half)) * log2_theta);
            double s, c;
            sincos(double(pos) * inv_freq, &s, &c);
            cs[pair] = make_double2(c, s);
        }
        return;
    }
    const T* src = table + size_t(id) * d;
    const int lo = blockIdx.x * 1024;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = lo + threadIdx.x + 256 * i;
        if (c < d) x[c] = float(src[c]);
    }
}

hipError_t launch_token_begin(int dtype, const void* table, int id, float* x, int d, double* cs, int head_dim, int pos, float theta,
                              hipStream_t st) {
    const dim3 grid((d + 1023) / 1024 + 1), block(256);
    const double l2 = log2(double(theta));
    if (dtype == 0) hipLaunchKernelGGL(token_begin_kernel<float>, grid, block, 0, st, (const float*)table, id, x, d, (double2*)cs, head_dim / 2, pos, l2);
    else hipLaunchKernelGGL(token_begin_kernel<bf16_t>, grid, block, 0, st, (const bf16_t*)table, id, x, d, (double2*)cs, head_dim / 2, pos, l2);
    return hipGetLastError();
}

// ------------------------------------------------------------------ one-token attention, keys split
// Grid (KV head g, split s).  The workgroup's four waves take the split's 64-key tiles in turn.
// Per tile: scores of the R query heads of the group against 64 keys (K rows are contiguous:
// KL lanes x 16 B per row, partial dots reduced across those lanes), online softmax with lane =
// key, then P.V with V^T rows (64 keys = VL lanes x 16 B, reduced across those lanes).  The waves'
// and then the splits' partial (max, sum, O) are merged by the usual rescaling.
constexpr int DEC_MAX_SPLITS = 128;

template <typename T, int HD, int R>
__global__ void __launch_bounds__(256, 2)
decode_attention_kernel(const float* __restrict__ q, float* __restrict__ part, int n_keys, int tiles_per_split,
                        KvView kv) {
    constexpr int E = Ld16<T>::N;
    constexpr int KL = HD / E, KPI = 64 / KL, NQI = 64 / KPI;   // lanes per K row, keys per instruction, instructions
    constexpr int VL = 64 / E, RPI = 64 / VL, NVI = HD / RPI;   // lanes per V^T row piece, rows per instruction
    __shared__ float sc[4][R][64];
    __shared__ float wo[4][R][HD];
    __shared__ float wm[4][R], wl[4][R];
    const int g = blockIdx.x, split = blockIdx.y, n_splits = gridDim.y;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n_tiles = (n_keys + 63) / 64;
    const int tile_lo = split * tiles_per_split, tile_hi = min(tile_lo + tiles_per_split, n_tiles);
    const float scale = rsqrtf(float(HD));
    const int pt = kv.page_tokens;
    const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;

    const int ksub = lane % KL, kq = lane / KL;
    const int vsub = lane % VL, vq = lane / VL;
    float o_acc[R][NVI];
    float m_run[R], l_run[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        m_run[j] = -1.0e30f;   // finite: a tile with every key masked then leaves exp(-inf - m) = 0, not NaN
        l_run[j] = 0.f;
#pragma unroll
        for (int i = 0; i < NVI; ++i) o_acc[j][i] = 0.f;
    }

    // uniform trip count for the four waves (barriers inside); a wave without a tile skips the work
    for (int base = tile_lo; base < tile_hi; base += 4) {
        const int tile = base + wave;
        const bool have = tile < tile_hi;
        const int key0 = tile * 64;
        const T* page = nullptr;
        int in_page0 = 0;
        if (have) {
            const int lpage = key0 / pt;
            in_page0 = key0 - lpage * pt;
            page = (const T*)kv.pool + (layer_base + kv.block_table[lpage]) * kv.page_elems();
        }
        // every K load of the tile is issued before the first is used (16 KB in flight together, not
        // one 1 KB round trip after another); the V^T loads go out as soon as the scores are formed,
        // so they fly during the softmax.  Registers are kept under 256 so two waves share a SIMD.
        uint4 kraw[NQI], vraw[NVI];
        if (have) {
            const T* kp = page + (size_t(g) * pt + in_page0) * HD;
            const T* vp = page + size_t(kv.n_kv) * pt * HD + size_t(g) * HD * pt + in_page0;
#pragma unroll
            for (int it = 0; it < NQI; ++it) kraw[it] = Ld16<T>::raw(kp + size_t(it * KPI + kq) * HD + ksub * E);
            float qreg[R][E];   // this lane's slice of the group's queries (L1-resident after the first tile)
#pragma unroll
            for (int j = 0; j < R; ++j)
#pragma unroll
                for (int e = 0; e < E; ++e) qreg[j][e] = q[size_t(g * R + j) * HD + ksub * E + e] * scale;
#pragma unroll
            for (int it = 0; it < NQI; ++it) {
                const int kt = it * KPI + kq;
                float kf[E];
                Ld16<T>::unpack(kraw[it], kf);
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    float d = 0.f;
#pragma unroll
                    for (int e = 0; e < E; ++e) d = __builtin_fmaf(kf[e], qreg[j][e], d);
                    d = group_sum<KL>(d);
                    if (ksub == 0) sc[wave][j][kt] = d;
                }
            }
#pragma unroll
            for (int it = 0; it < NVI; ++it) vraw[it] = Ld16<T>::raw(vp + size_t(it * RPI + vq) * pt + vsub * E);
        }
        __syncthreads();
        float corr[R], pl[R][E];
        if (have) {
            const bool valid = key0 + lane < n_keys;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const float s = valid ? sc[wave][j][lane] : -INFINITY;
                const float m_new = fmaxf(m_run[j], wmax(s));
                const float p = __expf(s - m_new);
                corr[j] = __expf(m_run[j] - m_new);
                l_run[j] = l_run[j] * corr[j] + wsum(p);
                m_run[j] = m_new;
                sc[wave][j][lane] = p;
            }
        }
        __syncthreads();
        if (have) {
#pragma unroll
            for (int j = 0; j < R; ++j)
#pragma unroll
                for (int e = 0; e < E; ++e) pl[j][e] = sc[wave][j][vsub * E + e];
#pragma unroll
            for (int it = 0; it < NVI; ++it) {
                float vf[E];
                Ld16<T>::unpack(vraw[it], vf);
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    float d = 0.f;
#pragma unroll
                    for (int e = 0; e < E; ++e) d = __builtin_fmaf(vf[e], pl[j][e], d);
                    d = group_sum<VL>(d);
                    o_acc[j][it] = o_acc[j][it] * corr[j] + d;
                }
            }
        }
        __syncthreads();   // sc is rewritten by the next tile
    }

    // merge the four waves, then hand the split's partial result to the combine kernel
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (lane == 0) { wm[wave][j] = m_run[j]; wl[wave][j] = l_run[j]; }
        if (vsub == 0)
#pragma unroll
            for (int it = 0; it < NVI; ++it) wo[wave][j][it * RPI + vq] = o_acc[j][it];
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < R * HD; idx += 256) {
        const int j = idx / HD, d = idx % HD;
        float m = wm[0][j];
#pragma unroll
        for (int w = 1; w < 4; ++w) m = fmaxf(m, wm[w][j]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float c = __expf(wm[w][j] - m);
            num += wo[w][j][d] * c;
            den += wl[w][j] * c;
        }
        float* dst = part + (size_t(g * R + j) * n_splits + split) * (HD + 2);
        dst[d] = num;
        if (d == 0) { dst[HD] = m; dst[HD + 1] = den; }
    }
}

// One workgroup per query head; thread (part, d), part < 4, adds up output element d over the splits part, part + 4, ...
// The per-split (max, sum) pairs are read by one lane each and reduced across the first wave, so no thread walks the
// splits one dependent load after another; a thread's first eight values are on their way meanwhile.  All latency: with one
// thread per output element 4.8 us at 32 splits of 32 heads, 4.0 so.
template <int HD>
__global__ void __launch_bounds__(4 * HD) decode_combine_kernel(const float* __restrict__ part, float* __restrict__ out,
                                                                int n_splits) {
    __shared__ float coef[DEC_MAX_SPLITS];
    __shared__ float den_s, sums[4][HD];
    const int h = blockIdx.x, d = threadIdx.x % HD, quarter = threadIdx.x / HD;
    const float* p = part + size_t(h) * n_splits * (HD + 2);
    float first[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) first[i] = quarter + 4 * i < n_splits ? p[(quarter + 4 * i) * (HD + 2) + d] : 0.f;
    if (threadIdx.x < 64) {   // first wave: splits x and x + 64
        const int x = threadIdx.x;
        const float m0 = x < n_splits ? p[x * (HD + 2) + HD] : -INFINITY;
        const float m1 = x + 64 < n_splits ? p[(x + 64) * (HD + 2) + HD] : -INFINITY;
        const float l0 = x < n_splits ? p[x * (HD + 2) + HD + 1] : 0.f, l1 = x + 64 < n_splits ? p[(x + 64) * (HD + 2) + HD + 1] : 0.f;
        const float m = wmax(fmaxf(m0, m1));
        const float c0 = x < n_splits ? __expf(m0 - m) : 0.f, c1 = x + 64 < n_splits ? __expf(m1 - m) : 0.f;
        const float den = wsum(l0 * c0 + l1 * c1);
        coef[x] = c0;
        coef[x + 64] = c1;
        if (x == 0) den_s = den;
    }
    __syncthreads();
    float num = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (quarter + 4 * i < n_splits) num += first[i] * coef[quarter + 4 * i];
#pragma unroll 8
    for (int s = quarter + 32; s < n_splits; s += 4) num += p[s * (HD + 2) + d] * coef[s];
    sums[quarter][d] = num;
    __syncthreads();
    if (quarter == 0) out[size_t(h) * HD + d] = (sums[0][d] + sums[1][d] + sums[2][d] + sums[3][d]) / den_s;
}

int decode_attention_splits(int n_keys, int n_kv) {
    const int n_tiles = (n_keys + 63) / 64;
    int want = std::max(1, 1024 / std::max(1, n_kv));            // about four workgroups per CU in total
    int splits = std::min({want, (n_tiles + 3) / 4, DEC_MAX_SPLITS});
    return std::max(1, splits);
}

size_t decode_attention_workspace_bytes(int n_q, int head_dim) {
    return size_t(n_q) * DEC_MAX_SPLITS * (head_dim + 2) * sizeof(float);
}

template <typename T, int HD>
static hipError_t decode_launch_r(int r, dim3 grid, hipStream_t st, const float* q, float* part, int n_keys, int tps,
                                  const KvView& kv) {
    switch (r) {
        case 1: hipLaunchKernelGGL((decode_attention_kernel<T, HD, 1>), grid, dim3(256), 0, st, q, part, n_keys, tps, kv); break;
        case 2: hipLaunchKernelGGL((decode_attention_kernel<T, HD, 2>), grid, dim3(256), 0, st, q, part, n_keys, tps, kv); break;
        case 4: hipLaunchKernelGGL((decode_attention_kernel<T, HD, 4>), grid, dim3(256), 0, st, q, part, n_keys, tps, kv); break;
        case 8: hipLaunchKernelGGL((decode_attention_kernel<T, HD, 8>), grid, dim3(256), 0, st, q, part, n_keys, tps, kv); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// q[n_q][hd] (float32, rotated) against keys [0, n_keys) of the layer; out[n_q][hd] float32.
// `part` must hold decode_attention_workspace_bytes().  bf16 pages with head_dim 128 go to the
// MFMA kernel (one workgroup per CU, each wave streaming its own tiles); everything else to the
// vector-ALU kernel above.
hipError_t launch_decode_attention(int dtype, const float* q, float* out, float* part, int n_q, int n_keys,
                                   const KvView& kv, hipStream_t st, bool generic_only) {
    if (n_keys <= 0 || n_q % kv.n_kv) return hipErrorInvalidValue;
    const int r = n_q / kv.n_kv;
    const int n_tiles = (n_keys + 63) / 64;
    const bool mfma = !generic_only && decode_attention_mfma_supported(dtype, kv.head_dim, kv.page_tokens, r);
    int splits = mfma ? std::max(1, std::min({256 / std::max(1, kv.n_kv), (n_tiles + 3) / 4, DEC_MAX_SPLITS}))
                      : decode_attention_splits(n_keys, kv.n_kv);
    const int tps = (n_tiles + splits - 1) / splits;
    const int used = (n_tiles + tps - 1) / tps;   // every launched split owns at least one tile
    dim3 grid(kv.n_kv, used);
    hipError_t e;
    if (mfma) e = launch_decode_attention_mfma(q, part, n_q, n_keys, tps, used, kv, st);
    else if (dtype == 0 && kv.head_dim == 64) e = decode_launch_r<float, 64>(r, grid, st, q, part, n_keys, tps, kv);
    else if (dtype == 0 && kv.head_dim == 128) e = decode_launch_r<float, 128>(r, grid, st, q, part, n_keys, tps, kv);
    else if (dtype == 1 && kv.head_dim == 64) e = decode_launch_r<bf16_t, 64>(r, grid, st, q, part, n_keys, tps, kv);
    else if (dtype == 1 && kv.head_dim == 128) e = decode_launch_r<bf16_t, 128>(r, grid, st, q, part, n_keys, tps, kv);
    else return hipErrorInvalidValue;
    if (e != hipSuccess) return e;
    if (kv.head_dim == 64) hipLaunchKernelGGL(decode_combine_kernel<64>, dim3(n_q), dim3(256), 0, st, part, out, used);
    else hipLaunchKernelGGL(decode_combine_kernel<128>, dim3(n_q), dim3(512), 0, st, part, out, used);
    return hipGetLastError();
}

// ------------------------------------------------------------------ argmax over the logits
// result[0] = index of the largest value (the lowest index among equal values).  Workgroups take 1024-element pieces in
// turn and leave their best in `best`; the one that draws the last ticket looks those through and puts the counter back.
// (One workgroup over 128 256 logits took 56 us, most of it waiting for one load after another.)
__device__ __forceinline__ void argmax_take(float x, int i, float* best, int* idx) {
    if (x > *best || (x == *best && i < *idx)) { *best = x; *idx = i; }
}
__device__ __forceinline__ void argmax_wave(float* best, int* idx) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ob = __shfl_xor(*best, o, 64);
        const int oi = __shfl_xor(*idx, o, 64);
        argmax_take(ob, oi, best, idx);
    }
}

__global__ void __launch_bounds__(256) argmax_kernel(const float* __restrict__ v, int n, unsigned long long* __restrict__ best_of,
                                                     unsigned* __restrict__ counter, int32_t* __restrict__ result) {
    __shared__ float bv[4];
    __shared__ int bi[4];
    __shared__ unsigned ticket;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float best = -INFINITY;
    int idx = 0x7fffffff;
    for (int base = blockIdx.x * 1024; base < n; base += gridDim.x * 1024)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = base + threadIdx.x + 256 * i;
            if (at < n) {
                const float x = v[at];
                argmax_take(x, at, &best, &idx);
            }
        }
    argmax_wave(&best, &idx);
    if (lane == 0) { bv[wave] = best; bi[wave] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) argmax_take(bv[w], bi[w], &best, &idx);
        __hip_atomic_store(&best_of[blockIdx.x], (unsigned long long)(unsigned)idx << 32 | __float_as_uint(best), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (ticket != gridDim.x - 1 || wave != 0) return;
    best = -INFINITY;
    idx = 0x7fffffff;
    for (int b = lane; b < int(gridDim.x); b += 64) {
        const unsigned long long p = __hip_atomic_load(&best_of[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        argmax_take(__uint_as_float(unsigned(p)), int(unsigned(p >> 32)), &best, &idx);
    }
    argmax_wave(&best, &idx);
    if (lane == 0) {
        result[0] = idx;
        __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

hipError_t launch_argmax(const float* v, int n, ArgmaxWs* ws, int32_t* result, hipStream_t st) {
    if (n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(argmax_kernel, dim3(std::min(ARGMAX_BLOCKS, (n + 1023) / 1024)), dim3(256), 0, st, v, n, ws->best, &ws->counter, result);
    return hipGetLastError();
}

}  // namespace cake
