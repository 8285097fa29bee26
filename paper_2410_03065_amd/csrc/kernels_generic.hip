// Generic device kernels: embedding gather, RMSNorm, rotary + KV page write, a plain
// LDS-tiled GEMM and a plain chunk-vs-prefix attention.  They accept float32 and bf16
// element types and any supported shape; float32 models run on them entirely, bf16
// models use them for the element-wise steps (the contractions go to the MFMA kernels).
//
// Operations follow the decoder block the benchmark shapes name (the paper, Sec. 3,
// states only Q = X W_Q, K = X W_K, V = X W_V and softmax(Q K^T / sqrt(d_k)) V):
// pre-RMSNorm, rotary embedding on adjacent pairs, grouped-query attention, SwiGLU.
#include "kernels.hpp"

namespace cake {

template <typename T> __device__ __forceinline__ float to_f(T v);
template <> __device__ __forceinline__ float to_f<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f<bf16_t>(bf16_t v) { return float(v); }
template <typename T> __device__ __forceinline__ T from_f(float v);
template <> __device__ __forceinline__ float from_f<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float v) { return bf16_t(v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// ------------------------------------------------------------------ RMSNorm
// y = x / sqrt(mean(x^2) + eps) * gain ; one 256-thread block per row.
template <typename T>
__global__ void __launch_bounds__(256) rmsnorm_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                                      T* __restrict__ out, int d, float eps) {
    __shared__ float part[4];
    const float* xr = x + size_t(blockIdx.x) * d;
    float s = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) { float v = xr[c]; s += v * v; }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    float tot = part[0] + part[1] + part[2] + part[3];
    float r = 1.0f / sqrtf(tot / float(d) + eps);
    T* o = out + size_t(blockIdx.x) * d;
    for (int c = threadIdx.x; c < d; c += 256) o[c] = from_f<T>(xr[c] * r * gain[c]);
}

// The norm of a row that the workgroup's threads hold in pieces, thread t the elements 4 t .. 4 t + 3 of every 1024.
template <typename T, int NV>
__device__ __forceinline__ void rmsnorm_row(const float4 (&v)[NV], float* part, const float* __restrict__ gain, T* __restrict__ o, float eps) {
    constexpr int d = NV * 1024;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    const float tot = part[0] + part[1] + part[2] + part[3];
    const float r = 1.0f / sqrtf(tot / float(d) + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c4 = threadIdx.x + 256 * i;
        const float4 g = ((const float4*)gain)[c4];
        const float y0 = v[i].x * r * g.x, y1 = v[i].y * r * g.y, y2 = v[i].z * r * g.z, y3 = v[i].w * r * g.w;
        if constexpr (sizeof(T) == 4) {
            ((float4*)o)[c4] = make_float4(y0, y1, y2, y3);
        } else {
            typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
            bf16x4_t w = {from_f<T>(y0), from_f<T>(y1), from_f<T>(y2), from_f<T>(y3)};
            ((bf16x4_t*)o)[c4] = w;
        }
    }
}

// Rows whose length is a multiple of 1024: every thread keeps its NV float4 pieces of the row in
// registers (one 16-byte load each, all in flight together), so the row is read once.  PARTS: the K ranges of the
// product in front of the norm, parts[n_parts][rows][d], are added to the residual stream on the way (in that order)
// and the sum is written back; bound by the ranges' way through memory (1024 x 4096 with four ranges 64 + 32 MB).
template <typename T, int NV, bool PARTS>
__global__ void __launch_bounds__(256) rmsnorm_vec_kernel(float* __restrict__ x, const float* __restrict__ parts, int n_parts,
                                                          const float* __restrict__ gain, T* __restrict__ out, float eps) {
    __shared__ float part[4];
    constexpr int d = NV * 1024;
    float4* xr = (float4*)(x + size_t(blockIdx.x) * d);
    float4 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = xr[threadIdx.x + 256 * i];
    if constexpr (PARTS) {
        const float4* pr = (const float4*)(parts + size_t(blockIdx.x) * d) + threadIdx.x;
        const size_t step = size_t(gridDim.x) * (d / 4);
#pragma unroll 4
        for (int p = 0; p < n_parts; ++p)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const float4 a = pr[p * step + 256 * i];
                v[i].x += a.x; v[i].y += a.y; v[i].z += a.z; v[i].w += a.w;
            }
#pragma unroll
        for (int i = 0; i < NV; ++i) xr[threadIdx.x + 256 * i] = v[i];
    }
    rmsnorm_row<T, NV>(v, part, gain, out + size_t(blockIdx.x) * d, eps);
}

template <typename T>
static bool launch_rmsnorm_vec(float* x, const float* parts, int n_parts, const float* gain, T* out, int rows, int d, float eps,
                               hipStream_t st) {
    if (d % 1024 != 0 || d > 8192 || ((uintptr_t(x) | uintptr_t(parts) | uintptr_t(gain) | uintptr_t(out)) & 15)) return false;
    switch (d / 1024) {
#define CAKE_RMS_CASE(NV)                                                                                                          \
    case NV:                                                                                                                       \
        if (n_parts) hipLaunchKernelGGL((rmsnorm_vec_kernel<T, NV, true>), dim3(rows), dim3(256), 0, st, x, parts, n_parts, gain, out, eps); \
        else hipLaunchKernelGGL((rmsnorm_vec_kernel<T, NV, false>), dim3(rows), dim3(256), 0, st, x, parts, 0, gain, out, eps);    \
        return true;
        CAKE_RMS_CASE(1) CAKE_RMS_CASE(2) CAKE_RMS_CASE(3) CAKE_RMS_CASE(4) CAKE_RMS_CASE(5) CAKE_RMS_CASE(6) CAKE_RMS_CASE(7)
        CAKE_RMS_CASE(8)
#undef CAKE_RMS_CASE
    }
    return false;
}

hipError_t launch_rmsnorm(int dtype, const float* x, const float* gain, void* out, int rows, int d, float eps,
                          hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    if (dtype == 0 ? launch_rmsnorm_vec((float*)x, nullptr, 0, gain, (float*)out, rows, d, eps, st)   // without parts x is only read
                   : launch_rmsnorm_vec((float*)x, nullptr, 0, gain, (bf16_t*)out, rows, d, eps, st))
        return hipGetLastError();
    if (dtype == 0) hipLaunchKernelGGL(rmsnorm_kernel<float>, dim3(rows), dim3(256), 0, st, x, gain, (float*)out, d, eps);
    else hipLaunchKernelGGL(rmsnorm_kernel<bf16_t>, dim3(rows), dim3(256), 0, st, x, gain, (bf16_t*)out, d, eps);
    return hipGetLastError();
}

// x[n] += parts[0][n] + parts[1][n] + ... in that order (store: x[n] = that sum); n a multiple of 4.
__global__ void __launch_bounds__(256) add_parts_kernel(float4* __restrict__ x, const float4* __restrict__ parts, int n_parts, size_t n4, bool store) {
    for (size_t i = blockIdx.x * size_t(256) + threadIdx.x; i < n4; i += gridDim.x * size_t(256)) {
        float4 v = store ? parts[i] : x[i];
#pragma unroll 4
        for (int p = store ? 1 : 0; p < n_parts; ++p) {
            const float4 a = parts[p * n4 + i];
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        x[i] = v;
    }
}

hipError_t launch_add_parts(float* x, const float* parts, int n_parts, size_t n, hipStream_t st, bool store) {
    if (n == 0 || n_parts <= 0) return hipSuccess;
    if (n % 4 || ((uintptr_t(x) | uintptr_t(parts)) & 15)) return hipErrorInvalidValue;
    const size_t blocks = (n / 4 + 255) / 256;
    hipLaunchKernelGGL(add_parts_kernel, dim3(unsigned(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st, (float4*)x, (const float4*)parts, n_parts, n / 4, store);
    return hipGetLastError();
}

hipError_t launch_rmsnorm_parts(int dtype, float* x, const float* parts, int n_parts, const float* gain, void* out, int rows, int d,
                                float eps, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    if (dtype == 0 ? launch_rmsnorm_vec(x, parts, n_parts, gain, (float*)out, rows, d, eps, st)
                   : launch_rmsnorm_vec(x, parts, n_parts, gain, (bf16_t*)out, rows, d, eps, st))
        return hipGetLastError();
    hipError_t e = launch_add_parts(x, parts, n_parts, size_t(rows) * d, st);
    return e != hipSuccess ? e : launch_rmsnorm(dtype, x, gain, out, rows, d, eps, st);
}

// ------------------------------------------------------------------ rotary table
// cs[row][pair] = (cos, sin) of (tok_begin + row) * theta^(-2*pair/head_dim).  The angle is
// formed in double precision: at position 65535 a float32 angle is off by ~4e-3 rad.
__device__ __forceinline__ void rope_table_entry(float2* __restrict__ cs, int idx, int tok_begin, int rows, int half, double log2_theta) {
    if (idx >= rows * half) return;
    int row = idx / half, pair = idx % half;
    double inv_freq = exp2(-(double(pair) / double(half)) * log2_theta);
    double ang = double(tok_begin + row) * inv_freq;
    double s, c;
    sincos(ang, &s, &c);
    cs[idx] = make_float2(float(c), float(s));
}

__global__ void __launch_bounds__(256) rope_table_kernel(float2* __restrict__ cs, int tok_begin, int rows, int half, double log2_theta) {
    rope_table_entry(cs, blockIdx.x * 256 + threadIdx.x, tok_begin, rows, half, log2_theta);
}

hipError_t launch_rope_table(float* cs, int tok_begin, int rows, int head_dim, float theta, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    int half = head_dim / 2, n = rows * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3((n + 255) / 256), dim3(256), 0, st, (float2*)cs, tok_begin, rows, half,
                       log2(double(theta)));
    return hipGetLastError();
}

// ------------------------------------------------------------------ what a prefill begins with
// One launch: the rows' embeddings (x), their first RMSNorm (h; NV 1024-element pieces of a row, NV = 0: no norm, NV = -1: no
// norm, bf16 rows read in pieces of 16 bytes; 137 rows of 3584 6.6 -> 4.0 us, 1024 rows 12.7 -> 11.2) and, by the workgroups
// after the rows', the rotary table.  They were three launches of 2 to 10 us at the start of a step, when the host is not
// ahead of the GPU yet.  Token ids: device memory, or (TokenIds) the launch's own arguments, which saves a short step the copy
// in front of it.  Two layers, us: 137 rows of the Llama3-8B shape 346 -> 335, 512 rows of the small model with heads of 64
// 313 -> 299, 256 rows of the tiny model 126 -> 119.
struct IdsInMemory {
    const int32_t* p;
    __device__ int32_t operator[](int row) const { return p[row]; }
};
struct IdsInArguments {
    TokenIds t;
    __device__ int32_t operator[](int row) const { return t.v[row]; }
};
template <typename T, int NV, typename Ids>
__global__ void __launch_bounds__(256)
prefill_begin_kernel(const T* __restrict__ table, const Ids ids, float* __restrict__ x, int d_any, int vocab, int rows,
                     const float* __restrict__ gain, T* __restrict__ out, float eps, float2* __restrict__ cs, int tok_begin, int half,
                     double log2_theta) {
    __shared__ float part[4];
    if (int(blockIdx.x) >= rows) {
        rope_table_entry(cs, (blockIdx.x - rows) * 256 + threadIdx.x, tok_begin, rows, half, log2_theta);
        return;
    }
    int id = ids[blockIdx.x];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
    if constexpr (NV == 0) {
        const T* src = table + size_t(id) * d_any;
        float* dst = x + size_t(blockIdx.x) * d_any;
        for (int c = threadIdx.x; c < d_any; c += 256) dst[c] = to_f<T>(src[c]);
    } else if constexpr (NV < 0) {
        const uint4* src = (const uint4*)(table + size_t(id) * d_any);
        float4* dst = (float4*)(x + size_t(blockIdx.x) * d_any);
        for (int c = threadIdx.x; c < d_any / 8; c += 256) {
            const uint4 v = src[c];
            dst[2 * c] = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                                     __uint_as_float(v.y & 0xFFFF0000u));
            dst[2 * c + 1] = make_float4(__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xFFFF0000u), __uint_as_float(v.w << 16),
                                         __uint_as_float(v.w & 0xFFFF0000u));
        }
    } else {
        constexpr int d = NV * 1024;
        typedef __attribute__((__vector_size__(4 * sizeof(T)))) T vec4_t;
        const vec4_t* src = (const vec4_t*)(table + size_t(id) * d);
        float4 v[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const vec4_t t = src[threadIdx.x + 256 * i];
            v[i] = make_float4(to_f<T>(t[0]), to_f<T>(t[1]), to_f<T>(t[2]), to_f<T>(t[3]));
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) ((float4*)(x + size_t(blockIdx.x) * d))[threadIdx.x + 256 * i] = v[i];
        rmsnorm_row<T, NV>(v, part, gain, out + size_t(blockIdx.x) * d, eps);
    }
}

template <typename T, int NV, typename Ids>
static void launch_begin(const PrefillBegin& b, const Ids& ids, hipStream_t st) {
    const int half = b.head_dim / 2;
    hipLaunchKernelGGL((prefill_begin_kernel<T, NV, Ids>), dim3(b.rows + (b.rows * half + 255) / 256), dim3(256), 0, st, (const T*)b.table, ids, b.x,
                       b.d, b.vocab, b.rows, b.gain, (T*)b.h, b.eps, (float2*)b.cs, b.tok_begin, half, log2(double(b.theta)));
}
template <typename T, typename Ids>
static hipError_t launch_begin_any(const PrefillBegin& b, bool norm, const Ids& ids, hipStream_t st) {
    if constexpr (sizeof(T) == 2) {
        if (!norm && b.d % 8 == 0 && ((uintptr_t(b.table) | uintptr_t(b.x)) & 15) == 0) {
            launch_begin<T, -1>(b, ids, st);
            return hipGetLastError();
        }
    }
    switch (norm ? b.d / 1024 : 0) {
        case 1: launch_begin<T, 1>(b, ids, st); break;
        case 2: launch_begin<T, 2>(b, ids, st); break;
        case 3: launch_begin<T, 3>(b, ids, st); break;
        case 4: launch_begin<T, 4>(b, ids, st); break;
        case 5: launch_begin<T, 5>(b, ids, st); break;
        case 6: launch_begin<T, 6>(b, ids, st); break;
        case 7: launch_begin<T, 7>(b, ids, st); break;
        case 8: launch_begin<T, 8>(b, ids, st); break;
        default: launch_begin<T, 0>(b, ids, st);
    }
    return hipGetLastError();
}

// whole pieces of 1024 elements, 16 bytes of x, h and the gains at once (8 of a bf16 table)
bool prefill_begin_norms(const PrefillBegin& b) {
    return b.gain && b.d % 1024 == 0 && b.d <= 8192 && ((uintptr_t(b.table) | uintptr_t(b.x) | uintptr_t(b.gain) | uintptr_t(b.h)) & 15) == 0;
}

hipError_t launch_prefill_begin(int dtype, const PrefillBegin& b, const int32_t* ids, const TokenIds* ids_by_value, hipStream_t st) {
    if (b.rows <= 0) return hipSuccess;
    if (ids_by_value && b.rows > TokenIds::MAX) return hipErrorInvalidValue;
    const bool norm = prefill_begin_norms(b);
    if (ids_by_value)
        return dtype == 0 ? launch_begin_any<float>(b, norm, IdsInArguments{*ids_by_value}, st)
                          : launch_begin_any<bf16_t>(b, norm, IdsInArguments{*ids_by_value}, st);
    return dtype == 0 ? launch_begin_any<float>(b, norm, IdsInMemory{ids}, st) : launch_begin_any<bf16_t>(b, norm, IdsInMemory{ids}, st);
}

// ------------------------------------------------------------------ rotary + KV page write
// grid.x: 64-token tiles aligned to absolute token index (so a tile never straddles a page);
// grid.y: head index in [0, n_q + 2 n_kv): query heads, then key heads, then value heads.
// K/V slots of the last tile that lie past the range are zeroed: attention reads whole
// 64-key tiles and masks by position, and 0 * NaN from stale memory would poison P V.
template <typename T, int HD>
__global__ void __launch_bounds__(256)
rope_kv_write_kernel(const float* __restrict__ qkv, const float2* __restrict__ cs, T* __restrict__ q, int n_q,
                     int tok_begin, int rows, KvView kv) {
    constexpr int HALF = HD / 2;
    __shared__ T vt[64][HD + 2];
    const int n_kv = kv.n_kv;
    const int ldq = (n_q + 2 * n_kv) * HD;
    const int head = blockIdx.y;
    const int tile_tok0 = (tok_begin / 64 + blockIdx.x) * 64;  // absolute
    const int lo = max(tile_tok0, tok_begin), hi = min(tile_tok0 + 64, tok_begin + rows);
    if (lo >= hi) return;
    const int lpage = tile_tok0 / kv.page_tokens;
    const int ppage = kv.block_table[lpage];
    const int in_page0 = tile_tok0 - lpage * kv.page_tokens;
    T* page = (T*)kv.pool + (size_t(kv.layer) * kv.n_physical_pages + ppage) * kv.page_elems();

    if (head < n_q + n_kv) {
        const bool is_q = head < n_q;
        for (int idx = threadIdx.x; idx < 64 * HALF; idx += 256) {
            int t = idx / HALF, pair = idx % HALF;
            int tok = tile_tok0 + t;
            if (tok < lo) continue;
            T* kdst = page + (size_t(head - n_q) * kv.page_tokens + in_page0 + t) * HD + 2 * pair;
            if (tok >= hi) {  // slots of this tile past the range: keep them finite for masked reads
                if (!is_q) { kdst[0] = from_f<T>(0.f); kdst[1] = from_f<T>(0.f); }
                continue;
            }
            int row = tok - tok_begin;
            float2 v = *(const float2*)(qkv + size_t(row) * ldq + head * HD + 2 * pair);
            float2 c = cs[row * HALF + pair];
            float o0 = v.x * c.x - v.y * c.y;
            float o1 = v.x * c.y + v.y * c.x;
            T* dst = is_q ? q + (size_t(head) * rows + row) * HD + 2 * pair : kdst;
            dst[0] = from_f<T>(o0);
            dst[1] = from_f<T>(o1);
        }
    } else {
        const int g = head - n_q - n_kv;
        for (int idx = threadIdx.x; idx < 64 * HD; idx += 256) {
            int t = idx / HD, e = idx % HD;
            int tok = tile_tok0 + t;
            float v = (tok >= lo && tok < hi) ? qkv[size_t(tok - tok_begin) * ldq + head * HD + e] : 0.f;
            vt[t][e] = from_f<T>(v);
        }
        __syncthreads();
        T* vpage = page + size_t(n_kv) * kv.page_tokens * HD + size_t(g) * HD * kv.page_tokens;
        for (int idx = threadIdx.x; idx < 64 * HD; idx += 256) {
            int e = idx / 64, t = idx % 64;
            int tok = tile_tok0 + t;
            if (tok >= lo) vpage[size_t(e) * kv.page_tokens + in_page0 + t] = vt[t][e];  // zeros past the range
        }
    }
}

// The same grid and semantics with 16-byte loads (4 consecutive elements = 2 rotary pairs per thread, HD / 4 threads per
// token row) and 8- or 16-byte stores; V^T leaves the LDS transpose in 16-byte pieces of consecutive tokens.  qkv may come
// as n_parts outputs, one per K range of the product, qkv[n_parts][rows][...], which are added up (in that order) as they
// are read.  A workgroup takes TOK tokens of a 64-token tile: all of them, or 16 where that leaves too few workgroups to
// hide the latency of the reads, which is what bounds it for small models (us, one pair or element per thread
// above and here: 512 rows of 48 bf16 heads of 64 9.2 and 4.9, 256 rows of 12 float32 heads of 64 8.5 and 3.0).
template <typename T, int HD, int TOK>
__global__ void __launch_bounds__(256)
rope_kv_write_vec_kernel(const float* __restrict__ qkv, int n_parts, const float2* __restrict__ cs, T* __restrict__ q,
                         int n_q, int tok_begin, int rows, KvView kv) {
    constexpr int HALF = HD / 2, TPR = HD / 4, RPP = 256 / TPR, PASSES = TOK / RPP;   // threads per row, rows per pass
    constexpr int E = 16 / sizeof(T), PP = TOK / E;                                   // tokens per V^T piece, pieces per head-dim row
    typedef __attribute__((__vector_size__(4 * sizeof(T)))) T vec4_t;
    typedef __attribute__((__vector_size__(16))) T piece_t;
    __shared__ T vt[TOK][HD + 4 / sizeof(T)];
    const int n_kv = kv.n_kv;
    const int ldq = (n_q + 2 * n_kv) * HD;
    const int head = blockIdx.y;
    const int tile_tok0 = tok_begin / 64 * 64 + blockIdx.x * TOK;  // absolute
    const int lo = max(tile_tok0, tok_begin), hi = min(tile_tok0 + TOK, tok_begin + rows);
    if (tile_tok0 + TOK <= tok_begin) return;   // (a piece wholly past the range still zeroes its K/V slots)
    const int lpage = tile_tok0 / kv.page_tokens;
    const int ppage = kv.block_table[lpage];
    const int in_page0 = tile_tok0 - lpage * kv.page_tokens;
    T* page = (T*)kv.pool + (size_t(kv.layer) * kv.n_physical_pages + ppage) * kv.page_elems();
    const int tx = threadIdx.x % TPR, ty = threadIdx.x / TPR;
    const size_t part_step = size_t(rows) * ldq;
    auto load = [&](int row) {
        const float* p = qkv + size_t(row) * ldq + head * HD + 4 * tx;
        float4 v = *(const float4*)p;
#pragma unroll 4
        for (int i = 1; i < n_parts; ++i) {
            const float4 a = *(const float4*)(p + i * part_step);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        return v;
    };

    if (head < n_q + n_kv) {
        const bool is_q = head < n_q;
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int t = ty + RPP * pass, tok = tile_tok0 + t;
            if (tok < lo) continue;
            T* kdst = page + (size_t(head - n_q) * kv.page_tokens + in_page0 + t) * HD + 4 * tx;
            if (tok >= hi) {  // slots of this tile past the range: keep them finite for masked reads
                if (!is_q) *(vec4_t*)kdst = vec4_t{0, 0, 0, 0};
                continue;
            }
            const int row = tok - tok_begin;
            const float4 v = load(row);
            const float4 c = *(const float4*)(cs + row * HALF + 2 * tx);   // (cos, sin) of pairs 2tx, 2tx+1
            vec4_t w = {from_f<T>(v.x * c.x - v.y * c.y), from_f<T>(v.x * c.y + v.y * c.x),
                        from_f<T>(v.z * c.z - v.w * c.w), from_f<T>(v.z * c.w + v.w * c.z)};
            T* dst = is_q ? q + (size_t(head) * rows + row) * HD + 4 * tx : kdst;
            *(vec4_t*)dst = w;
        }
    } else {
        const int g = head - n_q - n_kv;
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int t = ty + RPP * pass, tok = tile_tok0 + t;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (tok >= lo && tok < hi) v = load(tok - tok_begin);
            vt[t][4 * tx + 0] = from_f<T>(v.x); vt[t][4 * tx + 1] = from_f<T>(v.y);
            vt[t][4 * tx + 2] = from_f<T>(v.z); vt[t][4 * tx + 3] = from_f<T>(v.w);
        }
        __syncthreads();
        T* vpage = page + size_t(n_kv) * kv.page_tokens * HD + size_t(g) * HD * kv.page_tokens;
        // HD rows (head-dim index) x PP pieces of E tokens
#pragma unroll
        for (int i = 0; i < (HD * PP + 255) / 256; ++i) {
            const int piece = threadIdx.x + 256 * i, e = piece / PP, t0 = (piece % PP) * E;
            if (HD * PP % 256 != 0 && piece >= HD * PP) break;
            piece_t w;
#pragma unroll
            for (int k = 0; k < E; ++k) w[k] = vt[t0 + k][e];
            T* dst = vpage + size_t(e) * kv.page_tokens + in_page0 + t0;
            if (tile_tok0 + t0 >= lo) {
                *(piece_t*)dst = w;    // zeros past the range
            } else {                   // tokens before the range belong to an earlier call: leave them
#pragma unroll
                for (int k = 0; k < E; ++k)
                    if (tile_tok0 + t0 + k >= lo) dst[k] = w[k];
            }
        }
    }
}

template <typename T, int HD>
static void launch_rope_vec(dim3 grid, const float* qkv, int n_parts, const float2* cs, void* q, int n_q, int tok_begin, int rows,
                            const KvView& kv, hipStream_t st) {
    if (long(grid.x) * grid.y < 512)
        hipLaunchKernelGGL((rope_kv_write_vec_kernel<T, HD, 16>), dim3(4 * grid.x, grid.y), dim3(256), 0, st, qkv, n_parts, cs, (T*)q, n_q, tok_begin, rows, kv);
    else
        hipLaunchKernelGGL((rope_kv_write_vec_kernel<T, HD, 64>), grid, dim3(256), 0, st, qkv, n_parts, cs, (T*)q, n_q, tok_begin, rows, kv);
}

hipError_t launch_rope_kv_write(int dtype, const float* qkv, const float* cs, void* q, int n_q, int tok_begin,
                                int rows, const KvView& kv, hipStream_t st, int n_parts) {
    if (rows <= 0) return hipSuccess;
    int tiles = (tok_begin + rows - 1) / 64 - tok_begin / 64 + 1;
    dim3 grid(tiles, n_q + 2 * kv.n_kv), block(256);
    const float2* c2 = (const float2*)cs;
    const bool aligned = ((uintptr_t(qkv) | uintptr_t(cs) | uintptr_t(q) | uintptr_t(kv.pool)) & 15) == 0;
    if (aligned && (dtype == 0 || dtype == 1) && (kv.head_dim == 64 || kv.head_dim == 128)) {
        if (dtype == 0 && kv.head_dim == 64) launch_rope_vec<float, 64>(grid, qkv, n_parts, c2, q, n_q, tok_begin, rows, kv, st);
        else if (dtype == 0) launch_rope_vec<float, 128>(grid, qkv, n_parts, c2, q, n_q, tok_begin, rows, kv, st);
        else if (kv.head_dim == 64) launch_rope_vec<bf16_t, 64>(grid, qkv, n_parts, c2, q, n_q, tok_begin, rows, kv, st);
        else launch_rope_vec<bf16_t, 128>(grid, qkv, n_parts, c2, q, n_q, tok_begin, rows, kv, st);
        return hipGetLastError();
    }
    if (n_parts > 1) return hipErrorInvalidValue;
    if (dtype == 0 && kv.head_dim == 64)
        hipLaunchKernelGGL((rope_kv_write_kernel<float, 64>), grid, block, 0, st, qkv, c2, (float*)q, n_q, tok_begin, rows, kv);
    else if (dtype == 0 && kv.head_dim == 128)
        hipLaunchKernelGGL((rope_kv_write_kernel<float, 128>), grid, block, 0, st, qkv, c2, (float*)q, n_q, tok_begin, rows, kv);
    else if (dtype == 1 && kv.head_dim == 64)
        hipLaunchKernelGGL((rope_kv_write_kernel<bf16_t, 64>), grid, block, 0, st, qkv, c2, (bf16_t*)q, n_q, tok_begin, rows, kv);
    else if (dtype == 1 && kv.head_dim == 128)
        hipLaunchKernelGGL((rope_kv_write_kernel<bf16_t, 128>), grid, block, 0, st, qkv, c2, (bf16_t*)q, n_q, tok_begin, rows, kv);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// ------------------------------------------------------------------ plain GEMM
// out[M][N] = a[M][K] * w[N][K]^T with float32 accumulation.  64x64 tile, 16-deep slices
// through LDS, 4x4 outputs per thread.  K must be a multiple of 4.
template <typename T> struct Vec4;
template <> struct Vec4<float> { typedef float4 type; };
template <> struct Vec4<bf16_t> { typedef uint2 type; };

template <typename T>
__device__ __forceinline__ void load4(const T* p, float* o);
template <>
__device__ __forceinline__ void load4<float>(const float* p, float* o) {
    float4 v = *(const float4*)p;
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
template <>
__device__ __forceinline__ void load4<bf16_t>(const bf16_t* p, float* o) {
    uint2 v = *(const uint2*)p;
    o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
    o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

template <typename T, int EPI>
__global__ void __launch_bounds__(256)
gemm_generic_kernel(const T* __restrict__ a, const T* __restrict__ w, const T* __restrict__ w2, void* __restrict__ outv,
                    int M, int N, int K) {
    constexpr int BK = 16;
    __shared__ float As[BK][64 + 4];
    __shared__ float Ws[BK][64 + 4];
    __shared__ float W2s[EPI == EPI_SWIGLU ? BK : 1][64 + 4];
    const int tid = threadIdx.x;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int lr = tid >> 2, lk = (tid & 3) * 4;
    const int arow = min(m0 + lr, M - 1), wrow = min(n0 + lr, N - 1);
    const int ty = tid >> 4, tx = tid & 15;
    float acc[4][4] = {}, acc2[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += BK) {
        float va[4] = {0, 0, 0, 0}, vw[4] = {0, 0, 0, 0}, vw2[4] = {0, 0, 0, 0};
        if (k0 + lk < K) {
            load4<T>(a + size_t(arow) * K + k0 + lk, va);
            load4<T>(w + size_t(wrow) * K + k0 + lk, vw);
            if (EPI == EPI_SWIGLU) load4<T>(w2 + size_t(wrow) * K + k0 + lk, vw2);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            As[lk + i][lr] = va[i];
            Ws[lk + i][lr] = vw[i];
            if (EPI == EPI_SWIGLU) W2s[lk + i][lr] = vw2[i];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BK; ++k) {
            float ar[4], wr[4], w2r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ar[i] = As[k][ty * 4 + i];
                wr[i] = Ws[k][tx * 4 + i];
                if (EPI == EPI_SWIGLU) w2r[i] = W2s[k][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] = fmaf(ar[i], wr[j], acc[i][j]);
                    if (EPI == EPI_SWIGLU) acc2[i][j] = fmaf(ar[i], w2r[j], acc2[i][j]);
                }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int row = m0 + ty * 4 + i;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int col = n0 + tx * 4 + j;
            if (col >= N) continue;
            size_t o = size_t(row) * N + col;
            if (EPI == EPI_STORE_F32) ((float*)outv)[o] = acc[i][j];
            else if (EPI == EPI_RESIDUAL_F32) ((float*)outv)[o] += acc[i][j];
            else {
                float g = acc[i][j];
                ((T*)outv)[o] = from_f<T>(g / (1.0f + expf(-g)) * acc2[i][j]);
            }
        }
    }
}

template <typename T>
static hipError_t gemm_generic_t(int epi, const void* a, const void* w, const void* w2, void* out, int M, int N, int K,
                                 hipStream_t st) {
    dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
    const T *A = (const T*)a, *W = (const T*)w, *W2 = (const T*)w2;
    if (epi == EPI_STORE_F32) hipLaunchKernelGGL((gemm_generic_kernel<T, EPI_STORE_F32>), grid, block, 0, st, A, W, W2, out, M, N, K);
    else if (epi == EPI_RESIDUAL_F32) hipLaunchKernelGGL((gemm_generic_kernel<T, EPI_RESIDUAL_F32>), grid, block, 0, st, A, W, W2, out, M, N, K);
    else if (epi == EPI_SWIGLU) hipLaunchKernelGGL((gemm_generic_kernel<T, EPI_SWIGLU>), grid, block, 0, st, A, W, W2, out, M, N, K);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_gemm_generic(int dtype, int epi, const void* a, const void* w, const void* w2, void* out, int M,
                               int N, int K, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K <= 0 || (K & 3)) return hipErrorInvalidValue;
    return dtype == 0 ? gemm_generic_t<float>(epi, a, w, w2, out, M, N, K, st)
                      : gemm_generic_t<bf16_t>(epi, a, w, w2, out, M, N, K, st);
}

// ------------------------------------------------------------------ plain attention
// One wavefront per (query row, query head).  Keys are visited in groups of 64 (one key per
// lane for the scores); the running max / sum of the online softmax are wave-uniform; each
// lane owns HD/64 output dimensions for the P V accumulation.
template <typename T, int HD>
__global__ void __launch_bounds__(64)
attention_generic_kernel(const T* __restrict__ q, T* __restrict__ out, int n_q, int tok_begin, int rows, KvView kv) {
    constexpr int EPL = HD / 64;  // output dims per lane
    const int row = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int g = h / (n_q / kv.n_kv);
    const int qpos = tok_begin + row;
    const float scale = 1.0f / sqrtf(float(HD));
    float qr[HD];
    const T* qp = q + (size_t(h) * rows + row) * HD;
#pragma unroll
    for (int e = 0; e < HD; ++e) qr[e] = to_f<T>(qp[e]) * scale;
    float m_run = -INFINITY, l_run = 0.f, o[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) o[i] = 0.f;
    const int n_groups = qpos / 64 + 1;
    const int pt = kv.page_tokens;
    for (int grp = 0; grp < n_groups; ++grp) {
        const int key0 = grp * 64;
        const int lpage = key0 / pt;
        const int in_page0 = key0 - lpage * pt;
        const T* page = (const T*)kv.pool + (size_t(kv.layer) * kv.n_physical_pages + kv.block_table[lpage]) * kv.page_elems();
        const T* kp = page + (size_t(g) * pt + in_page0 + lane) * HD;
        const T* vp = page + size_t(kv.n_kv) * pt * HD + size_t(g) * HD * pt + in_page0;
        float s = -INFINITY;
        if (key0 + lane <= qpos) {
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < HD; ++e) acc = fmaf(qr[e], to_f<T>(kp[e]), acc);
            s = acc;
        }
        float m_new = fmaxf(m_run, wave_max(s));
        float p = (key0 + lane <= qpos) ? expf(s - m_new) : 0.f;
        float corr = expf(m_run - m_new);
        l_run = l_run * corr + wave_sum(p);
        m_run = m_new;
        const int n_valid = min(64, qpos - key0 + 1);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const T* vrow = vp + size_t(lane + 64 * i) * pt;
            float acc = o[i] * corr;
            for (int j = 0; j < n_valid; ++j) acc = fmaf(__shfl(p, j, 64), to_f<T>(vrow[j]), acc);
            o[i] = acc;
        }
    }
    T* op = out + size_t(row) * n_q * HD + h * HD;
#pragma unroll
    for (int i = 0; i < EPL; ++i) op[lane + 64 * i] = from_f<T>(o[i] / l_run);
}

hipError_t launch_attention_generic(int dtype, const void* q, void* out, int n_q, int tok_begin, int rows,
                                    const KvView& kv, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    dim3 grid(rows, n_q), block(64);
    if (dtype == 0 && kv.head_dim == 64)
        hipLaunchKernelGGL((attention_generic_kernel<float, 64>), grid, block, 0, st, (const float*)q, (float*)out, n_q, tok_begin, rows, kv);
    else if (dtype == 0 && kv.head_dim == 128)
        hipLaunchKernelGGL((attention_generic_kernel<float, 128>), grid, block, 0, st, (const float*)q, (float*)out, n_q, tok_begin, rows, kv);
    else if (dtype == 1 && kv.head_dim == 64)
        hipLaunchKernelGGL((attention_generic_kernel<bf16_t, 64>), grid, block, 0, st, (const bf16_t*)q, (bf16_t*)out, n_q, tok_begin, rows, kv);
    else if (dtype == 1 && kv.head_dim == 128)
        hipLaunchKernelGGL((attention_generic_kernel<bf16_t, 128>), grid, block, 0, st, (const bf16_t*)q, (bf16_t*)out, n_q, tok_begin, rows, kv);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace cake
