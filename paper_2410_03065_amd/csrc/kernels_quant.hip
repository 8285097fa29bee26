// Quantised stored KV on the load path (Sec. 5.5 combines KV compression with the method: a smaller
// stored KV loads faster, so the meet point moves towards the front).
//
// Store format per page, per layer, per K|V: codes [kv_head][token][hd] followed by float32
// scales [kv_head][token]; value = code * scale (one scale per token and KV head, symmetric,
// absmax / QMAX).  8-bit: one int8 code per element, QMAX 127.  4-bit: two codes per byte (element
// 2i in the low nibble, 2i+1 in the high nibble, two's complement), QMAX 7.  V is not transposed
// in the store; the pages hold V^T, so the kernels transpose V tiles through LDS.
//
// All are streaming kernels.  bf16 pages go 8 elements (16 bytes) at a time: HD / 8 neighbouring lanes hold a token
// row, its largest magnitude is found by exchanging among them, and V tiles pass through LDS in rows of HD + 2 elements
// (an odd number of 32-bit words: neither the rows written nor the columns read meet in a bank).  One element per thread
// and a quarter row strided through LDS took 14.4 us to quantise and 9.5 to expand a 256-token page of four resp. eight
// Llama3-8B layers; the kernels below take 12.5 for four pages in a launch, and 6.4.
#include <algorithm>

#include "kernels.hpp"

namespace cake {

namespace {
template <typename T> __device__ __forceinline__ T qfrom_f(float v);
template <> __device__ __forceinline__ float qfrom_f<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t qfrom_f<bf16_t>(float v) { return bf16_t(v); }
template <typename T> __device__ __forceinline__ float qto_f(T v);
template <> __device__ __forceinline__ float qto_f<float>(float v) { return v; }
template <> __device__ __forceinline__ float qto_f<bf16_t>(bf16_t v) { return float(v); }
// sign-extended nibble n (0 or 1) of a byte
__device__ __forceinline__ int nibble(unsigned b, int n) { return (int(b << (28 - 4 * n))) >> 28; }
}  // namespace

// Page images, image_bytes apart -> layer pages.  grid.x: (layer, K|V, kv_head); grid.y: 64-token tiles of the page;
// grid.z: images.
template <typename T, int HD, int BITS>
__global__ void __launch_bounds__(256)
dequant_page_kernel(const unsigned char* __restrict__ images, size_t image_bytes, KvView kv, PageRun run) {
    __shared__ float tile[64][HD + 1];
    constexpr int ROWB = HD * BITS / 8;          // code bytes per token row
    const int pt = kv.page_tokens, n_kv = kv.n_kv;
    const int g = blockIdx.x % n_kv, which = (blockIdx.x / n_kv) & 1, layer = blockIdx.x / (2 * n_kv);
    const int t0 = blockIdx.y * 64;
    const size_t slab = size_t(n_kv) * pt * (ROWB + 4);
    const unsigned char* base = images + blockIdx.z * image_bytes + (size_t(layer) * 2 + which) * slab;
    const unsigned char* codes = base + (size_t(g) * pt + t0) * ROWB;
    const float* scales = (const float*)(base + size_t(n_kv) * pt * ROWB) + size_t(g) * pt + t0;
    T* page = (T*)kv.pool + (size_t(layer) * kv.n_physical_pages + run.phys[blockIdx.z]) * kv.page_elems();
    // 64 tokens x HD elements, 4 per thread per pass (coalesced 4- or 2-byte reads)
    for (int idx = threadIdx.x * 4; idx < 64 * HD; idx += 256 * 4) {
        const int t = idx / HD, e = idx % HD;
        const float sc = scales[t];
        float v0, v1, v2, v3;
        if constexpr (BITS == 8) {
            const char4 c = *(const char4*)(codes + idx);
            v0 = float(c.x) * sc; v1 = float(c.y) * sc; v2 = float(c.z) * sc; v3 = float(c.w) * sc;
        } else {
            const unsigned c = *(const unsigned short*)(codes + idx / 2);
            v0 = float(nibble(c, 0)) * sc; v1 = float(nibble(c, 1)) * sc;
            v2 = float(nibble(c, 2)) * sc; v3 = float(nibble(c, 3)) * sc;
        }
        if (which == 0) {
            T* dst = page + (size_t(g) * pt + t0 + t) * HD + e;
            if constexpr (sizeof(T) == 2) {
                typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
                *(bf16x4_t*)dst = bf16x4_t{bf16_t(v0), bf16_t(v1), bf16_t(v2), bf16_t(v3)};
            } else {
                *(float4*)dst = make_float4(v0, v1, v2, v3);
            }
        } else {
            tile[t][e] = v0; tile[t][e + 1] = v1; tile[t][e + 2] = v2; tile[t][e + 3] = v3;
        }
    }
    if (which == 1) {
        __syncthreads();
        T* vpage = page + size_t(n_kv) * pt * HD + size_t(g) * HD * pt;
        for (int idx = threadIdx.x; idx < 64 * HD; idx += 256) {
            const int e = idx / 64, t = idx % 64;
            vpage[size_t(e) * pt + t0 + t] = qfrom_f<T>(tile[t][e]);
        }
    }
}

// What follows for bf16 pages.  A thread's 8 elements e0 .. e0+7 of token row t, t = 256 / (HD / 8) rows per pass.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 q_bf16x8;

template <int HD, int BITS>
__global__ void __launch_bounds__(256)
dequant_page_bf16_kernel(const unsigned char* __restrict__ images, size_t image_bytes, KvView kv, PageRun run) {
    __shared__ unsigned tile[64][HD / 2 + 1];     // bf16 pairs
    constexpr int ROWB = HD * BITS / 8, LPR = HD / 8, RPP = 256 / LPR;
    const int pt = kv.page_tokens, n_kv = kv.n_kv;
    const int g = blockIdx.x % n_kv, which = (blockIdx.x / n_kv) & 1, layer = blockIdx.x / (2 * n_kv);
    const int t0 = blockIdx.y * 64;
    const size_t slab = size_t(n_kv) * pt * (ROWB + 4);
    const unsigned char* base = images + blockIdx.z * image_bytes + (size_t(layer) * 2 + which) * slab;
    const unsigned char* codes = base + (size_t(g) * pt + t0) * ROWB;
    const float* scales = (const float*)(base + size_t(n_kv) * pt * ROWB) + size_t(g) * pt + t0;
    bf16_t* page = (bf16_t*)kv.pool + (size_t(layer) * kv.n_physical_pages + run.phys[blockIdx.z]) * kv.page_elems();
    const int e0 = (threadIdx.x % LPR) * 8, r0 = threadIdx.x / LPR;
    uint2 c[64 / RPP];
    float sc[64 / RPP];
#pragma unroll
    for (int i = 0; i < 64 / RPP; ++i) {
        const unsigned char* p = codes + (r0 + i * RPP) * ROWB + e0 * BITS / 8;
        if constexpr (BITS == 8) c[i] = *(const uint2*)p;
        else c[i] = make_uint2(*(const unsigned*)p, 0);
        sc[i] = scales[r0 + i * RPP];
    }
#pragma unroll
    for (int i = 0; i < 64 / RPP; ++i) {
        const int t = r0 + i * RPP;
        q_bf16x8 v;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const unsigned w = BITS == 8 && k >= 4 ? c[i].y : c[i].x;
            const int code = BITS == 8 ? int(w << (24 - 8 * (k & 3))) >> 24 : int(w << (28 - 4 * k)) >> 28;
            v[k] = bf16_t(float(code) * sc[i]);
        }
        if (which == 0) {
            *(q_bf16x8*)(page + (size_t(g) * pt + t0 + t) * HD + e0) = v;
        } else {
            unsigned w[4];
            __builtin_memcpy(w, &v, 16);
#pragma unroll
            for (int k = 0; k < 4; ++k) tile[t][e0 / 2 + k] = w[k];
        }
    }
    if (which == 1) {
        __syncthreads();
        bf16_t* vpage = page + size_t(n_kv) * pt * HD + size_t(g) * HD * pt + t0;
        const bf16_t* tb = (const bf16_t*)&tile[0][0];
#pragma unroll
        for (int i = 0; i < HD * 8 / 256; ++i) {   // 8 tokens of one head-dim element each
            const int piece = threadIdx.x + 256 * i, e = piece >> 3, t = (piece & 7) * 8;
            q_bf16x8 v;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = tb[(t + k) * (HD + 2) + e];
            *(q_bf16x8*)(vpage + size_t(e) * pt + t) = v;
        }
    }
}

// Logical pages first_page + z of `kv`, z < gridDim.z, into images[z].
template <int HD, int BITS>
__global__ void __launch_bounds__(256)
quant_pages_bf16_kernel(unsigned char* __restrict__ images, size_t image_bytes, KvView kv, int first_page) {
    __shared__ unsigned tile[64][HD / 2 + 1];
    constexpr int ROWB = HD * BITS / 8, LPR = HD / 8, RPP = 256 / LPR;
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    const int pt = kv.page_tokens, n_kv = kv.n_kv;
    const int g = blockIdx.x % n_kv, which = (blockIdx.x / n_kv) & 1, layer = blockIdx.x / (2 * n_kv);
    const int t0 = blockIdx.y * 64;
    const size_t slab = size_t(n_kv) * pt * (ROWB + 4);
    unsigned char* base = images + blockIdx.z * image_bytes + (size_t(layer) * 2 + which) * slab;
    unsigned char* codes = base + (size_t(g) * pt + t0) * ROWB;
    float* scales = (float*)(base + size_t(n_kv) * pt * ROWB) + size_t(g) * pt + t0;
    const bf16_t* page = (const bf16_t*)kv.pool + (size_t(layer) * kv.n_physical_pages + kv.block_table[first_page + blockIdx.z]) * kv.page_elems();
    const int e0 = (threadIdx.x % LPR) * 8, r0 = threadIdx.x / LPR;
    q_bf16x8 v[64 / RPP];
    if (which == 0) {
#pragma unroll
        for (int i = 0; i < 64 / RPP; ++i) v[i] = *(const q_bf16x8*)(page + (size_t(g) * pt + t0 + r0 + i * RPP) * HD + e0);
    } else {
        const bf16_t* vpage = page + size_t(n_kv) * pt * HD + size_t(g) * HD * pt + t0;
        bf16_t* tb = (bf16_t*)&tile[0][0];
#pragma unroll
        for (int i = 0; i < HD * 8 / 256; ++i) {
            const int piece = threadIdx.x + 256 * i, e = piece >> 3, t = (piece & 7) * 8;
            const q_bf16x8 x = *(const q_bf16x8*)(vpage + size_t(e) * pt + t);
#pragma unroll
            for (int k = 0; k < 8; ++k) tb[(t + k) * (HD + 2) + e] = x[k];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 64 / RPP; ++i) {
            unsigned w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = tile[r0 + i * RPP][e0 / 2 + k];
            __builtin_memcpy(&v[i], w, 16);
        }
    }
#pragma unroll
    for (int i = 0; i < 64 / RPP; ++i) {
        const int t = r0 + i * RPP;
        float amax = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) amax = fmaxf(amax, fabsf(float(v[i][k])));
#pragma unroll
        for (int o = 1; o < LPR; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        const float scale = amax / QMAX;
        const float safe = scale > 0.f ? scale : 1.0f;
        unsigned out[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float q = rintf(float(v[i][k]) / safe);
            q = fminf(fmaxf(q, -QMAX), QMAX);
            const int code = scale > 0.f ? int(q) : 0;
            if constexpr (BITS == 8) out[k >> 2] |= (unsigned(code) & 0xFFu) << (8 * (k & 3));
            else out[0] |= (unsigned(code) & 0xFu) << (4 * k);
        }
        unsigned char* dst = codes + size_t(t) * ROWB + e0 * BITS / 8;
        if constexpr (BITS == 8) *(uint2*)dst = make_uint2(out[0], out[1]);
        else *(unsigned*)dst = out[0];
        if (e0 == 0) scales[t] = scale;
    }
}

template <int BITS>
static hipError_t launch_dequant_bits(int dtype, const unsigned char* img, size_t image_bytes, const KvView& kv, const PageRun& run,
                                      int n_layers, hipStream_t st) {
    dim3 grid(n_layers * 2 * kv.n_kv, kv.page_tokens / 64, run.n), block(256);
    const bool wide = ((uintptr_t(img) | uintptr_t(kv.pool) | image_bytes) & 15) == 0;   // 8- and 16-byte accesses
    if (dtype == 0 && kv.head_dim == 64) hipLaunchKernelGGL((dequant_page_kernel<float, 64, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else if (dtype == 0 && kv.head_dim == 128) hipLaunchKernelGGL((dequant_page_kernel<float, 128, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else if (dtype == 1 && kv.head_dim == 64 && wide) hipLaunchKernelGGL((dequant_page_bf16_kernel<64, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else if (dtype == 1 && kv.head_dim == 128 && wide) hipLaunchKernelGGL((dequant_page_bf16_kernel<128, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else if (dtype == 1 && kv.head_dim == 64) hipLaunchKernelGGL((dequant_page_kernel<bf16_t, 64, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else if (dtype == 1 && kv.head_dim == 128) hipLaunchKernelGGL((dequant_page_kernel<bf16_t, 128, BITS>), grid, block, 0, st, img, image_bytes, kv, run);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_dequant_pages(int dtype, const void* images, size_t image_bytes, const KvView& kv, const PageRun& run, int n_layers,
                                int bits, hipStream_t st) {
    if (kv.page_tokens % 64 || run.n <= 0 || run.n > PageRun::MAX) return hipErrorInvalidValue;
    const unsigned char* img = (const unsigned char*)images;
    if (bits == 8) return launch_dequant_bits<8>(dtype, img, image_bytes, kv, run, n_layers, st);
    if (bits == 4) return launch_dequant_bits<4>(dtype, img, image_bytes, kv, run, n_layers, st);
    return hipErrorInvalidValue;
}

// Layer pages -> one page image (the tool that writes a store from a cache that is in HBM).
// Same grid.  Four threads share a token row: absmax over the row, scale = absmax / QMAX,
// code = round-half-even(x / scale) clipped to +-QMAX; a row of zeros gets scale 0 and codes 0.
template <typename T, int HD, int BITS>
__global__ void __launch_bounds__(256)
quant_page_kernel(unsigned char* __restrict__ image, KvView kv, int phys_page, int n_layers) {
    __shared__ float tile[64][HD + 1];
    constexpr int ROWB = HD * BITS / 8;
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    const int pt = kv.page_tokens, n_kv = kv.n_kv;
    const int g = blockIdx.x % n_kv, which = (blockIdx.x / n_kv) & 1, layer = blockIdx.x / (2 * n_kv);
    const int t0 = blockIdx.y * 64;
    const size_t slab = size_t(n_kv) * pt * (ROWB + 4);
    unsigned char* base = image + (size_t(layer) * 2 + which) * slab;
    unsigned char* codes = base + (size_t(g) * pt + t0) * ROWB;
    float* scales = (float*)(base + size_t(n_kv) * pt * ROWB) + size_t(g) * pt + t0;
    const T* page = (const T*)kv.pool + (size_t(layer) * kv.n_physical_pages + phys_page) * kv.page_elems();
    if (which == 0) {
        const T* src = page + (size_t(g) * pt + t0) * HD;
        for (int idx = threadIdx.x; idx < 64 * HD; idx += 256) tile[idx / HD][idx % HD] = qto_f<T>(src[idx]);
    } else {
        const T* vpage = page + size_t(n_kv) * pt * HD + size_t(g) * HD * pt;
        for (int idx = threadIdx.x; idx < 64 * HD; idx += 256) {
            const int e = idx / 64, t = idx % 64;
            tile[t][e] = qto_f<T>(vpage[size_t(e) * pt + t0 + t]);
        }
    }
    __syncthreads();
    const int t = threadIdx.x >> 2, part = threadIdx.x & 3;   // 4 threads per token row
    float amax = 0.f;
    for (int e = part; e < HD; e += 4) amax = fmaxf(amax, fabsf(tile[t][e]));
    amax = fmaxf(amax, __shfl_xor(amax, 1, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 2, 64));
    const float scale = amax / QMAX;
    const float safe = scale > 0.f ? scale : 1.0f;
    auto code = [&](int e) -> int {
        float q = rintf(tile[t][e] / safe);
        q = fminf(fmaxf(q, -QMAX), QMAX);
        return scale > 0.f ? int(q) : 0;
    };
    if constexpr (BITS == 8) {
        for (int e = part; e < HD; e += 4) codes[size_t(t) * ROWB + e] = (unsigned char)(signed char)code(e);
    } else {
        // a thread packs the element pairs (2b, 2b+1) of bytes b = part, part + 4, ...
        for (int b = part; b < HD / 2; b += 4)
            codes[size_t(t) * ROWB + b] = (unsigned char)((code(2 * b) & 0xF) | ((code(2 * b + 1) & 0xF) << 4));
    }
    if (part == 0) scales[t] = scale;
}

// images + z * image_bytes = the image of logical page first_page + z, z < n_pages (block_table_host: the physical pages,
// for the kernel that takes one at a time).
template <int BITS>
static hipError_t launch_quant_bits(int dtype, unsigned char* img, size_t image_bytes, const KvView& kv, const int32_t* block_table_host,
                                    int first_page, int n_pages, int n_layers, hipStream_t st) {
    dim3 grid(n_layers * 2 * kv.n_kv, kv.page_tokens / 64), block(256);
    if (dtype == 1 && ((uintptr_t(img) | uintptr_t(kv.pool) | image_bytes) & 15) == 0 && (kv.head_dim == 64 || kv.head_dim == 128)) {
        grid.z = n_pages;
        if (kv.head_dim == 64) hipLaunchKernelGGL((quant_pages_bf16_kernel<64, BITS>), grid, block, 0, st, img, image_bytes, kv, first_page);
        else hipLaunchKernelGGL((quant_pages_bf16_kernel<128, BITS>), grid, block, 0, st, img, image_bytes, kv, first_page);
        return hipGetLastError();
    }
    for (int p = 0; p < n_pages; ++p, img += image_bytes) {
        const int phys_page = block_table_host[first_page + p];
        if (dtype == 0 && kv.head_dim == 64) hipLaunchKernelGGL((quant_page_kernel<float, 64, BITS>), grid, block, 0, st, img, kv, phys_page, n_layers);
        else if (dtype == 0 && kv.head_dim == 128) hipLaunchKernelGGL((quant_page_kernel<float, 128, BITS>), grid, block, 0, st, img, kv, phys_page, n_layers);
        else if (dtype == 1 && kv.head_dim == 64) hipLaunchKernelGGL((quant_page_kernel<bf16_t, 64, BITS>), grid, block, 0, st, img, kv, phys_page, n_layers);
        else if (dtype == 1 && kv.head_dim == 128) hipLaunchKernelGGL((quant_page_kernel<bf16_t, 128, BITS>), grid, block, 0, st, img, kv, phys_page, n_layers);
        else return hipErrorInvalidValue;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_quant_pages(int dtype, void* images, size_t image_bytes, const KvView& kv, const int32_t* block_table_host, int first_page,
                              int n_pages, int n_layers, int bits, hipStream_t st) {
    if (kv.page_tokens % 64) return hipErrorInvalidValue;
    if (n_pages <= 0) return hipSuccess;
    unsigned char* img = (unsigned char*)images;
    if (bits == 8) return launch_quant_bits<8>(dtype, img, image_bytes, kv, block_table_host, first_page, n_pages, n_layers, st);
    if (bits == 4) return launch_quant_bits<4>(dtype, img, image_bytes, kv, block_table_host, first_page, n_pages, n_layers, st);
    return hipErrorInvalidValue;
}

// Raw images in device memory, image_bytes apart <-> layer pages: 16 KB (a divisor of every layer page) per workgroup and
// turn.  Streaming; a 256-token page of eight layers is 512 of these.
template <bool EXPORT>
__global__ void __launch_bounds__(256) move_pages_kernel(char* __restrict__ images, size_t image_bytes, KvView kv, PageRun run,
                                                         size_t layer_bytes, int n_layers) {
    const int per_layer = int(layer_bytes >> 14), n_items = per_layer * n_layers;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int layer = item / per_layer;
        const size_t off = size_t(item % per_layer) << 14;
        uint4* image = (uint4*)(images + blockIdx.y * image_bytes + layer * layer_bytes + off);
        uint4* page = (uint4*)((char*)kv.pool + (size_t(layer) * kv.n_physical_pages + run.phys[blockIdx.y]) * layer_bytes + off);
        const uint4* src = EXPORT ? page : image;
        uint4* dst = EXPORT ? image : page;
        uint4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = src[threadIdx.x + 256 * i];
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[threadIdx.x + 256 * i] = v[i];
    }
}

bool move_pages_supported(const void* images, size_t layer_bytes, const KvView& kv) {
    return layer_bytes && (layer_bytes & 16383) == 0 && ((uintptr_t(images) | uintptr_t(kv.pool)) & 15) == 0;
}

template <bool EXPORT>
static hipError_t launch_move_pages(char* images, size_t image_bytes, const KvView& kv, const PageRun& run, size_t layer_bytes, int n_layers,
                                    hipStream_t st) {
    if (!move_pages_supported(images, layer_bytes, kv) || (image_bytes & 15) || run.n <= 0 || run.n > PageRun::MAX) return hipErrorInvalidValue;
    const long items = long(layer_bytes >> 14) * n_layers;
    hipLaunchKernelGGL(move_pages_kernel<EXPORT>, dim3(unsigned(std::min(items, 2048L)), run.n), dim3(256), 0, st, images, image_bytes, kv, run,
                       layer_bytes, n_layers);
    return hipGetLastError();
}

hipError_t launch_import_pages(const void* images, size_t image_bytes, const KvView& kv, const PageRun& run, size_t layer_bytes,
                               int n_layers, hipStream_t st) {
    return launch_move_pages<false>((char*)images, image_bytes, kv, run, layer_bytes, n_layers, st);
}
hipError_t launch_export_pages(void* images, size_t image_bytes, const KvView& kv, const PageRun& run, size_t layer_bytes, int n_layers,
                               hipStream_t st) {
    return launch_move_pages<true>((char*)images, image_bytes, kv, run, layer_bytes, n_layers, st);
}

}  // namespace cake
