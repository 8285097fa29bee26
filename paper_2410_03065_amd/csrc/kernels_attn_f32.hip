// Float32 attention on the matrix cores, and the kernel that merges the key ranges of any attention launch that
// split its keys (Sec. 3 "Attention and KV cache", "Chunk Prefill").
//
// MFMA used: v_mfma_f32_32x32x2_f32 (float32 products and sums, 256 FLOP per clock and CU).  For D[32x32] +=
// A[32x2] * B[2x32] lane l supplies A[l%32][l/32] and B[l/32][l%32] and holds D[8*(v/4) + 4*(l/32) + v%4][l%32]
// in accumulator register v (0..15).
#include <algorithm>
#include <cfloat>

#include "kernels.hpp"

namespace cake {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// =====================================================================================
// One workgroup = 32 queries of one head over one range of keys; its four waves take the range's 32-key tiles in
// turn with private softmax state and are merged through LDS at the end.
//
// As in the bf16 kernels the score tile is formed transposed, S^T[key][query], so a lane owns one query and the
// probabilities in accumulator register v are already the B operand of the second product, O^T[hd][query] +=
// V^T[hd][key] P^T[key][query]: MFMA step v of a tile contracts the keys 8*(v/4) + v%4 (low half-wave) and
// 8*(v/4) + 4 + v%4 (high half-wave), so the V^T operands of four steps are one aligned 16-byte read per lane.
// Along the head dimension the contraction order is free as long as both operands share it: half-wave h takes
// elements 8j + 4h .. + 3, again 16 bytes per read.  Nothing is shared between waves, so nothing is staged in LDS.
//
// What bounds it: the float32 matrix rate where there are enough queries; for the few queries of a small model's
// chunk the number of waves, hence the key ranges (launch_attention_f32).  256 rows x 4 heads x 64 against 2048
// keys: 18 us with the merge, against 352 us for one wave per row and query head with a lane per key, whose 64
// lanes each walked a key row of their own (one cache line per lane and load).
//
// The exponentials are expf, not the hardware's exp2 of a product with log2 e: that product's rounding is worth
// |x| 2^-24 of e^x (3.4e-6 at probabilities of e^-80, 1.1e-7 now; 5 to 10 % of the time).
// =====================================================================================
constexpr int FQ = 32, FK = 32;

template <int HD>
__global__ void __launch_bounds__(256)
attention_f32_kernel(const float* __restrict__ q, float* __restrict__ out, float* __restrict__ part, int n_q, int tok_begin,
                     int rows, KvView kv, int tiles_per_split) {
    constexpr int NC = HD / 8, ND = HD / 32;   // 16-byte pieces of a key row per lane; 32-row blocks of V^T
    __shared__ float o_lds[4][HD][FQ];
    __shared__ float m_lds[4][FQ], l_lds[4][FQ];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int h = blockIdx.y, g = h / (n_q / kv.n_kv), q0 = blockIdx.x * FQ, split = blockIdx.z;
    const int pt = kv.page_tokens;
    const int my_pos = tok_begin + min(q0 + lrow, rows - 1);
    const int first_pos = tok_begin + q0, last_pos = tok_begin + min(q0 + FQ, rows) - 1;
    const int n_tiles = last_pos / FK + 1;
    const int tile_lo = split * tiles_per_split, tile_hi = min(tile_lo + tiles_per_split, n_tiles);
    const float scale = 1.0f / sqrtf(float(HD));

    float4 qr[NC];
    {
        const float* qp = q + (size_t(h) * rows + (my_pos - tok_begin)) * HD + 4 * lhalf;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const float4 v = *(const float4*)(qp + 8 * j);
            qr[j] = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
        }
    }
    const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;
    float4 kr[NC], vr[ND][4];
    auto tile_page = [&](int tile, int* in_page0) {
        const int key0 = tile * FK, lpage = key0 / pt;
        *in_page0 = key0 - lpage * pt;
        return (const float*)kv.pool + (layer_base + kv.block_table[lpage]) * kv.page_elems();
    };
    auto load_k = [&](int tile) {
        int in_page0;
        const float* kp = tile_page(tile, &in_page0) + (size_t(g) * pt + in_page0 + lrow) * HD + 4 * lhalf;
#pragma unroll
        for (int j = 0; j < NC; ++j) kr[j] = *(const float4*)(kp + 8 * j);
    };
    auto load_v = [&](int tile) {
        int in_page0;
        const float* vp = tile_page(tile, &in_page0) + size_t(kv.n_kv) * pt * HD + (size_t(g) * HD + lrow) * pt + in_page0 + 4 * lhalf;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int c = 0; c < 4; ++c) vr[d][c] = *(const float4*)(vp + size_t(32 * d) * pt + 8 * c);
    };
    auto mfma = [](float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); };

    const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    f32x16 o[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) o[d] = zero16;
    float m_run = -FLT_MAX, l_part = 0.f;   // finite start: a key hidden from a query then weighs exp(-inf - m) = 0
    int tile = tile_lo + wave;
    if (tile < tile_hi) load_k(tile);
    for (; tile < tile_hi; tile += 4) {
        load_v(tile);
        f32x16 s = zero16;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            s = mfma(kr[j].x, qr[j].x, s);
            s = mfma(kr[j].y, qr[j].y, s);
            s = mfma(kr[j].z, qr[j].z, s);
            s = mfma(kr[j].w, qr[j].w, s);
        }
        if (tile + 4 < tile_hi) load_k(tile + 4);
        const bool diagonal = (tile + 1) * FK > first_pos + 1;   // some key of the tile lies above some query's diagonal
        if (diagonal) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (tile * FK + 8 * (v >> 2) + 4 * lhalf + (v & 3) > my_pos) s[v] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const float corr = expf(m_run - m_new);
        m_run = m_new;
        l_part *= corr;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = expf(s[v] - m_new);
            l_part += s[v];
        }
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[d][v] *= corr;
        // A hidden key's probability is 0, but 0 * V is not where V holds an infinity or a NaN (a later token's, or
        // what a page held before): such a diagonal tile goes key by key, over the keys a query sees.
        if (diagonal) {
            float zero = 0.f;
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int c = 0; c < 4; ++c) zero += vr[d][c].x * 0.f + vr[d][c].y * 0.f + vr[d][c].z * 0.f + vr[d][c].w * 0.f;
            if (__builtin_amdgcn_ballot_w64(zero != 0.f) != 0) {
                int in_page0;
                const float* vp = tile_page(tile, &in_page0) + size_t(kv.n_kv) * pt * HD + (size_t(g) * HD + 4 * lhalf) * pt + in_page0;
                for (int key = 0; key < FK; ++key) {
                    float pk = 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (v == 4 * (key >> 3) + (key & 3)) pk = s[v];
                    pk = __shfl(pk, lrow + 32 * ((key >> 2) & 1), 64);
                    if (tile * FK + key <= my_pos) {
#pragma unroll
                        for (int d = 0; d < ND; ++d)
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                o[d][v] = fmaf(pk, vp[size_t(32 * d + 8 * (v >> 2) + (v & 3)) * pt + key], o[d][v]);
                    }
                }
                continue;
            }
        }
#pragma unroll
        for (int d = 0; d < ND; ++d) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                o[d] = mfma(vr[d][c].x, s[4 * c], o[d]);
                o[d] = mfma(vr[d][c].y, s[4 * c + 1], o[d]);
                o[d] = mfma(vr[d][c].z, s[4 * c + 2], o[d]);
                o[d] = mfma(vr[d][c].w, s[4 * c + 3], o[d]);
            }
        }
    }

    // merge the four waves: element (d, query) of the result is summed by one thread
    const float l_tot = l_part + __shfl_xor(l_part, 32, 64);
    if (lhalf == 0) { m_lds[wave][lrow] = m_run; l_lds[wave][lrow] = l_tot; }
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) o_lds[wave][32 * d + 8 * (v >> 2) + 4 * lhalf + (v & 3)][lrow] = o[d][v];
    __syncthreads();
    const int qi = threadIdx.x & 31, row = q0 + qi;
    float m = m_lds[0][qi], w[4], den = 0.f;
#pragma unroll
    for (int i = 1; i < 4; ++i) m = fmaxf(m, m_lds[i][qi]);
#pragma unroll
    for (int i = 0; i < 4; ++i) { w[i] = expf(m_lds[i][qi] - m); den += l_lds[i][qi] * w[i]; }
    if (row >= rows) return;
    const float inv = part ? 1.0f : 1.0f / den;
    float* dst = part ? part + ((size_t(split) * n_q + h) * rows + row) * (HD + 2) : out + (size_t(row) * n_q + h) * HD;
#pragma unroll
    for (int d = (threadIdx.x >> 5) * (HD / 8); d < ((threadIdx.x >> 5) + 1) * (HD / 8); ++d) {
        float x = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) x += o_lds[i][d][qi] * w[i];
        dst[d] = x * inv;
    }
    if (part && threadIdx.x < 32) { dst[HD] = m; dst[HD + 1] = den; }
}

// Merges the key ranges of a split attention launch: part[split][head][row] holds the unnormalised O (HD floats), the
// reference its exponentials were taken against and the row sum; a range in which the row saw no key has sum 0 and
// the lowest reference.
// One thread per two elements of a row: a stream over the parts, bound by the memory they come from.
template <typename T, int HD>
__global__ void __launch_bounds__(256)
attention_merge_kernel(const float* __restrict__ part, T* __restrict__ out, int n_q, int rows, int splits) {
    constexpr int TPR = HD / 2;                       // threads per (head, row)
    const int item = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, d = (threadIdx.x % TPR) * 2;
    if (item >= n_q * rows) return;
    const float* p = part + size_t(item) * (HD + 2);
    const size_t step = size_t(n_q) * rows * (HD + 2);
    float m = p[HD];
#pragma unroll 8
    for (int s = 1; s < splits; ++s) m = fmaxf(m, p[s * step + HD]);
    float den = 0.f, x0 = 0.f, x1 = 0.f;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) {
        const float2 ml = *(const float2*)(p + s * step + HD), o = *(const float2*)(p + s * step + d);
        const float w = expf(ml.x - m);
        den += ml.y * w;
        x0 += o.x * w;
        x1 += o.y * w;
    }
    const float inv = 1.0f / den;
    T* dst = out + (size_t(item % rows) * n_q + item / rows) * HD + d;
    dst[0] = T(x0 * inv);
    dst[1] = T(x1 * inv);
}

hipError_t launch_attention_merge(int dtype, int head_dim, const float* part, void* out, int n_q, int rows, int splits, hipStream_t st) {
    const int per = 256 / (head_dim / 2);
    const dim3 grid((n_q * rows + per - 1) / per), block(256);
    if (dtype == 0 && head_dim == 64) hipLaunchKernelGGL((attention_merge_kernel<float, 64>), grid, block, 0, st, part, (float*)out, n_q, rows, splits);
    else if (dtype == 0 && head_dim == 128) hipLaunchKernelGGL((attention_merge_kernel<float, 128>), grid, block, 0, st, part, (float*)out, n_q, rows, splits);
    else if (dtype == 1 && head_dim == 64) hipLaunchKernelGGL((attention_merge_kernel<bf16_t, 64>), grid, block, 0, st, part, (bf16_t*)out, n_q, rows, splits);
    else if (dtype == 1 && head_dim == 128) hipLaunchKernelGGL((attention_merge_kernel<bf16_t, 128>), grid, block, 0, st, part, (bf16_t*)out, n_q, rows, splits);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// 16-byte reads of q and of the pages.
bool attention_f32_supported(const void* q, const KvView& kv) {
    return (kv.head_dim == 64 || kv.head_dim == 128) && kv.page_tokens % 64 == 0 && ((uintptr_t(q) | uintptr_t(kv.pool)) & 15) == 0;
}

// Key ranges of ws.range_keys whatever the rows.  A row's sums are then over the same keys in the same order in every
// launch, however many rows and keys the launch has: a wave takes the same tiles of a range, a tile that a row does not
// see adds zeros to it, and so does a range.  (Prompts under one tile come here for the same reason, though a wave per
// row and head would be faster: 16 heads x 64, us: 8 rows of 8 keys 6.3 against 3.9, 24 of 24 6.1 against 5.3.)
// More rows than the ranges' parts fit (an op call beyond the context's chunk) take fewer, longer ranges.
hipError_t launch_attention_f32(const float* q, float* out, int n_q, int tok_begin, int rows, const KvView& kv, hipStream_t st,
                                const AttnWs& ws) {
    if (rows <= 0) return hipSuccess;
    float* part = ws.part;
    const int q_tiles = (rows + FQ - 1) / FQ, n_tiles = (tok_begin + rows - 1) / FK + 1;
    const size_t one = size_t(n_q) * rows * (kv.head_dim + 2) * sizeof(float);
    const size_t room = part ? std::max<size_t>(1, ws.bytes / one) : 1;
    int per = ws.range_keys > 0 ? std::max(1, ws.range_keys / FK) : n_tiles;
    if (size_t((n_tiles + per - 1) / per) > room) per = int((n_tiles + room - 1) / room);
    const int splits = (n_tiles + per - 1) / per;
    const dim3 grid(q_tiles, n_q, splits), block(256);
    float* p = splits > 1 ? part : nullptr;
    if (kv.head_dim == 64) hipLaunchKernelGGL(attention_f32_kernel<64>, grid, block, 0, st, q, out, p, n_q, tok_begin, rows, kv, per);
    else hipLaunchKernelGGL(attention_f32_kernel<128>, grid, block, 0, st, q, out, p, n_q, tok_begin, rows, kv, per);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    return launch_attention_merge(0, kv.head_dim, part, out, n_q, rows, splits, st);
}

}  // namespace cake
