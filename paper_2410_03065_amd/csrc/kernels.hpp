// Launchers of the device kernels.  Every launcher enqueues on `st` and returns the
// hipError_t of the launch.  Shapes are validated by the callers in cake_api.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cake {

typedef __bf16 bf16_t;

// Where a layer's K and V live: see the pool layout in cake.h.
struct KvView {
    void* pool;
    const int32_t* block_table;  // device
    int32_t page_tokens;
    int32_t n_physical_pages;
    int32_t n_kv;
    int32_t head_dim;
    int32_t layer;
    // elements per (layer, page): 2 * n_kv * page_tokens * head_dim
    __host__ __device__ size_t page_elems() const { return size_t(2) * n_kv * page_tokens * head_dim; }
};

enum GemmEpilogue { EPI_STORE_F32 = 0, EPI_RESIDUAL_F32 = 1, EPI_SWIGLU = 2 };

// ---- generic kernels (any supported shape) ----
// What a prefill begins with, in one launch: x = the rows' embeddings, cs = the rotary table of positions tok_begin ..; with a
// gain also h = the RMSNorm of x where d and the alignment allow it (prefill_begin_norms).  ids: device memory, or
// ids_by_value (at most TokenIds::MAX rows).
struct TokenIds { static constexpr int MAX = 512; int32_t v[MAX]; };   // 2 KB of a launch's 4 KB of arguments
struct PrefillBegin {
    const void* table; float* x; int rows, d, vocab;
    const float* gain; void* h; float eps;
    float* cs; int tok_begin, head_dim; float theta;
};
bool prefill_begin_norms(const PrefillBegin& b);
hipError_t launch_prefill_begin(int dtype, const PrefillBegin& b, const int32_t* ids, const TokenIds* ids_by_value, hipStream_t st);
hipError_t launch_rmsnorm(int dtype, const float* x, const float* gain, void* out, int rows, int d,
                          float eps, hipStream_t st);
hipError_t launch_rope_table(float* cs, int tok_begin, int rows, int head_dim, float theta,
                             hipStream_t st);
// n_parts > 1: qkv[n_parts][rows][...] is added up as it is read (16-byte aligned pointers only).
hipError_t launch_rope_kv_write(int dtype, const float* qkv, const float* cs, void* q, int n_q,
                                int tok_begin, int rows, const KvView& kv, hipStream_t st, int n_parts = 1);
// x += parts[0] + ... + parts[n_parts - 1] (each [rows][d], float32, 16-byte aligned), then the norm of the sum.
hipError_t launch_rmsnorm_parts(int dtype, float* x, const float* parts, int n_parts, const float* gain, void* out, int rows,
                                int d, float eps, hipStream_t st);
// x += (store: =) parts[0] + ... + parts[n_parts - 1], n floats each.
hipError_t launch_add_parts(float* x, const float* parts, int n_parts, size_t n, hipStream_t st, bool store = false);
hipError_t launch_gemm_generic(int dtype, int epi, const void* a, const void* w, const void* w2,
                               void* out, int M, int N, int K, hipStream_t st);
hipError_t launch_attention_generic(int dtype, const void* q, void* out, int n_q, int tok_begin,
                                    int rows, const KvView& kv, hipStream_t st);

// Where an attention launch may leave the parts of its key ranges: float32 workspace (part null: never divide the keys);
// launches sharing it must not overlap.  range_keys > 0: the keys are divided into ranges of that many whatever the
// number of rows, and a token's result does not depend on the step that it is computed in; 0: by a cost model.
struct AttnWs { float* part; size_t bytes; int range_keys; };

// ---- float32 on the matrix cores ----
bool attention_f32_supported(const void* q, const KvView& kv);
hipError_t launch_attention_f32(const float* q, float* out, int n_q, int tok_begin, int rows, const KvView& kv,
                                hipStream_t st, const AttnWs& ws);
// The RMSNorm in front of a product: its input is x / sqrt(mean(x^2) + eps) * gain (gain null: x as it is).
struct GemvNorm { const float* gain; float eps; };
// nm.gain: a is normed on the way (store and SwiGLU, where gemm_f32_norms_input says so for M rows or more; gain 16-byte
// aligned like a, w and w2).
bool gemm_f32_norms_input(int epi, int max_rows, int N, int K);
hipError_t launch_gemm_f32(int epi, const float* a, const float* w, const float* w2, float* out, int M, int N, int K,
                           hipStream_t st, const GemvNorm& nm = {nullptr, 0.f});
// Adds up the key ranges of a split attention launch: part[split][head][row][head_dim + 2] (O, reference of
// the exponentials, row sum) -> out[row][head][head_dim].
hipError_t launch_attention_merge(int dtype, int head_dim, const float* part, void* out, int n_q, int rows, int splits,
                                  hipStream_t st);

// ---- MFMA kernels (bf16) ----
bool gemm_mfma_supported(int epi, int M, int N, int K);
// Workspace of the split-K GEMMs: float32 parts of the tiles in flight, and one ticket counter per
// tile (zero between launches: the kernel puts it back).  Launches sharing it must not overlap.
struct GemmSplitWs {
    float* part;
    size_t part_bytes;
    unsigned* counters;
    int n_counters;
};
// cfg_override: -1 = choose the tile configuration from the shape; 0 and up = force one, unsplit (testing).
// ws: nullptr = never split K.  ksplit_override: 0 = by the cost model, 1 = never, 2/4/8 = that
// many K ranges wherever the shape and the workspace allow it.
hipError_t launch_gemm_mfma(int epi, const void* a, const void* w, const void* w2, void* out,
                            int M, int N, int K, hipStream_t st, int cfg_override = -1,
                            const GemmSplitWs* ws = nullptr, int ksplit_override = 0);
// What launch_gemm_mfma would launch: tile rows / columns and K ranges per tile.
void gemm_mfma_plan(int epi, int M, int N, int K, int cfg_override, const GemmSplitWs* ws, int ksplit_override,
                    int* bm, int* bn, int* ksplit);
// Does launch_gemm_mfma add up in the same order for every M from 1 to max_rows?
bool gemm_order_fixed(int epi, int max_rows, int N, int K, const GemmSplitWs* ws);
// out[ks][M][N] float32: one output per K range (K a multiple of 64 ks), for a consumer that adds them up; M <= 192, N a
// multiple of 128.
hipError_t launch_gemm_rows_parts(const void* a, const void* w, float* part, int M, int N, int K, int ks, hipStream_t st);
// How to leave a product (epi: store or residual) to its consumer: ksplit 0: not, launch_gemm_mfma is faster; else K in
// that many ranges on the kernel for few rows, on the persistent one or on the 128 x 128 or 128 x 192 tiles.  fused: the
// consumer reads the result anyway (an RMSNorm, the rotary step); otherwise a pass of its own adds the ranges up.
enum GemmPartsKind { GEMM_PARTS_ROWS = 0, GEMM_PARTS_P256 = 1, GEMM_PARTS_128 = 2, GEMM_PARTS_192 = 3 };
struct GemmPartsPlan { int ksplit; GemmPartsKind kind; };
GemmPartsPlan gemm_parts_plan(int epi, int M, int N, int K, const GemmSplitWs* ws, bool fused, bool rows_only = false);
hipError_t launch_gemm_parts(const GemmPartsPlan& plan, const void* a, const void* w, float* part, int M, int N, int K, hipStream_t st);
// MFMA-only yardstick kernel: out holds workgroups * 8 floats; see kernels_gemm.hip.
hipError_t launch_mfma_rate(float* out, int workgroups, int iters, hipStream_t st);
bool attention_mfma_supported(int head_dim, int page_tokens);
// variant: 0 = eight-wave kernel, 128, 64 or 32 queries per workgroup and the key ranges by a cost model; 1 = four-wave
// kernel; 2 / 3 = eight-wave kernel with 128 / 64 queries per workgroup (testing).
hipError_t launch_attention_mfma(const void* q, void* out, int n_q, int tok_begin, int rows,
                                 const KvView& kv, hipStream_t st, int variant, const AttnWs& ws);

// bf16, head_dim 64
bool attention_hd64_supported(const void* q, const void* out, int n_keys, const KvView& kv, const AttnWs& ws);
hipError_t launch_attention_hd64(const void* q, void* out, int n_q, int tok_begin, int rows, const KvView& kv,
                                 hipStream_t st, const AttnWs& ws);

bool decode_attention_mfma_supported(int dtype, int head_dim, int page_tokens, int r);
hipError_t launch_decode_attention_mfma(const float* q, float* part, int n_q, int n_keys, int tiles_per_split,
                                        int n_splits, const KvView& kv, hipStream_t st);

// ---- quantised stored KV (bits = 8 or 4): a page image (all layers) <-> the layer pages of a physical page ----
// Images side by side in device memory and the physical page of each.
struct PageRun { static constexpr int MAX = 32; int n; int32_t phys[MAX]; };
hipError_t launch_dequant_pages(int dtype, const void* images, size_t image_bytes, const KvView& kv, const PageRun& run, int n_layers,
                                int bits, hipStream_t st);
// raw images -> pages and pages -> raw images (images and pool 16-byte aligned, layer pages of whole 16 KB)
bool move_pages_supported(const void* images, size_t layer_bytes, const KvView& kv);
hipError_t launch_import_pages(const void* images, size_t image_bytes, const KvView& kv, const PageRun& run, size_t layer_bytes,
                               int n_layers, hipStream_t st);
hipError_t launch_export_pages(void* images, size_t image_bytes, const KvView& kv, const PageRun& run, size_t layer_bytes, int n_layers,
                               hipStream_t st);
// logical pages [first_page, first_page + n_pages) -> images, image_bytes apart
hipError_t launch_quant_pages(int dtype, void* images, size_t image_bytes, const KvView& kv, const int32_t* block_table_host,
                              int first_page, int n_pages, int n_layers, int bits, hipStream_t st);

// ---- first-token step (one row of activations: matrix-vector products, one-token attention) ----
// h = x (gain null: mode 1 only) or its RMSNorm (gain, eps; modes 0, 2, 3): out[n] (mode 0: =, 1: +=) sum_k h[k] w[n][k];
// mode 2: out[n] = silu(h.w[n]) * (h.w2[n]); mode 3: mode 0 with adjacent rows of a head rotated by cs[head_dim / 2]
// (cos, sin).  x, out float32.  host (mode 0): null, or pinned memory, 16-byte aligned, for a copy of the result.
hipError_t launch_gemv(int dtype, int mode, const GemvNorm& nm, const float* x, const void* w, const void* w2, float* out,
                       int N, int K, hipStream_t st, const double* cs = nullptr, int head_dim = 0, float* host = nullptr);
// x = row `id` of the embedding table; cs[head_dim / 2] = (cos, sin) of the rotary pairs at position pos.
hipError_t launch_token_begin(int dtype, const void* table, int id, float* x, int d, double* cs, int head_dim, int pos,
                              float theta, hipStream_t st);
size_t decode_attention_workspace_bytes(int n_q, int head_dim);
// generic_only: keep to the vector-ALU kernel (testing)
hipError_t launch_decode_attention(int dtype, const float* q, float* out, float* part, int n_q,
                                   int n_keys, const KvView& kv, hipStream_t st, bool generic_only = false);
// Device memory of launch_argmax; counter is zero between launches.
constexpr int ARGMAX_BLOCKS = 128;
struct ArgmaxWs { unsigned long long best[ARGMAX_BLOCKS]; unsigned counter; };
hipError_t launch_argmax(const float* v, int n, ArgmaxWs* ws, int32_t* result, hipStream_t st);

}  // namespace cake
