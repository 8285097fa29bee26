// bf16 MFMA attention for gfx950: chunk-vs-prefix causal attention over paged KV
// (Sec. 3 "Attention and KV cache", "Chunk Prefill": a chunk's queries attend to every cached
// key before and inside it).  Built with MFMA results kept in ordinary VGPRs, because the
// softmax reads every score on the vector ALUs.
//
// MFMA shape used throughout: v_mfma_f32_32x32x16_bf16.  For D[32x32] += A[32x16] * B[16x32]
// lane l supplies A[l%32][8*(l/32) .. +7] and B[8*(l/32) .. +7][l%32], and holds
// D[8*(v/4) + 4*(l/32) + v%4][l%32] in accumulator register v (0..15).
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "kernels.hpp"

namespace cake {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
// v_mfma_f32_16x16x32_bf16, D[16x16] += A[16x32] * B[32x16]: lane l supplies A[l%16][8*(l/16) .. +7] and
// B[8*(l/16) .. +7][l%16], and holds D[4*(l/16) + v][l%16] in accumulator register v (0..3).
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

#define CAKE_GLOBAL_AS __attribute__((address_space(1)))
#define CAKE_LDS_AS __attribute__((address_space(3)))

// =====================================================================================
// Attention: out[row][h*128 + :] = softmax_s(q_row . k_s / sqrt(128)) v_s over keys s <= tok_begin+row.
//
// Workgroup = 4 waves x 32 queries of one query head; keys are visited in tiles of 64 held in a
// ring of LDS stages filled by direct global->LDS loads from the K pages ([key][hd]) and the
// transposed V pages ([hd][key]).
//
// The score tile is formed transposed, S^T[key][query] = K[key][:] . Q[query][:], so a lane
// holds 32 keys of ONE query: the online-softmax statistics are per-lane scalars (one exchange
// with lane^32 for the max) and the probabilities are already laid out as the B operand
// P^T[key][query] of the second product O^T[hd][query] += V^T[hd][key] P^T[key][query].
// The K rows fed to the first MFMA are permuted within each group of 16 (rows 4-7 and 8-11
// swapped).  With that, accumulator registers v = 8*(j&1) .. +7 of key tile j>>1 hold, in the
// low / high half-wave, keys 16j + 0..7 / 16j + 8..15 -- exactly the 8 consecutive k-slots each
// half-wave must supply for 16-key step j, so P needs no shuffle and the V^T operand is one
// aligned 16-byte read.
//
// Pipeline per key tile: wait for the next tile's loads, barrier, refill the stage freed one
// tile ago, then issue the NEXT tile's score MFMAs and, in their shadow, run this tile's
// softmax on the vector ALUs, then this tile's P V MFMAs.  The output accumulators are rescaled
// only when some lane's running maximum moved (wave-uniform test).
// =====================================================================================
constexpr int AQ = 128;   // queries per workgroup
constexpr int AK = 64;    // keys per tile
constexpr int AHD = 128;  // head dim
constexpr int A_STAGES = 4;
constexpr int A_KBYTES = AK * AHD * 2, A_STAGE = 2 * A_KBYTES;
constexpr int A_PER_TILE = 8;  // wave-loads per wave per tile (4 K + 4 V)

__device__ __forceinline__ int sigma16(int x) { return (x & 3) | ((x & 4) << 1) | ((x & 8) >> 1); }

__global__ void __launch_bounds__(256)
attention_mfma_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ out, int n_q, int tok_begin, int rows,
                      KvView kv, int q_tiles) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int G = kv.n_kv, r = n_q / G;
    // Workgroups that share a KV head go to the same XCD (block b runs on XCD b % 8).
    int g, rest;
    if ((G & 7) == 0) {
        const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3, gpx = G >> 3;
        g = xcd + 8 * (idx % gpx);
        rest = idx / gpx;
    } else {
        g = blockIdx.x % G;
        rest = blockIdx.x / G;
    }
    const int h = g * r + rest % r;
    const int q0 = (rest / r) * AQ;
    const int pt = kv.page_tokens;

    const int my_row = min(q0 + wave * 32 + lrow, rows - 1);
    const int my_pos = tok_begin + my_row;
    const int wave_first_pos = tok_begin + min(q0 + wave * 32, rows - 1);
    const int wg_last_pos = tok_begin + min(q0 + AQ, rows) - 1;
    const int n_tiles = wg_last_pos / AK + 1;

    // Q^T operand: lane supplies q[my_row][16*ks + 8*lhalf .. +7]
    bf16x8 qreg[AHD / 16];
    {
        const bf16_t* qp = q + (size_t(h) * rows + my_row) * AHD + 8 * lhalf;
#pragma unroll
        for (int ks = 0; ks < AHD / 16; ++ks) qreg[ks] = *(const bf16x8*)(qp + 16 * ks);
    }

    // global->LDS sources.  K wave-load j covers rows 4j..4j+3 (256 B each, chunk c stored at c ^ (row & 15));
    // V^T wave-load j covers rows 8j..8j+7 (128 B each, chunk c stored at c ^ ((row >> 1) & 7)).
    unsigned koffg[4], voffg[4];   // byte offsets from the tile's K / V^T base
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int j = wave + 4 * i;
        int krow = 4 * j + (lane >> 4), kpos = lane & 15;
        koffg[i] = unsigned(krow * AHD + ((kpos ^ (krow & 15)) << 3)) * 2u;
        int vrow = 8 * j + (lane >> 3), vpos = lane & 7;
        voffg[i] = unsigned(vrow * pt + ((vpos ^ ((vrow >> 1) & 7)) << 3)) * 2u;
    }
    // Byte offset of every logical page this workgroup needs (this layer, this KV head's K block)
    // is put into LDS once: a global load in the issue path would share the vmcnt counter with
    // the tile loads and drain the whole ring.  The entry for the tile issued next is read one
    // tile ahead, so its LDS latency is off the issue path too.
    const int last_page = wg_last_pos / pt;
    unsigned long long* pg_lds = (unsigned long long*)(lds + A_STAGES * A_STAGE);
    {
        const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;
        const size_t page_bytes = kv.page_elems() * 2, k_head = size_t(g) * pt * AHD * 2;
        for (int i = tid; i <= last_page; i += 256) pg_lds[i] = (layer_base + kv.block_table[i]) * page_bytes + k_head;
    }
    __syncthreads();
    // from a page's K block of head g to its V^T block of head g
    const unsigned long long k_to_v = (size_t(G - g) * pt * AHD + size_t(g) * AHD * pt) * 2;
    unsigned long long pg_next = pg_lds[0];
    auto issue = [&](int stage, int kt) {
        const int key0 = kt * AK;
        const int lpage = key0 / pt;
        const unsigned in_page0 = unsigned(key0 - lpage * pt);
        // readfirstlane returns a signed int: go through unsigned, or offsets with bit 31 set sign-extend
        const unsigned long long lo = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(pg_next));
        const unsigned long long hi = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(pg_next >> 32));
        const char* kp = (const char*)kv.pool + ((hi << 32) | lo) + size_t(in_page0) * (AHD * 2);
        const char* vp = (const char*)kv.pool + ((hi << 32) | lo) + k_to_v + size_t(in_page0) * 2;
        pg_next = pg_lds[min((key0 + AK) / pt, last_page)];
        unsigned char* sa = lds + stage * A_STAGE;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(kp + size_t(koffg[i])),
                                             (CAKE_LDS_AS void*)(sa + (wave + 4 * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(vp + size_t(voffg[i])),
                                             (CAKE_LDS_AS void*)(sa + A_KBYTES + (wave + 4 * i) * 1024), 16, 0, 0);
    };

    // operand read offsets (per lane, in bytes from the start of a stage)
    const int sk = sigma16(lrow & 15);
    const int krow_base = (16 * (lrow >> 4) + sk) * (AHD * 2);   // + 32*t rows
    int kaddr[AHD / 16];
#pragma unroll
    for (int ks = 0; ks < AHD / 16; ++ks) kaddr[ks] = krow_base + (((2 * ks + lhalf) ^ sk) << 4);
    const int sv = (lrow >> 1) & 7;
    int vaddr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) vaddr[j] = A_KBYTES + lrow * (AK * 2) + (((2 * j + lhalf) ^ sv) << 4);

    f32x16 o[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[t][v] = 0.f;
    float m_run = -INFINITY, l_part = 0.f;
    const float sl2 = 0.08838834764831845f * 1.4426950408889634f;  // 1/sqrt(128) * log2(e)
    const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    // Running maximum of a score tile, in pieces so that it can be spread over MFMA groups:
    // (masking of the diagonal tiles), max over the lane's 32 scores, exchange with the partner
    // half-wave, correction factor for the old accumulators.
    float mx_cur = 0.f, corr_cur = 0.f;
    bool moved_cur = false;
    auto mask_tile = [&](f32x16* s, int kt) {
        const int key0 = kt * AK;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int key = key0 + 32 * t + (v & 7) + 8 * lhalf + 16 * (v >> 3);
                if (key > my_pos) s[t][v] = -INFINITY;
            }
    };
    auto part_max = [&](const f32x16* s, int part, float acc) {   // elements [8*part, 8*part+8) of the 32
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fmaxf(acc, s[part >> 1][8 * (part & 1) + i]);
        return acc;
    };
    // The exponentials use a reference value m_run per query that follows the running maximum
    // lazily: it is moved (and O, l rescaled) only when some lane's maximum has outgrown it by more
    // than 2^RESCALE_LOG2, so probabilities may reach 2^RESCALE_LOG2 instead of 1 -- harmless in
    // bf16 / fp32, and softmax is invariant to the reference.  Without this the rescale of the 64
    // accumulator registers would run on roughly every other tile.
    constexpr float RESCALE_LOG2 = 6.0f;
    auto finish_max = [&](float raw) {
        float mx = raw * sl2;
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));   // key 0 is visible to every query, so mx is finite
        moved_cur = mx > m_run + RESCALE_LOG2;    // -inf + 6 = -inf: the first tile always moves
        if (__builtin_amdgcn_ballot_w64(moved_cur) != 0) {
            mx = fmaxf(mx, m_run);
            corr_cur = __builtin_amdgcn_exp2f(m_run - mx);
            m_run = mx;
            moved_cur = true;
        } else {
            corr_cur = 1.0f;
        }
        mx_cur = m_run;
    };

    // One key tile = two MFMA phases of four groups each (4 LDS reads feeding 4 MFMAs per group);
    // a group's operands are read while the previous group's MFMAs run, and the vector-ALU work
    // is dealt out group by group so that it executes in the MFMAs' shadow:
    //   phase 1: S^T of tile kt+1  ||  exponentials + bf16 packing of tile kt (8 per group)
    //   phase 2: O^T += V^T P^T of tile kt  ||  (mask and) running max of tile kt+1
    // then the (rare) rescale of O by the correction of tile kt+1.
    auto step = [&](int kt, f32x16* s_cur, f32x16* s_nxt, auto masked_tag) {
        constexpr bool masked_next = decltype(masked_tag)::value;
        if (kt + A_STAGES - 2 < n_tiles) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((A_STAGES - 3) * A_PER_TILE));
        else asm volatile("s_waitcnt vmcnt(0)");
        __builtin_amdgcn_s_barrier();
        if (kt + A_STAGES - 1 < n_tiles) issue((kt + A_STAGES - 1) % A_STAGES, kt + A_STAGES - 1);

        const float mx = mx_cur;
        // past the last tile the score MFMAs read a stale stage; that result is never used
        const unsigned char* stk = lds + ((kt + 1) % A_STAGES) * A_STAGE;
        const unsigned char* stv = lds + (kt % A_STAGES) * A_STAGE;
        bf16x8 opa[4], opb[4], p[4];
        auto read_k = [&](bf16x8* dst, int grp) {   // ks = 2*grp, 2*grp+1 ; t = 0, 1
#pragma unroll
            for (int i = 0; i < 4; ++i)
                dst[i] = *(const bf16x8*)(stk + (i & 1) * 32 * (AHD * 2) + kaddr[2 * grp + (i >> 1)]);
        };
        auto read_v = [&](bf16x8* dst, int j) {      // t = 0..3
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i] = *(const bf16x8*)(stv + i * 32 * (AK * 2) + vaddr[j]);
        };
        auto mma_k = [&](const bf16x8* src, int grp) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ks = 2 * grp + (i >> 1), t = i & 1;
                s_nxt[t] = mfma32(src[i], qreg[ks], ks == 0 ? zero16 : s_nxt[t]);
            }
        };
        auto expo = [&](int grp) {                   // p[grp]: 8 probabilities of tile kt
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[grp >> 1][8 * (grp & 1) + i], sl2, -mx));
                l_part += e;
                p[grp][i] = bf16_t(e);
            }
        };
        // ---- phase 1
        read_k(opa, 0);
        __builtin_amdgcn_sched_barrier(0);
        read_k(opb, 1); mma_k(opa, 0); expo(0);
        __builtin_amdgcn_sched_barrier(0);
        read_k(opa, 2); mma_k(opb, 1); expo(1);
        __builtin_amdgcn_sched_barrier(0);
        read_k(opb, 3); mma_k(opa, 2); expo(2);
        __builtin_amdgcn_sched_barrier(0);
        read_v(opa, 0); mma_k(opb, 3); expo(3);
        __builtin_amdgcn_sched_barrier(0);
        // ---- phase 2
        float raw;
        if (masked_next) mask_tile(s_nxt, kt + 1);
        read_v(opb, 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = mfma32(opa[t], p[0], o[t]);
        raw = part_max(s_nxt, 0, s_nxt[0][0]);
        raw = part_max(s_nxt, 1, raw);
        __builtin_amdgcn_sched_barrier(0);
        read_v(opa, 2);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = mfma32(opb[t], p[1], o[t]);
        raw = part_max(s_nxt, 2, raw);
        raw = part_max(s_nxt, 3, raw);
        __builtin_amdgcn_sched_barrier(0);
        read_v(opb, 3);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = mfma32(opa[t], p[2], o[t]);
        finish_max(raw);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = mfma32(opb[t], p[3], o[t]);
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_amdgcn_ballot_w64(moved_cur) != 0) {
            l_part *= corr_cur;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[t][v] *= corr_cur;
        }
    };

    // prologue
#pragma unroll
    for (int st = 0; st < A_STAGES - 1; ++st)
        if (st < n_tiles) issue(st, st);
    if (n_tiles >= A_STAGES - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((A_STAGES - 2) * A_PER_TILE));
    else asm volatile("s_waitcnt vmcnt(0)");
    __builtin_amdgcn_s_barrier();
    f32x16 s_a[2], s_b[2];
    {
        const unsigned char* stk = lds;
#pragma unroll
        for (int ks = 0; ks < AHD / 16; ++ks)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf16x8 a = *(const bf16x8*)(stk + t * 32 * (AHD * 2) + kaddr[ks]);
                s_a[t] = mfma32(a, qreg[ks], ks == 0 ? zero16 : s_a[t]);
            }
    }
    // tiles below first_masked hold only keys every query of this wave may see
    const int first_masked = (wave_first_pos + 1) / AK;   // first tile with key0 + AK - 1 > wave_first_pos
    if (first_masked <= 0) mask_tile(s_a, 0);
    {
        float raw = s_a[0][0];
#pragma unroll
        for (int part = 0; part < 4; ++part) raw = part_max(s_a, part, raw);
        finish_max(raw);
    }
    // two tiles per trip so the score buffers alternate without copies
    int kt = 0;
    for (; kt + 2 < first_masked && kt + 1 < n_tiles; kt += 2) {
        step(kt, s_a, s_b, std::false_type{});
        step(kt + 1, s_b, s_a, std::false_type{});
    }
    for (; kt < n_tiles; kt += 2) {   // the few tiles on and past the diagonal
        step(kt, s_a, s_b, std::true_type{});
        if (kt + 1 < n_tiles) step(kt + 1, s_b, s_a, std::true_type{});
    }
    // finish: total row sum = this lane's partial + the partner half-wave's
    const float l_tot = l_part + __shfl_xor(l_part, 32, 64);
    const float inv = 1.0f / l_tot;
    const int row = q0 + wave * 32 + lrow;
    if (row < rows) {
        bf16_t* op = out + size_t(row) * n_q * AHD + h * AHD;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = bf16_t(o[t][4 * v4 + e] * inv);
                *(bf16x4*)(op + t * 32 + 8 * v4 + 4 * lhalf) = w;
            }
    }
}

// =====================================================================================
// Eight-wave variant: two waves per SIMD, so that one wave's softmax (vector ALU) runs while the
// other's MFMAs occupy the matrix pipe -- a single wave cannot overlap the two (an MFMA holds its
// own wave's issue for most of its duration).  A chunk of 1024 queries x 32 heads only offers
// 4 waves of 32 queries per CU, so the second wave group takes the other half of the KEYS: waves
// 0-3 visit key tiles 0, 2, 4, ..., waves 4-7 tiles 1, 3, 5, ... with private softmax state, and
// the two partial results are merged through LDS at the end (softmax over a union of key sets:
// rescale both to the common reference and add).
//
// The products are 16x16x32 MFMAs (two columns of 16 queries per wave): per FLOP they move a quarter of the accumulators
// of 32x32x16 ones, and this kernel runs at the power limit (1024 rows at 31744 keys, 32 heads on 8: 4.5 % less time).
// The two halves run half a step apart, a barrier between the phases of a step keeping them there: a SIMD then holds one
// wave whose scores are being formed beside the exponentials (vector work above the MFMAs') and one that only adds P V up,
// at lower priority.  Together they overlap, where two waves in the same phase first compete for the vector unit and then
// leave it idle (6 % more; with 32x32x16 MFMAs it gained nothing).  The maximum that is only compared with the reference
// is taken on integers (2 %).  Launches of few pairs are all fixed cost, so the last step forms no scores, row sums cross
// lanes without LDS and both columns' parts are read before either is stored (the first with 32x32x16 MFMAs, then these
// without and with that, us: 64 rows of 32 heads on 8 at 0 6.9, 7.3, 6.8, at 500 11.7, 12.4, 11.6; 1024 at 0 21.4, 21.2,
// 20.4).  494 -> 427 us for the launch above, 1.27 PFLOP/s; 1024 rows at 16000 250 -> 221; 509 rows of
// 32 KV heads at 7003 78 -> 70.  What bounds it now: one LDS read per two MFMAs, 3.5 vector instructions per two, one of
// them an exponential; a loop of just these on two waves per SIMD sustains 1.34 PFLOP/s.
//
// LDS: K ring of 2 x (two 16 KB tiles) and V^T ring of 2 x (two 16 KB tiles).  K of a tile pair
// is consumed one iteration before its V^T, so per iteration the V^T of pair i+1 and the K of
// pair i+2 are fetched, each into the buffer its group finished with in the previous iteration.
// Masked scores are -inf, the initial reference is a large FINITE negative: a row whose keys in
// one half are all above the diagonal then keeps exp2(-inf - finite) = 0 everywhere (no inf - inf),
// ends with O = 0, l = 0 and the initial reference, and the merge weighs that half by exactly 0.
// =====================================================================================
constexpr float A8_NEG = -1.0e30f;
constexpr int A8_RING = 2 * A_KBYTES;        // one ring slot: group A's tile then group B's tile
constexpr int A8_VBASE = 2 * A8_RING;        // V^T ring after the K ring
constexpr int A8_TABLE = 4 * A8_RING;        // page offsets after both rings

// side_by_side: the r query heads that share a KV head are laid side by side, query number x of KV head g is row x / r
// of head g r + x % r, so a workgroup's queries fill up across heads (137 rows of four heads: five tiles of 128 instead
// of eight).  Where that saves no tile a workgroup keeps to one head (1024 rows at 31744: 1 % less time).
// QW = query waves per half: 128, 64 or 32 queries per workgroup.
//
// Launches with too few query tiles for the chip divide the keys as well: blockIdx.y takes `pairs_per_split` pairs of
// key tiles and leaves its unnormalised result in `part` for attention_merge_kernel (SPLIT, an instantiation of its
// own: the unsplit loop's code stays as it is).
template <int QW, bool SPLIT>
__global__ void __launch_bounds__(128 * QW)
attention_mfma8_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ out, float* __restrict__ part, int n_q, int tok_begin,
                       int rows, KvView kv, int pairs_per_split, bool side_by_side) {
    constexpr int AQW = 32 * QW;        // queries per workgroup
    constexpr int PER = 16 / QW;        // wave-loads per wave per K (or V^T) tile
    constexpr int KN = QW == 4 ? 2 : 4, KE = QW == 1 ? 2 : 1;   // the K swizzle term of a wave's loads has KN values in turn, KE loads each
    constexpr int VP = QW >= 2 ? 1 : 2;                         // period after which the V^T term repeats
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave8 % QW, grp = wave8 / QW;
    const int l16 = lane & 15, lq = lane >> 4;
    const int G = kv.n_kv, r = n_q / G;
    int g, q0;
    if ((G & 7) == 0) {
        const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3, gpx = G >> 3;
        g = xcd + 8 * (idx % gpx);
        q0 = idx / gpx * AQW;
    } else {
        g = blockIdx.x % G;
        q0 = blockIdx.x / G * AQW;
    }
    const int pt = kv.page_tokens;

    // number of queries laid out, heads each stands across, first head; one head: q0 / AQW = q tile * r + head
    const int rr = side_by_side ? r : 1, n_queries = rows * rr;
    const int head0 = side_by_side ? g * r : g * r + (q0 / AQW) % r;
    if (!side_by_side) q0 = (q0 / AQW) / r * AQW;
    // this lane's two queries, one in each tile of 16 columns
    int my_row[2], h[2], my_pos[2];
    bool is_query[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int x = q0 + wave * 32 + 16 * c + l16, my_query = min(x, n_queries - 1);
        is_query[c] = x < n_queries;
        my_row[c] = rr == 1 ? my_query : my_query / rr;
        h[c] = head0 + (my_query - my_row[c] * rr);
        my_pos[c] = tok_begin + my_row[c];
    }
    const int wave_first_pos = tok_begin + min(q0 + wave * 32, n_queries - 1) / rr;
    const int wg_last_pos = tok_begin + (min(q0 + AQW, n_queries) - 1) / rr;
    const int n_tiles = wg_last_pos / AK + 1;
    const int pair_lo = SPLIT ? blockIdx.y * pairs_per_split : 0;
    const int n_pairs = SPLIT ? min(pair_lo + pairs_per_split, (n_tiles + 1) >> 1) : (n_tiles + 1) >> 1;
    auto my_part = [&](int c) { return part + ((size_t(blockIdx.y) * n_q + h[c]) * rows + my_row[c]) * (AHD + 2); };
    if (SPLIT && pair_lo >= n_pairs) {   // a range wholly above this workgroup's diagonal
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (grp == 0 && is_query[c]) {
                float* p = my_part(c);
                for (int d = lq * (AHD / 4); d < (lq + 1) * (AHD / 4); d += 2) *(float2*)(p + d) = make_float2(0.f, 0.f);
                if (lq == 0) *(float2*)(p + AHD) = make_float2(-FLT_MAX, 0.f);
            }
        return;
    }
    const int first_masked = (wave_first_pos + 1) / AK;   // first tile with a key some query of this wave must not see

    bf16x8 qreg[2][AHD / 32];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const bf16_t* qp = q + (size_t(h[c]) * rows + my_row[c]) * AHD + 8 * lq;
#pragma unroll
        for (int ks = 0; ks < AHD / 32; ++ks) qreg[c][ks] = *(const bf16x8*)(qp + 32 * ks);
    }
    {   // softmax scale and log2(e) go into Q once, so a score leaves the MFMA in the exponent's units
        const float sl2q = 0.08838834764831845f * 1.4426950408889634f;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int ks = 0; ks < AHD / 32; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) qreg[c][ks][e] = bf16_t(float(qreg[c][ks][e]) * sl2q);
    }
    // lane offsets of this wave's K / V^T wave-loads of a tile: load i covers 1 KB = key rows
    // 4j .. 4j+3 (V^T: head-dim rows 8j .. 8j+7) with j = wave + QW*i.  Chunk c of key row x is stored at
    // c ^ kswz(x), so that the sixteen rows a quarter-wave reads (x = 8 q + v, plus a constant) lie in sixteen
    // different chunks; of V^T row x at c ^ ((x >> 1) & 7).  Loads with the
    // same swizzle term are a wave-uniform distance apart.
    auto kswz = [](int x) { return (x & 3) | (x >> 1 & 12); };
    unsigned koffp[KN], voffp[VP];
#pragma unroll
    for (int i = 0; i < KN; ++i) {
        int krow = 4 * (wave + QW * KE * i) + (lane >> 4), kpos = lane & 15;
        koffp[i] = unsigned(krow * AHD + ((kpos ^ kswz(krow)) << 3)) * 2u;
    }
#pragma unroll
    for (int i = 0; i < VP; ++i) {
        int vrow = 8 * (wave + QW * i) + (lane >> 3), vpos = lane & 7;
        voffp[i] = unsigned(vrow * pt + ((vpos ^ ((vrow >> 1) & 7)) << 3)) * 2u;
    }
    const int last_page = wg_last_pos / pt;
    unsigned long long* pg_lds = (unsigned long long*)(lds + A8_TABLE);
    {
        const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;
        const size_t page_bytes = kv.page_elems() * 2, k_head = size_t(g) * pt * AHD * 2;
        for (int i = tid; i <= last_page; i += 128 * QW) pg_lds[i] = (layer_base + kv.block_table[i]) * page_bytes + k_head;
    }
    __syncthreads();
    const unsigned long long k_to_v = (size_t(G - g) * pt * AHD + size_t(g) * AHD * pt) * 2;
    // this wave group's tile of a pair; a tile past the end re-reads the last real one (it is fully masked)
    auto tile_of = [&](int pair) { return min(2 * pair + grp, n_tiles - 1); };
    auto page_base = [&](int tile, unsigned* in_page0) {
        const int key0 = tile * AK, lpage = key0 / pt;
        *in_page0 = unsigned(key0 - lpage * pt);
        const unsigned long long off = pg_lds[lpage];
        const unsigned long long lo = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(off));
        const unsigned long long hi = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(off >> 32));
        return (const char*)kv.pool + ((hi << 32) | lo);
    };
    auto issue_k = [&](int pair) {
        unsigned in_page0;
        const char* kp = page_base(tile_of(pair), &in_page0) + size_t(in_page0) * (AHD * 2);
        unsigned char* sa = lds + (pair & 1) * A8_RING + grp * A_KBYTES;
#pragma unroll
        for (int i = 0; i < PER; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(kp + size_t(i - i / KE % KN * KE) * (4 * QW * AHD * 2) + koffp[i / KE % KN]),
                                             (CAKE_LDS_AS void*)(sa + (wave + QW * i) * 1024), 16, 0, 0);
    };
    auto issue_v = [&](int pair) {
        unsigned in_page0;
        const char* vp = page_base(tile_of(pair), &in_page0) + k_to_v + size_t(in_page0) * 2;
        unsigned char* sa = lds + A8_VBASE + (pair & 1) * A8_RING + grp * A_KBYTES;
#pragma unroll
        for (int i = 0; i < PER; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(vp + size_t(i / VP) * (8 * QW * VP) * pt * 2 + voffp[i % VP]),
                                             (CAKE_LDS_AS void*)(sa + (wave + QW * i) * 1024), 16, 0, 0);
    };

    // Score tiles t = 2 j and 2 j + 1 (16 keys each) hold the keys 32 j + 8 q + v and 32 j + 8 q + 4 + v at their rows
    // 4 q + v, so that a lane's eight scores of the two are the eight consecutive keys 32 j + 8 lq .. + 7, which is what it
    // has to supply to the second product's k-step j.
    const int krow0 = 8 * (l16 >> 2) + (l16 & 3), sk = kswz(krow0);   // + 32 j + 4 (t & 1) changes no term of kswz
    int kaddr[AHD / 32], vaddr[2];
#pragma unroll
    for (int ks = 0; ks < AHD / 32; ++ks) kaddr[ks] = grp * A_KBYTES + krow0 * (AHD * 2) + (((4 * ks + lq) ^ sk) << 4);
    const int sv = (l16 >> 1) & 7;
#pragma unroll
    for (int j = 0; j < 2; ++j) vaddr[j] = A8_VBASE + grp * A_KBYTES + l16 * (AK * 2) + (((4 * j + lq) ^ sv) << 4);

    const f32x4 zero4 = {0, 0, 0, 0};
    f32x4 o[8][2];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) o[t][c] = zero4;
    // The running reference m_run of a query (log2 units) is SUBTRACTED INSIDE THE MFMA: the score
    // accumulators start from negm = -m_run instead of zero, so a finished score is already
    // s - m_run and the exponential needs no multiply-add of its own.  When the reference moves
    // (rarely, see RESCALE_LOG2) the scores formed against the old one are shifted by hand.
    float m_run[2] = {0.f, 0.f}, l_part[2] = {0.f, 0.f};
    f32x4 negm[2] = {zero4, zero4};
    float raw_cur = 0.f;
    constexpr float RESCALE_LOG2 = 6.0f;
    auto mask_tile = [&](f32x4 (*s)[2], int tile, const int* last_visible) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int limit = last_visible[c] - (tile * AK + 8 * lq);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (32 * (t >> 1) + 4 * (t & 1) + v > limit) s[t][c][v] = -INFINITY;
        }
    };
    auto part_max = [&](f32x4 (*s)[2], int c, int t, float acc) {   // tiles t and t + 1
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaxf(acc, s[t + (e >> 2)][c][e & 3]);
        return acc;
    };
    // raw[c]: this lane's largest score of query c -> the query's, of column tile 0 in lanes 0 .. 31 and of 1 in the others
    auto row_max = [&](const float* raw) {
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(raw[0]), __float_as_uint(raw[1]), false, false);
        const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
        return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    };
    // The same for the test against RESCALE_LOG2, on the bit patterns as integers: of values of which one is positive the
    // largest is found (where none is, some negative one), without the canonicalising that fmaxf costs.
    auto part_top = [&](f32x4 (*s)[2], int c, int t, int acc) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = max(acc, __float_as_int(s[t + (e >> 2)][c][e & 3]));
        return acc;
    };
    auto row_top = [&](const int* raw) {
        const auto a = __builtin_amdgcn_permlane32_swap(raw[0], raw[1], false, false);
        const int y = max(int(a[0]), int(a[1]));
        const auto b = __builtin_amdgcn_permlane16_swap(y, y, false, false);
        return __int_as_float(max(int(b[0]), int(b[1])));
    };
    auto spread = [&](float y, float* of) {   // that value back to all lanes of its column
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
        of[0] = __uint_as_float(a[0]);
        of[1] = __uint_as_float(a[1]);
    };

    // iteration i: this group's tile 2i+grp is in K slot i&1 (scores already formed) and V slot i&1.  The last one forms no
    // further scores (a launch of one pair: 0.5 us less)
    auto step = [&](auto last_step, int i, f32x4 (*s_cur)[2], f32x4 (*s_nxt)[2]) {
        constexpr bool LAST = decltype(last_step)::value;
        asm volatile("s_waitcnt vmcnt(0)");
        __builtin_amdgcn_s_barrier();
        if constexpr (!LAST) {
            issue_v(i + 1);
            if (i + 2 < n_pairs) issue_k(i + 2);
        }
        const unsigned char* stk = lds + ((i + 1) & 1) * A8_RING;
        const unsigned char* stv = lds + (i & 1) * A8_RING;
        bf16x8 opa[4], opb[4], p[4];   // p[2 j + c]
        auto read_k = [&](bf16x8* dst, int ks) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                dst[t] = *(const bf16x8*)(stk + (32 * (t >> 1) + 4 * (t & 1)) * (AHD * 2) + kaddr[ks]);
        };
        auto read_v = [&](bf16x8* dst, int u) {   // k-step u >> 1, head-dim tiles 4 (u & 1) .. + 3
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[e] = *(const bf16x8*)(stv + (4 * (u & 1) + e) * 16 * (AK * 2) + vaddr[u >> 1]);
        };
        auto mma_k = [&](const bf16x8* src, int ks) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int c = 0; c < 2; ++c) s_nxt[t][c] = mfma16(src[t], qreg[c][ks], ks == 0 ? negm[c] : s_nxt[t][c]);
        };
        auto mma_v = [&](const bf16x8* src, int u) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < 2; ++c) o[4 * (u & 1) + e][c] = mfma16(src[e], p[2 * (u >> 1) + c], o[4 * (u & 1) + e][c]);
        };
        auto expo = [&](int u) {
            const int j = u >> 1, c = u & 1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = __builtin_amdgcn_exp2f(s_cur[2 * j + (e >> 2)][c][e & 3]);
                l_part[c] += x;
                p[u][e] = bf16_t(x);
            }
        };
        if constexpr (LAST) {
            read_v(opa, 0);
            expo(0); expo(1); expo(2);
        } else {
            read_k(opa, 0);
            __builtin_amdgcn_sched_barrier(0);
            read_k(opb, 1); mma_k(opa, 0); expo(0);
            __builtin_amdgcn_sched_barrier(0);
            read_k(opa, 2); mma_k(opb, 1); expo(1);
            __builtin_amdgcn_sched_barrier(0);
            read_k(opb, 3); mma_k(opa, 2); expo(2);
            __builtin_amdgcn_sched_barrier(0);
            read_v(opa, 0); mma_k(opb, 3);
        }
        // the probabilities are only consumed after the branch below; pin them here, or the compiler
        // sinks the exponentials out of the block whose MFMAs they are meant to overlap with
#pragma unroll
        for (int e = 0; e < 3; ++e) asm volatile("" ::"v"(p[e]));
        asm volatile("" ::"v"(l_part[0]), "v"(l_part[1]));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (QW == 4) {   // the other half's step begins
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_setprio(0);
        }
        if constexpr (!LAST) {
            const int next_tile = 2 * (i + 1) + grp;
            if (next_tile >= first_masked) mask_tile(s_nxt, next_tile, my_pos);   // tiles past the end are blanked too
        }
        int raw[2];
        read_v(opb, 1);
        mma_v(opa, 0);
        expo(3);
        if constexpr (!LAST) {
            raw[0] = part_top(s_nxt, 0, 0, __float_as_int(s_nxt[0][0][0]));
            raw[0] = part_top(s_nxt, 0, 2, raw[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        read_v(opa, 2);
        mma_v(opb, 1);
        if constexpr (!LAST) {
            raw[1] = part_top(s_nxt, 1, 0, __float_as_int(s_nxt[0][1][0]));
            raw[1] = part_top(s_nxt, 1, 2, raw[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        read_v(opb, 3);
        mma_v(opa, 2);
        if constexpr (!LAST) raw_cur = row_top(raw);
        __builtin_amdgcn_sched_barrier(0);
        mma_v(opb, 3);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (QW == 4) __builtin_amdgcn_s_setprio(1);
        if (!LAST && __builtin_amdgcn_ballot_w64(raw_cur > RESCALE_LOG2) != 0) {
            float delta[2];
            spread(raw_cur, delta);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                delta[c] = delta[c] > RESCALE_LOG2 ? delta[c] : 0.f;   // of this query alone: a row's bits do not depend on the rows beside it
                const float corr = __builtin_amdgcn_exp2f(-delta[c]);
                m_run[c] += delta[c];
                l_part[c] *= corr;
#pragma unroll
                for (int t = 0; t < 8; ++t) o[t][c] *= f32x4{corr, corr, corr, corr};
#pragma unroll
                for (int t = 0; t < 4; ++t) s_nxt[t][c] -= f32x4{delta[c], delta[c], delta[c], delta[c]};   // formed against the old reference
                negm[c] = f32x4{-m_run[c], -m_run[c], -m_run[c], -m_run[c]};
            }
        }
    };

    // prologue: K, V of the first pair and K of the second in flight; K landed; scores and reference of the first tile
    issue_k(pair_lo);
    issue_v(pair_lo);
    if (pair_lo + 1 < n_pairs) {
        issue_k(pair_lo + 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER));
    } else {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER));
    }
    __builtin_amdgcn_s_barrier();
    f32x4 s_a[4][2], s_b[4][2];
    {
        const unsigned char* stk = lds + (pair_lo & 1) * A8_RING;
#pragma unroll
        for (int ks = 0; ks < AHD / 32; ++ks)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 a = *(const bf16x8*)(stk + (32 * (t >> 1) + 4 * (t & 1)) * (AHD * 2) + kaddr[ks]);
#pragma unroll
                for (int c = 0; c < 2; ++c) s_a[t][c] = mfma16(a, qreg[c][ks], ks == 0 ? zero4 : s_a[t][c]);
            }
    }
    if (2 * pair_lo + grp >= first_masked) mask_tile(s_a, 2 * pair_lo + grp, my_pos);
    {
        // the first tile fixes the reference exactly; a row that sees none of its keys (possible for
        // the second wave half only) keeps reference 0 and contributes nothing
        float raw[2], top[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) raw[c] = part_max(s_a, c, 2, part_max(s_a, c, 0, s_a[0][c][0]));
        spread(row_max(raw), top);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            m_run[c] = top[c] > -INFINITY ? top[c] : 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) s_a[t][c][v] -= m_run[c];
            negm[c] = f32x4{-m_run[c], -m_run[c], -m_run[c], -m_run[c]};
        }
    }
    if (QW == 4 && grp == 1) __builtin_amdgcn_s_barrier();   // half a step behind; the first half makes up for it at the end
    const std::integral_constant<bool, false> more;
    const std::integral_constant<bool, true> last;
    int pair = pair_lo;
    for (; pair + 2 < n_pairs; pair += 2) {   // two to a trip, so that the score buffers alternate without copies
        step(more, pair, s_a, s_b);
        step(more, pair + 1, s_b, s_a);
    }
    if (pair + 1 < n_pairs) {
        step(more, pair++, s_a, s_b);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) s_a[t][c] = s_b[t][c];
    }
    step(last, pair, s_a, s_b);
    if (QW == 4 && grp == 0) __builtin_amdgcn_s_barrier();

    // merge the two key halves: group B parks (O, l, reference) in LDS, group A combines and stores
    __syncthreads();
    float* park = (float*)lds + size_t(wave) * 68 * 64 + lane;
    float l_row[2];   // of the whole row, all of its lanes
    {
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_part[0]), __float_as_uint(l_part[1]), false, false);
        const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
        spread(__uint_as_float(b[0]) + __uint_as_float(b[1]), l_row);
    }
    if (grp == 1) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) park[(8 * t + 4 * c + v) * 64] = o[t][c][v];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            park[(64 + c) * 64] = l_row[c];
            park[(66 + c) * 64] = m_run[c];
        }
    }
    __syncthreads();
    if (grp == 0) {
        float ca[2], cb[2], m[2], l_tot[2], inv[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float l_b = park[(64 + c) * 64];
            const float m_b = l_b > 0.f ? park[(66 + c) * 64] : -1.0e30f;         // a half that saw no key has no reference
            m[c] = fmaxf(m_run[c], m_b);
            ca[c] = __builtin_amdgcn_exp2f(m_run[c] - m[c]);
            cb[c] = __builtin_amdgcn_exp2f(m_b - m[c]);
            // (sums written as fmaf, so that both instantiations round them alike)
            l_tot[c] = __builtin_fmaf(l_row[c], ca[c], l_b * cb[c]);
            inv[c] = SPLIT ? 1.0f : 1.0f / l_tot[c];
        }
        // before the branches, so that the columns do not wait for their reads one after the other
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) o[t][c][v] = __builtin_fmaf(o[t][c][v], ca[c], park[(8 * t + 4 * c + v) * 64] * cb[c]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (!is_query[c]) continue;
            if constexpr (SPLIT) {
                float* p = my_part(c);
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int v = 0; v < 4; v += 2) *(float2*)(p + t * 16 + 4 * lq + v) = make_float2(o[t][c][v], o[t][c][v + 1]);
                if (lq == 0) *(float2*)(p + AHD) = make_float2(l_tot[c] > 0.f ? m[c] * 0.6931471805599453f : -FLT_MAX, l_tot[c]);
            } else {
                bf16_t* op = out + size_t(my_row[c]) * n_q * AHD + h[c] * AHD;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    bf16x4 w;
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[v] = bf16_t(o[t][c][v] * inv[c]);
                    *(bf16x4*)(op + t * 16 + 4 * lq) = w;
                }
            }
        }
    }
}

// =====================================================================================
// Head dimension 64: eight waves as above (QW x 32 queries, the two wave halves on alternate 64-key tiles), K and
// V^T tiles of 8 KB in two LDS slots per half, filled one pair ahead by direct loads.
//
// Nothing is rounded that the one-wave-per-row kernel keeps in float32: the softmax scale stays out of Q (it is
// applied in the exponent's multiply-add) and a probability enters the second product as the sum of three bf16 values
// that hold its 24 bits, so P V takes three MFMAs per tile instead of one.  (Two values, 16 bits: 5 to 8 % less time, and
// two parts in a million more error of the bf16 result, 1.658401e-3 against 1.658399e-3.)
//
// What bounds it: the vector work per score (exponential, running sum, three cuts) beside 32 MFMAs per 64 x 32 scores.  Two
// workgroups share a CU, so that four waves per SIMD cover each other's waits.  512 rows x 32 heads (8 KV heads) against
// 2048 keys: 5203 -> 33 us with the merge, from the one-wave-per-row kernel; 1024 rows against 8192 keys 155 us.
// =====================================================================================
constexpr int H64_TILE = AK * 64 * 2, H64_GROUP = 4 * H64_TILE, H64_TABLE = 2 * H64_GROUP;

template <int QW>
__global__ void __launch_bounds__(128 * QW, QW == 4 ? 4 : 1)
attention_hd64_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ out, float* __restrict__ part, int n_q, int tok_begin,
                      int rows, KvView kv, int pairs_per_split) {
    constexpr int HD = 64, AQW = 32 * QW, PER = 8 / QW;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave8 % QW, grp = wave8 / QW;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int G = kv.n_kv, r = n_q / G;
    int g, rest;   // workgroups that share a KV head go to the same XCD
    if ((G & 7) == 0) {
        const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3, gpx = G >> 3;
        g = xcd + 8 * (idx % gpx);
        rest = idx / gpx;
    } else {
        g = blockIdx.x % G;
        rest = blockIdx.x / G;
    }
    const int h = g * r + rest % r, q0 = (rest / r) * AQW, split = blockIdx.y;
    const int pt = kv.page_tokens;
    const int my_pos = tok_begin + min(q0 + wave * 32 + lrow, rows - 1);
    const int wave_first_pos = tok_begin + min(q0 + wave * 32, rows - 1);
    const int wg_last_pos = tok_begin + min(q0 + AQW, rows) - 1;
    const int n_tiles = wg_last_pos / AK + 1;
    const int pair_lo = split * pairs_per_split, pair_hi = min(pair_lo + pairs_per_split, (n_tiles + 1) >> 1);
    const int first_masked = (wave_first_pos + 1) / AK;   // first tile with a key some query of this wave must not see

    bf16x8 qreg[HD / 16];
    {
        const bf16_t* qp = q + (size_t(h) * rows + (my_pos - tok_begin)) * HD + 8 * lhalf;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) qreg[ks] = *(const bf16x8*)(qp + 16 * ks);
    }
    // wave-load j of a tile covers its rows 8j .. 8j + 7 (128 B each); chunk c of row x is stored at c ^ ((x >> 1) & 7)
    unsigned koff[PER], voff[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int row = 8 * (wave + QW * i) + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        koff[i] = unsigned(row * HD + c * 8) * 2u;
        voff[i] = unsigned(row * pt + c * 8) * 2u;
    }
    unsigned long long* pg_lds = (unsigned long long*)(lds + H64_TABLE);
    {
        const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;
        const size_t page_bytes = kv.page_elems() * 2, k_head = size_t(g) * pt * HD * 2;
        for (int i = tid; i <= wg_last_pos / pt; i += 128 * QW) pg_lds[i] = (layer_base + kv.block_table[i]) * page_bytes + k_head;
    }
    __syncthreads();
    const unsigned long long k_to_v = (size_t(G - g) * pt * HD + size_t(g) * HD * pt) * 2;
    unsigned char* ring = lds + grp * H64_GROUP;          // slot s: K at 2 s tiles, V^T right after it
    auto page_of = [&](int key0) {                        // K block of head g in the page of a key (wave-uniform)
        const unsigned long long off = pg_lds[key0 / pt];
        const unsigned long long lo = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(off));
        const unsigned long long hi = (unsigned)__builtin_amdgcn_readfirstlane((int)unsigned(off >> 32));
        return (const char*)kv.pool + ((hi << 32) | lo);
    };
    auto issue = [&](int pair) {
        const int tile = min(2 * pair + grp, n_tiles - 1);   // a tile past the end re-reads the last one (it is masked)
        const char* page = page_of(tile * AK);
        const size_t in_page0 = size_t(tile * AK % pt);
        const char *kp = page + in_page0 * (HD * 2), *vp = page + k_to_v + in_page0 * 2;
        unsigned char* sa = ring + (pair & 1) * 2 * H64_TILE;
#pragma unroll
        for (int i = 0; i < PER; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(kp + koff[i]), (CAKE_LDS_AS void*)(sa + (wave + QW * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < PER; ++i)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(vp + voff[i]), (CAKE_LDS_AS void*)(sa + H64_TILE + (wave + QW * i) * 1024), 16, 0, 0);
    };
    const int sk = sigma16(lrow & 15), sv = (lrow >> 1) & 7;
    int kaddr[HD / 16], vaddr[4];
#pragma unroll
    for (int ks = 0; ks < HD / 16; ++ks) kaddr[ks] = (16 * (lrow >> 4) + sk) * 128 + (((2 * ks + lhalf) ^ ((sk >> 1) & 7)) << 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) vaddr[j] = H64_TILE + lrow * 128 + (((2 * j + lhalf) ^ sv) << 4);

    const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    f32x16 o[2] = {zero16, zero16};
    float m_run = -FLT_MAX, l_part = 0.f;
    const float sl2 = 0.125f * 1.4426950408889634f;   // 1/sqrt(64) * log2(e)
    constexpr float RESCALE_LOG2 = 6.0f;              // the reference follows the running maximum lazily, as above

    unsigned left_out = 0;   // tiles, counted from first_masked (a wave has at most four there)

    if (pair_lo < pair_hi) issue(pair_lo);
    for (int pair = pair_lo; pair < pair_hi; ++pair) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (pair + 1 < pair_hi) issue(pair + 1);
        const unsigned char* st = ring + (pair & 1) * 2 * H64_TILE;
        const int tile = 2 * pair + grp;
        f32x16 s[2];
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks)
#pragma unroll
            for (int t = 0; t < 2; ++t) s[t] = mfma32(*(const bf16x8*)(st + t * 32 * 128 + kaddr[ks]), qreg[ks], ks == 0 ? zero16 : s[t]);
        const bool masked = tile >= first_masked;   // also a tile past the end
        if (masked) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (tile * AK + 32 * t + (v & 7) + 8 * lhalf + 16 * (v >> 3) > my_pos) s[t][v] = -INFINITY;
        }
        float mx = s[0][0];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[t][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * sl2;
        const bool moved = mx > m_run + RESCALE_LOG2;   // each query's reference by itself, as above
        if (__builtin_amdgcn_ballot_w64(moved) != 0) {
            const float m_new = moved ? mx : m_run, corr = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_part *= corr;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[t][v] *= corr;
        }
        if (masked) {
            // A hidden key's probability is 0, but 0 * V is not where V holds an infinity or a NaN (a later token's, or
            // what a page held before): such a tile is left for the loop below.
            unsigned bad = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const u32x4 w = *(const u32x4*)(st + t * 32 * 128 + vaddr[j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) bad |= unsigned((w[e] & 0x7F80u) == 0x7F80u) | unsigned((w[e] & 0x7F800000u) == 0x7F800000u);
                }
            if (__builtin_amdgcn_ballot_w64(bad != 0) != 0) {
                left_out |= tile < n_tiles ? 1u << (tile - first_masked) : 0u;
                continue;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // x = hi + mid + lo exactly: its upper, middle and lower 8 significant bits, cut off one after the other
            unsigned w[3][4];
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                float x[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[j >> 1][8 * (j & 1) + i + e], sl2, -m_run));
                    l_part += x[e];
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    w[k][i / 2] = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302);
#pragma unroll
                    for (int e = 0; e < 2; ++e) x[e] -= __uint_as_float(__float_as_uint(x[e]) & 0xFFFF0000u);
                }
            }
            bf16x8 p[3];
            __builtin_memcpy(p, w, sizeof p);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bf16x8 v = *(const bf16x8*)(st + t * 32 * 128 + vaddr[j]);
#pragma unroll
                for (int k = 0; k < 3; ++k) o[t] = mfma32(v, p[k], o[t]);
            }
        }
    }

    // An infinity in V that a query does see: the lower parts of a probability may be 0, and 0 times the infinity is a NaN
    // where the probability times it is the infinity.  Such a range is taken again.
    bool nan = false;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; v += 2) nan |= __builtin_isunordered(o[t][v], o[t][v + 1]);
    const bool again = __builtin_amdgcn_ballot_w64(nan) != 0;
    if (again) {
        o[0] = o[1] = zero16;
        m_run = -FLT_MAX;
        l_part = 0.f;
    }
    // Tiles taken again or left out: key by key, over the keys a query sees, straight from the page
    // (wave-uniform bases and one lane offset, so that this loop costs the one above no registers).
    const int tile_end = again || left_out != 0 ? min(2 * pair_hi, n_tiles) : 0;
#pragma unroll 1
    for (int tile = 2 * pair_lo + grp; tile < tile_end; tile += 2) {
        if (!again && (tile < first_masked || (left_out >> (tile - first_masked) & 1) == 0)) continue;
        const int key0 = tile * AK;
        const char* page = page_of(key0);
        const unsigned in_page0 = unsigned(key0 % pt);
#pragma unroll 1
        for (int key = 0; key < AK; ++key) {
            const char* kp = page + size_t(in_page0 + key) * (HD * 2);
            const char* vp = page + k_to_v + size_t(in_page0 + key) * 2;
            float d = 0.f;   // this half-wave's 8 of every 16 elements, then the other's
#pragma unroll
            for (int ks = 0; ks < HD / 16; ++ks) {
                const bf16x8 kk = *(const bf16x8*)(kp + 32 * ks + unsigned(16 * lhalf));
#pragma unroll
                for (int e = 0; e < 8; ++e) d = __builtin_fmaf(float(kk[e]), float(qreg[ks][e]), d);
            }
            d += __shfl_xor(d, 32, 64);
            if (key0 + key > my_pos) continue;
            const float m_new = fmaxf(m_run, d * sl2), corr = __builtin_amdgcn_exp2f(m_run - m_new);
            const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(d, sl2, -m_new));
            m_run = m_new;
            l_part = l_part * corr + (lhalf == 0 ? x : 0.f);
            const unsigned lane_row = unsigned(8 * lhalf * pt);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const char* row = vp + size_t(32 * t + 8 * (v >> 2) + (v & 3)) * pt * 2;
                    o[t][v] = __builtin_fmaf(x, float(*(const bf16_t*)(row + lane_row)), o[t][v] * corr);
                }
        }
    }

    // merge the two key halves: the second parks (O, l, reference) in LDS, the first combines and stores
    __syncthreads();
    float* park = (float*)lds + size_t(wave) * 34 * 64 + lane;
    const float l_tot = l_part + __shfl_xor(l_part, 32, 64);
    if (grp == 1) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) park[(16 * t + v) * 64] = o[t][v];
        park[32 * 64] = l_tot;
        park[33 * 64] = m_run;
    }
    __syncthreads();
    const int row = q0 + wave * 32 + lrow;
    if (grp == 1 || row >= rows) return;
    const float m_b = park[33 * 64], m = fmaxf(m_run, m_b);
    const float ca = __builtin_amdgcn_exp2f(m_run - m), cb = __builtin_amdgcn_exp2f(m_b - m);
    const float den = l_tot * ca + park[32 * 64] * cb, inv = part ? 1.0f : 1.0f / den;
    float* pp = part + ((size_t(split) * n_q + h) * rows + row) * (HD + 2);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (o[t][4 * v4 + e] * ca + park[(16 * t + 4 * v4 + e) * 64] * cb) * inv;
            const int d = t * 32 + 8 * v4 + 4 * lhalf;
            if (part) {
                *(float2*)(pp + d) = make_float2(x[0], x[1]);
                *(float2*)(pp + d + 2) = make_float2(x[2], x[3]);
            } else {
                *(bf16x4*)(out + (size_t(row) * n_q + h) * HD + d) = bf16x4{bf16_t(x[0]), bf16_t(x[1]), bf16_t(x[2]), bf16_t(x[3])};
            }
        }
    if (part && lhalf == 0) *(float2*)(pp + HD) = make_float2(m * 0.6931471805599453f, den);
}

// =====================================================================================
// One-token attention on the matrix cores (first-token step; bf16 pages, head_dim 128).
//
// The "queries" of a workgroup are the r query heads that share KV head g, all at the same
// position; they fill r of the 16 C columns of transposed products as in the kernel of eight waves
// (S^T = K Q^T, O^T = V^T P^T in 16x16x32 MFMAs), the other columns stay zero.  That wastes most of the MFMA
// columns, which is free here: the kernel is bound by streaming the layer's K and V once.
// There is no reuse between waves, so nothing is
// staged in LDS: every lane loads its MFMA operand slices straight from the pages (K rows in the order of
// the eight-wave kernel, V^T row = head-dim index), a wave has the V^T tile of this step
// and the K tile of the next in flight while it works, and the W waves of a workgroup take
// the 32-key tiles of the workgroup's range in turn.  An operand of the 16-row MFMA is 64 bytes of each row; that of the
// 32-row one was 32, half of what a request fetches.  Partial (max, sum, O) per wave are merged
// through LDS and written per key range for the combine kernel.  Eight waves, two per SIMD, where their parts fit the
// LDS (up to 12 heads to a KV head), so that one's loads are out while the other works; else four.  us with the
// combine kernel (of one thread per output), 32-row and 16-row MFMAs: 32 heads on 8 at 32768 keys (134 MB) 37.7 and 34.4,
// at 8000 16.6 and 14.6, 32 on 32 at 16000 (262 MB) 55.9 and 51.
// =====================================================================================
constexpr int DK = 32;   // keys per tile

template <int W, int C>
__global__ void __launch_bounds__(64 * W)
decode_attention_mfma_kernel(const float* __restrict__ q, float* __restrict__ part, int n_q, int n_keys,
                             int tiles_per_split, KvView kv) {
    extern __shared__ float dlds[];   // [W][r][AHD + 2]: O, then max (natural-log units), then sum
    const int g = blockIdx.x, split = blockIdx.y, n_splits = gridDim.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: a page number comes by a scalar load and waits for no tile
    const int l16 = lane & 15, lq = lane >> 4;
    const int r = n_q / kv.n_kv;
    const int pt = kv.page_tokens;
    const int n_tiles = (n_keys + DK - 1) / DK;
    const int tile_lo = split * tiles_per_split * (AK / DK), tile_hi = min(tile_lo + tiles_per_split * (AK / DK), n_tiles);
    const float sl2 = 0.08838834764831845f * 1.4426950408889634f;

    const int krow = 8 * (l16 >> 2) + (l16 & 3);   // of score tile 0; four keys on in tile 1
    const size_t layer_base = size_t(kv.layer) * kv.n_physical_pages;
    bf16x8 kA[2][AHD / 32], vA[AHD / 16];
    auto tile_page = [&](int tile, int* in_page0) {
        const int key0 = tile * DK, lpage = key0 / pt;
        *in_page0 = key0 - lpage * pt;
        return (const bf16_t*)kv.pool + (layer_base + kv.block_table[lpage]) * kv.page_elems();
    };
    auto load_k = [&](int tile) {
        int in_page0;
        const bf16_t* kp = tile_page(tile, &in_page0) + (size_t(g) * pt + in_page0 + krow) * AHD + 8 * lq;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < AHD / 32; ++ks) kA[t][ks] = *(const bf16x8*)(kp + 4 * t * AHD + 32 * ks);
    };
    auto load_v = [&](int tile) {
        int in_page0;
        const bf16_t* vp = tile_page(tile, &in_page0) + size_t(kv.n_kv) * pt * AHD + (size_t(g) * AHD + l16) * pt + in_page0 + 8 * lq;
#pragma unroll
        for (int dt = 0; dt < AHD / 16; ++dt) vA[dt] = *(const bf16x8*)(vp + size_t(16 * dt) * pt);
    };

    const f32x4 zero4 = {0, 0, 0, 0};
    f32x4 o[AHD / 16][C];
    float m_run[C], l_part[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        m_run[c] = -1.0e30f;   // finite start: exp2(-inf - m) of a masked key is 0, never NaN
        l_part[c] = 0.f;
#pragma unroll
        for (int dt = 0; dt < AHD / 16; ++dt) o[dt][c] = zero4;
    }

    int tile = tile_lo + wave;
    if (tile < tile_hi) load_k(tile);
    bf16x8 qB[C][AHD / 32];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int ks = 0; ks < AHD / 32; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                qB[c][ks][e] = 16 * c + l16 < r ? bf16_t(q[size_t(g * r + 16 * c + l16) * AHD + 32 * ks + 8 * lq + e] * sl2) : bf16_t(0.f);
    for (; tile < tile_hi; tile += W) {
        load_v(tile);
        f32x4 s[2][C];
#pragma unroll
        for (int ks = 0; ks < AHD / 32; ++ks)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < C; ++c) s[t][c] = mfma16(kA[t][ks], qB[c][ks], ks == 0 ? zero4 : s[t][c]);
        if (tile + W < tile_hi) load_k(tile + W);
        if ((tile + 1) * DK > n_keys) {   // ragged last tile: keys past the prompt
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (tile * DK + 8 * lq + 4 * t + v >= n_keys) s[t][c][v] = -INFINITY;
        }
        bf16x8 pB[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float mx = s[0][c][0];
#pragma unroll
            for (int v = 1; v < 8; ++v) mx = fmaxf(mx, s[v >> 2][c][v & 3]);
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_new = fmaxf(m_run[c], mx);
            const float corr = __builtin_amdgcn_exp2f(m_run[c] - m_new);
            m_run[c] = m_new;
            if (__builtin_amdgcn_ballot_w64(corr != 1.0f) != 0) {   // what was summed so far moves to the new reference
                l_part[c] *= corr;
#pragma unroll
                for (int dt = 0; dt < AHD / 16; ++dt) o[dt][c] *= f32x4{corr, corr, corr, corr};
            }
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const float x = __builtin_amdgcn_exp2f(s[v >> 2][c][v & 3] - m_new);
                l_part[c] += x;
                pB[c][v] = bf16_t(x);
            }
        }
#pragma unroll
        for (int dt = 0; dt < AHD / 16; ++dt)
#pragma unroll
            for (int c = 0; c < C; ++c) o[dt][c] = mfma16(vA[dt], pB[c], o[dt][c]);
    }

    // merge the waves; column n of a wave belongs to query head g*r + n
#pragma unroll
    for (int c = 0; c < C; ++c) {
        float l_tot = l_part[c] + __shfl_xor(l_part[c], 16, 64);
        l_tot += __shfl_xor(l_tot, 32, 64);
        if (16 * c + l16 >= r) continue;
        float* w = dlds + size_t(wave * r + 16 * c + l16) * (AHD + 2);
#pragma unroll
        for (int dt = 0; dt < AHD / 16; ++dt)
#pragma unroll
            for (int v = 0; v < 4; ++v) w[16 * dt + 4 * lq + v] = o[dt][c][v];
        if (lq == 0) { w[AHD] = m_run[c] * 0.6931471805599453f; w[AHD + 1] = l_tot; }
    }
    __syncthreads();
    for (int idx = tid; idx < r * AHD; idx += 64 * W) {
        const int j = idx / AHD, d = idx % AHD;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) m = fmaxf(m, dlds[size_t(w * r + j) * (AHD + 2) + AHD]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float* src = dlds + size_t(w * r + j) * (AHD + 2);
            const float c = __expf(src[AHD] - m);
            num += src[d] * c;
            den += src[AHD + 1] * c;
        }
        float* dst = part + (size_t(g * r + j) * n_splits + split) * (AHD + 2);
        dst[d] = num;
        if (d == 0) { dst[AHD] = m; dst[AHD + 1] = den; }
    }
}

bool decode_attention_mfma_supported(int dtype, int head_dim, int page_tokens, int r) {
    return dtype == 1 && head_dim == AHD && page_tokens % AK == 0 && r >= 1 && r <= 32;
}

// Writes n_splits partial results per query head into `part` ([n_q][n_splits][head_dim + 2]).
hipError_t launch_decode_attention_mfma(const float* q, float* part, int n_q, int n_keys, int tiles_per_split,
                                        int n_splits, const KvView& kv, hipStream_t st) {
    const int r = n_q / kv.n_kv;
    const size_t wave_lds = size_t(r) * (AHD + 2) * sizeof(float);
    const dim3 grid(kv.n_kv, n_splits);
    if (r <= 12) hipLaunchKernelGGL((decode_attention_mfma_kernel<8, 1>), grid, dim3(512), 8 * wave_lds, st, q, part, n_q, n_keys, tiles_per_split, kv);
    else if (r <= 16) hipLaunchKernelGGL((decode_attention_mfma_kernel<4, 1>), grid, dim3(256), 4 * wave_lds, st, q, part, n_q, n_keys, tiles_per_split, kv);
    else hipLaunchKernelGGL((decode_attention_mfma_kernel<4, 2>), grid, dim3(256), 4 * wave_lds, st, q, part, n_q, n_keys, tiles_per_split, kv);
    return hipGetLastError();
}

bool attention_mfma_supported(int head_dim, int page_tokens) {
    return head_dim == AHD && page_tokens % AK == 0;
}

// How a launch is divided: queries per workgroup (32 qw) and key ranges, by the time of the busiest CU: a workgroup (one per
// CU) takes 1.98 us a pair of key tiles with 128 queries and 1.40 with 64 or fewer, 5.5 beyond its pairs, 9.5 where it leaves a
// part; key ranges cost the merge kernel and their parts' way through memory (about 4 bytes per ps each way).  These are
// prices of the kernel with 32x32x16 MFMAs.  The present one takes 1.42 us a pair (128 queries) and 1.23 (64, 32) and 7.1, 5.2
// and 4.7 beyond them, 1.54, 1.36 and 1.36 and 10.2, 8.6 and 8.2 where it leaves a part; over 490 launches (32 heads on 8 and 32,
// 64 on 8, 40 on 40, 24 on 8; 1 to 1024 rows behind 0 to 31744 keys) a choice takes 2.1 % more than the best, the worst 25 %
// (200 rows of 32 KV heads at 2000: 27.7 us, 22.2 in two ranges).  us undivided and divided, merge included, 32 heads on 8 KV
// heads: 8 rows at 4000 keys 50 and 17, 33 rows at 16000 175 and 29, 137 rows at 4000 53 and 26; 509 rows of 32 KV heads at
// 8000 101 and 73.
constexpr int A_LDS_MAX = 160 * 1024;
struct AttnPlan { int qw, splits, per; };   // 32 qw queries per workgroup, key ranges of `per` pairs
static AttnPlan attn_plan(int n_q, int n_kv, int tok_begin, int rows, const AttnWs& ws, int force_qw) {
    static const struct { int qw; double pair_us; } kinds[3] = {{4, 1.98}, {2, 1.40}, {1, 1.40}};
    const int n_pairs = (tok_begin + rows - 1) / (2 * AK) + 1;
    const double one = double(n_q) * rows * (AHD + 2) * sizeof(float);
    const int fixed = ws.range_keys / (2 * AK);   // pairs per range where the caller fixes it (and the parts fit)
    const bool use_fixed = fixed > 0 && ws.part && double((n_pairs + fixed - 1) / fixed) * one <= double(ws.bytes);
    AttnPlan best{4, 1, n_pairs};
    double best_us = 1e30;
    for (const auto& k : kinds) {
        if (force_qw && k.qw != force_qw) continue;
        const long wgs = (long(rows) * (n_q / n_kv) + 32 * k.qw - 1) / (32 * k.qw) * n_kv;
        for (int s = 1; s <= (use_fixed ? n_pairs : 32) && s <= n_pairs; ++s) {
            if (s > 1 && (!ws.part || s * one > double(ws.bytes))) break;
            const int per = use_fixed ? fixed : (n_pairs + s - 1) / s;
            if ((n_pairs + per - 1) / per != s) continue;
            double us = double((wgs * s + 255) / 256) * (per * k.pair_us + (s > 1 ? 9.5 : 5.5));
            if (s > 1) us = (us + 4.5 + 2.0 * s * one / 4.0e6) * 1.05;
            if (us < best_us) { best_us = us; best = AttnPlan{k.qw, s, per}; }
        }
    }
    return best;
}

template <int QW>
static hipError_t launch_mfma8(const bf16_t* q, bf16_t* out, float* part, int n_q, int tok_begin, int rows, const KvView& kv, int splits,
                               int per, int lds, hipStream_t st) {
    const int r = n_q / kv.n_kv, packed = (rows * r + 32 * QW - 1) / (32 * QW), apart = r * ((rows + 32 * QW - 1) / (32 * QW));
    const bool side_by_side = packed < apart;
    const int q_tiles = side_by_side ? packed : apart;
    auto kern = splits > 1 ? attention_mfma8_kernel<QW, true> : attention_mfma8_kernel<QW, false>;
    static bool attr_set[2] = {false, false};
    if (!attr_set[splits > 1]) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, A_LDS_MAX);
        if (e != hipSuccess) return e;
        attr_set[splits > 1] = true;
    }
    hipLaunchKernelGGL(kern, dim3(q_tiles * kv.n_kv, splits), dim3(128 * QW), lds, st, q, out, part, n_q, tok_begin, rows, kv, per, side_by_side);
    hipError_t e = hipGetLastError();
    return e != hipSuccess || splits == 1 ? e : launch_attention_merge(1, AHD, part, out, n_q, rows, splits, st);
}

hipError_t launch_attention_mfma(const void* q, void* out, int n_q, int tok_begin, int rows, const KvView& kv,
                                 hipStream_t st, int variant, const AttnWs& ws) {
    if (rows <= 0) return hipSuccess;
    const int table = 8 * ((tok_begin + rows - 1) / kv.page_tokens + 1);   // one 8-byte page offset per logical page
    if (variant == 1) {
        const int LDS = A_STAGES * A_STAGE + table, q_tiles = (rows + AQ - 1) / AQ;
        if (LDS > A_LDS_MAX) return hipErrorInvalidValue;
        static bool attr_set = false;
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)attention_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, A_LDS_MAX);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(attention_mfma_kernel, dim3(q_tiles * n_q), dim3(256), LDS, st, (const bf16_t*)q, (bf16_t*)out, n_q,
                           tok_begin, rows, kv, q_tiles);
        return hipGetLastError();
    }
    const int LDS = A8_TABLE + table;
    if (LDS > A_LDS_MAX) return hipErrorInvalidValue;
    const AttnPlan plan = attn_plan(n_q, kv.n_kv, tok_begin, rows, ws, variant == 2 ? 4 : variant == 3 ? 2 : 0);
    const bf16_t* Q = (const bf16_t*)q;
    if (plan.qw == 4) return launch_mfma8<4>(Q, (bf16_t*)out, ws.part, n_q, tok_begin, rows, kv, plan.splits, plan.per, LDS, st);
    if (plan.qw == 2) return launch_mfma8<2>(Q, (bf16_t*)out, ws.part, n_q, tok_begin, rows, kv, plan.splits, plan.per, LDS, st);
    return launch_mfma8<1>(Q, (bf16_t*)out, ws.part, n_q, tok_begin, rows, kv, plan.splits, plan.per, LDS, st);
}

// Head dimension 64, 16-byte reads of q, the pages and the result.  With fewer keys than 24 the one-wave-per-row kernel
// is as fast or faster (32 heads, us: 8 rows of 8 keys 5.6 here, 4.3 there; 16: 5.6, 5.2; 24: 5.6, 5.9), but not where a
// token's result must not depend on its step.  Queries per workgroup by the rows there are; key ranges until two
// workgroups per CU, as long as a range keeps four tile pairs and the parts fit the workspace, or fixed ones.
bool attention_hd64_supported(const void* q, const void* out, int n_keys, const KvView& kv, const AttnWs& ws) {
    const size_t table = 8 * (size_t(n_keys - 1) / kv.page_tokens + 1);
    return (n_keys >= 24 || ws.range_keys > 0) && kv.head_dim == 64 && kv.page_tokens % AK == 0 &&
           ((uintptr_t(q) | uintptr_t(out) | uintptr_t(kv.pool)) & 15) == 0 && H64_TABLE + table <= 160 * 1024;
}

template <int QW>
static hipError_t launch_hd64(const bf16_t* q, bf16_t* out, int n_q, int tok_begin, int rows, const KvView& kv, hipStream_t st,
                              const AttnWs& ws) {
    float* part = ws.part;
    const int q_tiles = (rows + 32 * QW - 1) / (32 * QW), n_pairs = (tok_begin + rows - 1) / (2 * AK) + 1;
    const int lds = H64_TABLE + 8 * ((tok_begin + rows - 1) / kv.page_tokens + 1);
    static bool attr_set = false;   // one flag per instantiation
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)attention_hd64_kernel<QW>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int fixed = ws.range_keys / (2 * AK);
    const int want = fixed ? (n_pairs + fixed - 1) / fixed : std::max(1, std::min(512 / std::max(1, q_tiles * n_q), n_pairs / 4));
    const size_t one = size_t(n_q) * rows * 66 * sizeof(float);
    const int room = part ? std::max(1, int(std::min<size_t>(size_t(want), ws.bytes / one))) : 1;
    const int per = fixed && room >= want ? fixed : (n_pairs + room - 1) / room;
    const int splits = (n_pairs + per - 1) / per;
    hipLaunchKernelGGL(attention_hd64_kernel<QW>, dim3(q_tiles * n_q, splits), dim3(128 * QW), lds, st, q, out, splits > 1 ? part : nullptr,
                       n_q, tok_begin, rows, kv, per);
    hipError_t e = hipGetLastError();
    return e != hipSuccess || splits == 1 ? e : launch_attention_merge(1, 64, part, out, n_q, rows, splits, st);
}

hipError_t launch_attention_hd64(const void* q, void* out, int n_q, int tok_begin, int rows, const KvView& kv, hipStream_t st,
                                 const AttnWs& ws) {
    if (rows <= 0) return hipSuccess;
    const bf16_t* Q = (const bf16_t*)q;
    if (rows <= 32) return launch_hd64<1>(Q, (bf16_t*)out, n_q, tok_begin, rows, kv, st, ws);
    if (rows <= 64) return launch_hd64<2>(Q, (bf16_t*)out, n_q, tok_begin, rows, kv, st, ws);
    return launch_hd64<4>(Q, (bf16_t*)out, n_q, tok_begin, rows, kv, st, ws);
}

}  // namespace cake
