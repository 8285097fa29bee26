// bf16 MFMA GEMMs for gfx950: the four projections of the decoder block
// (Sec. 3: Q = X W_Q, K = X W_K, V = X W_V, and the block's output and feed-forward products).
//
// MFMA shape used throughout: v_mfma_f32_32x32x16_bf16.  For D[32x32] += A[32x16] * B[16x32]
// lane l supplies A[l%32][8*(l/32) .. +7] and B[8*(l/32) .. +7][l%32], and holds
// D[8*(v/4) + 4*(l/32) + v%4][l%32] in accumulator register v (0..15).
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "gemm_p256.hpp"

namespace cake {

// =====================================================================================
// Persistent GEMM of 256 x 256 tiles, four waves: K ranges of a product, each stored as an output of its own (of the plain
// products with so many tiles those of short K too; see launch_p256 for the line to the kernel with eight waves).
//
// What bounds a 256 x 256 tile on this chip is the LDS port, then the texture addresser: with eight
// waves of 128 x 64 the operand reads plus the incoming tile data keep the LDS busy for as long as the
// MFMAs take, and a burst of loads after the slice barrier fills the addresser's FIFO, which blocks the
// issuing wave (and its MFMAs) until it drains.  So here:
//  * four waves of 128 x 128 (8 x 8 tiles of v_mfma_f32_16x16x32_bf16, 256 accumulator registers each):
//    16 operand reads per 64 MFMAs instead of 24, two thirds of the LDS read traffic;
//  * K in 64-deep slices (whole 128-byte lines from L2, half the requests of 32-deep slices), each slice
//    two 32 KB items (the A rows, the W rows) in a ring of five LDS slots filled by buffer loads to LDS;
//    row r of an item stores its 16-byte chunk c at c ^ ((r >> 1) & 7), so the sixteen rows a
//    quarter-wave reads hit all 64 banks once (the rows of an item are permuted in LDS, see tile_off);
//  * a slice is two phases of 64 MFMAs: phase A computes k-step 0 while the operands of k-step 1 are read
//    and the W item of slice g+2 is loaded; then one barrier (this slice's slots are free, the next slice
//    has landed); phase B computes k-step 1 while the first operands of slice g+1 are read and the A item
//    of slice g+2 is loaded into a slot just freed.  Inside a phase the source interleaves two operand
//    reads with one load, eight times, and sched_group_barrier pins 2 MFMAs between any two of them: no
//    burst anywhere (a load to LDS and an LDS read may not pass each other, so source order is issue
//    order);
//  * workgroups are persistent: each takes its tiles one after another, the loads of the next tile's first
//    slices are already in flight during the epilogue, and the grid is a whole number of rounds
//    (448 tiles -> 224 workgroups of two tiles).  Past the end of its tiles a workgroup's loads use an
//    empty buffer descriptor: they return zeros into slots nobody reads again, which keeps the load count
//    per phase, and with it the s_waitcnt arithmetic, the same in every iteration.
// Rows past M are read as zeros and their stores dropped by the buffer bounds checks.  Stores of four bytes, 64 of a row to
// a store: with 16 bytes to a lane (W as the MFMAs' first operand) 512 rows of 11008 -> 4096 in eight ranges take 60.8 us
// instead of 57.9, sum included.
// =====================================================================================
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
constexpr int P_ITEM = 256 * 128, P_SLOTS = 5, P_LDS = P_ITEM * P_SLOTS;
// An MFMA as an asm statement with the accumulator tied to an AGPR tuple: the 64 accumulators of a wave then
// fill the AGPR file exactly and stay where they are (left to itself the allocator rotates them through
// misaligned tuples with a hundred register copies per slice, each waiting for the MFMA that wrote its source),
// and, being volatile, the statements pin the order of the LDS reads and loads written between them: source
// order is issue order.  The compiler's hazard handling does not see them: the kernel puts the wait states
// between the last MFMA of an item and the first read of an accumulator itself.
__device__ __forceinline__ void p256_mfma(f32x4& c, const p256_frag_t& a, const p256_frag_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

__global__ void __launch_bounds__(256)
gemm_p256_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, float* __restrict__ out, int M, int N, int K,
                 int tiles_m, P256Plan plan, int tiles_per_wg, int ksplit) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int UNIT = 32;   // output columns per MFMA tile pair of a wave pair: panel of class c = c * UNIT columns
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lq = lane >> 4;
    // Items are numbered class-major (all 256-wide panels, then the 192-wide, then the 128-wide), within a class
    // panel-major, and over the K ranges range-major (item = range * tiles + tile).
    const int t8 = tiles_m * plan.n8, t6 = tiles_m * plan.n6, n_tiles = t8 + t6 + tiles_m * plan.n4;
    const int nb = n_tiles * ksplit, G = gridDim.x;
    // item u of this workgroup: one per round of G items.  Workgroup b runs on XCD b % 8: where the grid divides,
    // an XCD takes G / 8 consecutive items of a round (whole weight panels, shared through its L2).
    const bool by_xcd = (G & 7) == 0;
    const int in_round = by_xcd ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : int(blockIdx.x);
    auto item_of = [&](int u) { return u * G + in_round; };
    int n_mine = 0;
    for (int u = 0; u < tiles_per_wg; ++u)
        if (item_of(u) < nb) ++n_mine;
    if (n_mine == 0) return;
    // K ranges of whole 64-deep slices, the first n_long of them one slice longer
    const int nk_short = K / 64 / ksplit, n_long = K / 64 - nk_short * ksplit;
    auto slices_of = [&](int range) { return nk_short + (range < n_long); };
    auto first_k = [&](int range) { return (range * nk_short + min(range, n_long)) * 64; };
    // geometry of tile t: MFMA tiles per wave along N, first row of A, first column (in units of UNIT)
    auto tile_geom = [&](int t, int* nj, int* m0, int* col_units) {
        int c, p;
        if (t < t8) { c = 8; p = t; *col_units = 0; }
        else if (t < t8 + t6) { c = 6; p = t - t8; *col_units = 8 * plan.n8; }
        else { c = 4; p = t - t8 - t6; *col_units = 8 * plan.n8 + 6 * plan.n6; }
        *nj = c;
        *m0 = (p % tiles_m) * 256;
        *col_units += c * (p / tiles_m);
    };

    // ---- loads.  Wave-load wl = wave + 4 i of an item covers its rows 8 wl .. 8 wl + 7 (128 B each).
    const int lr = lane >> 3, lpos = lane & 7;
    const unsigned chunk = unsigned((lpos ^ (((wave & 1) << 2) + (lr >> 1))) << 4);
    const unsigned voff = unsigned((8 * wave + lr) * K * 2) + chunk, step = unsigned(32 * K * 2);
    // the item always has 256 rows of W: those past the panel lie outside the descriptor and arrive as zeros
    __amdgpu_buffer_rsrc_t ra, rw;
    int ka = 0, ua = 0, kw = 0, uw = 0, slot_a = 1, slot_w = 0, nk_a = 0, nk_w = 0;
    // descriptors start at the item's first row and first K element
    auto set_a = [&]() {
        const int q = item_of(ua), kbeg = first_k(q / n_tiles);
        nk_a = slices_of(q / n_tiles);
        int nj, m0, cu;
        tile_geom(q % n_tiles, &nj, &m0, &cu);
        ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + size_t(m0) * K + kbeg), 0, min(256, M - m0) * K * 2 - kbeg * 2, 0x00020000);
    };
    auto set_w = [&]() {
        const int q = item_of(uw), kbeg = first_k(q / n_tiles);
        nk_w = slices_of(q / n_tiles);
        int nj, m0, cu;
        tile_geom(q % n_tiles, &nj, &m0, &cu);
        rw = __builtin_amdgcn_make_buffer_rsrc((void*)(W + size_t(cu) * UNIT * K + kbeg), 0, nj * UNIT * K * 2 - kbeg * 2, 0x00020000);
    };
    auto next_a = [&]() {
        slot_a = slot_a >= P_SLOTS - 2 ? slot_a + 2 - P_SLOTS : slot_a + 2;
        if (++ka == nk_a) {
            ka = 0; ++ua;
            if (ua < n_mine) set_a();
            else ra = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0, 0x00020000);
        }
    };
    auto next_w = [&]() {
        slot_w = slot_w >= P_SLOTS - 2 ? slot_w + 2 - P_SLOTS : slot_w + 2;
        if (++kw == nk_w) {
            kw = 0; ++uw;
            if (uw < n_mine) set_w();
            else rw = __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, 0, 0x00020000);
        }
    };
    // wave-load l of an item: LDS base of its half of the wave's eight, the immediate offset picks one of four (the
    // builtin wants it as a literal)
    auto load_one = [&](__amdgpu_buffer_rsrc_t rs, unsigned char* dst, unsigned voff, int kk, unsigned step, int l)
                        __attribute__((always_inline)) {
        CAKE_LDS_AS void* d = (CAKE_LDS_AS void*)(dst + (l >> 2) * 4096);
        const unsigned so = kk * 128 + l * step - (l & 3) * 1024;
        switch (l & 3) {
            case 0: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 0, 0); break;
            case 1: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 1024, 0); break;
            case 2: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 2048, 0); break;
            default: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 3072, 0); break;
        }
    };
    auto load_item = [&](__amdgpu_buffer_rsrc_t rs, int slot, unsigned voff, int kk, unsigned step) {
        unsigned char* dst = lds + slot * P_ITEM + wave * 8192;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            load_one(rs, dst, voff, kk, step, r);
    };

    // ---- operand reads: MFMA tile i of this wave = rows 16 i .. 16 i + 15 of its share of the item (A: 128 rows from
    // 128 wm; W: 16 nj rows from 16 nj wn); k-step ks = chunks 4 ks .. 4 ks + 3
    const int sw = (l16 >> 1) & 7;
    // Where item row R sits in LDS: a wave's eight wave-loads of an item lie next to each other, 1 KB apart, so that
    // four of them share one value of M0 and differ in the instruction's immediate offset (which the hardware adds
    // to the LDS address and to the memory address alike; the scalar offset takes it off the latter again).  Every
    // write of M0 costs the one wave of a SIMD issue time: with one M0 per load the kernel ran 7 % longer.  Row
    // R = 32 r + 8 w + lr (wave-load r of wave w, row lr of its eight) is at byte 8192 w + 1024 r + 128 lr; for the
    // rows 16 i + l16 of MFMA tile i above a base that is a multiple of 32 rows that is
    // 8192 (2 (i & 1) + (l16 >> 3)) + 1024 (base / 32 + (i >> 1)) + 128 (l16 & 7).
    auto tile_off = [](int i) { return (i & 1) * 16384 + (i >> 1) * 1024; };
    const int lane_off = (l16 >> 3) * 8192 + (l16 & 7) * 128;
    const int a_lane = wm * 4096 + lane_off, b_lane = lane_off;
    int kch[2];
    kch[0] = (lq ^ sw) << 4;
    kch[1] = ((4 + lq) ^ sw) << 4;
    f32x4 acc[8][8];
    p256_frag_t a0[8], b0[8], a1[8], b1[8];
    // One phase of an item of class nj (a constant where this is called): the 8 nj MFMAs of a k-step on (a, b), with
    // the 8 + nj operand reads of the next k-step (into an, bn: W fragments first, they are needed by the first
    // MFMAs) and the eight wave-loads of one item dealt between them in `slots` places, two reads then a load,
    // at even distances, the last MFMAs after the last read.  b_wave: byte offset of this wave's W rows in an item,
    // of the class the fragments READ here belong to (the next item's in the last phase of an item).
    auto phase = [&](const int nj, const p256_frag_t* a, const p256_frag_t* b, p256_frag_t* an, p256_frag_t* bn, int sa, int sb,
                     int ks, int b_wave, __amdgpu_buffer_rsrc_t rs, int slot, unsigned voff, int kk, unsigned step)
                     __attribute__((always_inline)) {
        const unsigned char* pa = lds + sa * P_ITEM + a_lane + kch[ks];
        const unsigned char* pb = lds + sb * P_ITEM + b_wave + b_lane + kch[ks];
        unsigned char* dst = lds + slot * P_ITEM + wave * 8192;
        const int n_mfma = 8 * nj, reads = 8 + nj, slots = reads + 8, spread = n_mfma - (nj == 8 ? 16 : nj == 6 ? 8 : 6);
#pragma unroll
        for (int n = 0; n <= 64; ++n) {
#pragma unroll
            for (int sl = 0; sl < 24; ++sl) {
                if (sl < slots && ((sl + 1) * spread) / slots == n) {
                    const int grp = sl / 3, pos = sl % 3;
                    if (sl < 3 * (reads / 2) && pos < 2) {
                        const int r = 2 * grp + pos;
                        if (r < nj) bn[r] = *(const p256_frag_t*)(pb + tile_off(r));
                        else an[r - nj] = *(const p256_frag_t*)(pa + tile_off(r - nj));
                    } else {
                        const int l = sl < 3 * (reads / 2) ? grp : reads / 2 + (sl - 3 * (reads / 2));
                        load_one(rs, dst, voff, kk, step, l);
                    }
                }
            }
            if (n < n_mfma) p256_mfma(acc[n / nj][n % nj], a[n / nj], b[n % nj]);
        }
    };

    // prologue: items W0 A0 W1 A1 in flight (dummies past the end of the streams)
    set_a(); set_w();
    load_item(rw, slot_w, voff, kw, step); next_w();
    load_item(ra, slot_a, voff, ka, step); next_a();
    load_item(rw, slot_w, voff, kw, step); next_w();
    load_item(ra, slot_a, voff, ka, step); next_a();
    asm volatile("s_waitcnt vmcnt(16)");
    __builtin_amdgcn_s_barrier();
    int sa = 1, sb = 0;   // slots of the slice being consumed
    int nj_cur, m0_cur, cu_cur;
    tile_geom(item_of(0) % n_tiles, &nj_cur, &m0_cur, &cu_cur);
    {   // first operands of the first item
        const unsigned char* pa = lds + sa * P_ITEM + a_lane + kch[0];
        const unsigned char* pb = lds + sb * P_ITEM + wn * nj_cur * 512 + b_lane + kch[0];
#pragma unroll
        for (int j = 0; j < 8; ++j) b0[j] = *(const p256_frag_t*)(pb + tile_off(j));
#pragma unroll
        for (int i = 0; i < 8; ++i) a0[i] = *(const p256_frag_t*)(pa + tile_off(i));
    }
    // The K loop of an item of class nj (a constant at each of the three call sites)
    auto k_loop = [&](const int nj, const int nk, int b_wave, int b_wave_next) __attribute__((always_inline)) {
        for (int kt = 0; kt < nk; ++kt) {
            // phase A: k-step 0; operands of k-step 1; the W item of the slice after next (the weights come from HBM
            // and get the longer run-up: a slice and a half; the activations are L2 hits)
            phase(nj, a0, b0, a1, b1, sa, sb, 1, b_wave, rw, slot_w, voff, kw, step);
            next_w();
            // this wave has read all of this slice; the next slice must have landed: only the item just issued may be out
            asm volatile("s_waitcnt vmcnt(8)");
            __builtin_amdgcn_s_barrier();
            sa = sa >= P_SLOTS - 2 ? sa + 2 - P_SLOTS : sa + 2;
            sb = sb >= P_SLOTS - 2 ? sb + 2 - P_SLOTS : sb + 2;
            // phase B: k-step 1; first operands of the next slice; the A item of the slice after next into a freed slot
            phase(nj, a1, b1, a0, b0, sa, sb, 0, kt + 1 == nk ? b_wave_next : b_wave, ra, slot_a, voff, ka, step);
            next_a();
        }
    };
    // Epilogue of an item of class nj; accumulator (i, j)[v] is row 16 i + 4 lq + v, column 16 j + l16 of the wave's share
    auto epilogue = [&](const int nj, int q, int m0, int col_units) __attribute__((always_inline)) {
        // a K range is stored as an output of its own
        const __amdgpu_buffer_rsrc_t obuf = __builtin_amdgcn_make_buffer_rsrc(out + size_t(q / n_tiles) * M * N, 0, int(size_t(M) * N * 4), 0x00020000);
        const unsigned base = unsigned((m0 + wm * 128 + 4 * lq) * N + col_units * UNIT + wn * nj * 16 + l16) * 4u;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (j < nj) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][v]), obuf, base + unsigned((i * 16 + v) * N + j * 16) * 4u, 0, 0);
    };
    for (int u = 0; u < n_mine; ++u) {
        // cleared here and nowhere else, so that no accumulator value lives from one item to the next
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7");
        __builtin_amdgcn_sched_barrier(0);
        const int q = item_of(u);
        int nj_next = nj_cur, m0_next = 0, cu_next = 0;
        if (u + 1 < n_mine) tile_geom(item_of(u + 1) % n_tiles, &nj_next, &m0_next, &cu_next);
        const int nk = slices_of(q / n_tiles);
        const int b_wave = wn * nj_cur * 512, b_wave_next = wn * nj_next * 512;   // 16 nj rows = nj / 2 KB steps
        if (nj_cur == 8) k_loop(8, nk, b_wave, b_wave_next);
        else if (nj_cur == 6) k_loop(6, nk, b_wave, b_wave_next);
        else k_loop(4, nk, b_wave, b_wave_next);
        // The asm MFMAs are opaque to the compiler's hazard handling: let the last of them (four passes) retire
        // before the accumulators are read.
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 15");
        __builtin_amdgcn_sched_barrier(0);
        // (the next item's first slices are in flight during the epilogue)
        if (nj_cur == 8) epilogue(8, q, m0_cur, cu_cur);
        else if (nj_cur == 6) epilogue(6, q, m0_cur, cu_cur);
        else epilogue(4, q, m0_cur, cu_cur);
        nj_cur = nj_next; m0_cur = m0_next; cu_cur = cu_next;
        // loads and stores complete out of order with respect to each other: nothing is counted across them
        asm volatile("s_waitcnt vmcnt(0)");
    }
}

// =====================================================================================
// Yardstick: what the matrix pipes deliver with nothing else going on.  Every wave runs `iters`
// rounds of eight independent 32x32x16 bf16 MFMAs on operands it keeps in registers (no memory
// traffic, no LDS, no barriers); one value per wave is written so that the work is not dead.
// `acc[lane & 15]` at the end indexes a vector dynamically; the loop above keeps it in registers.
// =====================================================================================
__global__ void __launch_bounds__(512)
mfma_rate_kernel(float* __restrict__ out, int iters, unsigned seed) {
    const int lane = threadIdx.x & 63;
    // operands with the statistics of real data (what the pipes draw depends on how many bits toggle):
    // hashed values spread over [-2, 2), a different register set for every MFMA of a round, laid out
    // like one wave's 128x64 tile of the GEMM above (four A fragments, two B fragments)
    auto rnd = [&](unsigned k) {
        unsigned h = (k + seed) * 2654435761u; h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
        return bf16_t(float(int(h & 0xffff) - 32768) * (1.0f / 16384.0f));
    };
    bf16x8 a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) a[i][e] = rnd(unsigned((threadIdx.x * 4 + i) * 8 + e));
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) b[j][e] = rnd(0x9e3779b9u + unsigned((threadIdx.x * 2 + j) * 8 + e));
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(a[i], b[j], acc[i][j]);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) sum += acc[i][j][lane & 15];
    if (lane == 0) out[(size_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6] = sum;
}

// grid: `workgroups` workgroups of eight waves.  FLOPs = workgroups * 8 * iters * 8 * 32768.
hipError_t launch_mfma_rate(float* out, int workgroups, int iters, hipStream_t st) {
    hipLaunchKernelGGL(mfma_rate_kernel, dim3(workgroups), dim3(512), 0, st, out, iters, 12345u);
    return hipGetLastError();
}

// Tile configurations.  Chosen per GEMM by gemm_pick() from how well the grid fills 256 CUs.
struct GemmCfg { int bm, bn; };
// GCFG_128x128K: the 128x128 tile as two 128x64 halves, each shared by two waves that divide K (KW = 2)
// GCFG_P256: items of 256 rows on a persistent kernel (several per workgroup; launch_p256)
// GCFG_192x128: gate/up of 129 to 192 rows in one tile of all rows (137 rows of the Llama3-8B shape 56 us, 192 rows 58, against
// 62 and 63 on items of 256 rows; two bands of 128 take 82 and 89)
enum { GCFG_256x256 = 0, GCFG_256x128 = 1, GCFG_128x128 = 2, GCFG_128x192 = 3, GCFG_128x64 = 4, GCFG_128x128K = 5, GCFG_P256 = 6,
       GCFG_192x128 = 7, GCFG_COUNT = 8 };
static const GemmCfg kGemmCfg[GCFG_COUNT] = {{256, 256}, {256, 128}, {128, 128}, {128, 192}, {128, 64}, {128, 128}, {256, 256}, {192, 128}};

static P256Plan p256_plan(int epi, int tiles_m, int N);
static double p256_plan_cost(int tiles_m, int n8, int n6, int n4);

static int out_cols_per_tile(int cfg, int epi) { return epi == EPI_SWIGLU ? kGemmCfg[cfg].bn / 2 : kGemmCfg[cfg].bn; }

static bool gemm_cfg_ok(int cfg, int epi, int M, int N, int K) {
    if ((cfg == GCFG_128x192 || cfg == GCFG_128x64) && epi == EPI_SWIGLU) return false;   // odd n-tiles per wave: no gate/up pairs
    if (cfg == GCFG_128x128K && (epi == EPI_SWIGLU || (K % 64) != 0)) return false;
    if (cfg == GCFG_192x128 && (epi != EPI_SWIGLU || (K % 64) != 0)) return false;
    // the persistent kernel addresses everything through 32-bit buffer offsets
    // (its column panels are 256, 192 or 128 rows of W wide: N in units of 64, of 32 for SwiGLU)
    if (cfg == GCFG_P256)
        return M > 0 && N > 0 && K >= 64 && (K % 64) == 0 && double(M) * N * 4 < 2147483648.0 && double(K) * 512 < 2147483648.0 &&
               (N % (epi == EPI_SWIGLU ? 32 : 64)) == 0;
    return M > 0 && N > 0 && K >= 32 && (K % 32) == 0 && (N % out_cols_per_tile(cfg, epi)) == 0;
}

bool gemm_mfma_supported(int epi, int M, int N, int K) { return gemm_cfg_ok(GCFG_128x128, epi, M, N, K); }

// Cost model: the busiest CU runs ceil(workgroups / 256) of them one after another, each costing its
// tile area times its share of K divided by a per-shape efficiency (measured: larger tiles feed the
// MFMAs better because they pull fewer bytes per flop through L2), plus a fixed part (pipeline fill,
// epilogue).  With K split `ks` ways every workgroup writes its part and the one that finishes a tile
// reads ks parts back; that pays only where the unsplit choice is a small tile over a long K (the
// down projections of the 512-token-chunk and the 8192-wide shapes).  Unit: one 256x256 tile over
// K = 4096 costs 100 (about a microsecond each).
struct GemmChoice { int cfg, ksplit; };
static bool ksplit_ok(int cfg, int ks, int epi, int M, int N, int K, const GemmSplitWs* ws) {
    if (ks == 1) return true;
    if (!ws || !ws->part || !ws->counters || epi == EPI_SWIGLU) return false;
    if (K % ks || (K / ks) % 64 || K / ks < 512) return false;
    const GemmCfg& c = kGemmCfg[cfg];
    if (N % c.bn) return false;
    const long tiles = long((M + c.bm - 1) / c.bm) * (N / c.bn);
    return tiles <= ws->n_counters && size_t(tiles) * ks * c.bm * c.bn * sizeof(float) <= ws->part_bytes;
}
static GemmChoice gemm_pick(int epi, int M, int N, int K, const GemmSplitWs* ws, double* cost_out = nullptr) {
    // Measured TFLOP/s per busy CU, relative to 256x256; GCFG_P256 on four waves, which store plain products of under 100 slices.
    // The eight waves in turn that take the others, gate/up among them, are 5 to 11 % faster over 64 slices, 7 to 20 over 32.
    static const double eff[GCFG_COUNT] = {1.0, 0.60, 0.62, 0.80, 0.40, 0.65, 1.11, 0.72};
    GemmChoice best{GCFG_128x128, 1};
    double best_cost = 1e30;
    for (int cfg = GCFG_COUNT - 1; cfg >= 0; --cfg) {
        if (!gemm_cfg_ok(cfg, epi, M, N, K)) continue;
        const GemmCfg& c = kGemmCfg[cfg];
        if (cfg == GCFG_P256) {
            // The persistent kernels need a grid that fills the chip.  They are chosen unsplit only: with K split each range
            // becomes an output of its own, and products for which that pays go there by gemm_parts_plan (the path here
            // stays for forced use).
            const int tiles_m = (M + 255) / 256;
            const P256Plan plan = p256_plan(epi, tiles_m, N);
            const long items = long(tiles_m) * (plan.n8 + plan.n6 + plan.n4);
            if (items < 160) continue;
            // p256_plan_cost: the busiest workgroup's work in units of an eighth of a 256 x 256 tile
            const double cost = p256_plan_cost(tiles_m, plan.n8, plan.n6, plan.n4) * 12.5 * (double(K) / 4096.0) / eff[cfg] +
                                6.0 * double((items + 255) / 256);
            if (cost < best_cost) { best_cost = cost; best = GemmChoice{cfg, 1}; }
            continue;
        }
        const long tiles = long((M + c.bm - 1) / c.bm) * (N / out_cols_per_tile(cfg, epi));
        const double area = double(c.bm) * c.bn / 65536.0;
        for (int ks = 1; ks <= 8; ks *= 2) {
            if (!ksplit_ok(cfg, ks, epi, M, N, K, ws)) continue;
            const double rounds = double((tiles * ks + 255) / 256);
            double cost = rounds * (100.0 * area * (double(K) / ks / 4096.0) / eff[cfg] + 6.0);
            // measured: the parts cross the chip twice, at device scope; and a split must promise 8 % to be taken
            if (ks > 1) cost = (cost + 10.0 + 20.0 * area * ks) * 1.08;
            if (cost < best_cost) { best_cost = cost; best = GemmChoice{cfg, ks}; }
        }
    }
    if (cost_out) *cost_out = best_cost;
    return best;
}

// Panel widths of the persistent kernel for N columns and `tiles_m` row bands: counts of 8-, 6- and 4-tile panels
// with 8 n8 + 6 n6 + 4 n4 = N / unit that minimise the time of the busiest workgroup: items go out widest first,
// one per workgroup and round, so workgroup 0 takes the widest item of every round.  A narrow item is not
// faster in proportion (measured on four waves, 256 items over K = 4096: 108 us at 256 wide, 86 to 100 at 192, 70 to 74 at 128,
// and 1.2 us per slice at 128 wide over a long K against 1.46 at 256: the loads, reads and barriers of a slice
// stay the same), and every item costs an epilogue.
static double p256_plan_cost(int tiles_m, int n8, int n6, int n4) {
    const int c8 = tiles_m * n8, c6 = tiles_m * n6, nb = c8 + c6 + tiles_m * n4;
    const int rounds = (nb + 255) / 256, wgs = (nb + rounds - 1) / rounds;
    double cost = 0.0;
    for (int u = 0; u < rounds; ++u) {
        const int first = u * wgs;
        cost += (first < c8 ? 8.0 : first < c8 + c6 ? 7.0 : 6.2) + 0.4;
    }
    return cost;
}
static P256Plan p256_plan(int epi, int tiles_m, int N) {
    const int unit = epi == EPI_SWIGLU ? 16 : 32;
    if (N % (2 * unit)) return P256Plan{0, 0, 0};
    const int U = N / unit;
    struct Entry { int epi, tiles_m, N; P256Plan plan; };
    static std::mutex mu;
    static std::vector<Entry> cache;
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry& e : cache)
        if (e.epi == epi && e.tiles_m == tiles_m && e.N == N) return e.plan;
    P256Plan best{0, 0, 0};
    double best_cost = 1e30;
    for (int n8 = 0; 8 * n8 <= U; ++n8)
        for (int n6 = 0; 8 * n8 + 6 * n6 <= U; ++n6) {
            const int rem = U - 8 * n8 - 6 * n6;
            if (rem % 4) continue;
            const double c = p256_plan_cost(tiles_m, n8, n6, rem / 4);
            if (c < best_cost - 1e-9) { best_cost = c; best = P256Plan{n8, n6, rem / 4}; }
        }
    cache.push_back(Entry{epi, tiles_m, N, best});
    return best;
}

// 128 x 192, at most one workgroup per CU: the whole 160 KB of LDS as a ring of 64-deep slices, whose halves two waves
// take (120 KB in flight hide the latency of weights that come from HBM: 64 against 75 us for N = 6144).
static bool deep_192(int M, int N, int K, int ks) { return long((M + 127) / 128) * (N / 192) * ks <= 256 && (K / ks % 64) == 0; }

// The choice goes by M, and with it the order of a sum: K from end to end (every template tile in one K range), its
// slices' halves apart, 32 instead of 16 elements to an MFMA (the persistent kernel), K ranges apart.  Choices change at
// multiples of 64 rows only.
bool gemm_order_fixed(int epi, int max_rows, int N, int K, const GemmSplitWs* ws) {
    if (!gemm_mfma_supported(epi, 1, N, K)) return true;   // the generic kernel walks K in one order
    int first = -1;
    for (int M = 1; M <= max_rows; M += 64) {
        const GemmChoice ch = gemm_pick(epi, M, N, K, ws);
        const bool halves = ch.cfg == GCFG_128x128K || (ch.cfg == GCFG_128x192 && deep_192(M, N, K, ch.ksplit));
        const int order = 4 * ch.ksplit + (ch.cfg == GCFG_P256 ? 2 : halves ? 1 : 0);
        if (first >= 0 && order != first) return false;
        first = order;
    }
    return true;
}

// Items of 256 rows: on the eight waves in turn (kernels_gemm_pp.hip), but for float32 stores of items of under 100 slices, where
// its two phases of one group alone weigh as much as it gains.  Residual products and SwiGLU gain at every length.  us, four
// waves / in turn: residual 1024 rows -> 8192 over 1 slice 23.5 and 13.6, 16 slices 35 and 27, 32 slices 48 and 41; -> 16384 over 64
// slices 125 and 112, 128 slices 222 and 203; SwiGLU 1024 rows -> 14336 over 1 slice 23.5 and 14.4, 16 slices 64 and 53, 64
// slices 182 and 171.  Stores, each with the pass that adds the ranges up: 224 slices of 256 items 359.7 and 357.4, 128 of 128
// items 163 and 157, 112 of 256 items 203.5 and 202.2, 108 of 160 items 141.9 and 138.2; 75 of 192 items 111.2 and 110.4, 72 of
// 240 items 118.1 and 119.0, 64 of 256 items 119.6 and 120.9, 56 of 256 items 103.2 and 104.6,
// 43 of 128 items 67.0 and 68.2, 16 of 128 items 34.2 and 36.5.  Both give the same bits.
template <int EPI>
static hipError_t launch_p256(const bf16_t* A, const bf16_t* W, const bf16_t* W2, void* out, int M, int N, int K, const P256Plan& plan,
                              int ks, hipStream_t st) {
    if (EPI != EPI_STORE_F32 || K / 64 / ks >= 100) return launch_gemm_pp(EPI, A, W, W2, out, M, N, K, plan, ks, st);
    const int tiles_m = (M + 255) / 256, nb = tiles_m * (plan.n8 + plan.n6 + plan.n4) * ks;
    if (nb == 0) return hipErrorInvalidValue;
    // a whole number of rounds: every workgroup takes `rounds` items (the last may take one less)
    const int rounds = (nb + 255) / 256, wgs = (nb + rounds - 1) / rounds;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)gemm_p256_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, P_LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(gemm_p256_kernel, dim3(wgs), dim3(256), P_LDS, st, A, W, (float*)out, M, N, K, tiles_m, plan, rounds, ks);
    return hipGetLastError();
}

// K in `ks` ranges (whole slices of 64, as even as they go) on the persistent kernels, each range stored as an output of its
// own (256-wide panels).
static hipError_t launch_gemm_p256_parts(const void* a, const void* w, float* part, int M, int N, int K, int ks, hipStream_t st) {
    if (N % 256 || ks <= 0 || K / 64 < ks || !gemm_cfg_ok(GCFG_P256, EPI_STORE_F32, M, N, K)) return hipErrorInvalidValue;
    return launch_p256<EPI_STORE_F32>((const bf16_t*)a, (const bf16_t*)w, nullptr, part, M, N, K, P256Plan{N / 256, 0, 0}, ks, st);
}

template <int EPI>
static hipError_t gemm_launch_cfg(int cfg, int ks, const GemmSplitWs* ws, const bf16_t* A, const bf16_t* W, const bf16_t* W2,
                                  void* out, int M, int N, int K, hipStream_t st) {
    const long tiles128 = long((M + 127) / 128) * (N / (EPI == EPI_SWIGLU ? 64 : 128)) * ks;
    if (cfg == GCFG_P256) {
        if constexpr (EPI != EPI_SWIGLU) {
            if (ks > 1) {   // forced only: every range an output of its own, and a pass that adds them up
                const hipError_t e = launch_gemm_p256_parts(A, W, ws->part, M, N, K, ks, st);
                return e != hipSuccess ? e : launch_add_parts((float*)out, ws->part, ks, size_t(M) * N, st, EPI == EPI_STORE_F32);
            }
        }
        return launch_p256<EPI>(A, W, W2, out, M, N, K, p256_plan(EPI, (M + 255) / 256, N), 1, st);
    }
    switch (cfg) {
        case GCFG_256x256: return gemm_launch_t<4, 2, 2, 4, 32, 5, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
        case GCFG_256x128:
            if ((K / ks % 64) == 0) return gemm_launch_t<4, 2, 2, 2, 64, 3, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
            return gemm_launch_t<4, 2, 2, 2, 32, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
        case GCFG_128x192:
            if constexpr (EPI != EPI_SWIGLU) {
                if (deep_192(M, N, K, ks))
                    return gemm_launch_t<2, 3, 2, 2, 64, 4, EPI, 2>(A, W, W2, out, M, N, K, st, ks, ws);
                return gemm_launch_t<2, 3, 2, 2, 32, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
            } else {
                return hipErrorInvalidValue;
            }
        case GCFG_192x128:
            if constexpr (EPI == EPI_SWIGLU) return gemm_launch_t<3, 2, 2, 2, 64, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
            else return hipErrorInvalidValue;
        case GCFG_128x128K:
            if constexpr (EPI != EPI_SWIGLU) return gemm_launch_t<2, 2, 2, 2, 64, 5, EPI, 2>(A, W, W2, out, M, N, K, st, ks, ws);
            else return hipErrorInvalidValue;
        case GCFG_128x64:   // half-size chunks (M = 512): the only unsplit shape that still gives N = 4096 GEMMs 256 tiles
            if constexpr (EPI != EPI_SWIGLU) {
                if ((K / ks % 64) == 0) return gemm_launch_t<2, 1, 2, 2, 64, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
                return gemm_launch_t<2, 1, 2, 2, 32, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
            } else {
                return hipErrorInvalidValue;
            }
        default:
            // one workgroup per CU at most: spend the whole LDS on a deep ring of 64-deep slices
            // (96 KB in flight per CU); more tiles than CUs: 64 KB rings so two workgroups share a CU
            if (tiles128 <= 256 && (K / ks % 64) == 0) return gemm_launch_t<2, 2, 2, 2, 64, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
            return gemm_launch_t<2, 2, 2, 2, 32, 4, EPI>(A, W, W2, out, M, N, K, st, ks, ws);
    }
}

// K in `ks` ranges on the 128-row tiles whose slices two waves divide, each range stored as an output of its own.
static hipError_t launch_gemm_tile_parts(int bn, const void* a, const void* w, float* part, int M, int N, int K, int ks, hipStream_t st) {
    const bf16_t *A = (const bf16_t*)a, *W = (const bf16_t*)w;
    if (M <= 0 || N <= 0 || K <= 0 || ks <= 0 || N % bn || K % (64 * ks)) return hipErrorInvalidValue;
    if (bn == 128) return gemm_launch_t<2, 2, 2, 2, 64, 5, EPI_STORE_F32, 2>(A, W, nullptr, part, M, N, K, st, ks, nullptr, true);
    if (bn == 192) return gemm_launch_t<2, 3, 2, 2, 64, 4, EPI_STORE_F32, 2>(A, W, nullptr, part, M, N, K, st, ks, nullptr, true);
    return hipErrorInvalidValue;
}

// What a launch of launch_gemm_mfma takes, us, plain and with K split by ticket: a slice of the tile, a round beyond its slices,
// once, and a MB of the result that a residual product reads.  A launch of fewer workgroups than CUs runs its slices up to a
// fifth faster (L2).  Fitted, together with kWhole's, for the choices that they lead to, to 1464 measured products (39 shapes
// of 512 to 20480 x 2048 to 15360, 64 to 1024 rows, each plain and in two to eight ranges on every tile; fitted to half of the
// shapes, a choice on the others takes 1.8 to 2.0 % more than the best).  gemm_pick's prices, which only have to rank tiles,
// are up to 60 % above what launches take.
static double chip_fill(long wgs) { return 0.8 + 0.2 * double(wgs) / double((wgs + 255) / 256 * 256); }
static double plain_launch_us(const GemmChoice& ch, int epi, int M, int N, int K) {
    struct Price { double slice, round, once, residual_mb; };
    static const Price price[GCFG_COUNT][2] = {{{1.30, 3.0, 0.0, 0.50}, {2.12, 0.0, 0.3, 1.11}},      // 256 x 256
                                               {{1.00, 3.0, 0.0, 0.50}, {1.00, 0.0, 11.0, 0.80}},     // 256 x 128
                                               {{0.566, 2.0, 0.0, 0.45}, {0.634, 0.0, 10.9, 0.82}},   // 128 x 128
                                               {{0.693, 4.1, 0.0, 0.18}, {0.946, 0.0, 10.7, 0.49}},   // 128 x 192
                                               {{0.435, 3.5, 0.0, 1.02}, {0.401, 0.0, 9.4, 4.13}},    // 128 x 64
                                               {{0.566, 2.0, 0.0, 0.45}, {0.634, 0.0, 10.9, 0.82}},   // 128 x 128, waves along K
                                               {{0.853, 7.5, 0.0, 0.48}, {}},                         // persistent (four waves); gemm_pick leaves it unsplit
                                               {{0.693, 4.1, 0.0, 0.18}, {0.946, 0.0, 10.7, 0.49}}};  // 192 x 128 (gate/up only)
    const GemmCfg& c = kGemmCfg[ch.cfg];
    const Price& p = price[ch.cfg][ch.ksplit > 1];
    const long wgs = long((M + c.bm - 1) / c.bm) * (N / c.bn) * ch.ksplit;
    return double((wgs + 255) / 256) * (double(K) / 64 / ch.ksplit * p.slice * chip_fill(wgs) + p.round) + p.once +
           (epi == EPI_RESIDUAL_F32 ? double(M) * N * 4e-6 * p.residual_mb : 0.0);
}

// K ranges on the kernel for few rows: a slice takes 0.24 us + 0.075 us per 32 rows, HBM delivers the weights at 5.3 TB/s, L2
// the tiles at 10, or 0.05 per workgroup; a pass of its own that adds the ranges up reads and writes the result too.
// Whole tiles beyond that (kWhole): where the consumer adds the ranges up, against gemm_pick's price; where a pass does,
// against plain_launch_us.  Over those 1464 products a choice takes 1.5 % more than the best of all (against gemm_pick's prices
// it was 4.0 %, with 512 rows of 2048 -> 2048 at 20.7 us instead of 12.3).
// Both sides measured, us (the second without the consumer's part):
// down 8B (K = 14336 -> 4096) 1024 rows 133 and 87 in four ranges, 512 rows 81 and 51 in eight, 64 rows 40 and 24 in eight;
// down 70B 1024 rows 434 and 334 in two, 512 rows 284 and 183 in four; O 8B 512 rows 40 and 24 (128 x 128, two), 137 rows
// 32 and 16; QKV 8B 320 rows 37 and 27 (128 x 192, two), 137 rows 29 and 18; 512 rows of 8192 -> 2048 42 and 24 (128 x 128,
// four), of 2048 -> 2048 16 and 10, of 2048 -> 3072 21 and 12 (128 x 192, four).  No gain: 1024 rows of O 8B 43 and 39.
// rows_only: only the kernel for few rows.  Products of under 2048 columns stay with launch_gemm_mfma, where the order of
// their sums changes with M at fewer sizes, so that a narrow model's KV shows less of its steps; 64 rows of 4096 -> 1024
// would take 9.5 instead of 18.7.
GemmPartsPlan gemm_parts_plan(int epi, int M, int N, int K, const GemmSplitWs* ws, bool fused, bool rows_only) {
    GemmPartsPlan best{0, GEMM_PARTS_ROWS};
    if (epi == EPI_SWIGLU || !ws || !ws->part || M <= 0 || K % 64 || N % 128 || N < 2048) return best;
    double pick_cost;
    const GemmChoice plain = gemm_pick(epi, M, N, K, ws, &pick_cost);
    double best_us = pick_cost * 0.95;
    const double out_mb = double(M) * N * 4e-6;
    auto fits = [&](int ks) { return size_t(ks) * M * N * 4 <= ws->part_bytes; };
    auto take = [&](int ks, GemmPartsKind kind, double us) {
        if (us < best_us) { best_us = us; best = GemmPartsPlan{ks, kind}; }
    };
    if (M <= 192)
        for (int ks = 1; ks <= 8; ks *= 2) {
            if (K % (64 * ks) || !fits(ks)) continue;
            const double slices = double(K) / ks / 64;
            const int bm = (M + 31) / 32 * 32;
            const double tiles = N / 128, rounds = double((long(tiles) * ks + 255) / 256);
            if (bm >= 160 && tiles * ks < 160) continue;   // 137 and 192 rows of 11008 -> 4096 in four: 41 and 47 us, 38 and 42 without
            const double l2_rate = std::min(10.0, 0.05 * tiles * ks);   // TB/s
            const double after = (ks * out_mb + (fused ? 0.0 : 2.0 * out_mb)) / 4.5 + (fused ? 0.0 : 4.0) + ks * out_mb / 10.0;
            take(ks, GEMM_PARTS_ROWS, after + std::max(rounds * (slices * (0.24 + 0.075 * (bm / 32)) + 4.0),
                                                       std::max(double(N) * K * 2e-6 / 5.3 + 2.0, (bm + 128.0) * K * 2e-6 * tiles / l2_rate + 3.0)));
        }
    if (rows_only || (best.ksplit && M <= 192)) return best;
    // us per slice, per round, per MB of ranges, per MB of result and once; [1]: with a pass of its own
    struct Price { double slice, round, range_mb, out_mb, once; };
    static const struct { GemmPartsKind kind; int bm, bn; Price price[2]; } kWhole[3] = {
        {GEMM_PARTS_P256, 256, 256, {{1.40, 4.0, 1 / 4.5 + 1 / 10.0, 0.0, 0.0}, {1.14, 0.0, 0.315, 0.035, 8.1}}},
        {GEMM_PARTS_128, 128, 128, {{0.60, 4.0, 1 / 4.5 + 1 / 10.0, 0.0, 0.0}, {0.473, 0.0, 0.663, 0.033, 5.8}}},
        {GEMM_PARTS_192, 128, 192, {{0.72, 4.0, 1 / 4.5 + 1 / 10.0, 0.0, 0.0}, {0.605, 0.0, 0.501, 0.046, 6.4}}}};
    if (!fused) {
        // Unsplit 128 x 128 tiles, one to every CU, keep the order of their sums unless ranges promise a third (1024 rows of
        // 14336 -> 4096 137 us, in four ranges it would be 107; 512 of 28672 -> 8192 286 and 207).
        const bool one_each = plain.cfg == GCFG_128x128K && plain.ksplit == 1 && chip_fill(long((M + 127) / 128) * (N / 128)) > 0.98;
        best_us = plain_launch_us(plain, epi, M, N, K) * (one_each ? 0.66 : 0.945);
    }
    for (int ks = fused ? 1 : 2; ks <= 8; ++ks)
        for (const auto& t : kWhole) {
            if (N % t.bn || K / 64 < ks || !fits(ks)) continue;
            if (t.kind == GEMM_PARTS_P256 ? !gemm_cfg_ok(GCFG_P256, EPI_STORE_F32, M, N, K) : K % (64 * ks) != 0) continue;
            const Price& p = t.price[!fused];
            const long wgs = long(M + t.bm - 1) / t.bm * (N / t.bn) * ks;
            take(ks, t.kind, double((wgs + 255) / 256) * (std::ceil(double(K) / 64 / ks) * p.slice * chip_fill(wgs) + p.round) +
                                 ks * out_mb * p.range_mb + (epi == EPI_RESIDUAL_F32 ? 2.0 : 1.0) * out_mb * p.out_mb + p.once);
        }
    return best;
}

hipError_t launch_gemm_parts(const GemmPartsPlan& plan, const void* a, const void* w, float* part, int M, int N, int K, hipStream_t st) {
    switch (plan.kind) {
        case GEMM_PARTS_ROWS: return launch_gemm_rows_parts(a, w, part, M, N, K, plan.ksplit, st);
        case GEMM_PARTS_P256: return launch_gemm_p256_parts(a, w, part, M, N, K, plan.ksplit, st);
        case GEMM_PARTS_128: return launch_gemm_tile_parts(128, a, w, part, M, N, K, plan.ksplit, st);
        case GEMM_PARTS_192: return launch_gemm_tile_parts(192, a, w, part, M, N, K, plan.ksplit, st);
    }
    return hipErrorInvalidValue;
}

static GemmChoice gemm_choose(int epi, int M, int N, int K, int cfg_override, const GemmSplitWs* ws, int ksplit_override) {
    GemmChoice ch = gemm_pick(epi, M, N, K, ksplit_override == 1 ? nullptr : ws);
    if (cfg_override >= 0 && cfg_override < GCFG_COUNT && gemm_cfg_ok(cfg_override, epi, M, N, K)) ch = GemmChoice{cfg_override, 1};
    if (ksplit_override > 1 && gemm_cfg_ok(ch.cfg, epi, M, N, K) && ksplit_ok(ch.cfg, ksplit_override, epi, M, N, K, ws))
        ch.ksplit = ksplit_override;
    return ch;
}

void gemm_mfma_plan(int epi, int M, int N, int K, int cfg_override, const GemmSplitWs* ws, int ksplit_override,
                    int* bm, int* bn, int* ksplit) {
    const GemmChoice ch = gemm_choose(epi, M, N, K, cfg_override, ws, ksplit_override);
    *bm = kGemmCfg[ch.cfg].bm; *bn = kGemmCfg[ch.cfg].bn; *ksplit = ch.ksplit;
}

hipError_t launch_gemm_mfma(int epi, const void* a, const void* w, const void* w2, void* out, int M, int N, int K,
                            hipStream_t st, int cfg_override, const GemmSplitWs* ws, int ksplit_override) {
    const bf16_t *A = (const bf16_t*)a, *W = (const bf16_t*)w, *W2 = (const bf16_t*)w2;
    GemmChoice ch = gemm_choose(epi, M, N, K, cfg_override, ws, ksplit_override);
    if (ch.cfg == GCFG_P256 && (uintptr_t(out) & (epi == EPI_SWIGLU ? 1 : 3))) ch = GemmChoice{GCFG_128x128, 1};   // off whole elements
    if (ch.cfg == GCFG_P256 && (uintptr_t(out) & 15)) ch.ksplit = 1;   // forced K ranges: the pass that adds them up takes 16 bytes at once
    if (!gemm_cfg_ok(ch.cfg, epi, M, N, K)) return hipErrorInvalidValue;
    if (epi == EPI_SWIGLU) return gemm_launch_cfg<EPI_SWIGLU>(ch.cfg, 1, ws, A, W, W2, out, M, N, K, st);
    if (epi == EPI_RESIDUAL_F32) return gemm_launch_cfg<EPI_RESIDUAL_F32>(ch.cfg, ch.ksplit, ws, A, W, W2, out, M, N, K, st);
    if (epi == EPI_STORE_F32) return gemm_launch_cfg<EPI_STORE_F32>(ch.cfg, ch.ksplit, ws, A, W, W2, out, M, N, K, st);
    return hipErrorInvalidValue;
}

}  // namespace cake
