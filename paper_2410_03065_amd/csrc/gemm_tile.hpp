// The tiled bf16 MFMA GEMM kernel and its launch, shared by the sources that instantiate it (kernels_gemm.hip: the
// tiles of whole chunks; kernels_gemm_small.hip: few rows).
//
// MFMA shape used: v_mfma_f32_32x32x16_bf16.  For D[32x32] += A[32x16] * B[16x32]
// lane l supplies A[l%32][8*(l/32) .. +7] and B[8*(l/32) .. +7][l%32], and holds
// D[8*(v/4) + 4*(l/32) + v%4][l%32] in accumulator register v (0..15).
#pragma once
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace cake {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// =====================================================================================
// GEMM: out[M][N] = a[M][K] * w[N][K]^T, bf16 in, float32 accumulate.
//
// Workgroup tile BM x BN = (WAVES_M*WTM*32) x (WAVES_N*WTN*32); each wave owns WTM x WTN MFMA
// tiles.  K is consumed in BK-deep slices (32 or 64) held in a ring of STAGES LDS buffers that are filled
// by direct global->LDS loads (global_load_lds_dwordx4: 64 lanes x 16 B land contiguously, so
// the bank swizzle is applied by choosing which global chunk each lane fetches).  A slice row
// is 64 B or 128 B of 16-byte chunks; chunk c of row r is stored at c ^ ((r >> 2) & 3) resp.
// c ^ ((r >> 1) & 7), so the 16 rows that one quarter-wave reads with ds_read_b128 cover all
// 64 LDS banks once.  64-deep slices ask L2 for whole 128-byte lines (half as many requests).
//
// Software pipeline per slice (BK/16 MFMA steps of depth 16): while a step's MFMAs issue, the
// next step's operands are read; before the last step the wave waits for the NEXT slice's loads
// (vmcnt), meets the other waves at a bare s_barrier (no fence: a fence would drain every load in
// flight), refills the buffer freed one slice ago, and runs the last step's MFMAs while reading
// the next slice's first operands.  sched_group_barrier pins the 2-MFMA / 1-ds_read interleave.
//
// The block index is remapped so that workgroups that share a weight panel (the tiles_m tiles
// of one n-panel) sit on the same XCD and run at the same time: the panel is then fetched from
// HBM once and hit in that XCD's L2 by the others.
//
// Epilogues: store float32; add into a float32 residual stream; SwiGLU, where each wave's
// n-tiles alternate gate / up rows of the two weight matrices, so silu(gate) * up of one
// output column is formed in registers and the tile yields BN/2 output columns.
//
// Split K (ksplit > 1, not for SwiGLU): when a GEMM has too few large tiles to fill the chip, each
// tile is computed by ksplit workgroups, one per K range.  A workgroup writes its accumulators to
// its slot of a float32 workspace (in accumulator order, so the stores are contiguous), makes them
// visible device-wide and takes a ticket from the tile's counter; the one that draws the last
// ticket reads all parts back and adds them IN K-RANGE ORDER, so the result does not depend on
// which workgroup came last, runs the ordinary epilogue and puts the counter back to zero.  Nobody
// waits for anybody.  Launches that share a workspace must not overlap (one stream).  Without counters (float32 store
// only) each K range is stored as an output of its own, out[range][M][N], for a consumer that adds them up as it reads.
//
// Waves dividing K (KW = 2, 64-deep slices): every spatial part of the tile belongs to two waves,
// one taking the first two 16-deep steps of each slice, the other the last two.  The LDS traffic
// per MFMA is unchanged; what it buys is two waves per SIMD for a small tile (one CU's 128 x 128),
// so that one wave's waits (LDS, barrier) hide behind the other's MFMAs.  After the last slice the
// pair exchanges, through the idle ring, the 32-row bands each does not finish, and each runs the
// epilogue for its own bands.
// =====================================================================================
#define CAKE_GLOBAL_AS __attribute__((address_space(1)))
#define CAKE_LDS_AS __attribute__((address_space(3)))

// 16 consecutive rows must fall into 16 different 16-byte slots of a 256-byte bank window
template <int BK> __device__ __forceinline__ int gemm_swz(int row) { return BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3); }

template <int WTM, int WTN, int WAVES_M, int WAVES_N, int BK, int STAGES, int EPI, int KW>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N * KW)
gemm_mfma_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const bf16_t* __restrict__ W2,
                 void* __restrict__ outv, int M, int N, int K, int tiles_m, int tiles_n,
                 float* __restrict__ part, unsigned* __restrict__ counters, int ksplit) {
    constexpr int NWS = WAVES_M * WAVES_N;   // waves that divide the tile in space
    constexpr int NW = NWS * KW;             // times the waves that divide each slice along K
    constexpr int KS = BK / 16 / KW;         // 16-deep MFMA steps per slice and wave
    static_assert(KW == 1 || (KW == 2 && BK == 64), "K is divided between two waves at most, two steps each");
    static_assert(KW == 1 || STAGES * (WAVES_M * WTM + WAVES_N * WTN) * 32 * BK * 2 >= NWS * WTM * WTN * 4096, "the ring holds the exchange");
    constexpr int BM = WAVES_M * WTM * 32, BN = WAVES_N * WTN * 32;
    constexpr int ROWB = BK * 2, CPR = BK / 8, RPL = 64 / CPR;
    constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB, STAGE = A_BYTES + B_BYTES;
    constexpr int A_PER = A_BYTES / 1024 / NW, B_PER = B_BYTES / 1024 / NW, PER_TILE = A_PER + B_PER;
    static_assert((A_BYTES / 1024) % NW == 0 && (B_BYTES / 1024) % NW == 0, "slice loads must divide among the waves");
    static_assert(STAGES >= 3 && (STAGES - 2) * PER_TILE < 64, "vmcnt range");
    static_assert(EPI != EPI_SWIGLU || WTN % 2 == 0, "gate/up pairs");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave / NWS, wsp = wave % NWS;
    const int wm = wsp / WAVES_N, wn = wsp % WAVES_N;
    const int lrow = lane & 31, lhalf = lane >> 5;

    const int nb = tiles_m * tiles_n;
    const int bid = blockIdx.x;
    int t, kpart = 0;
    if (EPI == EPI_SWIGLU || ksplit == 1) {
        t = (nb % 8 == 0) ? (bid % 8) * (nb / 8) + bid / 8 : bid;
    } else if (8 % ksplit == 0 && nb % (8 / ksplit) == 0) {
        // block b runs on XCD b % 8: an XCD takes one K range of a group of whole weight panels
        const int xcd = bid & 7, per_group = nb / (8 / ksplit);
        kpart = xcd % ksplit;
        t = (xcd / ksplit) * per_group + (bid >> 3);
    } else {
        kpart = bid % ksplit;
        t = bid / ksplit;
    }
    const int tm = t % tiles_m, tn = t / tiles_m;
    const int k_begin = kpart * (K / ksplit);
    const int m0 = tm * BM;
    const int n0 = tn * (EPI == EPI_SWIGLU ? BN / 2 : BN);   // first output column of the tile

    // first row of weight-tile row `row` (for SwiGLU the tile's rows alternate between the two matrices)
    auto w_row = [&](int row) -> const bf16_t* {
        if (EPI == EPI_SWIGLU) {
            int wcol = row / (WTN * 32), j = (row / 32) % WTN, c = row % 32;
            return ((j & 1) ? W2 : W) + size_t(n0 + wcol * (WTN / 2) * 32 + (j >> 1) * 32 + c) * K + k_begin;
        }
        return W + size_t(n0 + row) * K + k_begin;
    };
    // global source of this lane for each 1 KB wave-load (16 rows x 64 B)
    const int lr = lane / CPR, lpos = lane % CPR;
    const bf16_t* ag[A_PER];
    const bf16_t* bg[B_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        int row = (wave + i * NW) * RPL + lr;
        ag[i] = A + size_t(min(m0 + row, M - 1)) * K + k_begin + (lpos ^ gemm_swz<BK>(row)) * 8;
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
        int row = (wave + i * NW) * RPL + lr;
        bg[i] = w_row(row) + (lpos ^ gemm_swz<BK>(row)) * 8;
    }
    // Wave-load idx of a slice (0 .. PER_TILE-1: the A loads, then the W loads) belongs to part idx % KS.  A slice
    // is not requested in one burst: the texture addresser takes 16 cycles per wave-load and a full address
    // FIFO blocks the issuing wave, MFMAs included.  Part 0 goes out after the barrier that frees the buffer,
    // part p in step p-1 of the following slice, each load between two operand reads.
    auto issue_one = [&](unsigned char* sa, int k0, int idx) {
        if (idx < A_PER)
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(ag[idx] + k0),
                                             (CAKE_LDS_AS void*)(sa + (wave + idx * NW) * 1024), 16, 0, 0);
        else
            __builtin_amdgcn_global_load_lds((const CAKE_GLOBAL_AS void*)(bg[idx - A_PER] + k0),
                                             (CAKE_LDS_AS void*)(sa + A_BYTES + (wave + (idx - A_PER) * NW) * 1024), 16, 0, 0);
    };
    auto issue = [&](int stage, int k0) {   // a whole slice at once (prologue)
        unsigned char* sa = lds + stage * STAGE;
#pragma unroll
        for (int idx = 0; idx < PER_TILE; ++idx) issue_one(sa, k0, idx);
    };
    constexpr int PART_MAX = (PER_TILE + KS - 1) / KS;

    f32x16 acc[WTM][WTN];
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int sw = gemm_swz<BK>(lrow);  // tile rows start at multiples of 32, so the swizzle depends on lrow only
    int koff[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) koff[ks] = ((2 * (kw * KS + ks) + lhalf) ^ sw) << 4;
    const int a_row_off = (wm * WTM * 32 + lrow) * ROWB;
    const int b_row_off = A_BYTES + (wn * WTN * 32 + lrow) * ROWB;
    auto rd = [&](bf16x8* a, bf16x8* bb, int stage, int koffv) {
        const unsigned char* st = lds + stage * STAGE;
#pragma unroll
        for (int i = 0; i < WTM; ++i) a[i] = *(const bf16x8*)(st + a_row_off + i * 32 * ROWB + koffv);
#pragma unroll
        for (int j = 0; j < WTN; ++j) bb[j] = *(const bf16x8*)(st + b_row_off + j * 32 * ROWB + koffv);
    };
    // the same reads with part `part` of the slice bound for `stage_ld` dealt between them (a load to LDS and an
    // LDS read may not pass each other, so this source order is the issue order)
    auto rd_ld = [&](bf16x8* a, bf16x8* bb, int stage, int koffv, int stage_ld, int k0, auto part_tag) {
        constexpr int PART = decltype(part_tag)::value;
        const unsigned char* st = lds + stage * STAGE;
        unsigned char* sa = lds + stage_ld * STAGE;
#pragma unroll
        for (int r = 0; r < WTM + WTN; ++r) {
            if (r < WTM) a[r] = *(const bf16x8*)(st + a_row_off + r * 32 * ROWB + koffv);
            else bb[r - WTM] = *(const bf16x8*)(st + b_row_off + (r - WTM) * 32 * ROWB + koffv);
            if (r < PART_MAX && PART + r * KS < PER_TILE) issue_one(sa, k0, PART + r * KS);
        }
    };
    auto mm = [&](const bf16x8* a, const bf16x8* bb) {
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < WTN; ++j) acc[i][j] = mfma32(a[i], bb[j], acc[i][j]);
    };
    auto interleave = [&]() {
#pragma unroll
        for (int i = 0; i < WTM + WTN; ++i) {
            if constexpr ((WTM * WTN) / (WTM + WTN) > 0)
                __builtin_amdgcn_sched_group_barrier(0x008, (WTM * WTN) / (WTM + WTN), 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                          // DS read
        }
    };

    auto interleave_ld = [&](auto part_tag) {
        constexpr int PART = decltype(part_tag)::value;
#pragma unroll
        for (int i = 0; i < WTM + WTN; ++i) {
            if constexpr ((WTM * WTN) / (WTM + WTN) > 0)
                __builtin_amdgcn_sched_group_barrier(0x008, (WTM * WTN) / (WTM + WTN), 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                          // DS read
            if (i < PART_MAX && PART + i * KS < PER_TILE) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // load
        }
    };
    static_assert(PART_MAX <= WTM + WTN, "one load per operand read at most");

    const int nk = K / ksplit / BK;
    // Slices 0 .. n_steady-1 each request the slice STAGES-1 ahead (part 0 in their last step, the other parts in
    // the first steps of the slice after them); the slices after that request nothing.
    const int n_steady = nk > STAGES - 1 ? nk - (STAGES - 1) : 0;
    // prologue: STAGES-1 slices in flight (of the last of them only part 0 if slice 0 will deal out the rest);
    // slice 0 landed; its step-0 operands in registers
#pragma unroll
    for (int st = 0; st < STAGES - 2; ++st)
        if (st < nk) issue(st, st * BK);
    if (STAGES - 2 < nk) {
        if (n_steady > 0) {
            unsigned char* sa = lds + (STAGES - 2) * STAGE;
#pragma unroll
            for (int r = 0; r < PART_MAX; ++r)
                if (r * KS < PER_TILE) issue_one(sa, (STAGES - 2) * BK, r * KS);
        } else {
            issue(STAGES - 2, (STAGES - 2) * BK);
        }
    }
    constexpr int PART0 = (PER_TILE + KS - 1) / KS;   // loads in part 0
    if (n_steady > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 3) * PER_TILE + PART0));
    else if (nk >= STAGES - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 2) * PER_TILE));
    else asm volatile("s_waitcnt vmcnt(0)");
    __builtin_amdgcn_s_barrier();
    bf16x8 opa[2][WTM], opb[2][WTN];   // operands of the current and the next step
    rd(opa[0], opb[0], 0, koff[0]);
    // One slice.  NEW: this slice requests part 0 of slice kt+STAGES-1 after its barrier.  DEFER: its first
    // steps request the remaining parts of slice kt+STAGES-2 (whose part 0 the slice before requested).
    auto slice = [&](int kt, auto new_tag, auto defer_tag) {
        constexpr bool NEW = decltype(new_tag)::value, DEFER = decltype(defer_tag)::value;
        const int cur = kt % STAGES;
        const int st_prev = (kt + STAGES - 2) % STAGES, k_prev = (kt + STAGES - 2) * BK;
        // steps 0 .. KS-2: this step's MFMAs, next step's operands from the same slice
        [&]<int... PS>(std::integer_sequence<int, PS...>) {
            ([&] {
                constexpr int ks = PS;
                if constexpr (DEFER) {
                    rd_ld(opa[(ks + 1) & 1], opb[(ks + 1) & 1], cur, koff[ks + 1], st_prev, k_prev, std::integral_constant<int, ks + 1>{});
                    mm(opa[ks & 1], opb[ks & 1]);
                    interleave_ld(std::integral_constant<int, ks + 1>{});
                } else {
                    rd(opa[(ks + 1) & 1], opb[(ks + 1) & 1], cur, koff[ks + 1]);
                    mm(opa[ks & 1], opb[ks & 1]);
                    interleave();
                }
            }(), ...);
        }(std::make_integer_sequence<int, KS - 1>{});
        // slice kt+1 must have landed before the last step reads its first operands: in the steady state everything
        // but the STAGES-3 slices after it may still be out
        if constexpr (NEW || DEFER) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 3) * PER_TILE));
        else asm volatile("s_waitcnt vmcnt(0)");
        __builtin_amdgcn_s_barrier();
        // every wave has finished reading slice kt-1: its buffer is refilled, starting now
        if constexpr (NEW) {
            rd_ld(opa[0], opb[0], (kt + 1) % STAGES, koff[0], (kt + STAGES - 1) % STAGES, (kt + STAGES - 1) * BK, std::integral_constant<int, 0>{});
            mm(opa[(KS - 1) & 1], opb[(KS - 1) & 1]);
            interleave_ld(std::integral_constant<int, 0>{});
        } else {
            // past the last slice this reads stale LDS that is never used
            rd(opa[0], opb[0], (kt + 1) % STAGES, koff[0]);
            mm(opa[(KS - 1) & 1], opb[(KS - 1) & 1]);
            interleave();
        }
    };
    {
        int kt = 0;
        for (; kt < n_steady; ++kt) slice(kt, std::true_type{}, std::true_type{});
        if (n_steady > 0) { slice(kt, std::false_type{}, std::true_type{}); ++kt; }
        for (; kt < nk; ++kt) slice(kt, std::false_type{}, std::false_type{});
    }

    // With K divided between two waves, wave kw finishes the 32-row bands i with (i & 1) == kw.
    auto band_is_mine = [&](int i) { return KW == 1 || (i & 1) == kw; };
    if constexpr (KW > 1) {
        // The two waves that shared a tile along K add up: each hands the other, through the ring (idle
        // by now), the bands it does not finish, and adds what it is handed (a + b = b + a exactly, so
        // the sum does not depend on which of the two holds it).
        static_assert(WTM % 2 == 0, "bands are dealt alternately");
        __syncthreads();
        float4* spot = (float4*)(lds + wsp * (WTM * WTN * 4096));
#pragma unroll
        for (int i = 0; i < WTM; ++i)
            if (!band_is_mine(i)) {
#pragma unroll
                for (int j = 0; j < WTN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        spot[((i * WTN + j) * 4 + q) * 64 + lane] =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < WTM; ++i)
            if (band_is_mine(i)) {
#pragma unroll
                for (int j = 0; j < WTN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 p = spot[((i * WTN + j) * 4 + q) * 64 + lane];
                        acc[i][j][4 * q] += p.x; acc[i][j][4 * q + 1] += p.y; acc[i][j][4 * q + 2] += p.z; acc[i][j][4 * q + 3] += p.w;
                    }
            }
    }
    const int tid_s = wsp * 64 + lane;   // thread index among the waves that hold a result

    if constexpr (EPI != EPI_SWIGLU) {
        if (ksplit > 1 && counters) {
            // Parts go through the workspace with device-scope accesses (the sc1 bit: written through to,
            // and read from, the level every XCD shares), so no cache-wide write-back or invalidate is
            // needed: a wave waits until its stores are acknowledged, the barrier collects all waves, then
            // one thread draws the ticket; the loads of the last workgroup are issued after its ticket.
            constexpr int TILE_B = BM * BN * 4, NT = NWS * 64;
            const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(part, 0, tiles_m * tiles_n * ksplit * TILE_B, 0x00020000);
            const unsigned slots = unsigned(t) * ksplit * TILE_B;
            const unsigned mine = slots + unsigned(kpart) * TILE_B;
            constexpr int DEVICE_SCOPE = 16;   // sc1
#pragma unroll
            for (int i = 0; i < WTM; ++i)
#pragma unroll
                for (int j = 0; j < WTN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (!band_is_mine(i)) continue;
                        u32x4 v = {__float_as_uint(acc[i][j][4 * q]), __float_as_uint(acc[i][j][4 * q + 1]),
                                   __float_as_uint(acc[i][j][4 * q + 2]), __float_as_uint(acc[i][j][4 * q + 3])};
                        __builtin_amdgcn_raw_buffer_store_b128(v, ws, mine + (((i * WTN + j) * 4 + q) * NT + tid_s) * 16, 0, DEVICE_SCOPE);
                    }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) *(volatile unsigned*)lds = __hip_atomic_fetch_add(&counters[t], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (*(volatile unsigned*)lds != unsigned(ksplit - 1)) return;
            // every part, this workgroup's too, comes from the workspace, in K-range order
            auto sum_parts = [&](auto nparts) {
                constexpr int NP = decltype(nparts)::value;
#pragma unroll
                for (int i = 0; i < WTM; ++i)
#pragma unroll
                    for (int j = 0; j < WTN; ++j) {
                        if (!band_is_mine(i)) continue;
                        u32x4 p[NP][4];
#pragma unroll
                        for (int sp = 0; sp < NP; ++sp)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                p[sp][q] = __builtin_amdgcn_raw_buffer_load_b128(ws, slots + sp * TILE_B + (((i * WTN + j) * 4 + q) * NT + tid_s) * 16, 0, DEVICE_SCOPE);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                float tot = __uint_as_float(p[0][q][e]);
#pragma unroll
                                for (int sp = 1; sp < NP; ++sp) tot += __uint_as_float(p[sp][q][e]);
                                acc[i][j][4 * q + e] = tot;
                            }
                    }
            };
            if (ksplit == 2) sum_parts(std::integral_constant<int, 2>{});
            else if (ksplit == 4) sum_parts(std::integral_constant<int, 4>{});
            else sum_parts(std::integral_constant<int, 8>{});
            if (tid == 0) counters[t] = 0;   // every ticket of this tile is drawn: ready for the next launch
        }
    }

    // epilogue
    if (EPI == EPI_STORE_F32 && !counters) outv = (float*)outv + size_t(kpart) * M * N;   // every K range to an output of its own
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
        if (!band_is_mine(i)) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            int row = m0 + (wm * WTM + i) * 32 + 8 * (v >> 2) + 4 * lhalf + (v & 3);
            if (row >= M) continue;
            if (EPI == EPI_SWIGLU) {
#pragma unroll
                for (int j = 0; j < WTN; j += 2) {
                    int col = n0 + wn * (WTN / 2) * 32 + (j >> 1) * 32 + lrow;
                    float g = acc[i][j][v], u = acc[i][j + 1][v];
                    // silu(g) * u; the hardware reciprocal (1 ulp) instead of an IEEE division: the result is rounded to bf16
                    ((bf16_t*)outv)[size_t(row) * N + col] = bf16_t(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
                }
            } else {
#pragma unroll
                for (int j = 0; j < WTN; ++j) {
                    int col = n0 + (wn * WTN + j) * 32 + lrow;
                    float* o = (float*)outv + size_t(row) * N + col;
                    if (EPI == EPI_RESIDUAL_F32) *o += acc[i][j][v];
                    else *o = acc[i][j][v];
                }
            }
        }
    }
}

template <int WTM, int WTN, int WAVES_M, int WAVES_N, int BK, int STAGES, int EPI, int KW = 1>
static hipError_t gemm_launch_t(const bf16_t* A, const bf16_t* W, const bf16_t* W2, void* out, int M, int N, int K,
                                hipStream_t st, int ksplit, const GemmSplitWs* ws, bool parts = false) {
    constexpr int BM = WAVES_M * WTM * 32, BN = WAVES_N * WTN * 32;
    constexpr int LDS = (BM + BN) * BK * 2 * STAGES;
    auto kern = gemm_mfma_kernel<WTM, WTN, WAVES_M, WAVES_N, BK, STAGES, EPI, KW>;
    static bool attr_set = false;   // one flag per instantiation
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / (EPI == EPI_SWIGLU ? BN / 2 : BN);
    if (ksplit > 1 && (K / ksplit) % BK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * ksplit), dim3(64 * WAVES_M * WAVES_N * KW), LDS, st, A, W, W2, out, M, N, K,
                       tiles_m, tiles_n, ksplit > 1 && !parts ? ws->part : nullptr, ksplit > 1 && !parts ? ws->counters : nullptr, ksplit);
    return hipGetLastError();
}

}  // namespace cake
