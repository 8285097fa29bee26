// bf16 products of work items of 256 rows on eight waves in turn: gate/up with SwiGLU, and the products whose items have long
// K ranges.
//
// A wave that forms MFMAs back to back does not get anything else issued: with one wave to a SIMD (the four-wave kernel in
// kernels_gemm.hip) every load to LDS between two MFMAs costs it about 50 cycles, 30 % of a slice.  Here a SIMD has two waves,
// of two groups, half a slice apart.  While a wave of one group forms the 64 MFMAs of its slice and nothing else, the wave of
// the other reads its operands of the next one (24 reads, 64 rows of A x 128 of W in 64-deep slices) and requests data for
// later ones (8 loads); then they change places.  One barrier at the end of every phase:
//
//     phase         2 g           2 g + 1       2 g + 2
//     group 0       reads g       products g    reads g + 1
//     group 1       products g-1  reads g       products g
//
// The price is LDS traffic, 24 reads per 64 MFMAs and wave instead of 16, and two phases of one group alone at the ends of an
// item.  Four waves / in turn, us: 1024 x 4096 -> 2 x 14336 with SwiGLU 192 and 179, 512 x 4096 -> 2 x 11008 86 and 80,
// 512 x 2048 -> 2 x 8192 37.5 and 31; 1024 x 8192 -> 8192 147 and 143.  What bounds it is the power limit and what a phase waits for
// lines from beyond L2: with no loads in the loop the first of these took 142 us where it took 181, with all of W from L2 164
// (MFMAs alone hold 1.9 GHz).  Not gained: W lines touched 3 to 8 slices ahead, into L2 (151 -> 145 us on one card, 149 -> 150 on
// another); raised wave priority in the product phase; the loads before or after all reads of a phase; half of A one slice
// ahead instead of two, and half of W two instead of one.
//
// LDS holds ten half items of 16 KB (128 rows of 128 bytes: whole lines from L2), a ring in the order in which they are
// requested.  Of slice g group 0 requests its own half of W two slices ahead (phase 2 g - 4) and group 1's half one ahead
// (2 g - 2), group 1 both halves of A two ahead (2 g - 3).  What phase p asks for takes the place of what was last read in
// phase p - 1 or before, and has three phases or more to arrive.
// Row r of a half stores its 16-byte chunk c at c ^ ((r >> 1) & 7), so the sixteen rows a quarter-wave reads hit all 64 banks
// once.  Buffer bounds: rows past M or past a panel arrive as zeros, and their stores are dropped.  Workgroups are
// persistent: the requests run on into the next item, past the last one through an empty descriptor, so that the counts in
// the waits are the same in every slice.  The waits count loads, which return in order; stores in flight can only make
// them wait for more.
// SwiGLU: the W rows of a half alternate between the two matrices in groups of sixteen (even MFMA tiles of a wave hold gate
// columns, odd ones the same columns of up), so an item yields half as many output columns, formed in registers.
// Stores of 16 bytes need a result on 4 bytes, which every float32 result is; ODD: a bf16 result that starts half-way between
// two words leaves in pieces of two and four bytes (1024 x 4096 -> 2 x 14336: 174 us on 4 bytes, 184 between two words, on
// 128 x 128 tiles 311).
#include <type_traits>
#include <utility>

#include "gemm_p256.hpp"

namespace cake {

constexpr int PP_HALF = 128 * 128, PP_SLOTS = 10, PP_LDS = PP_HALF * PP_SLOTS;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Accumulators by name.  MFMA tile T of a wave lives in a[4 T .. 4 T + 3] from the clearing to the epilogue: every statement
// that touches an AGPR is asm, and the build fails if the compiler places another (left to the register allocator the
// accumulators rotate through misaligned tuples with register copies that wait for the MFMA before them, or are spilled).
// Volatile statements keep their order, and with it that of the LDS reads and loads written between them; the wait states
// around an MFMA are the kernel's business.
template <int T> __device__ __forceinline__ void pp_mfma(const p256_frag_t& a, const p256_frag_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(a), "v"(b), "n"(4 * T), "n"(4 * T + 3));
}
template <int R> __device__ __forceinline__ void pp_clear() { asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(R)); }
template <int R> __device__ __forceinline__ float pp_read() {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(R));
    return x;
}
// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <int N, typename F> __device__ __forceinline__ void pp_each(F f) {
    [&]<int... X>(std::integer_sequence<int, X...>) { (f(std::integral_constant<int, X>{}), ...); }(std::make_integer_sequence<int, N>{});
}

template <int EPI, bool ODD>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2), amdgpu_num_vgpr(128)))
gemm_pp_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const bf16_t* __restrict__ W2,
                 void* __restrict__ outv, int M, int N, int K, int tiles_m, P256Plan plan, int tiles_per_wg, int ksplit) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int UNIT = EPI == EPI_SWIGLU ? 16 : 32;   // output columns per MFMA tile pair of a wave pair: panel of class c = c * UNIT columns
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, wm = wave & 3;           // group: half of the panel; wave: 64 of the band's rows
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

    // ---- loads.  Group 0 brings the W panel: stream 0 the half that group 1 reads, one slice ahead, stream 1 its own, two
    // slices ahead; group 1 the A band, two slices ahead: stream 0 its first 128 rows, stream 1 the others.
    // Wave-load i of wave wm covers rows 32 i + 8 wm .. + 7 of a half (128 B each).
    const int lr = lane >> 3, lpos = lane & 7;
    const unsigned chunk = unsigned((lpos ^ (((wave & 1) << 2) + (lr >> 1))) << 4);
    // W rows: plain, item row = panel row; SwiGLU, waves 0 and 1 of a group fetch gate rows, waves 2 and 3 up rows.  The
    // half always has 128 rows: those past the panel's half lie outside the descriptor and arrive as zeros.
    const bool pairs = EPI == EPI_SWIGLU && !grp;
    const unsigned voff = unsigned((8 * (pairs ? wave & 1 : wm) + lr) * K * 2) + chunk, step = unsigned((pairs ? 16 : 32) * K * 2);
    struct Stream { __amdgpu_buffer_rsrc_t rs; int k, u, nk; } st[2];
    // descriptors start at the half's first row and first K element
    auto set = [&](Stream& x, int which) __attribute__((always_inline)) {
        if (x.u >= n_mine) { x.rs = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0, 0x00020000); return; }
        const int q = item_of(x.u), kbeg = first_k(q / n_tiles);
        x.nk = slices_of(q / n_tiles);
        int nj, m0, cu;
        tile_geom(q % n_tiles, &nj, &m0, &cu);
        m0 += which * 128;
        const int nw = nj * (UNIT / 2);   // of the half: output columns
        const int rows = __builtin_amdgcn_readfirstlane(grp ? max(0, min(128, M - m0)) : nw);   // in a scalar register, like the descriptor
        const bf16_t* base = grp ? A + size_t(rows > 0 ? m0 : 0) * K
                                 : (EPI == EPI_SWIGLU && (wave & 2) ? W2 : W) + size_t(cu * UNIT + (1 - which) * nw) * K;
        x.rs = __builtin_amdgcn_make_buffer_rsrc((void*)(base + kbeg), 0, rows > 0 ? rows * K * 2 - kbeg * 2 : 0, 0x00020000);
    };
    auto next = [&](Stream& x, int which) __attribute__((always_inline)) {
        if (++x.k == x.nk) { x.k = 0; ++x.u; set(x, which); }
    };
    // wave-load i of a half: the immediate offset picks one of a wave's four kilobytes (the builtin wants it as a literal)
    auto load_one = [&](const Stream& x, int slot, int i) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rs = x.rs;
        CAKE_LDS_AS void* d = (CAKE_LDS_AS void*)(lds + slot * PP_HALF + wm * 4096);
        const unsigned so = x.k * 128 + i * step - i * 1024;
        switch (i) {
            case 0: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 0, 0); break;
            case 1: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 1024, 0); break;
            case 2: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 2048, 0); break;
            default: __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, d, 16, voff, so, 3072, 0); break;
        }
    };
    auto load_half = [&](int which, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load_one(st[which], slot, i);
        next(st[which], which);
    };

    // ---- operand reads: MFMA tile i of this wave = rows 64 wm + 16 i .. + 15 of the band; tile j = rows 16 j .. + 15 of its
    // group's half of the panel; k-step ks = chunks 4 ks .. 4 ks + 3.
    const int sw = (l16 >> 1) & 7;
    // Where row R of a half sits in LDS: a wave's four wave-loads lie next to each other, 1 KB apart, so that they share
    // one value of M0 and differ in the instruction's immediate offset (which the hardware adds to the LDS address and to
    // the memory address alike; the scalar offset takes it off the latter again).  Row R = 32 i + 8 w + lr (wave-load i of
    // wave w, row lr of its eight) is at byte 4096 w + 1024 i + 128 lr; for row l16 of tile t that is
    // 8192 (t & 1) + 1024 (t >> 1) + 4096 (l16 >> 3) + 128 (l16 & 7).
    auto tile_off = [](int t) { return (t & 1) * 8192 + (t >> 1) * 1024; };
    const int b_lane = (l16 >> 3) * 4096 + (l16 & 7) * 128, a_lane = b_lane + (wm & 1) * 2048;
    int kch[2];
    kch[0] = (lq ^ sw) << 4;
    kch[1] = ((4 + lq) ^ sw) << 4;
    p256_frag_t a[2][4], b[2][8];
    asm volatile("" ::: "a127");   // the accumulators: a0 .. a127

    // Slots of the ring: 4 s (group 0's half of W of slice s), + 5 (group 1's), + 2 (rows 0 .. 127 of A), + 3 (rows 128 ..), mod 10
    auto ring = [](int x) { return x >= PP_SLOTS ? x - PP_SLOTS : x; };
    int q4 = 0;   // 4 s mod 10 of the slice to be read next
    st[0].k = st[0].u = st[1].k = st[1].u = 0;
    set(st[0], 0); set(st[1], 1);
    if (!grp) { load_half(1, 0); load_half(0, 5); load_half(1, 4); }
    else { load_half(0, 2); load_half(1, 3); load_half(0, 6); load_half(1, 7); }
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (grp) __builtin_amdgcn_s_barrier();   // a phase behind

    constexpr int OUT_ELT = EPI == EPI_SWIGLU ? 2 : 4;
    // ODD: from the word that the result's first element shares
    __amdgpu_buffer_rsrc_t obuf = __builtin_amdgcn_make_buffer_rsrc((char*)outv - (ODD ? 2 : 0), 0, int(size_t(M) * N * OUT_ELT) + (ODD ? 2 : 0), 0x00020000);
    // The K loop of an item of class nj (a constant at each of the three call sites)
    auto k_loop = [&](auto nj_tag, const int nk) __attribute__((always_inline)) {
        constexpr int nj = decltype(nj_tag)::value;
        int left = nk;   // at least one: a loop that might run no slice gets a path that clears accumulators beside the MFMAs
        do {
            // reading phase: this slice's operands, and the requests for later slices between them
            {
                const unsigned char* pa = lds + ring(q4 + 2 + (wm >> 1)) * PP_HALF + a_lane;
                const unsigned char* pb = lds + ring(q4 + 5 * grp) * PP_HALF + b_lane;
                const int slot_x = ring(q4 + (grp ? 0 : 9)), slot_y = ring(q4 + (grp ? 1 : 8));
#pragma unroll
                for (int r = 0; r < 24; ++r) {   // k-step r / 12: W fragments, then A fragments
                    const int ks = r / 12, f = r % 12;
                    if (f < 8) { if (f < nj) b[ks][f] = *(const p256_frag_t*)(pb + tile_off(f) + kch[ks]); }
                    else a[ks][f - 8] = *(const p256_frag_t*)(pa + tile_off(f - 8) + kch[ks]);
                    if (r % 3 == 2) {
                        const int l = r / 3;
                        if (l < 4) load_one(st[0], slot_x, l);
                        else load_one(st[1], slot_y, l - 4);
                    }
                }
            }
            next(st[0], 0); next(st[1], 1);
            q4 = ring(q4 + 4);
            // The operands are here.  For the next phase: what group 0 requested a slice ago for group 1 (younger than that are
            // the other half of those eight requests and this phase's), and group 1's requests of a slice ago.
            asm volatile("s_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 .Lpp_r%=\n\ts_waitcnt vmcnt(8)\n.Lpp_r%=:\n\ts_waitcnt vmcnt(12) lgkmcnt(0)\n\ts_barrier" ::"s"(grp) : "memory", "scc");
            __builtin_amdgcn_sched_barrier(0);
            // product phase
            pp_each<2 * 4 * nj>([&](auto n) {
                constexpr int ks = n.value / (4 * nj), i = n.value / nj % 4, j = n.value % nj;
                pp_mfma<8 * i + j>(b[ks][j], a[ks][i]);
            });
            // For the next phase: group 0's own half of W, the last of its requests of a slice ago (group 1 has waited for its
            // own by now).  One statement with the barrier (none after an item's last slice): as branches of the loop
            // these would be laid out with copies of it.
            asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Lpp_w%=\n\ts_waitcnt vmcnt(8)\n.Lpp_w%=:\n\t"
                         "s_cmp_eq_u32 %1, 0\n\ts_cbranch_scc1 .Lpp_b%=\n\ts_barrier\n.Lpp_b%=:" ::"s"(grp), "s"(left - 1) : "memory", "scc");
            __builtin_amdgcn_sched_barrier(0);
        } while (--left);
    };
    // Epilogue of an item of class nj; accumulator (i, j)[v] is row 16 i + l16 of the wave's 64, column 16 j + 4 lq + v of
    // its group's half
    auto epilogue = [&](auto nj_tag, int q, int m0, int col_units) __attribute__((always_inline)) {
        constexpr int nj = decltype(nj_tag)::value;
        if constexpr (EPI == EPI_SWIGLU) {
            // silu(gate) * up from accumulator pairs (even j: gate, odd j: the same columns of up): a lane's four columns of
            // pair p, bf16, in two words.
            auto pair = [&](auto it, auto pt) __attribute__((always_inline)) {
                constexpr int t = 8 * it.value + 2 * pt.value;
                bf16x4 o;
                pp_each<4>([&](auto v) {
                    const float g = pp_read<4 * t + v.value>(), up = pp_read<4 * (t + 1) + v.value>();
                    // the hardware reciprocal (1 ulp) instead of an IEEE division: the result is rounded to bf16
                    o[v.value] = bf16_t(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * up);
                });
                u32x2 bits;
                __builtin_memcpy(&bits, &o, 8);
                return bits;
            };
            // Two pairs p, p + 1: lanes of lq 0 and 2 end up with eight columns of the first, 1 and 3 with eight of the second.
            auto two = [&](auto it, auto pt) __attribute__((always_inline)) {
                const u32x2 x = pair(it, pt), y = pair(it, std::integral_constant<int, pt.value + 1>{});
                const auto r0 = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false), r1 = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
                return u32x4{r0[0], r1[0], r0[1], r1[1]};
            };
            const int col = col_units * UNIT + grp * nj * 8 + 16 * (lq & 1) + 8 * (lq >> 1);
            pp_each<4>([&](auto it) {
                const int row = m0 + wm * 64 + 16 * it.value;
                if constexpr (ODD) {
                    pp_each<nj / 2>([&](auto pt) {
                        const u32x2 x = pair(it, pt);
                        const unsigned at = unsigned((row + l16) * N + col_units * UNIT + grp * nj * 8 + 16 * pt.value + 4 * lq) * 2u + 2u;
                        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)x[0], obuf, at, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b32(x[0] >> 16 | x[1] << 16, obuf, at + 2, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(x[1] >> 16), obuf, at + 6, 0, 0);
                    });
                    return;
                }
                const u32x4 x = two(it, std::integral_constant<int, 0>{});
                if constexpr (nj == 8) {   // whole 128-byte lines: eight rows in one store, the other eight in the next
                    const u32x4 y = two(it, std::integral_constant<int, 2>{});
                    u32x4 s0, s1;
                    pp_each<4>([&](auto v) {   // row_ror:8, lanes 8 to 15 and 0 to 7 of 16
                        s0[v.value] = __builtin_amdgcn_update_dpp(int(x[v.value]), int(y[v.value]), 0x128, 0xf, 0xc, false);
                        s1[v.value] = __builtin_amdgcn_update_dpp(int(y[v.value]), int(x[v.value]), 0x128, 0xf, 0x3, false);
                    });
                    const unsigned at = unsigned((row + (l16 & 7)) * N + col + 32 * (l16 >> 3)) * 2u;
                    __builtin_amdgcn_raw_buffer_store_b128(s0, obuf, at, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(s1, obuf, at + unsigned(8 * N) * 2u, 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b128(x, obuf, unsigned((row + l16) * N + col) * 2u, 0, 0);
                    if constexpr (nj == 6)
                        __builtin_amdgcn_raw_buffer_store_b64(pair(it, std::integral_constant<int, 2>{}), obuf,
                                                              unsigned((row + l16) * N + col_units * UNIT + grp * nj * 8 + 32 + 4 * lq) * 2u, 0, 0);
                }
            });
        } else {
            if constexpr (EPI == EPI_STORE_F32)   // a K range is stored as an output of its own
                obuf = __builtin_amdgcn_make_buffer_rsrc((float*)outv + size_t(q / n_tiles) * M * N, 0, int(size_t(M) * N * OUT_ELT), 0x00020000);
            // Two tiles side by side make whole 128-byte lines: eight rows of both in one store, the other eight in the next.
            const unsigned base = unsigned((m0 + wm * 64 + (l16 & 7)) * N + col_units * UNIT + grp * nj * 16 + 16 * (l16 >> 3) + 4 * lq) * 4u;
            pp_each<4>([&](auto band) {
                constexpr int i = band.value;
                // No scalar offset in the stores: the compiler then keeps the wait states between a 16-byte store and the next
                // write of its data registers, which the hardware needs with a scalar offset too (the accumulators read
                // right after it were stored in its place).
                const unsigned at = base + unsigned(i * 16 * N) * 4u, at8 = at + unsigned(8 * N) * 4u;
                u32x4 old[nj];
                if constexpr (EPI == EPI_RESIDUAL_F32) {   // all loads of a band of 16 rows in flight before the first add
#pragma unroll
                    for (int j = 0; j < nj; j += 2) {
                        old[j] = __builtin_amdgcn_raw_buffer_load_b128(obuf, at + j * 64, 0, 0);
                        old[j + 1] = __builtin_amdgcn_raw_buffer_load_b128(obuf, at8 + j * 64, 0, 0);
                    }
                }
                pp_each<nj / 2>([&](auto jt) {
                    constexpr int j = 2 * jt.value;
                    u32x4 x, y;
                    pp_each<4>([&](auto v) {
                        const int c0 = __float_as_int(pp_read<4 * (8 * i + j) + v.value>()), c1 = __float_as_int(pp_read<4 * (8 * i + j + 1) + v.value>());
                        x[v.value] = __builtin_amdgcn_update_dpp(c0, c1, 0x128, 0xf, 0xc, false);   // row_ror:8, lanes 8 to 15 of 16
                        y[v.value] = __builtin_amdgcn_update_dpp(c1, c0, 0x128, 0xf, 0x3, false);
                        if constexpr (EPI == EPI_RESIDUAL_F32) {
                            x[v.value] = __float_as_uint(__uint_as_float(x[v.value]) + __uint_as_float(old[j][v.value]));
                            y[v.value] = __float_as_uint(__uint_as_float(y[v.value]) + __uint_as_float(old[j + 1][v.value]));
                        }
                    });
                    __builtin_amdgcn_raw_buffer_store_b128(x, obuf, at + j * 64, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(y, obuf, at8 + j * 64, 0, 0);
                });
            });
        }
    };
    for (int u = 0; u < n_mine; ++u) {
        pp_each<128>([](auto r) { pp_clear<r.value>(); });
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7");
        __builtin_amdgcn_sched_barrier(0);
        const int q = item_of(u);
        int nj, m0, cu;
        tile_geom(q % n_tiles, &nj, &m0, &cu);
        const int nk = slices_of(q / n_tiles);
        auto item = [&](auto c) __attribute__((always_inline)) {
            k_loop(c, nk);
            // Group 0 writes its half while group 1 forms its last products, group 1 before it meets group 0 again.
            if (!grp) __builtin_amdgcn_s_barrier();
            // let the last MFMAs (four passes) retire before the accumulators are read
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15\n\ts_nop 15");
            __builtin_amdgcn_sched_barrier(0);
            epilogue(c, q, m0, cu);
        };
        if (nj == 8) item(std::integral_constant<int, 8>{});
        else if (nj == 6) item(std::integral_constant<int, 6>{});
        else item(std::integral_constant<int, 4>{});
        if (grp) __builtin_amdgcn_s_barrier();
    }
    if (!grp) __builtin_amdgcn_s_barrier();
    asm volatile("s_waitcnt vmcnt(0)");   // no load may still be on its way to LDS that is no longer this workgroup's
}


// A whole number of rounds over the CUs: every workgroup takes `rounds` items (the last may take one less).
template <int EPI, bool ODD = false>
static hipError_t launch_pp(const bf16_t* A, const bf16_t* W, const bf16_t* W2, void* out, int M, int N, int K, const P256Plan& plan,
                            int ks, hipStream_t st) {
    const int tiles_m = (M + 255) / 256, nb = tiles_m * (plan.n8 + plan.n6 + plan.n4) * ks;
    if (nb == 0 || (uintptr_t(out) & 3) != (ODD ? 2 : 0)) return hipErrorInvalidValue;
    const int rounds = (nb + 255) / 256, wgs = (nb + rounds - 1) / rounds;
    static bool attr_set = false;   // one flag per instantiation
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)gemm_pp_kernel<EPI, ODD>, hipFuncAttributeMaxDynamicSharedMemorySize, PP_LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_pp_kernel<EPI, ODD>), dim3(wgs), dim3(512), PP_LDS, st, A, W, W2, out, M, N, K, tiles_m, plan, rounds, ks);
    return hipGetLastError();
}

hipError_t launch_gemm_pp(int epi, const bf16_t* A, const bf16_t* W, const bf16_t* W2, void* out, int M, int N, int K,
                          const P256Plan& plan, int ks, hipStream_t st) {
    switch (epi) {
        case EPI_SWIGLU:
            if (uintptr_t(out) & 2) return launch_pp<EPI_SWIGLU, true>(A, W, W2, out, M, N, K, plan, 1, st);
            return launch_pp<EPI_SWIGLU>(A, W, W2, out, M, N, K, plan, 1, st);
        case EPI_RESIDUAL_F32: return launch_pp<EPI_RESIDUAL_F32>(A, W, W2, out, M, N, K, plan, 1, st);
        case EPI_STORE_F32: return launch_pp<EPI_STORE_F32>(A, W, W2, out, M, N, K, plan, ks, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace cake
