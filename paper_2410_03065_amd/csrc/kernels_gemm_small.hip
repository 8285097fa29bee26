// bf16 MFMA GEMMs that leave K ranges for their consumer to add up: out[range][M][N] float32.  The products in front of
// an RMSNorm (O, down) and of the rotary step (QKV) end in a kernel that reads their result anyway; where K has to be
// divided to fill the chip, that kernel adds the ranges as it reads, instead of the last workgroup of a tile (device
// scope stores, a ticket and a read-back: 10 us and more per launch) or a pass of its own.
//
// Few rows (up to 192: the products of a serving step's share of a short prompt, of a ragged last chunk): the weights
// are the work and come from HBM once.  One tile takes all rows (BM = M rounded up to 32; the tiles of whole chunks have
// 128 or 256) by 128 rows of W, the four waves side by side along N, in a ring that fills the CU's LDS (up to eight
// slices of 64).
#include <algorithm>

#include "gemm_tile.hpp"

namespace cake {

namespace {

constexpr int stages_of(int bm, int bn) { return std::min(8, 160 * 1024 / ((bm + bn) * 128)); }   // slices of 64 that fit the LDS

template <int WTM>
hipError_t launch_tile(const bf16_t* A, const bf16_t* W, float* part, int M, int N, int K, hipStream_t st, int ks) {
    return gemm_launch_t<WTM, 1, 1, 4, 64, stages_of(32 * WTM, 128), EPI_STORE_F32>(A, W, nullptr, part, M, N, K, st, ks, nullptr, true);
}

}  // namespace

hipError_t launch_gemm_rows_parts(const void* a, const void* w, float* part, int M, int N, int K, int ks, hipStream_t st) {
    const bf16_t *A = (const bf16_t*)a, *W = (const bf16_t*)w;
    if (M <= 0 || N <= 0 || K <= 0 || N % 128 || K % (64 * ks)) return hipErrorInvalidValue;
    switch ((M + 31) / 32) {
        case 1: return launch_tile<1>(A, W, part, M, N, K, st, ks);
        case 2: return launch_tile<2>(A, W, part, M, N, K, st, ks);
        case 3: return launch_tile<3>(A, W, part, M, N, K, st, ks);
        case 4: return launch_tile<4>(A, W, part, M, N, K, st, ks);
        case 5: return launch_tile<5>(A, W, part, M, N, K, st, ks);
        case 6: return launch_tile<6>(A, W, part, M, N, K, st, ks);
    }
    return hipErrorInvalidValue;
}

}  // namespace cake
