// What the two kernels for work items of 256 rows share: kernels_gemm.hip (four waves) and kernels_gemm_pp.hip (eight waves in
// turn).  Both add up a product in the same order, K from end to end in 32-deep MFMAs: their results are the same bits.
#pragma once
#include "gemm_tile.hpp"

namespace cake {

// Operand fragments are held as four 32-bit words (eight bf16 values along K).
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int p256_frag_t;

// Column panels.  The N dimension is cut into panels of 8, 6 or 4 MFMA tiles per wave (256, 192 or 128 rows of
// W; the widest first), so that the number of work items can be made a whole number of rounds over the CUs where
// 256-wide panels alone leave some idle (448 items on 256 CUs: 224 workgroups of two; with 64 panels of 256 and
// 64 of 192 every CU gets one item of each width, 7/8 of the time).  A work item is one panel x one band of 256
// rows of A (x one K range when K is split).
struct P256Plan { int n8, n6, n4; };

// kernels_gemm_pp.hip; out: on a whole element.  ks > 1 (float32 store): every K range an output of its own.
hipError_t launch_gemm_pp(int epi, const bf16_t* A, const bf16_t* W, const bf16_t* W2, void* out, int M, int N, int K,
                          const P256Plan& plan, int ks, hipStream_t st);

}  // namespace cake
