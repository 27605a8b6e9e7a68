// Problem statement and arguments shared by the grouped GEMMs (gemm2.hpp: bf16;
// gemm_f32.hpp: fp32; gfx950 MFMA, persistent blocks on an XCD-aware tile schedule).
//
// C[m][n] = sum_k A[m][k] * B[n][k] for every group (expert) e:
//   GROUP_M: the m range is expert e's rows [offsets[e], offsets[e+1]) (tokens);
//            K and N are fixed; A rows are K-contiguous; B is expert e's weight,
//            K-contiguous ([N][K], nn.Linear) or N-contiguous ([K][N]).
//   GROUP_K: the k range is expert e's rows (tokens); M and N are fixed; A and B
//            are both stored row-per-token ([K][M] and [K][N]); C is expert e's
//            weight gradient [M][N].
// The MFMA's first operand takes the B tile (n) and its second the A tile (m),
// so each lane's accumulator holds 4 consecutive n of one m: 8/16-byte stores.
#pragma once

#include "common.hpp"

namespace dmoe {

enum GroupMode { GROUP_M = 0, GROUP_K = 1 };
// EPI_SGD: C holds parameters; C <- C - lr * (A^T B) (the gradient is not stored)
enum Epilogue { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_ACT = 2, EPI_DACT = 3, EPI_SGD = 5 };

template <typename E>
struct GemmArgs {
  const E* A; int64_t lda;
  const E* B; int64_t ldb; int64_t b_gstride;      // GROUP_M: elements between experts' B
  void* C; int64_t ldc; int64_t c_gstride;         // GROUP_K: elements between experts' C
  void* C2;                                        // EPI_BIAS_ACT: activation output
  const E* bias; int64_t bias_gstride;             // EPI_BIAS*: per-expert bias [N]
  const E* aux;                                    // EPI_DACT: pre-activation, layout of C
  const int32_t* offsets;                          // [groups+1]
  const int32_t* tprefix;                          // [groups+1] prefix of tile units
  int tscale;                                      // tiles per unit of tprefix
  int groups;
  int M, N, K;                                     // fixed dims (M unused for GROUP_M, K for GROUP_K)
  int act;
  int chunked;                                     // XCD-chunked schedule (grid >= 8)
  float lr;                                        // EPI_SGD: step size
};

}  // namespace dmoe
