// Token GEMM for at most 8 rows (gemm_few.hip).
#pragma once
#include "kvpr_internal.h"

namespace kvpr {

bool takes_few_tokens(int M, int N, int K);   // launch_few_tokens is the kernel for this product

// y[M, N] = x[M, K] . W[N, K]^T + bias, K a multiple of 128: the first out_f32_cols features as float32 to y32
// [M, out_f32_cols], the others as float16 to y16 (row stride ld16), with a residual laid out as y16 added if there is one
struct FewTokens {
    const _Float16 *x, *W, *bias;
    float* y32;
    _Float16* y16;
    const _Float16* res;
    int64_t ld16;
    int M, N, K, out_f32_cols, relu;
};

// gated: W is [gate; up] of N / 2 features each (a multiple of 4), y16 [M, N / 2] = silu(x gate^T) * (x up^T); nothing else applies
int launch_few_tokens(const FewTokens& a, bool gated, hipStream_t st, const CopyJob& beside = CopyJob());

}  // namespace kvpr
