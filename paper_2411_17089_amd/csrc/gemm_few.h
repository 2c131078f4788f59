// Token GEMM for at most 8 rows (gemm_few.hip).
#pragma once
#include "kvpr_internal.h"

namespace kvpr {

bool takes_few_tokens(int M, int N, int K);   // launch_few_tokens is the kernel for this product by itself
bool few_tokens_along(int M, int N, int K);   // ... for this product with copies, the rotation or the gate along
bool few_tokens_norm(int M, int N, int K);    // ... and with a norm in front

// y[M, N] = x[M, K] . W[N, K]^T + bias, K a multiple of 128: the first out_f32_cols features as float32 to y32
// [M, out_f32_cols], the others as float16 to y16 (row stride ld16), with a residual laid out as y16 added if there is one
struct FewTokens {
    const _Float16 *x, *W, *bias;
    float* y32;
    _Float16* y16;
    const _Float16* res;
    int64_t ld16;
    int M, N, K, out_f32_cols, relu;
    // norm: x goes through LayerNorm (1) or RMSNorm (2) first, gains and offsets of K halfs; the normalised rows also go to xn if
    // it is not null
    int norm = 0;
    const _Float16 *norm_g = nullptr, *norm_b = nullptr;
    _Float16* xn = nullptr;
    // rotary form: (cos, sin) of the rows' position, head_dim / 2 pairs
    const float2* rope = nullptr;
    int head_dim = 0;
    // the kernels behind read (most of) W again
    bool w_again = false;
};

// Plain.  Gated: W is [gate; up] of N / 2 features each (a multiple of 4), y16 [M, N / 2] = silu(x gate^T) * (x up^T), no bias,
// residual or ReLU.  Rotary: W is [q; k; v] of N / 3 features each, in heads of head_dim; q and k are rotated, q goes to y32.
enum class FewForm { plain, gated, rotary };

int launch_few_tokens(const FewTokens& a, FewForm form, hipStream_t st, const CopyJob& beside = CopyJob());

}  // namespace kvpr
