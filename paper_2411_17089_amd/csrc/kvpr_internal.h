// Internal declarations shared by the translation units of libkvpr (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "copy_job.h"
#include "kvpr.h"

namespace kvpr {

// error plumbing: records text for kvpr_last_error() and returns `code`
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
#define KVPR_HIP(call)                                                                    \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess)                                                             \
            return ::kvpr::fail(KVPR_E_HIP, "%s failed: %s (%s:%d)", #call,               \
                                hipGetErrorString(e_), __FILE__, __LINE__);               \
    } while (0)

int compute_units();   // of the current device, read once

// kernels (each validates nothing: callers check shapes first)
int64_t gemm_workgroups(int64_t M, int N);   // that launch_gemm and launch_gemm_rope make of a product
double gemm_estimate_s(int64_t M, int N, int K);   // how long, to about a tenth
// `beside`: copies by extra workgroups of the launch, whose results the launch itself does not read
int launch_gemm(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K,
                int64_t ldc, hipStream_t st, const CopyJob& beside = CopyJob());
int launch_attention(const void* q, const void* kv, void* z, void* ws, int S, int batch, int hidden,
                     int n_heads, hipStream_t st, const CopyJob& beside = CopyJob());
size_t attention_workspace_bytes(int batch, int hidden, int n_heads, int S);
int launch_attention_mixed(const void* q, const void* kv16, const void* kvq, void* z, void* ws, int S, int split, int batch,
                           int hidden, int n_heads, int phase, hipStream_t st, const CopyJob& beside = CopyJob());
// A norm in front of a token GEMM, which then reads xn = norm(x) instead of its x: LayerNorm with offsets b, RMSNorm without.
// keep: the normalised rows are needed in xn afterwards.
struct TokenNorm {
    const void *x, *g, *b;
    void* xn;
    bool keep;
};
bool norm_goes_along(const TokenNorm& n, int M, int N, int K);     // in the product's own launch; else in one in front of it
int launch_norm(const TokenNorm& n, int rows, int h, hipStream_t st);
int launch_token_gemm_flags(const void* x, const void* w, const void* bias, void* y32, void* y16, int M, int N,
                            int K, int out_f32_cols, int64_t ld16, int flags /*bit 0: ReLU, 1: as with something along, 2: W is read again*/, hipStream_t st,
                            void* ws = nullptr, size_t ws_bytes = 0, const void* residual = nullptr, const CopyJob& beside = CopyJob(),
                            const TokenNorm* norm = nullptr);
int launch_token_qkv_rope(const void* x, const void* w, const void* bias, void* qk32, void* q32, void* kv16, int M, int h, int head_dim,
                          const void* table, int pos, hipStream_t st, void* ws, size_t ws_bytes, const CopyJob& beside = CopyJob(),
                          const TokenNorm* norm = nullptr, bool w_again = false);
int launch_token_gemm_gated(const void* x, const void* w, void* mid, void* y, int M, int f, int K, hipStream_t st, void* ws,
                            size_t ws_bytes, const TokenNorm* norm = nullptr);
size_t token_gemm_workspace_bytes(int M, int N);
int launch_fill_u16(void* p, size_t n_halfs, uint16_t pattern, hipStream_t st);
int launch_fill_random(void* p, size_t n_halfs, float scale, uint32_t seed, hipStream_t st);
int launch_layernorm(const void* x, const void* g, const void* b, void* y, int rows, int h, hipStream_t st);
int launch_argmax_gather(const float* logits, int M, int N, int32_t* tokens, const void* table, void* x_next, int h, hipStream_t st);
int launch_gemm_rope(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K, int64_t ldc,
                     const void* table, int rope_cols, int head_dim, int batch, int pos0, hipStream_t st, const CopyJob& beside = CopyJob());
int launch_rmsnorm(const void* x, const void* g, void* y, int rows, int h, hipStream_t st);
int launch_silu_mul(const void* gu, void* y, int rows, int f, hipStream_t st);
int launch_rope_token(const void* qk32, const void* table, int pos, int batch, int h, int head_dim, void* q32, void* k16,
                      int64_t ldk, hipStream_t st);
size_t int4_row_bytes(int cols);
int launch_quant_int4(const void* src, void* dst, int64_t rows, int cols, hipStream_t st);
int launch_dequant_int4(const void* src, void* dst, int64_t rows, int cols, hipStream_t st);
constexpr int kCopyThreads = 512;     // of the workgroups of the GEMM tiles and of the token GEMM that take copies along
int launch_copy(const CopyJob& job, int threads, hipStream_t st);
int launch_copy_bytes(const void* src, void* dst, size_t bytes, hipStream_t st, const void* src2 = nullptr, void* dst2 = nullptr,
                      size_t bytes2 = 0);
int launch_keep_warm(const void* w, size_t n_w, double seconds, double wall_clock_hz, void* sink, hipStream_t st);

}  // namespace kvpr
