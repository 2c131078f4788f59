// Small memory-bound helpers around the attention block: norms, greedy sampling, pattern fill.
#include "kvpr_internal.h"
#include "silu.h"
#include <algorithm>
#include <cstdint>
#include <math.h>

namespace kvpr {
namespace {

__global__ void fill_u16_kernel(uint16_t* __restrict__ p, size_t n, uint16_t pattern) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = pattern;
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

// 8 consecutive halfs; callers' own tensors need not be 16-byte aligned
template <bool ALIGNED>
__device__ __forceinline__ half8 load8(const _Float16* p) {
    if constexpr (ALIGNED) return *reinterpret_cast<const half8*>(p);
    half8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[e];
    return v;
}
template <bool ALIGNED>
__device__ __forceinline__ void store8(_Float16* p, half8 v) {
    if constexpr (ALIGNED) {
        *reinterpret_cast<half8*>(p) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = v[e];
    }
}

// sum over a workgroup of up to 16 waves; red: 16 floats
__device__ __forceinline__ float block_sum(float v, float* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    return s;
}

// LayerNorm / RMSNorm (RMS): one workgroup per row, one 16-byte piece of the row per thread, float32 statistics.  The
// decode token has few rows, so the kernel is a chain of latencies and not of bytes: the row, the gains and the offsets
// are all asked for at once and kept in registers (pieces beyond kKeep per thread are read again), instead of three
// passes over the row of one half per lane.  4096 columns, one row: 11.9 -> 6.1 us on average in a decode step.
constexpr int kKeep = 2;
template <bool RMS, bool ALIGNED>
__global__ __launch_bounds__(1024) void norm_kernel(const _Float16* __restrict__ x, const _Float16* __restrict__ g,
                                                    const _Float16* __restrict__ b, _Float16* __restrict__ y, int h, float eps) {
    const _Float16* xr = x + (int64_t)blockIdx.x * h;
    _Float16* yr = y + (int64_t)blockIdx.x * h;
    const int pieces = h / 8, nt = blockDim.x;
    __shared__ float red[16];
    half8 xv[kKeep], gv[kKeep], bv[kKeep];
#pragma unroll
    for (int r = 0; r < kKeep; ++r) {
        const int at = threadIdx.x + r * nt;
        if (at < pieces) {
            xv[r] = load8<ALIGNED>(xr + at * 8);
            gv[r] = load8<ALIGNED>(g + at * 8);
            if constexpr (!RMS) bv[r] = load8<ALIGNED>(b + at * 8);
        }
    }
    // f(piece) over this thread's pieces of the row
    auto each = [&](auto&& f) {
#pragma unroll
        for (int r = 0; r < kKeep; ++r)
            if ((int)threadIdx.x + r * nt < pieces) f(xv[r]);
        for (int at = threadIdx.x + kKeep * nt; at < pieces; at += nt) f(load8<ALIGNED>(xr + at * 8));
    };
    float mean = 0.f, s = 0.f;
    if constexpr (!RMS) {
        each([&](half8 v) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s += (float)v[e];
        });
        mean = block_sum(s, red) / h;
        s = 0.f;
    }
    each([&](half8 v) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float d = (float)v[e] - mean;
            s += d * d;
        }
    });
    const float rstd = rsqrtf(block_sum(s, red) / h + eps);
    auto out = [&](int at, half8 v, half8 gg, half8 bb) {
        half8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float t = ((float)v[e] - mean) * rstd * (float)gg[e];
            o[e] = (_Float16)(RMS ? t : t + (float)bb[e]);
        }
        store8<ALIGNED>(yr + at * 8, o);
    };
#pragma unroll
    for (int r = 0; r < kKeep; ++r)
        if ((int)threadIdx.x + r * nt < pieces) out(threadIdx.x + r * nt, xv[r], gv[r], bv[r]);
    for (int at = threadIdx.x + kKeep * nt; at < pieces; at += nt) {
        half8 bb{};
        if constexpr (!RMS) bb = load8<ALIGNED>(b + at * 8);
        out(at, load8<ALIGNED>(xr + at * 8), load8<ALIGNED>(g + at * 8), bb);
    }
}

template <bool RMS>
int launch_norm(const void* x, const void* g, const void* b, void* y, int rows, int h, hipStream_t st) {
    const unsigned threads = (unsigned)std::min(1024, (h / 8 + 63) / 64 * 64);
    const bool aligned = (((uintptr_t)x | (uintptr_t)g | (uintptr_t)b | (uintptr_t)y) & 15) == 0;   // rows are multiples of 16 bytes
    auto kern = aligned ? norm_kernel<RMS, true> : norm_kernel<RMS, false>;
    hipLaunchKernelGGL(kern, dim3(rows), dim3(threads), 0, st, (const _Float16*)x, (const _Float16*)g, (const _Float16*)b,
                       (_Float16*)y, h, 1e-5f);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

// uniform pseudo-random halfs in [-scale, scale): data for the profiler's timing runs (real-looking
// operand bits keep MFMA power draw, and with it the clock, representative)
__global__ void fill_random_kernel(_Float16* __restrict__ p, size_t n, float scale, uint32_t seed) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        uint32_t v = (uint32_t)i * 2654435761u + seed;
        v ^= v >> 16; v *= 0x7feb352du; v ^= v >> 15; v *= 0x846ca68bu; v ^= v >> 16;
        p[i] = (_Float16)(((float)(v >> 8) * (1.0f / 8388608.0f) - 1.0f) * scale);
    }
}

// Greedy sampling, and the embedding row of the token it gives (table may be null): one workgroup per row, lowest index
// wins ties.  One row of 50272 logits is 200 KB for one compute unit, so what counts is bytes in flight: 1024 threads with
// four 16-byte loads each instead of 256 with one of 4 bytes; the gather, which was a launch of its own, follows in the
// same workgroup.  One row of 50272: 53 us, and 8.5 for the gather -> 9.9.
// wide: rows of logits start at multiples of 16 bytes; wide_rows: so do rows of the table and of the output.
__global__ __launch_bounds__(1024) void argmax_gather_kernel(const float* __restrict__ logits, int N, int32_t* __restrict__ tokens,
                                                             const _Float16* __restrict__ table, _Float16* __restrict__ x_next, int h,
                                                             int wide, int wide_rows) {
    const float* row = logits + (int64_t)blockIdx.x * N;
    constexpr int NT = 1024, U = 4;
    const int tid = threadIdx.x;
    float best = -INFINITY;
    int bi = 0x7fffffff;
    auto take = [&](float v, int i) {
        if (v > best || (v == best && i < bi)) { best = v; bi = i; }
    };
    int done = 0;                                      // logits [0, done) were read in pieces of 4
    if (wide) {
        const int pieces = N / 4;
        const float4v* p = reinterpret_cast<const float4v*>(row);
        for (int at = tid; at < pieces; at += NT * U) {
            float4v v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p[min(at + u * NT, pieces - 1)];   // clamped ones count twice, which changes nothing
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) take(v[u][e], min(at + u * NT, pieces - 1) * 4 + e);
        }
        done = pieces * 4;
    }
    for (int i = done + tid; i < N; i += NT) take(row[i], i);
    __shared__ float sv[16];
    __shared__ int si[16];
    for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o), __shfl_xor(bi, o));
    if ((tid & 63) == 0) { sv[tid >> 6] = best; si[tid >> 6] = bi; }
    __syncthreads();
    best = sv[0];
    bi = si[0];
    for (int w = 1; w < NT / 64; ++w) take(sv[w], si[w]);
    if (best == -INFINITY) bi = 0x7fffffff;            // nothing above -inf (or only NaN): no token ...
    if (tid == 0) tokens[blockIdx.x] = bi;
    if (!table) return;
    _Float16* out = x_next + (int64_t)blockIdx.x * h;
    if (bi >= N) {                                     // ... and no embedding
        for (int i = tid; i < h; i += NT) out[i] = (_Float16)0.f;
        return;
    }
    const _Float16* src = table + (int64_t)bi * h;
    if (wide_rows)
        for (int i = tid; i < h / 8; i += NT) *reinterpret_cast<half8*>(out + i * 8) = *reinterpret_cast<const half8*>(src + i * 8);
    else
        for (int i = tid; i < h; i += NT) out[i] = src[i];
}

// gated FFN middle: gu [rows, 2f] = [gate | up]  ->  y [rows, f] = silu(gate) * up
__global__ void silu_mul_kernel(const _Float16* __restrict__ gu, _Float16* __restrict__ y, int f, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t row = i / f, col = i - row * f;
    y[i] = (_Float16)silu_mul((float)gu[row * 2 * f + col], (float)gu[row * 2 * f + f + col]);
}

// rotary embedding of the decode token: qk [batch, 2h] float32 = [q | k] before rotation, position `pos` for
// every sequence; q goes out as float32 [batch, h], k as float16 with row stride ldk (a row of the cache).
// One thread per (row, pair): element i of a head pairs with element i + HD/2.
__global__ void rope_token_kernel(const float* __restrict__ qk, const float2* __restrict__ table, int pos, int h, int hd,
                                  float* __restrict__ q_out, _Float16* __restrict__ k_out, int64_t ldk, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int half_h = h / 2, half_d = hd / 2;
    const size_t row = i / half_h;
    const int p = (int)(i - row * half_h);
    const int head = p / half_d, f = p - head * half_d;
    const int c1 = head * hd + f, c2 = c1 + half_d;
    const float2 cs = table[(size_t)pos * half_d + f];
    const float* qr = qk + row * 2 * h;
    const float q1 = qr[c1], q2 = qr[c2], k1 = qr[h + c1], k2 = qr[h + c2];
    q_out[row * h + c1] = q1 * cs.x - q2 * cs.y;
    q_out[row * h + c2] = q2 * cs.x + q1 * cs.y;
    k_out[row * ldk + c1] = (_Float16)(k1 * cs.x - k2 * cs.y);
    k_out[row * ldk + c2] = (_Float16)(k2 * cs.x + k1 * cs.y);
}

}  // namespace

int launch_rmsnorm(const void* x, const void* g, void* y, int rows, int h, hipStream_t st) {
    return launch_norm<true>(x, g, nullptr, y, rows, h, st);
}

int launch_silu_mul(const void* gu, void* y, int rows, int f, hipStream_t st) {
    const size_t n = (size_t)rows * f;
    hipLaunchKernelGGL(silu_mul_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const _Float16*)gu, (_Float16*)y, f, n);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int launch_rope_token(const void* qk32, const void* table, int pos, int batch, int h, int head_dim, void* q32, void* k16,
                      int64_t ldk, hipStream_t st) {
    const size_t n = (size_t)batch * (h / 2);
    hipLaunchKernelGGL(rope_token_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const float*)qk32,
                       (const float2*)table, pos, h, head_dim, (float*)q32, (_Float16*)k16, ldk, n);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int launch_argmax_gather(const float* logits, int M, int N, int32_t* tokens, const void* table, void* x_next, int h, hipStream_t st) {
    const int wide = N % 4 == 0 && ((uintptr_t)logits & 15) == 0;
    const int wide_rows = h % 8 == 0 && (((uintptr_t)table | (uintptr_t)x_next) & 15) == 0;
    hipLaunchKernelGGL(argmax_gather_kernel, dim3(M), dim3(1024), 0, st, logits, N, tokens, (const _Float16*)table, (_Float16*)x_next,
                       h, wide, wide_rows);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int launch_fill_u16(void* p, size_t n_halfs, uint16_t pattern, hipStream_t st) {
    if (n_halfs == 0) return KVPR_OK;
    size_t blocks = (n_halfs + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u16_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (uint16_t*)p, n_halfs, pattern);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int launch_fill_random(void* p, size_t n_halfs, float scale, uint32_t seed, hipStream_t st) {
    if (n_halfs == 0) return KVPR_OK;
    size_t blocks = (n_halfs + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(fill_random_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (_Float16*)p, n_halfs, scale, seed);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int launch_layernorm(const void* x, const void* g, const void* b, void* y, int rows, int h, hipStream_t st) {
    return launch_norm<false>(x, g, b, y, rows, h, st);
}

// plain copy of up to two ranges, one launch for both: the new K|V row and the new activation row of a layer go to the host
// together, and each launch is about 4 us of a call that launches bound
__global__ void copy_kernel(CopyJob job) { run_copy_job(job, blockIdx.x); }

int launch_copy(const CopyJob& job, int threads, hipStream_t st) {
    if (job.blocks == 0) return KVPR_OK;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)job.blocks), dim3((unsigned)threads), 0, st, job);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

// At most 64 workgroups of 256 lanes, 256 KiB on the way: more of them only crowd the link (single-layer calls in a row / waited
// for, cache alone, 512 / 256 / 64 workgroups: hidden 4096, batch 10, 1.6 MiB 85 / 80 / 77 and 108 / 103 / 95 us; hidden 768, batch 8,
// 1.4 MiB 76 / 72 / 68 and 86 / 82 / 80).
constexpr int kCopyBytesThreads = 256, kCopyBytesBlocks = 64;

int launch_copy_bytes(const void* src, void* dst, size_t bytes, hipStream_t st, const void* src2, void* dst2, size_t bytes2) {
    return launch_copy(copy_job(kCopyBytesThreads, src, dst, bytes, src2, dst2, bytes2, kCopyBytesBlocks), kCopyBytesThreads, st);
}

}  // namespace kvpr

// for tests: workgroups of launch_copy_bytes
extern "C" int kvpr_debug_copy_workgroups(size_t bytes, size_t bytes2) {
    return kvpr::copy_job(kvpr::kCopyBytesThreads, nullptr, nullptr, bytes, nullptr, nullptr, bytes2, kvpr::kCopyBytesBlocks).blocks;
}
