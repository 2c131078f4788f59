// Group-wise 4-bit codec for the host store (Sec. 4.4 "KV Cache Compression").
//
// The paper names the scheme without fixing a format; this library's format is:
//   - a group is 64 consecutive columns of one row (a [K|V] row of one sequence, or an activation row);
//   - mn = min(group), mx = max(group) (float16 values, exact), scale = float16((mx - mn) / 15);
//     code = clamp(rint((x - mn) / scale), 0, 15), all in float32 with IEEE division and
//     round-half-to-even; a group with scale == 0 has all codes 0;
//   - dequantised value = float16(code * scale + mn) (code * scale is exact in float32);
//   - a packed row of C columns is C/2 code bytes (element 2k in the low nibble of byte k, 2k+1 in
//     the high nibble) followed by C/64 pairs (scale, mn) of float16: 9C/16 bytes.
//
// Both kernels stream.  Packing was bound by its arithmetic (two IEEE divisions per 8 values and one per value: 205 us for
// 32768 rows of 8192, 3.4 TB/s), so a lane takes 16 values, the group is 4 lanes, and the divisions are a product with the
// reciprocal and one remainder step, which gives the correctly rounded quotient here (see quotient()).  Unpacking takes 8
// values a lane so that its 16-byte stores are contiguous over the wave.  Rows are found with a 32-bit multiplication.
// Packing and unpacking those rows together: 296 -> 241 us, 5.7 TB/s of the 1.38 GB moved.
#include "kvpr_internal.h"

namespace kvpr {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned int word2 __attribute__((ext_vector_type(2), aligned(4)));   // packed rows are multiples of 4 bytes only

constexpr int QUANT_PIECES = 2, DEQUANT_PIECES = 4;     // independent pieces of 16 / 8 values a thread has in flight

// index / per_row for index < 2^31: (index * mul) >> (32 + shift), mul = ceil(2^(32 + shift) / per_row)
struct RowOf {
    uint32_t mul, shift, per_row;
    __device__ uint32_t operator()(uint32_t index) const { return __umulhi(index, mul) >> shift; }
};

// The correctly rounded a / b for |b| of at most 11 significant bits, r = 1 / b to an ulp or two, nothing under- or
// overflowing.  a - q b is exact, so the sum before its rounding is off by about 2^-22 units in the last place, while a
// quotient by 11 bits that is no midpoint between two floats is at least 2^-12 away from one; none is a midpoint.
__device__ __forceinline__ float quotient(float a, float b, float r) {
    const float q = a * r;
    return fmaf(fmaf(-q, b, a), r, q);
}

template <int CTRL>
__device__ __forceinline__ float across(float v) {       // the value of another lane of the same row of 16
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// 16 codes of one lane's values v[0..15] with the group's scale and minimum
__device__ __forceinline__ word2 codes16(const half8 v[2], float scale, float mn) {
    word2 w = {0, 0};
    if (!(scale > 0.f)) return w;
    const float r = __builtin_amdgcn_rcpf(scale);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float part[2];                                   // four codes each as one number below 2^16
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float c[4];
#pragma unroll
            // a NaN (a NaN value, or an infinite scale) gives code 0: fmed3 returns the smallest of its numbers then
            for (int e = 0; e < 4; ++e)
                c[e] = rintf(__builtin_amdgcn_fmed3f(quotient((float)v[i][4 * j + e] - mn, scale, r), 0.f, 15.f));
            part[j] = fmaf(fmaf(c[3], 16.f, c[2]), 256.f, fmaf(c[1], 16.f, c[0]));
        }
        w[i] = (uint32_t)part[0] | (uint32_t)part[1] << 16;
    }
    return w;
}

__global__ __launch_bounds__(256) void quant_int4_kernel(const _Float16* __restrict__ src, uint8_t* __restrict__ dst,
                                                         uint32_t n, RowOf row_of, int packed_row_bytes) {
    const uint32_t t0 = blockIdx.x * (256u * QUANT_PIECES) + threadIdx.x;
    half8 v[QUANT_PIECES][2];
#pragma unroll
    for (int u = 0; u < QUANT_PIECES; ++u) {
        const uint32_t t = t0 + u * 256u;
        const half8* p = reinterpret_cast<const half8*>(src) + (size_t)(t < n ? t : 0) * 2;
        v[u][0] = __builtin_nontemporal_load(p);
        v[u][1] = __builtin_nontemporal_load(p + 1);
    }
#pragma unroll
    for (int u = 0; u < QUANT_PIECES; ++u) {
        const half8 lo = __builtin_elementwise_min(v[u][0], v[u][1]), hi = __builtin_elementwise_max(v[u][0], v[u][1]);
        float mn = (float)lo[0], mx = (float)hi[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            mn = fminf(mn, (float)lo[i]);
            mx = fmaxf(mx, (float)hi[i]);
        }
        // quad_perm [1,0,3,2] and [2,3,0,1]: the 4 lanes of the group (n is a multiple of 4, they live together)
        mn = fminf(mn, across<0xB1>(mn)); mx = fmaxf(mx, across<0xB1>(mx));
        mn = fminf(mn, across<0x4E>(mn)); mx = fmaxf(mx, across<0x4E>(mx));
        const float range = mx - mn;
        const float step = fabsf(range) < INFINITY ? quotient(range, 15.f, 1.f / 15.f) : range;
        const _Float16 scale16 = (_Float16)step;
        const word2 w = codes16(v[u], (float)scale16, mn);
        const uint32_t t = t0 + u * 256u;
        if (t >= n) continue;
        const uint32_t row = row_of(t), j = t - row * row_of.per_row;
        uint8_t* out = dst + (size_t)row * packed_row_bytes;
        *reinterpret_cast<word2*>(out + j * 8) = w;
        if ((j & 3) == 0) {
            union { _Float16 h[2]; uint32_t u; } meta;
            meta.h[0] = scale16;
            meta.h[1] = (_Float16)mn;
            *reinterpret_cast<uint32_t*>(out + row_of.per_row * 8 + j) = meta.u;
        }
    }
}

__global__ __launch_bounds__(256) void dequant_int4_kernel(const uint8_t* __restrict__ src, _Float16* __restrict__ dst,
                                                           uint32_t n, RowOf row_of, int packed_row_bytes) {
    const uint32_t t0 = blockIdx.x * (256u * DEQUANT_PIECES) + threadIdx.x;
    uint32_t word[DEQUANT_PIECES];
    union { _Float16 h[2]; uint32_t u; } meta[DEQUANT_PIECES];
#pragma unroll
    for (int u = 0; u < DEQUANT_PIECES; ++u) {
        const uint32_t t = t0 + u * 256u < n ? t0 + u * 256u : 0;
        const uint32_t row = row_of(t), j = t - row * row_of.per_row;
        const uint8_t* in = src + (size_t)row * packed_row_bytes;
        word[u] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(in + j * 4));
        meta[u].u = *reinterpret_cast<const uint32_t*>(in + row_of.per_row * 4 + (j >> 3) * 4);
    }
#pragma unroll
    for (int u = 0; u < DEQUANT_PIECES; ++u) {
        const uint32_t t = t0 + u * 256u;
        if (t >= n) continue;
        const float scale = (float)meta[u].h[0], mn = (float)meta[u].h[1];
        half8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (_Float16)((float)((word[u] >> (4 * i)) & 15u) * scale + mn);
        *reinterpret_cast<half8*>(dst + (size_t)t * 8) = v;
    }
}

// launch(first row, pieces, RowOf): one launch per run of rows whose pieces of `values` columns can be counted in 31 bits
template <class F>
int for_row_runs(int64_t rows, int cols, int values, F launch) {
    RowOf row_of{0, 0, (uint32_t)(cols / values)};
    if (row_of.per_row < 4) return KVPR_OK;              // fewer columns than a group
    uint32_t log2 = 0;
    while ((1u << log2) < row_of.per_row) ++log2;        // 2 or more
    row_of.shift = log2 - 1;
    row_of.mul = (uint32_t)(((1ull << (31 + log2)) + row_of.per_row - 1) / row_of.per_row);
    const int64_t run = 0x7FFF0000u / row_of.per_row;
    for (int64_t r = 0; r < rows; r += run) {
        launch(r, (uint32_t)((rows - r < run ? rows - r : run) * row_of.per_row), row_of);
        KVPR_HIP(hipGetLastError());
    }
    return KVPR_OK;
}

}  // namespace

size_t int4_row_bytes(int cols) { return (size_t)cols / 2 + (size_t)cols / 16; }

int launch_quant_int4(const void* src, void* dst, int64_t rows, int cols, hipStream_t st) {
    const size_t packed = int4_row_bytes(cols);
    return for_row_runs(rows, cols, 16, [&](int64_t r, uint32_t n, RowOf row_of) {
        const unsigned grid = (n + 256u * QUANT_PIECES - 1) / (256u * QUANT_PIECES);
        hipLaunchKernelGGL(quant_int4_kernel, dim3(grid), dim3(256), 0, st, (const _Float16*)src + (size_t)r * cols,
                           (uint8_t*)dst + (size_t)r * packed, n, row_of, (int)packed);
    });
}

int launch_dequant_int4(const void* src, void* dst, int64_t rows, int cols, hipStream_t st) {
    const size_t packed = int4_row_bytes(cols);
    return for_row_runs(rows, cols, 8, [&](int64_t r, uint32_t n, RowOf row_of) {
        const unsigned grid = (n + 256u * DEQUANT_PIECES - 1) / (256u * DEQUANT_PIECES);
        hipLaunchKernelGGL(dequant_int4_kernel, dim3(grid), dim3(256), 0, st, (const uint8_t*)src + (size_t)r * packed,
                           (_Float16*)dst + (size_t)r * cols, n, row_of, (int)packed);
    });
}

}  // namespace kvpr
