// Copies of a few rows between device memory and mapped pinned host memory, as a kernel of their own or as extra workgroups of
// a launch that is going out anyway.  Beside a launch they cost what they take over the link, if that; alone they are a launch
// more in a chain of launches, 4 us each.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace kvpr {

struct CopyRange {
    const unsigned char* src;
    unsigned char* dst;
    size_t bytes;
};

// blocks = 0: nothing to copy
struct CopyJob {
    CopyRange a{nullptr, nullptr, 0}, b{nullptr, nullptr, 0};
    int blocks = 0, width = 16;      // workgroups, bytes a lane moves at a time
    int blocks_a = 0;                // the first ones copy a and the others b, at the same time; 0: all of them a, then b
};

// width: the widest piece all pointers are aligned to (packed 4-bit rows are multiples of 8 bytes, not always of 16; a
// caller's tensor may start anywhere).  threads: of the workgroups that will run it.  64 of 512 lanes have 512 KiB on the
// way, four times what the link takes in the 2 us to its first byte.
inline CopyJob copy_job(int threads, const void* src, void* dst, size_t bytes, const void* src2 = nullptr, void* dst2 = nullptr,
                        size_t bytes2 = 0, int most = 64) {
    CopyJob j;
    j.a = {(const unsigned char*)src, (unsigned char*)dst, bytes};
    if (bytes2) j.b = {(const unsigned char*)src2, (unsigned char*)dst2, bytes2};
    uintptr_t all = (uintptr_t)j.b.src | (uintptr_t)j.b.dst;
    if (bytes) all |= (uintptr_t)src | (uintptr_t)dst;
    j.width = (all & 15) == 0 ? 16 : (all & 7) == 0 ? 8 : (all & 3) == 0 ? 4 : 1;
    const size_t per = (size_t)threads * 16, n = (bytes + bytes2 + per - 1) / per;
    j.blocks = (int)(n < (size_t)most ? n : most);
    return j;
}

// Two ranges that cross the link in opposite directions, each with workgroups of its own, of 512 lanes.  Beside a product 32 in
// and 8 out: writes need few (8 alone 53 of the 56 GB/s that 16 reach), and more of them hold the reads back (a prefill of 512
// positions, batch 8, hidden 4096 with 8 / 16 / 32 out: 1.60 / 1.65 / 1.70 ms; with 4: 1.88).
inline CopyJob copy_both_ways(const void* in, void* in_to, size_t in_bytes, const void* out, void* out_to, size_t out_bytes) {
    const CopyJob i = copy_job(512, in, in_to, in_bytes, nullptr, nullptr, 0, 32), o = copy_job(512, out, out_to, out_bytes, nullptr, nullptr, 0, 8);
    if (i.blocks == 0) return o;
    if (o.blocks == 0) return i;
    CopyJob j;
    j.a = i.a;
    j.b = o.a;
    j.blocks_a = i.blocks;
    j.blocks = i.blocks + o.blocks;
    j.width = i.width < o.width ? i.width : o.width;
    return j;
}

template <class T>
__device__ __forceinline__ void copy_range(const CopyRange& r, size_t first, size_t stride) {
    const size_t n = r.bytes / sizeof(T);
    for (size_t i = first; i < n; i += stride) reinterpret_cast<T*>(r.dst)[i] = reinterpret_cast<const T*>(r.src)[i];
    for (size_t i = n * sizeof(T) + first; i < r.bytes; i += stride) r.dst[i] = r.src[i];
}

// the share of workgroup `block` of j.blocks
__device__ __forceinline__ void run_copy_job(const CopyJob& j, int block) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const size_t first = (size_t)block * blockDim.x + threadIdx.x, stride = (size_t)j.blocks * blockDim.x;
    auto both = [&](auto piece) {
        using T = decltype(piece);
        if (j.blocks_a) {
            if (block < j.blocks_a) copy_range<T>(j.a, first, (size_t)j.blocks_a * blockDim.x);
            else copy_range<T>(j.b, first - (size_t)j.blocks_a * blockDim.x, (size_t)(j.blocks - j.blocks_a) * blockDim.x);
            return;
        }
        copy_range<T>(j.a, first, stride);
        // the second range starts with the lanes that the first one has left over
        const size_t used = (j.a.bytes / sizeof(T)) % stride;
        copy_range<T>(j.b, first >= used ? first - used : first + stride - used, stride);
    };
    if (j.width == 16) both(u4{});
    else if (j.width == 8) both(u2{});
    else if (j.width == 4) both(0u);
    else both((unsigned char)0);
}

}  // namespace kvpr
