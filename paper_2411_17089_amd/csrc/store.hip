// Host store (Sec. 3.3 "pinned memory"): writing rows, borrowing the pinned arrays, and the prefill stand-in.
#include "context.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

using kvpr::fail;
using kvpr::check_weights;

extern "C" int kvpr_store_write(kvpr_ctx* c, int layer, int t0, int t1, const void* x_host, const void* kv_host) {
    if (!c) return fail(KVPR_E_INVAL, "ctx is null");
    if (layer < 0 || layer >= c->slots()) return fail(KVPR_E_RANGE, "layer %d outside [0, %d)", layer, c->slots());
    if (t0 < 0 || t1 < t0 || t1 > c->d.max_seq) return fail(KVPR_E_RANGE, "rows [%d, %d) outside [0, %d]", t0, t1, c->d.max_seq);
    // decodes may still be touching the store: reading it on the copy stream, writing new rows on the store stream or, while
    // those are few, on the compute stream in front of ev_free (inline_store).  The caller's other work on the compute
    // stream is not waited for.
    KVPR_HIP(hipStreamSynchronize(c->copy));
    KVPR_HIP(hipStreamSynchronize(c->store));
    for (int i = 0; i < c->nbuf; ++i)
        if (c->free_recorded[i]) KVPR_HIP(hipEventSynchronize(c->ev_free[i]));
    const size_t xr = c->x_row_halfs(), kr = c->kv_row_halfs();
    const size_t xsb = c->x_store_bytes(), ksb = c->kv_store_bytes();
    const size_t n = (size_t)(t1 - t0);
    // an array kept compressed is packed on the GPU (one codec implementation): float16 rows up, packed rows down
    auto write_packed = [&](const void* src, half* dev, char* stage, char* dst, size_t row_halfs, size_t row_store_bytes,
                            int cols) -> int {
        KVPR_HIP(hipDeviceSynchronize());
        KVPR_HIP(hipMemcpy(dev, src, n * row_halfs * sizeof(half), hipMemcpyHostToDevice));
        if (int rc = kvpr::launch_quant_int4(dev, stage, (int64_t)n * c->d.batch, cols, c->compute)) return rc;
        KVPR_HIP(hipMemcpyAsync(dst, stage, n * row_store_bytes, hipMemcpyDeviceToHost, c->compute));
        KVPR_HIP(hipStreamSynchronize(c->compute));
        return KVPR_OK;
    };
    if (x_host && n > 0) {
        if (c->qx) {
            if (int rc = write_packed(x_host, c->dx[0], c->dxq[0], c->hx[layer] + (size_t)t0 * xsb, xr, xsb, c->d.hidden)) return rc;
        } else {
            memcpy(c->hx[layer] + (size_t)t0 * xsb, x_host, n * xsb);
        }
    }
    if (x_host && t0 <= c->x_rows[layer]) c->x_rows[layer] = std::max(c->x_rows[layer], t1);
    if (kv_host && n > 0) {
        if (c->qkv) {
            if (int rc = write_packed(kv_host, c->dkv[0], c->dkvq[0], c->hkv[layer] + (size_t)t0 * ksb, kr, ksb, 2 * c->d.hidden)) return rc;
        } else {
            memcpy(c->hkv[layer] + (size_t)t0 * ksb, kv_host, n * ksb);
        }
    }
    if (kv_host && t0 <= c->kv_rows[layer]) c->kv_rows[layer] = std::max(c->kv_rows[layer], t1);
    return KVPR_OK;
}

extern "C" int kvpr_store_ptrs(kvpr_ctx* c, int layer, void** x_host, void** kv_host) {
    if (!c) return fail(KVPR_E_INVAL, "ctx is null");
    if (layer < 0 || layer >= c->slots()) return fail(KVPR_E_RANGE, "layer %d outside [0, %d)", layer, c->slots());
    if (x_host) *x_host = c->hx[layer];
    if (kv_host) *kv_host = c->hkv[layer];
    // the caller may now write any row directly: treat all rows as holding data
    c->x_rows[layer] = c->d.max_seq;
    c->kv_rows[layer] = c->d.max_seq;
    return KVPR_OK;
}

constexpr double kPrefillFirst = 1.5 * (1 << 20);     // bytes of activations of the first run, at least
constexpr int kPrefillRuns = 24;
// Above this many bytes of rows the helper stays one copy, one product, one copy.  The memory of a context that was destroyed
// before is given back in the background for some 20 ms, and copies by the DMA engines meanwhile run at 30 instead of 57 GB/s (with
// or without this helper; not if the old contexts are kept or 0.1 s pass).  Small contexts are done with that at once; the slow helper
// covers that time for the large ones, and a fast one does not.  Contexts one after the other of which one of the first three decodes
// was slow, in runs / in one piece: 37, 64 and 94 MiB of rows 0 / 1 of 144, 105 MiB 1 / 0 of 60, 125 and 127 MiB 14 and 4 / 0 of 60, 175
// MiB 11 / 5 of 60.  What the runs gain beyond (30.4 -> 20.5 ms for 1024 positions, batch 32, hidden 7168) a program that makes one
// large context after the other would lose in the decodes that follow.
constexpr size_t kPrefillInRuns = size_t(96) << 20;

// Positions go in runs whose copies are workgroups of the products' launches (0: one DMA copy in, one product, one DMA copy out).  A
// kernel's copies save the engines' start, some 14 us, but rows go out at 45 - 50 instead of 57 GB/s, so runs have to gain that back:
// by what lies beside them, the product and the other direction.  One run has nothing beside its copies: better up to 3 MiB of rows.
// A narrow product hides little: with float16 rows, one after the other / in runs, hidden 256 9 MiB 289 / 320 us, 35 MiB 1022 / 1027;
// hidden 768 9 MiB 296 / 322, 14 MiB 444 / 468, 25 MiB 750 / 753, 32 MiB 955 / 931; hidden 1024 15 MiB 463 / 474, 45 MiB 1309 / 1176;
// hidden 2048 7 MiB 249 / 246, 14 MiB 442 / 401.  Packed rows are few, and their codec is beside nothing in either form: 0.8 - 1.01 of the time.
static int prefill_runs(int seq, int hidden, size_t x_row_bytes, size_t kv_row_bytes, bool packed_rows) {
    const size_t x = seq * x_row_bytes, kv = seq * kv_row_bytes, least = size_t(3) << 20, mib = size_t(1) << 20;
    if (kv > kPrefillInRuns) return 0;
    int runs = 1;
    while (runs < kPrefillRuns && (double)x * (std::sqrt(2.0) - 1.0) >= kPrefillFirst * (std::pow(2.0, 0.5 * (runs + 1)) - 1.0)) ++runs;
    if (kv > least && (runs == 1 || (!packed_rows && kv + hidden * (mib / 60) < 40 * mib))) return 0;
    return runs;
}

extern "C" int kvpr_store_prefill_kv(kvpr_ctx* c, int layer, int seq, const kvpr_layer_weights* w) {
    if (!c) return fail(KVPR_E_INVAL, "ctx is null");
    if (layer < 0 || layer >= c->slots()) return fail(KVPR_E_RANGE, "layer %d outside [0, %d)", layer, c->slots());
    if (seq < 0 || seq > c->d.max_seq) return fail(KVPR_E_RANGE, "seq %d outside [0, %d]", seq, c->d.max_seq);
    if (int rc = check_weights(c, w, false)) return rc;
    if (c->x_rows[layer] < seq) return fail(KVPR_E_STATE, "layer %d: only %d activation rows written", layer, c->x_rows[layer]);
    if (seq == 0) return KVPR_OK;
    const int h = c->d.hidden, b = c->d.batch;
    const size_t xr = c->x_row_halfs(), kr = c->kv_row_halfs(), xsb = c->x_store_bytes(), ksb = c->kv_store_bytes();
    KVPR_HIP(hipDeviceSynchronize());
    char *x_stage = c->qx ? c->dxq[0] : (char*)c->dx[0], *kv_stage = c->qkv ? c->dkvq[0] : (char*)c->dkv[0];
    const half* wkv = (const half*)w->wqkv + (size_t)h * h;
    const half* bkv = w->bqkv ? (const half*)w->bqkv + h : nullptr;
    // positions [p0, p1): the activations as the store returns them (dequantised if it keeps them packed), their rows as it takes them
    auto rows_of = [&](int p0, int p1, const kvpr::CopyJob& beside) -> int {
        const int64_t rows = (int64_t)(p1 - p0) * b;
        half *x = c->dx[0] + p0 * xr, *kv = c->dkv[0] + p0 * kr;
        if (c->qx)
            if (int rc = kvpr::launch_dequant_int4(x_stage + p0 * xsb, x, rows, h, c->compute)) return rc;
        if (int rc = c->llama ? kvpr::launch_gemm_rope(x, wkv, bkv, kv, rows, 2 * h, h, 2 * (int64_t)h, c->rope_tab, h, c->d.head_dim, b, p0,
                                                       c->compute, beside)
                              : kvpr::launch_gemm(x, wkv, bkv, kv, rows, 2 * h, h, 2 * (int64_t)h, c->compute, beside))
            return rc;
        return c->qkv ? kvpr::launch_quant_int4(kv, kv_stage + p0 * ksb, rows, 2 * h, c->compute) : KVPR_OK;
    };
    const int runs = c->prefill_runs = prefill_runs(seq, h, xsb, ksb, c->qkv);
    if (runs == 0) {
        KVPR_HIP(hipMemcpyAsync(x_stage, c->hx[layer], (size_t)seq * xsb, hipMemcpyHostToDevice, c->compute));
        if (int rc = rows_of(0, seq, kvpr::CopyJob())) return rc;
        KVPR_HIP(hipMemcpyAsync(c->hkv[layer], kv_stage, (size_t)seq * ksb, hipMemcpyDeviceToHost, c->compute));
    } else {
        // Runs of positions, in order: beside the product of one run the activations of the next come in and the rows of the one
        // before go out, by workgroups of the same launch.  The link carries both directions at once and the product hides
        // under them.  Every launch costs the link about 20 us of start and end, and nothing goes out before the first two runs
        // are in: the first is small and each is 1.4 times as long as the one before, for which the activations of one run
        // take as long to come in as the rows two runs before it to go out.  512 positions, batch 8, hidden 4096: 2.00 ms one
        // after the other, 1.80 in 16 equal runs, 1.58 in these.
        auto bound = [&](int r) {
            return r >= runs ? seq : (int)(seq * (std::pow(2.0, 0.5 * r) - 1.0) / (std::pow(2.0, 0.5 * runs) - 1.0));
        };
        // the activations of run `in` and the rows of run `out` (none outside [0, runs))
        auto copies = [&](int in, int out) {
            const size_t i0 = bound(in), i1 = bound(in + 1), o0 = out < 0 ? 0 : bound(out), o1 = out < 0 ? 0 : bound(out + 1);
            return kvpr::copy_both_ways(c->hx[layer] + i0 * xsb, x_stage + i0 * xsb, (i1 - i0) * xsb,
                                        kv_stage + o0 * ksb, c->hkv[layer] + o0 * ksb, (o1 - o0) * ksb);
        };
        if (int rc = kvpr::launch_copy(copies(0, -1), kvpr::kCopyThreads, c->compute)) return rc;
        for (int r = 0; r < runs; ++r)
            if (int rc = rows_of(bound(r), bound(r + 1), copies(r + 1, r - 1))) return rc;
        const size_t last = bound(runs - 1);
        if (int rc = kvpr::launch_copy(kvpr::copy_job(kvpr::kCopyThreads, kv_stage + last * ksb, c->hkv[layer] + last * ksb, (seq - last) * ksb,
                                                      nullptr, nullptr, 0, 16),
                                       kvpr::kCopyThreads, c->compute))
            return rc;
    }
    KVPR_HIP(hipStreamSynchronize(c->compute));
    c->kv_rows[layer] = std::max(c->kv_rows[layer], seq);
    return KVPR_OK;
}

// for tests: the rule, and what the last call of a context took
extern "C" int kvpr_debug_prefill_rule(int seq, int hidden, size_t x_row_bytes, size_t kv_row_bytes, int packed_rows) {
    return prefill_runs(seq, hidden, x_row_bytes, kv_row_bytes, packed_rows != 0);
}
extern "C" int kvpr_debug_prefill_runs(kvpr_ctx* c) { return c->prefill_runs; }
