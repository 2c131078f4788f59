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
    // decodes may still be touching the store
    KVPR_HIP(hipStreamSynchronize(c->compute));
    KVPR_HIP(hipStreamSynchronize(c->copy));
    KVPR_HIP(hipStreamSynchronize(c->store));
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

extern "C" int kvpr_store_prefill_kv(kvpr_ctx* c, int layer, int seq, const kvpr_layer_weights* w) {
    if (!c) return fail(KVPR_E_INVAL, "ctx is null");
    if (layer < 0 || layer >= c->slots()) return fail(KVPR_E_RANGE, "layer %d outside [0, %d)", layer, c->slots());
    if (seq < 0 || seq > c->d.max_seq) return fail(KVPR_E_RANGE, "seq %d outside [0, %d]", seq, c->d.max_seq);
    if (int rc = check_weights(c, w, false)) return rc;
    if (c->x_rows[layer] < seq) return fail(KVPR_E_STATE, "layer %d: only %d activation rows written", layer, c->x_rows[layer]);
    if (seq == 0) return KVPR_OK;
    const int h = c->d.hidden;
    const size_t xsb = c->x_store_bytes(), ksb = c->kv_store_bytes();
    KVPR_HIP(hipDeviceSynchronize());
    // Up to 8 runs of positions, at least 2 MiB of activations each, so that activations coming in, projection and rows going
    // out overlap: the link carries both directions at once, and the rows out are the longest of the three.  512 positions,
    // batch 8, hidden 4096 in one run: 2000 us (590 in, 200, 1180 out); in 8: 1540.
    // The activations are what the store returns (dequantised if it keeps them packed).
    const int runs = (int)std::clamp<size_t>((size_t)seq * xsb >> 21, 1, std::min(8, seq));
    const hipStream_t in = runs > 1 ? c->copy : c->compute, out = runs > 1 ? c->store : c->compute;
    auto first = [&](int j) { return (size_t)((int64_t)seq * j / runs); };
    char* x_stage = c->qx ? c->dxq[0] : (char*)c->dx[0];
    char* kv_stage = c->qkv ? c->dkvq[0] : (char*)c->dkv[0];
    for (int j = 0; j < runs; ++j) {
        const size_t t = first(j);
        KVPR_HIP(hipMemcpyAsync(x_stage + t * xsb, c->hx[layer] + t * xsb, (first(j + 1) - t) * xsb, hipMemcpyHostToDevice, in));
        if (runs > 1) KVPR_HIP(hipEventRecord(c->ev_chunk[0][j], in));
    }
    const half* wkv = (const half*)w->wqkv + (size_t)h * h;
    const half* bkv = w->bqkv ? (const half*)w->bqkv + h : nullptr;
    for (int j = 0; j < runs; ++j) {
        const size_t t = first(j), n = first(j + 1) - t;
        const int64_t rows = (int64_t)n * c->d.batch;
        half *x = c->dx[0] + t * c->x_row_halfs(), *kv = c->dkv[0] + t * c->kv_row_halfs();
        if (runs > 1) KVPR_HIP(hipStreamWaitEvent(c->compute, c->ev_chunk[0][j], 0));
        if (c->qx)
            if (int rc = kvpr::launch_dequant_int4(x_stage + t * xsb, x, rows, h, c->compute)) return rc;
        if (int rc = c->llama ? kvpr::launch_gemm_rope(x, wkv, bkv, kv, rows, 2 * h, h, 2 * (int64_t)h, c->rope_tab, h, c->d.head_dim,
                                                       c->d.batch, (int)t, c->compute)
                              : kvpr::launch_gemm(x, wkv, bkv, kv, rows, 2 * h, h, 2 * (int64_t)h, c->compute))
            return rc;
        if (c->qkv)
            if (int rc = kvpr::launch_quant_int4(kv, kv_stage + t * ksb, rows, 2 * h, c->compute)) return rc;
        if (runs > 1) {
            KVPR_HIP(hipEventRecord(c->ev_chunk[1][j], c->compute));
            KVPR_HIP(hipStreamWaitEvent(out, c->ev_chunk[1][j], 0));
        }
        KVPR_HIP(hipMemcpyAsync(c->hkv[layer] + t * ksb, kv_stage + t * ksb, n * ksb, hipMemcpyDeviceToHost, out));
    }
    KVPR_HIP(hipStreamSynchronize(out));
    c->kv_rows[layer] = std::max(c->kv_rows[layer], seq);
    return KVPR_OK;
}
