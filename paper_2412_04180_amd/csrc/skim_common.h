// Internal declarations shared by the translation units of libskim (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "skim.h"

struct skim_ctx {
    int device;
    hipStream_t stream;
    void *ws;
    size_t ws_bytes;
    int lds_limit;      // max LDS bytes one workgroup may use on this device
    int num_cu;
    char err[512];
    // optional per-kernel timing of the clustering calls (skim_profile_enable)
    int profiling;
    hipEvent_t ev[3];    // before sort, between sort and Lloyd, after Lloyd
    int ev_valid;
    size_t sort_lds_enabled[6];   // dynamic LDS size each variant of the sort kernel has been allowed so far (through this context)
    size_t lloyd_lds_enabled[4];  // likewise of the iteration kernels that keep rows in LDS
    int greedy_lds_enabled, xtx_lds_enabled, gemm3_lds_enabled;   // the larger dynamic-LDS limit of these kernels has been set through this context
    int validate;        // check W, S, alpha of the clustering calls for values the method is not defined on
    void *pack_scratch;  // this device's address of the static scratch of skim_pack_static
    int *sort_counters;  // device memory owned by the context: units of work handed out by the running sort_kernel, zero between
                         // launches (whoever takes the last one clears it)
};

#define SKIM_FAIL(ctx, code, ...)                                   \
    do {                                                            \
        snprintf((ctx)->err, sizeof((ctx)->err), __VA_ARGS__);      \
        return (code);                                              \
    } while (0)

#define SKIM_HIP(ctx, call)                                                                  \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            SKIM_FAIL(ctx, SKIM_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_));     \
    } while (0)

// Makes `device` current for the calling thread; returns SKIM_ERR_HIP on failure.
static inline skim_status skim_enter(skim_ctx *ctx) {
    if (!ctx) return SKIM_ERR_ARG;
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) SKIM_FAIL(ctx, SKIM_ERR_HIP, "hipSetDevice failed: %s", hipGetErrorString(e));
    ctx->err[0] = 0;
    return SKIM_OK;
}

// Workspace carving: 256-byte aligned pieces of the registered buffer.
struct skim_ws_cursor {
    char *base;
    size_t off, cap;
    void *take(size_t bytes) {
        size_t a = (off + 255) & ~(size_t)255;
        if (a + bytes > cap) return nullptr;
        off = a + bytes;
        return base + a;
    }
};

static inline int skim_block_offset(int bmin, int b) {  // start of block b inside a row of the *_all arrays
    return (1 << b) - (1 << bmin);
}

// Looks up this device's address of the static scratch of skim_pack_static (the device must be current).
skim_status skim_pack_static_setup(skim_ctx *ctx);

// How the iterations of skim_error_table and skim_cluster_rows take a matrix of n rows of m columns: keys per piece (4 or 8) of rows that
// are kept in LDS, 0 for rows in global memory.  The labels are the same either way, centroids and errors to the last digits.  For tests.
extern "C" int skim_cluster_pieces(const skim_ctx *ctx, int64_t n, int64_t m);

// Labels that are worked out from the clusters' upper bounds instead of read: 2^bits bounds per row at upper + i *
// upper_stride (bits = 0: labels are read), with the clusters' centroids at centroids + i * centroid_stride; labels_out (may be
// NULL) receives them.
struct skim_label_bounds {
    int bits = 0;
    const float *upper = nullptr;
    int64_t upper_stride = 0;
    const double *centroids = nullptr;
    int64_t centroid_stride = 0;
    uint8_t *labels_out = nullptr;
};

// skim_layer_loss with the per-row losses written at a stride (row i at row_loss[i * row_stride]).  loss may be
// NULL.  h_ready: the pieces of H are where the last such call with the same n, m left them in the workspace.
skim_status skim_layer_loss_strided(skim_ctx *ctx, const float *W, const float *S, const float *alpha, const float *H,
                                    int64_t n, int64_t m, int64_t ld, const uint8_t *labels,
                                    const skim_label_bounds &bounds, double *loss,
                                    double *row_loss, int64_t row_stride, bool h_ready);

// Room for the partial tiles of a scale step on any layer of at most n rows and m columns.
size_t skim_dwh_slot_bytes(int64_t n, int64_t m);

// What no call on an n x m matrix can do without: skim_workspace_bytes less those partial tiles.
size_t skim_workspace_least(int64_t n, int64_t m);
