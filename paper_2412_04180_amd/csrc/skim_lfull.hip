// Error pre-recording with the layer-wise error (Alg. 3, pre-recording loop with Err(.) in its L-full
// form, Sec. 3.4 and the remark under Alg. 1): for every bit width the rows are clustered as
// in skim_error_table, each weight gets the label of its cluster, and the error of channel i
// is dW_i H dW_i^T.  Composition of the clustering call and the layer-loss kernels, which work the
// labels out themselves; one contraction dW * H per bit width.
#include "skim_common.h"

extern "C" skim_status skim_error_table_lfull(skim_ctx *ctx, const float *W, const float *S, const float *alpha,
                                              const float *H, int64_t n, int64_t m, int64_t ld, int bmin, int bmax,
                                              int iters, double *E_full, double *E_sdiag, double *centroids_all,
                                              float *upper_all, uint8_t *labels_work) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!W || !S || !H || !E_full || !centroids_all || !upper_all || !labels_work)
        SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_error_table_lfull: W, S, H, E_full, centroids_all, upper_all, labels_work must not be NULL");
    if (bmin < 1 || bmax > SKIM_MAX_BITS || bmin > bmax) SKIM_FAIL(ctx, SKIM_ERR_ARG, "bit range [%d,%d] outside 1..4", bmin, bmax);
    if (n < 1) SKIM_FAIL(ctx, SKIM_ERR_SHAPE, "n = %lld out of range", (long long)n);
    if (ctx->ws_bytes < skim_workspace_least(n, m))
        SKIM_FAIL(ctx, SKIM_ERR_WORKSPACE, "workspace missing or smaller than skim_workspace_bytes(n, m)");
    const int nb = bmax - bmin + 1;
    // the tail of the workspace holds what must survive the calls below (they carve from its start)
    const size_t tail_bytes = (((size_t)n * nb * sizeof(double) + 255) & ~(size_t)255);
    char *tail = (char *)ctx->ws + ((ctx->ws_bytes - tail_bytes) & ~(size_t)255);
    double *sdiag = E_sdiag ? E_sdiag : (double *)tail;
    if ((st = skim_error_table(ctx, W, S, alpha, n, m, ld, bmin, bmax, iters, sdiag, centroids_all, upper_all)) != SKIM_OK)
        return st;
    const int stride = (2 << bmax) - (1 << bmin);
    for (int b = bmin; b <= bmax; ++b) {
        const int off = (1 << b) - (1 << bmin);
        // the labels are those of the clusters' upper bounds; the caller's buffer holds the last bit width's on return
        skim_label_bounds bounds;
        bounds.bits = b;
        bounds.upper = upper_all + off;
        bounds.upper_stride = stride;
        bounds.labels_out = b == bmax ? labels_work : nullptr;
        // the centroids are the clustering's, the weighted means of these labels; a cluster whose members carry no
        // sensitivity mass keeps the one it was left with (the value the packed codebook holds)
        bounds.centroids = centroids_all + off;
        bounds.centroid_stride = stride;
        if ((st = skim_layer_loss_strided(ctx, W, S, alpha, H, n, m, ld, nullptr, bounds, nullptr, E_full + (b - bmin), nb,
                                          b > bmin)) != SKIM_OK)
            return st;
    }
    return SKIM_OK;
}
