// Choice of the greedy search parameters by profiling a sample of the checkpoint (Section 5.2,
// "Parameter selection"): quantize the sampled rows with a grid of parameter values, compute the
// mean l2 error of each, keep the value at which the improvement over plain min/max quantization
// tapers off.  All values of num_bins are tried in one launch, then all ratios (cnr_sample_errors): two
// synchronizations, since the second grid depends on the first one's choice.  What happens here on the
// host is the comparison of a dozen means.
#include "cnr_common.h"

namespace {

size_t align16(size_t v) { return (v + 15u) & ~(size_t)15u; }

// The caller's scratch.  Only partial sums of errors go there, at most one per workgroup and point (fewer
// points or workgroups take part where a small sample's scratch holds fewer); its size, one encoded sample
// with its errors, is part of the interface and stays as it was.
size_t scratch_bytes(uint64_t n, uint32_t dim, int bits) {
    return 2 * align16(n * sizeof(float)) + align16(n * cnr_packed_row_bytes(dim, bits)) + align16(n * sizeof(double)) + 16;
}

// Index of the smallest grid value whose improvement 1 - E / E_naive is within `taper` (relative) of
// the best improvement on the grid; the first one when nothing improves on min/max.
uint32_t taper_choice(const double *errors, uint32_t n, double naive, double taper) {
    double best = 0.0;
    for (uint32_t i = 0; i < n; ++i) {
        const double gain = naive > 0.0 ? 1.0 - errors[i] / naive : 0.0;
        if (i == 0 || gain > best) best = gain;
    }
    if (!(best > 0.0)) return 0;
    for (uint32_t i = 0; i < n; ++i) {
        const double gain = naive > 0.0 ? 1.0 - errors[i] / naive : 0.0;
        if (gain >= (1.0 - taper) * best) return i;
    }
    return n - 1;
}

}  // namespace

extern "C" {

size_t cnr_select_scratch_bytes(uint64_t n_sample, uint32_t dim, int bits) {
    if (cnr_packed_row_bytes(dim, bits) == 0) return 0;
    return scratch_bytes(n_sample, dim, bits);
}

cnr_status cnr_select_greedy_params(cnr_ctx *ctx, const float *table, uint64_t n_rows, uint32_t dim,
                                    const uint32_t *sample_ids, uint64_t n_sample, int bits,
                                    const uint32_t *bins_grid, uint32_t n_bins, const float *ratio_grid,
                                    uint32_t n_ratios, double taper, void *scratch, cnr_greedy_params *chosen,
                                    double *report, void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (!cnr_valid_bits(bits)) return CNR_E_BITS;
    if (dim == 0 || dim % 4 || dim > CNR_MAX_DIM || ((uint64_t)dim * (uint64_t)bits) % 8) return CNR_E_DIM;
    if (!chosen || !bins_grid || !ratio_grid || n_bins == 0 || n_ratios == 0 || n_sample == 0 || !scratch ||
        !(taper >= 0.0 && taper < 1.0))
        return CNR_E_INVALID;
    if (n_bins > CNR_SELECT_MAX_GRID || n_ratios > CNR_SELECT_MAX_GRID) return CNR_E_INVALID;
    if ((uintptr_t)scratch % 16) return CNR_E_ALIGN;
    if (!table || n_rows == 0 || n_rows >= (1ull << 32)) return CNR_E_INVALID;
    if (((uintptr_t)table % 16) || ((uintptr_t)sample_ids % 16)) return CNR_E_ALIGN;
    hipStream_t hs = as_stream(stream);

    // mean l2 errors of the sample under m sets of parameters, written to pinned memory by the kernel
    cnr_search_params points[1 + CNR_SELECT_MAX_GRID];
    auto mean_errors = [&](uint32_t m) -> cnr_status {
        cnr_status r = cnr_sample_errors(ctx, table, n_rows, dim, sample_ids, n_sample, bits, points, m,
                                         static_cast<double *>(scratch), scratch_bytes(n_sample, dim, bits) / sizeof(double),
                                         ctx->host_means, hs);
        // also when a launch failed: those before it still write the scratch and the context's means
        const hipError_t e = hipStreamSynchronize(hs);
        return r != CNR_OK ? r : cnr_hip_status(ctx, e);
    };

    points[0] = {0, 1.0f};  // min/max
    for (uint32_t i = 0; i < n_bins; ++i) points[1 + i] = {cnr_greedy_iterations(bins_grid[i], 1.0f), (float)bins_grid[i]};  // ratio 1
    if ((st = mean_errors(1 + n_bins)) != CNR_OK) return st;
    const double naive = ctx->host_means[0];
    for (uint32_t i = 0; report && i <= n_bins; ++i) report[i] = ctx->host_means[i];
    chosen->num_bins = bins_grid[taper_choice(ctx->host_means + 1, n_bins, naive, taper)];
    for (uint32_t i = 0; i < n_ratios; ++i)  // then the ratio, at that num_bins
        points[i] = {cnr_greedy_iterations(chosen->num_bins, ratio_grid[i]), (float)chosen->num_bins};
    if ((st = mean_errors(n_ratios)) != CNR_OK) return st;
    const double *errors = ctx->host_means;
    for (uint32_t i = 0; report && i < n_ratios; ++i) report[1 + n_bins + i] = errors[i];
    chosen->ratio = ratio_grid[taper_choice(errors, n_ratios, naive, taper)];
    return CNR_OK;
}

}  // extern "C"
