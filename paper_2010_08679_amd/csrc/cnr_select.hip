// Choice of the greedy search parameters by profiling a sample of the checkpoint (Section 5.2,
// "Parameter selection"): quantize the sampled rows with a grid of parameter values, compute the
// mean l2 error of each, keep the value at which the improvement over plain min/max quantization
// tapers off.  The ratios are tried at the chosen num_bins, but a search of fewer iterations is the beginning of
// a longer one: on grids of ordinary size every num_bins is searched once, with a stop at every ratio's
// iterations (cnr_sample_errors), and one launch and one synchronization serve both choices.  Larger grids take one for num_bins and
// another for the ratios.  What happens here on the host is the comparison of a dozen means.
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

    // mean l2 errors of the sample at m points, written to pinned memory by the kernel
    cnr_search_params points[1 + CNR_SELECT_MAX_GRID];
    const uint64_t max_sums = scratch_bytes(n_sample, dim, bits) / sizeof(double);
    auto mean_errors = [&](uint32_t m) -> cnr_status {
        cnr_status r = cnr_sample_errors(ctx, table, n_rows, dim, sample_ids, n_sample, bits, points, m,
                                         static_cast<double *>(scratch), max_sums, ctx->host_means, hs);
        // also when a launch failed: those before it still write the scratch and the context's means
        const hipError_t e = hipStreamSynchronize(hs);
        return r != CNR_OK ? r : cnr_hip_status(ctx, e);
    };
    const double *means = ctx->host_means;
    double naive, by_bins[CNR_SELECT_MAX_GRID], by_ratio[CNR_SELECT_MAX_GRID];
    uint32_t best;

    // The ratios in ascending order, each once, and 1 among them, at which num_bins is chosen.  (None below 0, no NaN: no iterations either.)
    auto plain = [](float ratio) { return ratio > 0.0f ? ratio : 0.0f; };
    float ratios[CNR_SELECT_MAX_GRID + 1] = {1.0f};
    uint32_t n_stops = 1;
    bool has_one = false;
    for (uint32_t r = 0; r < n_ratios; ++r) {
        const float ratio = plain(ratio_grid[r]);
        has_one = has_one || ratio == 1.0f;
        uint32_t k = n_stops;
        while (k && ratios[k - 1] > ratio) --k;
        if (k && ratios[k - 1] == ratio) continue;
        for (uint32_t i = n_stops++; i > k; --i) ratios[i] = ratios[i - 1];
        ratios[k] = ratio;
    }
    auto stop_of = [&](float ratio) {
        uint32_t k = 0;
        while (ratios[k] != plain(ratio)) ++k;
        return k;
    };

    const uint64_t n_points = 1 + (uint64_t)n_bins * n_stops;
    const uint64_t workgroups = cnr_sample_workgroups(cnr_sample_lanes(dim, n_sample, n_bins), n_sample);
    if (n_points <= kSearchBatch && n_points * (workgroups > 4 ? workgroups : 4) <= max_sums) {
        // Both grids in a launch, one search for each num_bins: as long as the scratch has room for all sums with as many workgroups as the
        // sample calls for, or four where that is more (four and three values: at every row length from 21 rows on).  2.5 K rows of 64, 3 bits, four and three
        // values 64 -> 43 us; 100 to 20 K rows of 8 to 320 elements 1.1 to 1.9 times as fast.  With fewer workgroups than that a
        // wave searches several rows one after the other, which costs more than the second launch.
        points[0] = {0, (float)bins_grid[0]};  // min/max
        for (uint32_t i = 0; i < n_bins; ++i)
            for (uint32_t k = 0; k < n_stops; ++k)
                points[1 + i * n_stops + k] = {cnr_greedy_iterations(bins_grid[i], ratios[k]), (float)bins_grid[i]};
        if ((st = mean_errors((uint32_t)n_points)) != CNR_OK) return st;
        naive = means[0];
        for (uint32_t i = 0; i < n_bins; ++i) by_bins[i] = means[1 + i * n_stops + stop_of(1.0f)];
        best = taper_choice(by_bins, n_bins, naive, taper);
        for (uint32_t r = 0; r < n_ratios; ++r) by_ratio[r] = means[1 + best * n_stops + stop_of(ratio_grid[r])];
    } else {
        points[0] = {0, 1.0f};
        for (uint32_t i = 0; i < n_bins; ++i) points[1 + i] = {cnr_greedy_iterations(bins_grid[i], 1.0f), (float)bins_grid[i]};
        if ((st = mean_errors(1 + n_bins)) != CNR_OK) return st;
        naive = means[0];
        for (uint32_t i = 0; i < n_bins; ++i) by_bins[i] = means[1 + i];
        best = taper_choice(by_bins, n_bins, naive, taper);
        // One search for all ratios, or, in descending order, one for each while they have room side by side: the stops of one
        // search are behind each other.
        const bool apart = n_ratios * cnr_sample_workgroups(cnr_sample_lanes(dim, n_sample, n_ratios), n_sample) <= 4u * (uint64_t)ctx->n_cu;
        uint32_t slot[CNR_SELECT_MAX_GRID + 1], m = 0;
        for (uint32_t i = 0; i < n_stops; ++i) {
            const uint32_t k = apart ? n_stops - 1 - i : i;
            if (ratios[k] == 1.0f && !has_one) continue;
            points[m] = {cnr_greedy_iterations(bins_grid[best], ratios[k]), (float)bins_grid[best]};
            slot[k] = m++;
        }
        if ((st = mean_errors(m)) != CNR_OK) return st;
        for (uint32_t r = 0; r < n_ratios; ++r) by_ratio[r] = means[slot[stop_of(ratio_grid[r])]];
    }
    chosen->num_bins = bins_grid[best];
    if (report) {
        report[0] = naive;
        for (uint32_t i = 0; i < n_bins; ++i) report[1 + i] = by_bins[i];
        for (uint32_t r = 0; r < n_ratios; ++r) report[1 + n_bins + r] = by_ratio[r];
    }
    chosen->ratio = ratio_grid[taper_choice(by_ratio, n_ratios, naive, taper)];
    return CNR_OK;
}

}  // extern "C"
