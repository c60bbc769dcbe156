// The launches that cnr_select_greedy_params asks for, against the room in the caller's scratch: no launch's sums overrun it, and a sample
// gets all the workgroups its rows call for in every launch of up to 31 values of num_bins.
#include <stdio.h>

#include "cnr_common.h"

static uint64_t n_sample;
static uint32_t dim;
static int calls, bits, overruns, short_of_workgroups;

cnr_status cnr_enter(cnr_ctx *) { return CNR_OK; }
cnr_status cnr_hip_status(cnr_ctx *, hipError_t e) { return e == hipSuccess ? CNR_OK : CNR_E_HIP; }
cnr_status cnr_sample_errors(cnr_ctx *, const float *, uint64_t, uint32_t, const uint32_t *, uint64_t, int, const cnr_search_params *p,
                             uint32_t n, double *, uint64_t max_sums, double *mean_out, hipStream_t) {
    ++calls;
    for (uint32_t i = 0; i < n; ++i) mean_out[i] = 1.0 / (1 + i);
    uint32_t searches = 0;
    for (uint32_t i = 0; i < n; ++i) searches += !i || p[i].num_bins_f != p[i - 1].num_bins_f || p[i].n_iter < p[i - 1].n_iter;
    const uint32_t lanes = cnr_sample_lanes(dim, n_sample, searches), grid = cnr_sample_grid(lanes, n_sample, n, max_sums);
    overruns += n > kSearchBatch || !grid || (uint64_t)grid * n > max_sums || max_sums * 8 > cnr_select_scratch_bytes(n_sample, dim, bits);
    short_of_workgroups += grid < cnr_sample_workgroups(lanes, n_sample);
    return CNR_OK;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
extern "C" size_t cnr_packed_row_bytes(uint32_t d, int b) { return (size_t)d * b / 8; }
extern "C" uint32_t cnr_greedy_iterations(uint32_t num_bins, float ratio) { return (uint32_t)(ratio * (float)(num_bins - 1)); }

int main() {
    static double means[1 + CNR_SELECT_MAX_GRID];
    static float table[4] __attribute__((aligned(16)));
    static uint32_t ids[4] __attribute__((aligned(16)));
    static char scratch[16] __attribute__((aligned(16)));
    cnr_ctx ctx = {};
    ctx.host_means = means;
    ctx.n_cu = 256;
    const float ratios[] = {0.3f, 0.6f, 1.0f};
    const uint64_t sizes[] = {33, 64, 100, 256, 500, 1000, 1001, 2047, 2500, 4096, 20000, 30000, 100000, 1000000};
    const int widths[] = {2, 3, 4, 8};
    for (int b : widths)
        for (uint32_t d = 4; d <= 2048; d += 4)
            for (uint64_t n : sizes)
                for (uint32_t n_bins = 1; n_bins <= 31; ++n_bins) {
                    if (d * b % 8) continue;
                    uint32_t bins[31];
                    for (uint32_t i = 0; i < n_bins; ++i) bins[i] = 10 + 2 * i;
                    cnr_greedy_params chosen = {};
                    bits = b, dim = d, n_sample = n, calls = overruns = short_of_workgroups = 0;
                    if (cnr_select_greedy_params(&ctx, table, n + 1, d, ids, n, b, bins, n_bins, ratios, 3, 0.05, scratch, &chosen, nullptr, nullptr) != CNR_OK) return 1;
                    const int want = n_bins <= 10 ? 1 : 2;  // both grids in one launch of up to 32 points (33 rows: where it fits)
                    if (overruns || short_of_workgroups || (calls != want && n >= 64)) {
                        printf("%d bits, rows of %u, %llu of them, %u values: %d launches, %d overrun, %d short of workgroups\n", b, d, (unsigned long long)n,
                               n_bins, calls, overruns, short_of_workgroups);
                        return 1;
                    }
                }
    return 0;
}
