// Both ways of cnr_select_greedy_params (both grids in one launch, or one after the other) against the choice made point by point,
// over grids in any order, with repeated values, without ratio 1, with ratios that give no iterations.  The kernels are a
// stand-in: a point's error is a function of its iterations and num_bins.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include "cnr_common.h"

static int calls;
static uint64_t room;  // what the caller's scratch holds, in sums

cnr_status cnr_enter(cnr_ctx *) { return CNR_OK; }
cnr_status cnr_hip_status(cnr_ctx *, hipError_t e) { return e == hipSuccess ? CNR_OK : CNR_E_HIP; }
static double error_of(uint32_t n_iter, float num_bins) { return 1.0 + 0.4 * sin(n_iter * 0.37 + 1.0) / (1.0 + 0.05 * n_iter) + 0.1 * cos((n_iter ? num_bins : 0.0f) * 0.9); }
cnr_status cnr_sample_errors(cnr_ctx *, const float *, uint64_t, uint32_t, const uint32_t *, uint64_t, int, const cnr_search_params *p,
                             uint32_t n, double *, uint64_t max_sums, double *mean_out, hipStream_t) {
    ++calls;
    room = max_sums;
    for (uint32_t i = 0; i < n; ++i) mean_out[i] = error_of(p[i].n_iter, p[i].num_bins_f);
    return CNR_OK;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
extern "C" size_t cnr_packed_row_bytes(uint32_t dim, int bits) { return (size_t)dim * bits / 8; }
extern "C" uint32_t cnr_greedy_iterations(uint32_t num_bins, float ratio) {
    if (num_bins < 2) return 0;
    const double want = ceil((double)ratio * (double)num_bins - 1e-4);
    if (!(want > 0.0)) return 0;
    return (uint32_t)(want < num_bins - 1.0 ? want : num_bins - 1.0);
}
static uint32_t taper(const double *e, uint32_t n, double naive, double t) {
    double best = 0.0;
    for (uint32_t i = 0; i < n; ++i)
        if (i == 0 || 1.0 - e[i] / naive > best) best = 1.0 - e[i] / naive;
    if (!(best > 0.0)) return 0;
    for (uint32_t i = 0; i < n; ++i)
        if (1.0 - e[i] / naive >= (1.0 - t) * best) return i;
    return n - 1;
}

int main() {
    static double means[1 + CNR_SELECT_MAX_GRID], report[1 + 2 * CNR_SELECT_MAX_GRID];
    static float table[4] __attribute__((aligned(16)));
    static uint32_t ids[4] __attribute__((aligned(16)));
    static char scratch[16] __attribute__((aligned(16)));
    cnr_ctx ctx = {};
    ctx.host_means = means;
    ctx.n_cu = 256;
    srand(1);
    int seen[2] = {0, 0};
    const uint32_t dims[] = {4, 16, 36, 64, 128, 200, 256, 1152};
    for (int trial = 0; trial < 20000; ++trial) {
        uint32_t bins[CNR_SELECT_MAX_GRID];
        float ratios[CNR_SELECT_MAX_GRID];
        const bool large = trial % 10 == 0;
        const uint32_t nb = 1 + rand() % (large ? 64 : 6), nr = 1 + rand() % (large ? 64 : 5);
        for (uint32_t i = 0; i < nb; ++i) bins[i] = rand() % 8 ? 2 + rand() % 60 : rand() % 3;
        for (uint32_t i = 0; i < nr; ++i) {
            const float odd[] = {1.0f, 0.0f, -0.5f, 1.5f, NAN, -0.0f};
            ratios[i] = rand() % 3 ? (rand() % 20) / 20.0f : odd[rand() % 6];
        }
        const uint32_t dim = dims[rand() % 8];
        const uint64_t n = 1 + rand() % (rand() % 2 ? 9 : 30000);
        const int bits = dim % 8 ? 4 : 3;
        cnr_greedy_params chosen = {};
        calls = 0;
        if (cnr_select_greedy_params(&ctx, table, n + 1, dim, ids, n, bits, bins, nb, ratios, nr, 0.05, scratch, &chosen, report, nullptr) != CNR_OK) return 1;
        double eb[CNR_SELECT_MAX_GRID], er[CNR_SELECT_MAX_GRID];
        const double naive = error_of(0, 1.0f);
        for (uint32_t i = 0; i < nb; ++i) eb[i] = error_of(cnr_greedy_iterations(bins[i], 1.0f), (float)bins[i]);
        const uint32_t b = taper(eb, nb, naive, 0.05);
        for (uint32_t r = 0; r < nr; ++r) er[r] = error_of(cnr_greedy_iterations(bins[b], ratios[r]), (float)bins[b]);
        const uint32_t r = taper(er, nr, naive, 0.05);
        bool same = report[0] == naive && chosen.num_bins == bins[b] && (chosen.ratio == ratios[r] || (isnan(chosen.ratio) && isnan(ratios[r])));
        for (uint32_t i = 0; i < nb; ++i) same = same && report[1 + i] == eb[i];
        for (uint32_t i = 0; i < nr; ++i) same = same && report[1 + nb + i] == er[i];
        if (!same || calls < 1 || calls > 2 || room < 4) {
            printf("trial %d: %u bins, %u ratios, dim %u, n %llu, %d calls\n", trial, nb, nr, dim, (unsigned long long)n, calls);
            return 1;
        }
        ++seen[calls - 1];
    }
    return seen[0] < 1000 || seen[1] < 1000;
}
