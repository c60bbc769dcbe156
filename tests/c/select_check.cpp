// The host side of cnr_select_greedy_params, linked with stand-ins for the kernels and the runtime: when a
// launch fails the call must wait for what was enqueued before it, which may still write the caller's scratch
// and the context's pinned means, before it returns the failure.
#include <stdio.h>

#include "cnr_common.h"

static int calls, fail_at;     // calls of cnr_sample_errors; the one that fails
static bool work_in_flight;    // enqueued since the last synchronization

cnr_status cnr_enter(cnr_ctx *) { return CNR_OK; }
cnr_status cnr_hip_status(cnr_ctx *, hipError_t e) { return e == hipSuccess ? CNR_OK : CNR_E_HIP; }
cnr_status cnr_sample_errors(cnr_ctx *, const float *, uint64_t, uint32_t, const uint32_t *, uint64_t, int, const cnr_search_params *,
                             uint32_t n_params, double *, uint64_t, double *mean_out, hipStream_t) {
    work_in_flight = true;
    for (uint32_t i = 0; i < n_params; ++i) mean_out[i] = 1.0 / (1 + i);
    return ++calls == fail_at ? CNR_E_HIP : CNR_OK;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t) {
    work_in_flight = false;
    return hipSuccess;
}
extern "C" size_t cnr_packed_row_bytes(uint32_t dim, int bits) { return (size_t)dim * bits / 8; }
extern "C" uint32_t cnr_greedy_iterations(uint32_t num_bins, float) { return num_bins ? num_bins - 1 : 0; }

int main() {
    static double means[1 + CNR_SELECT_MAX_GRID], report[6];
    static float table[64 * 4] __attribute__((aligned(16)));
    static uint32_t ids[4] __attribute__((aligned(16)));
    static char scratch[1024] __attribute__((aligned(16)));
    const uint32_t bins[] = {10, 25, 45};
    const float ratios[] = {0.5f, 1.0f};
    cnr_ctx ctx = {};
    ctx.host_means = means;
    for (fail_at = 0; fail_at <= 2; ++fail_at) {  // 0: none fails
        calls = 0;
        cnr_greedy_params chosen;
        const cnr_status st = cnr_select_greedy_params(&ctx, table, 4, 64, ids, 4, 4, bins, 3, ratios, 2, 0.05, scratch, &chosen, report, nullptr);
        if (st != (fail_at ? CNR_E_HIP : CNR_OK) || calls != (fail_at == 1 ? 1 : 2) || work_in_flight) {
            printf("launch %d fails: status %d after %d launches, work in flight: %d\n", fail_at, (int)st, calls, (int)work_in_flight);
            return 1;
        }
    }
    return 0;
}
