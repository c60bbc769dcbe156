// Which way the long look-up streams of a call go: through bitmap slices in LDS, and in how many parts, or through flag bytes.  Host code
// without the GPU's headers.
#ifndef CNR_MARK_RULE_H
#define CNR_MARK_RULE_H

#include <cmath>

#include "cnr.h"

// A slice: the rows whose bitmap fills a compute unit's LDS.
constexpr uint32_t kSliceWords = 40960;
constexpr uint64_t kSliceRows = 32ull * kSliceWords;
constexpr uint64_t kSliceTeamMax = 16;    // tables of more slices than this always take the flag bytes
constexpr uint32_t kStreamParts = 8;      // parts of a stream that every scratch has room for (slabs)
constexpr uint32_t kStreamPartsMax = 32;  // parts of a stream at most
// The scratch of a table: one byte per row (eight slabs, or the flag bytes), and never less than 32
// slabs of one whole slice, so that a table of one or two slices, whose 8 or 16 workgroups would
// leave most of the chip idle, can be shared out over 32 or 16 parts of its stream instead.
constexpr uint64_t kScratchFloorBytes = (uint64_t)kStreamPartsMax * kSliceWords * 4u;
static inline uint64_t mark_scratch_bytes(uint64_t n_rows) {
    const uint64_t words = (n_rows + 31u) / 32u;
    const uint64_t per_row = words * 32u, slabs32 = words * 4u * kStreamPartsMax;
    const uint64_t floor = slabs32 < kScratchFloorBytes ? slabs32 : kScratchFloorBytes;
    return per_row > floor ? per_row : floor;
}
// The most parts (a multiple of eight) a table's scratch has slabs for.
static inline uint32_t slice_parts_max(uint64_t n_rows) {
    const uint64_t words = (n_rows + 31u) / 32u;
    if (words == 0) return kStreamParts;
    const uint64_t fit = (mark_scratch_bytes(n_rows) / (words * 4u)) & ~7ull;
    return (uint32_t)(fit > kStreamPartsMax ? kStreamPartsMax : fit < kStreamParts ? kStreamParts : fit);
}
// The parts of one table's stream where the call's streams are cut into `want`.
static inline uint32_t slice_parts(uint64_t n_rows, uint32_t want) {
    const uint32_t most = slice_parts_max(n_rows);
    return want < most ? want : most;
}
static inline uint64_t slices_of(const cnr_table_job &j) { return (j.n_rows + kSliceRows - 1) / kSliceRows; }
// Streams for which a pass over the table's scratch is worth it.
static inline bool bulk_stream(const cnr_table_job &j) { return j.mark_scratch && j.n_rows && j.n_indices > j.n_rows / 256 + 65536; }

// Parts that the long streams of these tables are cut into, all together, for slices; 0: flag bytes.  Estimates in us:
//   slices   two launches, 0.6 for each MB of slabs that the workgroups write and the fold reads and zeroes, 0.23 for each part, which the
//            fold takes one after the other, and the longest part of a stream at 82 ps a look-up of 32 bits, 124 one of 64, once for every
//            round the workgroups need on the chip.  Few parts for short streams (8 tables of 1.3 M rows, 131 K look-ups each: 13 us in four parts, 30 in
//            thirty-two), many for long ones (4.2 M look-ups: 158 and 65, 61 in sixteen).  Hot rows queue in LDS, which shorter parts
//            share out (Zipf(1.2): a look-up costs half as much again, and workgroups beyond the first round meet a chip that waits for a few), so
//            the number of parts is chosen as if all did.
//   flags    two launches, 0.3 for each MB of flags, and a look-up as the stream is: 17 ps for one that gets past the table of
//            lately flagged rows, and of those there are more the larger the tables are together.  Zipf(1.05): 1.7 to 7 ps on average;
//            Zipf(1.2) half of that; without repeats 4.5 to 15 (flags of up to 2 MB in all stay in the L2), the first ones less.
// Flags are taken where they are faster at Zipf(1.05), with one exception: in a call whose look-ups cost less through slices than through flags
// (several tables, whose slices fill the chip) flags gain by launches and slabs alone, a few us, and may lose as much again for every
// look-up, so there they are taken only if a stream without repeats loses no more than a fifth of the time by it.  (In other calls every
// look-up of a skewed stream gains: two tables of 4 M rows, 10 M look-ups each, Zipf(1.2) 77 against 201, without repeats 308 against 137.)
// Measured over 884 calls of 64-bit look-ups, 1 to 16 tables of 60 K to 16 M rows and 70 K to 30 M look-ups each, against parts that fill the
// chip and slabs and launches taken as free: 1.32 times as fast with Zipf(1.05), 1.36 with Zipf(1.2), 1.20 without repeats; two skewed streams and
// six without repeats 5 to 10 % slower, one more a third.  335 of 32 bits: 1.37, 1.45 and 1.22.  Without the exception, and with other figures, a batch could lose: three
// tables of 4 M rows, 1.5 M look-ups each, 25 -> 39 us, without repeats 32 -> 78.
static inline uint32_t bulk_mark_parts(const cnr_table_job *jobs, uint32_t n_jobs, uint32_t index_bytes, uint32_t n_cu) {
    auto eligible = [](const cnr_table_job &j) { return bulk_stream(j) && slices_of(j) <= kSliceTeamMax; };
    double flag_mb = 0.0, look_ups = 0.0;  // both in millions
    for (uint32_t i = 0; i < n_jobs; ++i)
        if (eligible(jobs[i])) {
            flag_mb += 1e-6 * (double)jobs[i].n_rows;
            look_ups += 1e-6 * (double)jobs[i].n_indices;
        }
    if (look_ups == 0.0) return 0;
    auto between = [](double v, double least, double most) { return v < least ? least : v > most ? most : v; };
    const double size = std::log2(flag_mb), width = index_bytes == 4 ? 0.95 : 1.0;
    const double skewed = width * between(2.5 + 1.3 * size, 1.7, 7.2) * look_ups, flags_us = width * (7.4 + 0.29 * flag_mb) + skewed;
    const double stores = between(-1.0 + 7.0 * size, 4.5, 15.0) * look_ups;
    const double no_repeats_us = width * (8.8 + 0.24 * flag_mb + (stores < 12.0 ? 0.75 * stores : stores - 3.0));
    double slices_us = HUGE_VAL, least_stream_us = HUGE_VAL, least_us = HUGE_VAL;
    uint32_t parts = 0;
    for (uint32_t want = 2; want <= kStreamPartsMax; want *= 2) {
        uint64_t workgroups = 0, slab_words = 0, longest = 0;
        uint32_t most = 0;
        for (uint32_t i = 0; i < n_jobs; ++i) {
            if (!eligible(jobs[i])) continue;
            const uint32_t p = slice_parts(jobs[i].n_rows, want);
            if (p > most) most = p;
            workgroups += slices_of(jobs[i]) * p;
            slab_words += (jobs[i].n_rows + 31u) / 32u * p;
            if (jobs[i].n_indices / p > longest) longest = jobs[i].n_indices / p;
        }
        const double other_us = 6.7 + 0.23 * most + 0.59e-6 * 4.0 * (double)slab_words;
        const double part_us = (40.0 + 10.5 * index_bytes) * 1e-6 * (double)longest, rounds = (double)workgroups / n_cu;
        const double stream_us = part_us * std::ceil(rounds);
        if (other_us + stream_us < slices_us) slices_us = other_us + stream_us;
        if (stream_us < least_stream_us) least_stream_us = stream_us;
        const double skewed_us = other_us + 1.5 * part_us * (rounds > 1.0 ? rounds : 1.0);
        if (skewed_us < least_us) {
            least_us = skewed_us;
            parts = want;
        }
    }
    const bool faster = flags_us <= 1.1 * slices_us;
    const bool look_ups_gain = least_stream_us >= skewed;
    return faster && (look_ups_gain || no_repeats_us <= 1.2 * slices_us) ? 0 : parts;
}

#endif
