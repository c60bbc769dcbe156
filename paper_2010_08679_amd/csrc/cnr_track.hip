// Tracking bit-vector (Section 5.1.1) and its compaction into the incremental view (Section 5.1).
//
// Every kernel here takes a batch of tables (a GPU holds several embedding tables, Section 2.1, and
// a checkpoint covers all of them): a workgroup's y index selects the table, its x index the share
// of that table's work, so the tables of a batch run side by side in one launch.  The single-table
// entry points are batches of one.
#include "cnr_common.h"
#include "cnr_mark_rule.h"

#include <type_traits>

// Per-tile counts of cnr_compact_dirty_noalloc: a fixed array in the library's device image instead
// of a buffer from the caller.  Every GPU that loads the library holds its own copy at its own
// address.  In host code this name is only a handle for hipGetSymbolAddress, never a device address:
// kernels get the looked-up pointer (cnr_ctx::static_scratch) as an argument like any other scratch.
static __device__ __align__(256) uint32_t scratch[CNR_NOALLOC_SCRATCH_BYTES / sizeof(uint32_t)];

namespace {

struct TrackJob {
    uint32_t *bitmap;
    uint64_t n_rows;
    const void *idx;      // mark: look-up indices
    uint64_t n_idx;
    uint8_t *flags;       // mark, bulk route: the scratch (flag bytes or slabs), zero on entry and on exit
    uint32_t parts;       // mark, LDS slices: workgroups that share this table's stream = slabs to fold
    uint32_t *row_ids;    // compact
    uint64_t capacity;
    uint64_t *n_dirty;
    uint32_t *block_count;
};
struct TrackBatch {
    TrackJob job[CNR_MAX_BATCH];
    uint32_t grid_x;  // workgroups per table
};

__global__ void __launch_bounds__(kBlock) clear_kernel(const TrackBatch b) {
    const TrackJob &t = b.job[wg_y()];
    const uint64_t n = (t.n_rows + 31u) / 32u;
    const uint64_t stride = (uint64_t)b.grid_x * kBlock;
    for (uint64_t i = (uint64_t)wg_x() * kBlock + tid_x(); i < n; i += stride) t.bitmap[i] = 0u;
}

// ---------------------------------------------------------------------------------------------
// mark: one bit per looked-up row.
//
// The index stream is read once, coalesced (each lane four indices per pass, all in flight).
// Hot rows repeat many times under a skewed lookup distribution, so the word is tested with a
// plain load first and the atomic OR is issued only for bits not yet seen as set: a stale zero
// merely costs a redundant OR, and bits never go back to zero while marking.  After a clear every
// look-up of a hot row sees a zero, and the ORs of one address complete one after the other, 12 ns
// each: so a workgroup's look-ups that want an OR first agree on one of those that name the same row.  Each
// leaves its number in a slot of LDS that its row selects, and gives way to the number that it finds
// there afterwards if that one's row is the same.  (Where two rows share a slot one of them may issue
// more than one.)  And all words of a pass are loaded before its first OR, which the compiler would not move a load past.
// 8 tables of 1 M rows, 40,960 Zipf(1.1) look-ups each: first call after a clear 44 -> 11 us, mean of 32 calls 12.1 -> 6.5 (3.5
// where all bits are set); one table of 100 K rows, 4096 look-ups 6.5 -> 3.0; 1.5 M look-ups of different rows in no order into 5 M
// 128 -> 92.  Where the bitmap is larger than the caches and nothing repeats, an OR that follows its word's load at once is faster: 500 K different rows in
// no order of 64 M 24 -> 27, of 256 M 24 -> 29, without the agreement and its barriers as well (Zipf(1.05) look-ups into 64 M, 131 K: 45 -> 9).
// A list of rows in order has no repeats either, but its ORs meet in few words, up to 32 of a wave in one, and the loads ahead of them made that worse (750 K
// of 2.5 M rows 31.2 -> 33.0 us, 1 M of 1 M 84 -> 102).  So a wave whose rows ascend collects the bits of each word first, and
// its first lane there issues the OR: 6.0 and 4.7 us.  Other waves pay a comparison with the lane before, while they wait for the words.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kMarkUnroll = 4, kMarkSlots = 4096;
// Whether this lane's row is above the one of the lane before.
__device__ __forceinline__ bool lane_ascends(uint32_t r) {
    const uint32_t left = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
    return r > left || (tid_x() & (kWave - 1)) == 0;
}
template <typename IdxT>
__global__ void __launch_bounds__(kBlock) mark_kernel(const TrackBatch b, cnr_dev_errors *err) {
    __shared__ uint16_t slot[kMarkSlots];
    __shared__ uint32_t row[kBlock * kMarkUnroll];
    const TrackJob &t = b.job[wg_y()];
    uint32_t *__restrict__ bitmap = t.bitmap;
    const IdxT *__restrict__ idx = static_cast<const IdxT *>(t.idx);
    const uint64_t n_rows = t.n_rows, n = t.n_idx;
    const uint64_t stride = (uint64_t)b.grid_x * kBlock;
    const uint32_t tid = tid_x();
    unsigned bad = 0;
    for (uint64_t first = (uint64_t)wg_x() * kBlock; first < n; first += stride * kMarkUnroll) {
        IdxT v[kMarkUnroll];
        uint32_t word[kMarkUnroll];
#pragma unroll
        for (uint32_t u = 0; u < kMarkUnroll; ++u) {
            const uint64_t p = first + tid + (uint64_t)u * stride;
            v[u] = p < n ? idx[p] : (IdxT)0;
        }
#pragma unroll
        for (uint32_t u = 0; u < kMarkUnroll; ++u) {
            const uint64_t p = first + tid + (uint64_t)u * stride;
            const int64_t r = (int64_t)v[u];
            const bool valid = r >= 0 && (uint64_t)r < n_rows;
            if (p < n && !valid) ++bad;
            word[u] = p < n && valid ? bitmap[(uint64_t)r >> 5] : ~0u;
        }
        bool ascending = true;
#pragma unroll
        for (uint32_t u = 0; u < kMarkUnroll; ++u) ascending = ascending && lane_ascends((uint32_t)v[u]);
        // (Expected not to: the code then lies apart.  In the way of the others it cost every call 0.15 us.)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!ascending) == 0, 0)) {
#pragma unroll
            for (uint32_t u = 0; u < kMarkUnroll; ++u) {
                const uint32_t r = (uint32_t)v[u];
                uint32_t bits = ~word[u] & (1u << (r & 31u));
#pragma unroll
                for (int off = 1; off < 32; off *= 2) {  // at most 32 lanes have a word in common
                    const uint32_t theirs = (uint32_t)__shfl_down((int)bits, off);
                    if ((uint32_t)__shfl_down((int)r, off) >> 5 == r >> 5) bits |= theirs;
                }
                const uint32_t left = (uint32_t)__shfl_up((int)r, 1);
                if (bits && (left >> 5 != r >> 5 || (tid & (kWave - 1)) == 0)) atomicOr(bitmap + (r >> 5), bits);
                word[u] = ~0u;
            }
        }
        bool wants[kMarkUnroll];
#pragma unroll
        for (uint32_t u = 0; u < kMarkUnroll; ++u) {
            const uint32_t r = (uint32_t)v[u];  // n_rows < 2^32
            wants[u] = !(word[u] & (1u << (r & 31u)));
            if (wants[u]) {
                row[u * kBlock + tid] = r;
                slot[r * 0x9E3779B1u >> 20] = (uint16_t)(u * kBlock + tid);
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < kMarkUnroll; ++u) {
            const uint32_t r = (uint32_t)v[u];
            if (wants[u]) {
                const uint32_t k = slot[r * 0x9E3779B1u >> 20];
                if (k == u * kBlock + tid || row[k] != r) atomicOr(bitmap + (r >> 5), 1u << (r & 31u));
            }
        }
        __syncthreads();  // the slots are read before the next pass's look-ups write them
    }
    // one atomic per wave that saw out-of-range indices
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
    if (bad && (tid & (kWave - 1)) == 0) atomicAdd(&err->n_bad_indices, (unsigned long long)bad);
}

// ---------------------------------------------------------------------------------------------
// mark, bulk variants: no device-scope atomics.  The first, for tables too large for the second.
//
// On this GPU the L2 caches of the eight XCDs are not coherent with each other, so a device-scope
// atomic OR is carried out at the memory side: each one costs a 64-byte read and a 32-byte write
// there, and a few million of them dominate a checkpoint.  Plain byte stores do not have that
// problem: different threads may write different bytes of one cache line from anywhere, and
// writing the same value twice is harmless.  So a long index stream is first scattered into one
// flag byte per row (scratch, all zero on entry), and a second kernel folds the flag bytes into
// the bitmap 32 rows per thread, with plain read-modify-write because every bitmap word has exactly
// one owner there, and zeroes the bytes it found set so that the scratch is clean again.
// ---------------------------------------------------------------------------------------------
// Most look-ups of a skewed stream repeat a row that the same compute unit has flagged already, and a
// scattered byte store is the expensive part (each one is a request of its own to the L2, about 17 ps
// of the whole chip's time).  So a workgroup keeps, in 128 KB of LDS, a direct-mapped table of the
// rows it has flagged lately: h = row * odd constant (a bijection on 32 bits), slot = high 16 bits of
// h, and the slot holds the low 16 bits, so slot and content together name exactly one row.  A
// look-up that finds its own row there is dropped, any other one takes the slot over and stores its
// flag byte.  A row found in the table has had its store issued (or about to be issued, in program
// order) by the lane that put it there, so nothing is ever lost; collisions only cost a repeated
// store.  The content 0xFFFF marks an empty slot; the one row in 65,536 whose own low bits are
// 0xFFFF bypasses the table.  One workgroup of kSeenThreads threads per compute unit (the table
// fills the LDS; two smaller tables per unit do worse, each sees half the repeats); the stream is
// read as 16-byte vectors.
constexpr int kSeenThreads = 1024;
constexpr uint32_t kSeenSlots = 65536;

template <typename IdxT>
__global__ void __launch_bounds__(kSeenThreads) mark_flags_kernel(const TrackBatch b, cnr_dev_errors *err) {
    constexpr int kVec = 16 / (int)sizeof(IdxT);
    typedef IdxT vec_t __attribute__((ext_vector_type(kVec)));
    constexpr int kUnroll = 4;
    __shared__ uint16_t seen[kSeenSlots];
    const TrackJob &t = b.job[wg_y()];
    uint8_t *__restrict__ flags = t.flags;
    const uint32_t n_rows = (uint32_t)t.n_rows;  // the host checks n_rows < 2^32
    const uint32_t tid = tid_x();
    for (uint32_t i = tid; i < kSeenSlots / 2; i += kSeenThreads) reinterpret_cast<uint32_t *>(seen)[i] = 0xFFFFFFFFu;
    __syncthreads();

    // the stream as [head][16-byte vectors][tail]: head and tail are fewer than kVec elements each
    const IdxT *idx = static_cast<const IdxT *>(t.idx);
    const uint64_t n = t.n_idx;
    uint64_t head = ((16u - (uint32_t)((uintptr_t)idx & 15u)) & 15u) / sizeof(IdxT);
    if (head > n) head = n;
    const vec_t *vecs = reinterpret_cast<const vec_t *>(idx + head);
    const uint64_t n_vec = (n - head) / kVec;
    const uint64_t tail = head + n_vec * kVec;

    unsigned bad = 0;
    auto look_up = [&](IdxT v) {
        bool valid = (uint32_t)v < n_rows;
        if constexpr (sizeof(IdxT) == 8) valid = valid && ((uint64_t)v >> 32) == 0;
        else valid = valid && v >= 0;
        if (!valid) {
            ++bad;
            return;
        }
        const uint32_t r = (uint32_t)v;
        const uint32_t h = r * 0x9E3779B1u;
        const uint32_t slot = h >> 16, low = h & 0xFFFFu;
        if (seen[slot] != low || low == 0xFFFFu) {
            seen[slot] = (uint16_t)low;
            flags[r] = 1;
        }
    };
    const uint64_t stride = (uint64_t)b.grid_x * kSeenThreads;
    for (uint64_t p = (uint64_t)wg_x() * kSeenThreads + tid; p < n_vec; p += stride * kUnroll) {
        vec_t v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint64_t q = p + (uint64_t)u * stride;
            if (q < n_vec) v[u] = load_stream<vec_t>(vecs + q);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint64_t q = p + (uint64_t)u * stride;
            if (q < n_vec) {
#pragma unroll
                for (int e = 0; e < kVec; ++e) look_up(v[u][e]);
            }
        }
    }
    if (wg_x() == 0) {
        if (tid < head) look_up(idx[tid]);
        else if (tid - head < n - tail) look_up(idx[tail + (tid - head)]);
    }
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
    if (bad && (tid & (kWave - 1)) == 0) atomicAdd(&err->n_bad_indices, (unsigned long long)bad);
}

// ---------------------------------------------------------------------------------------------
// mark, second bulk variant, for tables of up to a few tens of millions of rows: bitmap slices in LDS.
//
// A workgroup owns kSliceRows consecutive rows of one table as a bitmap in LDS (all 160 KB of a
// compute unit) and one part of the table's index stream (a half down to a thirty-second, see
// bulk_mark_parts): it reads its share of the stream, sets the bits of the
// look-ups that fall into its rows with LDS atomics, and stores the slice to slab s (= its part of
// the stream) of the scratch buffer, partial bitmaps that fold_slabs_kernel ORs into the bitmap and
// zeroes again.  Nothing is scattered to memory; the price is that the W = ceil(n_rows / kSliceRows)
// workgroups of a team read the same part of the stream.  Workgroups are dealt to the eight XCDs in
// turn along x; where the number of parts is a multiple of eight, x & 7 names both the part (mod 8)
// and the XCD: a team shares its part of the stream through one L2 and memory is read once.  (Two or four parts, for streams so
// short that this does not matter, put a team on four or two XCDs.)
// Where every table is one slice there is no team to share with, and STREAM reads with the non-temporal
// hint: 8 tables of 1 M rows, 8.2 M look-ups each, from memory 167 -> 107 us, 1 M look-ups 49 -> 38 (with
// teams of four it costs 20 %: 415 -> 502 us for 8 x 5 M rows, 20 M look-ups).
// ---------------------------------------------------------------------------------------------
constexpr int kSliceThreads = 1024;

template <typename IdxT, bool STREAM>
__global__ void __launch_bounds__(kSliceThreads) mark_slices_kernel(const TrackBatch b, cnr_dev_errors *err) {
    constexpr int kVec = 16 / (int)sizeof(IdxT);
    typedef IdxT vec_t __attribute__((ext_vector_type(kVec)));
    constexpr int kUnroll = 4;
    __shared__ uint32_t bits[kSliceWords];
    const TrackJob &t = b.job[wg_y()];
    const uint32_t part = wg_x() % t.parts, w = wg_x() / t.parts;
    const uint32_t n_rows = (uint32_t)t.n_rows;
    const uint64_t first = (uint64_t)w * kSliceRows;
    if (first >= t.n_rows) return;  // the whole workgroup: tables of a batch differ in size
    const uint32_t lo = (uint32_t)first;
    const uint32_t span = n_rows - lo < kSliceRows ? n_rows - lo : (uint32_t)kSliceRows;
    const uint32_t tid = tid_x();
    for (uint32_t i = tid; i < kSliceWords; i += kSliceThreads) bits[i] = 0u;
    __syncthreads();

    // the stream as [head][16-byte vectors][tail]: head and tail are fewer than kVec elements each
    const IdxT *idx = static_cast<const IdxT *>(t.idx);
    const uint64_t n = t.n_idx;
    uint64_t head = ((16u - (uint32_t)((uintptr_t)idx & 15u)) & 15u) / sizeof(IdxT);
    if (head > n) head = n;
    const vec_t *vecs = reinterpret_cast<const vec_t *>(idx + head);
    const uint64_t n_vec = (n - head) / kVec;
    const uint64_t tail = head + n_vec * kVec;
    const uint64_t per_part = (n_vec + t.parts - 1u) / t.parts;
    const uint64_t v0 = part * per_part;
    const uint64_t v1 = v0 + per_part < n_vec ? v0 + per_part : n_vec;

    unsigned bad = 0;
    // COUNT: also count the indices outside the table (the team's first workgroup does, for its part
    // of the stream).  A look-up inside this slice is inside the table, so the bit needs no more
    // than the slice test.
    auto run = [&](auto count_tag) {
        constexpr bool COUNT = decltype(count_tag)::value;
        auto look_up = [&](IdxT v) {
            const uint32_t d = (uint32_t)v - lo;
            bool mine = d < span;
            if constexpr (sizeof(IdxT) == 8) mine = mine && ((uint64_t)v >> 32) == 0;
            if (mine)
                __hip_atomic_fetch_or(&bits[d >> 5], 1u << (d & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if constexpr (COUNT) {
                bool valid = (uint32_t)v < n_rows;
                if constexpr (sizeof(IdxT) == 8) valid = valid && ((uint64_t)v >> 32) == 0;
                bad += valid ? 0u : 1u;
            }
        };
        for (uint64_t p = v0 + tid; p < v1; p += (uint64_t)kSliceThreads * kUnroll) {
            vec_t v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint64_t q = p + (uint64_t)u * kSliceThreads;
                if (q < v1) v[u] = STREAM ? load_stream<vec_t>(vecs + q) : vecs[q];
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint64_t q = p + (uint64_t)u * kSliceThreads;
                if (q < v1) {
#pragma unroll
                    for (int e = 0; e < kVec; ++e) look_up(v[u][e]);
                }
            }
        }
        if (part == 0) {
            if (tid < head) look_up(idx[tid]);
            else if (tid - head < n - tail) look_up(idx[tail + (tid - head)]);
        }
    };
    if (w == 0) run(std::true_type{});
    else run(std::false_type{});
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
    if (bad && (tid & (kWave - 1)) == 0) atomicAdd(&err->n_bad_indices, (unsigned long long)bad);
    __syncthreads();

    const uint64_t n_words = (t.n_rows + 31u) / 32u;
    uint32_t *slab = reinterpret_cast<uint32_t *>(t.flags) + part * n_words + (uint64_t)w * kSliceWords;
    const uint32_t words = (span + 31u) / 32u;
    for (uint32_t i = tid; i < words; i += kSliceThreads) slab[i] = bits[i];
}

// bitmap |= OR of the table's slabs; the slabs are left all zero.
__global__ void __launch_bounds__(kBlock) fold_slabs_kernel(const TrackBatch b) {
    const TrackJob &t = b.job[wg_y()];
    uint32_t *__restrict__ slabs = reinterpret_cast<uint32_t *>(t.flags);
    uint32_t *__restrict__ bitmap = t.bitmap;
    const uint64_t n_words = (t.n_rows + 31u) / 32u;
    const uint64_t stride = (uint64_t)b.grid_x * kBlock;
    for (uint64_t i = (uint64_t)wg_x() * kBlock + tid_x(); i < n_words; i += stride) {
        uint32_t acc = 0;
        for (uint32_t s = 0; s < t.parts; ++s) {
            acc |= slabs[s * n_words + i];
            slabs[s * n_words + i] = 0u;
        }
        if (acc) bitmap[i] |= acc;
    }
}

// Eight flag bytes (each 0 or 1) to eight bits, first byte in bit 0.
__device__ __forceinline__ uint32_t flags_to_bits(uint64_t eight) {
    return (uint32_t)((eight * 0x0102040810204080ull) >> 56);
}

__global__ void __launch_bounds__(kBlock) fold_flags_kernel(const TrackBatch b) {
    const TrackJob &t = b.job[wg_y()];
    uint8_t *__restrict__ flags = t.flags;
    uint32_t *__restrict__ bitmap = t.bitmap;
    const uint64_t n_words = (t.n_rows + 31u) / 32u;
    const uint64_t stride = (uint64_t)b.grid_x * kBlock;
    for (uint64_t w = (uint64_t)wg_x() * kBlock + tid_x(); w < n_words; w += stride) {
        ulonglong2 *src = reinterpret_cast<ulonglong2 *>(flags + 32u * w);
        const ulonglong2 a = src[0], b = src[1];
        if ((a.x | a.y | b.x | b.y) == 0) continue;
        const uint32_t bits = flags_to_bits(a.x) | (flags_to_bits(a.y) << 8) | (flags_to_bits(b.x) << 16) |
                              (flags_to_bits(b.y) << 24);
        bitmap[w] |= bits;
        src[0] = make_ulonglong2(0, 0);
        src[1] = make_ulonglong2(0, 0);
    }
}

// ---------------------------------------------------------------------------------------------
// compact: set-bit positions in ascending order.
//
// Two kernels, or the second one alone, no inter-workgroup waiting.  Each workgroup owns kBlock consecutive 64-bit bitmap
// words (one per thread = 16384 rows).
//   count:   population count of the tile -> block_count[b]
//   scatter: base = sum of block_count[0..b) (read back by every workgroup; at most a few thousand
//            values), exclusive scan of the per-thread counts inside the workgroup (wave shuffles +
//            one LDS step across the four waves), then every lane walks the set bits of its own
//            word and writes their row numbers, as 16-bit offsets from the tile's first row, to its
//            place in an LDS copy of the tile's part of the list, which the workgroup then stores
//            to the list with every lane writing consecutive ids.
// Tables of up to kSelfCountTiles tiles (1 M rows) need the second kernel only: there a workgroup counts
// the bits of all earlier tiles itself, at most 128 KB of bitmap out of the L2, which takes less than the
// launch it saves (one table: 100 K rows 7.9 -> 5.7 us, 1 M rows 8.3 -> 7.3; eight tables of 1 M 9.8 -> 9.0; at 96
// tiles 8.2 -> 7.5, at 128 no difference, at 256 8.2 -> 11.5).  What is counted grows with the square of a table's
// tiles and with the tables of the launch: kSelfCountPairs is where that meets the launch (in graph replays, 16
// tables of 48 tiles 7.9 -> 7.2 us, 12 of 56 7.9 and 7.8, 10 of 64 7.8 -> 8.3, 16 of 64 8.8 -> 10.5).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint64_t load_tile_word(const uint32_t *__restrict__ bitmap,
                                                   uint64_t n_rows, uint64_t n_words32, uint64_t w64) {
    const uint64_t i0 = 2 * w64, i1 = 2 * w64 + 1;
    uint64_t lo = i0 < n_words32 ? bitmap[i0] : 0u;
    uint64_t hi = i1 < n_words32 ? bitmap[i1] : 0u;
    uint64_t w = lo | (hi << 32);
    // ignore bits at positions >= n_rows
    const uint64_t first_row = w64 * 64u;
    if (first_row >= n_rows) return 0;
    const uint64_t live = n_rows - first_row;
    if (live < 64u) w &= (~0ull) >> (64u - live);
    return w;
}

__device__ __forceinline__ unsigned block_sum_u32(unsigned v, unsigned *lds /* kWavesPerBlock */) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const int wave = tid_x() / kWave;
    __syncthreads();
    if ((tid_x() & (kWave - 1)) == 0) lds[wave] = v;
    __syncthreads();
    unsigned t = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
    return t;
}

// Tiles of one table; an empty table still has one, so that its count is written.
__device__ __forceinline__ uint64_t compact_tiles(uint64_t n_rows) {
    const uint64_t tiles = (n_rows + kCompactRowsPerBlock - 1) / kCompactRowsPerBlock;
    return tiles ? tiles : 1;
}

__global__ void __launch_bounds__(kBlock) compact_count_kernel(const TrackBatch b) {
    __shared__ unsigned lds[kWavesPerBlock];
    const TrackJob &t = b.job[wg_y()];
    const uint64_t n_rows = t.n_rows, n_words32 = (n_rows + 31u) / 32u;
    if (wg_x() >= compact_tiles(n_rows)) return;  // uniform over the workgroup
    const uint32_t *__restrict__ bitmap = t.bitmap;
    uint32_t *__restrict__ block_count = t.block_count;
    const uint64_t w64 = (uint64_t)wg_x() * kBlock + tid_x();
    const unsigned c = __popcll(load_tile_word(bitmap, n_rows, n_words32, w64));
    const unsigned total = block_sum_u32(c, lds);
    if (tid_x() == 0) block_count[wg_x()] = total;
}

constexpr uint64_t kSelfCountTiles = 64, kSelfCountPairs = 9 * kSelfCountTiles * kSelfCountTiles;

// This thread's share of the set bits in the first `tiles` (whole) tiles of a bitmap.
__device__ __forceinline__ unsigned count_tiles_share(const uint32_t *__restrict__ bitmap, uint32_t tiles) {
    constexpr uint32_t kWordsPerTile = kCompactRowsPerBlock / 32;
    const uint32_t words = tiles * kWordsPerTile;
    unsigned c = 0;
    if (((uintptr_t)bitmap & 15u) == 0) {  // uniform
        const u32x4 *p = reinterpret_cast<const u32x4 *>(bitmap);
        const uint32_t n = words / 4;  // a multiple of kBlock / 2
        constexpr uint32_t kAhead = 8;
        for (uint32_t i = tid_x(); i < n; i += kBlock * kAhead) {
            u32x4 v[kAhead];
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) v[k] = i + k * kBlock < n ? p[i + k * kBlock] : u32x4{0, 0, 0, 0};
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) c += __popc(v[k].x) + __popc(v[k].y) + __popc(v[k].z) + __popc(v[k].w);
        }
    } else {
        for (uint32_t i = tid_x(); i < words; i += kBlock) c += __popc(bitmap[i]);
    }
    return c;
}

// COUNTED: block_count holds the tiles' counts; else the workgroup counts the tiles before its own.
template <bool COUNTED>
__global__ void __launch_bounds__(kBlock) compact_scatter_kernel(const TrackBatch b, cnr_dev_errors *err) {
    __shared__ unsigned lds[kWavesPerBlock];
    __shared__ unsigned wave_total[kWavesPerBlock];
    __shared__ uint16_t tile_ids[kCompactRowsPerBlock];
    const TrackJob &t = b.job[wg_y()];
    const uint64_t n_rows = t.n_rows, n_words32 = (n_rows + 31u) / 32u, capacity = t.capacity;
    const uint64_t tiles = compact_tiles(n_rows);
    if (wg_x() >= tiles) return;  // uniform over the workgroup
    const uint32_t *__restrict__ bitmap = t.bitmap;
    const uint32_t *__restrict__ block_count = t.block_count;
    uint32_t *__restrict__ row_ids = t.row_ids;
    uint64_t *__restrict__ n_dirty = t.n_dirty;
    const int lane = tid_x() & (kWave - 1);
    const int wave = tid_x() / kWave;

    // dirty rows in all earlier tiles
    unsigned part = 0;
    if constexpr (COUNTED) {
        for (unsigned b = tid_x(); b < wg_x(); b += kBlock) part += block_count[b];
    } else {
        part = count_tiles_share(bitmap, wg_x());
    }
    const uint64_t base = block_sum_u32(part, lds);

    const uint64_t w64 = (uint64_t)wg_x() * kBlock + tid_x();
    const uint64_t word = load_tile_word(bitmap, n_rows, n_words32, w64);
    const unsigned c = __popcll(word);

    // inclusive scan of c over the wave
    unsigned incl = c;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) wave_total[wave] = incl;
    __syncthreads();
    unsigned before_wave = 0, block_total = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) {
        const unsigned t = wave_total[k];
        if (k < wave) before_wave += t;
        block_total += t;
    }
    const unsigned excl = before_wave + incl - c;  // dirty rows of this tile before my word

    if (wg_x() == tiles - 1 && tid_x() == 0) {
        const uint64_t total = base + block_total;
        *n_dirty = total;
        if (total > capacity) raise_flag(err, CNR_FLAG_CAPACITY);
    }

    // ids of the tile in ascending order, as 16-bit offsets from its first row, into LDS: every lane
    // walks the set bits of its own word ...
    {
        uint64_t rest = word;
        unsigned k = excl;
        const uint32_t off0 = tid_x() * 64u;
        while (rest) {
            tile_ids[k++] = (uint16_t)(off0 + (uint32_t)__builtin_ctzll(rest));
            rest &= rest - 1;
        }
    }
    __syncthreads();
    // ... and from there to the list, every lane storing
    const uint64_t tile_row0 = (uint64_t)wg_x() * kCompactRowsPerBlock;
    for (unsigned p = tid_x(); p < block_total; p += kBlock) {
        const uint64_t pos = base + p;
        if (pos < capacity) row_ids[pos] = (uint32_t)(tile_row0 + tile_ids[p]);
    }
}

// Workgroups per table for a grid-stride kernel over a batch: enough for the largest share of work,
// at most an equal part of `blocks_per_cu` workgroups per compute unit.
unsigned batch_grid_x(const cnr_ctx *ctx, uint64_t max_items, uint64_t per_block, unsigned blocks_per_cu,
                      uint32_t n_jobs) {
    uint64_t need = (max_items + per_block - 1) / per_block;
    uint64_t cap = (uint64_t)ctx->n_cu * blocks_per_cu / n_jobs;
    if (cap < 1) cap = 1;
    if (need < 1) need = 1;
    return (unsigned)(need < cap ? need : cap);
}

cnr_status check_tracked_table(const cnr_table_job &j) {
    if (j.n_rows >= (1ull << 32)) return CNR_E_INVALID;
    if (!j.bitmap && j.n_rows) return CNR_E_INVALID;
    if ((uintptr_t)j.bitmap % 4) return CNR_E_ALIGN;
    return CNR_OK;
}

}  // namespace

extern "C" {

size_t cnr_mark_scratch_bytes(uint64_t n_rows) { return (size_t)mark_scratch_bytes(n_rows); }

cnr_status cnr_clear_bitmap_batch(cnr_ctx *ctx, const cnr_table_job *jobs, uint32_t n_jobs, void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (n_jobs && !jobs) return CNR_E_INVALID;
    for (uint32_t i = 0; i < n_jobs; ++i)
        if ((st = check_tracked_table(jobs[i])) != CNR_OK) return st;
    for (uint32_t first = 0; first < n_jobs; first += CNR_MAX_BATCH) {
        TrackBatch b = {};
        uint32_t n = 0;
        uint64_t max_words = 0;
        for (uint32_t i = first; i < n_jobs && i < first + CNR_MAX_BATCH; ++i) {
            if (jobs[i].n_rows == 0) continue;
            b.job[n].bitmap = jobs[i].bitmap;
            b.job[n].n_rows = jobs[i].n_rows;
            const uint64_t words = cnr_bitmap_words(jobs[i].n_rows);
            if (words > max_words) max_words = words;
            ++n;
        }
        if (n == 0) continue;
        b.grid_x = batch_grid_x(ctx, max_words, kBlock * 4, 4, n);
        hipLaunchKernelGGL(clear_kernel, dim3(b.grid_x, n), dim3(kBlock), 0, as_stream(stream), b);
        if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
    }
    return CNR_OK;
}

cnr_status cnr_clear_bitmap(cnr_ctx *ctx, uint32_t *bitmap, uint64_t n_rows, void *stream) {
    cnr_table_job j = {};
    j.bitmap = bitmap;
    j.n_rows = n_rows;
    return cnr_clear_bitmap_batch(ctx, &j, 1, stream);
}

cnr_status cnr_mark_touched_batch(cnr_ctx *ctx, const cnr_table_job *jobs, uint32_t n_jobs,
                                  cnr_index_type type, void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (type != CNR_IDX_I32 && type != CNR_IDX_I64) return CNR_E_INVALID;
    if (n_jobs && !jobs) return CNR_E_INVALID;
    const uintptr_t align = type == CNR_IDX_I64 ? 8 : 4;
    for (uint32_t i = 0; i < n_jobs; ++i) {
        const cnr_table_job &j = jobs[i];
        if (j.n_rows >= (1ull << 32)) return CNR_E_INVALID;
        if (j.n_indices == 0) continue;
        if (!j.indices || (!j.bitmap && j.n_rows)) return CNR_E_INVALID;
        if (((uintptr_t)j.indices % align) || ((uintptr_t)j.bitmap % 4) || ((uintptr_t)j.mark_scratch % 16))
            return CNR_E_ALIGN;
    }
    hipStream_t s = as_stream(stream);
    for (uint32_t first = 0; first < n_jobs; first += CNR_MAX_BATCH) {
        // Three routes.  Short streams: atomic ORs on the bitmap (about 16 G atomics/s; the other two
        // pay a pass over n_rows bytes or more).  Long streams: bitmap slices in LDS, or one flag byte per row
        // and a fold, as bulk_mark_parts estimates.
        const uint32_t n_here = n_jobs - first < CNR_MAX_BATCH ? n_jobs - first : CNR_MAX_BATCH;
        const uint32_t want_parts = bulk_mark_parts(jobs + first, n_here, type == CNR_IDX_I64 ? 8 : 4, (uint32_t)ctx->n_cu);  // 0: flag bytes
        TrackBatch slices = {}, bulk = {}, direct = {};
        uint32_t n_slices = 0, n_bulk = 0, n_direct = 0;
        bool slices_one = true;     // every table of the slices route is one slice
        uint64_t slices_bytes = 0;  // their streams in all
        uint64_t slices_words = 0, slices_team = 0, bulk_idx = 0, bulk_words = 0, direct_idx = 0;
        for (uint32_t i = first; i < n_jobs && i < first + CNR_MAX_BATCH; ++i) {
            const cnr_table_job &j = jobs[i];
            if (j.n_indices == 0) continue;
            const bool long_stream = bulk_stream(j);
            const uint64_t team = slices_of(j);
            const bool use_slices = long_stream && team <= kSliceTeamMax && want_parts != 0;
            TrackJob &t = use_slices ? slices.job[n_slices++] : long_stream ? bulk.job[n_bulk++] : direct.job[n_direct++];
            t.bitmap = j.bitmap;
            t.n_rows = j.n_rows;
            t.idx = j.indices;
            t.n_idx = j.n_indices;
            t.flags = (uint8_t *)j.mark_scratch;
            const uint64_t words = cnr_bitmap_words(j.n_rows);
            if (use_slices) {
                t.parts = slice_parts(j.n_rows, want_parts);
                if (team * t.parts > slices_team) slices_team = team * t.parts;
                if (team > 1) slices_one = false;
                slices_bytes += j.n_indices * (type == CNR_IDX_I64 ? 8u : 4u);
                if (words > slices_words) slices_words = words;
            } else if (long_stream) {
                if (j.n_indices > bulk_idx) bulk_idx = j.n_indices;
                if (words > bulk_words) bulk_words = words;
            } else if (j.n_indices > direct_idx) {
                direct_idx = j.n_indices;
            }
        }
        if (n_slices) {
            const dim3 grid((unsigned)slices_team, n_slices);  // the most workgroups any table of the launch has
            // Long streams are read past the caches.  With the hint, streams of 64 to 256 MB take 0.56-0.90 of the time
            // where they come from memory (a window's look-ups, marked after other work), 0.93-1.06 where they were
            // written just before and 0.88-1.18 where they are read a second time in a row (the memory-side cache
            // holds 256 MB; eight tables at most 1.09); from 384 MB on it is never the slower way.  Below 64 MB the
            // whole gain is a few microseconds and streams found in the cache are the rule.
            const bool stream = slices_one && slices_bytes >= (64ull << 20);
            if (type == CNR_IDX_I64)
                hipLaunchKernelGGL((stream ? mark_slices_kernel<int64_t, true> : mark_slices_kernel<int64_t, false>), grid,
                                   dim3(kSliceThreads), 0, s, slices, ctx->dev_err);
            else
                hipLaunchKernelGGL((stream ? mark_slices_kernel<int32_t, true> : mark_slices_kernel<int32_t, false>), grid,
                                   dim3(kSliceThreads), 0, s, slices, ctx->dev_err);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
            slices.grid_x = batch_grid_x(ctx, slices_words, kBlock, 8, n_slices);
            hipLaunchKernelGGL(fold_slabs_kernel, dim3(slices.grid_x, n_slices), dim3(kBlock), 0, s, slices);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
        }
        if (n_bulk) {
            // one workgroup per compute unit in all (each fills a unit's LDS), shared out over the tables
            bulk.grid_x = batch_grid_x(ctx, bulk_idx, (uint64_t)kSeenThreads * 8, 1, n_bulk);
            const dim3 grid(bulk.grid_x, n_bulk);
            if (type == CNR_IDX_I64)
                hipLaunchKernelGGL(mark_flags_kernel<int64_t>, grid, dim3(kSeenThreads), 0, s, bulk, ctx->dev_err);
            else
                hipLaunchKernelGGL(mark_flags_kernel<int32_t>, grid, dim3(kSeenThreads), 0, s, bulk, ctx->dev_err);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
            bulk.grid_x = batch_grid_x(ctx, bulk_words, kBlock, 8, n_bulk);
            hipLaunchKernelGGL(fold_flags_kernel, dim3(bulk.grid_x, n_bulk), dim3(kBlock), 0, s, bulk);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
        }
        if (n_direct) {
            direct.grid_x = batch_grid_x(ctx, direct_idx, (uint64_t)kBlock * kMarkUnroll, 8, n_direct);
            const dim3 grid(direct.grid_x, n_direct);
            if (type == CNR_IDX_I64)
                hipLaunchKernelGGL(mark_kernel<int64_t>, grid, dim3(kBlock), 0, s, direct, ctx->dev_err);
            else
                hipLaunchKernelGGL(mark_kernel<int32_t>, grid, dim3(kBlock), 0, s, direct, ctx->dev_err);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
        }
    }
    return CNR_OK;
}

cnr_status cnr_mark_touched(cnr_ctx *ctx, uint32_t *bitmap, uint64_t n_rows, const void *indices,
                            uint64_t n_indices, cnr_index_type type, void *scratch, void *stream) {
    cnr_table_job j = {};
    j.bitmap = bitmap;
    j.n_rows = n_rows;
    j.indices = indices;
    j.n_indices = n_indices;
    j.mark_scratch = scratch;
    return cnr_mark_touched_batch(ctx, &j, 1, type, stream);
}

cnr_status cnr_compact_dirty_batch(cnr_ctx *ctx, const cnr_table_job *jobs, uint32_t n_jobs, void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (n_jobs && !jobs) return CNR_E_INVALID;
    for (uint32_t i = 0; i < n_jobs; ++i) {
        const cnr_table_job &j = jobs[i];
        if (!j.n_dirty_dev || !j.compact_scratch || j.n_rows >= (1ull << 32)) return CNR_E_INVALID;
        if ((!j.bitmap && j.n_rows) || (!j.row_ids && j.capacity)) return CNR_E_INVALID;
        if (((uintptr_t)j.bitmap % 4) || ((uintptr_t)j.row_ids % 4) || ((uintptr_t)j.n_dirty_dev % 8) ||
            ((uintptr_t)j.compact_scratch % 8))
            return CNR_E_ALIGN;
    }
    for (uint32_t first = 0; first < n_jobs; first += CNR_MAX_BATCH) {
        TrackBatch b = {};
        uint32_t n = 0;
        uint64_t max_tiles = 1, tile_pairs = 0;
        for (uint32_t i = first; i < n_jobs && i < first + CNR_MAX_BATCH; ++i, ++n) {
            const cnr_table_job &j = jobs[i];
            b.job[n].bitmap = j.bitmap;
            b.job[n].n_rows = j.n_rows;
            b.job[n].row_ids = j.row_ids;
            b.job[n].capacity = j.capacity;
            b.job[n].n_dirty = j.n_dirty_dev;
            b.job[n].block_count = (uint32_t *)j.compact_scratch;
            const uint64_t tiles = (j.n_rows + kCompactRowsPerBlock - 1) / kCompactRowsPerBlock;
            if (tiles > max_tiles) max_tiles = tiles;
            tile_pairs += tiles * tiles;
        }
        b.grid_x = (uint32_t)max_tiles;
        const dim3 grid(b.grid_x, n);
        if (max_tiles <= kSelfCountTiles && tile_pairs <= kSelfCountPairs) {
            hipLaunchKernelGGL(compact_scatter_kernel<false>, grid, dim3(kBlock), 0, as_stream(stream), b, ctx->dev_err);
        } else {
            hipLaunchKernelGGL(compact_count_kernel, grid, dim3(kBlock), 0, as_stream(stream), b);
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
            hipLaunchKernelGGL(compact_scatter_kernel<true>, grid, dim3(kBlock), 0, as_stream(stream), b, ctx->dev_err);
        }
        if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
    }
    return CNR_OK;
}

cnr_status cnr_compact_dirty(cnr_ctx *ctx, const uint32_t *bitmap, uint64_t n_rows,
                             uint32_t *row_ids, uint64_t capacity, uint64_t *n_dirty_dev,
                             void *scratch, void *stream) {
    cnr_table_job j = {};
    j.bitmap = const_cast<uint32_t *>(bitmap);
    j.n_rows = n_rows;
    j.row_ids = row_ids;
    j.capacity = capacity;
    j.n_dirty_dev = n_dirty_dev;
    j.compact_scratch = scratch;
    return cnr_compact_dirty_batch(ctx, &j, 1, stream);
}

cnr_status cnr_compact_dirty_noalloc(cnr_ctx *ctx, const uint32_t *bitmap, uint64_t n_rows,
                                     uint32_t *row_ids, uint64_t capacity, uint64_t *n_dirty_dev,
                                     void *stream) {
    if (!ctx) return CNR_E_INVALID;
    if (n_rows > CNR_NOALLOC_MAX_ROWS) return CNR_E_TOO_LARGE;
    static_assert(CNR_NOALLOC_SCRATCH_BYTES >= (CNR_NOALLOC_MAX_ROWS / kCompactRowsPerBlock) * sizeof(uint32_t) + 8u,
                  "the fixed scratch holds one count per tile of the largest table");
    if (!ctx->static_scratch || cnr_scratch_bytes(n_rows) > CNR_NOALLOC_SCRATCH_BYTES) return CNR_E_INVALID;
    // from here on the plain call with this device's array as its scratch: argument checks and two
    // kernel launches at most, no allocation
    return cnr_compact_dirty(ctx, bitmap, n_rows, row_ids, capacity, n_dirty_dev, ctx->static_scratch, stream);
}

}  // extern "C"

cnr_status cnr_bind_static_scratch(cnr_ctx *ctx) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return cnr_hip_status(ctx, e);
    if (!p) return cnr_hip_status(ctx, hipErrorInvalidSymbol);
    ctx->static_scratch = p;
    return CNR_OK;
}
