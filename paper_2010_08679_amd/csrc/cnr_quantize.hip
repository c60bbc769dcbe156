// Gather + per-row uniform quantization F_Q + dense packing (Section 5.2, Approaches 1 and 3).
//
// Arithmetic contract (what makes the output comparable with a plain CPU statement of the
// formulas): fp32 throughout, one rounding per operation (the build disables contraction into fused
// multiply-adds), round-half-even, fp32 denormals kept; row minimum, maximum, scale and bias are
// bit-exact; codes may differ from the divide-and-round definition by one step where the quotient
// lies within rounding distance of a half-integer (see the tile kernel).  Error sums that only rank
// candidate ranges are accumulated in fp64.
#include <type_traits>

#include "cnr_common.h"

namespace {

enum { kModeMinMax = CNR_RANGE_MINMAX, kModeGreedy = CNR_RANGE_GREEDY, kModeSymmetric = CNR_RANGE_SYMMETRIC };

// Arguments shared by the quantize kernels.
struct QuantArgs {
    const float *table;
    uint64_t n_rows;
    uint32_t dim;
    const uint32_t *row_ids;
    const uint64_t *n_dev;
    uint64_t n_max;
    int mode;
    uint32_t n_iter;   // greedy iterations
    float num_bins_f;  // greedy num_bins
    float *scale, *bias, *row_min, *row_max;
    uint8_t *codes, *packed;
    cnr_dev_errors *err;
    uint32_t n_waves;  // waves of the grid = the stride of a wave through the list, in passes
};

__device__ __forceinline__ uint64_t row_count(const QuantArgs &a) { return live_rows(a.n_dev, a.n_max); }

// Code of one element as a float in [0, qmax] (F_Q of Section 5.2: clip, subtract the zero point,
// divide by the scale, round).
__device__ __forceinline__ float fq_code_f(float x, float lo, float hi, float scale, float qmaxf) {
    const float c = fminf(fmaxf(x, lo), hi);
    const float t = (c - lo) / scale;
    float q = fminf(fmaxf(rintf(t), 0.0f), qmaxf);
    return scale == 0.0f ? 0.0f : q;
}

// x = scale * x_q + zero_point, product and sum rounded separately.
__device__ __forceinline__ float fq_value(float qf, float scale, float bias) {
    const float p = scale * qf;
    return p + bias;
}

__device__ __forceinline__ double fq_sq_err(float x, float lo, float hi, float scale, float qmaxf) {
    const float d = x - fq_value(fq_code_f(x, lo, hi, scale, qmaxf), scale, lo);
    return (double)d * (double)d;
}

// ---------------------------------------------------------------------------------------------
// Tile kernel (min/max and symmetric range), dim = 64 * M.  Bound by HBM.
//
// A wave works on sixteen consecutive dirty rows per pass, in two lane layouts with a transpose
// through LDS between them:
//   load layout     sixteen lanes share a row: lane l of group g holds elements 64c + 4l .. + 3 of
//                   rows 4g .. 4g + 3 of the pass, so every 16-byte load instruction reads 256
//                   contiguous bytes per row;
//   compute layout  four lanes share a row: lane j of row rho holds the sixteen consecutive elements
//                   64c + 16j .. + 15 of every 64-element chunk c.  The row minimum and maximum then
//                   need only two cross-lane steps, the row's parameters are computed where they are
//                   used, and a lane's sixteen codes are 2 * BITS contiguous bytes of the packed row,
//                   so a wave's packed output is one contiguous run.
// The transpose is private to the wave (LDS operations of one wave complete in order, so no
// barrier is needed); a row's four quarters sit 80 bytes apart and rows 320 bytes apart, which
// spreads the lanes that the LDS serves together over its banks in both directions (what conflicts
// remain cost a few LDS cycles per instruction, far from limiting).
//
// The kernel has to stay clear of the vector-ALU issue limit (a wave64 instruction occupies a SIMD
// for four cycles) to run at the speed of its memory traffic, so the per-element work is pared down:
//   - an element's code is round((x - lo) * (1/scale)); adding 1.5 * 2^23 does the rounding
//     (half-to-even) and leaves the integer in the low mantissa bits, so four codes are merged by
//     three shift-adds and one subtraction of the merged constant.  The product differs from the
//     correctly rounded quotient by at most 1.5 ulp, which can move a code only when the quotient
//     sits within that distance of a half-integer (a few elements in a million at 4 bits); at 8
//     bits, where quotients are larger, one FMA residual step on the quotient removes that too;
//   - the reciprocal must be a normal number: rows with a scale outside [2^-100, 2^100] (denormal
//     or near-overflow ranges) are brought there by an exact power-of-two factor applied to both
//     x - lo and the scale, and a wave takes that variant only if one of its sixteen rows needs it;
//   - rows past the end of the list and row ids outside the table are handled by clamping the
//     addresses that are read and masking what is stored, not by branches.
// ---------------------------------------------------------------------------------------------
// Shapes.  Q = dim / 16.  Rows of 64 elements and more (Q = 4 * M) go through the tile in M chunks of
// 64 elements, with 16 rows per pass, 16 lanes per row in the load layout and 4 in the compute
// layout, as described above.  Rows of 32 and 16 elements (Q = 2, 1) keep 4 KB per pass by taking
// 32 and 64 rows per pass: 8 and 4 lanes per row in the load layout, 2 and 1 in the compute layout
// (a lane still holds 16 consecutive elements).
template <int Q>
struct TileShape {
    static_assert(Q == 1 || Q == 2 || (Q >= 4 && Q % 4 == 0), "row length");
    static constexpr int DIM = 16 * Q;
    static constexpr int LC = Q >= 4 ? 4 : Q;        // lanes per row, compute layout
    static constexpr int M = Q >= 4 ? Q / 4 : 1;     // chunks per row
    static constexpr int CHUNK = DIM / M;            // elements per chunk: 64, 32 or 16
    static constexpr int LR = CHUNK / 4;             // lanes per row, load layout
    static constexpr int ROWS = kWave / LC;          // rows per pass: 16, 32 or 64
    static constexpr int ROW_BYTES = 80 * (CHUNK / 16);  // tile: 16 elements + 16 bytes per segment
};
constexpr int kTileBytes = 5120;  // one wave: ROWS * ROW_BYTES for every shape

template <int LC>
__device__ __forceinline__ float row_lanes_min(float v) {  // over the LC lanes of a row
    if constexpr (LC >= 2) v = fminf(v, dpp_f<0xB1>(v));
    if constexpr (LC >= 4) v = fminf(v, dpp_f<0x4E>(v));
    return v;
}
template <int LC>
__device__ __forceinline__ float row_lanes_max(float v) {
    if constexpr (LC >= 2) v = fmaxf(v, dpp_f<0xB1>(v));
    if constexpr (LC >= 4) v = fmaxf(v, dpp_f<0x4E>(v));
    return v;
}

// Quantizes and stores this lane's 16 * M elements of row k (compute layout): x[c][i] holds elements
// CHUNK * c + 16j + 4i .. + 3.
template <int Q, int BITS>
__device__ __forceinline__ void encode_row_share(const QuantArgs &a, uint64_t k, bool live, int j,
                                                 const float4 (&x)[TileShape<Q>::M][4]) {
    using S = TileShape<Q>;
    constexpr int M = S::M, LC = S::LC, DIM = S::DIM;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    constexpr uint64_t P = (uint64_t)DIM * BITS / 8;  // packed bytes per row
    constexpr float MAGIC = 12582912.0f;              // 1.5 * 2^23: x + MAGIC rounds x to an integer
    constexpr uint32_t MAGIC_BITS = 0x4B400000u;      // bit pattern of MAGIC
    // what four magic-biased codes add up to when merged with shifts of B, 2B, 3B bits
    constexpr uint32_t MERGED_BIAS = MAGIC_BITS * (1u + (1u << BITS) + (1u << (2 * BITS)) + (1u << (3 * BITS)));
    constexpr uint32_t MERGED_BIAS8 = MAGIC_BITS * (1u + (1u << 8) + (1u << 16) + (1u << 24));

    // ---- row minimum / maximum
    float mn = x[0][0].x, mx = x[0][0].x;
#pragma unroll
    for (int c = 0; c < M; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            mn = fminf(fminf(mn, x[c][i].x), fminf(x[c][i].y, fminf(x[c][i].z, x[c][i].w)));
            mx = fmaxf(fmaxf(mx, x[c][i].x), fmaxf(x[c][i].y, fmaxf(x[c][i].z, x[c][i].w)));
        }
    const float X_min = row_lanes_min<LC>(mn) + 0.0f;  // -0.0 -> +0.0
    const float X_max = row_lanes_max<LC>(mx) + 0.0f;
    float lo = X_min, hi = X_max;
    if (a.mode == kModeSymmetric) {
        const float m = fmaxf(fabsf(X_min), fabsf(X_max));
        lo = -m + 0.0f;
        hi = m;
    }

    // ---- the row's parameters: with four lanes per row, lane 0 writes scale, lane 1 bias, lanes 2, 3
    // min, max; with fewer, the lanes there are share them out
    const float scale = (hi - lo) / QMAXF;
    if constexpr (LC == 4) {
        float *dst = j == 0 ? a.scale : j == 1 ? a.bias : j == 2 ? a.row_min : a.row_max;
        const float v = j == 0 ? scale : j == 1 ? lo : j == 2 ? X_min : X_max;
        if (dst && live) store_stream<float>(dst + k, v);
    } else {
        if (live && j == 0) store_stream<float>(a.scale + k, scale);
        if (live && j == LC - 1) store_stream<float>(a.bias + k, lo);
        if (live && j == 0 && a.row_min) store_stream<float>(a.row_min + k, X_min);
        if (live && j == LC - 1 && a.row_max) store_stream<float>(a.row_max + k, X_max);
    }
    const float f = scale < 0x1p-100f ? 0x1p120f : scale > 0x1p100f ? 0x1p-120f : 1.0f;
    const float fscale = scale * f;
    const float inv = scale == 0.0f ? 0.0f : 1.0f / fscale;  // scale 0: every code 0

    // ---- quantize; h[c][i] = the four codes of x[c][i], first element lowest
    uint32_t h[M][4];
    auto quantize_by_reciprocal = [&](auto rescale) {
        constexpr bool RESCALE = decltype(rescale)::value;
        // magic-biased code of one element: MAGIC_BITS + round((x - lo) / scale)
        auto biased = [&](float xv) -> uint32_t {
            float d0 = xv - lo;
            if constexpr (RESCALE) d0 *= f;
            float t = d0 * inv;
            if constexpr (BITS == 8) t = fmaf(fmaf(-t, fscale, d0), inv, t);
            return __float_as_uint(t + MAGIC);
        };
#pragma unroll
        for (int c = 0; c < M; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 v = x[c][i];
                const uint32_t b0 = biased(v.x), b1 = biased(v.y), b2 = biased(v.z), b3 = biased(v.w);
                uint32_t m = (b3 << BITS) + b2;
                m = (m << BITS) + b1;
                h[c][i] = (m << BITS) + b0 - MERGED_BIAS;
                if (a.codes && live)  // one code per byte as well (uniform branch)
                    *reinterpret_cast<uint32_t *>(a.codes + k * (uint64_t)DIM + S::CHUNK * c + 16 * j + 4 * i) =
                        (((((b3 << 8) + b2) << 8) + b1) << 8) + b0 - MERGED_BIAS8;
            }
    };
    if (__builtin_amdgcn_ballot_w64(f != 1.0f) != 0)
        quantize_by_reciprocal(std::true_type{});
    else
        quantize_by_reciprocal(std::false_type{});

#pragma unroll
    for (int c = 0; c < M; ++c) {
        // ---- packed codes: this lane's bits are 2 * BITS contiguous bytes of the row
        if (a.packed) {
            uint8_t *dst = a.packed + k * P + (2 * BITS * LC) * c + (2 * BITS) * j;
            if constexpr (BITS == 8) {
                if (live) store_stream<u32x4>(dst, u32x4{h[c][0], h[c][1], h[c][2], h[c][3]});
            } else if constexpr (BITS == 4) {
                if (live) store_stream<u32x2>(dst, u32x2{h[c][0] | (h[c][1] << 16), h[c][2] | (h[c][3] << 16)});
            } else if constexpr (BITS == 2) {
                if (live) store_stream<uint32_t>(dst, h[c][0] | (h[c][1] << 8) | (h[c][2] << 16) | (h[c][3] << 24));
            } else {  // 3 bits: 48 bits per lane; even lanes append their right neighbour's 48 bits
                const uint32_t w0 = h[c][0] | (h[c][1] << 12) | (h[c][2] << 24);  // stream bits 0..31
                const uint32_t w1 = (h[c][2] >> 8) | (h[c][3] << 4);              // stream bits 32..47
                if constexpr (LC == 1) {  // the row is this lane's 48 bits alone
                    uint16_t *d2 = reinterpret_cast<uint16_t *>(dst);
                    if (live) {
                        d2[0] = (uint16_t)w0;
                        d2[1] = (uint16_t)(w0 >> 16);
                        d2[2] = (uint16_t)w1;
                    }
                } else {
                    const uint32_t n0 = (uint32_t)dpp_i<0xB1>((int)w0);  // lane ^ 1
                    const uint32_t n1 = (uint32_t)dpp_i<0xB1>((int)w1);
                    if (live && !(j & 1)) {
                        uint32_t *d3 = reinterpret_cast<uint32_t *>(dst);
                        store_stream<uint32_t>(d3, w0);
                        store_stream<uint32_t>(d3 + 1, w1 | (n0 << 16));
                        store_stream<uint32_t>(d3 + 2, (n0 >> 16) | (n1 << 16));
                    }
                }
            }
        }
    }
}

// Row ids a lane needs for one pass: of the four rows it helps to load, and of the row it encodes.
struct PassIds {
    uint32_t rid[4];
    uint32_t own;
};

// Ids of pass `pass` of ROWS rows (which must hold at least one row).  Rows past the end repeat the
// last row of the pass; nothing of theirs is stored.
template <int ROWS>
__device__ __forceinline__ void load_pass_ids(const QuantArgs &a, uint64_t n, uint64_t pass, int g, int rho, PassIds &o) {
    const uint64_t base = pass * (uint64_t)ROWS;
    const uint64_t left = n - base;
    const uint32_t rows = left < (uint64_t)ROWS ? (uint32_t)left : (uint32_t)ROWS;  // uniform
    const uint32_t own_i = (uint32_t)rho < rows ? (uint32_t)rho : rows - 1u;
    uint32_t idx[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) idx[u] = (uint32_t)(4 * g + u) < rows ? (uint32_t)(4 * g + u) : rows - 1u;
    if (!a.row_ids) {  // row k of the list is row k of the table; beyond 2^32 - 1: outside any table
        const uint64_t ko = base + own_i;
        o.own = ko > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)ko;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t ku = base + idx[u];
            o.rid[u] = ku > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)ku;
        }
        return;
    }
    o.own = a.row_ids[base + own_i];
    if (rows == (uint32_t)ROWS) {  // one 16-byte load
        const uint4 v = *reinterpret_cast<const uint4 *>(a.row_ids + base + 4u * (uint32_t)g);
        o.rid[0] = v.x; o.rid[1] = v.y; o.rid[2] = v.z; o.rid[3] = v.w;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) o.rid[u] = a.row_ids[base + idx[u]];
    }
}

template <int Q, int BITS>
__device__ __forceinline__ void encode_table(const QuantArgs &a, unsigned char *tile /* this wave's kTileBytes of LDS */) {
    using S = TileShape<Q>;
    constexpr int DIM = S::DIM, M = S::M, ROWS = S::ROWS;
    const uint64_t n = row_count(a);
    const int lane = tid_x() & (kWave - 1);
    const int g = lane / S::LR, l = lane % S::LR;   // load layout: group (four rows), lane in group
    const int rho = lane / S::LC, j = lane % S::LC; // compute layout: row of the pass, share of the row
    const uint32_t last_row = (uint32_t)a.n_rows - 1u;  // the host checks 1 <= n_rows < 2^32
    unsigned char *const wr = tile + (4 * g) * S::ROW_BYTES + (l >> 2) * 80 + (l & 3) * 16;
    const unsigned char *const rd = tile + rho * S::ROW_BYTES + j * 80;

    // Requests this lane's share of the rows of a pass (ids outside the table read the last row
    // instead).
    f32x4 ld[4][M];
    auto gather = [&](const PassIds &ids) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t r = ids.rid[u] < last_row ? ids.rid[u] : last_row;
            const float *src = a.table + (uint64_t)r * DIM + 4u * (uint32_t)l;
#pragma unroll
            for (int c = 0; c < M; ++c) ld[u][c] = load_stream<f32x4>(src + S::CHUNK * c);
        }
    };

    // Software pipeline: while a pass is transposed, quantized and stored, the rows of the wave's
    // next pass and the ids of the one after that are on their way.
    const uint32_t n_waves = a.n_waves;
    uint64_t pass = wave_in_grid();
    if (pass * ROWS >= n) return;
    PassIds ids;
    load_pass_ids<ROWS>(a, n, pass, g, rho, ids);
    gather(ids);
    uint32_t own = ids.own;
    uint64_t next = pass + n_waves;
    if (next * ROWS < n) load_pass_ids<ROWS>(a, n, next, g, rho, ids);
    for (;;) {
        const uint64_t base = pass * (uint64_t)ROWS;  // first row of the pass (uniform)
        const uint64_t left = n - base;
        const uint32_t rows = left < (uint64_t)ROWS ? (uint32_t)left : (uint32_t)ROWS;
        const bool in_table = own <= last_row;
        const bool live = (uint32_t)rho < rows && in_table;
        if ((uint32_t)rho < rows && !in_table && j == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);

        // ---- transpose through the wave's LDS tile, one chunk at a time
        float4 x[M][4];
#pragma unroll
        for (int c = 0; c < M; ++c) {
#pragma unroll
            for (int u = 0; u < 4; ++u) *reinterpret_cast<f32x4 *>(wr + u * S::ROW_BYTES) = ld[u][c];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 4; ++i) x[c][i] = *reinterpret_cast<const float4 *>(rd + 16 * i);
            __builtin_amdgcn_wave_barrier();
        }

        // ---- the load registers are free again: request the next pass
        const bool has_next = next * ROWS < n;  // uniform
        const uint64_t next2 = next + n_waves;
        if (has_next) {
            gather(ids);
            own = ids.own;
            if (next2 * ROWS < n) load_pass_ids<ROWS>(a, n, next2, g, rho, ids);
        }

        encode_row_share<Q, BITS>(a, base + (uint32_t)rho, live, j, x);
        if (!has_next) break;
        pass = next;
        next = next2;
    }
}

// One launch takes up to CNR_MAX_BATCH tables (grid y = table; a slice of a long list counts as a
// table).  Workgroups are handed out x first, so the tables of a launch are swept one after the
// other by all compute units, each on one moving front, with nothing idle between them; a table
// that needs fewer workgroups than the largest of the launch sends the surplus home at once.
// The register budget is pinned to 6 / 4 / 2 waves per SIMD for rows of up to 64 / 128 / 256
// elements: left alone, the compiler lands a few registers to either side of those limits from one
// small change to the next.
template <int N = CNR_MAX_BATCH>
struct QuantBatchArgs {
    QuantArgs job[N];
};
template <int Q, int BITS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(Q <= 4 ? 6 : Q == 8 ? 4 : 2, Q <= 4 ? 6 : Q == 8 ? 4 : 2)))
quantize_tile_kernel(const QuantBatchArgs<> b) {
    __shared__ __align__(16) unsigned char tiles[kWavesPerBlock * kTileBytes];
    // A job behind a reference is loaded again inside the loop, which costs rows of 64 and 256 elements 2 to 7 % (141 K rows of
    // 64, 4 bits, 8.0 -> 7.8 us, 4.2 M 226.4 -> 219.7, at 8 bits 247.5 -> 236.5; 35 K rows of 256 9.8 -> 9.3, 1.05 M 225.9 -> 219.5);
    // rows of 16, 32 and 128 are level (128 at 1.05 M rows 0.4 % slower with a copy).
    using Job = std::conditional_t<Q == 4 || Q == 16, const QuantArgs, const QuantArgs &>;
    Job a = b.job[wg_y()];
    if (wg_x() * kWavesPerBlock >= a.n_waves) return;
    encode_table<Q, BITS>(a, tiles + (tid_x() / kWave) * kTileBytes);
}

// ---------------------------------------------------------------------------------------------
// Greedy range search (Approach 3), dim = 16 * G * L in {16, 32, 64, 128, 256}: L lanes per row, G
// groups of sixteen elements per lane.  Bound by vector-ALU issue: up to 1 + 2 * n_iter candidate ranges are
// tried per row (ClipBound ends most searches early).
//
// Every lane owns 16 * G consecutive elements (4 * G 16-byte loads) of one row, L neighbouring lanes
// own the row, a wave handles 64 / L consecutive dirty rows per pass.  A candidate's error is summed
// over a lane's registers and then over the L lanes with log2(L) DPP exchanges, and a group's sixteen
// codes are exactly 2 * BITS contiguous bytes of the packed row.  What a candidate costs beyond its
// elements (its scale and reciprocal, the exchange between lanes, the comparison) is paid once per
// lane, so more elements per lane mean less of it: with 64 instead of 16 (G = 4; a row of 64 floats
// is then one lane's, with no exchange at all) a long list takes 13 % less time.  A lane then works four times
// as long on a row, so short lists, which cannot fill the SIMDs either way, keep G = 1.  The rows are read in this
// layout directly (each lane its own 64 * G bytes): the kernel is far from the memory system's limits,
// so the transpose through LDS that the tile kernel pays for coalesced loads would buy nothing.
// A candidate is evaluated with the cheapest sequence that still ranks candidates as F_Q would: eight
// vector instructions per element (struct Candidate).  What they cost differs (a loop of nothing but one kind
// takes 1.3 ns per instruction, wave and SIMD for an add or subtract, 1.2 for a multiply with the clamp modifier, 1.9
// for a median, a round or a conversion, 2.0 for a fused multiply-add, 2.05 in fp64; mixed, as here, they take
// less than these add up to, so the figures rank the kinds and are no occupancy), so
// the clip is the free clamp to [0, 1] of the multiply by 1 / (qmax * scale), the rounding is the fused
// multiply-add by qmax onto 2^23, and that biased code, with -2^23 * scale as the addend, gives the
// rounded product scale * code in one fused multiply-add more.  The sequence with a median for the clip
// and a round instruction (nine instructions) took 12.2 ns per element and candidate, this one takes 9.8
// in a loop of its own and 9.2 here; at the published vector rates (fp32 two clocks a wave, fp64 four) the eight
// cannot take less than 7.5.  1.5 M rows of 64, 199 candidates: 3.28 -> 2.70 ms.
// The candidate's scale is range / (2^b - 1) correctly rounded (reciprocal multiply plus one FMA
// residual step), 1 / (qmax * scale) likewise, and the quotient, three roundings in all, is within
// 1.5 ulp of the exact one, which can move a code of a candidate only where the quotient lies that
// close to a half-integer (about 3 elements in a million at 4 bits) and then changes the candidate's
// error by about 1e-7 of itself: a search leaves the path of the divide-as-written sequence only if
// that coincides with two candidates that close, about one row in a few million.  Everything behind the code (product, sum, difference, square, fp64 sum) is
// rounded as the definition rounds it.  A wave holding a row whose scale lies outside [2^-100, 2^100], or
// whose span is only a few float spacings wide, divides instead.  The final codes of the chosen range
// are produced by division, exactly as F_Q is written.
// ---------------------------------------------------------------------------------------------
template <int L>
__device__ __forceinline__ float lanes_min(float v) {
    if constexpr (L >= 2) v = fminf(v, dpp_f<0xB1>(v));
    if constexpr (L >= 4) v = fminf(v, dpp_f<0x4E>(v));
    if constexpr (L >= 8) v = fminf(v, dpp_f<0x141>(v));
    if constexpr (L >= 16) v = fminf(v, dpp_f<0x140>(v));
    if constexpr (L >= 32) v = fminf(v, __shfl_xor(v, 16));
    if constexpr (L >= 64) v = fminf(v, __shfl_xor(v, 32));
    return v;
}
template <int L>
__device__ __forceinline__ float lanes_max(float v) {
    if constexpr (L >= 2) v = fmaxf(v, dpp_f<0xB1>(v));
    if constexpr (L >= 4) v = fmaxf(v, dpp_f<0x4E>(v));
    if constexpr (L >= 8) v = fmaxf(v, dpp_f<0x141>(v));
    if constexpr (L >= 16) v = fmaxf(v, dpp_f<0x140>(v));
    if constexpr (L >= 32) v = fmaxf(v, __shfl_xor(v, 16));
    if constexpr (L >= 64) v = fmaxf(v, __shfl_xor(v, 32));
    return v;
}
template <int L>
__device__ __forceinline__ float lanes_sum(float v) {
    if constexpr (L >= 2) v += dpp_f<0xB1>(v);
    if constexpr (L >= 4) v += dpp_f<0x4E>(v);
    if constexpr (L >= 8) v += dpp_f<0x141>(v);
    if constexpr (L >= 16) v += dpp_f<0x140>(v);
    if constexpr (L >= 32) v += __shfl_xor(v, 16);
    if constexpr (L >= 64) v += __shfl_xor(v, 32);
    return v;
}
template <int L>
__device__ __forceinline__ double lanes_sum(double v) {
    if constexpr (L >= 2) v += dpp_d<0xB1>(v);
    if constexpr (L >= 4) v += dpp_d<0x4E>(v);
    if constexpr (L >= 8) v += dpp_d<0x141>(v);
    if constexpr (L >= 16) v += dpp_d<0x140>(v);
    if constexpr (L >= 32) v += __shfl_xor(v, 16);
    if constexpr (L >= 64) v += __shfl_xor(v, 32);
    return v;
}

// One candidate range: what the error of an element needs.
template <int BITS>
struct Candidate {
    static constexpr float QMAXF = (float)((1 << BITS) - 1);
    float lo, scale, inv;  // inv = 1 / (qmax * scale)
    float unbias;          // -2^23 * scale
    __device__ __forceinline__ Candidate(float c_lo, float c_hi) {
        constexpr float INV_QMAX = 1.0f / QMAXF;
        const float range = c_hi - c_lo;
        const float q0 = range * INV_QMAX;
        lo = c_lo;
        scale = fmaf(fmaf(-q0, QMAXF, range), INV_QMAX, q0);
        const float full = scale * QMAXF, rest = fmaf(scale, QMAXF, -full);  // qmax * scale in two pieces
        const float r0 = __builtin_amdgcn_rcpf(full);
        inv = scale == 0.0f ? 0.0f : fmaf(fmaf(-rest, r0, fmaf(-full, r0, 1.0f)), r0, r0);
        unbias = scale * -0x1p23f;
    }
    // acc += (x - F_Q(x) de-quantized)^2 of N elements (eight, or four that are left over).  Left to itself the compiler strings the
    // eight instructions of one element behind each other, each waiting for the one before; the barriers
    // keep them in stages of eight independent ones (2.99 -> 2.70 ms on the list above; stages of four or
    // sixteen 2.97).
    template <int N>
    __device__ __forceinline__ void add_err(double &acc, const float (&x)[N]) const {
        float t[N];
        double d[N];
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = x[i] - lo;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = __builtin_amdgcn_fmed3f(t[i] * inv, 0.0f, 1.0f);  // the multiply's clamp modifier
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = fmaf(t[i], QMAXF, 0x1p23f);  // 2^23 + code
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = fmaf(t[i], scale, unbias);   // scale * code
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = t[i] + lo;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = x[i] - t[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) d[i] = (double)t[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) acc = fma(d[i], d[i], acc);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// An error counts as the smaller of two when it is below tie_factor(dim) times the other.  Two candidate
// ranges can have exactly the same error: where a step is a whole number of code steps, moving the range by
// a step moves its grid onto itself, and the row's two ends, clipped by a step each, swap their errors.  The
// fp64 sums of such a pair differ by their rounding alone, which depends on the lanes that a row is spread
// over, that is on the length of the list; taken for a difference it gave the same row another range in a
// longer list (rows with one far element at either end: 12 in 1000 of 16 floats at 2 bits and 4 bins, 2 of 200 at 3 and 12).  A sum has at most min(dim, 72) roundings
// on its way in every kernel here (17 units in one lane, and the exchange between lanes), so equal sums are
// found equal, and a tie moves the upper bound wherever the row is searched.  (CPU emulation, 120 K rows of
// 4 to 1000 elements: sums that differ at all do so by more than 2^-47 of themselves.)
inline double tie_factor(uint32_t dim) { return 1.0 - (double)(dim < 72u ? dim : 72u) * 0x1p-52; }

// Whether a wave's rows (this lane's with range [lo, hi]) have to be searched with divisions, as F_Q is
// written.  Scales outside [2^-100, 2^100] are: their reciprocals are no normal numbers.  So are narrow
// rows: the bounds are moved by cumulative fp32 additions, each rounded to the spacing of the bounds'
// magnitude, so after k moves a bound sits up to k/2 spacings off the exact lattice.  Where the step is not
// many spacings wide (a row whose span is tiny against its magnitude) a candidate range can close or turn
// inside out before the search ends, and there the clamped quotient of the fast sequence is no longer that
// of min(max(x, lo), hi).  Safe when range >= num_bins^2 spacings (twice the drift num_bins moves allow).
__device__ __forceinline__ bool search_divides(float lo, float hi, float num_bins_f, float qmaxf) {
    const float s0 = (hi - lo) * (1.0f / qmaxf);
    const bool odd_scale = s0 != 0.0f && !(s0 >= 0x1p-100f && s0 <= 0x1p100f);
    const float mag = fmaxf(fabsf(lo), fabsf(hi));
    const bool narrow = hi != lo && (hi - lo) < num_bins_f * num_bins_f * (mag * 0x1p-23f);
    // the last candidates are up to num_bins times narrower than the first
    return __builtin_amdgcn_ballot_w64(odd_scale || narrow) != 0 || num_bins_f > kFastSearchBins;
}

// What ends a search early: a lower bound for the error of every candidate still to come.  Candidate ranges are
// nested, so an element that a range clips stays clipped, at least as far, in all later ones, and
// its clipping error is part of their errors.  Each lane keeps the smallest and the largest element of every N-th
// part of its share of the row and adds up the squares of what those are clipped by; every candidate still to come lies within one of
// the next iteration's two, so once the row's sums for both reach the
// best error, no later candidate can be strictly smaller and the range is the one that the whole search would end
// with.  It holds for the computed errors as well: below, a clipped element's code is 0, its restored value
// the candidate's bound itself, and the difference is rounded here as there; above, the restored value scale * qmax + lo
// lies within seven half-spacings of the row's largest magnitude of the candidate's bound, and `slack` is twice
// that and more.  The sums here are in fp32, of differences in units of a power of two near the row's range; 2^-16
// covers their rounding.  (All this for scales that are normal numbers: the sequence without divisions.)
// 1.5 M rows of 64 at 100 bins and 4 bits stop after 20 of 99 iterations (with every element's clipping error: 20 too,
// the row's two ends alone: 20), at 2 bits and 25 bins after 17 of 24, at 8 bits before the first: 2.69 -> 0.63 ms and 0.73 -> 0.56.  Asked about the
// current range instead of the next two, every search took one iteration more: 1.5 M rows of 64 at 3 bits and 25 bins 377 -> 352 us now,
// 4 bits and 45 bins 358 -> 333, 100 bins 653 -> 630, 1.2 M rows of 16 58 -> 47, 8 bits 32 -> 27 (0.3 M rows of 64 29 -> 24).  Rows of 8
// to 512 elements at 4 bits and 45 bins 1.4 to 6 times as fast as without an end, at 8 bits 4 to 5 times.  At 2 bits it depends on the rows: whole
// searches of 1024 elements 1.6 times as fast on evenly spread values, 1.3 on normal ones, and a few per cent slower than without an end where outliers
// let the search go on to nine tenths of its iterations (25 bins: 1 K rows of 1024 23.5 -> 24.9 us, of 320 15.8 -> 16.2; 10 K and more
// within 3 %), as are searches that stop by themselves about where rows would be finished (1 K rows of 320 at 4 bits, 45 bins, ratio 0.4, 13.1 -> 14.6).
// Short lists are up to 13 % slower or 10 % faster by where their loop lies in the code: a few waves then wait for their own
// instructions (1.7 K rows of 16 at 2 bits and 94 bins 14.0 us where the loop begins at byte 36 of a line of 128, 16.2 at byte 116, 15.6 at 0; the
// same instructions).  Loops aligned throughout win and lose as much: rows of 96 38.8 -> 34.6, of 24 19.5 -> 21.4, 1.5 M rows of 64 at 100 bins 626 -> 668.
template <int N>
struct ClipBound {
    float mn[N], mx[N];
    float unit, slack;
    double enough;  // the bound is compared with the best error times this
    // Ends that no element has: parts may stay empty.
    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int g = 0; g < N; ++g) {
            mn[g] = __builtin_huge_valf();
            mx[g] = -__builtin_huge_valf();
        }
    }
    __device__ __forceinline__ void start(int g, const float4 &v) {
        mn[g] = mx[g] = v.x;
        take(g, v);
    }
    __device__ __forceinline__ void take(int g, const float4 &v) {
        mn[g] = fminf(mn[g], fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
        mx[g] = fmaxf(mx[g], fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
    }
    __device__ __forceinline__ float lane_min() const {
        float v = mn[0];
#pragma unroll
        for (int g = 1; g < N; ++g) v = fminf(v, mn[g]);
        return v;
    }
    __device__ __forceinline__ float lane_max() const {
        float v = mx[0];
#pragma unroll
        for (int g = 1; g < N; ++g) v = fmaxf(v, mx[g]);
        return v;
    }
    // To units of the row's range [lo, hi].
    __device__ __forceinline__ void rescale(float lo, float hi) {
        const uint32_t exponent = __float_as_uint(hi - lo) >> 23;  // 1 to 253, or 0 for a constant row
        unit = hi == lo ? 1.0f : __uint_as_float((254u - exponent) << 23);
        slack = fmaxf(fabsf(lo), fabsf(hi)) * unit * 0x1p-20f;
        enough = (double)unit * (double)unit * (1.0 + 0x1p-16);
#pragma unroll
        for (int g = 0; g < N; ++g) {
            mn[g] *= unit;
            mx[g] *= unit;
        }
    }
    // Whether what a row of L lanes is clipped by at [lo, hi] comes to its best error.  All lanes have to call it.
    template <int L>
    __device__ __forceinline__ bool reached(float lo, float hi, double best) const {
        const float from = lo * unit, to = fmaf(hi, unit, slack);
        float e = 0.0f;
#pragma unroll
        for (int g = 0; g < N; ++g) {
            const float below = fmaxf(from - mn[g], 0.0f), above = fmaxf(mx[g] - to, 0.0f);
            e = fmaf(below, below, e);
            e = fmaf(above, above, e);
        }
        return (double)lanes_sum<L>(e) >= best * enough;
    }
};
// Whether it is worth asking: a candidate's error is well above the bound, since the elements within its range
// have errors too.  (At 2 bits a search stops where its error is about 1.2 times the best, at 4 bits 1.7; an eighth
// of a binade more in the errors' upper halves is 1.06 to 1.125 times.)  ZERO: where the best may be 0, no later error can be
// smaller, and the question is worth asking whatever the error.
template <bool ZERO>
__device__ __forceinline__ bool may_be_done(double error, double best) {
    const int b = __double2hiint(best);
    return __double2hiint(error) >= b + (ZERO ? min(b, 1 << 17) : 1 << 17);
}

// The 24 code bits of a pair of units at 3 bits.
__device__ __forceinline__ void store_pair3(uint8_t *out, uint32_t pair, uint32_t w) {
    uint8_t *o3 = out + 3 * pair;
    o3[0] = (uint8_t)w;
    o3[1] = (uint8_t)(w >> 8);
    o3[2] = (uint8_t)(w >> 16);
}
// Stores the 4 * BITS code bits h of unit u (elements 4u .. 4u + 3) of a packed row.  At 3 bits units come
// in pairs (dim % 8 == 0): unit u + 1 is lane + 1's, and the lane of the even one stores both; all lanes
// have to call it.
template <int BITS>
__device__ __forceinline__ void store_unit_codes(uint8_t *out, uint32_t u, uint32_t h, bool store) {
    if constexpr (BITS == 8) {
        if (store) *reinterpret_cast<uint32_t *>(out + 4 * u) = h;
    } else if constexpr (BITS == 4) {
        if (store) *reinterpret_cast<uint16_t *>(out + 2 * u) = (uint16_t)h;
    } else if constexpr (BITS == 2) {
        if (store) out[u] = (uint8_t)h;
    } else {
        const uint32_t nb = (uint32_t)dpp_i<0xB1>((int)h);  // lane ^ 1: unit u + 1
        if (store && !(u & 1)) store_pair3(out, u >> 1, h | (nb << 12));
    }
}

// Rows of the n of a list that the waves of a grid of n_waves search.
template <int L, int BITS, int G, bool ENDS>
__device__ __forceinline__ void search_rows(const QuantArgs &a, double less /* tie_factor(dim) */, uint64_t n, uint32_t n_waves) {
    constexpr int EPL = 16 * G;  // elements per lane
    constexpr int DIM = EPL * L;
    constexpr int kRowsPerPass = kWave / L;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    constexpr uint64_t P = (uint64_t)DIM * BITS / 8;  // packed bytes per row
    const int lane = tid_x() & (kWave - 1);
    const int j = lane % L;  // lane within the row
    for (uint64_t pass = wave_in_grid(); pass * kRowsPerPass < n; pass += n_waves) {
        const uint64_t k = pass * kRowsPerPass + lane / L;
        // ---- gather
        uint64_t rid = 0;
        bool live = k < n;
        if (live) {
            rid = a.row_ids ? (uint64_t)a.row_ids[k] : k;
            if (rid >= a.n_rows) {
                if (j == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);
                live = false;
                rid = 0;
            }
        }
        float4 x[4 * G];
        {
            const float *src = a.table + rid * (uint64_t)DIM + (uint64_t)(EPL * j);
#pragma unroll
            for (int i = 0; i < 4 * G; ++i) x[i] = *reinterpret_cast<const float4 *>(src + 4 * i);
        }

        // ---- row minimum / maximum
        ClipBound<G> clip;
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) i % 4 ? clip.take(i / 4, x[i]) : clip.start(i / 4, x[i]);
        const float X_min = lanes_min<L>(clip.lane_min()) + 0.0f;  // -0.0 -> +0.0
        const float X_max = lanes_max<L>(clip.lane_max()) + 0.0f;
        float lo = X_min, hi = X_max;

        // ---- the search: shrink from whichever side hurts less, remember the best range seen
        auto search = [&](auto fast_tag) {
            constexpr bool FAST = decltype(fast_tag)::value;
            auto row_err = [&](float c_lo, float c_hi) -> double {
                double e = 0.0;
                if constexpr (FAST) {
                    const Candidate<BITS> c(c_lo, c_hi);
#pragma unroll
                    for (int i = 0; i < 4 * G; i += 2)
                        c.template add_err<8>(e, {x[i].x, x[i].y, x[i].z, x[i].w, x[i + 1].x, x[i + 1].y, x[i + 1].z, x[i + 1].w});
                } else {
                    const float s = (c_hi - c_lo) / QMAXF;
#pragma unroll
                    for (int i = 0; i < 4 * G; ++i) {
                        e += fq_sq_err(x[i].x, c_lo, c_hi, s, QMAXF);
                        e += fq_sq_err(x[i].y, c_lo, c_hi, s, QMAXF);
                        e += fq_sq_err(x[i].z, c_lo, c_hi, s, QMAXF);
                        e += fq_sq_err(x[i].w, c_lo, c_hi, s, QMAXF);
                    }
                }
                return lanes_sum<L>(e);
            };
            float cur_lo = lo, cur_hi = hi;
            const float step = (hi - lo) / a.num_bins_f;
            if constexpr (FAST && ENDS) clip.rescale(lo, hi);
            double best = row_err(lo, hi);
            // Rows that keep the wave searching.  Not those without an error from the start: constant rows, or two values far
            // apart; one such row in 64 kept every wave of a list to its last iteration (1.5 M rows of 64 at 4 bits and 100 bins 2580 us
            // with them, 655 now, 660 without any).  (ZERO instead of this mask: rows of 16 at 3 bits 131 -> 146 us.)
            const bool open = live & (best != 0.0);
            uint32_t n_iter = a.n_iter;
            auto finished = [&]() -> bool {  // the wave: neither of the next two ranges can lead any row below its best
                if (__builtin_amdgcn_ballot_w64(open & !clip.template reached<L>(cur_lo + step, cur_hi, best)) != 0) return false;
                return __builtin_amdgcn_ballot_w64(open & !clip.template reached<L>(cur_lo, cur_hi - step, best)) == 0;
            };
            // At 8 bits a step is several code steps as a rule, and no iteration is needed.  (Asked at 2 to 4 bits too, where it takes 10 bins
            // or fewer for that, 1.5 M rows of 64 at 100 bins took 650 us instead of 630.)
            if constexpr (FAST && ENDS && BITS == 8) {
                if (finished()) n_iter = 0;
            }
            for (uint32_t it = 0; it < n_iter; ++it) {
                const float c_lo = cur_lo + step;
                const float c_hi = cur_hi - step;
                const double limit = best * less;
                const double e_lo = row_err(c_lo, cur_hi);
                const double e_hi = row_err(cur_lo, c_hi);
                const bool move_lo = e_lo < e_hi * less;
                cur_lo = move_lo ? c_lo : cur_lo;
                cur_hi = move_lo ? cur_hi : c_hi;
                const double e = move_lo ? e_lo : e_hi;
                const bool found = e < limit;
                best = found ? e : best;
                lo = found ? cur_lo : lo;
                hi = found ? cur_hi : hi;
                if constexpr (FAST && ENDS) {
                    if (__builtin_amdgcn_ballot_w64(open & !may_be_done<false>(e, best)) == 0 && finished()) n_iter = it;
                }
            }
        };
        if (search_divides(lo, hi, a.num_bins_f, QMAXF))
            search(std::false_type{});
        else
            search(std::true_type{});

        // ---- per-row parameters: lane 0 of the row writes scale, lane 1 bias, lanes 2, 3 min, max
        // (with fewer than four lanes per row, the lanes there are share them out)
        const float scale = (hi - lo) / QMAXF;
        if constexpr (L >= 4) {
            float *dst = j == 0 ? a.scale : j == 1 ? a.bias : j == 2 ? a.row_min : a.row_max;
            const float v = j == 0 ? scale : j == 1 ? lo : j == 2 ? X_min : X_max;
            if (j < 4 && dst && live) dst[k] = v;
        } else {
            if (live && j == 0) a.scale[k] = scale;
            if (live && j == L - 1) a.bias[k] = lo;
            if (live && j == 0 && a.row_min) a.row_min[k] = X_min;
            if (live && j == L - 1 && a.row_max) a.row_max[k] = X_max;
        }

        // ---- final codes by F_Q as written, sixteen elements at a time; h[i] = four codes, first element
        // lowest.  Packed, this lane's bits are bytes [2 * BITS * G * j, 2 * BITS * G * (j + 1)) of the row,
        // 2 * BITS bytes per group of sixteen elements
        uint8_t *const packed = a.packed ? a.packed + k * P + 2 * BITS * G * j : nullptr;
        uint32_t even_w0 = 0, even_w1 = 0;  // 3 bits: the 48 bits of the group before
#pragma unroll
        for (int g = 0; g < G; ++g) {
            uint32_t h[4], h8[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 v = x[4 * g + i];
                const uint32_t q0 = (uint32_t)fq_code_f(v.x, lo, hi, scale, QMAXF);
                const uint32_t q1 = (uint32_t)fq_code_f(v.y, lo, hi, scale, QMAXF);
                const uint32_t q2 = (uint32_t)fq_code_f(v.z, lo, hi, scale, QMAXF);
                const uint32_t q3 = (uint32_t)fq_code_f(v.w, lo, hi, scale, QMAXF);
                h[i] = q0 | (q1 << BITS) | (q2 << (2 * BITS)) | (q3 << (3 * BITS));
                h8[i] = q0 | (q1 << 8) | (q2 << 16) | (q3 << 24);
            }
            if (a.codes && live)
                *reinterpret_cast<uint4 *>(a.codes + k * (uint64_t)DIM + EPL * j + 16 * g) = make_uint4(h8[0], h8[1], h8[2], h8[3]);
            if (!packed) continue;  // uniform
            uint8_t *dst = packed + 2 * BITS * g;
            if constexpr (BITS == 8) {
                if (live) *reinterpret_cast<uint4 *>(dst) = make_uint4(h[0], h[1], h[2], h[3]);
            } else if constexpr (BITS == 4) {
                if (live) *reinterpret_cast<uint2 *>(dst) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            } else if constexpr (BITS == 2) {
                if (live) *reinterpret_cast<uint32_t *>(dst) = h[0] | (h[1] << 8) | (h[2] << 16) | (h[3] << 24);
            } else {  // 3 bits: 48 bits per group
                const uint32_t w0 = h[0] | (h[1] << 12) | (h[2] << 24);  // stream bits 0..31 of the group
                const uint32_t w1 = (h[2] >> 8) | (h[3] << 4);           // stream bits 32..47
                if constexpr (G >= 2) {  // two groups make three whole words
                    if (g & 1) {
                        uint32_t *d3 = reinterpret_cast<uint32_t *>(dst - 6);
                        if (live) {
                            d3[0] = even_w0;
                            d3[1] = even_w1 | (w0 << 16);
                            d3[2] = (w0 >> 16) | (w1 << 16);
                        }
                    } else {
                        even_w0 = w0;
                        even_w1 = w1;
                    }
                } else if constexpr (L == 1) {  // the row is this lane's 48 bits alone
                    uint16_t *d2 = reinterpret_cast<uint16_t *>(dst);
                    if (live) {
                        d2[0] = (uint16_t)w0;
                        d2[1] = (uint16_t)(w0 >> 16);
                        d2[2] = (uint16_t)w1;
                    }
                } else {  // even lanes append their right neighbour's 48 bits
                    const uint32_t n0 = (uint32_t)dpp_i<0xB1>((int)w0);  // lane ^ 1
                    const uint32_t n1 = (uint32_t)dpp_i<0xB1>((int)w1);
                    if (live && !(j & 1)) {
                        uint32_t *d3 = reinterpret_cast<uint32_t *>(dst);
                        d3[0] = w0;
                        d3[1] = w1 | (n0 << 16);
                        d3[2] = (n0 >> 16) | (n1 << 16);
                    }
                }
            }
        }
    }
}

template <int L, int BITS, int G, bool ENDS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(L == 1 && G == 4 ? 3 : G == 4 ? 4 : 5, 8))) quantize_greedy_kernel(const QuantArgs a, double less) {
    search_rows<L, BITS, G, ENDS>(a, less, row_count(a), a.n_waves);
}
// Lists whose length only the device knows, in buffers that may hold long ones: fewer than `line` rows go as L_NARROW lanes of sixteen elements
// each, more as L_WIDE of 16 * G_WIDE.  Two launches, of which one found that the list was the other's, were 2 to 5 us more (500 rows of 64 at 45 bins
// and 4 bits in a capacity of 655 K 11.7 -> 9.0 us, 52 K 23.5 -> 21.0, 131 K rows of 256 208 -> 196).  Together the forms have the registers of the
// wide one, which costs lists below the line a wave per SIMD and no time that shows.
template <int L_NARROW, int L_WIDE, int G_WIDE, int BITS, bool ENDS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(L_WIDE == 1 && G_WIDE == 4 ? 3 : 4, 8)))
quantize_greedy_pair_kernel(const QuantArgs a, double less, uint64_t line, uint32_t narrow_waves) {
    const uint64_t n = row_count(a);
    if (n >= line) search_rows<L_WIDE, BITS, G_WIDE, ENDS>(a, less, n, a.n_waves);
    else if (wave_in_grid() < narrow_waves) search_rows<L_NARROW, BITS, 1, ENDS>(a, less, n, narrow_waves);
}

// ---------------------------------------------------------------------------------------------
// Greedy search at any other dim (dim % 4 == 0, dim * bits % 8 == 0): L lanes per row, lane j holds the
// row's 16-byte units j, j + L, ... in registers, up to UMAX of them that every lane has plus the last,
// which only some have.  How many there are is known at run time and the same for all lanes, so the units
// are walked in pairs (eight elements, as above) behind uniform branches; an odd unit and the partial one
// follow as fours, and a lane without a partial unit evaluates elements that equal the candidate's lower
// bound, whose error is zero.  Candidates go through one copy of the code: the un-shrunk range first,
// then the two of every iteration, in turn or side by side.  Same bound and same arithmetic as the kernel
// above.
// Side by side (DUAL): a short list is bound not by issue but by one candidate's chain of dependent
// instructions (range to scale to reciprocal, the sum over the lanes, the comparison), so two groups of L
// lanes hold the row, one evaluates the raised lower bound and the other the lowered upper one.  (A wave
// per row that re-read the row from cache and divided for every element: 100 K rows of 96 at 49
// candidates 874 us, this 106 us.)  The waves that waves_per_eu asks for cost spilled registers: in the 16-unit forms 2 at
// 2 bits and 30 at 3 and 4, in some 8-unit forms 4 to 8, where a search may end early 10 to 12 and 6 to 8 more for the ends it keeps, and 2 to 26 in the
// kernels of both forms.
// All of them are stored and reloaded outside the loop over the candidates, once per pass.
// ---------------------------------------------------------------------------------------------
// What the same lane of the row's other group of L lanes holds.  (The mirrors reverse the lanes, which is
// the same for values that all lanes of a group agree on.)
template <int L>
__device__ __forceinline__ double other_group(double v) {
    if constexpr (L == 4) return dpp_d<0x141>(v);
    else if constexpr (L == 8) return dpp_d<0x140>(v);
    else return __shfl_xor(v, L);
}

template <int L, int UMAX, bool DUAL>
struct RowUnits {
    static_assert(UMAX % 2 == 0, "units are walked in pairs");
    static_assert(!DUAL || L <= 32, "two groups of lanes fit a wave");
    static constexpr int LANES = DUAL ? 2 * L : L;  // per row
    float4 x[UMAX];   // units j + L * t, t < 2 * pairs
    float4 odd;       // unit j + L * 2 * pairs, if has_odd
    float4 tail;      // unit j + L * n_full, if in_tail
    const float4 *row;
    uint32_t n4, j;
    uint32_t pairs;
    bool has_odd, has_tail;  // uniform
    bool in_tail;            // this lane
    ClipBound<(UMAX + 3) / 4> clip;

    __device__ __forceinline__ void load(const float4 *row_, uint32_t n4_, uint32_t j_) {
        row = row_;
        n4 = n4_;
        j = j_;
        const uint32_t n_full = n4 / L;
        pairs = n_full / 2;
        has_odd = n_full & 1;
        has_tail = n4 % L != 0;
        in_tail = j + L * n_full < n4;
#pragma unroll
        for (int t = 0; t < UMAX; t += 2)
            if ((uint32_t)t < 2 * pairs) {
                x[t] = row[j + L * t];
                x[t + 1] = row[j + L * (t + 1)];
            }
        tail = row[in_tail ? j + L * n_full : n4 - 1];  // a unit of the row in any case, though only an in_tail lane's counts
        odd = tail;
        if (has_odd) odd = row[j + L * (n_full - 1)];
    }
    __device__ __forceinline__ void range(float &mn, float &mx) {
        clip.reset();
        if (in_tail) clip.take(0, tail);
        if (has_odd) clip.take(0, odd);
#pragma unroll
        for (int t = 0; t < UMAX; t += 2)
            if ((uint32_t)t < 2 * pairs) {
                clip.take(t / 4, x[t]);
                clip.take(t / 4, x[t + 1]);
            }
        mn = lanes_min<L>(clip.lane_min()) + 0.0f;  // -0.0 -> +0.0
        mx = lanes_max<L>(clip.lane_max()) + 0.0f;
        if (mn > mx) mn = mx = tail.x;  // none of the row's elements is above or below anything: all of them are NaN, and so is its range
    }
    // Squared l2 error of the row under F_Q with the range [c_lo, c_hi], in every lane.
    template <int BITS, bool FAST>
    __device__ __forceinline__ double sq_err(float c_lo, float c_hi) const {
        double e = 0.0;
        if constexpr (FAST) {
            const Candidate<BITS> c(c_lo, c_hi);
#pragma unroll
            for (int t = 0; t < UMAX; t += 2)
                if ((uint32_t)t < 2 * pairs)
                    c.template add_err<8>(e, {x[t].x, x[t].y, x[t].z, x[t].w, x[t + 1].x, x[t + 1].y, x[t + 1].z, x[t + 1].w});
            if (has_odd) c.template add_err<4>(e, {odd.x, odd.y, odd.z, odd.w});
            if (has_tail)
                c.template add_err<4>(e, {in_tail ? tail.x : c_lo, in_tail ? tail.y : c_lo, in_tail ? tail.z : c_lo, in_tail ? tail.w : c_lo});
        } else {
            constexpr float QMAXF = (float)((1 << BITS) - 1);
            const float s = (c_hi - c_lo) / QMAXF;
            for (uint32_t u = j; u < n4; u += L) {  // rare, and its code is long: a loop that re-reads the row
                const float4 v = row[u];
                e += fq_sq_err(v.x, c_lo, c_hi, s, QMAXF);
                e += fq_sq_err(v.y, c_lo, c_hi, s, QMAXF);
                e += fq_sq_err(v.z, c_lo, c_hi, s, QMAXF);
                e += fq_sq_err(v.w, c_lo, c_hi, s, QMAXF);
            }
        }
        return lanes_sum<L>(e);
    }
    // The search (header: cnr_greedy_params): [lo, hi] comes in as the row's range and leaves as the chosen one;
    // rows that are not live do not keep it going.  ENDS: it ends early where it can.
    template <int BITS, bool FAST, bool ENDS>
    __device__ __forceinline__ void search(uint32_t n_iter, float num_bins_f, double less, bool live, float &lo, float &hi) {
        Search<BITS, FAST, ENDS> s(*this, num_bins_f, less, live, lo, hi);
        s.run(n_iter, lo, hi);
    }
    // A search in steps: run(n, ...) takes it on to the end of iteration n, where [lo, hi] is what a search of n iterations
    // ends with.
    template <int BITS, bool FAST, bool ENDS>
    struct Search {
        using Count = std::conditional_t<FAST, uint32_t, uint64_t>;
        RowUnits &row;
        const float step;
        const double less;
        const uint64_t live_rows;
        const bool upper;  // this lane's group lowers the upper bound
        float cur_lo, cur_hi;
        // The first candidate is an iteration whose step is zero.
        float move = 0.0f;
        double best = __builtin_huge_val(), e_lo = best;
        Count c = 0;
        bool over = false;  // the wave's rows are finished: more iterations change nothing

        __device__ __forceinline__ Search(RowUnits &row_, float num_bins_f, double less_, bool live, float lo, float hi)
            : row(row_), step((hi - lo) / num_bins_f), less(less_), live_rows(__builtin_amdgcn_ballot_w64(live)), upper(DUAL && (tid_x() / L) & 1),
              cur_lo(lo), cur_hi(hi) {
            if constexpr (FAST && ENDS) row.clip.rescale(lo, hi);
        }
        __device__ __forceinline__ void run(uint32_t n_iter, float &lo, float &hi) {
            Count last = last_candidate<Count>(n_iter, DUAL);
            for (; c <= last; ++c) {
                const bool raise = DUAL ? !upper : (c & 1);  // uniform, but for DUAL
                const float c_lo = raise ? cur_lo + move : cur_lo;
                const float c_hi = raise ? cur_hi : cur_hi - move;
                const double limit = best * less;
                double e = row.template sq_err<BITS, FAST>(c_lo, c_hi);
                if (!DUAL && raise) {
                    e_lo = e;
                } else {
                    if constexpr (DUAL) {
                        const double o = other_group<L>(e);
                        e_lo = upper ? o : e;
                        e = upper ? e : o;
                    }
                    const bool move_lo = e_lo < e * less;
                    cur_hi = move_lo ? cur_hi : cur_hi - move;
                    cur_lo = move_lo ? cur_lo + move : cur_lo;
                    const double better = move_lo ? e_lo : e;
                    const bool found = better < limit;
                    best = found ? better : best;
                    lo = found ? cur_lo : lo;
                    hi = found ? cur_hi : hi;
                    move = step;
                    if constexpr (FAST && ENDS) {
                        if ((BITS == 8 && c == 0) || (__builtin_amdgcn_ballot_w64(!may_be_done<true>(better, best)) & live_rows) == 0) {
                            // side by side, each group asks for the bound that it moves
                            bool going = (__builtin_amdgcn_ballot_w64(!row.clip.template reached<L>(upper ? cur_lo : cur_lo + step, upper ? cur_hi - step : cur_hi, best)) & live_rows) != 0;
                            if (!DUAL && !going)
                                going = (__builtin_amdgcn_ballot_w64(!row.clip.template reached<L>(cur_lo, cur_hi - step, best)) & live_rows) != 0;
                            if (!going) {
                                last = c;
                                over = true;
                            }
                        }
                    }
                }
            }
        }
    };
};

template <int L, int UMAX, bool DUAL, int BITS, bool ENDS>
__device__ __forceinline__ void search_unit_rows(const QuantArgs &a, double less /* tie_factor(dim) */, uint64_t n, uint32_t n_waves) {
    using Row = RowUnits<L, UMAX, DUAL>;
    constexpr int kRowsPerPass = kWave / Row::LANES;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    const uint32_t dim = a.dim, n4 = dim / 4;
    const uint64_t P = (uint64_t)dim * BITS / 8;
    const int lane = tid_x() & (kWave - 1);
    const uint32_t j = lane % L;
    for (uint64_t pass = wave_in_grid(); pass * kRowsPerPass < n; pass += n_waves) {
        const uint64_t k = pass * kRowsPerPass + lane / Row::LANES;
        uint64_t rid = 0;
        bool live = k < n;
        if (live) {
            rid = a.row_ids ? (uint64_t)a.row_ids[k] : k;
            if (rid >= a.n_rows) {
                if (lane % Row::LANES == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);
                live = false;
                rid = 0;
            }
        }
        Row row;
        row.load(reinterpret_cast<const float4 *>(a.table + rid * (uint64_t)dim), n4, j);
        float X_min, X_max;
        row.range(X_min, X_max);
        float lo = X_min, hi = X_max;
        if (search_divides(lo, hi, a.num_bins_f, QMAXF))
            row.template search<BITS, false, ENDS>(a.n_iter, a.num_bins_f, less, live, lo, hi);
        else
            row.template search<BITS, true, ENDS>(a.n_iter, a.num_bins_f, less, live, lo, hi);

        if constexpr (DUAL) live = live && !((lane / L) & 1);  // one of the row's two groups stores
        const float scale = (hi - lo) / QMAXF;
        {
            // lane j of the row writes parameter j, or with fewer than four lanes j, j + L, ...
#pragma unroll
            for (uint32_t p = j; p < 4; p += L) {
                float *dst = p == 0 ? a.scale : p == 1 ? a.bias : p == 2 ? a.row_min : a.row_max;
                const float v = p == 0 ? scale : p == 1 ? lo : p == 2 ? X_min : X_max;
                if (dst && live) dst[k] = v;
            }
        }
        // ---- final codes by F_Q as written, unit by unit; all lanes run it (3 bits: units u and u + 1, of
        // neighbouring lanes or, where a lane has the whole row, behind each other, make three bytes)
        uint32_t before = 0;
        auto emit = [&](const float4 &v, uint32_t u, bool mine) {
            const uint32_t q0 = (uint32_t)fq_code_f(v.x, lo, hi, scale, QMAXF);
            const uint32_t q1 = (uint32_t)fq_code_f(v.y, lo, hi, scale, QMAXF);
            const uint32_t q2 = (uint32_t)fq_code_f(v.z, lo, hi, scale, QMAXF);
            const uint32_t q3 = (uint32_t)fq_code_f(v.w, lo, hi, scale, QMAXF);
            const uint32_t h = q0 | (q1 << BITS) | (q2 << (2 * BITS)) | (q3 << (3 * BITS));
            const bool store = mine && live;
            if (a.codes && store)
                *reinterpret_cast<uint32_t *>(a.codes + k * (uint64_t)dim + 4 * u) = q0 | (q1 << 8) | (q2 << 16) | (q3 << 24);
            if (!a.packed) return;
            uint8_t *const out = a.packed + k * P;
            if constexpr (L == 1 && BITS == 3) {  // dim % 8 == 0: an even number of units
                if (store && (u & 1)) store_pair3(out, u >> 1, before | (h << 12));
                before = h;
            } else {
                store_unit_codes<BITS>(out, u, h, store);
            }
        };
        const uint32_t n_full = n4 / L;
#pragma unroll
        for (int t = 0; t < UMAX; ++t)
            if ((uint32_t)t < 2 * row.pairs) emit(row.x[t], j + L * t, true);
        if (row.has_odd) emit(row.odd, j + L * (n_full - 1), true);
        if (row.has_tail) emit(row.tail, j + L * n_full, row.in_tail);
    }
}

// Lists of n_from to n_below - 1 rows; the others are another launch's.
template <int L, int UMAX, bool DUAL, int BITS, bool ENDS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(UMAX > 8 ? 3 : 4, 8)))
quantize_greedy_units_kernel(const QuantArgs a, double less, uint64_t n_from, uint64_t n_below) {
    const uint64_t n = row_count(a);
    if (n >= n_from && n < n_below) search_unit_rows<L, UMAX, DUAL, BITS, ENDS>(a, less, n, a.n_waves);
}
// Both forms, as above (500 rows of 96 at 45 bins and 4 bits in a capacity of 133 K 11.9 -> 9.2 us, 25 K 27.6 -> 25.2, 106 K 58.8 -> 55.3).  Where the long form has
// sixteen units its registers leave three waves per SIMD, and the short form, throughput-bound just below the line, loses more than a launch with
// that (36 K rows of 144 48.7 against 52.9 us, 10 K of 640 71 and 77, 14 K of 1000 145 and 158; with the line anywhere from where it is to three quarters of
// that): there the two stay apart.
template <int L_NARROW, int U_NARROW, int L_WIDE, int U_WIDE, int BITS, bool ENDS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(U_WIDE > 8 ? 3 : 4, 8)))
quantize_greedy_units_pair_kernel(const QuantArgs a, double less, uint64_t line, uint32_t narrow_waves) {
    const uint64_t n = row_count(a);
    if (n >= line) search_unit_rows<L_WIDE, U_WIDE, false, BITS, ENDS>(a, less, n, a.n_waves);
    else if (wave_in_grid() < narrow_waves) search_unit_rows<L_NARROW, U_NARROW, true, BITS, ENDS>(a, less, n, narrow_waves);
}

// ---------------------------------------------------------------------------------------------
// Mean l2 error of a sample under several greedy parameters at once (parameter selection): the search of
// the kernel above, the restored row's error in place of its codes, nothing stored but one sum per
// workgroup and point.  Grid y = searches, side by side: a sample of a few thousand rows
// leaves the chip mostly idle, and the launch takes as long as its longest search.  What a search of fewer iterations ends with
// is what a longer one has found by then, so one search serves every point that differs in its ratio alone: it stops at
// each of them and works out the errors, unless no row of the wave has found a better range since the last one.
// One sum per workgroup, not per wave: with four times the sums the caller's scratch is full four times as early, and fewer waves then take a sample
// in several passes (31 values of num_bins at 2 bits, 256 rows of 40: 65 us against 95, 2.5 K rows of 64: 134 and 152; where either fits, level).
// One launch per set of parameters with the codes stored, read back and compared (encode, error, mean and a synchronization
// each) took 354 us for 2.5 K rows of 64 and eight points; all values of num_bins in one launch and all ratios in another,
// a search each, 64 us, this 43.
// ---------------------------------------------------------------------------------------------
struct SelectArgs {
    const float *table;
    uint64_t n_rows;
    uint32_t dim;
    const uint32_t *row_ids;
    uint64_t n;
    double less;   // tie_factor(dim)
    double *sums;  // [points][workgroups along x]
    uint32_t grid;  // workgroups along x
    cnr_dev_errors *err;
    cnr_search_params points[kSearchBatch];
    uint8_t first[kSearchBatch + 1];  // search y has the points first[y] .. first[y + 1) - 1, in ascending order of iterations
};
template <int L, int UMAX, bool DUAL, int BITS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(UMAX > 8 ? 3 : 4, 8)))
sample_error_kernel(const SelectArgs a) {
    using Row = RowUnits<L, UMAX, DUAL>;
    constexpr int kRowsPerPass = kWave / Row::LANES;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    const uint32_t p0 = a.first[wg_y()], p1 = a.first[wg_y() + 1];
    const float num_bins_f = a.points[p0].num_bins_f;
    const uint32_t n4 = a.dim / 4;
    const int lane = tid_x() & (kWave - 1);
    const uint32_t j = lane % L;
    const uint32_t n_waves = a.grid * kWavesPerBlock;
    __shared__ double wave_sums[kWavesPerBlock][kSearchBatch];
    double *const sums = wave_sums[tid_x() / kWave];
    bool add_up = false;  // not the first pass
    if ((uint64_t)wave_in_grid() * kRowsPerPass >= a.n && lane < (int)kSearchBatch) sums[lane] = 0.0;  // a wave beyond the last row
    for (uint64_t pass = wave_in_grid(); pass * kRowsPerPass < a.n; pass += n_waves) {
        const uint64_t k = pass * kRowsPerPass + lane / Row::LANES;
        uint64_t rid = 0;
        bool live = k < a.n;
        if (live) {
            rid = a.row_ids ? (uint64_t)a.row_ids[k] : k;
            if (rid >= a.n_rows) {
                if (lane % Row::LANES == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);
                live = false;
                rid = 0;
            }
        }
        Row row;
        row.load(reinterpret_cast<const float4 *>(a.table + rid * (uint64_t)a.dim), n4, j);
        float lo, hi;
        row.range(lo, hi);
        auto points = [&](auto fast_tag) {
            typename Row::template Search<BITS, decltype(fast_tag)::value, true> search(row, num_bins_f, a.less, live, lo, hi);
            double sum = 0.0;
            for (uint32_t p = p0; p < p1; ++p) {
                const float lo_before = lo, hi_before = hi;
                const uint32_t n_iter = a.points[p].n_iter;
                if (n_iter && !search.over) search.run(n_iter, lo, hi);
                if (p == p0 || __builtin_amdgcn_ballot_w64(lo != lo_before || hi != hi_before) != 0) {
                    const float scale = (hi - lo) / QMAXF;
                    double e = 0.0;
                    auto add = [&](const float4 &v) {
                        const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const double d = (double)x[i] - (double)fq_value(fq_code_f(x[i], lo, hi, scale, QMAXF), scale, lo);
                            e = fma(d, d, e);
                        }
                    };
#pragma unroll
                    for (int t = 0; t < UMAX; ++t)
                        if ((uint32_t)t < 2 * row.pairs) add(row.x[t]);
                    if (row.has_odd) add(row.odd);
                    if (row.has_tail && row.in_tail) add(row.tail);
                    e = lanes_sum<L>(e);
                    sum = live && lane % Row::LANES == 0 ? sqrt(e) : 0.0;
                    for (int off = 32; off >= Row::LANES; off >>= 1) sum += __shfl_xor(sum, off);
                }
                if (lane == 0) sums[p] = add_up ? sums[p] + sum : sum;
            }
        };
        if (search_divides(lo, hi, num_bins_f, QMAXF)) points(std::false_type{});
        else points(std::true_type{});
        add_up = true;
    }
    __syncthreads();
    const uint32_t p = p0 + tid_x();
    if (p < p1) a.sums[(uint64_t)p * a.grid + wg_x()] = (wave_sums[0][p] + wave_sums[1][p]) + (wave_sums[2][p] + wave_sums[3][p]);
}
static_assert(kWavesPerBlock == 4 && kSearchBatch <= kWave && kSearchBatch <= kBlock, "");
// mean_out[p] = (the sums of point p, added up in a fixed order) / n; one workgroup per p.
__global__ void __launch_bounds__(kBlock) sample_mean_kernel(const double *sums, uint32_t per_set, double n, double *mean_out) {
    __shared__ double part[kBlock];
    double acc = 0.0;
    for (uint32_t i = tid_x(); i < per_set; i += kBlock) acc += sums[(uint64_t)wg_x() * per_set + i];
    part[tid_x()] = acc;
    __syncthreads();
    for (int half = kBlock / 2; half > 0; half >>= 1) {
        if ((int)tid_x() < half) part[tid_x()] += part[tid_x() + half];
        __syncthreads();
    }
    if (tid_x() == 0) mean_out[wg_x()] = part[0] / n;
}

// ---------------------------------------------------------------------------------------------
// Other row lengths, min/max and symmetric range.  Same arithmetic as the tile kernel; bound by the
// memory traffic, on short lists by the chain of one row's loads and the fetch of the kernel's own code.
//
// Up to 512 elements (quantize_units_kernel): LPR lanes per row, U 16-byte units of it per lane (unit j +
// LPR * t, so that a load instruction reads 16 * LPR contiguous bytes per row), read once and held in
// registers: SB steps of 64 / LPR rows are on their way at a time, and the other waves of the compute unit
// hide their latency.  The row's range takes log2(LPR) cross-lane steps.  A unit's 4 * BITS code bits are
// too few to store one by one, so a wave collects the codes of ROWS rows (a multiple of sixteen, hence
// whole 16-byte pieces at any row length and width), which are one contiguous run of the output, in its
// own piece of LDS and writes them out 16 bytes per lane.  750 K rows of 96, 4 bits: read twice and
// stored by twos of bytes 130 us, this 66 us (5.1 TB/s); rows
// of 8 to 512 elements 1.3 to 2.5 times as fast.
//
// Longer rows, and short lists: one row (or 64 / LPR short ones) per wave and pass (encode_strided).  It fills
// the chip sooner and is less code, but it reads a row twice and its last trip through a row stores as little as
// one unit, 1 to 4 bytes.  On lists of up to 6144 waves of it (SHORT_ROWS: 98 K rows of 4 to 16 elements, 6 K of more than 128) the units
// kernel goes that way itself, whether the host knows the length or not: 1 K rows of 24 / 96 / 200
// elements 3.4 / 3.2 / 4.3 us in units, 2.7 / 2.8 / 3.0 this way; 16 K rows of 96 3.8 and 4.5.
// ---------------------------------------------------------------------------------------------
// Code of one element, biased by the pattern of 1.5 * 2^23 (see the tile kernel).
template <int BITS>
__device__ __forceinline__ uint32_t biased_code(float x, float lo, float f, float fscale, float inv) {
    const float d0 = (x - lo) * f;
    float t = d0 * inv;
    if constexpr (BITS == 8) t = fmaf(fmaf(-t, fscale, d0), inv, t);
    return __float_as_uint(t + 12582912.0f);
}
// The 4 * BITS code bits of a unit, and its codes one per byte.
template <int BITS>
__device__ __forceinline__ uint32_t unit_codes(const f32x4 &v, float lo, float f, float fscale, float inv, uint32_t &bytes) {
    constexpr uint32_t MAGIC_BITS = 0x4B400000u;
    constexpr uint32_t MERGED_BIAS = MAGIC_BITS * (1u + (1u << BITS) + (1u << (2 * BITS)) + (1u << (3 * BITS)));
    constexpr uint32_t MERGED_BIAS8 = MAGIC_BITS * (1u + (1u << 8) + (1u << 16) + (1u << 24));
    const uint32_t b0 = biased_code<BITS>(v.x, lo, f, fscale, inv), b1 = biased_code<BITS>(v.y, lo, f, fscale, inv);
    const uint32_t b2 = biased_code<BITS>(v.z, lo, f, fscale, inv), b3 = biased_code<BITS>(v.w, lo, f, fscale, inv);
    bytes = (((((b3 << 8) + b2) << 8) + b1) << 8) + b0 - MERGED_BIAS8;
    uint32_t m = (b3 << BITS) + b2;
    m = (m << BITS) + b1;
    return (m << BITS) + b0 - MERGED_BIAS;
}

// LPR lanes per row, 64 / LPR rows per wave and pass; the row is read twice, for its range and to quantize, the
// second time from cache, and its codes go straight to memory.
template <int LPR, int BITS>
__device__ __forceinline__ void encode_strided(const QuantArgs &a, uint64_t n) {
    constexpr int kRowsPerPass = kWave / LPR;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    const uint32_t dim = a.dim, n4 = dim / 4;      // 16-byte units per row
    const uint64_t P = (uint64_t)dim * BITS / 8;   // packed bytes per row
    const int lane = tid_x() & (kWave - 1);
    const uint32_t j = lane % LPR;
    const uint32_t last_row = (uint32_t)a.n_rows - 1u;
    const uint32_t n_waves = a.n_waves;
    for (uint64_t pass = wave_in_grid(); pass * kRowsPerPass < n; pass += n_waves) {
        const uint64_t k = pass * kRowsPerPass + lane / LPR;
        const uint64_t kc = k < n ? k : n - 1;     // rows past the end repeat the last one; nothing of theirs is stored
        const uint32_t rid = a.row_ids ? a.row_ids[kc] : kc > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)kc;
        const bool in_table = rid <= last_row;
        const bool live = k < n && in_table;
        if (k < n && !in_table && j == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);
        const f32x4 *row = reinterpret_cast<const f32x4 *>(a.table + (uint64_t)(in_table ? rid : last_row) * dim);

        // ---- row minimum / maximum (every lane starts from the row's first unit, so idle lanes are neutral)
        const f32x4 first = row[0];
        float mn = fminf(fminf(first.x, first.y), fminf(first.z, first.w));
        float mx = fmaxf(fmaxf(first.x, first.y), fmaxf(first.z, first.w));
        for (uint32_t u = j; u < n4; u += LPR) {
            const f32x4 v = row[u];
            mn = fminf(fminf(mn, v.x), fminf(v.y, fminf(v.z, v.w)));
            mx = fmaxf(fmaxf(mx, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
        }
        const float X_min = lanes_min<LPR>(mn) + 0.0f;  // -0.0 -> +0.0
        const float X_max = lanes_max<LPR>(mx) + 0.0f;
        float lo = X_min, hi = X_max;
        if (a.mode == kModeSymmetric) {
            const float m = fmaxf(fabsf(X_min), fabsf(X_max));
            lo = -m + 0.0f;
            hi = m;
        }
        const float scale = (hi - lo) / QMAXF;
        {
            float *dst = j == 0 ? a.scale : j == 1 ? a.bias : j == 2 ? a.row_min : a.row_max;
            const float v = j == 0 ? scale : j == 1 ? lo : j == 2 ? X_min : X_max;
            if (j < 4 && dst && live) dst[k] = v;
        }
        const float f = scale < 0x1p-100f ? 0x1p120f : scale > 0x1p100f ? 0x1p-120f : 1.0f;
        const float fscale = scale * f;
        const float inv = scale == 0.0f ? 0.0f : 1.0f / fscale;  // scale 0: every code 0

        // ---- quantize unit by unit; all lanes take every trip so that the 3-bit exchange has partners
        const uint32_t trips = (n4 + LPR - 1) / LPR;
        for (uint32_t trip = 0; trip < trips; ++trip) {
            const uint32_t u = j + trip * LPR;
            const bool mine = u < n4;
            uint32_t bytes;
            const uint32_t h = unit_codes<BITS>(row[mine ? u : 0], lo, f, fscale, inv, bytes);
            const bool store = mine && live;
            if (a.codes && store) *reinterpret_cast<uint32_t *>(a.codes + k * (uint64_t)dim + 4 * u) = bytes;
            if (a.packed) store_unit_codes<BITS>(a.packed + k * P, u, h, store);
        }
    }
}
// Tables of a batch in one launch, as for the tile kernel: small tables are bound by their launches (the encode of eight
// tables of 29 K rows of 8 34.5 us one table per launch, 14.6 all in one; 16 x 20 K rows of 96 66 -> 28; 2 x 2 M 137 -> 133).
// Both the launch of one table (N = 1) and that of several exist: sixteen tables' arguments are 2 KB for each launch to
// bring along (0.2 to 0.6 us of 6), and a job is copied out of them, since one that stays behind a reference is
// loaded again inside the loops (1.5 M rows of 24 50 -> 56 us).
template <int N>
__device__ __forceinline__ QuantArgs job_of(const QuantBatchArgs<N> &b) {
    if constexpr (N == 1) return b.job[0];
    else return b.job[wg_y()];
}
template <int BITS, int N>
__global__ void __launch_bounds__(kBlock) quantize_strided_kernel(const QuantBatchArgs<N> b) {
    const QuantArgs a = job_of(b);
    if (N > 1 && wg_x() * kWavesPerBlock >= a.n_waves) return;  // fewer workgroups than the launch's largest table
    encode_strided<kWave, BITS>(a, row_count(a));
}

constexpr uint64_t kShortEncodeWaves = 6144;
template <int LPR, int U, int SB, int BITS>
struct UnitsShape {
    static constexpr int RPS = kWave / LPR;                                  // rows per step
    static constexpr int STEPS = LPR == 4 ? SB : LPR == 8 ? (SB > 2 ? SB : 2) : 4;
    static constexpr int ROWS = RPS * STEPS;                                 // rows per wave and pass
    static_assert(ROWS % 16 == 0 && STEPS % SB == 0, "whole 16-byte pieces");
    static constexpr int STAGE = ROWS * LPR * U * BITS / 2;                  // LDS per wave
    static constexpr int SHORT_LPR = LPR * U <= 4 ? 4 : LPR * U <= 8 ? 8 : LPR * U <= 16 ? 16 : LPR * U <= 32 ? 32 : 64;
    static constexpr uint64_t SHORT_ROWS = kShortEncodeWaves * (kWave / SHORT_LPR);
};
template <int LPR, int U, int SB, int BITS, int N>
__global__ void __launch_bounds__(kBlock) quantize_units_kernel(const QuantBatchArgs<N> b) {
    using S = UnitsShape<LPR, U, SB, BITS>;
    const QuantArgs a = job_of(b);
    if (N > 1 && wg_x() * kWavesPerBlock >= a.n_waves) return;
    constexpr int RPS = S::RPS, ROWS = S::ROWS;
    constexpr float QMAXF = (float)((1 << BITS) - 1);
    __shared__ __align__(16) uint8_t stages[kWavesPerBlock * S::STAGE];
    uint8_t *const stage = stages + (tid_x() / kWave) * S::STAGE;
    const uint64_t n = row_count(a);
    if (n <= S::SHORT_ROWS) return encode_strided<S::SHORT_LPR, BITS>(a, n);
    const uint32_t dim = a.dim, n4 = dim / 4;      // 16-byte units per row, at most LPR * U
    const uint32_t P = dim * BITS / 8;             // packed bytes per row
    const int lane = tid_x() & (kWave - 1);
    const uint32_t j = lane % LPR, rho = lane / LPR;
    const uint32_t last_row = (uint32_t)a.n_rows - 1u;
    const uint32_t n_waves = a.n_waves;
    for (uint64_t pass = wave_in_grid(); pass * ROWS < n; pass += n_waves) {
        const uint64_t base = pass * ROWS;
        const uint32_t left = n - base < (uint64_t)ROWS ? (uint32_t)(n - base) : (uint32_t)ROWS;  // uniform
        bool all_in_table = true;
#pragma unroll
        for (int s0 = 0; s0 < S::STEPS; s0 += SB) {
            uint32_t rid[SB];
            f32x4 x[SB][U];
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                const uint32_t r = (s0 + s) * RPS + rho;
                const uint64_t k = base + (r < left ? r : left - 1);  // rows past the end repeat the last one; nothing of theirs is stored
                rid[s] = a.row_ids ? a.row_ids[k] : k > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)k;
            }
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                const float *row = a.table + (uint64_t)(rid[s] < last_row ? rid[s] : last_row) * dim;
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t u = j + LPR * t;
                    x[s][t] = load_stream<f32x4>(row + 4 * (u < n4 ? u : n4 - 1));  // past the row's end: its last unit again
                }
            }
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                const uint32_t r = (s0 + s) * RPS + rho;
                const uint64_t k = base + r;
                const bool in_table = rid[s] <= last_row, live = r < left && in_table;
                if (r < left && !in_table) {
                    all_in_table = false;
                    if (j == 0) raise_flag(a.err, CNR_FLAG_ROW_ID);
                }
                // ---- row minimum / maximum, parameters
                float mn = x[s][0].x, mx = x[s][0].x;
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const f32x4 v = x[s][t];
                    mn = fminf(fminf(mn, v.x), fminf(v.y, fminf(v.z, v.w)));
                    mx = fmaxf(fmaxf(mx, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
                }
                const float X_min = lanes_min<LPR>(mn) + 0.0f;  // -0.0 -> +0.0
                const float X_max = lanes_max<LPR>(mx) + 0.0f;
                float lo = X_min, hi = X_max;
                if (a.mode == kModeSymmetric) {
                    const float m = fmaxf(fabsf(X_min), fabsf(X_max));
                    lo = -m + 0.0f;
                    hi = m;
                }
                const float scale = (hi - lo) / QMAXF;
                {
                    float *dst = j == 0 ? a.scale : j == 1 ? a.bias : j == 2 ? a.row_min : a.row_max;
                    const float v = j == 0 ? scale : j == 1 ? lo : j == 2 ? X_min : X_max;
                    if (j < 4 && dst && live) store_stream<float>(dst + k, v);
                }
                const float f = scale < 0x1p-100f ? 0x1p120f : scale > 0x1p100f ? 0x1p-120f : 1.0f;
                const float fscale = scale * f;
                const float inv = scale == 0.0f ? 0.0f : 1.0f / fscale;  // scale 0: every code 0
                // ---- codes, into the wave's stage
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t u = j + LPR * t;
                    uint32_t bytes;
                    const uint32_t h = unit_codes<BITS>(x[s][t], lo, f, fscale, inv, bytes);
                    if (a.codes && u < n4 && live) *reinterpret_cast<uint32_t *>(a.codes + k * (uint64_t)dim + 4 * u) = bytes;
                    if (a.packed) store_unit_codes<BITS>(stage + r * P, u, h, u < n4);
                }
            }
        }
        if (!a.packed) continue;
        // ---- the packed rows of the pass: one run of left * P bytes
        __builtin_amdgcn_wave_barrier();  // LDS operations of one wave complete in order
        uint8_t *const out = a.packed + base * P;
        const uint32_t bytes = left * P;
        if (__builtin_amdgcn_ballot_w64(!all_in_table) == 0) {
            for (uint32_t off = 16u * lane; off + 16u <= bytes; off += 16u * kWave)
                store_stream<u32x4>(out + off, *reinterpret_cast<const u32x4 *>(stage + off));
            const uint32_t rest = bytes & 15u;
            if ((uint32_t)lane < rest) out[bytes - rest + lane] = stage[bytes - rest + lane];
        } else {  // rows outside the table leave their place in the output as it is
            for (uint32_t r = 0; r < left; ++r) {
                const uint64_t k = base + r;
                const uint64_t id = a.row_ids ? (uint64_t)a.row_ids[k] : k;
                if (id >= a.n_rows) continue;
                for (uint32_t b = lane; b < P; b += kWave) out[r * P + b] = stage[r * P + b];
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------------------------
// Stand-alone dense packing of one-code-per-byte input: one output byte per thread-visit.
// ---------------------------------------------------------------------------------------------
template <int BITS>
__global__ void __launch_bounds__(kBlock)
pack_kernel(const uint8_t *__restrict__ codes, const uint64_t *__restrict__ n_dev, uint64_t n_max,
            uint32_t dim, uint8_t *__restrict__ packed, uint64_t stride) {
    uint64_t n = n_max;
    if (n_dev) {
        const uint64_t nd = *n_dev;
        n = nd < n_max ? nd : n_max;
    }
    const uint64_t P = (uint64_t)dim * BITS / 8;
    const uint64_t total = n * P;
    for (uint64_t o = (uint64_t)wg_x() * kBlock + tid_x(); o < total; o += stride) {
        const uint64_t k = o / P, b = o - k * P;
        const uint8_t *row = codes + k * (uint64_t)dim;
        const uint32_t first = (uint32_t)((8 * b) / BITS);
        const uint32_t last = (uint32_t)((8 * b + 7) / BITS);
        uint32_t byte = 0;
        for (uint32_t e = first; e <= last; ++e) {
            const uint32_t code = row[e] & ((1u << BITS) - 1u);
            const int shift = (int)(e * BITS) - (int)(8 * b);
            byte |= shift >= 0 ? (code << shift) : (code >> -shift);
        }
        packed[o] = (uint8_t)byte;
    }
}

// n tables (or slices) in one launch: every one with the grid its own list calls for (cnr_row_grid).
template <int Q, int BITS>
void launch_tile(QuantBatchArgs<> &b, uint32_t n, hipStream_t s) {
    unsigned grid = 1;
    for (uint32_t i = 0; i < n; ++i) {
        const unsigned g = cnr_row_grid(b.job[i].n_max, (uint64_t)TileShape<Q>::ROWS * kWavesPerBlock);
        b.job[i].n_waves = g * kWavesPerBlock;
        if (g > grid) grid = g;
    }
    hipLaunchKernelGGL((quantize_tile_kernel<Q, BITS>), dim3(grid, n), dim3(kBlock), 0, s, b);
}
template <int BITS>
void launch_tile_bits(QuantBatchArgs<> &b, uint32_t n, uint32_t dim, hipStream_t s) {
    switch (dim) {
        case 16: return launch_tile<1, BITS>(b, n, s);
        case 32: return launch_tile<2, BITS>(b, n, s);
        case 64: return launch_tile<4, BITS>(b, n, s);
        case 128: return launch_tile<8, BITS>(b, n, s);
        default: return launch_tile<16, BITS>(b, n, s);
    }
}
inline void launch_tile_any(QuantBatchArgs<> &b, uint32_t n, uint32_t dim, int bits, hipStream_t s) {
    switch (bits) {
        case 2: return launch_tile_bits<2>(b, n, dim, s);
        case 3: return launch_tile_bits<3>(b, n, dim, s);
        case 4: return launch_tile_bits<4>(b, n, dim, s);
        default: return launch_tile_bits<8>(b, n, dim, s);
    }
}

// Whether a search can end before its last iteration: one that covers only the first part of its num_bins moves (a ratio well
// below 1) is over before any but clustered rows could be finished, and would keep the ends and ask for nothing.  Evenly spread
// rows, which finish first, do so after 0.48 to 0.52 of the moves at 2 bits, 0.28 to 0.32 at 3, 0.17 to 0.2 at 4, at 8 bits after one or two
// moves; normal ones after 0.6, 0.35 and 0.2 of them and later.  (Rows of up to 32 elements sooner: they always ask.)  With the questions and
// without: 20 K rows of 40 elements, 3 bits, ratio 0.3 20.7 and 18.0 us, of 1024 136 and 129; 1 K of 320 at 2 bits, ratio 0.5, 11.4 and 10.8;
// 78 K of 256 at 4 bits, ratio 0.17, 74.3 and 70.4.
template <int BITS>
constexpr float kEarliestEnd = BITS == 2 ? 0.52f : BITS == 3 ? 0.32f : BITS == 4 ? 0.18f : 0.0f;
template <int BITS>
bool may_end_early(const QuantArgs &a) { return a.dim <= 32 || (float)a.n_iter > kEarliestEnd<BITS> * a.num_bins_f; }

template <int L, int BITS, int G>
void launch_greedy(QuantArgs &a, hipStream_t s) {
    // the large grid here too: the search is bound by arithmetic, but workgroups handed out as others
    // finish even out the end of the launch (4 % on a 1.5 M-row list)
    const unsigned grid = cnr_row_grid(a.n_max, (uint64_t)(kWave / L) * kWavesPerBlock);
    a.n_waves = grid * kWavesPerBlock;
    if constexpr (BITS != 8 && 16 * G * L > 32) {
        if (!may_end_early<BITS>(a)) {
            hipLaunchKernelGGL((quantize_greedy_kernel<L, BITS, G, false>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim));
            return;
        }
    }
    hipLaunchKernelGGL((quantize_greedy_kernel<L, BITS, G, true>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim));
}
template <int L_NARROW, int L_WIDE, int G_WIDE, int BITS>
void launch_greedy_pair(QuantArgs &a, hipStream_t s, uint64_t line) {
    const unsigned wide = cnr_row_grid(a.n_max, (uint64_t)(kWave / L_WIDE) * kWavesPerBlock);
    const unsigned narrow = cnr_row_grid(line, (uint64_t)(kWave / L_NARROW) * kWavesPerBlock);
    const unsigned grid = wide > narrow ? wide : narrow;
    a.n_waves = grid * kWavesPerBlock;
    if constexpr (BITS != 8 && 16 * L_NARROW > 32) {
        if (!may_end_early<BITS>(a)) {
            hipLaunchKernelGGL((quantize_greedy_pair_kernel<L_NARROW, L_WIDE, G_WIDE, BITS, false>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), line, narrow * kWavesPerBlock);
            return;
        }
    }
    hipLaunchKernelGGL((quantize_greedy_pair_kernel<L_NARROW, L_WIDE, G_WIDE, BITS, true>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), line, narrow * kWavesPerBlock);
}
// Long lists give every lane 64 elements (32 at dim 32); short ones keep 16 per lane, four times the
// lanes per row and a quarter of the time per row, which is what counts while the list cannot fill
// the SIMDs anyway.  The break-even lies at 8 M elements at 2 to 4 bits, whether searches end early or not (rows of 64, 45 bins, 4 bits:
// 93 K rows 32.1 us with 16 elements per lane, 40.6 with 64, 131 K 41.6 and 41.1, 262 K 77.0 and 72.0; 3 bits 52.3 and 66.9, 68.4 and
// 68.5, 129 and 119; rows of 256 at 16 K, 33 K and 66 K 38.7 and 44.2, 71.0 and 66.5, 134 and 118; rows of 32 level from 4 M on).
// At 8 bits it depends on the number of bins (100 bins: rows of 64 16.2 and 18.4 at 8 M, 26.9 and 29.9 at 16 M, level at 32 M;
// rows of 256 22.3 and 21.3, 39.7 and 36.0; 20 bins: 15.0 and 16.0, level from 16 M on).  Where the
// length is a count on the device and the capacity allows a long list, the kernel has both forms.
template <int L_NARROW, int L_WIDE, int G_WIDE, int BITS>
void launch_greedy_by_length(QuantArgs &a, hipStream_t s) {
    const uint64_t wide_rows = (1ull << 23) / a.dim;
    if (a.n_max < wide_rows) launch_greedy<L_NARROW, BITS, 1>(a, s);
    else if (a.n_dev) launch_greedy_pair<L_NARROW, L_WIDE, G_WIDE, BITS>(a, s, wide_rows);
    else launch_greedy<L_WIDE, BITS, G_WIDE>(a, s);
}

template <int L, int UMAX, bool DUAL, int BITS>
void launch_greedy_units_shape(QuantArgs &a, hipStream_t s, uint64_t n_from, uint64_t n_below) {
    const uint64_t most = a.n_max < n_below ? a.n_max : n_below;
    const unsigned grid = cnr_row_grid(most, (uint64_t)(kWave / RowUnits<L, UMAX, DUAL>::LANES) * kWavesPerBlock);
    a.n_waves = grid * kWavesPerBlock;
    if constexpr (BITS != 8 && L > 1 && UMAX > 2) {  // the others have rows of up to 32 elements
        if (!may_end_early<BITS>(a)) {
            hipLaunchKernelGGL((quantize_greedy_units_kernel<L, UMAX, DUAL, BITS, false>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), n_from, n_below);
            return;
        }
    }
    hipLaunchKernelGGL((quantize_greedy_units_kernel<L, UMAX, DUAL, BITS, true>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), n_from, n_below);
}
template <int L_NARROW, int U_NARROW, int L_WIDE, int U_WIDE, int BITS>
void launch_greedy_units_pair(QuantArgs &a, hipStream_t s, uint64_t line) {
    const unsigned wide = cnr_row_grid(a.n_max, (uint64_t)(kWave / RowUnits<L_WIDE, U_WIDE, false>::LANES) * kWavesPerBlock);
    const unsigned narrow = cnr_row_grid(line, (uint64_t)(kWave / RowUnits<L_NARROW, U_NARROW, true>::LANES) * kWavesPerBlock);
    const unsigned grid = wide > narrow ? wide : narrow;
    a.n_waves = grid * kWavesPerBlock;
    if constexpr (BITS != 8 && U_NARROW > 2) {
        if (!may_end_early<BITS>(a)) {
            hipLaunchKernelGGL((quantize_greedy_units_pair_kernel<L_NARROW, U_NARROW, L_WIDE, U_WIDE, BITS, false>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), line, narrow * kWavesPerBlock);
            return;
        }
    }
    hipLaunchKernelGGL((quantize_greedy_units_pair_kernel<L_NARROW, U_NARROW, L_WIDE, U_WIDE, BITS, true>), dim3(grid), dim3(kBlock), 0, s, a, tie_factor(a.dim), line, narrow * kWavesPerBlock);
}
// Other row lengths: long lists give a row as few lanes as hold it; short ones give it two groups of 4 to
// 32 lanes, which evaluate the two candidates of an iteration side by side (17 instead of 23 us for
// the shortest lists of rows of 96 at 25 bins, a single group of 16 lanes taking one after the other).
// The line lies where the long form's waves fill the chip: 768 waves of short rows, or, since a lane with
// many units works longer on its row, a number in proportion to them (up to 26.6 K rows where four lanes hold
// up to eight units each).  Measured break-evens, 25 and 45 bins: rows of 24 at 45 K rows, of 48 at 25 K, of 60
// at 40 K, of 72 at 22 K, of 96 to 140 at 26-28 K, of 144 to 268 within 8 % of each other from 30 K to 90 K, of
// 288 and 320 at 7 K, of 384 at 8-10 K, of 640 at 15 K, of 1000 at 19 K.  Rows of 272 to 284 keep two groups of eight
// at any length: sixteen lanes would hold four units and a nearly empty fifth (20-30 % slower from 6 K to 31 K rows).
// At 8 bits a search ends after an iteration or two, so two groups save little and the line lies lower (rows of 24 at 22 K
// rows, of 48 at 12 K, of 96 at 9 K, of 200 at 21 K, of 640 at 5 K; 20 K rows of 96 9.3 us in two groups, 7.9 in one), and so it does
// for rows of 4 to 16 elements, whose long form is four elements' chain and no exchange between lanes (rows of 8 at 20-30 K;
// 40 K of them 8.5 and 6.5).
template <int BITS>
void launch_greedy_units(QuantArgs &a, hipStream_t s) {
    const uint32_t n4 = a.dim / 4;
    const uint32_t lanes = n4 <= 8 ? 1 : n4 <= 17 ? 2 : n4 < 68 ? 4 : n4 <= 271 ? 16 : 64;
    const uint64_t fill = 49152u / lanes, busy = (lanes >= 4 ? 20480ull : 8192ull) * n4 / (lanes * lanes);
    uint64_t wide_rows = fill > busy ? fill : busy;
    if (lanes == 4 && n4 < 36 && wide_rows > 26624) wide_rows = 26624;
    if (n4 <= 4) wide_rows /= 2;
    if (BITS == 8) wide_rows = wide_rows * 2 / 5;
    if (n4 >= 68 && n4 < 72) wide_rows = ~0ull;
    const bool may_be_wide = lanes == 64 || a.n_max >= wide_rows;
    const bool may_be_narrow = lanes != 64 && (!may_be_wide || a.n_dev != nullptr);
    if (may_be_wide && may_be_narrow && n4 < 36) {
        if (lanes == 1) launch_greedy_units_pair<4, 2, 1, 8, BITS>(a, s, wide_rows);
        else if (lanes == 2) launch_greedy_units_pair<8, 8, 2, 8, BITS>(a, s, wide_rows);
        else launch_greedy_units_pair<8, 8, 4, 8, BITS>(a, s, wide_rows);
        return;
    }
    const uint64_t below = may_be_wide ? wide_rows : ~0ull, from = may_be_narrow ? wide_rows : 0;
    if (may_be_narrow) {
        if (n4 <= 8) launch_greedy_units_shape<4, 2, true, BITS>(a, s, 0, below);
        else if (n4 < 72) launch_greedy_units_shape<8, 8, true, BITS>(a, s, 0, below);
        else launch_greedy_units_shape<32, 8, true, BITS>(a, s, 0, below);
    }
    if (may_be_wide) {
        if (lanes == 1) launch_greedy_units_shape<1, 8, false, BITS>(a, s, from, ~0ull);
        else if (lanes == 2) launch_greedy_units_shape<2, 8, false, BITS>(a, s, from, ~0ull);
        else if (n4 < 36) launch_greedy_units_shape<4, 8, false, BITS>(a, s, from, ~0ull);
        else if (lanes == 4) launch_greedy_units_shape<4, 16, false, BITS>(a, s, from, ~0ull);
        else if (lanes == 16) launch_greedy_units_shape<16, 16, false, BITS>(a, s, from, ~0ull);
        else launch_greedy_units_shape<64, 16, false, BITS>(a, s, from, ~0ull);
    }
}

// Lists so short that two groups of lanes per row, one candidate each, still leave room on the chip (three
// waves per SIMD), at the lengths that the kernels above otherwise search with one: 45 bins, 1 K rows of
// 16 to 128 elements 28-30 -> 12-25 us, of 256 30 -> 24; at the line both take the same.  A search of few
// iterations gains less than the wider spread of its rows costs, so the line comes down with it (up to 10 bins,
// 12 K rows of 64 8.8 us in one group, 9.6 in two, 6 K rows 8.8 and 7.9; up to 4 bins, 3 K rows of 128 5.4 and 5.9).
// At 8 bits a search ends after an iteration or two and one group is level or better for rows of 64 and more (12 K of them 4.8
// against 5.8 us) and beyond 6 K shorter rows (4.6 against 4.1-4.3 below, 4.6 and 4.5-4.9 at 12 K).  At 3 and 4 bits rows of 64 whose
// search may end early have the line at two waves per SIMD: they hold half of what rows of 128 do in the same form, and one that ends is
// over sooner (4 bits, 100 bins: 8 K rows 14.5 us in two groups, 17.4 in one, 9 K 17.6 and 17.3; 45 bins 9.7 and 10.0, 11.6 and 10.0; 3 bits,
// 45 bins 13.3 and 15.5, 16.0 and 15.4).  Partial searches keep three (100 bins, ratio 0.3, 8 K rows 16.7 and 20.8, 12 K 20.5 and 20.8), and
// so do the other lengths, searched whole or not (12 K rows of 128 at 4 bits, 100 bins, 29.4 and 32.7, 20 K of 16 8.4 and 10.6).
// Only where the host's bound on the length says so: another launch to choose from on the device would cost
// the longer lists more.
template <int BITS>
bool launch_greedy_short(QuantArgs &a, hipStream_t s) {
    const uint32_t lanes = a.dim <= 32 ? 8 : a.dim <= 128 ? 16 : 32;
    uint32_t many = 196608u / lanes >> (BITS == 8 ? 2 : 0);
    if (a.dim == 64 && BITS != 2 && a.n_iter >= 16 && may_end_early<BITS>(a)) many = many * 2 / 3;
    const uint32_t most = a.n_iter >= 16 ? many : a.dim <= 64 ? (a.n_iter >= 3 ? many / 2 : many / 4) : a.n_iter >= 8 ? many / 4 : 0;
    if (a.n_max > most || (BITS == 8 && a.dim > 32)) return false;
    if (a.dim == 16 || a.dim == 32) {
        launch_greedy_units_shape<4, 2, true, BITS>(a, s, 0, ~0ull);
        return true;
    }
    if constexpr (BITS != 8) {
        switch (a.dim) {
            case 64:
            case 128: launch_greedy_units_shape<8, 8, true, BITS>(a, s, 0, ~0ull); return true;
            case 256: launch_greedy_units_shape<16, 4, true, BITS>(a, s, 0, ~0ull); return true;
        }
    }
    return false;
}

// n tables in one launch: every one with the grid its own list calls for.
template <int LPR, int U, int SB, int BITS>
void launch_units(QuantBatchArgs<> &b, uint32_t n, hipStream_t s) {
    using S = UnitsShape<LPR, U, SB, BITS>;
    unsigned most = 1;
    for (uint32_t i = 0; i < n; ++i) {
        QuantArgs &a = b.job[i];
        const unsigned grid_long = cnr_row_grid(a.n_max, (uint64_t)S::ROWS * kWavesPerBlock);
        const unsigned grid_short = cnr_row_grid(a.n_max < S::SHORT_ROWS ? a.n_max : S::SHORT_ROWS, (uint64_t)(kWave / S::SHORT_LPR) * kWavesPerBlock);
        unsigned grid = grid_long > grid_short ? grid_long : grid_short;
        // Where only the device knows the length it may be far below the capacity, and then the workgroups beyond the
        // count are most of the time: half the usual cap (1 K rows of 96 in a capacity of 5 M 7.1 -> 4.5 us, 250 K rows
        // 25.9 -> 24.6, 1.5 M rows 122 -> 127).
        if (a.n_dev && grid > kRowKernelMaxBlocks / 2) grid = kRowKernelMaxBlocks / 2;
        a.n_waves = grid * kWavesPerBlock;
        if (grid > most) most = grid;
    }
    if (n == 1) hipLaunchKernelGGL((quantize_units_kernel<LPR, U, SB, BITS, 1>), dim3(most), dim3(kBlock), 0, s, QuantBatchArgs<1>{{b.job[0]}});
    else hipLaunchKernelGGL((quantize_units_kernel<LPR, U, SB, BITS, CNR_MAX_BATCH>), dim3(most, n), dim3(kBlock), 0, s, b);
}

// The greedy search, which takes one table per launch.
template <int BITS>
void launch_greedy_bits(QuantArgs &a, hipStream_t s) {
    if (launch_greedy_short<BITS>(a, s)) return;
    if (a.dim == 16) return launch_greedy<1, BITS, 1>(a, s);
    if (a.dim == 32) return launch_greedy_by_length<2, 1, 2, BITS>(a, s);
    if (a.dim == 64) return launch_greedy_by_length<4, 1, 4, BITS>(a, s);
    if (a.dim == 128) return launch_greedy_by_length<8, 2, 4, BITS>(a, s);
    if (a.dim == 256) return launch_greedy_by_length<16, 4, 4, BITS>(a, s);
    return launch_greedy_units<BITS>(a, s);
}

// Min/max or symmetric ranges at row lengths the tile kernel does not take.
//
// Longest list that goes a row per wave: rows of more than 512 elements, and the lists of more than 192 on which the
// registers that the units kernel holds keep too few rows in flight.  Measured break-evens: rows of 200 and 252 at 13 K and
// 15 K, of 264 and 320 at 16 K, of 384 at 20 K, of 448 at 45 K, of 512 at 70 K (12 K rows: 6.0 against 9.2 us).
inline uint64_t rows_by_wave(uint32_t dim) {
    const uint32_t n4 = dim / 4;
    return n4 > 128 ? ~0ull : n4 <= 48 ? 0 : n4 <= 80 ? 12288 : 8192ull << ((n4 - 65) / 16);
}
template <int BITS>
void launch_strided(cnr_ctx *ctx, QuantBatchArgs<> &b, uint32_t n, hipStream_t s) {
    unsigned most = 1;
    for (uint32_t i = 0; i < n; ++i) {
        const unsigned grid = cnr_grid(ctx, b.job[i].n_max, kWavesPerBlock, cnr_resident_blocks_per_cu<quantize_strided_kernel<BITS, 1>>());
        b.job[i].n_waves = grid * kWavesPerBlock;
        if (grid > most) most = grid;
    }
    if (n == 1) hipLaunchKernelGGL((quantize_strided_kernel<BITS, 1>), dim3(most), dim3(kBlock), 0, s, QuantBatchArgs<1>{{b.job[0]}});
    else hipLaunchKernelGGL((quantize_strided_kernel<BITS, CNR_MAX_BATCH>), dim3(most, n), dim3(kBlock), 0, s, b);
}
// Few idle lanes at every length (units of a row: lanes x units per lane), and 64 registers of row data or
// fewer on their way per lane
template <int BITS>
void launch_units_any(QuantBatchArgs<> &b, uint32_t n, uint32_t dim, hipStream_t s) {
    const uint32_t n4 = dim / 4;
    if (n4 <= 4) return launch_units<4, 1, 4, BITS>(b, n, s);
    if (n4 <= 8) return launch_units<8, 1, 4, BITS>(b, n, s);
    if (n4 <= 12) return launch_units<4, 3, 2, BITS>(b, n, s);
    if (n4 <= 16) return launch_units<8, 2, 4, BITS>(b, n, s);
    if (n4 <= 24) return launch_units<8, 3, 2, BITS>(b, n, s);
    if (n4 <= 32) return launch_units<8, 4, 2, BITS>(b, n, s);
    if (n4 <= 40) return launch_units<8, 5, 2, BITS>(b, n, s);
    if (n4 <= 48) return launch_units<8, 6, 2, BITS>(b, n, s);
    if (n4 <= 56) return launch_units<8, 7, 2, BITS>(b, n, s);
    if (n4 <= 64) return launch_units<8, 8, 2, BITS>(b, n, s);
    if (n4 <= 80) return launch_units<16, 5, 2, BITS>(b, n, s);
    if (n4 <= 96) return launch_units<16, 6, 2, BITS>(b, n, s);
    if (n4 <= 112) return launch_units<16, 7, 2, BITS>(b, n, s);
    return launch_units<16, 8, 2, BITS>(b, n, s);
}
// by_wave: every table of the launch is one of rows_by_wave or fewer rows
template <int BITS>
void launch_rows(cnr_ctx *ctx, QuantBatchArgs<> &b, uint32_t n, uint32_t dim, bool by_wave, hipStream_t s) {
    if (by_wave) launch_strided<BITS>(ctx, b, n, s);
    else launch_units_any<BITS>(b, n, dim, s);
}

template <int BITS>
cnr_status launch_sample_errors(cnr_ctx *ctx, SelectArgs &a, uint32_t n_points, uint32_t n_searches, uint64_t max_sums, double *mean_out, hipStream_t s) {
    const uint32_t n4 = a.dim / 4;
    const uint32_t lanes = cnr_sample_lanes(a.dim, a.n, n_searches);
    a.grid = cnr_sample_grid(lanes, a.n, n_points, max_sums);
    const dim3 g(a.grid, n_searches);
    if (lanes == 4 && n4 < 36) hipLaunchKernelGGL((sample_error_kernel<4, 8, false, BITS>), g, dim3(kBlock), 0, s, a);
    else if (lanes == 4) hipLaunchKernelGGL((sample_error_kernel<4, 16, false, BITS>), g, dim3(kBlock), 0, s, a);
    else if (lanes == 8) hipLaunchKernelGGL((sample_error_kernel<4, 2, true, BITS>), g, dim3(kBlock), 0, s, a);
    else if (lanes == 16) hipLaunchKernelGGL((sample_error_kernel<8, 8, true, BITS>), g, dim3(kBlock), 0, s, a);
    else if (lanes == 32) hipLaunchKernelGGL((sample_error_kernel<16, 4, true, BITS>), g, dim3(kBlock), 0, s, a);
    else if (n4 < 288) hipLaunchKernelGGL((sample_error_kernel<32, 8, true, BITS>), g, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((sample_error_kernel<64, 16, false, BITS>), g, dim3(kBlock), 0, s, a);
    cnr_status st = cnr_launch_status(ctx);
    if (st != CNR_OK) return st;
    hipLaunchKernelGGL(sample_mean_kernel, dim3(n_points), dim3(kBlock), 0, s, a.sums, a.grid, (double)a.n, mean_out);
    return cnr_launch_status(ctx);
}

}  // namespace

cnr_status cnr_sample_errors(cnr_ctx *ctx, const float *table, uint64_t n_rows, uint32_t dim, const uint32_t *row_ids,
                             uint64_t n, int bits, const cnr_search_params *points, uint32_t n_points, double *sums,
                             uint64_t max_sums, double *mean_out, hipStream_t s) {
    for (uint32_t done = 0; done < n_points;) {
        uint32_t m = n_points - done;
        if (m > kSearchBatch) m = kSearchBatch;
        if (m > max_sums) m = (uint32_t)max_sums;  // >= 1
        SelectArgs a = {table, n_rows, dim, row_ids, n, tie_factor(dim), sums, 0, ctx->dev_err, {}, {}};
        uint32_t n_searches = 0;
        for (uint32_t i = 0; i < m; ++i) {
            a.points[i] = points[done + i];
            const bool goes_on = i && a.points[i].num_bins_f == a.points[i - 1].num_bins_f && a.points[i].n_iter >= a.points[i - 1].n_iter;
            if (!goes_on) a.first[n_searches++] = (uint8_t)i;
        }
        a.first[n_searches] = (uint8_t)m;
        cnr_status st;
        switch (bits) {
            case 2: st = launch_sample_errors<2>(ctx, a, m, n_searches, max_sums, mean_out + done, s); break;
            case 3: st = launch_sample_errors<3>(ctx, a, m, n_searches, max_sums, mean_out + done, s); break;
            case 4: st = launch_sample_errors<4>(ctx, a, m, n_searches, max_sums, mean_out + done, s); break;
            default: st = launch_sample_errors<8>(ctx, a, m, n_searches, max_sums, mean_out + done, s); break;
        }
        if (st != CNR_OK) return st;
        done += m;
    }
    return CNR_OK;
}

extern "C" {

cnr_status cnr_quantize_rows_batch(cnr_ctx *ctx, const cnr_table_job *jobs, uint32_t n_jobs, uint32_t dim,
                                   int bits, cnr_range_mode mode, const cnr_greedy_params *greedy,
                                   void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (!cnr_valid_bits(bits)) return CNR_E_BITS;
    if (dim == 0 || dim % 4 || dim > CNR_MAX_DIM || ((uint64_t)dim * (uint64_t)bits) % 8) return CNR_E_DIM;
    if (mode != CNR_RANGE_MINMAX && mode != CNR_RANGE_GREEDY && mode != CNR_RANGE_SYMMETRIC) return CNR_E_INVALID;
    if (mode == CNR_RANGE_GREEDY && !greedy) return CNR_E_INVALID;
    if (n_jobs && !jobs) return CNR_E_INVALID;
    for (uint32_t i = 0; i < n_jobs; ++i) {
        const cnr_table_job &j = jobs[i];
        if (j.capacity == 0) continue;
        if (!j.table || !j.scale || !j.bias || j.n_rows == 0 || j.n_rows >= (1ull << 32)) return CNR_E_INVALID;
        if (((uintptr_t)j.table % 16) || ((uintptr_t)j.packed % 16) || ((uintptr_t)j.codes_u8 % 16) ||
            ((uintptr_t)j.scale % 4) || ((uintptr_t)j.bias % 4) || ((uintptr_t)j.row_min % 4) ||
            ((uintptr_t)j.row_max % 4) || ((uintptr_t)j.row_ids % 16) || ((uintptr_t)j.n_dirty_dev % 8))
            return CNR_E_ALIGN;
    }
    hipStream_t s = as_stream(stream);
    const uint32_t n_iter = mode == CNR_RANGE_GREEDY ? cnr_greedy_iterations(greedy->num_bins, greedy->ratio) : 0;
    const uint64_t prb = (uint64_t)dim * (uint64_t)bits / 8u;
    // rows k0 .. k0 + m - 1 of job j's list as arguments of its own
    auto part = [&](const cnr_table_job &j, uint64_t k0, uint64_t m) {
        QuantArgs a = {};
        a.dim = dim;
        if (j.row_ids) {
            a.table = j.table; a.n_rows = j.n_rows; a.row_ids = j.row_ids + k0;
        } else {  // no id list: the table from row k0 on
            a.table = j.table + k0 * dim; a.n_rows = j.n_rows - k0; a.row_ids = nullptr;
        }
        a.n_dev = j.n_dirty_dev; a.n_max = m;
        a.mode = (int)mode; a.n_iter = n_iter;
        a.num_bins_f = mode == CNR_RANGE_GREEDY ? (float)greedy->num_bins : 1.0f;
        a.scale = j.scale + k0; a.bias = j.bias + k0;
        a.row_min = j.row_min ? j.row_min + k0 : nullptr;
        a.row_max = j.row_max ? j.row_max + k0 : nullptr;
        a.codes = j.codes_u8 ? j.codes_u8 + k0 * dim : nullptr;
        a.packed = j.packed ? j.packed + k0 * prb : nullptr;
        a.err = ctx->dev_err;
        return a;
    };
    if (n_iter) {  // greedy search: one launch per table
        for (uint32_t i = 0; i < n_jobs; ++i) {
            const cnr_table_job &j = jobs[i];
            if (j.capacity == 0) continue;
            QuantArgs a = part(j, 0, j.capacity);
            switch (bits) {
                case 2: launch_greedy_bits<2>(a, s); break;
                case 3: launch_greedy_bits<3>(a, s); break;
                case 4: launch_greedy_bits<4>(a, s); break;
                default: launch_greedy_bits<8>(a, s); break;
            }
            if ((st = cnr_launch_status(ctx)) != CNR_OK) return st;
        }
        return CNR_OK;
    }
    // Up to CNR_MAX_BATCH tables per launch.  Small tables (rows of at most kSideBySideBytes at capacity) and large
    // ones go into launches of their own kind, so that a small table is not given a large one's grid, and
    // so do the tables that go a row per wave; for the tile kernel a list whose length the host knows is cut into
    // slices (cnr_slice_rows), each a table of the launch.
    const bool tile_dim = dim == 16 || dim == 32 || dim == 64 || dim == 128 || dim == 256;
    const uint64_t wave_rows = tile_dim ? 0 : rows_by_wave(dim);
    QuantBatchArgs<> b;  // 2 KB; what a launch reads of it is written before
    for (int kind = 0; kind < (wave_rows ? 4 : 2); ++kind) {
        const bool large = kind & 1, by_wave = kind & 2;
        uint32_t n = 0;
        auto flush = [&]() -> cnr_status {
            if (n == 0) return CNR_OK;
            if (tile_dim) launch_tile_any(b, n, dim, bits, s);
            else if (bits == 2) launch_rows<2>(ctx, b, n, dim, by_wave, s);
            else if (bits == 3) launch_rows<3>(ctx, b, n, dim, by_wave, s);
            else if (bits == 4) launch_rows<4>(ctx, b, n, dim, by_wave, s);
            else launch_rows<8>(ctx, b, n, dim, by_wave, s);
            n = 0;
            return cnr_launch_status(ctx);
        };
        for (uint32_t i = 0; i < n_jobs; ++i) {
            const cnr_table_job &j = jobs[i];
            if (j.capacity == 0 || (j.capacity * 4ull * dim > kSideBySideBytes) != large || (j.capacity <= wave_rows) != by_wave) continue;
            const bool sliceable = tile_dim && !j.n_dirty_dev && (j.row_ids || j.capacity <= j.n_rows);
            const uint64_t step = sliceable ? cnr_slice_rows(j.capacity, dim) : j.capacity;
            for (uint64_t k0 = 0; k0 < j.capacity; k0 += step) {
                b.job[n++] = part(j, k0, j.capacity - k0 < step ? j.capacity - k0 : step);
                if (n == CNR_MAX_BATCH && (st = flush()) != CNR_OK) return st;
            }
        }
        if ((st = flush()) != CNR_OK) return st;
    }
    return CNR_OK;
}

cnr_status cnr_quantize_rows(cnr_ctx *ctx, const float *table, uint64_t n_rows, uint32_t dim,
                             const uint32_t *row_ids, const uint64_t *n_dev, uint64_t n_max,
                             int bits, cnr_range_mode mode, const cnr_greedy_params *greedy,
                             float *scale, float *bias, float *row_min, float *row_max,
                             uint8_t *codes_u8, uint8_t *packed, void *stream) {
    cnr_table_job j = {};
    j.table = const_cast<float *>(table);
    j.n_rows = n_rows;
    j.row_ids = const_cast<uint32_t *>(row_ids);
    j.n_dirty_dev = const_cast<uint64_t *>(n_dev);
    j.capacity = n_max;
    j.scale = scale; j.bias = bias; j.row_min = row_min; j.row_max = row_max;
    j.codes_u8 = codes_u8; j.packed = packed;
    return cnr_quantize_rows_batch(ctx, &j, 1, dim, bits, mode, greedy, stream);
}

cnr_status cnr_pack(cnr_ctx *ctx, const uint8_t *codes_u8, const uint64_t *n_dev, uint64_t n_max,
                    uint32_t dim, int bits, uint8_t *packed, void *stream) {
    cnr_status st = cnr_enter(ctx);
    if (st != CNR_OK) return st;
    if (!cnr_valid_bits(bits)) return CNR_E_BITS;
    if (dim == 0 || dim > CNR_MAX_DIM || ((uint64_t)dim * (uint64_t)bits) % 8) return CNR_E_DIM;
    if (n_max == 0) return CNR_OK;
    if (!codes_u8 || !packed) return CNR_E_INVALID;
    if ((uintptr_t)n_dev % 8) return CNR_E_ALIGN;
    const uint64_t bytes = n_max * cnr_packed_row_bytes(dim, bits);
    const unsigned grid = cnr_grid(ctx, bytes, kBlock, 16);
    hipStream_t s = as_stream(stream);
    switch (bits) {
        case 2: hipLaunchKernelGGL(pack_kernel<2>, dim3(grid), dim3(kBlock), 0, s, codes_u8, n_dev, n_max, dim, packed, (uint64_t)grid * kBlock); break;
        case 3: hipLaunchKernelGGL(pack_kernel<3>, dim3(grid), dim3(kBlock), 0, s, codes_u8, n_dev, n_max, dim, packed, (uint64_t)grid * kBlock); break;
        case 4: hipLaunchKernelGGL(pack_kernel<4>, dim3(grid), dim3(kBlock), 0, s, codes_u8, n_dev, n_max, dim, packed, (uint64_t)grid * kBlock); break;
        default: hipLaunchKernelGGL(pack_kernel<8>, dim3(grid), dim3(kBlock), 0, s, codes_u8, n_dev, n_max, dim, packed, (uint64_t)grid * kBlock); break;
    }
    return cnr_launch_status(ctx);
}

}  // extern "C"
