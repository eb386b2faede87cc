// Pre-alignment filter (score-only mode).
//
// The least edit distance between the whole read and any substring of the
// reference, on vertical differences (diff_window.h): E(i) = the read's
// distance to the best prefix of the reference from column i on, for the
// columns from the last to the first, with no table and no traceback. A pair
// takes G lanes, each with 64 rows of the read, lane G-1 its first 64 bases:
// lane l is a column behind lane l-1, which hands it the horizontal difference
// of its last row (the block form of the recurrence, in the paper that
// diff_window.h names). A step costs a lane about 38 instructions, whatever k
// is, and G lanes of a wavefront share it, so a wavefront holds 64 / G pairs
// and a short batch of long reads still fills the chip: issue-bound. 20,000
// reads of 250 bases take 44 us and 4,000 of 1,000 bases 86 us; with a lane per
// row of the distance (64 rows whatever k is, 12 instructions per word) they
// took 948 and 2406 us.
#pragma once

#include "diff_window.h"

constexpr int kFilterSteps = 32;  // columns per block

// The 2-bit codes of 32 bases of a packed stream of nbytes bytes from base
// `base` on, base k in bits 2k, 2k+1; bases outside the stream read as 0.
__device__ __forceinline__ u64 packed_bases(const uint8_t* s, uint64_t nbytes, int64_t base) {
    const int64_t q = base >> 2;
    uint32_t w[3] = {0u, 0u, 0u};
    if (q >= 0 && (uint64_t)q + 12 <= nbytes) {
        __builtin_memcpy(w, s + q, 12);
    } else {
        for (int k = 0; k < 9; ++k) {
            const int64_t at = q + k;
            if (at >= 0 && (uint64_t)at < nbytes) w[k / 4] |= (uint32_t)s[at] << (8 * (k % 4));
        }
    }
    const int sh = 2 * (int)(base & 3);
    const u64 lo = ((u64)w[1] << 32) | w[0];
    return sh ? (lo >> sh) | ((u64)w[2] << (64 - sh)) : lo;
}

// Bit planes of the 64 bases from `base` on.
__device__ __forceinline__ void packed_planes(const uint8_t* s, uint64_t nbytes, int64_t base, u64& lo, u64& hi) {
    lo = hi = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u64 w = packed_bases(s, nbytes, base + 32 * h);
        const uint32_t w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32);
        lo |= (u64)(even_bits(w0) | (even_bits(w1) << 16)) << (32 * h);
        hi |= (u64)(even_bits(w0 >> 1) | (even_bits(w1 >> 1) << 16)) << (32 * h);
    }
}

// Value of the lane before in the wavefront's row of 16 lanes (lane 0 of the
// row: 0); `keep` is 0 in the first lane of a group.
__device__ __forceinline__ uint32_t from_lane_before(uint32_t x, uint32_t keep) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppRowShr1, 0xF, 0xF, true) & keep;
}

struct FilterLane {
    DiffColumn c;
    uint32_t ph, mh;  // top halves of the last step's Ph, Mh
    int score;
};

// kFilterSteps columns, the rightmost first. text: bases of the block's columns;
// out: bit t set where column t of the block lies outside the reference.
// CHAIN: the rows below this lane's are the lane's before. Returns the least
// (score << 6 | column of the block), valid in a group's last lane.
template <bool EDGE, bool CHAIN>
__device__ __forceinline__ uint32_t filter_block(FilterLane& f, u64 a, u64 b, u64 pad, uint32_t keep,
                                                 u64 text, uint32_t out) {
    const uint32_t tw[2] = {here((uint32_t)text), here((uint32_t)(text >> 32))};
    uint32_t best = ~0u;
#pragma unroll
    for (int x = kFilterSteps - 1; x >= 0; --x) {
        const uint32_t ph = CHAIN ? from_lane_before(f.ph, keep) : 0u;
        const uint32_t mh = CHAIN ? from_lane_before(f.mh, keep) : 0u;
        u64 ne = a ^ both(bit_mask(tw[x / 16], 2 * (x % 16)));
        uint32_t off = 0u;
        if constexpr (EDGE) {
            off = bit_mask(out, x);
            ne |= both(off);
        }
        u64 Eq = bit_op<~(kA | (kB ^ kC))>(ne, b, both(bit_mask(tw[x / 16], 2 * (x % 16) + 1)));
        Eq |= pad;
        // a column step whose row below the first changes by (ph, mh) at bit 31
        Eq |= (u64)(mh >> 31);
        const u64 sum = (Eq & f.c.Pv) + f.c.Pv;
        const u64 D0 = bit_op<(kA ^ kB) | kC>(sum, f.c.Pv, Eq | f.c.Mv);
        const u64 Ph = bit_op<kA | ~(kB | kC)>(f.c.Mv, D0, f.c.Pv);
        const u64 Mh = f.c.Pv & D0;
        const uint32_t pl = (uint32_t)Ph, ml = (uint32_t)Mh;
        f.ph = (uint32_t)(Ph >> 32);
        f.mh = (uint32_t)(Mh >> 32);
        const u64 Ps = ((u64)__builtin_amdgcn_alignbit(f.ph, pl, 31) << 32) |
                       __builtin_amdgcn_alignbit(pl, ph, 31);
        const u64 Ms = ((u64)__builtin_amdgcn_alignbit(f.mh, ml, 31) << 32) |
                       __builtin_amdgcn_alignbit(ml, mh, 31);
        f.c.Pv = bit_op<kA | ~(kB | kC)>(Ms, D0, Ps);
        f.c.Mv = Ps & D0;
        f.score += (int)(f.ph >> 31) + ((int32_t)f.mh >> 31);
        uint32_t key = ((uint32_t)f.score << 6) + (uint32_t)x;
        if constexpr (EDGE) key |= off;  // columns outside the reference are no start
        best = min(best, key);
    }
    return best;
}

template <int G>
__global__ __launch_bounds__(64) void k_filter(const uint8_t* reads, const uint64_t* read_off,
                                               const uint8_t* refs, const uint64_t* ref_off,
                                               uint64_t n_pairs, int32_t K, int32_t* dist,
                                               uint32_t* start) {
    const int lane = threadIdx.x & 63;
    const int gl = lane & (G - 1);
    const uint64_t pair = (uint64_t)blockIdx.x * (64 / G) + (uint64_t)(lane / G);
    const bool have = pair < n_pairs;
    const uint64_t rb = have ? read_off[pair] : 0, fb = have ? ref_off[pair] : 0;
    const int m = have ? (int)(read_off[pair + 1] - rb) : 0;
    const int n = have ? (int)(ref_off[pair + 1] - fb) : 0;
    const uint64_t read_bytes = (read_off[n_pairs] + 3) / 4, ref_bytes = (ref_off[n_pairs] + 3) / 4;
    // this lane's rows: read bases j0 .. j0 + 63, the first at bit 63; rows past
    // the read match everything and stay at 0
    const int j0 = 64 * (G - 1 - gl);
    const int rows = clampi(m - j0, 0, 64);
    const u64 pad = rows == 64 ? 0ull : ~0ull >> rows;
    u64 a = 0, b = 0;
    if (rows > 0) {
        u64 lo, hi;
        packed_planes(reads, read_bytes, (int64_t)rb + j0, lo, hi);
        a = __builtin_bitreverse64(lo);
        b = __builtin_bitreverse64(hi);
    }
    FilterLane f{{~pad, 0ull}, 0u, 0u, m};
    const uint32_t keep = gl ? ~0u : 0u;
    int best = m, col = n;  // the empty substring at the reference's end
    // block: this lane's columns top, top - 1, .. top - kFilterSteps + 1
    int top = n - 1 + gl;
    int left = n > 0 ? n + G - 1 : 0;  // steps the group still has to take
    u64 next = packed_bases(refs, ref_bytes, (int64_t)fb + top - (kFilterSteps - 1));
    while (__ballot(left > 0) != 0ull) {
        const int c0 = top - (kFilterSteps - 1);
        const u64 text = next;
        // the next block's bases arrive while this one's columns are computed
        if (left > kFilterSteps) next = packed_bases(refs, ref_bytes, (int64_t)fb + c0 - kFilterSteps);
        // column c0 + t lies in the reference for -c0 <= t < n - c0
        uint32_t out = 0u;
        if (top >= n) out |= n - c0 <= 0 ? ~0u : ~0u << (n - c0);
        if (c0 < 0) out |= c0 <= -kFilterSteps ? ~0u : ~(~0u << -c0);
        const uint32_t k = __ballot(out != 0u) != 0ull ? filter_block<true, true>(f, a, b, pad, keep, text, out)
                                                       : filter_block<false, true>(f, a, b, pad, keep, text, 0u);
        // a later block lies further left, so it wins ties
        if (k != ~0u && (int)(k >> 6) <= best) {
            best = (int)(k >> 6);
            col = c0 + (int)(k & 63u);
        }
        top -= kFilterSteps;
        left -= kFilterSteps;
    }
    if (have && gl == G - 1) {
        const bool ok = best <= K;
        dist[pair] = ok ? best : -1;
        start[pair] = ok ? (uint32_t)col : 0u;
    }
}

int filter_words(uint32_t max_read_len) {
    return max_read_len <= 64 ? 1 : max_read_len <= 128 ? 2 : max_read_len <= 256 ? 4
         : max_read_len <= 512 ? 8 : max_read_len <= 1024 ? 16 : 0;
}

hipError_t launch_filter(const uint8_t* reads, const uint64_t* read_off, const uint8_t* refs,
                         const uint64_t* ref_off, uint64_t n_pairs, uint32_t max_read_len,
                         int32_t k, int32_t* dist, uint32_t* start, hipStream_t s) {
    if (n_pairs == 0) return hipSuccess;
    const int G = filter_words(max_read_len);  // a lane per 64 read bases
    const int K = k < 63 ? k : 63;
    if (G == 0) return hipErrorInvalidValue;
    const uint64_t per = 64 / (uint64_t)G;
    const dim3 grid((unsigned)((n_pairs + per - 1) / per)), block(64);
    switch (G) {
        case 1: hipLaunchKernelGGL(k_filter<1>, grid, block, 0, s, reads, read_off, refs, ref_off, n_pairs, K, dist, start); break;
        case 2: hipLaunchKernelGGL(k_filter<2>, grid, block, 0, s, reads, read_off, refs, ref_off, n_pairs, K, dist, start); break;
        case 4: hipLaunchKernelGGL(k_filter<4>, grid, block, 0, s, reads, read_off, refs, ref_off, n_pairs, K, dist, start); break;
        case 8: hipLaunchKernelGGL(k_filter<8>, grid, block, 0, s, reads, read_off, refs, ref_off, n_pairs, K, dist, start); break;
        default: hipLaunchKernelGGL(k_filter<16>, grid, block, 0, s, reads, read_off, refs, ref_off, n_pairs, K, dist, start); break;
    }
    return hipGetLastError();
}
