// One pair per wavefront: start search and windows in one kernel, for the plain
// form and for batches too small to fill the chip a pair per lane.
//
// A window on diagonals. E(i, j) is the distance of diff_window.h. Along a
// diagonal (j - i fixed) it never grows towards the end, so the cells with E <=
// d are those from a first text base f_d on; level d is one number per
// diagonal, and with a diagonal per lane a level is one step for all of them:
//   f_d(t) = the least i from which the bases of diagonal t match up to
//            min(f_d-1(t) - 1, f_d-1(t + 1), f_d-1(t - 1) - 1)
// (a substitution, an insertion or a deletion before a cell of the level
// below), and level 0 starts from the read window's end. (Ukkonen, Algorithms
// for approximate string matching, 1985, from the end and with a free text
// end.) d* is the first level that reaches (0, 0). The traceback asks for E of
// neighbouring cells against d - 1 only, which is f_d-1 of their diagonals. A
// level costs 14 instructions, about 90 cycles of a wavefront that has its SIMD
// to itself, and an edit of the traceback 31 scalar ones, so a window costs by
// its distance: about 1.7 us at d* = 6 and 4.4 us at d* = 33 (unrelated bases),
// where a lane's column-by-column step (diff_window.h) takes 5 us, for up to 64
// pairs at once. 67 reads of 30 kb: 15.1 ms in row tables -> 2.6.
//
// An alignment of d edits from (0, 0) stays on diagonals -(d + nw - mw) / 2 .. d:
// past -x it needs x deletions, and then x + mw - nw insertions to reach the
// read window's end. So 64 diagonals from -kBandBelow on give the exact answer
// up to d = 42 (two full windows), and the rare rest is done again with all 128.
#pragma once

#include "diff_window.h"

constexpr int kBandBelow = 21;
// A diagonal's levels 0..64 (and one computed past them), one byte each, side by side: only its
// lane writes and reads them, four at a time on the way back (17 words apart,
// so the lanes' words lie in different banks).
constexpr int kWaveLevels = 68;
constexpr int kWaveLdsBytes = kWaveLevels * 128;

// Cross-lane moves over the whole wavefront. Values the others call with are
// the same in every lane (lane numbers, and what readlane returns).
__device__ __forceinline__ int read_lane(int v, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readlane(v, lane);
#else
    return __shfl(v, lane);
#endif
}
__device__ __forceinline__ u64 read_lane64(u64 v, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    // built from its halves, which two shifts and an or would cost moves for
    typedef uint32_t halves __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(u64, halves{(uint32_t)read_lane((int)v, lane), (uint32_t)read_lane((int)(v >> 32), lane)});
#else
    return ((u64)(uint32_t)read_lane((int)(v >> 32), lane) << 32) | (uint32_t)read_lane((int)v, lane);
#endif
}
__device__ __forceinline__ uint32_t write_lane(uint32_t old, uint32_t v, int at, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    (void)lane;
    asm("v_writelane_b32 %0, %1, %2" : "+v"(old) : "s"(v), "{m0}"(at));
    return old;
#else
    return lane == at ? v : old;
#endif
}
// Zeros below the lowest set bit, 64 or more when there is none.
__device__ __forceinline__ uint32_t trailing_zeros(u64 v) {
#if defined(__HIP_DEVICE_COMPILE__)
    int r;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(v));  // -1 for 0
    return (uint32_t)r;
#else
    return v ? (uint32_t)__builtin_ctzll(v) : ~0u;
#endif
}
// The next (previous) lane's value; the last (first) lane gets `edge`.
__device__ __forceinline__ int lane_above(int v, int edge, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    (void)lane;
    return __builtin_amdgcn_update_dpp(edge, v, 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
#else
    const int x = __shfl(v, (lane + 1) & 63);
    return lane == 63 ? edge : x;
#endif
}
__device__ __forceinline__ int lane_below(int v, int edge, int lane) {
    (void)lane;
    return __builtin_amdgcn_update_dpp(edge, v, kDppWaveShr1, 0xF, 0xF, false);
}
// The same with 0 at the edge.
__device__ __forceinline__ int lane_above0(int v, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    (void)lane;
    return __builtin_amdgcn_update_dpp(0, v, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
#else
    return lane_above(v, 0, lane);
#endif
}
__device__ __forceinline__ int lane_below0(int v, int lane) {
    (void)lane;
    return __builtin_amdgcn_update_dpp(0, v, kDppWaveShr1, 0xF, 0xF, true);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ u64 uniform64(u64 v) {
    return ((u64)(uint32_t)uniform((int)(v >> 32)) << 32) | (uint32_t)uniform((int)v);
}
__device__ __forceinline__ u64 wave_min(u64 v, int lane) {
    for (int s = 1; s < 64; s <<= 1) v = min(v, (u64)__shfl(v, lane ^ s));
    return uniform64(v);
}

// A sequence read forward in blocks of 64 bases: two blocks as bit planes, the
// same in every lane, and the codes of the block after them on their way, one
// base per lane.
struct WaveSeq {
    const uint8_t* s;
    uint64_t base;  // stream offset of the sequence
    int len, block;
    u64 lo0, lo1, hi0, hi1;
    int next;  // the byte that holds the lane's code, shifted only when it is used
};
__device__ __forceinline__ int wave_seq_byte(const WaveSeq& q, int block, int lane) {
    const int64_t at = (int64_t)block * 64 + lane;
    return at < (int64_t)q.len ? (int)q.s[(q.base + (uint64_t)at) >> 2] : 0;
}
__device__ __forceinline__ int wave_seq_code(const WaveSeq& q, int byte, int lane) {
    return byte >> (2 * (int)((q.base + (uint64_t)lane) & 3u));  // blocks are whole bytes long
}
__device__ __forceinline__ void wave_seq_open(WaveSeq& q, const uint8_t* s, uint64_t base, int len, int at,
                                              int lane) {
    q.s = s;
    q.base = base;
    q.len = len;
    q.block = at >> 6;
    const int b0 = wave_seq_byte(q, q.block, lane), b1 = wave_seq_byte(q, q.block + 1, lane);
    q.next = wave_seq_byte(q, q.block + 2, lane);
    const int c0 = wave_seq_code(q, b0, lane), c1 = wave_seq_code(q, b1, lane);
    q.lo0 = __ballot(c0 & 1);
    q.hi0 = __ballot(c0 & 2);
    q.lo1 = __ballot(c1 & 1);
    q.hi1 = __ballot(c1 & 2);
}
// The 64 bases from `at` on (at most a block further than the last call's).
__device__ __forceinline__ void wave_seq_window(WaveSeq& q, int at, int lane, u64& lo, u64& hi) {
    if ((at >> 6) != q.block) {
        q.lo0 = q.lo1;
        q.hi0 = q.hi1;
        const int c = wave_seq_code(q, q.next, lane);
        q.lo1 = __ballot(c & 1);
        q.hi1 = __ballot(c & 2);
        ++q.block;
        q.next = wave_seq_byte(q, q.block + 2, lane);
    }
    lo = funnel64(q.lo0, q.lo1, at & 63);
    hi = funnel64(q.hi0, q.hi1, at & 63);
}

// The diagonals of a window: lane l of set s holds diagonal t = 64 s + l - below
// (text base i with read base j = i + t). A diagonal's cells are numbered from
// its first one: a = min(i, j), so all words and levels start at 0. Behind the
// text the diagonals go on with cells that always differ, up to the read
// window's end: an edit there costs what the insertion it stands for does, so
// no distance changes, and every diagonal that can be used has a level 0.
template <int SETS> struct WaveWindow {
    static constexpr int below = SETS == 1 ? kBandBelow : 63;  // two sets: -63 .. 64
    u64 ne[SETS];  // bit a: the bases of the diagonal's cell a differ
};

template <int SETS>
__device__ __forceinline__ void wave_window(WaveWindow<SETS>& w, u64 pl, u64 ph, u64 tl, u64 th, int nw, int lane) {
    const u64 text = nw < 64 ? ~(~0ull << nw) : ~0ull;
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int t = 64 * s + lane - WaveWindow<SETS>::below;
        const int r = max(t, 0) & 63, l = max(-t, 0);  // diagonal 64 has no cell to compare
        w.ne[s] = ((pl >> r) ^ (tl >> l)) | ((ph >> r) ^ (th >> l)) | ~(text >> l);
    }
}

// Zeros above the highest set bit, and at most `most`.
__device__ __forceinline__ int leading_zeros(u64 v, int most) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t h, l;  // ~0 for 0
    asm("v_ffbh_u32 %0, %1" : "=v"(h) : "v"((uint32_t)(v >> 32)));
    asm("v_ffbh_u32 %0, %1" : "=v"(l) : "v"((uint32_t)v));
    return (int)min(min(h, __builtin_elementwise_add_sat(l, 32u)), (uint32_t)most);
#else
    return v ? min(__builtin_clzll(v), most) : most;
#endif
}

// Levels 0.. into lev; returns the first that reaches (0, 0), or -1 when none up
// to d_max does. A level's f is held as g = 64 - f: the shift that brings the
// cell before f to the top (modulo 64), 0 for a diagonal beyond the band, whose
// neighbours learn nothing from it.
template <int SETS>
__device__ __forceinline__ int wave_levels(const WaveWindow<SETS>& w, uint8_t* lev, int mw, int d_max, int lane) {
    constexpr int below = WaveWindow<SETS>::below;
    int g[SETS], above[SETS], under[SETS];
    uint8_t* out[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int t = 64 * s + lane - below;
        g[s] = min(64 - mw + max(t, 0), 64);
        // a step away from the main diagonal's side shortens a by one
        above[s] = t < 0;
        under[s] = t > 0;
        out[s] = lev + (64 * s + lane) * kWaveLevels;
    }
    // matches before cell f, then the level's byte; returns g of (0, 0)'s
    // diagonal, 64 when the level reaches it
    auto extend = [&](int d) -> int {
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            g[s] += leading_zeros(w.ne[s] << (g[s] & 63), 64 - g[s]);
            out[s][d] = (uint8_t)g[s];
        }
        return read_lane(g[below / 64], below & 63);
    };
    auto level = [&](int d) -> int {  // d > 0: from the level before
        int up[SETS], dn[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            up[s] = s + 1 < SETS ? lane_above(g[s], read_lane(g[s + 1 < SETS ? s + 1 : s], 0), lane)
                                 : lane_above0(g[s], lane);
            dn[s] = s > 0 ? lane_below(g[s], read_lane(g[s > 0 ? s - 1 : s], 63), lane) : lane_below0(g[s], lane);
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s) g[s] = min(max(max(g[s] + 1, dn[s] + under[s]), up[s] + above[s]), 64);
        return extend(d);
    };
    if (extend(0) == 64) return 0;
    if (d_max < 1) return -1;
    // two levels a turn, so that the first one's answer is read while the second
    // is computed; what has reached (0, 0) stays there
    int d = 1, first, second;
    do {
        first = level(d);
        second = level(d + 1);
        d += 2;
    } while (second != 64 && d <= d_max);
    return first == 64 ? d - 2 : second == 64 && d - 1 <= d_max ? d - 1 : -1;
}

// The runs of a pair's CIGAR, the same in every lane.
struct WaveRuns {
    int cur_op;
    uint32_t cur_len, written, room;
    uint32_t* at;
};
__device__ __forceinline__ void wave_put(const WaveRuns& r, uint32_t index, uint32_t len, int op) {
    if (index < r.room) r.at[index] = (len << 2) | (uint32_t)op;
}
__device__ __forceinline__ void wave_run(WaveRuns& r, int op, int len, int lane) {
    if (op != r.cur_op) {
        if (r.cur_op >= 0) {
            if (lane == 0) wave_put(r, r.written, r.cur_len, r.cur_op);
            ++r.written;
        }
        r.cur_op = op;
        r.cur_len = 0u;
    }
    r.cur_len += (uint32_t)len;
}

// An edit of a traceback: the text base it stands at, its op, and what it adds
// to the text base and (the signed rest) to the diagonal.
constexpr int kEditOp = 6, kEditText = 8, kEditDiag = 9;
constexpr int kEditSub = (int)GENASM_OP_MISMATCH << kEditOp | 1 << kEditText;
constexpr int kEditIns = (int)GENASM_OP_INS << kEditOp | 1 << kEditDiag;
constexpr int kEditDel = (int)GENASM_OP_DEL << kEditOp | 1 << kEditText | -(1 << kEditDiag);

// Appends a window's n edits, one per lane, all at once: an edit starts a run
// unless it follows one of the same op without a match between; a run's place
// is the number of runs before it and its length the distance to the next start.
__device__ __forceinline__ void wave_edits(WaveRuns& r, int n, int edit, int lane) {
    const int op = (edit >> kEditOp) & 3, i = edit & 63;
    // behind the edit before; kept out of the subtraction, which the compiler would
    // make a v_subrev_u32_dpp of: on this card that gives shifted(s1) - s0 where s1 -
    // shifted(s0) is meant (with s1 = 10000 (lane + 1) and s0 = 100 + lane, lane 2
    // got 20000 - 102, not 30000 - 101)
    const int after = (int)here((uint32_t)lane_below0(i + ((edit >> kEditText) & 1), lane));
    const int matches = i - after;
    const bool have = lane < n;
    const int before = lane_below(op, -1, lane);
    const bool m = have && matches > 0, start = have && (matches > 0 || op != before);
    const u64 M = __ballot(m), S = __ballot(start);
    const u64 below = (1ull << lane) - 1ull;
    const int first_op = (M & 1ull) ? (int)GENASM_OP_MATCH : read_lane(op, 0);
    uint32_t open = 0u;  // length the first run takes over from the open one
    if (r.cur_op == first_op) {
        open = r.cur_len;
    } else if (r.cur_op >= 0) {
        if (lane == 0) wave_put(r, r.written, r.cur_len, r.cur_op);
        ++r.written;
    }
    const int last = 63 - __builtin_clzll(S);  // the last run stays open
    const u64 later = lane < 63 ? S >> (lane + 1) : 0ull;
    const int len = later ? 1 + __builtin_ctzll(later) : n - lane;
    const uint32_t at = r.written + (uint32_t)(__builtin_popcountll(M & below) + __builtin_popcountll(S & below));
    if (m) wave_put(r, at, (uint32_t)matches + (lane == 0 ? open : 0u), (int)GENASM_OP_MATCH);
    if (start && lane != last)
        wave_put(r, at + (m ? 1u : 0u), (uint32_t)len + (lane == 0 && !m ? open : 0u), op);
    r.written += (uint32_t)(__builtin_popcountll(M) + __builtin_popcountll(S)) - 1u;
    r.cur_op = read_lane(op, last);
    r.cur_len = (uint32_t)(n - last) + (last == 0 && !(M & 1ull) ? open : 0u);
}

// Traceback of a window of distance d from (0, 0); returns the edits it
// commits. Each edit lowers d by one, so the levels are read in order, four to a
// word, and the word after the next is on its way.
template <int SETS>
__device__ __forceinline__ int wave_trace(const WaveWindow<SETS>& w, const uint8_t* lev, int mw, int nw, int d,
                                          int L, int lane, WaveRuns& runs, int& i_end, int& j_end) {
    constexpr int below = WaveWindow<SETS>::below;
    const int j_max = min(mw, L), i_max = min(L, nw);
    int level = d - 1;  // the one the next edit asks
    const int lead = 8 * (3 - (level & 3));  // so that it is the top byte of its word
    u64 ne[SETS];       // bit i of it: text base i and the diagonal's read base differ
    int last[SETS];     // the diagonal's last committed text base, and one more
    uint32_t f64[SETS], word[SETS], next[SETS];
    uint32_t f[SETS], fi[SETS];  // four levels' first text bases, here and on the next diagonal
    auto load = [&](int at, int s) -> uint32_t {
        return *reinterpret_cast<const uint32_t*>(lev + (64 * s + lane) * kWaveLevels + (max(at, 0) & ~3));
    };
    // a level of the word is the diagonal's first text base plus 64 - g; bytes
    // above the level asked may be stale and don't reach those below
    auto fields = [&] {
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            f[s] = (uint32_t)(((((u64)(f64[s] - word[s])) << 32 | (f64[s] - next[s])) << lead) >> 32);
            word[s] = next[s];
            next[s] = load(level - 8, s);
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s)
            fi[s] = (uint32_t)lane_above((int)f[s], s + 1 < SETS ? read_lane((int)f[s + 1 < SETS ? s + 1 : s], 0) : -1,
                                         lane);
        level -= 4;
    };
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int t = 64 * s + lane - below, l = max(-t, 0);
        ne[s] = w.ne[s] << l;
        last[s] = min(i_max, j_max - t);
        f64[s] = (uint32_t)(64 + l) * 0x01010101u;
        word[s] = load(level, s);
        next[s] = load(level - 4, s);
    }
    int i = 0, x = below;  // text base and diagonal index: read base j = i + x - below
    int n = 0;
    int edit = 0;          // lane e: edit e
    // the matches, and the edit after them unless they end at the diagonal's last
    // committed cell (the next step inside, so that each has one branch)
    auto step = [&](int byte, auto&& then) {
        u64 differ = 0;
        int end = 0, fs = 0, fn = 0;
#pragma unroll
        for (int s = 0; s < SETS; ++s)
            if (SETS == 1 || (x >> 6) == s) {
                differ = read_lane64(ne[s], x & 63);
                end = read_lane(last[s], x & 63);
                fs = read_lane((int)f[s], x & 63);
                fn = read_lane((int)fi[s], x & 63);
            }
        // (at 64, the end of all, the mask is full)
        i = max(i, (int)min(trailing_zeros(differ & (~0ull << (i & 63))), (uint32_t)end));
        if (i == end) return;
        int e = ((fn >> (8 * byte)) & 0xFF) <= i ? kEditIns : kEditDel;
        e = ((fs >> (8 * byte)) & 0xFF) <= i + 1 ? kEditSub : e;
        edit = (int)write_lane((uint32_t)edit, (uint32_t)(e | i), n, lane);
        ++n;
        i += (e >> kEditText) & 1;
        x += e >> kEditDiag;
        then();
    };
    // i + j grows with every edit, so the loop ends
    bool more;
    do {
        fields();
        more = false;
        step(3, [&] { step(2, [&] { step(1, [&] { step(0, [&] { more = true; }); }); }); });
    } while (more);
    const int j = i + x - below;
    int tail = i;
    if (n > 0) {
        const int e = read_lane(edit, n - 1);
        tail -= (e & 63) + ((e >> kEditText) & 1);
        wave_edits(runs, n, edit, lane);
    }
    if (tail > 0) wave_run(runs, (int)GENASM_OP_MATCH, tail, lane);
    // past the text only insertions are left
    const int rest = i < L && j < j_max ? j_max - j : 0;
    if (rest > 0) wave_run(runs, (int)GENASM_OP_INS, rest, lane);
    i_end = i;
    j_end = j + rest;
    return n + rest;
}

// A window: distance (-1: above K) and, when it is solved, its traceback. STATS:
// `solved` is the clock between the two.
template <int SETS, bool STATS>
__device__ __forceinline__ int wave_solve(u64 pl, u64 ph, u64 tl, u64 th, int mw, int nw, int K, int L,
                                          uint8_t* lev, int lane, WaveRuns& runs, int& edits, int& i_end,
                                          int& j_end, bool& exact, u64& solved) {
    WaveWindow<SETS> w;
    wave_window<SETS>(w, pl, ph, tl, th, nw, lane);
    const int d_max = SETS == 1 ? min(K, 63 - kBandBelow) : K;
    const int d = wave_levels<SETS>(w, lev, mw, d_max, lane);
    if constexpr (STATS) solved = clock64();
    exact = SETS == 2;
    if (SETS == 1) {
        // no answer within K edits is one too when the band holds all of them
        const int e = d >= 0 ? d : d_max;
        exact = min(e, (e + nw - mw) / 2) <= kBandBelow && (d >= 0 || K <= 63 - kBandBelow);
    }
    if (!exact || d < 0) return -1;
    edits = wave_trace<SETS>(w, lev, mw, nw, d, L, lane, runs, i_end, j_end);
    return d;
}

// Long references. However long the references are on average, one may be as
// long as the rest together, so a pair's own lanes search no more than its first
// search_own columns, and the chunks after those get lanes of their own: 2,000 reads of 100 bases, one of them with a reference of 10 Mb, took 9.76
// ms (100,000 of 250: 488 ms) when its pair's lanes searched all of it, against
// 0.42 (2.04) by chunks of 4,096 columns on the row tables, and 0.15 (0.38) so.
//
// The chunks' lanes need no list. With chunks of C columns, lane x stands at base
// (x + 1) C of the batch's references; a reference of n columns holds at least
// floor(n / C) such places, as many as its columns past search_own take as long as
// C <= search_own. Sets the pair, its first place and the first column of lane x's
// chunk; false if there is none.
__device__ __forceinline__ bool search_tail(const AlignParams& P, uint64_t x, uint64_t& pair, int64_t& c0,
                                            uint64_t& first) {
    const int log = P.search_tail_log;
    const uint64_t at = (x + 1) << log, org = P.ref_off[0];
    uint64_t lo = 0, hi = P.n_pairs - 1;  // the first pair whose reference ends at `at` or later
    while (lo < hi) {
        const uint64_t mid = (lo + hi) / 2;
        if (P.ref_off[mid + 1] - org >= at) hi = mid;
        else lo = mid + 1;
    }
    const uint64_t a = P.ref_off[lo] - org, b = P.ref_off[lo + 1] - org;
    pair = lo;
    first = a >> log;
    const uint64_t c = P.search_own + ((x - first) << log);
    c0 = (int64_t)c;
    return at <= b && c < b - a;
}

// Start search of `cols` output columns from c0 on of a lane's pair; see search_part. A hit within Kr rows reaches at most m1 + Kr columns. All lanes
// of the wavefront call this together. Returns row << 32 | column.
__device__ __forceinline__ u64 wave_search(const AlignParams& P, const PairCursor& pc, int m1, int Kr, u64 pl,
                                           u64 ph, int64_t c0, int cols) {
    const uint64_t bytes = (P.ref_off[P.n_pairs] + 3) / 4;
    const int e = (int)min((int64_t)pc.n, c0 + cols + m1 + Kr);
    int nb = c0 < pc.n ? (int)((e - c0 + 31) / 32) : 0;
    const u64 a = __builtin_bitreverse64(pl), b = __builtin_bitreverse64(ph);
    const u64 pad = m1 < 64 ? (1ull << (64 - m1)) - 1 : 0ull;
    FilterLane f{{~pad, 0ull}, 0u, 0u, m1};
    u64 key = ~0ull;
    u64 next = nb > 0 ? packed_bases(P.refs, bytes, (int64_t)pc.fb + c0 + 32 * (nb - 1)) : 0ull;
    while (__ballot(nb > 0) != 0ull) {
        const int64_t col = c0 + 32 * (int64_t)(nb - 1);
        const u64 text = next;
        if (nb > 1) next = packed_bases(P.refs, bytes, (int64_t)pc.fb + col - 32);
        const int64_t valid = e - col;
        const uint32_t out = nb > 0 && valid >= 32 ? 0u : nb > 0 ? ~0u << (int)valid : ~0u;
        const uint32_t k = __ballot(out != 0u) != 0ull ? filter_block<true, false>(f, a, b, pad, 0u, text, out)
                                                       : filter_block<false, false>(f, a, b, pad, 0u, text, 0u);
        if (k != ~0u) key = min(key, ((u64)(k >> 6) << 32) | (u64)(uint32_t)(col + (int64_t)(k & 63u)));
        --nb;
    }
    return key;
}

// Adds a wavefront's least key over `parts` parts of a long reference (its pair's
// own columns, or a chunk a lane) to the others'. True in the wavefront that is
// the last: `key` is then the least of all, and the slot is as it was. Nothing
// waits for the others.
__device__ __forceinline__ bool tail_last(const AlignParams& P, uint64_t first, int n, uint32_t parts, u64& key, int lane) {
    SearchTailSlot* slot = P.tail_slots + first;
    const uint32_t all = 2u + (((uint32_t)n - (uint32_t)P.search_own - 1u) >> P.search_tail_log);
    u64 best = 0;
    int last = 0;
    if (lane == 0) {
        atomicMax(&slot->best, ~key);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        last = atomicAdd(&slot->done, (u64)parts) + parts == all;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (last) {
            // (given back by atomics too: other slots of the line are in use meanwhile)
            best = atomicMin(&slot->best, 0ull);
            atomicAdd(&slot->done, 0ull - all);
        }
    }
    if (!uniform(last)) return false;
    key = ~uniform64(best);
    return true;
}

// The windows of a pair from the state `st` on, to its end or (serving) to the
// end of its turn, and its result or state.
template <bool STATS, bool SERVE>
__device__ __forceinline__ void wave_pair_windows(const AlignParams& P, uint64_t pair, const PairCursor& pc, int col,
                                                  PairState st, uint8_t* lev, int lane, TurnClock& turn) {
    const uint64_t base = uniform64(pair_run_base(P, pair));
    const uint64_t limit = min(P.cigar_cap, base + (uint64_t)pc.m + (uint64_t)pc.n);
    WaveRuns runs{st.cur_op, st.cur_len, st.written,
                  (uint32_t)uniform((int)(limit > base ? limit - base : 0ull)), P.cigar + base};
    WaveSeq rd, rf;
    u64 pl, ph, tl, th;
    int ti = st.ti, pj = st.pj, score = st.score;
    uint32_t nwin = st.nwin, done_here = 0u;
    wave_seq_open(rd, P.reads, pc.rb, pc.m, pj, lane);
    wave_seq_open(rf, P.refs, pc.fb, pc.n, ti, lane);
    bool failed = false, internal = false, park = false;
    u64 st_wops = 0, st_cells = 0, st_table = 0, st_tb = 0, st_steps = 0, cyc_dc = 0, cyc_tb = 0;
    u64 cyc_start = 0, wall_start = 0;
    if constexpr (STATS) {
        cyc_start = clock64();
        wall_start = wall_clock64();
    }
    // every window commits at least one base, so a pair has at most m + n
    const uint32_t max_windows = (uint32_t)pc.m + (uint32_t)pc.n;
    while (pj < pc.m && !park) {
        if (nwin >= max_windows) {
            failed = internal = true;
            break;
        }
        const int mw = min(P.W, pc.m - pj), nw = min(P.W, pc.n - ti);
        if (!audit_ok(P, pair, kAuditWindow, P.W >= 2 && P.W <= 64 && mw >= 1 && nw >= 0)) {
            failed = internal = true;
            break;
        }
        ++nwin;
        ++done_here;
        u64 cyc0 = 0, solved = 0;
        if constexpr (STATS) cyc0 = solved = clock64();
        wave_seq_window(rd, pj, lane, pl, ph);
        wave_seq_window(rf, ti, lane, tl, th);
        int edits = 0, i_end = 0, j_end = 0, d;
        if (nw == 0) {  // past the text: insertions only
            d = mw <= P.K ? mw : -1;
            edits = j_end = min(mw, P.L);
            if (d >= 0) wave_run(runs, (int)GENASM_OP_INS, edits, lane);
        } else {
            bool exact = false;
            d = wave_solve<1, STATS>(pl, ph, tl, th, mw, nw, P.K, P.L, lev, lane, runs, edits, i_end, j_end, exact,
                                     solved);
            if (!exact)
                d = wave_solve<2, STATS>(pl, ph, tl, th, mw, nw, P.K, P.L, lev, lane, runs, edits, i_end, j_end, exact,
                                         solved);
        }
        if constexpr (STATS) {
            cyc_dc += solved - cyc0;
            cyc_tb += clock64() - solved;
            st_cells += (u64)mw * nw;
            st_steps += (u64)nw;
        }
        if (d < 0) {
            failed = true;
            break;
        }
        if constexpr (STATS) {
            st_wops += (u64)nw * (2 + 6 * (u64)d);
            st_table += (u64)(d + 1) * (min(nw, P.L) + 1);
            st_tb += 2 * (u64)edits;
        }
        score += edits;
        ti += i_end;
        pj += j_end;
        if constexpr (SERVE) {
            // a turn takes at least one window and starts none once it has ended
            park = pj < pc.m && ((turn.active && turn.over()) ||
                                 (P.window_budget != 0u && done_here >= P.window_budget));
        }
    }
    if (lane != 0) return;
    if (!park) {
        if (!failed && runs.cur_op >= 0) {
            wave_put(runs, runs.written, runs.cur_len, runs.cur_op);
            ++runs.written;
        }
        const bool overflow = runs.written > runs.room;
        genasm_result r;
        r.edit_distance = failed ? -1 : score;
        r.ref_begin = failed ? 0u : (uint32_t)col;
        r.ref_end = failed ? 0u : (uint32_t)ti;
        r.cigar_len = failed || overflow ? 0u : runs.written;
        r.n_windows = nwin;
        r.cigar_off = base;
        r.flags = (overflow && !failed ? GENASM_FLAG_CIGAR_OVERFLOW : 0u) | (internal ? GENASM_FLAG_INTERNAL : 0u);
        P.out[pair] = r;
    }
    if constexpr (STATS) {
        u64* stp = P.stats + pair * kStatCount;
        stp[kStatWindowWordOps] += st_wops;
        stp[kStatWindowCells] += st_cells;
        stp[kStatTableWords] += st_table;
        stp[kStatTbReads] += st_tb;
        stp[kStatWindowLaneSteps] += st_steps;
        stp[kStatWindows] += nwin;
        stp[kStatDcCycles] += cyc_dc;
        stp[kStatTbCycles] += cyc_tb;
        stp[kStatPairCycles] += clock64() - cyc_start;
        stp[kStatPairStart] = wall_start;
        stp[kStatPairEnd] = wall_clock64();
    }
    if constexpr (SERVE) {
        P.state[pair] = PairState{ti, pj, score, nwin, runs.written, runs.cur_op, runs.cur_len,
                                  kStateStarted | (park ? 0u : kStateDone) | (failed ? kStateFailed : 0u) |
                                      (internal ? kStateInternal : 0u)};
        if (P.fin_list) {
            if (!park) P.fin_list[atomicAdd(P.fin_len, 1u)] = (uint32_t)pair;
            else if (done_here <= 1u) P.next_hot[atomicAdd(P.next_len + kCounterEasyLen, 1u)] = (uint32_t)pair;
            else P.next_cold[atomicAdd(P.next_len + kCounterHardLen, 1u)] = (uint32_t)pair;
        }
    }
}

__device__ __forceinline__ PairCursor wave_cursor(const AlignParams& P, uint64_t pair) {
    PairCursor pc = pair_cursor(P, pair);
    pc.rb = uniform64(pc.rb);
    pc.fb = uniform64(pc.fb);
    pc.m = uniform(pc.m);
    pc.n = uniform(pc.n);
    return pc;
}

// A pair from its search's least key on.
template <bool STATS>
__device__ __forceinline__ void wave_pair_from_key(const AlignParams& P, uint64_t pair, const PairCursor& pc, u64 key,
                                                   uint8_t* lev, int lane) {
    const int m1 = min(P.W, pc.m);
    const int Kr = min(P.K, m1 - 1);
    key = (int)(key >> 32) <= Kr ? key : ~0ull;
    int row = -1, col = 0;
    if (key != ~0ull) {
        row = (int)(key >> 32);
        col = (int)(uint32_t)key;
    } else if (m1 <= P.K) {
        row = m1;  // row m1 hits in every column
    }
    if (STATS && lane == 0) search_stats(P, pair, pc.n, m1, row >= 0 ? row : Kr, (u64)pc.n, true);
    if (row < 0) {
        if (lane == 0) finish_without_windows(P, pair, -1);
        return;
    }
    TurnClock none;
    wave_pair_windows<STATS, false>(P, pair, pc, col, fresh_state(col), lev, lane, none);
}

// Workgroup i takes pair i. CHUNKS: the workgroups after the pairs search the
// chunks of long references, a lane per chunk; the last wavefront to finish a
// pair's search takes its windows. (An instance of its own, and the windows twice in
// it: with the chunks' code around them short calls took up to 0.4 us longer.)
template <bool STATS, bool CHUNKS>
__global__ __launch_bounds__(64) void k_pair_wave(AlignParams P) {
    extern __shared__ u64 smem[];
    uint8_t* lev = reinterpret_cast<uint8_t*>(smem);
    const int lane = threadIdx.x & 63;
    const uint64_t pair = blockIdx.x;
    u64 pl, ph;
    if (!CHUNKS || pair < P.n_pairs) {
        if (pair >= P.n_pairs) return;
        const PairCursor pc = wave_cursor(P, pair);
        if (pc.m == 0) {
            if (lane == 0) finish_without_windows(P, pair, 0);
            return;
        }
        WaveSeq rd;
        wave_seq_open(rd, P.reads, pc.rb, pc.m, 0, lane);
        wave_seq_window(rd, 0, lane, pl, ph);
        const bool more = CHUNKS && pc.n > (int)P.search_own;
        const int m1 = min(P.W, pc.m), cols = max(((more ? (int)P.search_own : pc.n) + 63) / 64, 1);
        const int64_t c0 = (int64_t)lane * cols;
        u64 key = wave_min(wave_search(P, pc, m1, min(P.K, m1 - 1), pl, ph, c0, cols), lane);
        if (CHUNKS && more && !tail_last(P, (P.ref_off[pair] - P.ref_off[0]) >> P.search_tail_log, pc.n, 1u, key, lane)) return;
        wave_pair_from_key<STATS>(P, pair, pc, key, lev, lane);
        return;
    }
    const uint64_t x = (pair - P.n_pairs) * 64 + (uint64_t)lane;
    uint64_t of = 0, first = 0;
    int64_t c0 = 0;
    PairCursor pc{0, 0, 0, 0, 0, 0};
    bool have = x < P.search_tails && search_tail(P, x, of, c0, first);
    pl = ph = 0;
    if (have) {
        pc = pair_cursor(P, of);
        have = pc.m > 0;
        if (!have) pc.n = 0;  // nothing to search
        packed_planes(P.reads, (P.read_off[P.n_pairs] + 3) / 4, (int64_t)pc.rb, pl, ph);
    }
    u64 todo = __ballot(have);
    if (todo == 0ull) return;
    const int m1 = min(P.W, pc.m);
    const u64 lane_key = wave_search(P, pc, m1, min(P.K, m1 - 1), pl, ph, c0, 1 << P.search_tail_log);
    while (todo != 0ull) {
        const int at = __builtin_ctzll(todo);
        const uint64_t p = (uint32_t)read_lane((int)of, at);
        const u64 mine = __ballot(have && of == p);
        todo &= ~mine;
        u64 key = wave_min(have && of == p ? lane_key : ~0ull, lane);
        const PairCursor pu = wave_cursor(P, p);
        if (tail_last(P, read_lane64(first, at), pu.n, (uint32_t)__builtin_popcountll(mine), key, lane))
            wave_pair_from_key<STATS>(P, p, pu, key, lev, lane);
    }
}

// How many first pairs of the order take a wavefront each in the window kernel,
// looked for at 64 places at once (the order is by classes of length, so that
// neighbours may be out of order; all wavefronts get the same number).
__device__ __forceinline__ int long_count(const AlignParams& P, int lane) {
    if (P.long_pairs == 0) return 0;
    const int step = (P.long_pairs + 63) / 64, at = lane * step;
    const bool is = at < P.long_pairs && pair_cursor(P, P.order[at]).m > P.long_bases;
    const u64 other = ~__ballot(is);
    return min(other ? __builtin_ctzll(other) * step : P.long_pairs, P.long_pairs);
}

// The window kernel's wavefronts that take a pair each (see k_windows_lane): one
// of the longest pairs of a batch, or (serving) a share of the resident pairs.
template <bool STATS>
__device__ __forceinline__ void windows_long(const AlignParams& P, uint8_t* lev, int at, int n_long, int lane) {
    if (at >= n_long) return;
    const uint64_t pair = P.order[at];
    if (search_outcome(P, pair) < 0) return;  // the same in every lane
#if defined(GENASM_DEBUG)
    if (P.audit && lane == 0) atomicAdd(P.audit + pair, kAuditTake);  // queue audit
#endif
    const int col = uniform((int)P.search[pair].col);
    TurnClock none;
    wave_pair_windows<STATS, false>(P, pair, wave_cursor(P, pair), col, fresh_state(col), lev, lane, none);
}

__device__ __forceinline__ void windows_few(const AlignParams& P, uint8_t* lev, uint32_t n_hot, uint32_t n,
                                            uint32_t first, uint32_t stride, int lane) {
    TurnClock turn;
    turn.open(P);
    for (uint32_t at = first; at < n; at += stride) {
        const uint64_t pair = (uint32_t)uniform((int)(at < n_hot ? P.easy_list[at] : P.hard_list[at - n_hot]));
        const int row = uniform(P.search[pair].row), col = uniform((int)P.search[pair].col);
        const PairState s = P.state[pair];
        PairState st{uniform(s.ti), uniform(s.pj), uniform(s.score), (uint32_t)uniform((int)s.nwin),
                     (uint32_t)uniform((int)s.written), uniform(s.cur_op), (uint32_t)uniform((int)s.cur_len),
                     (uint32_t)uniform((int)s.flags)};
        if (row < 0 || (st.flags & kStateDone)) continue;
        if (!(st.flags & kStateStarted)) st = fresh_state(col);
        wave_pair_windows<false, true>(P, pair, wave_cursor(P, pair), col, st, lev, lane, turn);
    }
}
