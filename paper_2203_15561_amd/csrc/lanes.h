// Kernels that take one pair per lane: the start search and the windows, on
// vertical differences (diff_window.h).
#pragma once

#include "diff_window.h"
#include "filter.h"
#include "wave_pair.h"

static_assert(kLaneCols == kLanePathCommit, "the launch rule and the kernels agree");

// ---------------------------------------------------------------------------
// Windows
// ---------------------------------------------------------------------------

// The run-length CIGAR of a pair: the open run, and the runs already written.
struct RunOut {
    int cur_op;        // -1 before the pair's first op
    uint32_t cur_len, written, room;
    uint32_t* at;      // the pair's elements
    bool overflow;
};

__device__ __forceinline__ void close_run(RunOut& r) {
    if (r.written < r.room) r.at[r.written] = (r.cur_len << 2) | (uint32_t)r.cur_op;
    else r.overflow = true;
    ++r.written;
}

// A run of len > 0 ops; none of len 0. The run it closes goes to device memory.
__device__ __forceinline__ void append_run(RunOut& r, int op, uint32_t len) {
    const bool closes = len != 0u && op != r.cur_op;
    if (closes && r.written < r.room) r.at[r.written] = (r.cur_len << 2) | (uint32_t)r.cur_op;
    r.written += closes ? 1u : 0u;
    r.cur_len = (closes ? 0u : r.cur_len) + len;
    r.cur_op = len != 0u ? op : r.cur_op;
}

// Appends a window's path to the pair's runs, a run of matches and the run of
// edits after it at a time. Within a window a deletion is never next to an
// insertion or before a substitution (the earlier of the two edges in the order
// S, I, D would have been valid a cell before), so the next event in the read
// and the next in the text are never at the same cell.
//
// A wavefront takes as many turns as its lane with the most runs, about 30 with
// unrelated pairs in the batch, and every branch costs it more than the few
// instructions behind it: masks instead (20,000 pairs of 10 kb, 30% of them
// unrelated: 15,800 -> 8,300 cycles a window, where the other wavefront takes
// 12,600).
__device__ __forceinline__ void append_path(u64 ins, u64 sub, u64 del, int j, int i, RunOut& r) {
    constexpr int kDelOrIns = (int)GENASM_OP_MISMATCH;
    static_assert(GENASM_OP_INS == kDelOrIns + 1 && GENASM_OP_DEL == kDelOrIns + 2, "ops in order");
    // a pair's first run joins an empty one of its own op
    if (r.cur_op < 0)
        r.cur_op = del & 1u ? (int)GENASM_OP_DEL : ins & 1u ? (int)GENASM_OP_INS
                   : sub & 1u ? (int)GENASM_OP_MISMATCH : (int)GENASM_OP_MATCH;
    for (int it = 0; it < 2 * kLaneCols + 2 && (i | j) != 0; ++it) {  // i, j: bases left
        const int k = min(ctz64(ins | sub | del), j);
        ins >>= k;
        sub >>= k;
        del >>= k;
        i -= k;
        j -= k;
        append_run(r, (int)GENASM_OP_MATCH, (uint32_t)k);
        // the run of the edit there; one of more than 31 takes another turn
        const int dl = (int)del, nl = (int)ins, sl = (int)sub;
        const int d = -(dl & 1), n = -(nl & 1);
        const int edits = (d & dl) | (~d & ((n & nl) | (~n & sl & ~dl)));
        const int run = __builtin_ctz((unsigned)~edits | 0x80000000u);
        const int dj = run & ~d, di = run & ~n;
        ins >>= dj;
        sub >>= dj;
        del >>= di;
        j -= dj;
        i -= di;
        append_run(r, kDelOrIns - n - 2 * d, (uint32_t)run);
    }
    r.overflow = r.overflow || r.written > r.room;
}

// A window handed from the wavefront that computes it to the one that writes
// its CIGAR: its path, and i_end, j_end << 8 and kMail* bits.
constexpr uint32_t kMailWindow = 1u << 16;    // the lane computed a window
constexpr uint32_t kMailFailed = 1u << 17;    // it has no solution within K (no path)
constexpr uint32_t kMailInternal = 1u << 18;  // it committed nothing (never expected)
constexpr uint32_t kMailEnd = 1u << 19;       // the pair's last window
constexpr uint32_t kMailPark = 1u << 20;      // serving: the pair's turn ends
constexpr uint32_t kMailHot = 1u << 21;       // serving: it advanced one window only
// Everything is kept twice, a window's fields by the parity of the window and a
// pair's by that of its round of pairs: the writer reads a copy before it comes to
// its next barrier, so a copy may be filled again once another barrier has passed.
// A round can be one window long, with one barrier in all, and the next round's
// fields are filled before there is another.
struct LaneMail {
    u64 ins[2][64], sub[2][64], del[2][64];
    uint32_t info[2][64];
    uint32_t more[2];
    int32_t col[2][64];   // the pair's start column, -1: no window work
    uint32_t pair[2][64];
    int32_t ti[2][64];    // its text cursor and window count when the launch took it up
    uint32_t nwin[2][64];
};

// Workgroup barrier for what is handed over in LDS. The wavefronts share nothing
// in device memory, so their loads and stores there stay in flight across it
// (a __syncthreads would wait for the next window's words).
__device__ __forceinline__ void mail_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#else
    __syncthreads();
#endif
}

// A lane's pairs: lane l of the b-th workgroup of lanes takes list position
// b * lanes + l, then every (their number) * lanes further on. Serving: the
// resident pairs, those that advanced least first; otherwise all pairs, longest
// reads first if ordered, from the first that doesn't take a wavefront on.
struct LaneShare {
    uint64_t n, stride, first;
    uint32_t n_hot;
    int lanes, n_long, long_blocks;
};
template <bool SERVE>
__device__ __forceinline__ LaneShare lane_share(const AlignParams& P, int lane) {
    LaneShare s;
    s.n_hot = 0;
    s.n_long = s.long_blocks = 0;
    if constexpr (SERVE) {
        s.n_hot = __hip_atomic_load(P.counters + kCounterEasyLen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s.n = s.n_hot + (uint64_t)__hip_atomic_load(P.counters + kCounterHardLen, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        // spread over the whole grid
        s.lanes = (int)max((uint64_t)1, min((uint64_t)64, (s.n + gridDim.x - 1) / gridDim.x));
    } else {
        s.n = P.n_pairs;
        s.lanes = P.pair_lanes;
        s.n_long = long_count(P, lane);
        s.long_blocks = (s.n_long + 1) / 2;
        s.stride = (uint64_t)((int)gridDim.x - s.long_blocks) * s.lanes;
        s.first = (uint64_t)s.n_long + (uint64_t)((int)blockIdx.x - s.long_blocks) * s.lanes;
        return s;
    }
    s.stride = (uint64_t)gridDim.x * s.lanes;
    s.first = (uint64_t)blockIdx.x * s.lanes;
    return s;
}

// A lane's place in the bit planes of a sequence: the words of its window and
// the word after them, which the next window may need. That word is loaded by
// every lane for every window, wanted or not: a load under a condition ends in
// moves that wait for it (two waits a window; without them 20,000 pairs of 10
// kb take 1.60 ms instead of 1.67, 50,000 uneven ones 3.47 instead of 3.69).
// Words up to q + 2 exist for any place in a sequence, and for q = 0.
struct LaneSeq {
    u64 lo0, lo1, lo2, hi0, hi1, hi2;
    uint64_t q;
};
__device__ __forceinline__ void lane_seq_ahead(LaneSeq& c, const u64* lo, const u64* hi) {
    c.lo2 = lo[c.q + 2];
    c.hi2 = hi[c.q + 2];
}
__device__ __forceinline__ void lane_seq_open(LaneSeq& c, const u64* lo, const u64* hi, uint64_t bit) {
    c.q = bit >> 6;
    c.lo0 = lo[c.q];
    c.lo1 = lo[c.q + 1];
    c.hi0 = hi[c.q];
    c.hi1 = hi[c.q + 1];
    lane_seq_ahead(c, lo, hi);
}
// To the window at `bit`, at most one word on.
__device__ __forceinline__ void lane_seq_move(LaneSeq& c, const u64* lo, const u64* hi, uint64_t bit) {
    const bool on = (bit >> 6) != c.q;
    c.lo0 = on ? c.lo1 : c.lo0;
    c.lo1 = on ? c.lo2 : c.lo1;
    c.hi0 = on ? c.hi1 : c.hi0;
    c.hi1 = on ? c.hi2 : c.hi1;
    c.q += on ? 1 : 0;
#if defined(__HIP_DEVICE_COMPILE__)
    // the old words are done with before the loads, which can then take their
    // registers (or moves at the loop's end would wait again)
    asm volatile("" : "+v"(c.lo1), "+v"(c.hi1) : : "memory");
#endif
    lane_seq_ahead(c, lo, hi);
}
__device__ __forceinline__ void lane_seq_window(const LaneSeq& c, uint64_t bit, u64& wlo, u64& whi) {
    wlo = funnel64(c.lo0, c.lo1, (int)(bit & 63));
    whi = funnel64(c.hi0, c.hi1, (int)(bit & 63));
}

// The wavefront that computes the windows.
template <bool STATS, bool SERVE>
__device__ __forceinline__ void windows_compute(const AlignParams& P, const LaneShare& share, LaneMail& mail,
                                                int lane) {
    const uint64_t rorg = P.planes_from_off0 ? (P.read_off[0] & ~63ull) : 0;
    const uint64_t forg = P.planes_from_off0 ? (P.ref_off[0] & ~63ull) : 0;
    TurnClock turn;
    if constexpr (SERVE) turn.open(P);
    int buf = 0, round = 0;  // parities
    for (uint64_t first = share.first; first < share.n; first += share.stride, round ^= 1) {
        const uint64_t at = first + lane;
        bool have = lane < share.lanes && at < share.n;
        uint64_t pair = 0;
        PairState st = fresh_state(0);
        int col = -1;
        if (have) {
            if constexpr (SERVE) {
                pair = at < share.n_hot ? P.easy_list[at] : P.hard_list[at - share.n_hot];
                const SearchOut so = P.search[pair];
                st = P.state[pair];
                have = so.row >= 0 && !(st.flags & kStateDone);
                if (have) {
                    col = (int)so.col;
                    if (!(st.flags & kStateStarted)) st = fresh_state(col);
                }
            } else {
                pair = P.order ? P.order[at] : at;
                have = search_outcome(P, pair) >= 0;
                if (have) {
                    col = (int)P.search[pair].col;
                    st = fresh_state(col);
                }
            }
        }
        mail.col[round][lane] = col;
        mail.pair[round][lane] = (uint32_t)pair;
        mail.ti[round][lane] = st.ti;
        mail.nwin[round][lane] = st.nwin;
        PairCursor pc{0, 0, 0, 0, 0, 0};
        uint64_t rb = 0, fb = 0;  // the places of the lane's window in the planes
        uint32_t max_windows = 0, done_here = 0;
        if (have) {
#if defined(GENASM_DEBUG)
            if (P.audit) atomicAdd(P.audit + pair, kAuditTake);  // queue audit
#endif
            pc = pair_cursor(P, pair);
            max_windows = (uint32_t)pc.m + (uint32_t)pc.n + 1u;
            rb = pc.rb - rorg + st.pj;
            fb = pc.fb - forg + st.ti;
        }
        LaneSeq rc, fc;
        lane_seq_open(rc, P.read_lo, P.read_hi, rb);
        lane_seq_open(fc, P.ref_lo, P.ref_hi, fb);
        u64 st_wops = 0, st_cells = 0, st_table = 0, st_tb = 0, st_steps = 0, cyc_dc = 0;
        u64 cyc_start = 0, wall_start = 0;
        if constexpr (STATS) {
            cyc_start = clock64();
            wall_start = wall_clock64();
        }
        bool any = true;
        while (any) {
            const int mw = have ? min(P.W, pc.m - st.pj) : 64;
            const int nw = have ? min(P.W, pc.n - st.ti) : 64;
            u64 cyc0 = 0;
            if constexpr (STATS) cyc0 = clock64();
            u64 pl, ph, tl, th;
            lane_seq_window(rc, rb, pl, ph);
            lane_seq_window(fc, fb, tl, th);
            // Past the text only insertions are left, which needs no table: an
            // unrelated pair spends up to half its windows there, and the steps
            // for short windows cost all 64 lanes a seventh more (20,000 pairs of
            // 10 kb, 30% unrelated: 14,600 -> 13,100 cycles a window).
            const bool spent = nw == 0;
            const bool ragged = __ballot(!spent && (mw < 64 || nw < 64)) != 0ull;
            WindowPath w = ragged ? window_path<true>(pl, ph, tl, th, mw, nw, P.L)
                                  : window_path<false>(pl, ph, tl, th, mw, nw, P.L);
            if (spent) {
                w.j_end = min(mw, P.L);
                w.ins = ~0ull >> (64 - w.j_end);
                w.sub = w.del = 0ull;
                w.i_end = 0;
                w.dist = mw;
            }
            bool over = false;
            if constexpr (SERVE) over = turn.active && turn.over();
            uint32_t info = 0u;
            if (have) {
                if constexpr (STATS) st_cells += (u64)mw * nw;
                info = kMailWindow | (uint32_t)w.i_end | ((uint32_t)w.j_end << 8);
                ++st.nwin;
                ++done_here;
                // every window commits at least one base, so a pair has at most m + n
                if (st.nwin > max_windows || w.i_end + w.j_end == 0) info |= kMailInternal | kMailFailed;
                else if (w.dist > P.K) info |= kMailFailed;
                if (info & kMailFailed) {
                    info |= kMailEnd;
                } else {
                    st.ti += w.i_end;
                    st.pj += w.j_end;
                    if (st.pj >= pc.m) {
                        info |= kMailEnd;
                    } else {
                        rb += (uint64_t)w.j_end;
                        fb += (uint64_t)w.i_end;
                    }
                    if constexpr (STATS) {
                        st_wops += (u64)nw * (2 + 6 * w.dist);
                        st_table += (u64)(w.dist + 1) * (min(nw, P.L) + 1);
                        st_tb += 2u * (__builtin_popcountll(w.ins) + __builtin_popcountll(w.sub) +
                                       __builtin_popcountll(w.del));
                        st_steps += (u64)nw;
                        cyc_dc += clock64() - cyc0;
                    }
                }
                if constexpr (SERVE) {
                    // every pair advances at least one window per launch; none starts
                    // once its turn has ended
                    if (!(info & kMailEnd) &&
                        (over || (P.window_budget != 0u && done_here >= P.window_budget)))
                        info |= kMailPark | (done_here <= 1u ? kMailHot : 0u);
                    if (info & (kMailEnd | kMailPark)) {
                        PairState* ps = P.state + pair;
                        ps->ti = st.ti;
                        ps->pj = st.pj;
                        ps->nwin = st.nwin;
                    }
                }
                if (info & (kMailEnd | kMailPark)) {
                    have = false;
                    if constexpr (STATS) {
                        u64* stp = P.stats + pair * kStatCount;
                        stp[kStatWindowWordOps] += st_wops;
                        stp[kStatWindowCells] += st_cells;
                        stp[kStatTableWords] += st_table;
                        stp[kStatTbReads] += st_tb;
                        stp[kStatWindowLaneSteps] += st_steps;
                        stp[kStatWindows] += done_here;
                        stp[kStatDcCycles] += cyc_dc;
                        stp[kStatPairCycles] += clock64() - cyc_start;
                        if (!stp[kStatPairStart]) stp[kStatPairStart] = wall_start;
                        stp[kStatPairEnd] = wall_clock64();
                    }
                }
            }
            lane_seq_move(rc, P.read_lo, P.read_hi, rb);
            lane_seq_move(fc, P.ref_lo, P.ref_hi, fb);
            mail.ins[buf][lane] = w.ins;
            mail.sub[buf][lane] = w.sub;
            mail.del[buf][lane] = w.del;
            mail.info[buf][lane] = info;
            any = __ballot(have) != 0ull;
            if (lane == 0) mail.more[buf] = any ? 1u : 0u;
            buf ^= 1;
            mail_barrier();
        }
    }
}

// The wavefront that writes the CIGARs and results, a window behind the other.
template <bool STATS, bool SERVE>
__device__ __forceinline__ void windows_write(const AlignParams& P, const LaneShare& share, const LaneMail& mail,
                                              int lane) {
    int buf = 0, round = 0;
    for (uint64_t first = share.first; first < share.n; first += share.stride, round ^= 1) {
        bool more = true, opened = false;
        uint64_t pair = 0, base = 0;
        PairState st = fresh_state(0);
        RunOut run{-1, 0u, 0u, 0u, nullptr, false};
        int col = -1;
        u64 cyc_tb = 0;
        while (more) {
            mail_barrier();
            if (!opened) {
                opened = true;
                col = mail.col[round][lane];
                pair = mail.pair[round][lane];
                if (col >= 0) {
                    const PairCursor pc = pair_cursor(P, pair);
                    base = pair_run_base(P, pair);
                    const uint64_t limit = min(P.cigar_cap, base + (uint64_t)pc.m + (uint64_t)pc.n);
                    st = fresh_state(col);
                    if constexpr (SERVE) {
                        // ti, pj and nwin are the other wavefront's to read and write
                        const PairState* ps = P.state + pair;
                        if (ps->flags & kStateStarted) {
                            st.score = ps->score;
                            st.written = ps->written;
                            st.cur_op = ps->cur_op;
                            st.cur_len = ps->cur_len;
                            st.flags = ps->flags;
                        }
                    }
                    st.ti = mail.ti[round][lane];
                    st.nwin = mail.nwin[round][lane];
                    run = RunOut{st.cur_op, st.cur_len, st.written,
                                 (uint32_t)(limit > base ? limit - base : 0ull), P.cigar + base,
                                 (st.flags & kStateOverflow) != 0};
                }
            }
            more = mail.more[buf] != 0u;
            const uint32_t info = mail.info[buf][lane];
            const u64 cyc0 = STATS ? clock64() : 0ull;
            if (info & kMailWindow) {
                if (!(info & kMailFailed)) {
                    const u64 ins = mail.ins[buf][lane], sub = mail.sub[buf][lane], del = mail.del[buf][lane];
                    st.score += __builtin_popcountll(ins) + __builtin_popcountll(sub) +
                                __builtin_popcountll(del);
                    append_path(ins, sub, del, (int)((info >> 8) & 0xFFu), (int)(info & 0xFFu), run);
                    st.ti += (int)(info & 0xFFu);
                }
                ++st.nwin;
                if constexpr (STATS) cyc_tb += clock64() - cyc0;
                const bool failed = (info & kMailFailed) != 0u;
                if (info & kMailEnd) {
                    if (!failed && run.cur_op >= 0) close_run(run);
                    genasm_result r;
                    r.edit_distance = failed ? -1 : st.score;
                    r.ref_begin = failed ? 0u : (uint32_t)col;
                    r.ref_end = failed ? 0u : (uint32_t)st.ti;
                    r.cigar_len = failed || run.overflow ? 0u : run.written;
                    r.n_windows = st.nwin;
                    r.cigar_off = base;
                    r.flags = (run.overflow && !failed ? GENASM_FLAG_CIGAR_OVERFLOW : 0u) |
                              (info & kMailInternal ? GENASM_FLAG_INTERNAL : 0u);
                    P.out[pair] = r;
                    if constexpr (STATS) P.stats[pair * kStatCount + kStatTbCycles] += cyc_tb;
                }
                if constexpr (SERVE) {
                    if (info & (kMailEnd | kMailPark)) {
                        PairState* ps = P.state + pair;
                        ps->score = st.score;
                        ps->written = run.written;
                        ps->cur_op = run.cur_op;
                        ps->cur_len = run.cur_len;
                        ps->flags = st.flags | (run.overflow ? kStateOverflow : 0u) |
                                    (failed ? kStateFailed : 0u) |
                                    (info & kMailInternal ? kStateInternal : 0u) |
                                    (info & kMailEnd ? kStateDone : 0u);
                    }
                }
            }
            if constexpr (SERVE) {
                // the finished list, or the pair's list for the next iteration
                const bool fin = (info & kMailEnd) != 0u;
                const bool hot = (info & kMailPark) && (info & kMailHot);
                const bool cold = (info & kMailPark) && !(info & kMailHot);
                if (P.fin_list && __ballot(fin || hot || cold) != 0ull) {
                    const uint32_t pf = wave_append(P.fin_len, fin);
                    if (fin) P.fin_list[pf] = (uint32_t)pair;
                    const uint32_t p1 = wave_append(P.next_len + kCounterEasyLen, hot);
                    if (hot) P.next_hot[p1] = (uint32_t)pair;
                    const uint32_t p2 = wave_append(P.next_len + kCounterHardLen, cold);
                    if (cold) P.next_cold[p2] = (uint32_t)pair;
                }
            }
            buf ^= 1;
        }
    }
}

// A workgroup's LDS: the mail and its roles, or the levels of its two wavefronts.
constexpr int kLaneLdsBytes = 2 * kWaveLdsBytes;
constexpr int kRolesAt = kLaneLdsBytes / 4 - 4;  // words: two SIMDs, the role, the claim
static_assert(sizeof(LaneMail) <= 4 * kRolesAt, "layout");

// Which wavefront of a workgroup computes, where three or four workgroups share a
// compute unit: the SIMDs that its wavefronts get depend on what ran there before,
// and two computing wavefronts on one SIMD take longer than one of each. A word per
// compute unit counts the roles on its SIMDs (a byte each: computing, and writing
// from bit 4 on); a workgroup claims the better of its two ways round. The words
// steer only: whatever they hold, a workgroup has one wavefront of each kind.
__device__ __forceinline__ uint32_t* cu_word(const AlignParams& P, uint32_t& simd) {
#if defined(__HIP_DEVICE_COMPILE__)
    // HW_ID: SIMD in bits 4..5, compute unit and shader engine in 8..15; XCC_ID
    const uint32_t id = __builtin_amdgcn_s_getreg(4 | 31 << 11), xcd = __builtin_amdgcn_s_getreg(20 | 31 << 11);
#else
    const uint32_t id = ((blockIdx.x + (threadIdx.x >> 6)) & 3u) << 4, xcd = 0u;
#endif
    simd = (id >> 4) & 3u;
    return P.cu_roles + (((id >> 8) & 0xFFu) | (xcd & 15u) << 8);
}
__device__ __forceinline__ int claim_roles(const AlignParams& P, uint32_t* roles, int wave, int lane) {
    uint32_t simd;
    uint32_t* word = cu_word(P, simd);
    if (lane == 0) roles[wave] = simd;
    mail_barrier();
    if (wave == 0 && lane == 0) {
        const uint32_t a = 8u * roles[0], b = 8u * roles[1];
        const uint32_t first = (1u << a) + (16u << b), second = (1u << b) + (16u << a);
        const uint32_t old = atomicAdd(word, first);
        // two computing wavefronts on a SIMD are the worst, two writing ones leave a
        // later workgroup no better place
        auto load = [&](uint32_t compute, uint32_t write) {
            const uint32_t c = old >> compute, w = old >> write;
            return 4u * (c & 15u) + ((c >> 4) & 15u) + (w & 15u) + 2u * ((w >> 4) & 15u);
        };
        const bool turned = load(b, a) < load(a, b);
        if (turned) atomicAdd(word, second - first);
        roles[2] = turned ? 1u : 0u;
        roles[3] = turned ? second : first;
    }
    mail_barrier();
    return uniform((int)roles[2]);
}
__device__ __forceinline__ void release_roles(const AlignParams& P, const uint32_t* roles, int lane) {
    uint32_t simd;
    uint32_t* word = cu_word(P, simd);
    if (lane == 0) atomicAdd(word, 0u - roles[3]);
}

// Window kernel, two wavefronts per workgroup and one pair per lane of them:
// one computes the windows, the other turns each window's path into CIGAR runs
// while the next window is computed.
//
// A lane's window takes 5.2 us (12,600 cycles: about 2,500 instructions, of which
// one wavefront of a SIMD issues one per 4.5 cycles, so their number bounds it)
// and a batch as long as its longest pair. The first workgroups
// therefore take the longest pairs a wavefront each, if the lengths are uneven
// (wave_pair.h: 1.7 us a window); so do all workgroups of a serving iteration with
// no more resident pairs than wavefronts (eight times as many with small windows).
//
// ALONE: a wavefront takes more than half of a SIMD's registers, so that no two
// share one. Where a compute unit's next workgroup starts is not fixed (most often on
// a free pair of SIMDs or with the last one's second, now and then with its first),
// and a computing wavefront that shares its SIMD takes 1.7 times as long, and the
// batch with it (30,000 pairs of 10 kb: windows 1.37 ms, 2.35 when the roles went by
// the workgroup's number and one unit in a hundred had two of them on a SIMD).
template <bool STATS, bool SERVE, bool ALONE>
__global__ __launch_bounds__(128, ALONE ? 1 : 2) void k_windows_lane(AlignParams P) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (ALONE) asm volatile("" : : : "a127");
#endif
    extern __shared__ u64 smem[];
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
    uint8_t* lev = reinterpret_cast<uint8_t*>(smem) + wave * kWaveLdsBytes;
    const LaneShare share = lane_share<SERVE>(P, lane);
    if constexpr (SERVE) {
        // small windows: several pairs a wavefront one after the other (5,000 mixed
        // requests, W 8, O 7: 5.6 ms against 10.6 on lanes and 10.8 on the row tables)
        if (share.n <= (P.W <= 8 ? 16ull : 2ull) * gridDim.x) {
            windows_few(P, lev, share.n_hot, (uint32_t)share.n, (uint32_t)blockIdx.x + (uint32_t)wave * gridDim.x,
                        2u * gridDim.x, lane);
            return;
        }
    } else if ((int)blockIdx.x < share.long_blocks) {
        windows_long<STATS>(P, lev, (int)blockIdx.x * 2 + wave, share.n_long, lane);
        return;
    }
    LaneMail& mail = *reinterpret_cast<LaneMail*>(smem);
    const bool claim = !SERVE && !ALONE && P.cu_roles && share.first < share.n;
    uint32_t* roles = reinterpret_cast<uint32_t*>(smem) + kRolesAt;
    const int computes = claim ? claim_roles(P, roles, wave, lane) : 0;
    if (wave == computes) windows_compute<STATS, SERVE>(P, share, mail, lane);
    else windows_write<STATS, SERVE>(P, share, mail, lane);
    if (claim && wave == computes) release_roles(P, roles, lane);
}

// ---------------------------------------------------------------------------
// Start search
// ---------------------------------------------------------------------------

// Lane t searches part t mod `parts` of pair t / parts (parts a power of two):
// `cols` output columns (a multiple of 64) from part * cols on, in blocks of 64
// columns from the right. E over the first read window's m1 bases at a column
// within m1 + m1 columns of the text end depends on no column further right
// (an alignment of at most m1 edits reaches at most 2 m1 text bases), so a part
// starts 128 columns past its last output column. Columns it computes past its
// own are never below their true value, so they need no check; columns past
// the reference match nothing and stay at m1, which is no hit. The pair's key
// (row << 32 | column) is the least over its parts: least row, then leftmost
// column.
template <bool RAGGED>
__device__ __forceinline__ uint32_t search_block(DiffColumn& c, int& score, u64 a, u64 b, u64 pad,
                                                 const TextBlock& text) {
    uint32_t best = ~0u;
#pragma unroll
    for (int i = 63; i >= 0; --i) {
        u64 out;
        const u64 Eq = equal_rows<RAGGED>(a, b, pad, text, i, out);
        u64 D0, Ph, Mh;
        diff_step(c, Eq, D0, Ph, Mh);
        score += (int)((uint32_t)(Ph >> 32) >> 31) + ((int32_t)(uint32_t)(Mh >> 32) >> 31);
        best = min(best, ((uint32_t)score << 6) + (uint32_t)i);
    }
    return best;
}

// Searches output columns [c0, c0 + cols) of a pair (lanes without `have`: none)
// and combines its least key. All lanes of the wavefront call this together.
__device__ __forceinline__ void search_part(const AlignParams& P, bool have, uint64_t pair, const PairCursor& pc,
                                            int c0, uint64_t cols) {
    const int m1 = min(P.W, pc.m);
    const int e = (int)min((uint64_t)pc.n, (uint64_t)c0 + cols + 128);
    int nb = have ? (e - c0 + 63) / 64 : 0;
    const uint64_t rorg = P.planes_from_off0 ? (P.read_off[0] & ~63ull) : 0;
    const uint64_t forg = P.planes_from_off0 ? (P.ref_off[0] & ~63ull) : 0;
    u64 a = 0, b = 0, pad = 0;
    u64 lo1 = 0, hi1 = 0, lo0 = 0, hi0 = 0;  // words q + 1 and q of the block's text
    const uint64_t bit0 = pc.fb - forg + (uint64_t)c0;
    const int sh = (int)(bit0 & 63);
    uint64_t q = (bit0 >> 6) + (uint64_t)(nb > 0 ? nb - 1 : 0);
    if (have) {
        SeqCursor rc;
        u64 pl, ph;
        seq_open(rc, P.read_lo, P.read_hi, pc.rb - rorg);
        seq_window(rc, P.read_lo, P.read_hi, pc.rb - rorg, pl, ph);
        a = __builtin_bitreverse64(pl);
        b = __builtin_bitreverse64(ph);
        pad = m1 < 64 ? (1ull << (64 - m1)) - 1 : 0ull;
        lo1 = P.ref_lo[q + 1];
        hi1 = P.ref_hi[q + 1];
        lo0 = P.ref_lo[q];
        hi0 = P.ref_hi[q];
    }
    DiffColumn c{~pad, 0ull};
    int score = m1;
    u64 key = ~0ull;
    bool active = have;
    while (__ballot(active) != 0ull) {
        const u64 tl = funnel64(lo0, lo1, sh), th = funnel64(hi0, hi1, sh);
        lo1 = lo0;
        hi1 = hi0;
        const int col = c0 + 64 * (nb - 1);
        if (active && nb > 1) {  // the next block's words
            --q;
            lo0 = P.ref_lo[q];
            hi0 = P.ref_hi[q];
        }
        const int left = e - col;  // valid columns of the block
        const u64 past = left < 64 ? ~0ull << max(left, 0) : 0ull;
        const bool ragged = __ballot(active && (left < 64 || m1 < 64)) != 0ull;
        const uint32_t k = ragged ? search_block<true>(c, score, a, b, pad, text_block(tl, th, past))
                                  : search_block<false>(c, score, a, b, 0ull, text_block(tl, th, 0ull));
        if (active) {
            const u64 cand = ((u64)(k >> 6) << 32) | (u64)(uint32_t)(col + (int)(k & 63u));
            key = min(key, cand);
            --nb;
            active = nb > 0;
        }
    }
    if (!have) return;
    if ((int)(key >> 32) <= min(P.K, m1 - 1)) atomicMin(P.search_key + pair, key);
    if (P.stats) atomicAdd(P.stats + pair * kStatCount + kStatSearchLaneSteps, (u64)(e - c0));
}

__host__ __device__ __forceinline__ uint64_t search_part_blocks(const AlignParams& P) {
    return ((P.n_pairs << P.search_parts_log) + 63) / 64;
}

__global__ __launch_bounds__(64) void k_search_lane(AlignParams P) {
    uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool have;
    uint64_t pair = 0, cols = 1ull << P.search_tail_log;
    int64_t c0 = 0;
    PairCursor pc{0, 0, 0, 0, 0, 0};
    if (blockIdx.x < search_part_blocks(P)) {
        const uint64_t at = t >> P.search_parts_log;
        const uint32_t part = (uint32_t)(t & ((1ull << P.search_parts_log) - 1));
        have = at < P.n_pairs;
        if (have) {
            pair = P.order ? P.order[at] : at;
            pc = pair_cursor(P, pair);
            const uint64_t per = (((uint64_t)pc.n + (1ull << P.search_parts_log) - 1) >> P.search_parts_log);
            cols = min(max((uint64_t)64, (per + 63) & ~63ull), (uint64_t)P.search_part_cols);
            c0 = (int64_t)(part * cols);
        }
    } else {
        t -= search_part_blocks(P) * 64;
        uint64_t first;
        have = t < P.search_tails && search_tail(P, t, pair, c0, first);
        if (have) pc = pair_cursor(P, pair);
    }
    have = have && pc.m > 0 && c0 < (int64_t)pc.n;
    search_part(P, have, pair, pc, have ? (int)c0 : 0, cols);
}

// Serving: the items of k_search_items (pair << 24 | chunk), one per lane.
__global__ __launch_bounds__(64) void k_search_lane_items(AlignParams P) {
    const uint32_t n_items = __hip_atomic_load(P.counters + kCounterListBase, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
    for (uint64_t first = (uint64_t)blockIdx.x * 64; first < n_items; first += (uint64_t)gridDim.x * 64) {
        const uint64_t at = first + threadIdx.x;
        bool have = at < n_items;
        uint64_t pair = 0;
        int c0 = 0;
        PairCursor pc{0, 0, 0, 0, 0, 0};
        if (have) {
            const uint64_t it = P.items_in[at];
            pair = it >> 24;
            c0 = (int)((uint32_t)(it & 0xffffffull) * P.search_chunk);
            pc = pair_cursor(P, pair);
            have = c0 < pc.n;
        }
        search_part(P, have, pair, pc, c0, P.search_chunk);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

__global__ void k_lane_prep(const uint8_t* reads, const uint64_t* d_read, uint64_t n_read, u64* rlo,
                            u64* rhi, uint64_t rw, const uint8_t* refs, const uint64_t* d_ref,
                            uint64_t n_ref, u64* flo, u64* fhi, uint64_t fw, u64* key, uint64_t n_pairs,
                            uint32_t* cu_roles) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_pairs) key[t] = ~0ull;
    if (cu_roles && t < kCuRoles) cu_roles[t] = 0u;
    const bool rd = t < rw;
    const uint64_t w = rd ? t : t - rw;
    if (!rd && w >= fw) return;
    const uint64_t b0 = rd ? d_read[0] : d_ref[0];
    u64 x, y;
    plane_word(rd ? reads : refs, (b0 + (rd ? n_read : n_ref) + 3) / 4, (b0 >> 6) + w, x, y);
    (rd ? rlo : flo)[w] = x;
    (rd ? rhi : fhi)[w] = y;
}
