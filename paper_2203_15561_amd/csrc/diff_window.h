// A window's distance and traceback on vertical differences, in one lane.
//
// The window's dynamic program. E(i, j) is the least number of edits that
// aligns the read window's bases from j on to a prefix of the text window's
// bases from i on (E(i, mw) = 0, E(nw, j) = mw - j); bit p of GenASM's R[d][i]
// is 0 exactly when E(i, mw-1-p) <= d, so E holds all its rows at once: d* is
// E(0, 0), and a traceback that stands at a cell with d = E(i, j) edits left
// (it starts so, and every edge it takes keeps it so) finds the first valid
// edge in the order match, substitution, insertion, deletion as
//   match         the two bases agree,
//   substitution  E(i+1, j+1) = E(i, j) - 1,
//   insertion     E(i, j+1)   = E(i, j) - 1,
//   deletion      otherwise (some edge is valid at every cell).
// E's neighbours differ by at most one, so a column is two bit vectors, the
// rows where it grows (Pv) and falls (Mv) along the read, and a column step is
// the published bit-vector recurrence for approximate matching (Myers, A fast
// bit-vector algorithm for approximate string matching based on dynamic
// programming, 1999, in Hyyro's form with the diagonal-zero vector D0, 2003).
// A step costs about 25 32-bit instructions whatever d* is, where 64-bit rows
// cost 12 per row and column, and the traceback needs two bits per cell
// whatever d* is, where the rows need one word per row and column: the 40
// columns a window commits stay in registers, with no LDS table and no spill.
//
// Bit order. In a column, bit 63 - j stands for read base j (so the recurrence
// carries from the read window's end towards its start, and a short window's
// unused low bits act as rows of value 0). The traceback's words are the same
// bits reversed, bit j for read base j.
#pragma once

// Text columns a window keeps for its traceback (it commits at most W - O of
// either sequence); the traceback's words hold 32 + 8 read bases.
constexpr int kLaneCols = 40;

// All ones when bit b of w is set, else 0 (b a constant once unrolled).
__device__ __forceinline__ uint32_t bit_mask(uint32_t w, int b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_sbfe((int)w, b, 1);
#else
    return (uint32_t)((int32_t)(w << (31 - b)) >> 31);
#endif
}

__device__ __forceinline__ u64 both(uint32_t m) { return ((u64)m << 32) | m; }

// Any three-input bitwise function, one v_bitop3_b32 per half (the compiler
// makes two instructions or a half-rate v_bfi_b32 of most of them). T is the
// function applied to the bytes kA, kB, kC.
constexpr uint32_t kA = 0xF0, kB = 0xCC, kC = 0xAA;
template <uint32_t T>
__device__ __forceinline__ uint32_t bit_op(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, T & 0xFF);
#else
    uint32_t r = 0;
    for (int k = 0; k < 8; ++k)
        if ((T >> k) & 1u) r |= ((k & 4) ? a : ~a) & ((k & 2) ? b : ~b) & ((k & 1) ? c : ~c);
    return r;
#endif
}
template <uint32_t T>
__device__ __forceinline__ u64 bit_op(u64 a, u64 b, u64 c) {
    const uint32_t lo = bit_op<T>((uint32_t)a, (uint32_t)b, (uint32_t)c);
    const uint32_t hi = bit_op<T>((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32));
    return ((u64)hi << 32) | lo;
}

// x << 1 in one instruction (the compiler's two-instruction form issues slower).
__device__ __forceinline__ u64 shl1(u64 x) {
#if defined(__HIP_DEVICE_COMPILE__)
    u64 r;
    asm("v_lshlrev_b64 %0, 1, %1" : "=v"(r) : "v"(x));
    return r;
#else
    return x << 1;
#endif
}

// Keeps the scheduler from moving instructions across: over a whole window's
// straight-line code it would hoist what does not depend on the recurrence and
// take more registers than a wavefront has.
__device__ __forceinline__ void sched_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}

__device__ __forceinline__ uint32_t reverse32(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_bitreverse32(x);
#else
    return (uint32_t)(__builtin_bitreverse64((u64)x) >> 32);
#endif
}

// Has x computed here: the compiler would sink the traceback's words into the
// traceback's blocks and keep all the words they are made of until then.
__device__ __forceinline__ uint32_t here(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
    return x;
}

// One column of vertical differences.
struct DiffColumn {
    u64 Pv, Mv;
};

// Steps to the next text column, whose base equals the read's at the set bits
// of Eq. D0: the rows whose value equals the diagonal neighbour's in the column
// before; Ph, Mh: the rows whose value grew or fell against that column.
__device__ __forceinline__ void diff_step(DiffColumn& c, u64 Eq, u64& D0, u64& Ph, u64& Mh) {
    const u64 sum = (Eq & c.Pv) + c.Pv;
    D0 = bit_op<(kA ^ kB) | kC>(sum, c.Pv, Eq | c.Mv);
    Ph = bit_op<kA | ~(kB | kC)>(c.Mv, D0, c.Pv);
    Mh = c.Pv & D0;
    const u64 Ps = shl1(Ph), Ms = shl1(Mh);  // row 0 is 0 in every column: nothing shifts in
    c.Pv = bit_op<kA | ~(kB | kC)>(Ms, D0, Ps);
    c.Mv = Ps & D0;
}

// One window's alignment: bit j of `ins` / `sub` for a read base that is
// inserted / substituted, bit i of `del` for a deleted text base, every other
// base up to (i_end, j_end) matched.
struct WindowPath {
    u64 ins, sub, del;
    int i_end, j_end, dist;
};

// The path's state between text columns: `cur` has the bit of the read base it
// stands at (0 once it has left the read bases the window may commit).
struct PathWalk {
    u64 cur, ins, sub;
    uint32_t stay[2];  // columns that didn't move it, the latest in bit 0: 0..31 and 32..39
};

// bits << 1, and a set bit 0 if x is 0; x has at most one bit. Two instructions
// (its halves' sum less one has its top bit set for 0 only; then a funnel shift)
// that pass nothing through a condition register: a vector instruction may read one
// that another wrote only two wait states later. The sum is spelt out: with the
// compiler's own, a serving burst of 1,024 mixed requests, which runs none of it,
// took 2.7% longer (3908 -> 4017 us), other scalar registers being spilled in its
// loops.
__device__ __forceinline__ uint32_t shift_in_zero(uint32_t bits, u64 x) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t less_one;
    asm("v_add3_u32 %0, %1, %2, -1" : "=v"(less_one) : "v"((uint32_t)x), "v"((uint32_t)(x >> 32)));
    return __builtin_amdgcn_alignbit(bits, less_one, 31);
#else
    return (bits << 1) | (((uint32_t)x + (uint32_t)(x >> 32) - 1u) >> 31);
#endif
}

// One text column of the traceback: adding the position to the insertion cells
// carries it over a run of them to the next other cell; a match or substitution
// moves it on by one (it is added to itself), a deletion leaves it.
template <int i>
__device__ __forceinline__ void path_step(PathWalk& w, u64 U, u64 V, u64 live) {
    const u64 I = U & V;
    const u64 sum = I + w.cur;
    const u64 at = bit_op<kA & ~kB & kC>(sum, I, live);
    w.ins = bit_op<kA | (kB & ~kC)>(w.ins, I, sum);
    w.sub = bit_op<kA | (kB & kC)>(w.sub, at, U);
    const u64 move = at & ~V;
    w.stay[i / 32] = shift_in_zero(w.stay[i / 32], move);
    w.cur = at + move;
}

// The traceback's bits of a window: for column i, the cells of read bases 0..31
// in U[i] (substitution or insertion) and V[i] (insertion or deletion), and of
// bases 32..39 as bytes of H[i / 2] (U, V of the even column from the high
// byte on, then of the odd one, kept reversed), so that a window's 40 columns
// take 100 registers and two wavefronts fit a SIMD.
struct PathTable {
    uint32_t U[kLaneCols], V[kLaneCols], H[kLaneCols / 2];
};

// Bytes of a, b picked by the four selectors of sel (0..3: b, 4..7: a).
__device__ __forceinline__ uint32_t pick_bytes(uint32_t a, uint32_t b, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_perm(a, b, sel);
#else
    const u64 v = ((u64)a << 32) | b;
    uint32_t r = 0;
    for (int k = 0; k < 4; ++k) r |= (uint32_t)((v >> (8 * ((sel >> (8 * k)) & 7))) & 0xFF) << (8 * k);
    return r;
#endif
}

// Stores column i's words (bit 63 - j for read base j); columns come in
// descending order, so the odd column of a pair comes first.
template <int i>
__device__ __forceinline__ void table_put(PathTable& t, u64 u, u64 v) {
    t.U[i] = here(reverse32((uint32_t)(u >> 32)));
    t.V[i] = here(reverse32((uint32_t)(v >> 32)));
    const uint32_t top = pick_bytes((uint32_t)u, (uint32_t)v, 0x07030C0C);  // bytes 3 of u, v on top
    if constexpr (i & 1) t.H[i / 2] = here(top);
    else t.H[i / 2] = here(reverse32(pick_bytes(top, t.H[i / 2], 0x07060302)));
}

template <int i, int end>
__device__ __forceinline__ void path_steps(PathWalk& w, const PathTable& t, u64 live, int L) {
    if constexpr (i < end) {
        if (i < L) {
            const uint32_t h = t.H[i / 2] >> (i & 1 ? 16 : 0);
            path_step<i>(w, ((u64)h << 32) | t.U[i], ((u64)(h >> 8) << 32) | t.V[i], live);
        }
        path_steps<i + 1, end>(w, t, live, L);
    }
}
template <int i>
__device__ __forceinline__ void path_blocks(PathWalk& w, const PathTable& t, u64 live, int L) {
    if constexpr (i < kLaneCols) {
        // whole blocks of 8 columns without a branch per column
        if (i + 8 <= L) path_steps<i, i + 8>(w, t, live, kLaneCols);
        else path_steps<i, i + 8>(w, t, live, L);
        path_blocks<i + 8>(w, t, live, L);
    }
}

// 64 text columns as halves of their bit planes: lo[i / 32] bit i % 32 is bit 0
// of base i's code, hi bit 1, past set where there is no base.
struct TextBlock {
    uint32_t lo[2], hi[2], past[2];
};
__device__ __forceinline__ TextBlock text_block(u64 tl, u64 th, u64 past) {
    // halves of their own, so that a column's bit is one sign-extending extract
    return TextBlock{{here((uint32_t)tl), here((uint32_t)(tl >> 32))},
                     {here((uint32_t)th), here((uint32_t)(th >> 32))},
                     {here((uint32_t)past), here((uint32_t)(past >> 32))}};
}

// The read bases equal to text base i (a, b: the read's planes, pad: rows past
// the read, which match everything); `out` is all ones past the text.
template <bool RAGGED>
__device__ __forceinline__ u64 equal_rows(u64 a, u64 b, u64 pad, const TextBlock& t, int i, u64& out) {
    u64 ne = a ^ both(bit_mask(t.lo[i / 32], i & 31));
    out = 0ull;
    if constexpr (RAGGED) {
        out = both(bit_mask(t.past[i / 32], i & 31));
        ne |= out;
    }
    u64 Eq = bit_op<~(kA | (kB ^ kC))>(ne, b, both(bit_mask(t.hi[i / 32], i & 31)));
    if constexpr (RAGGED) Eq |= pad;
    return Eq;
}

// Text columns i..0 of a window's dynamic program.
template <bool RAGGED, int i>
__device__ __forceinline__ void window_columns(DiffColumn& c, PathTable& t, u64 a, u64 b, u64 pad,
                                               const TextBlock& text) {
    if constexpr (i >= 0) {
        u64 out;
        const u64 Eq = equal_rows<RAGGED>(a, b, pad, text, i, out);
        u64 D0, Ph, Mh;
        diff_step(c, Eq, D0, Ph, Mh);
        if constexpr (i < kLaneCols) {
            u64 u = bit_op<~kA | (kB & ~kC)>(D0, c.Pv, Eq), v = bit_op<kA & ~kB & kC>(D0, Eq, D0);
            if constexpr (RAGGED) {
                u |= out;
                v |= out;
            }
            table_put<i>(t, u, v);
        }
        if constexpr (i % 4 == 0) sched_fence();
        window_columns<RAGGED, i - 1>(c, t, a, b, pad, text);
    }
}

// Computes a window and its traceback. pl, ph, tl, th: bit planes of the read
// and text windows (bit k: base k). RAGGED: mw or nw may be below 64; otherwise
// both are 64. Text columns at or past nw match nothing, which keeps them at
// the initial column, and a traceback that reaches them only inserts. L <=
// kLaneCols.
template <bool RAGGED>
__device__ __forceinline__ WindowPath window_path(u64 pl, u64 ph, u64 tl, u64 th, int mw, int nw,
                                                  int L) {
    const u64 a = __builtin_bitreverse64(pl), b = __builtin_bitreverse64(ph);
    const u64 pad = RAGGED && mw < 64 ? (1ull << (64 - mw)) - 1 : 0ull;  // rows past the read window
    const u64 past = RAGGED && nw < 64 ? ~0ull << nw : 0ull;             // columns past the text
    DiffColumn c{~pad, 0ull};
    PathTable t;
    window_columns<RAGGED, 63>(c, t, a, b, pad, text_block(tl, th, past));
    WindowPath w;
    w.dist = __builtin_popcountll(c.Pv) - __builtin_popcountll(c.Mv);
    const int j_max = RAGGED ? min(mw, L) : L;
    const u64 live = ~0ull >> (64 - j_max);
    PathWalk p{1ull, 0ull, 0ull, {0u, 0u}};
    path_blocks<0>(p, t, live, L);
    w.ins = p.ins & live;
    w.sub = p.sub;
    // column i's bit back to bit i. A path that left its read bases stays at none
    // from the column after its last move on (no deletion comes right before the
    // insertions it may have left with).
    const int tail = max(L - 32, 0);
    u64 stay = ((u64)(tail ? reverse32(p.stay[1]) >> (32 - tail) : 0u) << 32) |
               (reverse32(p.stay[0]) >> (32 - min(L, 32)));
    const u64 moved = ~stay & (~0ull >> (64 - L));
    if (p.cur == 0ull) stay &= moved ? ~0ull >> __builtin_clzll(moved) : 0ull;
    w.del = stay;
    w.j_end = min(ctz64(p.cur), j_max);
    w.i_end = w.j_end - __builtin_popcountll(w.ins) + __builtin_popcountll(w.del);
    return w;
}
