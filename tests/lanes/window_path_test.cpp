// window_path (one lane's window on vertical differences) against a textbook
// dynamic program and a cell-by-cell traceback: random windows of every length,
// every commit limit, related and unrelated sequences.
//   window_path_test SEED COUNT
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

typedef unsigned long long u64;
using std::max;
using std::min;
#define __device__
#define __forceinline__ inline
static u64 reverse64(u64 x) {
    u64 r = 0;
    for (int b = 0; b < 64; ++b) r |= ((x >> b) & 1ull) << (63 - b);
    return r;
}
#define __builtin_bitreverse64 reverse64
static int ctz64(u64 x) { return x ? __builtin_ctzll(x) : 64; }
#include "../../paper_2203_15561_amd/csrc/diff_window.h"

static u64 state;
static uint32_t rnd(uint32_t n) {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)((state >> 33) % n);
}

struct Want {
    u64 ins, sub, del;
    int i, j, dist;
};

static Want textbook(const int* P, const int* T, int mw, int nw, int L) {
    static int E[65][65];
    for (int i = nw; i >= 0; --i)
        for (int j = mw; j >= 0; --j) {
            if (j == mw) E[i][j] = 0;
            else if (i == nw) E[i][j] = mw - j;
            else E[i][j] = min(min(E[i + 1][j], E[i][j + 1]) + 1, E[i + 1][j + 1] + (P[j] != T[i]));
        }
    Want w{0, 0, 0, 0, 0, E[0][0]};
    int d = w.dist;
    while (w.j < min(mw, L) && w.i < L) {
        const bool in = w.i < nw;
        if (in && P[w.j] == T[w.i]) {
            ++w.i, ++w.j;
            continue;
        }
        if (in && E[w.i + 1][w.j + 1] <= d - 1) w.sub |= 1ull << w.j, ++w.i, ++w.j;
        else if (E[w.i][w.j + 1] <= d - 1) w.ins |= 1ull << w.j, ++w.j;
        else w.del |= 1ull << w.i, ++w.i;
        --d;
    }
    return w;
}

static bool same(const WindowPath& g, const Want& w) {
    return g.ins == w.ins && g.sub == w.sub && g.del == w.del && g.i_end == w.i && g.j_end == w.j &&
           g.dist == w.dist;
}

int main(int argc, char** argv) {
    if (argc != 3) return 2;
    state = (u64)atoll(argv[1]);
    const int count = atoi(argv[2]);
    for (int it = 0; it < count; ++it) {
        int P[64], T[64];
        const int mw = rnd(3) ? 64 : 1 + (int)rnd(64), nw = rnd(3) ? 64 : (int)rnd(65);
        const int L = rnd(2) ? kLaneCols : 1 + (int)rnd(kLaneCols);
        const int letters = 1 + (int)rnd(4);  // few letters: long runs of ties
        for (int& t : T) t = (int)rnd((uint32_t)letters);
        const uint32_t rate = it % 5 == 0 ? 1000 : rnd(400);
        int s = 0;
        for (int& p : P) {
            if (rnd(1000) < rate) {
                const uint32_t kind = rnd(3);
                p = (int)rnd((uint32_t)letters);
                if (kind == 0) ++s;
                else if (kind == 1) s += 1 + (int)rnd(3), p = T[s & 63], ++s;
            } else {
                p = T[s & 63];
                ++s;
            }
        }
        u64 pl = 0, ph = 0, tl = 0, th = 0;
        for (int k = 0; k < 64; ++k) {
            pl |= (u64)(P[k] & 1) << k;
            ph |= (u64)(P[k] >> 1) << k;
            tl |= (u64)(T[k] & 1) << k;
            th |= (u64)(T[k] >> 1) << k;
        }
        const Want w = textbook(P, T, mw, nw, L);
        const WindowPath r = window_path<true>(pl, ph, tl, th, mw, nw, L);
        const WindowPath f = mw == 64 && nw == 64 ? window_path<false>(pl, ph, tl, th, mw, nw, L) : r;
        if (!same(r, w) || !same(f, w)) {
            printf("window %d differs: mw %d nw %d L %d, distance %d, want %d\n", it, mw, nw, L, r.dist, w.dist);
            return 1;
        }
    }
    printf("ok %d\n", count);
    return 0;
}
