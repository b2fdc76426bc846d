// Host check of the narrow form (narrow_form in na_launch.h, MaskRows in na_stage.h, compiled for
// the host).  Reads problems from stdin, one line each:
//   rank, then per axis: extent window dilation causal wave_tile waves
// and prints per line whether the launchers take the form, and the wave tile it cuts.  For each
// problem it is taken for, every wave of every tile of every dilation group is walked as the
// kernels walk it: what the table, the operands and the wave's eight columns let through must be
// each query's neighbours (win_start .. win_last), no more and no fewer.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "na_launch.h"
#include "na_stage.h"

using namespace na;

static void fail(const char* what, const Geo& g, int rank) {
    std::printf("FAIL %s:", what);
    for (int a = 0; a < rank; ++a)
        std::printf(" L=%d k=%d d=%d c=%d T=%d WT=%d", g.L[a], g.k[a], g.d[a], g.causal[a], g.T[a],
                    g.WT[a]);
    std::printf("\n");
    std::exit(1);
}

// Calls f(c) for every c of [0, n0) x [0, n1) x [0, n2).
template <class F>
static void each(const int* n, F f) {
    int c[3];
    for (c[0] = 0; c[0] < n[0]; ++c[0])
        for (c[1] = 0; c[1] < n[1]; ++c[1])
            for (c[2] = 0; c[2] < n[2]; ++c[2]) f(c);
}

template <int R>
static long check(const Geo& g) {
    long pairs = 0;
    each(g.d, [&](const int* gc) {
        int n[3];
        for (int a = 0; a < 3; ++a) n[a] = group_len(g.L[a], g.d[a], gc[a]);
        each(g.nt, [&](const int* tc) {
            int to[3], lo[3], E[3] = {1, 1, 1};
            for (int a = 0; a < 3; ++a) {
                to[a] = tc[a] * g.T[a];
                if (to[a] >= n[a]) return;
                const int last = (to[a] + g.T[a] < n[a] ? to[a] + g.T[a] : n[a]) - 1;
                lo[a] = win_start(to[a], n[a], g.k[a], g.causal[a]);
                E[a] = win_last(last, n[a], g.k[a], g.causal[a]) + 1 - lo[a];
            }
            if (E[R - 1] > 16) fail("a halo row is longer than a block", g, R);
            int nb = 1;
            for (int a = 0; a < R - 1; ++a) nb *= E[a];
            if (nb > g.tab_rows) fail("more rows than the table has", g, R);
            each(g.WGd, [&](const int* wc) {
                MaskRows<R> m;
                int wo[3], l[3], inner_lo = 0;
                for (int a = 0; a < 3; ++a) {
                    wo[a] = to[a] + wc[a] * g.WT[a];
                    if (wo[a] >= n[a]) return;
                    l[a] = (wo[a] + g.WT[a] < n[a] ? wo[a] + g.WT[a] : n[a]) - 1;
                    const bool c = g.causal[a];
                    const int sf = win_start(wo[a], n[a], g.k[a], c);
                    const int sl = win_start(l[a], n[a], g.k[a], c);
                    const int ef = win_last(wo[a], n[a], g.k[a], c);
                    const int el = win_last(l[a], n[a], g.k[a], c);
                    if (a < R - 1) m.set(a, sf - lo[a], el + 1 - sf, sl - sf, ef + 1 - sf);
                    if (a == R - 1) {
                        inner_lo = sf - lo[a];
                        if (el - sf + 1 > 8) fail("a wave needs more than eight columns", g, R);
                    }
                }
                const int z = R - 2;
                if (m.slot[z] + m.nlow[z] + m.len[z] - m.nfirst[z] > 15) fail("slots", g, R);
                const int col0 = inner_lo < 8 ? inner_lo : 8;
                each(g.WT, [&](const int* qc) {
                    int p[3], qs[3], s[3], e[3];
                    unsigned op = MaskRows<R>::operand();
                    for (int a = 0; a < 3; ++a) {
                        p[a] = wo[a] + qc[a];
                        if (p[a] >= n[a]) return;
                        const bool c = g.causal[a];
                        qs[a] = mask_start(p[a], n[a], g.k[a], c) - lo[a];
                        s[a] = win_start(p[a], n[a], g.k[a], c) - lo[a];
                        e[a] = win_last(p[a], n[a], g.k[a], c) - lo[a];
                        if (a < R - 1) op = m.operand(op, a, qs[a], qs[a] + g.k[a] - 1);
                    }
                    int rows[3] = {1, 1, 1};
                    for (int a = 0; a < R - 1; ++a) rows[a] = E[a];
                    each(rows, [&](const int* oc) {
                        bool outer = true;
                        for (int a = 0; a < R - 1; ++a)
                            outer = outer && oc[a] >= s[a] && oc[a] <= e[a];
                        if (outer != ((m.row_slots(oc) & op) == 0)) fail("outer mask", g, R);
                        for (int x = 0; x < E[R - 1]; ++x, ++pairs) {
                            const bool want = x >= s[R - 1] && x <= e[R - 1];
                            const bool got = x >= col0 && x < col0 + 8 &&
                                             (unsigned)(x - qs[R - 1]) < (unsigned)g.k[R - 1];
                            if (want != got) fail("inner mask", g, R);
                        }
                    });
                });
            });
        });
    });
    return pairs;
}

int main() {
    int rank;
    long pairs = 0;
    while (std::scanf("%d", &rank) == 1) {
        Geo g;
        std::memset(&g, 0, sizeof g);
        int nb = 1;
        for (int a = 0; a < 3; ++a) {
            g.L[a] = g.k[a] = g.d[a] = g.WT[a] = g.WGd[a] = 1;
            if (a < rank && std::scanf("%d %d %d %d %d %d", &g.L[a], &g.k[a], &g.d[a],
                                       &g.causal[a], &g.WT[a], &g.WGd[a]) != 6)
                return 2;
            g.T[a] = g.WT[a] * g.WGd[a];
            const int n = group_len(g.L[a], g.d[a], 0);
            g.nt[a] = (n + g.T[a] - 1) / g.T[a];
        }
        nb = max_halo_blocks(g, rank);
        const bool taken = narrow_form(g, rank, nb);
        std::printf("%d %d %d %d\n", taken, g.WT[0], g.WT[1], g.WT[2]);
        if (taken) pairs += rank == 2 ? check<2>(g) : check<3>(g);
    }
    std::printf("pairs %ld\n", pairs);
    return 0;
}
