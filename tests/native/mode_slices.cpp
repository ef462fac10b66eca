// Holds every load of the mode products to its buffer: all slices' offsets of modeslice.h, walked as the
// kernel walks them, over mode sizes 1 .. 300 and trailing sizes 1 .. 40, both types, every tile.
#include <algorithm>
#include <cstdio>
#include <initializer_list>

#include "modeslice.h"

using cola::ModeSlices;

static long long checked = 0;
static int failures = 0;

static void fail(const char* what, int vw, int kt, int nt, int nk, long B, long G, long at, long end) {
    if (++failures <= 20)
        std::printf("%s: VW %d KT %d tile %d nk %d B %ld G %ld: element %ld of %ld\n", what, vw, kt, nt, nk, B, G, at, end);
}

template <int VW, int KT, int WM, int WN, bool ROWS>
static void check(int nk, long B, long G) {
    using S = ModeSlices<VW, KT, WM, WN, ROWS>;
    const long total = ROWS ? G * nk : G * nk * B;
    const long M = ROWS ? G : nk, N = ROWS ? nk : B;
    const long mts = (M + S::MT - 1) / S::MT, nts = (N + S::NT - 1) / S::NT;
    auto in = [&](const char* what, long at) {
        ++checked;
        if (at < 0 || at + VW > total) fail(what, VW, KT, ROWS ? S::MT : S::NT, nk, B, G, at, total);
    };
    for (long g : {0L, ROWS ? 0L : G - 1})
        for (long mt : {0L, mts - 1})
            for (long nt : {0L, nts - 1}) {
                const S s{nk, B, G, mt * S::MT, nt * S::NT, g};
                const int ns = s.slices();
                const long last = s.x_base() + (ns - 1) * s.x_step();
                for (int tid = 0; tid < S::THREADS; ++tid) {
                    for (int q = 0; q < S::XV; ++q) {
                        for (int u : {0, ns - 2}) {
                            if (u < 0 || u >= ns - 1) continue;
                            in("slice", s.x_base() + u * s.x_step() + s.x_at(tid, q));
                            const int k = s.panel_k(tid, q), c = s.panel_col(tid);      // stored columns: their own place
                            if (!ROWS && s.n0 + c < B && s.x_at(tid, q) != k * B + c)
                                fail("moved", VW, KT, S::NT, nk, B, G, s.x_at(tid, q), k * B + c);
                        }
                        in("last slice", last + s.x_last(tid, q));
                        in("after the last slice", last + s.x_idle_at(tid, q));
                        const long early = s.x_last_wanted(tid, q) - s.x_last(tid, q);
                        if (early > 0 && !s.x_clamped()) fail("not put back", VW, KT, S::NT, nk, B, G, early, 0);
                    }
                    for (int q = 0; q < S::FV; ++q) {        // the factor, padded by 128 bytes
                        const long f = (ROWS ? s.n0 : s.m0) * nk + s.f_at(tid, q) + (ns - 1) * KT;
                        const long pad = 128 / (VW == 2 ? 8 : 4);
                        if (f < 0 || f + VW > (long)nk * nk + pad) fail("factor", VW, KT, S::MT, nk, B, G, f, nk * nk);
                    }
                }
            }
}

template <int VW, int KT>
static void type(int es) {
    for (int nk = 1; nk <= 300; ++nk) {
        for (long B = 1; B <= 40; ++B)
            for (long G : {1L, 3L}) {
                if (cola::mode_needs_general<VW, KT>(false, nk, B, G, es)) continue;
                check<VW, KT, 4, 1, false>(nk, B, G);
                check<VW, KT, 3, 2, false>(nk, B, G);
                check<VW, KT, 1, 4, false>(nk, B, G);
            }
        for (long G : {1L, 2L, 31L, 33L, 65L, 129L}) {
            if (cola::mode_needs_general<VW, KT>(true, nk, 1, G, es)) continue;
            check<VW, KT, 1, 4, true>(nk, 1, G);
            check<VW, KT, 2, 3, true>(nk, 1, G);
            check<VW, KT, 4, 1, true>(nk, 1, G);
        }
    }
}

int main() {
    type<2, 16>(8);
    type<4, 32>(4);
    std::printf("%lld loads, %d outside\n", checked, failures);
    return failures ? 1 : 0;
}
