// Prints what the host-side tile rules (kernels.hpp) choose, for tests/test_tile_rules.py.  One line of standard input is one call:
//   step <fp8> <M> <D> <F> <experts> <offset 0> ... <offset n>   -> tiles of eq. (1), eq. (4), eqs. (3), (7), weight gradients in launches of their own; do they share;
//                                                                   tile of eq. (3) in a forward call
//   forward <M> <D> <F> <experts> <offset 0> ... <offset n>      -> tile of eq. (1) in a bf16 call; does it read X as it is on packed weights, does it on others; are its
//                                                                   preparing passes one launch
//   shares <M> <D> <F> <T>                                       -> does the router's step share launches; are its preparing passes one launch
//   share <fp8> <M> <D> <F> <experts> <T>                        -> do they share launches
//   router <M> <D> <F> <T>                                       -> tile of its eqs. (1), (4)
//   split <T> <N> <F>                                            -> workgroups per tile of eq. (3) at M = 8
//   rowx <M> <D> <F> <T>                                         -> does a forward call on packed weights read X as it is (-1: the tile does not)
//   plain <T> <N> <K>                                            -> tile of a 2:4 contraction with a plain store
#include <stdio.h>
#include <string.h>

#include "../paper_2602_06183_amd/csrc/kernels.hpp"

using namespace sffn;

int main() {
    char what[16];
    while (scanf("%15s", what) == 1) {
        long a, b, c, d, e;
        if (!strcmp(what, "plain")) {
            if (scanf("%ld %ld %ld", &a, &b, &c) != 3) return 1;
            const int steps = (int)(c / 64);
            printf("%d\n", pick_gemm_tile(b, a, steps, GemmGroup(), small_round(kGemmPlain, steps), true, last_round(kGemmPlain, steps)));
            continue;
        }
        if (!strcmp(what, "rowx")) {
            if (scanf("%ld %ld %ld %ld", &a, &b, &c, &d) != 4) return 1;
            const int tile = step_tiles(d, b, c, (int)a, 1, false).g;
            printf("%d\n", tile == 256 ? -1 : (int)forward_reads_x(d, b, c, (int)a, true, tile));
            continue;
        }
        if (!strcmp(what, "split")) {
            if (scanf("%ld %ld %ld", &a, &b, &c) != 3) return 1;
            printf("%d\n", plan_vnm8(a, b, (int)(c / 64), 0, false).n);
            continue;
        }
        if (!strcmp(what, "router")) {
            if (scanf("%ld %ld %ld %ld", &a, &b, &c, &d) != 4) return 1;
            GemmGroup g;
            g.n = (int)(a / 4);
            g.role = 1;
            const int steps = (int)(b / 64);
            printf("%d\n", pick_gemm_tile(4 * c / a, (d + 63) / 64 * 64 + 16 * a, steps, g, small_round(kGemmRouter, steps), true, last_round(kGemmRouter, steps)));
            continue;
        }
        if (!strcmp(what, "shares")) {
            if (scanf("%ld %ld %ld %ld", &a, &b, &c, &d) != 4) return 1;
            const int64_t rows = (d + 63) / 64 * 64 + 16 * a;
            printf("%d %d\n", (int)router_shares(rows, b, c, (int)a), (int)prologue_together(rows, b, c, 1));
            continue;
        }
        if (!strcmp(what, "forward")) {
            if (scanf("%ld %ld %ld %ld", &b, &c, &d, &e) != 4 || e > GemmGroup::kMaxExperts) return 1;
            GemmGroup g;
            g.n = e > 1 ? (int)e : 0;
            for (int i = 0; i <= e; ++i) if (scanf("%d", &g.seg[i]) != 1) return 1;
            const int64_t T = g.seg[e];
            StepTiles t = step_tiles(T, c, d, (int)b, (int)e, false);
            refine_tiles(&t, c, d, (int)b, g, false);
            printf("%d %d %d %d\n", t.g, (int)forward_reads_x(T, c, e * d, (int)b, true, t.g), (int)forward_reads_x(T, c, e * d, (int)b, false, t.g),
                   (int)(t.mix || prologue_together(T, c, d, e)));
            continue;
        }
        if (!strcmp(what, "share")) {
            long T;
            if (scanf("%ld %ld %ld %ld %ld %ld", &a, &b, &c, &d, &e, &T) != 6) return 1;
            printf("%d\n", (int)step_tiles(T, c, d, (int)b, (int)e, a != 0).mix);
            continue;
        }
        if (scanf("%ld %ld %ld %ld %ld", &a, &b, &c, &d, &e) != 5 || e > GemmGroup::kMaxExperts) return 1;
        GemmGroup g;
        g.n = e > 1 ? (int)e : 0;
        for (int i = 0; i <= e; ++i) if (scanf("%d", &g.seg[i]) != 1) return 1;
        StepTiles t = step_tiles(g.seg[e], c, d, (int)b, (int)e, a != 0, false);
        StepTiles whole = step_tiles(g.seg[e], c, d, (int)b, (int)e, a != 0);
        refine_tiles(&t, c, d, (int)b, g, a != 0);
        refine_tiles(&whole, c, d, (int)b, g, a != 0);
        printf("%d %d %d %d %d %d\n", t.g, t.g_bwd, t.v, t.w, (int)whole.mix, whole.v_alone);
    }
    return 0;
}
