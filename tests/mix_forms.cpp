// Prints which contractions of a step's shared launches take tall tiles (mix_plan.hpp), for tests/test_mix_forms.py.  One line of standard input is one call:
//   <fp8> <M> <D> <F> <T>   -> does the step share launches; the forms of eqs. (3), (5), (4), of (5), (4) and of (7), (8)
//   alone <fp8> <T> <N> <F> -> eqs. (3), (7) and (bf16) (5), (8) in launches of their own: the tile that the rules choose, is it a tall one instead (64 tiles, three workgroups a CU: no)
//   streams <T> <D> <F>     -> do the epilogues' stores go past the caches
//   play <slots> <n> <time> <alone> ... (three times)   -> time of the launch
#include <stdio.h>
#include <string.h>

#include "../paper_2602_06183_amd/csrc/kernels.hpp"

using namespace sffn;

static unsigned tiles(long a, long ea, long b, long eb) { return (unsigned)((a + ea - 1) / ea * ((b + eb - 1) / eb)); }

int main() {
    char first[16];
    while (scanf("%15s", first) == 1) {
        if (!strcmp(first, "play")) {
            float slots;
            MixUnit u[3];
            if (scanf("%f", &slots) != 1) return 1;
            for (MixUnit& x : u) if (scanf("%f %f %f", &x.n, &x.time, &x.alone) != 3) return 1;
            printf("%.4f\n", mix_time(u, 3, slots));
            continue;
        }
        if (!strcmp(first, "streams")) {
            long T, D, F;
            if (scanf("%ld %ld %ld", &T, &D, &F) != 3) return 1;
            printf("%d\n", (int)streams_between(T, D, F, 1, 2 * T * F));
            continue;
        }
        if (!strcmp(first, "alone")) {
            long f8, T, N, F;
            if (scanf("%ld %ld %ld %ld", &f8, &T, &N, &F) != 4) return 1;
            const AloneTiles& k = f8 ? kAloneActivationFp8 : kAloneActivationBf16;
            const int steps = (int)(F / (f8 ? 128 : 64)), v = plan_vnm8(T, N, steps, 0, f8 != 0).tile, w = pick_wgrad_tile(F, N, T, 0, true, f8 != 0);
            const unsigned n512 = (unsigned)(0.93f * (float)tiles(T, 512, N, 128)), n256 = tiles(T, 256, N, 256);
            const bool v_tall = v != 64 && tall_alone(k, v == 256 ? rounds_of_large(n512 < n256 ? n512 : n256, k.part) : 0.0f, tiles(T, 128, N, 128), tiles(T, 256, N, 128), steps);
            const bool w_tall = !f8 && w != 64 && !wgrad_three_a_cu(F, N, T, 0, w) &&
                                tall_alone(kAloneGradientBf16, w == 256 ? rounds_of_large(tiles(F, 256, N, 256), kAloneGradientBf16.part) : 0.0f, tiles(F, 128, N, 128), tiles(F, 256, N, 128), (int)(T / 64));
            printf("%d %d %d %d\n", v, (int)v_tall, w, (int)w_tall);
            continue;
        }
        const int fp8 = first[0] == '1';
        long M, D, F, T;
        if (scanf("%ld %ld %ld %ld", &M, &D, &F, &T) != 4) return 1;
        const StepTiles t = step_tiles(T, D, F, (int)M, 1, fp8 != 0);
        const int unit = fp8 ? 128 : 64, kc = (int)(4 * F / M);
        MixCount v, w, g = {0, tiles(F, M == 64 ? 256 : 128, T, 128), M == 64 ? 0 : tiles(F, 256, T, 128), (int)(D / unit)};
        if (M == 8) v = t.v == 64 ? MixCount{tiles(T, 64, D, 64), 0, 0, (int)(F / unit) / 4} : MixCount{0, tiles(T, 128, D, 128), tiles(T, 256, D, 128), (int)(F / unit)};
        else v = t.v == 64 ? MixCount{tiles(T, 64, D, 64), 0, 0, kc / 64 / 4} : MixCount{0, tiles(T, 64, D, 256), 0, kc / unit};
        w = t.w == 64 ? MixCount{tiles(F, 64, D, 64), 0, 0, (int)(T / 64) / 4} : MixCount{0, tiles(F, 128, D, 128), tiles(F, 256, D, 128), (int)(T / unit)};
        MixTiles k = M == 8 ? (fp8 ? kMixFp8 : kMixBf16) : fp8 ? kMixWideFp8 : kMixWideBf16;
        if (M == 64) k.g[0] = fp8 ? kMixTallFp8 : kMixTallBf16;
        const float slots = t.w == 64 && !fp8 ? 32.0f : 64.0f;
        printf("%d", (int)t.mix);
        for (int what : {kMixForwardTail, kMixBackwardHead, kMixBackwardTail})
            printf(" %u", mix_form(k, what, what != kMixBackwardHead ? v : MixCount(), w, what != kMixBackwardTail ? g : MixCount(), slots,
                                   2.0f * ((float)F * D * (what == kMixBackwardTail ? 2.0f : 3.6f) + (float)T * (2.0f * D + F))));
        printf("\n");
    }
    return 0;
}
