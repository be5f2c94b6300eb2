// Which contractions of a shared launch (StepTiles in kernels.hpp) take tiles of 256 x 128 in the place of 128 x 128.  Two workgroups of either, four wavefronts each, fit a CU.  The tall ones
// fetch a third (eqs. (4), (5), (8)) to two fifths (eqs. (3), (7)) fewer bytes per product; half as many tiles fill the chip worse.  Same sums in the same order, same bits.
#pragma once

namespace sffn {

enum { kMixForwardTail = 0, kMixBackwardHead = 1, kMixBackwardTail = 2 };      // {(3), (5), (4)}, {(5), (4)}, {(7), (8)}

// What a tile takes (us): fixed + step x stages beside another one on its CU, `alone` of that without.
struct MixTile { float fixed, step, alone; };
struct MixUnit { float n, time, alone; };                      // a contraction: its tiles on the fullest XCD, what one takes
inline MixUnit mix_unit(const MixTile& t, unsigned tiles, int stages) { return {(float)((tiles + 7) / 8), t.fixed + t.step * (float)stages, t.alone}; }

// The launch played through on one XCD: `slots` workgroups at a time, started in order wherever a slot is free.
inline float mix_time(const MixUnit* u, int m, float slots) {
    struct { float left, n, alone; } run[96];                  // tiles that started together
    int r = 0, c = 0;
    float now = 0.0f, idle = slots, wait = m ? u[0].n : 0.0f;
    for (;;) {
        while (c < m && idle > 0.0f) {
            if (wait <= 0.0f) { if (++c < m) wait = u[c].n; continue; }
            if (r == 96) return now;                           // (a round of the chip starts as a few groups: not met)
            const float k = wait < idle ? wait : idle;
            run[r].left = u[c].time; run[r].n = k; run[r].alone = u[c].alone;
            ++r; idle -= k; wait -= k;
        }
        if (r == 0) return now;
        // the part of the tiles that counts as alone on its CU: all of them, or half of those that are (the end waits for those that are not)
        const float busy = slots - idle, lone = busy <= 0.5f * slots ? 1.0f : 0.5f * idle / busy;
        auto pace = [&](int i) { return lone * run[i].alone + 1.0f - lone; };
        float next = 1e30f;
        for (int i = 0; i < r; ++i) { const float d = run[i].left * pace(i); next = d < next ? d : next; }
        now += next;
        int kept = 0;
        for (int i = 0; i < r; ++i) {
            run[i].left -= next / pace(i);
            if (run[i].left <= 1e-3f * next) idle += run[i].n;
            else run[kept++] = run[i];
        }
        r = kept;
    }
}

// The tiles of a kind of step: 64, then 128 and tall (eqs. (3), (7) on gathered rows: 64 x 256, no tall form); us per MB of the launch's bytes (those that bf16 would have).
// Fitted to the shared launches of 540 steps (T 64 - 12000, D 256 - 7000, up to 6e11 token-weight elements), each with every contraction on either tile: standard deviation 6 - 8 %.  What is
// chosen takes, of tiles of 128 everywhere (the best form of each):
//   bf16, M = 8           from 1000 tokens on 0.909 (0.899), 300 - 1000 0.947 (0.933), below 0.986 (0.965)
//   codes, M = 8          0.942 (0.925), 0.959 (0.936), 0.993 (0.969)
//   M = 16, 32, 64        bf16 0.969 (0.960), 0.958 (0.947), 0.967 (0.959); codes 0.980 (0.968), 0.956 (0.945), 0.977 (0.965)
// The bytes are those of one expert's weight where there are several: all of them hold every form down alike where tall ones save operand bytes (142 backward calls of 4 and 8 experts 0.973, with
// the bytes of all 0.981).
// Eqs. (3), (5), (4) and (7), (8) at M = 8: T = 1216, D = 5248, F = 17536 491 -> 411 us and 324 -> 256, T = 1344, D = 2240, F = 7424 92 -> 87 and 62 -> 57; with few tiles tall ones take
// longer, a step of T = 2176, D = 832, F = 2752 76 us, all tall 85.
// few: a launch of eqs. (3), (5), (4) with 64 tiles in eq. (3), up to three stages in eq. (5) and between one and that many rounds of the chip stays on 128: the estimate has the workgroups past the
// first round wait for a whole one, but the 64 tiles, first and short, make way for them at once.  Steps at M = 8 in bf16, 128 / tall: 1.02 rounds (T = 128, D = 1280, F = 5568) 47.5 / 51.2 us, 1.03
// (T = 64, D = 1408, F = 5312) 45.9 / 49.0, 1.21 (T = 192, D = 1536, F = 4992) 51.2 / 53.5, 1.30 (T = 128, D = 1664, F = 5568) 52.6 / 50.8; with more stages the shorter launch is worth more: T = 448,
// D = 1472, F = 3648 0.87 of the time on tall tiles.  231 steps of 1.0 - 1.25 rounds, of the time on 128: 0.962, the longest 1.02; tall always 0.965, 1.08.  Not for experts (26 steps 1.05 of the time
// on tall tiles), on codes (0.995 -> 0.998) and for wider blocks (tall 0.96 - 0.98 in four of five).
struct MixTiles { MixTile v64, v[2], w64, w[2], g[2]; float bytes, few = 0.0f; };
constexpr MixTiles kMixBf16 = {{3.77f, 0.227f, 0.86f}, {{0.0f, 0.434f, 0.674f}, {0.19f, 0.518f, 0.757f}}, {3.81f, 0.522f, 0.939f}, {{5.37f, 0.758f, 0.495f}, {9.28f, 1.373f, 0.45f}},
                               {{1.65f, 0.652f, 0.658f}, {3.68f, 1.01f, 0.808f}}, 0.23f, 1.25f};
constexpr MixTiles kMixFp8 = {{4.83f, 0.342f, 0.575f}, {{0.11f, 0.506f, 0.466f}, {1.74f, 0.708f, 0.485f}}, {9.17f, 0.68f, 0.384f}, {{5.17f, 0.667f, 0.591f}, {8.96f, 1.106f, 0.589f}},
                              {{4.46f, 0.575f, 0.92f}, {9.4f, 0.972f, 0.76f}}, 0.176f};
constexpr MixTiles kMixWideBf16 = {{0.94f, 4.41f, 0.364f}, {{0.0f, 1.348f, 0.566f}, {}}, {}, {{4.27f, 0.598f, 0.603f}, {5.85f, 1.046f, 0.626f}}, {{2.19f, 0.617f, 0.699f}, {3.43f, 1.109f, 0.744f}}, 0.207f};
constexpr MixTiles kMixWideFp8 = {{}, {{0.04f, 1.103f, 0.666f}, {}}, {8.3f, 0.757f, 0.3f}, {{3.43f, 0.719f, 0.547f}, {5.99f, 1.279f, 0.549f}}, {{2.49f, 0.683f, 0.727f}, {5.98f, 1.009f, 0.788f}}, 0.124f};
// Weight gradients that are added to float32 sums: a tile reads and writes eight bytes an element behind its last product, a tall one twice as many, so that where every CU has one tile the launch waits
// for that.  Backward calls, 128 / tall: T = 320, D = 1088, F = 4096 32.4 / 38.0 us, M = 32, T = 448, D = 896, F = 3072 1.15 of the time, 8 experts of 72 tokens 1.15; T = 256, D = 2752,
// F = 7360 112 / 94.  Fitted to 535 such calls (T 64 - 8192, 1 - 8 experts, every M) on each form; over 1660 others, of 128 everywhere: M = 8 0.990 (0.987 the best forms), experts 0.990 (0.984),
// M = 16, 32, 64 0.991 (0.988), nine launches of 3300 longer than 1.02, none than 1.034; with the constants above, over the first 535: 0.991, 1.00 and 0.998, one launch in 14 longer than 1.02, up to 1.15.
constexpr MixTiles kMixBf16Sums = {kMixBf16.v64, {kMixBf16.v[0], kMixBf16.v[1]}, {5.47f, 0.522f, 0.939f}, {{6.69f, 0.758f, 0.571f}, {12.27f, 1.373f, 0.799f}}, {kMixBf16.g[0], kMixBf16.g[1]}, 0.16f};
constexpr MixTiles kMixWideBf16Sums = {kMixWideBf16.v64, {kMixWideBf16.v[0], {}}, {}, {{6.85f, 0.598f, 0.388f}, {11.06f, 1.046f, 0.928f}}, {kMixWideBf16.g[0], kMixWideBf16.g[1]}, 0.2f};
// M = 64: eq. (4) is on 256 x 128 as it is
constexpr MixTile kMixTallBf16 = {4.14f, 0.996f, 0.71f}, kMixTallFp8 = {4.3f, 1.075f, 0.761f};

// A contraction of the launch: its tiles of each kind (0: not offered; 64: one kind) and the stages of one.
struct MixCount { unsigned n64, n128, tall; int stages; };
// What a tall form has to save: two runs of one form differ by 1 - 2 %; beside 64 tiles of eqs. (3), (7), where the estimate is off by more (T = 128, D = 1344, F = 4608 16.1 us, 19.6 with tall
// tiles in eq. (5), which it takes for 0.91 of the time), a tenth.
constexpr float kMixSave = 0.04f, kMixSaveBeside64 = 0.1f;
// Bits 0, 1, 2: eqs. (3) / (7), (5) / (8), (4) on tall tiles; eq. (4) only where all the others that have them are (built so).  slots: workgroups at a time on an XCD; bytes: of the launch.
// Past 16 rounds of the chip the largest form is taken unseen.
inline unsigned mix_form(const MixTiles& k, int what, const MixCount& v, const MixCount& w, const MixCount& g, float slots, float bytes) {
    MixUnit u[3][2];
    int bit[3], m = 0;
    float all = 0.0f;
    auto add = [&](int b, const MixTile& t64, const MixTile (&t)[2], const MixCount& c) {
        u[m][0] = c.n64 ? mix_unit(t64, c.n64, c.stages) : mix_unit(t[0], c.n128, c.stages);
        u[m][1] = c.tall ? mix_unit(t[1], c.tall, c.stages) : u[m][0];
        all += u[m][0].n;
        bit[m++] = b;
    };
    const bool has_v = what != kMixBackwardHead, w_first = has_v && w.stages > v.stages;
    if (w_first || !has_v) add(1, k.w64, k.w, w);
    if (has_v) add(0, k.v64, k.v, v);
    if (has_v && !w_first) add(1, k.w64, k.w, w);
    if (what != kMixBackwardTail) add(2, k.g[0], k.g, g);
    if (all <= 0.5f * slots) return 0;                         // (a CU for each)
    if (what == kMixForwardTail && v.n64 && w.stages <= 3 && all > slots && all <= k.few * slots) return 0;
    const unsigned may = (has_v && v.tall ? 1u : 0u) | (w.tall ? 2u : 0u), most = may | (what != kMixBackwardTail && g.tall && w.tall && (v.tall || !has_v || !v.n64) ? 4u : 0u);
    if (all > 16.0f * slots) return most;
    unsigned best = 0;
    float shortest = 0.0f;
    for (unsigned f = 0; f < 8; ++f) {
        if ((f & ~most) || ((f & 4u) && f != most)) continue;
        MixUnit on[3];
        for (int i = 0; i < m; ++i) on[i] = u[i][f >> bit[i] & 1u];
        float t = mix_time(on, m, slots);
        t = t < k.bytes * 1e-6f * bytes ? k.bytes * 1e-6f * bytes : t;
        if (f == 0) shortest = (1.0f - (has_v && v.n64 ? kMixSaveBeside64 : kMixSave)) * t;
        else if (t < shortest) { shortest = t; best = f; }
    }
    return best;
}

// A contraction in a launch of its own, on the large tile (a round of 256 at a time: fixed + step x stages; a last round of few tiles `part` of that and up), on 128 or on tall tiles; `start` comes
// on top of each.  Fitted to launches inside 130 steps of any size (T 128 - 16384, D 320 - 8192) on each tile; tall tiles where the estimate saves `save`.  Over the tile that the rules of
// kernels.hpp choose: eqs. (3), (7) 0.943 of the time in bf16 and 0.961 on codes over all of them, none longer (T = 1664, D = 3968, F = 15616 155 us on the large tile, 169 on 128, 119;
// T = 2304, D = 1856, F = 4864 41, 41, 34); eqs. (5), (8) in bf16 0.90 where they are chosen, one in nine, none above 0.945 (T = 2944, D = 3456, F = 9344 151 -> 137), on codes nothing;
// eqs. (1), (4) 0.994, not built.  Experts, not among the 130: their gradients are offered it nearly always where a step shares no launches, 22 backward calls 0.95, none above 1.00; with float32 sums
// 87 calls 0.994, none above 1.02, without experts 15 calls 0.975.
struct AloneTiles { MixTile large; float part; MixTile small, tall; float large_start, small_start, tall_start, save; };
constexpr AloneTiles kAloneActivationBf16 = {{0.0f, 0.636f, 1.0f}, 0.621f, {0.0f, 0.582f, 0.501f}, {0.0f, 0.759f, 0.492f}, 8.15f, 5.56f, 6.88f, 0.06f};
constexpr AloneTiles kAloneActivationFp8 = {{0.0f, 0.705f, 1.0f}, 0.69f, {0.0f, 0.629f, 0.476f}, {0.0f, 0.844f, 0.495f}, 9.2f, 6.46f, 7.95f, 0.06f};
constexpr AloneTiles kAloneGradientBf16 = {{6.46f, 1.258f, 1.0f}, 0.778f, {2.74f, 0.715f, 0.534f}, {4.53f, 1.255f, 0.546f}, 3.73f, 5.93f, 6.05f, 0.05f};
// large: rounds of the large tile, or 0 where `small` tiles of 128 are chosen
inline bool tall_alone(const AloneTiles& k, float large, unsigned small, unsigned tall, int stages) {
    if (tall > 8192) return false;                             // (16 rounds: what they end in no longer counts)
    const MixUnit t = mix_unit(k.tall, tall, stages), s = mix_unit(k.small, small, stages);
    const float now = large > 0.0f ? k.large_start + large * (k.large.fixed + k.large.step * (float)stages) : k.small_start + mix_time(&s, 1, 64.0f);
    return k.tall_start + mix_time(&t, 1, 64.0f) < (1.0f - k.save) * now;
}

}  // namespace sffn
