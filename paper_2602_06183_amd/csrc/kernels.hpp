// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <initializer_list>

namespace sffn {

// Fused V:N:M epilogue of the two GEMMs whose output feeds the activation sparsifier (ffn_sparse_step only).
//   mode 1 (eq. (1) -> eq. (2) + Section 2.3): the tile of y1 is squared-ReLU'd and compressed in place: outputs the
//          canonical V:N:M y2 (vals, meta, colidx), y1 at the kept slots (ykept, same indexing as vals), the plain
//          2:4 view (v24, m24; blocked layout) and the transposed y2v compacted to the four kept hidden units of every
//          (64-token block, group of 8) (at; [F / 2, T], blocked layout; see gemm_wgrad.hip).
//   mode 2 (eq. (4) -> eq. (6)): the tile of dy2 meets (meta, colidx, ykept) and becomes dy1 in y2's slots: outputs
//          vals (= dy1 values), v24 / m24 and at as above.
//   store_dense: also write the dense GEMM output (y1 / dy2) to `out`.
struct VnmEpilogue {
    int mode = 0;                   // 0: no V:N:M epilogue, only the dense output
    int store_dense = 1;
    uint16_t* vals = nullptr;
    uint8_t* meta = nullptr;
    uint8_t* colidx = nullptr;
    uint8_t* kmask = nullptr;       // mode 1: one byte per (64-token block, group of 8): bit c = column c of the group is kept
    uint16_t* ykept = nullptr;
    uint16_t* v24 = nullptr;
    uint8_t* m24 = nullptr;
    uint16_t* at = nullptr;
    // mode 3 (Section 3.3, neuron-level experts; grouped launch, A = one expert's hidden units in compact-column order):
    //        the tile of y1c gets the bias of its hidden units, is squared-ReLU'd and 2:4-pruned on every four consecutive
    //        compact columns: outputs vals, meta; padding rows (perm < 0) come out as zeros; `out` = y1c [rows, F] if store_dense.
    // mode 4 (the same experts, backward): the tile of dy2c meets (meta, ykept = the stored y1c [rows, F]) and becomes dy1 in y2's
    //        slots: outputs vals (canonical) and v24 (the same, blocked); `out` = dy2c if store_dense.
    //        Both, with `at`: the survivors as a dense transposed matrix [F, at_ld tokens], blocked, zeros at the dropped positions.
    // mode 5 / 6 (blocks of M = 2^logM = 16, 32, 64 columns, Table 5): as modes 1 / 2 with outputs vals, meta, colidx (mode 5), ykept
    //        ([T/64][F/64][64 tokens][64/M blocks] pairs), `at` + kmask (mode 5) exactly as for modes 1 / 2 (a block of M columns keeps 4, so no
    //        group of 8 hidden units keeps more than 4); no v24 / m24 (eqs. (3), (7) gather the kept rows of the dense operand from the
    //        canonical arrays).
    const int32_t* perm = nullptr;
    int logM = 3;
    // fp8 operands (launch_gemm_fp8_blocked, modes 1 / 2): the survivors leave as E4M3 codes quantised with 1 / scale = inv_out: mode 1 writes
    // vals as codes [T, F / 4], mode 2 keeps vals = dy1 in bf16; both write the codes into vcb.  ykept, at, kmask, colidx, meta stay as in the bf16 modes.
    // fp8 modes 5 / 6: vals = the survivors' codes [T, 2 F / M] in both directions (the operand of the gathered-row kernel); the rest as above.
    float inv_out = 1.0f;
    int at_fp8 = 0;                 // fp8 modes 1 / 2: `at` receives codes (pairs in the blocked layout, [F / 2, T]) instead of bf16
    float* amax = nullptr;          // fp8 modes 1 / 2: amax slots for the survivors' magnitudes (y2 / dy1)
    // modes 1 / 2: the operands of the V:2:8 activation GEMM (gemm_vnm8.hip; layouts: vcb_off, mcb_off, cixt_off in common.hpp, fp8: vcb8_off, ...):
    // vcb = the survivors (both modes; fp8: their codes), mcb = their metadata and cixt = the regrouped kept-column offsets (mode 1; mode 2 reuses them)
    int64_t at_ld = 0;
    int at_kept = 0;                // modes 5 / 6, bf16, M = 32, 64: `at` receives only the kept rows, in the order of gemm_wgrad_wide_body.hpp; no `kmask`
    uint16_t* vcb = nullptr;
    uint8_t* mcb = nullptr;
    uint8_t* cixt = nullptr;
};

// Grouped (mixture-of-experts) form of a contraction: the token axis is cut into n consecutive segments, one per
// expert (offsets seg[0] = 0 <= ... <= seg[n] = all tokens, multiples of 64), and each segment meets its own
// expert's weight operand.  `role` says which axis of the NT contraction the tokens are:
//   0: the i rows (A is token-indexed, B is the expert's weight matrix, out rows are tokens);
//   1: the j rows (A is the expert's packed weight matrix, B is token-indexed);
//   2: the contraction axis (A and B are [., all tokens] matrices, every expert gets its own output).
// Strides are per expert, in elements of the pointed-to type.  Token-indexed tensors always carry all tokens.
struct GemmGroup {
    static constexpr int kMaxExperts = 64;
    int n = 0;                      // 0: ordinary single contraction
    int role = 0;
    int64_t a_stride = 0, m_stride = 0, b_stride = 0, bias_stride = 0, out_stride = 0;
    // role 2 on row-major operands (weight gradients of the neuron-level experts, Section 3.3): output index i of expert e is
    // compact column i of its hidden units and lands at hidden unit (i / 4) * M + 4 e + i % 4 of the one shared output (0: off)
    int map_logM = 0;
    // roles 0 / none with the i-major output: row i goes to row out_row_map[i] of the output (negative: not stored)
    const int32_t* out_row_map = nullptr;
    // Segment offsets kept on the device (written by an earlier kernel of the same call, e.g. the router's grouping): when set,
    // the kernels read seg_dev[0..n] instead of seg[], and the launch is sized for the worst case of `cap_rows` token rows in n
    // runs (workgroups past the real tile count exit at once).  gemm_v2.hip kernels and the router's helpers only.
    const int32_t* seg_dev = nullptr;
    int64_t cap_rows = 0;
    int32_t seg[kMaxExperts + 1] = {0};
};

// arguments of the tile kernels' units (gemm_*_body.hpp; tiles_m / tiles_n are filled in at the launch)
struct GemmV2Args {
    const uint16_t* a_vals; const uint8_t* a_meta; const uint16_t* B; const float* bias;
    int Ra, Rb, K; uint16_t* out; int64_t ldo; int tiles_m, tiles_n; VnmEpilogue ep; GemmGroup grp; float alpha;
};
// Split: n workgroups per output tile, each on a range of the contraction (split.hpp); part: float32 sums, count: zeroed counters
struct Split { float* part = nullptr; unsigned* count = nullptr; int n = 1; };
struct Vnm8Args {
    const uint16_t* vcb; const uint8_t* mcb; const uint8_t* cixt; const uint8_t* Wk; int ldw, T, N, F; uint16_t* out; int64_t ldo; int tiles_m, tiles_n;
    GemmGroup grp; float alpha; Split split;
};
struct GatherArgs {
    const void* a_vals; const uint8_t* a_meta; const uint8_t* colidx; const void* Wk; int ldw, T, N, Kc, logM, tiles_n; float alpha; uint16_t* out; int64_t ldo; GemmGroup grp;
    Split split;
};
struct WgradArgs {
    const uint16_t* atc; const uint8_t* kmask; const uint16_t* G; float alpha; int F, N, T; uint16_t* out; int64_t ldo; int tiles_m, tiles_n; GemmGroup grp;
};

// Tiles of a step's contractions: g, g_bwd = eqs. (1), (4), v = eqs. (3), (7) (v_split workgroups each), w = eqs. (5), (8).  mix: the contractions that do not depend on each other
// share launches (sharing_pays, step_mix_*.hip): eqs. (3), (5), (4) in one and eqs. (7), (8) in another (a backward call: eqs. (5), (4), then (7), (8)).  Eq. (4) then takes the 128 tile
// and its results need operand buffers of their own, since eqs. (3), (5) still read those of eq. (1).
// v_alone: the tile of eq. (3) where it has a launch of its own all the same (forward calls); the same bits as on v.
struct StepTiles { int g = 0, g_bwd = 0, v = 0, v_alone = 0, v_split = 1, w = 0; bool mix = false; };
inline StepTiles step_tiles(int64_t T, int64_t D, int64_t F, int M, int experts, bool fp8, bool may_share = true);
enum { kMixForwardTail = 0, kMixBackwardHead = 1, kMixBackwardTail = 2 };      // {(3), (5), (4)}, {(5), (4)}, {(7), (8)}
// M = 8: v8 (else null: va); acc32: not with kMixForwardTail
hipError_t launch_step_mix_bf16(int what, int logM, const StepTiles& t, bool acc32, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s);
// (amax: with kMixBackwardTail, the fold of the step's maxima in the same launch)
struct AmaxFold { const float* p[6]; int n[6], stride[6]; float* out; int count; };
hipError_t launch_amax_fold(const AmaxFold& a, hipStream_t s);
hipError_t launch_step_mix_fp8(int what, int logM, const StepTiles& t, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s,
                               const AmaxFold* amax = nullptr);

// The passes that only depend on the step's inputs, in one launch (prologue.hip): the blocked copies of X and dY and their transposes, the pruning of W1
// and W2.  Absent parts: null X / dY / W1 / W2.  experts: W1, W2 are stacks of that many matrices.
struct PrologueArgs {
    int T, D, F, experts, mode;
    int t_layout;                   // of xt, dyt: 1 = blocked, 2 = lane_off (common.hpp)
    const uint16_t *X, *dY; uint16_t *xt, *xb, *dyt, *dyb;
    const uint16_t* W1; uint16_t *w1v, *w1vb; uint8_t *w1m, *w1mb;
    const uint16_t* W2; uint16_t *w2v, *w2vb, *w2t; uint8_t *w2m, *w2mb;
    unsigned* counters;             // kSplitCounters of them are cleared, or null
};
hipError_t launch_step_prologue(const PrologueArgs& a, hipStream_t s);
// The step's preparing passes: all in one launch while X, dY, W1 and W2 together stay below 96 MiB, else in three parts (X and W1 | W2 | dY)
inline bool prologue_together(int64_t T, int64_t D, int64_t F, int64_t E) { return 2 * (2 * T * D + 2 * E * F * D) < ((int64_t)96 << 20); }
// Eq. (1) with X row-major and the passes `behind` in the same launch (forward_x.hip); tile 64 or 128.
hipError_t launch_forward_x(const uint16_t* a_vals, const uint8_t* a_meta, const float* bias, const uint16_t* X, uint16_t* out, const VnmEpilogue& ep,
                            const PrologueArgs& behind, hipStream_t s, const GemmGroup* grp, int tile);
// Taken on both: what the row-major rows cost the loop (128-byte lines instead of 1 KB blocks) is less than a launch in front of it.  Forward calls on packed weights, 160
// shapes 0.88 of the time with the copy of X, none above 1.00: T = 64, D = 2048, F = 8192 40.7 us with the copy, 37.7 without; T = 4096, D = 256, F = 1024 22.1 / 17.9; T = 16320,
// D = 704, F = 2304, M = 16 101 / 97; M = 64, T = 4096, D = 512, F = 2048 27.3 / 20.6.  But the 64 tile of M = 64 (128 hidden units to a wavefront, two stages) does
// not cover the longer loads where the weights do not come from L2 (T = 64, F = 6144, D = 3072 37.0 / 36.3, D = 3584 41.8 / 43.2; F = 8192, D = 2560 38.2 / 41.3; T = 128, F = 4096,
// D = 3328 38.5 / 36.5, D = 4352 45.0 / 46.3).
// With weights to prune up to 6 Mi elements of tokens and weights, 3.5 Mi on 64 tiles: behind the tiles the pass over W2 runs two workgroups a CU (64 tiles: one),
// which is less than its rate alone.  A whole step: T = 512, D = 448, F = 1728 38 / 35 us; T = 64, D = 768, F = 2880 44 / 41; T = 128, D = 1088, F = 4096, M = 64
// 61 / 64; T = 128, D = 1216, F = 5120, M = 16 53 / 58; T = 128, D = 1856, F = 6080 86 / 98.
inline bool forward_reads_x(int64_t T, int64_t D, int64_t F, int M, bool packed, int tile) {
    if (tile == 256 || (M == 64 && tile == 64 && (T + 64) * D * F > 2650000000)) return false;
    return packed || (T + F) * D <= ((int64_t)(tile == 64 ? 7 : 12) << 19);
}
// The same for the fp8 step (prologue_fp8.hip).  t_codes: xt, dyt as codes instead of bf16.  Canonical codes / metadata (w1c, w1m, w2c, w2m) may be null.
// amax_*: one float per workgroup of the part (fp8_parts: x and dy have as many), slots_*: the epilogues' slots, cleared by the parts over X / dY; null: not wanted.
struct Fp8PrologueArgs {
    int T, D, F, experts, mode, t_codes;
    float inv_x, inv_dy, inv_w1, inv_w2;
    const uint16_t *X, *dY; uint8_t *xt, *xq, *dyt, *dyq;
    const uint16_t* W1; uint8_t *w1c, *w1m, *w1b, *w1mb, *w1q;
    const uint16_t* W2; uint8_t *w2c, *w2m, *w2b, *w2mb, *w2q;
    float *amax_x, *amax_w1, *amax_w2, *amax_dy, *slots_y2, *slots_dy1;
    unsigned* counters;             // as above
};
struct Fp8Parts { int x, w1, w2; };
Fp8Parts fp8_parts(int64_t T, int64_t D, int64_t F, int64_t experts);
hipError_t launch_fp8_prologue(const Fp8PrologueArgs& a, hipStream_t s);

// Edge of the square output tile of a contraction with n256 / n128 / n64 tiles of each size and `steps` trips of its main loop.  A round = one tile on
// every slot of the chip: 256 tiles of 256 x 256 (one workgroup per CU), 512 of 128 x 128 (two per CU).  A round of small tiles takes `w128` of a round of
// large ones (measured, see below: more bytes from L2 per product), so the large tile wins on whole rounds and the small one where the
// outputs do not fill the chip or leave the last round nearly empty.  64 x 64 tiles split the contraction over their four wavefronts: best
// while there are at most `most64` of them and the contraction is long enough to be worth splitting.  last: what a last round of small tiles takes, as a
// part of a full one, when it leaves every workgroup a CU of its own; slope: and from there in line up to a full one.
inline int pick_tile(float rounds256, unsigned n128, unsigned n64, int steps, float w128, unsigned most64, int least_steps, float last = 1.0f, bool slope = false) {
    if (n64 <= most64 && steps >= least_steps) return 64;
    const unsigned rest = n128 % 512;
    const float part = rest == 0 ? 0.0f : rest <= 256 ? last : slope ? last + (1.0f - last) * (float)(rest - 256) / 256.0f : 1.0f;
    return w128 * ((float)(n128 / 512) + part) < rounds256 ? 128 : 256;
}
inline float large_rounds(unsigned n256) { return (float)((n256 + 255) / 256); }

// tiles along the tokens when they come in `groups` segments (0: one), taken as equally long: a host and a device segment table choose alike
inline int64_t token_tiles(int64_t T, int groups, int64_t edge) {
    const int64_t n = groups ? groups : 1;
    return n * (((T + n - 1) / n + edge - 1) / edge);
}
// What a round of 128 tiles takes of a round of 256 tiles in gemm_v2, by the trips of the main loop: plain stores, or the V:N:M epilogues of eqs. (1) and
// (4), whose part of a tile overlaps with the other workgroup's main loop (the router's are shorter).  The longer the contraction the more the bytes from L2
// count, of which the small tile needs twice as many per product.  Fitted to 400 shapes (T 64 - 16000, D 256 - 6000, 1 - 8 experts; bf16, and fp8 by its own
// trips of 128, with weights of its own), over which what is chosen takes 0.05 - 0.1 % longer than the better tile of each.  Some of them, on 256 / 128 tiles:
//   eq. (1)  T = 5504, D = 768, F = 3072 43 / 37 us; T = 8192, D = 960, F = 3008 57 / 57; T = 2816, D = 2624, F = 7488 92 / 97; 8 x 512 tokens, D = 3840,
//            F = 12672 292 / 370
//   eq. (4)  33 / 31; 54 / 59; 79 / 91; 285 / 371
//   fp8      eq. (1) T = 3072, D = 3712, F = 11136 132 / 123; T = 6784, D = 2560, F = 7936 147 / 142; eq. (4) T = 9152, D = 1408, F = 3712 69 / 65
//   M = 16   eq. (4) T = 2560, D = 1984, F = 7936 67.5 / 63.0
//   router   T = 8192, D = 2048, F = 8192, M = 16 95 / 86, eq. (4) 94 / 92; T = 4096, D = 4096, F = 16384 147 / 161, 149 / 160
//   plain    26 trips 0.71, 46 0.73, 64 0.76 - 0.80, 86 0.89, 114 0.94 (T = 8000, N = 2560, K = 7296: 239 / 293 us)
// last_round: what the last round takes when it has at most 256 small tiles, one per CU (plain stores: 0.6 up to 48 trips, the router's eq. (3), 288 / 1120 tiles
// of K = 2048: 76 / 68 us; T = 8000, N = 2560, K = 7296 has 320 / 1260).
// Blocks of M = 64 columns want 128 hidden units in one wavefront, so that their small tile is 256 hidden units x 128 tokens (`tall`): a round of them, two
// per CU, is about the work of one of 256 tiles, and alone on its CU such a tile takes 0.85 - 1.1 of a 256 tile (bf16: 5 trips 0.91, 13 0.94, 33 0.98, eq.
// (4) 0.04 more; fp8: 2 trips 0.84, 14 0.87 - 0.9, 26 0.95).  Over 150 shapes what is chosen takes 0.02 % longer than the better tile (bf16) and 0.15 % (fp8):
// fp8 T = 8384, D = 1280, F = 4096 eq. (1) 64.4 us on 256, 59.0 on 256 x 128; T = 3392, D = 5120, F = 14336 190 / 172, eq. (4) 174 / 163; bf16 T = 11712,
// D = 1152, F = 3072 75.9 / 73.5; T = 2944, D = 4416, F = 18432 292 / 320.
enum { kGemmPlain = 0, kGemmForward = 1, kGemmBackward = 2, kGemmRouter = 3 };
inline float small_round(int what, int steps, int M = 8, bool fp8 = false) {
    const float n = (float)steps;
    float w;
    if (what == kGemmPlain) return n < 110.0f ? 0.68f + 0.002f * n : 0.90f;
    if (what == kGemmRouter) w = 0.53f + 0.0031f * n;
    else if (M == 64) return !fp8 ? 1.02f : n < 47.5f ? 0.96f + 0.004f * n : 1.15f;
    else if (what == kGemmForward) w = 0.50f + (fp8 ? 0.004f : 0.006f) * n;
    else w = fp8 ? 0.54f + 0.006f * n : M == 8 ? 0.62f + 0.006f * n : 0.56f + 0.004f * n;
    return w < 0.74f ? w : 0.74f;
}
inline float last_round(int what, int steps, int M = 8, bool fp8 = false) {
    if (what == kGemmPlain) return steps <= 48 ? 0.6f : 1.0f;
    if (what == kGemmRouter || M != 64) return fp8 ? 0.8f : 0.75f;
    return (fp8 ? 0.82f + 0.003f * (float)steps : 0.86f + 0.004f * (float)steps + (what == kGemmBackward ? 0.03f : 0.0f)) / small_round(what, steps, M, fp8);
}
// gemm_v2 (i x j outputs); w128, last: see pick_tile.  64 tiles: T = 64, D = 2048, F = 8192 (32 / 64 / 128 tiles): eqs. (1), (4) 43 / 33 us on 256 tiles,
// 21 / 18 on 128, 17 / 14 on 64; with more than 256 of them they lose to 128 (T = 128, D = 1984, F = 8512, 266 of them: 25 and 19 us).
inline int pick_gemm_tile(int64_t Ra, int64_t Rb, int steps, const GemmGroup& g, float w128, bool split, float last = 1.0f, bool tall = false) {
    auto tiles = [&](int64_t ei, int64_t ej) {
        return (unsigned)(token_tiles(Ra, g.n && g.role == 0 ? g.n : 0, ei) * token_tiles(Rb, g.n && g.role == 1 ? g.n : 0, ej) * (g.role == 2 && g.n ? g.n : 1));
    };
    return pick_tile(large_rounds(tiles(256, 256)), tiles(tall ? 256 : 128, 128), tiles(64, 64), steps, w128, split ? 256 : 0, 16, last);
}
// eqs. (1), (4) with their epilogues; M: columns per V:N:M block
inline int pick_epilogue_tile(int64_t F, int64_t T, int steps, const GemmGroup& g, int what, int M, bool fp8) {
    return pick_gemm_tile(F, T, steps, g, small_round(what, steps, M, fp8), true, last_round(what, steps, M, fp8), M == 64);
}
// V:2:8 activation GEMM.  The large tile is 512 tokens x 128 columns or 256 x 256 (gemm_vnm8.hip), 0.93 and 1 a round: four fifths of what a stage of the second
// fetches are the dense slab.  A round of 128 tiles, two per CU, takes more of that the longer the contraction, one per CU 0.86 at most (codes: 0.66).  Large /
// 128: T = 1600, N = 4864, F = 19584 (152 / 494 tiles) 369 us, 444; T = 2688, N = 2816, F = 9024 (126 / 462) 162, 170; T = 15360, N = 448, F = 1856 (120 / 480)
// 24 / 22; T = 896, N = 3904, F = 17280 (62 / 217) 1 / 0.75; T = 1792, N = 2816, F = 12096 (88 / 308) 1 / 0.86; T = 2048, N = 4800, F = 16896 (152 / 608) 1 / 1.49; codes, T = 3840, N = 2048, F = 7936 (120 / 480)
// 1 / 0.85.  Over 270 shapes what is chosen takes 0.2 % longer than the better of the two.  T = 1024, N = 1408, F = 4928 (24 / 88 / 352): 55, 33, and 29 on
// 64 tiles; T = 64, N = 2048, F = 8192 (8 / 16 / 32): 83, 49, 28.
// More than 256 of the 64 tiles: only for long contractions of bf16 (T = 256, N = 5824, F = 24704, 364 of them: 169 us, 192 on 128 tiles; 24 trips: a third
// slower than 128, 44: 15 %, 63 - 84: even, but in a shared launch 128 tiles are better up to there: T = 1664, D = 1216, F = 4032 the step 147 us, 106 on 128);
// fp8 loses to every other tile there (T = 4864, N = 384, F = 1408, 456 of them: 18.5 us, 10.6 on 128, 16.0 on 256).
inline float vnm8_rounds(unsigned n512, unsigned n256) { const float a = 0.93f * large_rounds(n512), b = large_rounds(n256); return a < b ? a : b; }
inline float vnm8_small_round(int steps, bool fp8) {
    const float w = fp8 ? 0.64f + 0.0012f * (float)steps : 0.63f + 0.0025f * (float)steps, most = fp8 ? 0.86f : 1.2f;
    return w < most ? w : most;
}
inline float vnm8_last_round(int steps, bool fp8) { const float w = vnm8_small_round(steps, fp8), last = fp8 ? 0.66f : 0.86f; return last < w ? last / w : 1.0f; }
inline int pick_vnm8_tile(int64_t T, int64_t N, int steps, int groups, bool fp8) {
    auto tiles = [&](int64_t edge) { return (unsigned)(token_tiles(T, groups, edge) * ((N + edge - 1) / edge)); };
    const float large = vnm8_rounds((unsigned)(token_tiles(T, groups, 512) * ((N + 127) / 128)), tiles(256));
    return pick_tile(large, tiles(128), tiles(64), steps, vnm8_small_round(steps, fp8), !fp8 && steps >= 84 ? 512 : 256, 8, vnm8_last_round(steps, fp8), true);
}
// gathered-row activation GEMM: 64 tokens x 256 columns, or 64 x 64
// (T = 256, N = 1024, F = 4096, M = 16: 19 us and 12 us; T = N = 1024: 20 and 12; T = 512, N = 4096, F = 16384: 90 and 67; T = 1984, N = 1344, M = 32: 14 and 23)
inline int pick_gather_tile(int64_t T, int64_t N, int steps) { return (T / 64) * ((N + 63) / 64) <= 512 && steps >= 6 ? 64 : 256; }

// Tile and number of workgroups per tile of eqs. (3), (7).  Estimated from what a stage of a tile takes (us): us64 for a 64 tile (one workgroup per
// CU, its four wavefronts together), 0.42 for a 128 tile alone on its CU, 0.58 for two of them; splitting costs 6 us and writes and reads
// `n` float32 copies of the output (at most kSplitMost bytes) at 4 TB/s.  Taken where that saves 15 % and more.  T = 64, N = 4096, F = 16384: 94 -> 38 us
// (4 splits; from HBM instead of the last-level cache: 90 -> 60), N = 2048, F = 8192: 28 -> 16 (8 splits); fp8: 40 -> 23; M = 16: 41 -> 22.  Not where eqs.
// (3), (7) share a launch: its workgroups fill the chip as it is (T = 192, N = 1024, F = 4096: the step 64 us, 74 with 5 splits).
// At most 1024 workgroups: with more, each with its start and its sums, the estimate is off (T = 384, N = 3072, F = 10752: 60 us undivided, 59 with 3 splits,
// 69 with 4; T = 256, N = 4736, F = 16320: 70, 72 and 80).
constexpr int64_t kSplitMost = (int64_t)32 << 20, kSplitMostGroups = 1024;
struct SplitPlan { int tile, n; };
inline SplitPlan plan_split(int64_t T, int64_t N, int steps, int tile, float us64) {
    auto tiles = [&](int64_t edge) { return ((T + edge - 1) / edge) * ((N + edge - 1) / edge); };
    auto cost = [&](int edge, int n) {
        const int64_t w = tiles(edge) * n;
        const float rounds = edge == 64 ? us64 * (float)((w + 255) / 256) : 0.58f * (float)(w / 512) + (w % 512 == 0 ? 0.0f : w % 512 <= 256 ? 0.42f : 0.58f);
        return rounds * (float)((steps + n - 1) / n) + (n > 1 ? 6.0f + (float)(tiles(edge) * edge * edge) * 8.0f * (float)n / 4.0e6f : 0.0f);
    };
    SplitPlan best = {tile, 1};
    if (tile == 256) return best;
    float least = 0.85f * cost(tile, 1);
    for (int n = 2; n <= 16 && steps / n >= 8 && tiles(64) * n <= kSplitMostGroups && tiles(64) * 64 * 64 * 4 * n <= kSplitMost; ++n) {
        const float c = cost(64, n);
        if (c < least) { least = c; best = {64, n}; }
    }
    return best;
}
inline SplitPlan plan_vnm8(int64_t T, int64_t N, int steps, int groups, bool fp8) {
    const int tile = pick_vnm8_tile(T, N, steps, groups, fp8);
    return groups ? SplitPlan{tile, 1} : plan_split(T, N, steps, tile, 0.205f);
}
inline SplitPlan plan_gather(int64_t T, int64_t N, int steps, int groups) {
    const int tile = pick_gather_tile(T, N, steps);
    return groups ? SplitPlan{tile, 1} : plan_split(T, N, steps, tile, 0.5f);
}
// bytes of the sums and, behind them, of the counters (one per tile: with 2 and more splits of 8 and more stages there are at most kSplitMost / 32 KB)
inline size_t split_part_bytes(const SplitPlan& p, int64_t T, int64_t N) {
    return p.n > 1 ? (size_t)(((T + p.tile - 1) / p.tile) * ((N + p.tile - 1) / p.tile)) * p.tile * p.tile * 4 * p.n : 0;
}
constexpr int kSplitCounters = 1024;
inline size_t split_bytes(const SplitPlan& p, int64_t T, int64_t N) { return p.n > 1 ? split_part_bytes(p, T, N) + kSplitCounters * sizeof(unsigned) : 0; }
inline Split split_at(void* p, const SplitPlan& plan, int64_t T, int64_t N) {
    Split s;
    if (plan.n > 1) { s.part = (float*)p; s.count = (unsigned*)((unsigned char*)p + split_part_bytes(plan, T, N)); s.n = plan.n; }
    return s;
}
// weight gradients.  F = 8192, N = 2048, T = 2048 (256 / 1024 tiles): 55 us on 256 tiles, 60 on 128; F = 4096, N = 1024, T = 8192 (64 / 256 / 1024): 145, 65,
// and 91 on 64 tiles; F = 1024, N = 256, T = 16384 (4 / 16 / 64): 277, 109, 39
inline int pick_wgrad_tile(int64_t F, int64_t N, int64_t T, int experts, bool split_ok) {
    const unsigned e = experts ? (unsigned)experts : 1u;
    auto tiles = [&](int64_t edge) { return (unsigned)((F + edge - 1) / edge * ((N + edge - 1) / edge)) * e; };
    return pick_tile(large_rounds(tiles(256)), tiles(128), tiles(64), (int)(T / 64 / e), 0.58f, split_ok ? 256 : 0, 12);
}

// Weight gradients of few tokens, bf16, launches of their own: 128 tiles on a ring of two stages, three workgroups a CU (768 tiles at a time), so that the stores of one
// tile run under the loads of two others.  A tile of few stages is mostly its start and its stores: T = 64, N = 7040, F = 23552 85 / 82 us on 256 tiles / 128 tiles of three
// stages, 62 on this form; T = 256 119 / 122, 101; T = 512, N = 1728, F = 5504 18 / 17, 16; T = 1024, N = 4032, F = 13440 101 / 102, 96; into float32 T = 384, N = 4608,
// F = 20160 174 / 170, 158.  Tiles that two workgroups a CU hold at once gain nothing (T = 448, N = 704, F = 2432, 114 of them: 13 / 7.4 / 8.3; 374 at T = 512: 16 / 12.2 / 11.9), nor does it pay where large
// tiles just fill their rounds (T = 768, N = 1920, F = 7296, 232 of them: 23.0 / 24.7 / 25.9; T = 1280, N = 2944, F = 10368, 492: 65 / 69 / 69).  Above 20 token blocks not measured but for
// T = 1984, N = 4096, F = 14336 (178 / 177 / 174) and T = 4096, N = 2048, F = 8192 (93 / 104 / 109).  Not for experts, whose tiles are of different lengths (8 of 630
// tokens on average, D = 1536, F = 4992: the step 591 us, 606 with it).  Codes: 200 registers, two workgroups a CU; with 168 they spill (T = 1216, a whole step a quarter slower).
// The order of the sums is that of the other tiles: same bits.
inline bool wgrad_three_a_cu(int64_t F, int64_t N, int64_t T, int experts, int tile) {
    auto tiles = [&](int64_t edge) { return (unsigned)((F + edge - 1) / edge * ((N + edge - 1) / edge)); };
    const unsigned n = tiles(128), rest = n % 768;
    if (experts || tile == 64 || T > 1280 || n <= (T > 512 ? 512u : 320u)) return false;
    if (tile == 128) return true;
    // a round of 768 in rounds of 256 large tiles; the last one takes less where it leaves the workgroups of a CU alone
    const float rounds = (float)(n / 768) + (rest == 0 ? 0.0f : rest <= 256 ? 0.65f : rest <= 512 ? 0.9f : 1.0f);
    return rounds * (0.68f + 0.07f * (float)T / 768.0f) < large_rounds(tiles(256));
}

// Weight gradients on the kept rows only (gemm_wgrad_wide_body.hpp; bf16, launches of their own), from 320 tokens per expert on: with fewer the matrix work that
// is saved is less than clearing a tile in LDS and reading it out again (F = 16384, N = 4096, M = 32: 50 us for 50 at 256 tokens, 51 for 54 at 320, 173 for 354 at 4096;
// M = 64: 43 for 45 at 192; F = 8192, N = 2048, M = 32: 17.9 for 17.4 at 256, 17.9 for 18.4 at 320, 22.4 for 30.7 at 1024).
inline bool wgrad_on_kept_rows(int64_t T, int64_t F, int M, int64_t experts) { return M >= 32 && F % (8 * M) == 0 && T >= 320 * experts; }

// Do eqs. (3), (5), (4) and (7), (8) take less time as two launches than as five?  Both are estimated (us).  A launch by itself takes `start` and its rounds
// over the chip, 256 large or 512 small tiles at a time (a last round of fewer less than a full one), or the time of the weights' bytes where few
// tokens meet them.  A shared launch takes the sum of its small tiles spread over the chip and `end` of the last unit's tile; no less than `lone` of a tile behind
// what comes before it, nor than the bytes of all its units.  Tiles and splits are those that the separate launches have.  Eqs. (5), (8) of bf16 blocks of 32 and
// 64 columns multiply the kept rows only where they have launches of their own, 8 and 16 times fewer products: M = 64, T = 11520, D = 896, F = 2048 the step 172 us apart,
// 286 together; T = 7680, D = 832, F = 3072 142 / 210; M = 32, T = 5312, D = 1152, F = 3584 148 / 185; small ones share all the same (M = 64, T = 1280, D = 448,
// F = 2048 51 / 44).
// The constants are fitted to whole steps of 28000 drawn shapes (T 64 - 16384, D 256 - 8192, 1 - 32 experts of uneven length, every M, bf16 and codes), each run both
// ways.  Over 4000 others what is chosen takes 0.10 % longer than the better form (one expert 0.10 % in bf16, 0.04 % on codes), one call in 180 4 % and more, the
// worst 12 %; always sharing would take 2.3 % longer, never 16 %.  Over 487 measured apart from both: 0.18 %, forward and backward calls after one another, whose eq. (3)
// has a launch of its own as in a step with float32 accumulation, 0.11 %.  T = 1984, D = 1344, F = 4160 167 us apart, 140 together; codes, T = 6848, D = 2304, F = 8192
// 671 / 686.  Near even it errs either way, mostly where 64 - 640 tokens meet large weights (T = 192, D = 5504, F = 17408, M = 32 497 / 536, shared) and on experts, whose
// lengths it does not know (8 of them, T = 640, D = 1600, F = 6720 419 / 465, shared); the worst have splits to lose (see step_tiles).
struct StepCosts {
    struct Line { float fixed, step; float operator()(float steps) const { return fixed + step * steps; } };       // us of a tile, and of it per trip of its main loop
    float start;
    struct { float v, w, g, g_tall; } lone;             // by unit: eqs. (3) / (7), (5) / (8), (4), (4) at M = 64
    struct { float v, w, g; } end;
    struct { float v, rows, g, w; } last;               // a last round of at most 256 small tiles: M = 8, M >= 16 in eqs. (3), (7), eq. (4), eqs. (5), (8)
    float knee, part;                                   // ... of just over 256; a last round of a few large tiles
    float two_v, two_w;                                 // a 64 tile in a shared launch, as a part of a 128 tile's slot
    struct { float v, g, w, all; } bytes;               // us per million weights read or written; all: of a shared launch's units together
    Line large4, large4_mid, large4_tall, small4, small4_mid, tall4, tiny4;        // 256 (M = 8; 16, 32; 64), 128 (two a CU; M = 8; 16, 32), M = 64: 256 x 128 (two a CU), 64
    Line large3, small3, tiny3, rows3, tiny_rows3;      // M = 8: 512 x 128 or 256, 128, 64; M >= 16: 64 x 256 (two a CU), 64
    Line large5, small5, tiny5, kept32, kept64;         // 256, 128, 64; on the kept rows
};
constexpr StepCosts kStepBf16 = {3.34f, {0.51f, 0.556f, 0.869f, 0.968f}, {0.402f, 0.411f, 0.436f}, {0.664f, 0.788f, 0.653f, 0.591f}, 0.882f, 0.856f, 2.69f, 1.98f, {0.263f, 0.285f, 0.485f, 1.12f},
                                 {8.92f, 0.722f}, {11.6f, 0.825f}, {7.85f, 0.511f}, {5.16f, 0.407f}, {4.99f, 0.639f}, {4.73f, 0.86f}, {11.8f, 0.0731f},
                                 {15.4f, 0.632f}, {2.0f, 0.69f}, {3.59f, 0.103f}, {3.2f, 1.49f}, {4.31f, 0.338f}, {6.46f, 1.17f}, {4.09f, 0.63f}, {4.46f, 0.164f}, {5.62f, 0.201f}, {7.12f, 0.229f}};
constexpr StepCosts kStepFp8 = {4.84f, {0.421f, 0.727f, 1.24f, 0.658f}, {0.297f, 0.255f, 0.254f}, {0.618f, 0.683f, 0.639f, 0.631f}, 1.0f, 0.942f, 2.75f, 1.9f, {0.247f, 0.26f, 0.452f, 1.03f},
                                 {11.8f, 0.858f}, {16.0f, 0.776f}, {13.6f, 0.8f}, {6.33f, 0.52f}, {7.82f, 0.545f}, {8.93f, 0.977f}, {1.9f, 0.15f},
                                 {11.0f, 0.608f}, {3.16f, 0.586f}, {3.4f, 0.206f}, {2.86f, 1.28f}, {4.0f, 0.38f}, {6.57f, 0.503f}, {4.15f, 0.29f}, {3.27f, 0.0483f}, {}, {}};
// t: the tiles of the separate launches; v: that of eqs. (3), (7) in the shared ones (256: the next smaller there)
inline bool sharing_pays(int64_t T, int64_t D, int64_t F, int M, int groups, bool fp8, const StepTiles& t, int v) {
    const StepCosts& c = fp8 ? kStepFp8 : kStepBf16;
    const int unit = fp8 ? 128 : 64, e = groups ? groups : 1;
    const float sg = (float)(D / unit), sv = (float)(M == 8 ? F / unit : 4 * F / M / unit), sw = (float)T / 64.0f / (float)e;
    auto across = [](int64_t n, int64_t edge) { return (float)((n + edge - 1) / edge); };
    // tiles along the tokens: experts end anywhere in their last tile, half a tile on average
    auto tokens = [&](int64_t edge) { return groups ? (float)T / (float)edge + 0.5f * (float)groups * (1.0f - 64.0f / (float)edge) : across(T, edge); };
    auto large = [&](float n) {
        const float all = ceilf(n), full = floorf(all / 256.0f), rest = all - 256.0f * full;
        return rest == 0.0f ? full : full + c.part + (1.0f - c.part) * rest / 256.0f;
    };
    auto small = [&](float n, float last) {
        const float all = ceilf(n), full = floorf(all / 512.0f), rest = all - 512.0f * full;
        return rest == 0.0f ? full : rest <= 256.0f ? full + last : full + last + (1.0f - last) * (c.knee + (1.0f - c.knee) * (rest - 256.0f) / 256.0f);
    };
    auto more = [](float a, float b) { return a > b ? a : b; };
    struct Unit { float tile, tiles, lone, end; };                      // of the shared launches
    const float weights = (float)(D * F * e) * 1e-6f;
    float alone3, alone4, alone5;
    Unit u3, u4, u5;
    {
        const StepCosts::Line big = M == 8 ? c.large4 : M == 64 ? c.large4_tall : c.large4_mid, two = M == 8 ? c.small4 : M == 64 ? c.tall4 : c.small4_mid;
        const float n = across(F, M == 64 ? 256 : 128) * tokens(128);
        u4 = {two(sg), n, M == 64 ? c.lone.g_tall : c.lone.g, c.end.g};
        alone4 = t.g_bwd == 256 ? large(across(F, 256) * tokens(256)) * big(sg) : t.g_bwd == 128 ? small(n, c.last.g) * u4.tile : large(across(F, 64) * tokens(64)) * c.tiny4(sg);
    }
    float rows = 1.0f;                                                  // the part of the weights that any token block keeps
    if (M == 8) {
        const float n = across(D, 128) * tokens(128), n64 = across(D, 64) * tokens(64);
        const float n512 = 0.93f * large(across(D, 128) * tokens(512)), n256 = large(across(D, 256) * tokens(256));
        alone3 = t.v == 256 ? (n512 < n256 ? n512 : n256) * c.large3(sv) : t.v == 128 ? small(n, c.last.v) * c.small3(sv) : large(n64 * (float)t.v_split) * c.tiny3(sv / (float)t.v_split);
        u3 = v == 64 ? Unit{c.two_v * c.tiny3(sv), n64, c.lone.v, c.end.v} : Unit{c.small3(sv), n, c.lone.v, c.end.v};
    } else {
        const float n = across(T, 64) * across(D, 256), n64 = across(T, 64) * across(D, 64);
        alone3 = t.v == 256 ? small(n, c.last.rows) * c.rows3(sv) : large(n64 * (float)t.v_split) * c.tiny_rows3(sv / (float)t.v_split);
        u3 = v == 64 ? Unit{c.two_v * c.tiny_rows3(sv), n64, c.lone.v, c.end.v} : Unit{c.rows3(sv), n, c.lone.v, c.end.v};
        rows -= powf(1.0f - 4.0f / (float)M, more(sw, 1.0f));
    }
    {
        const float n = (float)e * across(F, 128) * across(D, 128), n64 = (float)e * across(F, 64) * across(D, 64);
        if (!fp8 && wgrad_on_kept_rows(T, F, M, e)) alone5 = large((float)e * across(F, 512) * across(D, 64)) * (M == 32 ? c.kept32(sw) : c.kept64(sw));
        else alone5 = t.w == 256 ? large((float)e * across(F, 256) * across(D, 256)) * c.large5(sw) : t.w == 128 ? small(n, c.last.w) * c.small5(sw) : large(n64) * c.tiny5(sw);
        u5 = t.w == 64 ? Unit{c.two_w * c.tiny5(sw), n64, c.lone.w, c.end.w} : Unit{c.small5(sw), n, c.lone.w, c.end.w};
    }
    if (t.v_split > 1) alone3 += 1.5f;
    const float b3 = c.bytes.v * weights * rows, b4 = c.bytes.g * weights, b5 = c.bytes.w * weights;
    auto shared = [&](std::initializer_list<Unit> units, float bytes) {
        float before = 0.0f, last = 0.0f;
        for (const Unit& u : units) {
            const float work = u.tiles * u.tile / 512.0f;
            last = more(last, before + more(u.lone * u.tile, work + u.end * u.tile));
            before += work;
        }
        return c.start + more(last, c.bytes.all * bytes);
    };
    return shared({u3, u5, u4}, b3 + b4 + b5) + shared({u3, u5}, b3 + b5) < 5.0f * c.start + more(alone4, b4) + 2.0f * (more(alone3, b3) + more(alone5, b5));
}

// may_share: false where the shared launches are not built for the call
inline StepTiles step_tiles(int64_t T, int64_t D, int64_t F, int M, int experts, bool fp8, bool may_share) {
    StepTiles t;
    const int unit = fp8 ? 128 : 64, steps = (int)(D / unit);
    GemmGroup g;
    g.role = 1; g.n = experts > 1 ? experts : 0;
    t.g = pick_epilogue_tile(F, T, steps, g, kGemmForward, M, fp8);
    t.g_bwd = pick_epilogue_tile(F, T, steps, g, kGemmBackward, M, fp8);
    // (the gathered-row kernel on codes has the 256-column tile only, so wide fp8 blocks neither take 64 x 64 tiles nor split: not built)
    const SplitPlan v = M == 8 ? plan_vnm8(T, D, (int)(F / unit), g.n, fp8) : fp8 ? SplitPlan{256, 1} : plan_gather(T, D, (int)(4 * F / M / 64), g.n);
    t.v = M == 8 ? pick_vnm8_tile(T, D, (int)(F / unit), g.n, fp8) : fp8 ? 256 : pick_gather_tile(T, D, (int)(4 * F / M / 64));
    t.w = pick_wgrad_tile(F, D, T, experts > 1 ? experts : 0, M == 8 || fp8);
    const int v_shared = t.v;
    t.v = v.tile; t.v_split = v.n;
    // Shared launches do not split eqs. (3), (7), and calls of either pass alone have to sum as the whole step does: a forward call would lose its split (T = 64, D = 2048,
    // F = 6784: the step 89 us apart, 84 together, a forward call on packed weights 25 and 34).  So steps with splits share only where no contraction wants the large tile,
    // which is where they gain most (T = 64, D = 960, F = 4224: 62 / 47, the forward call 21 / 23).
    const bool loses_split = v.n > 1 && (t.w == 256 || pick_gemm_tile(F, T, steps, g, 0.56f, true) == 256);
    t.mix = may_share && !loses_split && sharing_pays(T, D, F, M, g.n, fp8, t, v_shared);
    t.v_alone = t.mix ? v_shared : v.tile;
    if (t.mix) {
        t.g_bwd = 128;
        t.v = M == 8 && v_shared == 256 ? 128 : v_shared; t.v_split = 1;
        if (t.w == 256) t.w = 128;
    }
    return t;
}

// the same once the experts' segments are known: 256 or 128 by the exact number of tiles (the two give the same bits; sharing launches and splitting
// contractions were decided from the sizes alone, and shared launches keep their tiles).  8 experts x 128 tokens, D = 3840, F = 12672: eqs. (3), (7) 181, 138 us on 128 tiles, 221, 191 on 256.
inline void refine_tiles(StepTiles* t, int64_t D, int64_t F, int M, const GemmGroup& g, bool fp8) {
    if (!g.n) return;
    auto count = [&](int64_t other, int64_t other_edge, int64_t edge) {
        int64_t n = 0;
        for (int e = 0; e < g.n; ++e) n += (g.seg[e + 1] - g.seg[e] + edge - 1) / edge;
        return (unsigned)(n * ((other + other_edge - 1) / other_edge));
    };
    auto pick = [&](int what) {
        const int steps = (int)(D / (fp8 ? 128 : 64));
        return pick_tile(large_rounds(count(F, 256, 256)), count(F, M == 64 ? 256 : 128, 128), ~0u, 0, small_round(what, steps, M, fp8), 0, 0, last_round(what, steps, M, fp8));
    };
    if (t->g != 64) t->g = pick(kGemmForward);
    if (t->g_bwd != 64 && !t->mix) t->g_bwd = pick(kGemmBackward);
    if (M == 8 && t->v != 64) {
        const int steps = (int)(F / (fp8 ? 128 : 64));
        t->v_alone = pick_tile(vnm8_rounds(count(D, 128, 512), count(D, 256, 256)), count(D, 128, 128), ~0u, 0, vnm8_small_round(steps, fp8), 0, 0, vnm8_last_round(steps, fp8), true);
        if (!t->mix) t->v = t->v_alone;
    }
}

// Does the router's step share launches?  Where eqs. (1), (4) and (3), (7) all run on 128 tiles.  Grouped by expert they have a few tiles more than fill the
// chip, so that the last round of each is nearly empty: T = 8192, D = 2048, F = 8192, M = 16 (1056 tiles each, 512 at a time) eqs. (4) and (3) 90 + 68 us apart,
// 137 together; eq. (7) and the transpose of dW2 72 + 12, 77; the step 542 / 522; T = 1792, D = 640, F = 1920, M = 8 110 / 94; T = 128, D = 704, F = 2560,
// M = 16 90 / 78.  Of 100 drawn calls 57 share, in 0.90 of the time apart, the slowest 1.02 (T = 13952, D = 1216, F = 5248, M = 8 734 / 748).  Up to 48 Mi elements of tokens and weights: the passes that ride along run two workgroups a CU, which
// is less than their rate alone (T = 320, D = 4928, F = 21888, M = 8 811 us apart, 894 together).
inline bool router_shares(int64_t rows, int64_t D, int64_t F, int M) {
    if ((rows + F) * D > ((int64_t)48 << 20)) return false;
    GemmGroup g;
    g.n = M / 4; g.role = 1;
    const int64_t Kc = 4 * F / M;
    const int steps = (int)(D / 64), steps3 = (int)(Kc / 64);
    if (pick_gemm_tile(Kc, rows, steps, g, small_round(kGemmRouter, steps), true, last_round(kGemmRouter, steps)) != 128) return false;
    g.role = 0;
    return pick_gemm_tile(rows, D, steps3, g, small_round(kGemmPlain, steps3), true, last_round(kGemmPlain, steps3)) == 128;
}

hipError_t launch_prune24(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, int mode, uint16_t* vals,
                          uint8_t* meta, hipStream_t stream);
hipError_t launch_dsqrelu_vnm(const uint16_t* dy2, const uint16_t* y1, const uint8_t* meta, const uint8_t* colidx,
                              int64_t T, int64_t F, uint16_t* dvals, hipStream_t s);
// 2:4 prune-and-pack: canonical outputs plus the blocked copies the GEMMs read
hipError_t launch_prune24_step(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, int mode, uint16_t* vals,
                               uint8_t* meta, uint16_t* vblk, uint8_t* mblk, hipStream_t stream,
                               int cluster_M = 0);    // cluster_M (trans = 0): rows come out expert-major, see scans.hpp
// vnm_general.hip: the stand-alone compressor for M in {8, 16, 32, 64}, and eq. (6) / 2:4 re-expression / transposed expansion for M in {16, 32, 64}.
hipError_t launch_sqrelu_vnm_compress_m(const uint16_t* y1, int64_t T, int64_t F, int M, uint16_t* vals, uint8_t* meta, uint8_t* colidx,
                                        hipStream_t s);
hipError_t launch_dsqrelu_vnm_m(const uint16_t* dy2, const uint16_t* y1, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F,
                                int M, uint16_t* dvals, hipStream_t s);
hipError_t launch_vnm_to_24_m(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M,
                              uint16_t* vals24, uint8_t* meta24, hipStream_t s);
hipError_t launch_vnm_expand_t_m(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M,
                                 uint16_t* out, hipStream_t s);
// eqs. (3), (7) with the rows of the dense operand gathered per token block (gemm_gather.hip):
// out[t, n] = sum over the kept columns f of A[t, f] * Wk[f, n]; Wk = [F, ldw] (contraction index = row).
// vnm_spmm_gather_ok: shapes the kernel covers (4 F / M a multiple of 64 and at most 7168); others take the plain-2:4 route.
bool vnm_spmm_gather_ok(int64_t T, int64_t N, int64_t F, int M);
// grp (role 0, host segment table): the token blocks of segment e take expert e's matrix Wk + e * b_stride.
hipError_t launch_vnm_spmm_gather(const uint16_t* a_vals, const uint8_t* a_meta, const uint8_t* colidx, const uint16_t* Wk, int64_t ldw,
                                  int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, const Split* split = nullptr);
// eqs. (3), (7) for M = 8 on a 256-token tile (gemm_vnm8.hip): the activation as the epilogues' vcb / mcb / cixt arrays, Wk = [F, ldw] with the
// contraction index as row; T, N, F multiples of 64.  grp as above (b_stride in elements).
bool vnm8_gemm_ok(int64_t T, int64_t N, int64_t F, int64_t ldw);
hipError_t launch_vnm8_gemm(const uint16_t* vcb, const uint8_t* mcb, const uint8_t* cixt, const uint16_t* Wk, int64_t ldw, int64_t T, int64_t N,
                            int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, int tile = 0, const Split* split = nullptr);
// vnm.hip: the canonical V:2:8 arrays (vals [T, F/4], meta [T, F/16], colidx [T/64, F/8, 4]) regrouped into those units; with W [R, C] (row stride ld)
// also its transpose wt [C, R]; counters (or null): kSplitCounters of them are cleared
hipError_t launch_vnm8_repack(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, uint16_t* vcb, uint8_t* mcb,
                              uint8_t* cixt, const uint16_t* W, int64_t R, int64_t C, int64_t ld, uint16_t* wt, unsigned* counters, hipStream_t s);
// (fp8 step: codes; F a multiple of 128, Wq = [F, ldw bytes], out = bf16(alpha * sum); the arrays in the layouts of vcb8_off, mcb8_off, cixt8_off)
bool vnm8_gemm_fp8_ok(int64_t T, int64_t N, int64_t F, int64_t ldw);
// fp8.hip: the canonical fp8 V:2:8 arrays (codes [T, F/4], meta, colidx) regrouped into those units; F a multiple of 128
hipError_t launch_vnm8_repack_fp8(const uint8_t* codes, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, uint8_t* vcb, uint8_t* mcb,
                                  uint8_t* cixt, hipStream_t s);
hipError_t launch_vnm8_gemm_fp8(const uint8_t* vcb, const uint8_t* mcb, const uint8_t* cixt, const uint8_t* Wq, int64_t ldw, float alpha, int64_t T,
                                int64_t N, int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, int tile = 0, const Split* split = nullptr);
// The same on E4M3 codes: a_codes [T, 2 F / M] + the same metadata and column offsets, Wq = codes [F, ldw bytes], out = bf16(alpha * sum);
// 4 F / M a multiple of 128; b_stride of grp in bytes.
bool vnm_spmm_gather_fp8_ok(int64_t T, int64_t N, int64_t F, int M);
hipError_t launch_vnm_spmm_gather_fp8(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* colidx, const uint8_t* Wq, int64_t ldw, float alpha,
                                      int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr);
hipError_t launch_vnm_to_24(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F,
                            uint16_t* vals24, uint8_t* meta24, hipStream_t s);
// vnm.hip: the transposed operand of eqs. (5), (8) from the canonical arrays: kept = 0: at [F / 2, T], mask [T / 64, F / 8] for launch_wgrad_vnm;
// kept = 1 (M = 32, 64, F a multiple of 8 M): at [4 F / M, T] for launch_wgrad_wide; and gt = the transpose of G [T, N] in
// the layout that kernel reads
hipError_t launch_vnm_compact_t(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M, int kept, uint16_t* at,
                                uint8_t* mask, const uint16_t* G, int64_t N, uint16_t* gt, hipStream_t s);
// blocked: out in the blocked operand layout (1) or in the order of lane_off (2, common.hpp); out_same: also a blocked copy of `in`; counters: as above
hipError_t launch_transpose(const uint16_t* in, int64_t R, int64_t C, int64_t ld, uint16_t* out, int blocked, uint16_t* out_same, hipStream_t s, unsigned* counters = nullptr);
hipError_t launch_clear_counters(unsigned* counters, hipStream_t s);

// C[i, j] = sum_k A[i, k] * B[j, k]  (both operands K-contiguous).
//   sparse_a: A given as 2:4 packed (a_vals [Ra, K/2], a_meta [Ra, K/8]) and multiplied on the
//             structured-sparse matrix cores; else a_vals is a dense [Ra, K] matrix.
//   out_i_contig: 1 -> out[j * ldo + i] (+ bias[i]);  0 -> out[i * ldo + j].
//   launch_spmm_blocked: A packed 2:4; both operands (and the metadata) are in the blocked layout of common.hpp;
//   out_i_contig must be 0 (eqs. (3), (7) of the fused step).
// eq. (1) / eq. (4) with the fused epilogue above: A packed 2:4 [Ra = F rows], B = [Rb = T rows], all blocked; out [T, F].
// grp (optional, blocked launchers only): grouped form, see GemmGroup; Ra / Rb / K then count all tokens on the token axis.
hipError_t launch_gemm_vnm_epilogue(const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias, int64_t F,
                                    int64_t T, int64_t K, uint16_t* out, const VnmEpilogue& ep, hipStream_t s,
                                    const GemmGroup* grp = nullptr, int tile = 0);
hipError_t launch_spmm_blocked(const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias, int64_t Ra, int64_t Rb,
                               int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr);
hipError_t launch_gemm_nt(int sparse_a, const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias,
                          int64_t Ra, int64_t Rb, int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s);
// eqs. (5), (8) of the neuron-level router: out[i * ldo + j] = sum over expert e's rows of at[i, row] * G[j, row], both blocked, dense [Kc, rows] and [N, rows];
// grp: role 2 (every expert contracts over its own run of rows, output rows by map_logM)
hipError_t launch_wgrad_router(const uint16_t* at, const uint16_t* G, int64_t Kc, int64_t N, int64_t rows, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup& grp);

// eqs. (5), (8): C[f, n] = sum_t A[t, f] * G[t, n] with A given as `atc` (compacted transposed activation written by the
// V:N:M epilogue) + kmask (kept-column bit masks, [T / 64, F / 8]), G = [N rows, T] in the blocked layout; out_i_contig: out[n * ldo + f], else out[f * ldo + n].
// grp (role 2): every expert contracts over its own token segment into its own output (out_stride).
// Section 3.3 / Alg. 3 (router.hip): routing scores + top-1, stable grouping by expert, permuted X, colidx of the result.
hipError_t launch_venom_route(const uint16_t* X, const uint16_t* means, int64_t T, int64_t D, int E, int32_t* expert, float* scores,
                              hipStream_t s);
hipError_t launch_venom_permute(const int32_t* expert, int64_t T, int E, int64_t cap, int32_t* blockcnt, int32_t* seg, int32_t* perm,
                                int32_t* row_of_token, hipStream_t s);
hipError_t launch_venom_gather_x(const uint16_t* X, const int32_t* perm, int64_t cap, int64_t D, uint16_t* xb, hipStream_t s);
struct TailFill {                   // up to five arrays of `rows` rows whose tail rows get a fill word
    int n = 0;
    uint32_t* p[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
    int64_t row_words[5] = {0, 0, 0, 0, 0};
    uint32_t v[5] = {0, 0, 0, 0, 0};
    void add(void* ptr, int64_t row_bytes, uint8_t byte) { p[n] = (uint32_t*)ptr; row_words[n] = row_bytes / 4; v[n] = 0x01010101u * byte; ++n; }
};
hipError_t launch_fill_tail_rows(const TailFill& f, int64_t first, int64_t rows, hipStream_t s);
// Everything the router's step prepares, in one launch (router.hip): permuted X and dY, row-major transposed and blocked; the experts' weights: W1 and
// W2.T pruned and packed expert-major (blocked), and the experts' slices of W2 and W1.T as [D, 4 F / M] matrices (blocked); colidx and the rows past
// the last run.  Absent parts: null X / dY / W1 / W2 / colidx.  seg: the run offsets (seg or seg_dev); at most max_tail rows lie past the last run.
struct RouterPrologueArgs {
    int rows, D, F, logM, mode;
    const int32_t* perm;
    const uint16_t *X, *dY; uint16_t *xt, *xb, *dyt, *dyb;
    const uint16_t* W1; uint16_t *w1vb, *w1t; uint8_t* w1mb;
    const uint16_t* W2; uint16_t *w2vb, *w2e; uint8_t* w2mb;
    uint8_t* colidx; TailFill tail; int max_tail;
    GemmGroup seg;
};
hipError_t launch_router_prologue(const RouterPrologueArgs& a, hipStream_t s);
// Shared launches of the router's step (router_mix.hip): eq. (1) with preparing passes that later launches read; eqs. (4) and (3); eq. (7) with the transpose of
// dW2.T [F, D].  128 tiles.
hipError_t launch_router_y1(const GemmV2Args& g1, const RouterPrologueArgs& p, hipStream_t s);
hipError_t launch_router_dy2_y3(const GemmV2Args& g4, const GemmV2Args& g3, hipStream_t s);
hipError_t launch_router_dx(const GemmV2Args& g7, const uint16_t* dw2t, int64_t F, int64_t D, uint16_t* dW2, hipStream_t s);
hipError_t launch_venom_colidx(const GemmGroup& g, int64_t cap, int64_t groups, uint8_t* colidx, hipStream_t s);

// fp8 operands (fp8.hip; Section 3.4's closing paragraph): E4M3 codes, inv = 1 / scale; amax (optional, device float) receives the largest
// magnitude quantised through an atomic max.
hipError_t launch_quantize_fp8(const uint16_t* src, int64_t n, float inv, uint8_t* codes, float* amax, hipStream_t s);
hipError_t launch_prune24_fp8(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, int mode, float inv, uint8_t* codes, uint8_t* meta,
                              float* amax, hipStream_t s);
hipError_t launch_sqrelu_vnm_compress_fp8(const uint16_t* y1, int64_t T, int64_t F, int M, float inv, uint8_t* codes, uint8_t* meta, uint8_t* colidx,
                                          float* amax, hipStream_t s);
hipError_t launch_vnm_to_24_fp8(const uint8_t* codes, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M, uint8_t* codes24,
                                uint8_t* meta24, hipStream_t s);
hipError_t launch_transpose_u8(const uint8_t* in, int64_t R, int64_t C, int64_t ld, uint8_t* out, hipStream_t s);
// C[i, j] = alpha * sum_k dec(A[i, k]) * dec(B[j, k]) (+ bias[i] when out_i_contig) on v_smfmac_f32_16x16x128_fp8_fp8: A packed 2:4 codes
// [Ra, K/2] + metadata [Ra, K/8], B codes [Rb, K], both row-major; K a multiple of 128; out bf16 as launch_gemm_nt.
hipError_t launch_spmm24_fp8(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* Bq, const float* bias, float alpha, int64_t Ra, int64_t Rb,
                             int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s);

// The same contraction on operands in the blocked layout with a pair of codes per 2-byte element (the fused fp8 step): a_codes = packed 2:4
// codes [Ra, K/2], a_meta in the fp8 metadata units of common.hpp, Bq = codes [Rb, K]; eq. (1) / eq. (4) with the fused V:N:M epilogue ep
// (mode 1 or 2: M = 8; mode 5 or 6: M = 2^logM = 16, 32, 64), Ra = hidden units, Rb = tokens, out [T, F] if ep->store_dense.
hipError_t launch_gemm_fp8_blocked(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* Bq, const float* bias, float alpha, int64_t Ra,
                                   int64_t Rb, int64_t K, uint16_t* out, int64_t ldo, const VnmEpilogue* ep, hipStream_t s, const GemmGroup* grp = nullptr, int tile = 0);
// the same on E4M3 codes (atc: compact transposed codes [F / 2, T], Gq [N, T], both in the blocked pair layout): out = bf16(alpha * sum)
hipError_t launch_wgrad_vnm_fp8(const uint8_t* atc, const uint8_t* kmask, const uint8_t* Gq, float alpha, int64_t F, int64_t N, int64_t T,
                                int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, bool acc32 = false, bool split_ok = true, int tile = 0);
// split_ok = false: never split a tile's contraction over wavefronts (the wide blocks' fused path sums in the order of the unfused one)
// acc32: `out` is a float32 matrix of the same shape (ldo in float32 elements; grouped form: out_stride in float32 elements) that the
// result is added to, out32 += alpha * sum, instead of a bf16 matrix that is overwritten
hipError_t launch_wgrad_vnm(const uint16_t* atc, const uint8_t* kmask, const uint16_t* G, int64_t F, int64_t N, int64_t T,
                            int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, bool acc32 = false, bool split_ok = true, int tile = 0);


// the same for blocks of M = 2^logM = 32, 64 columns on the kept rows only: at_kept = the epilogues' `at` with at_kept set, [4 F / M rows, T];
// colidx = the packed activation's; 4 F / M a multiple of 32.  Same sums, bit for bit, as launch_wgrad_vnm on the other form of `at`.
hipError_t launch_wgrad_wide(const uint16_t* at_kept, const uint8_t* colidx, const uint16_t* G, int64_t F, int64_t N, int64_t T, int logM, int out_i_contig, uint16_t* out,
                             int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, bool acc32 = false);

}  // namespace sffn
