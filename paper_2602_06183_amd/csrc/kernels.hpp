// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <initializer_list>
#include "mix_plan.hpp"

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
    int stream = 0;                 // modes 1 / 2 (bf16), 3 / 4: at, ykept, vcb, vals go out non-temporal (streams_between)
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
    // role 2 on dense blocked operands (weight gradients of the neuron-level experts, Section 3.3): output index i of expert e is
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
    GemmGroup grp; float alpha; Split split; int past = 0;
};
struct GatherArgs {
    const void* a_vals; const uint8_t* a_meta; const uint8_t* colidx; const void* Wk; int ldw, T, N, Kc, logM, tiles_n; float alpha; uint16_t* out; int64_t ldo; GemmGroup grp;
    Split split; int past = 0;
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
// Do the epilogues at M = 8 in bf16, and the router's, store what later launches read (`between`: bytes of a direction, prepared copies) non-temporal?  Where that and the inputs are more than the
// last-level cache of 256 MiB holds: ordinary stores then push the operands that the tiles share out of it, and are themselves gone before they are read.  Where all of it fits the readers find
// it there.  Steps, ordinary / non-temporal: T = 8192, D = 2048, F = 8192 (256 MiB) 907 / 894 us, T = 9664, D = 2752, F = 6016 (274) 1252 / 1228, T = 10496, D = 576, F = 13120 (313) 794 / 768,
// T = D = 8192, F = 28672 11034 / 10963; T = 896, D = 1792, F = 5184 (50) 110 / 124, T = 6720, D = 2752, F = 7488 (245) 1147 / 1165; the router's, T = 8192, D = 2048, F = 8192, M = 16 498 / 492,
// T = 10240, D = 576, F = 2560, M = 8 202 / 221.  Over 37 drawn steps that it takes 0.992, two of them 0.7 and 1.0 % longer.  M = 16, 32, 64 0.97 - 0.99 and codes 1.00 of the rate: not there.
inline bool streams_between(int64_t T, int64_t D, int64_t F, int64_t E, int64_t between) { return 4 * (T * D + E * F * D) + between >= (int64_t)250 << 20; }
// Eq. (1) with X row-major and the passes `behind` in the same launch (forward_x.hip); tile 64 or 128.
hipError_t launch_forward_x(const uint16_t* a_vals, const uint8_t* a_meta, const float* bias, const uint16_t* X, uint16_t* out, const VnmEpilogue& ep,
                            const PrologueArgs& behind, hipStream_t s, const GemmGroup* grp, int tile);
// Taken on both: what the row-major rows cost the loop (128-byte lines instead of 1 KB blocks) is less than a launch in front of it.  Forward calls on packed weights, 370
// shapes, three sets of weights and inputs in turn: 0.91 of the time with the copy of X, one in 18 2 % and more above it, the worst 1.09: T = 64, D = 2048, F = 8192, M = 64 27.0 us with the
// copy, 23.5 without; T = 4096, D = 512, F = 2048, M = 64 25.3 / 19.3; T = 384, D = 5696, F = 12288, M = 32 91.6 / 100.
// With weights to prune the passes over W2, X.T and dY run behind the tiles: two workgroups a CU beside 128 tiles, one beside 64 tiles, which is less than their rate alone.  On 128 tiles up to
// 6 Mi elements of tokens and weights, on 64 tiles while tiles and passes are 384 workgroups (M = 64: up to 3.5 Mi elements).  A whole step, with the copy / without: T = 512, D = 256, F = 1024 27.2 / 25.4 us;
// T = 448, D = 704, F = 2304 34.1 / 37.2; M = 32, T = 320, D = 768, F = 3072 37.2 / 40.9; on 128 tiles 38.3 / 36.8.
inline bool forward_reads_x(int64_t T, int64_t D, int64_t F, int64_t E, int M, bool packed, int tile) {
    if (tile == 256) return false;
    if (packed) return true;
    if (tile == 64 && M != 64) return ((F + 63) / 64) * (T / 64) + (2 * T + E * F) * D / 4096 <= 384;
    return (T + E * F) * D <= ((int64_t)(tile == 64 ? 7 : 12) << 19);
}
// Where eq. (1) also prunes the rows of W1 that it reads, so that no launch is in front of it: on 64 tiles while a wavefront has two stages of the contraction at most.  The pruning, 25 to 33
// instructions a group of four and done again for every 64 tokens, and the longer trip of twice the bytes cost eq. (1) 1 us a stage, the launch 3.  A step, with the launch / without:
// T = 512, D = 256, F = 1024 26.2 / 24.5 us, T = 192, D = 384, F = 1728 24.3 / 23.4, T = 64, D = 448, F = 1600 23.2 / 22.5; with eight stages for four wavefronts nothing is left of it
// (T = 256, D = 512, F = 1600 26.4 / 26.3, T = 576, D = 512, F = 1856 32.0 / 32.2).  At M = 8: wider blocks have 64 tiles from 16 stages on only.
inline bool forward_prunes_w1(int64_t D, int M, bool packed, int tile) { return !packed && tile == 64 && M == 8 && D <= 448; }
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
// part of a full one, when it leaves every workgroup a CU of its own.
inline int pick_tile(float rounds256, unsigned n128, unsigned n64, int steps, float w128, unsigned most64, int least_steps, float last = 1.0f) {
    if (n64 <= most64 && steps >= least_steps) return 64;
    const unsigned rest = n128 % 512;
    const float part = rest == 0 ? 0.0f : rest <= 256 ? last : 1.0f;
    return w128 * ((float)(n128 / 512) + part) < rounds256 ? 128 : 256;
}
inline float large_rounds(unsigned n256) { return (float)((n256 + 255) / 256); }

// tiles along the tokens when they come in `groups` segments (0: one), taken as equally long: a host and a device segment table choose alike
inline int64_t token_tiles(int64_t T, int groups, int64_t edge) {
    const int64_t n = groups ? groups : 1;
    return n * (((T + n - 1) / n + edge - 1) / edge);
}
// Plain stores and the router's epilogues: what a round of 128 tiles takes of a round of 256 tiles in gemm_v2, by the trips of the main loop.  The longer the contraction the more
// the bytes from L2 count, of which the small tile needs twice as many per product.
//   router   T = 8192, D = 2048, F = 8192, M = 16 95 / 86 us on 256 / 128 tiles, eq. (4) 94 / 92; T = 4096, D = 4096, F = 16384 147 / 161, 149 / 160
//   plain    26 trips 0.71, 46 0.73, 64 0.76 - 0.80, 86 0.89, 114 0.94 (T = 8000, N = 2560, K = 7296: 239 / 293 us)
// last_round: what the last round takes when it has at most 256 small tiles, one per CU (plain stores: 0.6 up to 48 trips, the router's eq. (3), 288 / 1120 tiles
// of K = 2048: 76 / 68 us; T = 8000, N = 2560, K = 7296 has 320 / 1260).
enum { kGemmPlain = 0, kGemmForward = 1, kGemmBackward = 2, kGemmRouter = 3 };
inline float small_round(int what, int steps) {
    const float n = (float)steps;
    if (what == kGemmPlain) return n < 110.0f ? 0.68f + 0.002f * n : 0.90f;
    const float w = 0.53f + 0.0031f * n;
    return w < 0.74f ? w : 0.74f;
}
inline float last_round(int what, int steps) { return what == kGemmPlain ? (steps <= 48 ? 0.6f : 1.0f) : 0.75f; }
// gemm_v2 (i x j outputs); w128, last: see pick_tile.  64 tiles: T = 64, D = 2048, F = 8192 (32 / 64 / 128 tiles): eqs. (1), (4) 43 / 33 us on 256 tiles,
// 21 / 18 on 128, 17 / 14 on 64; with more than 256 of them they lose to 128 (T = 128, D = 1984, F = 8512, 266 of them: 25 and 19 us).
inline int pick_gemm_tile(int64_t Ra, int64_t Rb, int steps, const GemmGroup& g, float w128, bool split, float last = 1.0f) {
    auto tiles = [&](int64_t ei, int64_t ej) {
        return (unsigned)(token_tiles(Ra, g.n && g.role == 0 ? g.n : 0, ei) * token_tiles(Rb, g.n && g.role == 1 ? g.n : 0, ej) * (g.role == 2 && g.n ? g.n : 1));
    };
    return pick_tile(large_rounds(tiles(256, 256)), tiles(128, 128), tiles(64, 64), steps, w128, split ? 256 : 0, 16, last);
}
// Eqs. (1), (4) with their epilogues, and eqs. (3), (7) at M = 8: the tile whose launch is estimated to be the shortest.  A launch takes the rounds of its tiles over the chip, 256 large or 512
// small ones at a time, times what such a tile takes: a fixed part and a part per trip of its main loop.  A last round of few tiles takes less than a full one: `part` of it with one large tile,
// and from there in line; `last` of it with up to 256 small tiles, a CU for each, and from `knee` on in line with more.  64 tiles: 256 at a time, a last round beyond the first one `more` of a full one.
// The epilogue of a small tile overlaps with the other workgroup's main loop; the longer the contraction the more the bytes from L2 count, of which it needs twice as many per product; the
// four wavefronts of a 64 tile share its contraction and its epilogue.  M = 64: one wavefront has to hold 128 hidden units, so that the small tile is 256 hidden units x 128
// tokens and the 64 tile 128 x 64.
// Fitted to launches inside whole steps of 3300 drawn shapes (T 64 - 10000, D 256 - 8192, 1 - 8 experts) on every tile, three sets of inputs and weights in turn: over them what is chosen takes
// 0.4 / 0.3 % longer than the best tile of each (eqs. (1) / (4), M = 8; wider blocks 1.0 / 0.4, codes 0.4 / 0.2) and 0.6 % (eqs. (3), (7)).  On 256 / 128 / 64 tiles:
//   eq. (1)  T = 2816, D = 2624, F = 7488 87.2 / 88.2 / 194 us; T = 832, D = 5376, F = 19008 145 / 158 / 250; T = 128, D = 960, F = 3776 24.7 / 13.5 / 10.7; codes, T = 128, D = 1920, F = 6272 28.1 / 16.3 / 12.1
//   eq. (4)  T = 64, D = 4288, F = 16704 52.0 / 36.2 / 44.1; M = 64, T = 192, D = 3456, F = 9216 45.6 / 47.8 / 29.9
struct TileTimes { float large, large_step, part, small, small_step, last, knee, tiny, tiny_step, more; };        // us
constexpr TileTimes kForwardBf16[3] = {{15.5f, 0.704f, 0.982f, 7.92f, 0.53f, 0.865f, 1.0f, 5.7f, 0.201f, 1.0f}, {15.8f, 0.672f, 0.807f, 8.53f, 0.485f, 0.815f, 1.0f, 8.21f, 0.146f, 0.604f},
                                       {12.8f, 0.648f, 1.0f, 10.3f, 0.745f, 0.976f, 1.0f, 15.9f, 0.309f, 0.46f}};            // M = 8; 16, 32; 64
constexpr TileTimes kForwardFp8[3] = {{23.7f, 0.718f, 0.822f, 10.3f, 0.609f, 0.775f, 1.0f, 7.13f, 0.172f, 0.655f}, {19.7f, 0.615f, 0.833f, 10.2f, 0.445f, 0.91f, 1.0f, 9.81f, 0.145f, 0.465f},
                                      {15.9f, 0.673f, 0.979f, 13.0f, 0.815f, 0.972f, 1.0f, 16.8f, 0.379f, 0.601f}};
constexpr TileTimes kBackwardBf16[3] = {{16.9f, 0.61f, 0.864f, 8.47f, 0.562f, 0.594f, 1.0f, 4.87f, 0.165f, 0.746f}, {13.0f, 0.771f, 0.848f, 7.92f, 0.552f, 0.758f, 1.0f, 7.34f, 0.228f, 0.333f},
                                        {10.1f, 0.781f, 0.903f, 7.08f, 1.04f, 0.856f, 1.0f, 10.6f, 0.384f, 0.502f}};
constexpr TileTimes kBackwardFp8[3] = {{17.4f, 0.522f, 1.0f, 7.71f, 0.547f, 0.828f, 1.0f, 5.29f, 0.222f, 0.674f}, {13.2f, 0.749f, 0.963f, 8.07f, 0.532f, 0.944f, 1.0f, 10.3f, 0.166f, 0.216f},
                                       {12.0f, 0.69f, 0.978f, 10.0f, 0.913f, 0.885f, 1.0f, 12.5f, 0.44f, 0.518f}};
inline const TileTimes& epilogue_times(int what, int M, bool fp8) {
    const int m = M == 8 ? 0 : M == 64 ? 2 : 1;
    return what == kGemmForward ? (fp8 ? kForwardFp8 : kForwardBf16)[m] : (fp8 ? kBackwardFp8 : kBackwardBf16)[m];
}
inline float rounds_of_large(unsigned n, float part) {
    const unsigned rest = n % 256;
    return (float)(n / 256) + (rest == 0 ? 0.0f : part + (1.0f - part) * (float)rest / 256.0f);
}
inline float rounds_of_small(unsigned n, float last, float knee = 1.0f) {
    const unsigned rest = n % 512;
    return (float)(n / 512) + (rest == 0 ? 0.0f : rest <= 256 ? last : knee + (1.0f - knee) * (float)(rest - 256) / 256.0f);
}
inline float rounds_of_tiny(unsigned n, float more) {
    const unsigned rest = n % 256;
    return n <= 256 ? 1.0f : (float)(n / 256) + (rest == 0 ? 0.0f : more + (1.0f - more) * (float)rest / 256.0f);
}
// large: rounds of the large tile; small, tiny: of 128 and 64 tiles (negative: not offered); before: what only the large tile needs in front of it
inline int shortest(const TileTimes& c, int steps, float large, float small, float tiny, float before = 0.0f) {
    const float n = (float)steps, a = before + large * (c.large + c.large_step * n), b = small * (c.small + c.small_step * n), t = tiny * (c.tiny + c.tiny_step * n);
    return tiny >= 0.0f && t < a && t < b ? 64 : b < a ? 128 : 256;
}
// On 128 tiles eq. (1) of a small step reads X as it is and the passes that nothing waits for stand behind it (forward_reads_x), so that the large tile has to save more than the launch in front
// of it: T = 7424, D = 320, F = 1152 74.7 us the step on 256, 69.9 on 128; T = 4928, D = 512, F = 1728 89.9 / 84.7.
inline float copy_of_x(int what, bool fp8, int64_t T, int64_t D, int64_t F, int64_t E) { return what == kGemmForward && !fp8 && (T + E * F) * D <= ((int64_t)12 << 19) ? 4.5f : 0.0f; }
// eqs. (1), (4); M: columns per V:N:M block
inline int pick_epilogue_tile(int64_t F, int64_t T, int steps, const GemmGroup& g, int what, int M, bool fp8) {
    const TileTimes& c = epilogue_times(what, M, fp8);
    auto tiles = [&](int64_t ef, int64_t et) { return (unsigned)((F + ef - 1) / ef * token_tiles(T, g.n, et)); };
    // (eq. (1) in bf16 at M = 16, 32: a short contraction gains less from four wavefronts than the preparing passes behind the tiles lose beside them; see forward_reads_x)
    const bool tiny = what != kGemmForward || fp8 || M == 8 || M == 64 || steps >= 16;
    return shortest(c, steps, rounds_of_large(tiles(256, 256), c.part), rounds_of_small(tiles(M == 64 ? 256 : 128, 128), c.last), tiny ? rounds_of_tiny(tiles(M == 64 ? 128 : 64, 64), c.more) : -1.0f,
                    copy_of_x(what, fp8, T, (int64_t)steps * (fp8 ? 128 : 64), F, g.n ? g.n : 1));
}
// V:2:8 activation GEMM.  The large tile is 512 tokens x 128 columns or 256 x 256 (gemm_vnm8.hip), 0.93 and 1 a round: four fifths of what a stage of the second
// fetches are the dense slab.  64 tiles hold the kept rows only, two workgroups a CU, from 8 trips on.  Large / 128 / 64: eqs. (3) and (7) together: T = 896, N = 1600, F = 4032 67 / 46 / 35 us;
// T = 832, N = 5376, F = 19008 374 / 438 / 378; T = 2816, N = 2624, F = 7488 132 / 149 / 192; codes, T = 448, N = 5120, F = 14336 212 / 149 / 113.
constexpr TileTimes kActivationBf16 = {3.59f, 0.62f, 0.991f, 3.02f, 0.77f, 0.541f, 0.699f, 1.78f, 0.275f, 0.932f}, kActivationFp8 = {9.77f, 0.592f, 1.0f, 3.57f, 0.66f, 0.559f, 0.873f, 2.01f, 0.366f, 0.943f};
// rounds of the 64 tiles, two workgroups a CU: `one` where each has a CU to itself; beyond 512 the next starts wherever one ends
inline float vnm8_tiny_rounds(unsigned n, float one, float more) { return n <= 256 ? one : n <= 512 ? 1.0f : 1.0f + (float)(n - 512) / 512.0f * more; }
inline float vnm8_rounds(unsigned n512, unsigned n256) { const float a = 0.93f * large_rounds(n512), b = large_rounds(n256); return a < b ? a : b; }
inline int shortest_vnm8(unsigned n512, unsigned n256, unsigned n128, unsigned n64, int steps, bool tiny_ok, bool fp8) {
    const TileTimes& c = fp8 ? kActivationFp8 : kActivationBf16;
    const float a = 0.93f * rounds_of_large(n512, c.part), b = rounds_of_large(n256, c.part);
    return shortest(c, steps, a < b ? a : b, rounds_of_small(n128, c.last, c.knee), tiny_ok && steps >= 8 ? vnm8_tiny_rounds(n64, fp8 ? 0.883f : 0.731f, c.more) : -1.0f);
}
inline int pick_vnm8_tile(int64_t T, int64_t N, int steps, int groups, bool fp8, bool tiny_ok = true) {
    auto tiles = [&](int64_t et, int64_t en) { return (unsigned)(token_tiles(T, groups, et) * ((N + en - 1) / en)); };
    return shortest_vnm8(tiles(512, 128), tiles(256, 256), tiles(128, 128), tiles(64, 64), steps, tiny_ok, fp8);
}
// gathered-row activation GEMM: 64 tokens x 256 columns, or 64 x 64
// (T = 256, N = 1024, F = 4096, M = 16: 19 us and 12 us; T = N = 1024: 20 and 12; T = 512, N = 4096, F = 16384: 90 and 67; T = 1984, N = 1344, M = 32: 14 and 23)
inline int pick_gather_tile(int64_t T, int64_t N, int steps) { return (T / 64) * ((N + 63) / 64) <= 512 && steps >= 6 ? 64 : 256; }

// Tile and number of workgroups per tile of eqs. (3), (7).  Splitting a 64 tile costs a fixed time and writes and reads `n` float32 copies of the output (at most kSplitMost bytes).  Not
// where eqs. (3), (7) share a launch: its workgroups fill the chip as it is (T = 192, N = 1024, F = 4096: the step 64 us, 74 with 5 splits).
// At most 1024 workgroups: with more, each with its start and its sums, the estimates are off.
constexpr int64_t kSplitMost = (int64_t)32 << 20, kSplitMostGroups = 1024;
struct SplitPlan { int tile, n; };
template <class Cost>
inline SplitPlan plan_split(int64_t T, int64_t N, int steps, int tile, float undivided, Cost split) {
    const int64_t tiles = ((T + 63) / 64) * ((N + 63) / 64);
    SplitPlan best = {tile, 1};
    if (tile == 256) return best;
    float least = undivided;
    for (int n = 2; n <= 16 && steps / n >= 8 && tiles * n <= kSplitMostGroups && tiles * 64 * 64 * 4 * n <= kSplitMost; ++n) {
        const float c = split(tiles * n, (float)((steps + n - 1) / n));
        if (c < least) { least = c; best = {64, n}; }
    }
    return best;
}
// M = 8: a launch takes 5.6 us, and 0.257 us a stage of a round of 512 of the 64 tiles, 0.42 of that with a CU for each; the sums 3.7 us and 10 ns per workgroup.  Taken where that saves
// 5 %.  (The counts, 6 of those 10 ns, have been spread over lines since: over 70 calls of 64 to 512 tokens what is chosen now takes 0.65 % longer than the best number of splits, always undivided 2.0 %.)  Fitted to 99 calls with 1 to 16 splits (what is chosen takes 2.0 % longer than the best of each, always undivided 10.6 %): T = 64, N = 4544, F = 19520 42.0 us undivided, 25.3 with 3,
// 27.4 with 7; T = 256, N = 4352, F = 19584 83.6, 60.5 with 3; T = 64, N = 896, F = 3648 9.6, 11.3 with 7.
inline SplitPlan plan_vnm8(int64_t T, int64_t N, int steps, int groups, bool fp8) {
    const int tile = pick_vnm8_tile(T, N, steps, groups, fp8);
    if (groups) return {tile, 1};
    auto launch = [](int64_t w, float stages) { return 5.6f + 0.257f * rounds_of_small((unsigned)w, 0.42f) * stages; };
    const TileTimes& c = fp8 ? kActivationFp8 : kActivationBf16;
    const int64_t n64 = ((T + 63) / 64) * ((N + 63) / 64), n128 = ((T + 127) / 128) * ((N + 127) / 128);
    const float undivided = tile == 64 ? launch(n64, (float)steps) : rounds_of_small((unsigned)n128, c.last, c.knee) * (c.small + c.small_step * (float)steps);
    return plan_split(T, N, steps, tile, 0.95f * undivided, [&](int64_t w, float stages) { return launch(w, stages) + 3.7f + 0.01f * (float)w; });
}
// M >= 16: 0.5 us a stage of a 64 tile, one workgroup per CU; the sums 6 us and their bytes at 4 TB/s.  Taken where that saves
// 15 % and more.  T = 64, N = 4096, F = 16384, M = 16: 41 -> 22 us.
inline SplitPlan plan_gather(int64_t T, int64_t N, int steps, int groups) {
    const int tile = pick_gather_tile(T, N, steps);
    if (groups) return {tile, 1};
    auto split = [](int64_t w, float stages) { return 0.5f * (float)((w + 255) / 256) * stages + 6.0f + (float)(w * 64 * 64) * 8.0f / 4.0e6f; };
    return plan_split(T, N, steps, tile, 0.85f * 0.5f * (float)((((T + 63) / 64) * ((N + 63) / 64) + 255) / 256) * (float)steps, split);
}
// bytes of the sums and, behind them, of the counters (a word per tile, spread over the lines: with 2 and more splits of 8 and more stages there are at most kSplitMost / 32 KB)
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
// Weight gradients: as eqs. (1), (4) above, a trip being a token block, over 1500 of those shapes (0.3 % longer than the best form of each).  Few tokens: 128 tiles on a ring of two
// stages, three workgroups a CU (768 tiles at a time), so that the stores of one tile run under the loads of two others; a tile of few stages is mostly its start and its stores.  On
// 256 / 128 / 64 tiles / three a CU: T = 64, N = 7040, F = 23552 85 / 82 us, three 62; T = 128, N = 3328, F = 8768 22.3 / 23.2 / 118 / 19.4; T = 704, N = 384, F = 1408 19.8 / 10.8 / 9.7 / 12.9;
// T = 4096, N = 704, F = 2048 71.9 / 31.5 / 27.9 / 43.0.  Not for experts, whose tiles are of different lengths (8 of 630 tokens on average, D = 1536, F = 4992: the step 591 us, 606 with
// it).  Codes: 200 registers, two workgroups a CU; with 168 they spill (T = 1216, a whole step a quarter slower).  The order of the sums is that of the other tiles: same bits.
constexpr TileTimes kGradientBf16 = {10.7f, 0.88f, 1.0f, 6.25f, 0.498f, 0.715f, 1.0f, 4.65f, 0.125f, 0.96f};
constexpr float kThreeFixed = 5.64f, kThreeStep = 0.873f, kThreeLast = 0.698f;
inline int pick_wgrad_tile(int64_t F, int64_t N, int64_t T, int experts, bool split_ok, bool fp8) {
    const unsigned e = experts ? (unsigned)experts : 1u;
    const int steps = (int)(T / 64 / e);
    auto tiles = [&](int64_t edge) { return (unsigned)((F + edge - 1) / edge * ((N + edge - 1) / edge)) * e; };
    if (fp8) return pick_tile(large_rounds(tiles(256)), tiles(128), tiles(64), steps, 0.58f, split_ok ? 256 : 0, 12);
    const TileTimes& c = kGradientBf16;
    return shortest(c, steps, rounds_of_large(tiles(256), c.part), rounds_of_small(tiles(128), c.last), split_ok && steps >= 12 ? rounds_of_tiny(tiles(64), c.more) : -1.0f);
}
// tile: what the rule above chooses
inline bool wgrad_three_a_cu(int64_t F, int64_t N, int64_t T, int experts, int tile) {
    if (experts || tile == 64) return false;
    auto tiles = [&](int64_t edge) { return (unsigned)((F + edge - 1) / edge * ((N + edge - 1) / edge)); };
    const TileTimes& c = kGradientBf16;
    const float steps = (float)(T / 64), three = (float)(tiles(128) / 768) + (tiles(128) % 768 == 0 ? 0.0f : tiles(128) % 768 <= 512 ? kThreeLast : 1.0f);
    return three * (kThreeFixed + kThreeStep * steps) < (tile == 256 ? rounds_of_large(tiles(256), c.part) * (c.large + c.large_step * steps) : rounds_of_small(tiles(128), c.last) * (c.small + c.small_step * steps));
}

// Weight gradients on the kept rows only (gemm_wgrad_wide_body.hpp; bf16, launches of their own), from 320 tokens per expert on: with fewer the matrix work that
// is saved is less than clearing a tile in LDS and reading it out again (F = 16384, N = 4096, M = 32: 50 us for 50 at 256 tokens, 51 for 54 at 320, 173 for 354 at 4096;
// M = 64: 43 for 45 at 192; F = 8192, N = 2048, M = 32: 17.9 for 17.4 at 256, 17.9 for 18.4 at 320, 22.4 for 30.7 at 1024).
inline bool wgrad_on_kept_rows(int64_t T, int64_t F, int M, int64_t experts) { return M >= 32 && F % (8 * M) == 0 && T >= 320 * experts; }

// Do eqs. (3), (5), (4) and (7), (8) take less time as two launches than as five?  Both are estimated (us).  A launch by itself takes `start` and its rounds
// over the chip, 256 large or 512 small tiles at a time (a last round of fewer less than a full one), or the time of the weights' bytes where few
// tokens meet them.  A shared launch takes the sum of its small tiles spread over the chip and `end` of the last unit's tile; no less than `lone` of a tile behind
// what comes before it, nor than the bytes of all its units.  Tiles and splits are those that the separate launches have.  Eqs. (5), (8) of bf16 blocks of 32 and
// 64 columns multiply the kept rows only where they have launches of their own, 8 and 16 times fewer products: M = 64, T = 11520, D = 896, F = 2048 the step 192 us apart,
// 254 together; T = 7680, D = 832, F = 3072 158 / 193; M = 32, T = 5312, D = 1152, F = 3584 175 / 198; small ones share all the same (M = 64, T = 1280, D = 448,
// F = 2048 51 / 44).
// The constants are fitted to whole steps, and to their forward and backward calls after one another, of 3487 shapes (T 64 - 16384, D 256 - 8192, 1 - 32 experts of uneven length, every M, bf16
// and codes, at most 1e11 token-weight elements), each run both ways with three sets of inputs and weights in turn; some no longer stand for the part that they are named after.  Over
// 2062 others what it chooses by itself takes 0.38 % longer than the better form in bf16 and 0.09 % on codes (the two calls 0.35 and 0.08 %, a forward call on packed weights 1.2 and 1.0 %: it takes the step's
// tile in eq. (3), see step_tiles), one step in 36 4 % and more, the worst 25 %; always sharing would take 4.3 % longer in bf16 and, as far as these sizes go, nothing on codes.  T = 1984, D = 1344, F = 4160 181 us apart, 150 together.
// (All of that on tiles of 128 in the shared launches.  With the tall ones of mix_plan.hpp in both forms, over 69 steps in bf16, 57 with experts and 149 on codes: 0.27, 0.30 and 0.37 % longer than
// the better form, 9 of them 4 % and more, the worst 12 %.)
// It errs mostly on experts, whose lengths it does not know (32 of them, T = 15104, D = 448, F = 1792, M = 16 411 / 322, apart), and on steps that have splits to lose (see step_tiles).
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
constexpr StepCosts kStepBf16 = {9.8f, {0.356f, 0.673f, 1.11f, 1.16f}, {0.297f, 0.157f, 1.0f}, {0.533f, 0.584f, 0.247f, 0.587f}, 0.3f, 0.269f, 1.98f, 4.51f, {0.338f, 0.0682f, 0.883f, 1.12f},
                                 {29.0f, 0.501f}, {28.6f, 0.767f}, {5.31f, 0.598f}, {14.9f, 0.276f}, {21.4f, 0.33f}, {21.9f, 0.461f}, {2.49f, 0.0356f},
                                 {13.0f, 0.747f}, {2.15f, 0.529f}, {0.175f, 0.324f}, {0.787f, 2.52f}, {4.61f, 0.308f}, {9.72f, 1.88f}, {5.5f, 0.958f}, {0.632f, 0.0131f}, {6.72f, 0.579f}, {5.64f, 0.669f}};
constexpr StepCosts kStepFp8 = {7.23f, {0.588f, 0.82f, 1.38f, 1.44f}, {0.33f, 0.432f, 0.927f}, {0.568f, 0.489f, 0.541f, 0.624f}, 0.699f, 0.433f, 1.9f, 1.47f, {0.207f, 0.321f, 0.979f, 0.986f},
                                {21.4f, 0.641f}, {26.8f, 0.367f}, {14.1f, 0.269f}, {12.1f, 0.39f}, {12.6f, 0.294f}, {13.1f, 0.286f}, {7.05f, 0.222f},
                                {12.8f, 0.345f}, {2.27f, 0.275f}, {3.09f, 0.19f}, {2.01f, 0.619f}, {3.52f, 0.416f}, {14.6f, 0.408f}, {7.85f, 0.193f}, {2.52f, 0.034f}, {}, {}};
// Steps of more than 1e10 token-weight elements: the mean of that estimate and of one fitted to 28000 shapes of any size, on somewhat slower kernels.  The first leaves its range and shares
// launches that fill the chip by themselves (T = 8192, D = 2048, F = 8576 1105 us apart, 1213 together; M = 16, T = 15936, D = 5760, F = 20480 11199 / 12103), the second errs the other way.
// 812 steps of 4e10 to 1.9e12, longer than the better form: bf16 0.31 % (the first alone 0.64, the second 0.48, never sharing 1.8), codes 0.23 % (0.55, 0.29, 4.1).
constexpr double kLargeStep = 1e10;
constexpr StepCosts kAnySizeBf16 = {3.34f, {0.51f, 0.556f, 0.869f, 0.968f}, {0.402f, 0.411f, 0.436f}, {0.664f, 0.788f, 0.653f, 0.591f}, 0.882f, 0.856f, 2.69f, 1.98f, {0.263f, 0.285f, 0.485f, 1.12f},
                                      {8.92f, 0.722f}, {11.6f, 0.825f}, {7.85f, 0.511f}, {5.16f, 0.407f}, {4.99f, 0.639f}, {4.73f, 0.86f}, {11.8f, 0.0731f},
                                      {15.4f, 0.632f}, {2.0f, 0.69f}, {3.59f, 0.103f}, {3.2f, 1.49f}, {4.31f, 0.338f}, {6.46f, 1.17f}, {4.09f, 0.63f}, {4.46f, 0.164f}, {5.62f, 0.201f}, {7.12f, 0.229f}};
constexpr StepCosts kAnySizeFp8 = {4.84f, {0.421f, 0.727f, 1.24f, 0.658f}, {0.297f, 0.255f, 0.254f}, {0.618f, 0.683f, 0.639f, 0.631f}, 1.0f, 0.942f, 2.75f, 1.9f, {0.247f, 0.26f, 0.452f, 1.03f},
                                      {11.8f, 0.858f}, {16.0f, 0.776f}, {13.6f, 0.8f}, {6.33f, 0.52f}, {7.82f, 0.545f}, {8.93f, 0.977f}, {1.9f, 0.15f},
                                      {11.0f, 0.608f}, {3.16f, 0.586f}, {3.4f, 0.206f}, {2.86f, 1.28f}, {4.0f, 0.38f}, {6.57f, 0.503f}, {4.15f, 0.29f}, {3.27f, 0.0483f}, {}, {}};
// t: the tiles of the separate launches; v, w: those of eqs. (3), (7) and (5), (8) in the shared ones (256: the next smaller there)
inline float shared_to_apart(const StepCosts& c, int64_t T, int64_t D, int64_t F, int M, int groups, bool fp8, const StepTiles& t, int v, int w) {
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
        else alone5 = t.w == 256 ? large((float)e * across(F, 256) * across(D, 256)) * c.large5(sw) : w != 64 ? small(n, c.last.w) * c.small5(sw) : large(n64) * c.tiny5(sw);
        u5 = w == 64 ? Unit{c.two_w * c.tiny5(sw), n64, c.lone.w, c.end.w} : Unit{c.small5(sw), n, c.lone.w, c.end.w};
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
    return (shared({u3, u5, u4}, b3 + b4 + b5) + shared({u3, u5}, b3 + b5)) / (5.0f * c.start + more(alone4, b4) + 2.0f * (more(alone3, b3) + more(alone5, b5)));
}
inline bool sharing_pays(int64_t T, int64_t D, int64_t F, int M, int groups, bool fp8, const StepTiles& t, int v, int w) {
    const float r = shared_to_apart(fp8 ? kStepFp8 : kStepBf16, T, D, F, M, groups, fp8, t, v, w);
    if ((double)T * (double)D * (double)F <= kLargeStep) return r < 1.0f;
    return r * shared_to_apart(fp8 ? kAnySizeFp8 : kAnySizeBf16, T, D, F, M, groups, fp8, t, v, w) < 1.0f;
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
    t.w = pick_wgrad_tile(F, D, T, experts > 1 ? experts : 0, M == 8 || fp8, fp8);
    // Beside eqs. (5), (8) the 64 tiles of eqs. (3), (7) gain only while there are few of them: behind more the launch is full with either, and theirs take longer per product.  The step on 64
    // tiles over that on 128 (medians of 260 drawn calls), 60 - 256 of the first: bf16 0.89, codes 0.98; up to 512 1.03 both, bf16 of 84 and more stages 0.98; above 1.04 and 1.07.
    int v_shared = t.v;
    if (M == 8 && v_shared == 64 && token_tiles(T, g.n, 64) * ((D + 63) / 64) > (!fp8 && F / unit >= 84 ? 512 : 256)) v_shared = pick_vnm8_tile(T, D, (int)(F / unit), g.n, fp8, false);
    // 64 tiles of eqs. (5), (8) in bf16 put a shared launch at one workgroup a CU (156,672 bytes of LDS): only while each has a CU of its own.  T = 3136, D = 832, F = 2304 (468 of them) 106 us the step, on 128 tiles 82; T = 6016, D = 768, F = 2496 161 / 132.
    const int w_shared = t.w == 64 && (experts > 1 ? experts : 1) * ((F + 63) / 64) * ((D + 63) / 64) > 256 ? 128 : t.w;
    t.v = v.tile; t.v_split = v.n;
    // Shared launches do not split eqs. (3), (7), and calls of either pass alone have to sum as the whole step does: a forward call would lose its split (T = 64, D = 2048,
    // F = 6784: the step 87 us apart, 74 together, a forward call on packed weights 20 and 23).  So steps with splits share only where no contraction wants the large tile,
    // which is where they gain most (T = 64, D = 960, F = 4224: 54 / 39, the forward call 17 / 17).
    const bool loses_split = v.n > 1 && (t.w == 256 || t.g == 256 || t.g_bwd == 256);
    t.mix = may_share && !loses_split && sharing_pays(T, D, F, M, g.n, fp8, t, v_shared, w_shared);
    t.v_alone = t.mix ? v_shared : v.tile;
    if (t.mix) {
        t.g_bwd = 128;
        t.v = M == 8 && v_shared == 256 ? 128 : v_shared; t.v_split = 1;
        t.w = w_shared == 256 ? 128 : w_shared;
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
        const TileTimes& c = epilogue_times(what, M, fp8);
        return shortest(c, (int)(D / (fp8 ? 128 : 64)), rounds_of_large(count(F, 256, 256), c.part), rounds_of_small(count(F, M == 64 ? 256 : 128, 128), c.last), -1.0f, copy_of_x(what, fp8, g.seg[g.n], D, F, g.n));
    };
    if (t->g != 64) t->g = pick(kGemmForward);
    if (t->g_bwd != 64 && !t->mix) t->g_bwd = pick(kGemmBackward);
    if (M == 8 && t->v != 64) {
        t->v_alone = shortest_vnm8(count(D, 128, 512), count(D, 256, 256), count(D, 128, 128), 0, (int)(F / (fp8 ? 128 : 64)), false, fp8);
        if (!t->mix) t->v = t->v_alone;
    }
}

// Does the router's step share launches?  Where eqs. (1), (4) and (3), (7) all run on 128 tiles.  Grouped by expert they have a few tiles more than fill the
// chip, so that the last round of each is nearly empty: T = 8192, D = 2048, F = 8192, M = 16 (1056 tiles each, 512 at a time) eqs. (4) and (3) 90 + 68 us apart,
// 137 together; eq. (7) and the transpose of dW2 72 + 12, 77; the step 542 / 522; T = 1792, D = 640, F = 1920, M = 8 110 / 94; T = 128, D = 704, F = 2560,
// M = 16 90 / 78.  M = 8 (two experts of half the hidden units): not above 6 Ki rows (T = 12544, D = 448, F = 1408 196 / 207; T = 7488, D = 512, F = 2304 160 / 164).  Of 100 drawn calls 54 share, in 0.90 of the time apart,
// the slowest 1.03 (T = 3904, D = 768, F = 3328, M = 8 132 / 136).  Up to 48 Mi elements of tokens and weights: the passes that ride along run two workgroups a CU, which
// is less than their rate alone (T = 320, D = 4928, F = 21888, M = 8 811 us apart, 894 together).
inline bool router_shares(int64_t rows, int64_t D, int64_t F, int M) {
    if ((rows + F) * D > ((int64_t)48 << 20) || (M == 8 && rows > 6 << 10)) return false;
    GemmGroup g;
    g.n = M / 4; g.role = 1;
    const int64_t Kc = 4 * F / M;
    const int steps = (int)(D / 64), steps3 = (int)(Kc / 64);
    if (pick_gemm_tile(Kc, rows, steps, g, small_round(kGemmRouter, steps), true, last_round(kGemmRouter, steps)) != 128) return false;
    g.role = 0;
    return pick_gemm_tile(rows, D, steps3, g, small_round(kGemmPlain, steps3), true, last_round(kGemmPlain, steps3)) == 128;
}

// Do the stand-alone packing operations read their operands past the caches?  Where these are as large as the last-level cache, which then holds none of them, whoever wrote them, but takes time to be
// filled.  Ordinary / past, operands in turn: SquaredReLU and compression of 448 MiB 113 / 100 us, of 512 126 / 111, of 896 223 / 195, eq. (6) on 256 MiB 52 / 50, on 1 GiB 207 / 193, pruning of
// 448 MiB along rows 128 / 115, across 177 / 140; the same one over and over alike.  Smaller ones are found there: 64 MiB of y1 18 / 19, the same 128 MiB at M = 16 over and over 25 / 29.
inline bool reads_past(int64_t bytes) { return bytes >= (int64_t)256 << 20; }
// Do the results of the stand-alone eqs. (1), (4) leave non-temporally?  Where they are as large as the last-level cache, so that the next kernel does not find them there: spmm24_fwd, then
// SquaredReLU and compression, ordinary / non-temporal: y1 of 256 MiB 649 / 578 us, of 512 1365 / 1191; of 128 181 / 184, of 64 95.5 / 96.7, of 1 9.9 / 10.2 (8 to 16 MiB 17.9 / 17.2, 25.8 / 24.7: not
// taken, Y3 of that size loses 7 %).
inline bool stores_past(int64_t bytes) { return bytes >= (int64_t)256 << 20; }
// Do Y3 and dX of a step?  From 16 MiB on, half of what the L2s hold together: the next layer's passes read them once, in order, and are no slower, while the step gains.  Of the time with ordinary
// stores, bf16 and M = 32 at 16 - 64 MiB: the step alone 0.971 - 1.000, with residuals added to both 0.978 - 1.006, two layers in a row 0.960 - 1.004, two forward calls in a row 0.985 - 1.016; below, up
// to 1.016, 1.013, 1.034 and 1.055 (T = 6144, D = 1024, F = 4096 159 -> 168 us the forward calls).  Codes 0.97 - 1.01 at any size.  Not the stand-alone vnm_spmm: spmm24_fwd, which reads its operand from
// many tiles, takes 2 - 9 % longer on such a result at every size.
inline bool results_past(int64_t T, int64_t D) { return 2 * T * D >= (int64_t)16 << 20; }
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
                                  int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, const Split* split = nullptr, bool past = false);
// eqs. (3), (7) for M = 8 on a 256-token tile (gemm_vnm8.hip): the activation as the epilogues' vcb / mcb / cixt arrays, Wk = [F, ldw] with the
// contraction index as row; T, N, F multiples of 64.  grp as above (b_stride in elements).
bool vnm8_gemm_ok(int64_t T, int64_t N, int64_t F, int64_t ldw);
hipError_t launch_vnm8_gemm(const uint16_t* vcb, const uint8_t* mcb, const uint8_t* cixt, const uint16_t* Wk, int64_t ldw, int64_t T, int64_t N,
                            int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, int tile = 0, const Split* split = nullptr, bool past = false);
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
                                int64_t N, int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, int tile = 0, const Split* split = nullptr, bool past = false);
// The same on E4M3 codes: a_codes [T, 2 F / M] + the same metadata and column offsets, Wq = codes [F, ldw bytes], out = bf16(alpha * sum);
// 4 F / M a multiple of 128; b_stride of grp in bytes.
bool vnm_spmm_gather_fp8_ok(int64_t T, int64_t N, int64_t F, int M);
hipError_t launch_vnm_spmm_gather_fp8(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* colidx, const uint8_t* Wq, int64_t ldw, float alpha,
                                      int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, bool past = false);
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
                               int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp = nullptr, bool past = false);
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
