// Pipelined tile kernel: C[i, j] = sum_k A[i, k] * B[j, k].  Workgroup tiles of 256 x 256, 128 x 128 and 64 x 64 outputs (pick_tile in
// kernels.hpp has the rule), operand tiles streamed HBM -> LDS with global_load_lds_dwordx4 into a ring of LDS stages (no register
// staging), XOR-swizzled 16-byte chunks so that the b128 fragment reads are bank-conflict free without padding.
//   256 x 256: 8 wavefronts (2 along i x 4 along j, 128 x 64 each, two wavefronts per SIMD so one hides the other's LDS latency).
//   128 x 128: 4 wavefronts of 64 x 64, two workgroups per CU: four times the workgroups for outputs that do not give every CU a 256 tile.
//   64 x 64:   4 wavefronts that share the tile's contraction (see Tile): outputs of a few tiles, where the latency of one wavefront's
//              trip along k is the whole cost.
//   SPARSE: A packed 2:4 -> v_smfmac_f32_16x16x64_bf16; ring of 3 stages of 64 k.  Eqs. (1), (3), (4), (7):
//           in the fused step on blocked operands (eqs. (1), (4) with the V:N:M epilogue), stand-alone on row-major ones.
//   dense : v_mfma_f32_16x16x32_bf16; ring of 4 stages of 32 k.  The weight gradients of the router's step on blocked operands, those of the unfused path on
//           row-major ones (those of the fused steps and the stand-alone vnm_wgrad: gemm_wgrad.hip, gemm_wgrad_wide.hip).
// The 16 x 16 instructions do the same products as the 32 x 32 ones for less power (registers only, random operands: smfmac 3350 -> 3720 dense-equivalent TFLOP/s, on codes
// 6200 -> 6970, dense 1850 -> 2070), and a whole stage is one of them per fragment pair.
// Register layouts of the two instructions are documented in lds_dma.hpp.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"
#include "vnm_select.hpp"

namespace sffn {

// FP8 (structured-sparse kernel): both operands are 1-byte E4M3 codes, row-major (stand-alone entry points) or blocked with a pair
// of codes per 2-byte element (fused fp8 step); the metadata is row-major [R, K/8] for row-major operands and in 512-byte units
// (m8blk_off, common.hpp) for blocked ones: 16-byte row pieces fetched one by one cost 17 % of eq. (3) at the 70B-scale layer.  In BYTES the tiles are those of
// the bf16 kernel (a stage is 128 k instead of 64: 64 survivor bytes per A row, 128 bytes per B row, and the fragment a lane of
// v_smfmac_f32_16x16x128_fp8_fp8 wants is the same 16 / 2 x 16 bytes), so the kernel runs with K counted in byte pairs and only
// the metadata differs: 16 survivors per lane and step need a whole 32-bit index word, 16 bytes per row and stage.
// Workgroup tile: WVM x WVN wavefronts of WM x 64 outputs each.  KW > 1 (with one wavefront per tile): KW wavefronts share one output tile,
// wavefront g contracting main-loop steps g, g + KW, ... in a ring of its own; the partial sums meet in LDS before the epilogue.
template <int WVM_, int WVN_, int WM_, int NST_, int KW_>
struct Tile {
    static constexpr int WVM = WVM_, WVN = WVN_, WM = WM_, NST = NST_, KW = KW_;
    static constexpr int NW = WVM * WVN, BM = WVM * WM, BN = WVN * 64, THREADS = 64 * NW * KW;
    static_assert(KW == 1 || NW == 1, "a shared output tile belongs to single wavefronts");
};
// MG: row-major 2:4 metadata fetched for four stages at a time, into two buffers behind the ring (see issue())
// PRUNE: A is the weight itself, which the wavefronts prune as they read it (see below): the stages hold B only
template <bool SPARSE, bool FP8, class TL, bool MG = false, bool PRUNE = false>
struct Cfg {
    static constexpr int BM = TL::BM, BN = TL::BN;
    static constexpr int BK = SPARSE ? 64 : 32;
    static constexpr int NSTAGE = TL::NST;
    static constexpr int A_ROW = 64;                        // bytes per A row per stage (32 survivors or 32 dense k)
    static constexpr int B_ROW = SPARSE ? 128 : 64;
    static constexpr int META_ROW = FP8 ? 16 : 8;
    static constexpr int A_BYTES = PRUNE ? 0 : BM * A_ROW, B_BYTES = BN * B_ROW, META_BYTES = SPARSE && !MG && !PRUNE ? BM * META_ROW : 0;
    static constexpr int GROUP_BYTES = MG ? BM * 32 : 0;    // 32 metadata bytes of every A row = 256 k
    static constexpr int STAGE = A_BYTES + B_BYTES + META_BYTES;
    static constexpr int A_LD = A_BYTES / 1024 / TL::NW, B_LD = B_BYTES / 1024 / TL::NW, M_LD = SPARSE && !PRUNE ? BM / 32 / TL::NW : 0;   // loads per wave per stage
    static constexpr int LOADS = A_LD + B_LD + M_LD * (FP8 ? 2 : 1);       // (MG: one fewer in stages that bring no metadata)
};

template <bool SPARSE, bool OUT_I_CONTIG, int EPI, bool BLOCKED, bool FP8, class TL, bool MG = false, bool PRUNE = false>
struct GemmV2Lds {
    using C = Cfg<SPARSE, FP8, TL, MG, PRUNE>;
    static constexpr int EPI_LDS = (EPI != 0) ? TL::NW * (64 + 32) * (64 * 2 + 16) : 0;        // the epilogues' scratch (see below) when the ring is shorter
    static constexpr int RING = TL::KW * C::NSTAGE * C::STAGE + 2 * C::GROUP_BYTES;
    static constexpr int SUMS = PRUNE ? TL::KW * (TL::WM / 16) * 4 * 4 * 256 + EPI_LDS : 0;     // the partial sums of a shared tile and the scratch, where the ring does not hold them
    static constexpr int LONGER = RING > EPI_LDS ? RING : EPI_LDS, BYTES = LONGER > SUMS ? LONGER : SUMS;
};
// pid / n_pid: this workgroup's id and the number of workgroups of the contraction (a launch may hold several contractions)
// BROW: B row-major although A is blocked (forward_x.hip)
// PRUNE: 1 + SFFN_MODE of a contraction whose A (a_vals) is the unpruned row-major weight (forward_x.hip): a lane's 16 k of a row are four whole groups, which it prunes in registers.  All of a
// wavefront's stages are in flight at once, at most NST of them (K <= 64 KW NST).
template <bool SPARSE, bool OUT_I_CONTIG, int EPI, bool BLOCKED, bool FP8, class TL, bool BROW, bool MG, int PRUNE>
__device__ __forceinline__ void gemm_nt_v2_body(unsigned char* __restrict__ smem, int pid, int n_pid,
                                                        const uint16_t* __restrict__ a_vals, const uint8_t* __restrict__ a_meta,
                                                        const uint16_t* __restrict__ B, const float* __restrict__ bias,
                                                        int Ra, int Rb, int K, uint16_t* __restrict__ out, int64_t ldo,
                                                        int tiles_m, int tiles_n, const VnmEpilogue& ep, const GemmGroup& grp, float alpha) {
    static_assert(EPI == 0 || (SPARSE && OUT_I_CONTIG && BLOCKED), "the V:N:M epilogues belong to the 2:4-weight GEMMs of the fused step");
    // EPI 16 + log2(M) / 32 + log2(M): the forward (eq. (2) + compression) / backward (eq. (6)) epilogue for blocks of M = 16, 32, 64 columns
    constexpr bool GEN_F = EPI >= 16 && EPI < 32, GEN_B = EPI >= 32;
    constexpr int LOGM = (GEN_F || GEN_B) ? (EPI & 15) : 3;
    static_assert(!(GEN_F || GEN_B) || (LOGM >= 4 && LOGM <= 6), "wide V:N:M blocks: M = 16, 32 or 64");
    static_assert(!FP8 || (SPARSE && (EPI == 0 || (BLOCKED && (EPI == 1 || EPI == 2 || GEN_F || GEN_B)))), "fp8 operands: structured-sparse kernel; the step's fused epilogues");
    constexpr bool blocked = BLOCKED, blockedB = BLOCKED && !BROW;       // operands in the blocked layout of common.hpp (fused step) or row-major (stand-alone entry points)
    static_assert(!MG || (SPARSE && !BLOCKED && !FP8 && TL::KW == 1 && TL::NST == 3 && TL::WM * TL::WVM == 32 * TL::NW), "metadata of four stages: row-major bf16, 32 rows a wavefront");
    static_assert(!PRUNE || (BROW && TL::KW > 1 && !FP8), "the weight itself: 64 tiles of eq. (1) in bf16, on row-major operands");
    using C = Cfg<SPARSE, FP8, TL, MG, PRUNE != 0>;
    constexpr int BM = C::BM, BN = C::BN, WM = TL::WM, WN = 64, FM = WM / 16, FN = 4, NH = WM / 64, KW = TL::KW;
    static_assert(LOGM < 6 || WM == 128, "the two blocks of 64 columns that share a metadata byte belong to one wavefront");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: everything derived from it stays in SGPRs
    const int kg = KW > 1 ? wave : 0, wt = KW > 1 ? 0 : wave;      // this wavefront's share of the contraction / place in the tile
    const int wm = wt / TL::WVN, wn = wt % TL::WVN;
    const int l16 = lane & 15, lq = lane >> 4;
    unsigned char* const ring = smem + kg * (C::NSTAGE * C::STAGE);
    const uint32_t ring_lds = lds_addr(smem) + kg * (C::NSTAGE * C::STAGE);

    // Workgroup -> tile.  Consecutive workgroup ids go to different XCDs; the remap gives each XCD a run of
    // consecutive logical ids, and logical ids walk bands of 4 tile rows, so an XCD's L2 sees few operand panels.
    int L = xcd_run(pid, n_pid);
    // Grouped form: find the expert of this tile and narrow the problem to its token segment.
    const int Kld = K;                   // K extent of the stored operands (block-row stride)
#define SEG(i) (grp.seg_dev ? uniform(grp.seg_dev[i]) : grp.seg[i])
    const int tok_ld = grp.n ? SEG(grp.n) : Rb;       // tokens in the token-indexed outputs of the V:N:M epilogue
    int i_base = 0, j_base = 0;
    int expert_id = 0;
    if (!SPARSE && BLOCKED && grp.n && grp.role == 2) {
        // every expert has its own tiles_m x tiles_n output and contracts over its own k range (whole chunks of 32) of the shared operands
        const int per = tiles_m * tiles_n;
        expert_id = uniform(L / per);
        L -= expert_id * per;
        if (expert_id >= grp.n) return;
        const int k0 = SEG(expert_id);
        K = SEG(expert_id + 1) - k0;
        a_vals += (int64_t)k0 * 16; B += (int64_t)k0 * 16;
        out += expert_id * grp.out_stride;
    } else if (grp.n) {
        int e = 0;
        {
            const int other = grp.role == 0 ? tiles_n : tiles_m;
            int cnt = 0;
            for (; e < grp.n; ++e) {
                cnt = ((SEG(e + 1) - SEG(e) + (grp.role == 0 ? BM : BN) - 1) / (grp.role == 0 ? BM : BN)) * other;
                if (L < cnt) break;
                L -= cnt;
            }
            if (e == grp.n) return;      // (the launcher sizes the grid exactly; kept as a guard)
            if (grp.role == 0) { tiles_m = uniform(cnt / other); i_base = SEG(e); Ra = SEG(e + 1); }
            else               { tiles_n = uniform(cnt / other); j_base = SEG(e); Rb = SEG(e + 1); }
#undef SEG
        }
        if (grp.role != 0) { a_vals += e * grp.a_stride; if (SPARSE) a_meta += e * grp.m_stride; }
        if (grp.role != 1) B += e * grp.b_stride;
        if (bias) bias += e * grp.bias_stride;
        out += e * grp.out_stride;
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, SFFN_TILE_GROUP, tm, tn);
    const int i0 = i_base + tm * BM, j0 = j_base + tn * BN;
    const int lda = SPARSE ? Kld / 2 : Kld;

    // ---- per-lane source addresses of the DMA loads.  A wave-wide load fills 1 KB of LDS = 16 tile rows x
    //      64 bytes; lane l lands at (row l / 4, 16-byte chunk l % 4) and therefore fetches the chunk that the
    //      XOR swizzle assigns to that slot.  Row-major sources: 16 row segments per load; blocked sources
    //      (common.hpp): the 16 rows x 64 bytes are one contiguous block.  Tile rows past the matrix edge
    //      are clamped into it: they only feed outputs that are never stored. --------------------------
    constexpr int A_LD = C::A_LD, B_LD = C::B_LD, M_LD = C::M_LD;          // issues per wave and stage
    // Row-major operands of the sparse kernel: a B row's 64 k of a stage are one 128-byte line, fetched whole (8 rows per
    // load, tile [256][128 bytes], 16-byte chunks swizzled by (row / 2) % 8) rather than as two 64-byte halves.
    constexpr bool lineB = SPARSE && !blockedB;
    uint64_t a_base[A_LD > 0 ? A_LD : 1], b_base[B_LD], m_base[M_LD > 0 ? M_LD : 1];     // wave-uniform byte addresses of kt = 0
    uint32_t a_lane, b_lane, m_lane;                     // per-lane byte offsets
    uint32_t a_kstep, b_kstep, m_kstep;                  // bytes per main-loop step
    {
        const int rb = lane >> 2;                                        // row inside the 16-row group
        const int c = (lane & 3) ^ swz4(rb >> 2);                        // source chunk for this lane's LDS slot
        const int KCa = SPARSE ? Kld / 64 : Kld / 32, KCb = Kld / 32;    // 32-element chunks per row
#pragma unroll
        for (int n = 0; n < A_LD; ++n) {
            int gr = i0 + (wt * A_LD + n) * 16; gr = gr < Ra ? gr : Ra - 16;
            a_base[n] = uniform64(blocked ? a_vals + ((int64_t)(gr >> 4) * KCa << 9) : a_vals + (int64_t)gr * lda);
        }
#pragma unroll
        for (int n = 0; n < B_LD; ++n) {
            // SPARSE: a stage holds 64 k of B as two half-tiles (k 0-31, k 32-63), each laid out like the A tile
            const int bk = wt * B_LD + n, h = SPARSE ? bk / (BN / 16) : 0;
            int gr = j0 + (bk % (BN / 16)) * 16; gr = gr < Rb ? gr : Rb - 16;
            if (lineB) { gr = j0 + bk * 8; gr = gr < Rb ? gr : Rb - 8; }
            b_base[n] = uniform64(blockedB ? B + (((int64_t)(gr >> 4) * KCb + h) << 9) : lineB ? B + (int64_t)gr * Kld : B + (int64_t)gr * Kld + h * 32);
        }
        a_lane = blocked ? (rb * 32 + c * 8) * 2 : (uint32_t)(rb * lda + c * 8) * 2;
        b_lane = blockedB ? (rb * 32 + c * 8) * 2 : (uint32_t)(rb * Kld + c * 8) * 2;
        if (lineB) {        // lane -> (row lane / 8 of the load's 8 rows, slot lane % 8); tile row = 8 * load + row; odd loads: the line's other half
            const int r8 = lane >> 3, slot = lane & 7;
            b_lane = (uint32_t)(r8 * Kld + ((slot ^ (r8 >> 1)) * 8)) * 2;
        }
        // metadata: one 4-byte-per-lane load brings 32 rows x 64 k; blocked: one unit of common.hpp, lane-linear;
        // row-major: lane -> (row lane / 2, 4-byte half lane % 2), landing as [row][8 bytes]
        m_lane = blocked ? lane * 4 : (uint32_t)((lane >> 1) * (Kld / 8) + (lane & 1) * 4);
        // fp8: a row has Kld / 4 metadata bytes, 16 per stage; one load brings 16 rows (lane -> row lane / 4, word lane % 4), two per wave
        if (FP8) m_lane = (uint32_t)((lane >> 2) * (Kld / 4) + (lane & 3) * 4);
#pragma unroll
        for (int n = 0; n < M_LD; ++n) {
            int gr = i0 + (wt * M_LD + n) * 32; gr = gr < Ra ? gr : Ra - 32;
            m_base[n] = uniform64(FP8 ? (blocked ? a_meta + (int64_t)(gr >> 5) * (Kld / 64) * 512 : a_meta + (int64_t)gr * (Kld / 4))
                                      : blocked ? a_meta + ((int64_t)(gr >> 5) * (Kld / 64) << 8) : a_meta + (int64_t)gr * (Kld / 8));
        }
        a_kstep = blocked ? 1024 : 64;
        b_kstep = blockedB ? 1024 * (C::BK / 32) : C::BK * 2;
        m_kstep = (blocked && !FP8) ? 256 : C::META_ROW;
        if (MG) m_lane = (uint32_t)((lane >> 1) * (Kld / 8) + (((lane & 1) ^ ((lane >> 4) & 1)) << 4));      // row lane / 2, 16-byte half swizzled by (row / 8) % 2
        if (FP8 && blocked) {       // fp8 metadata units of common.hpp (m8blk_off): 512 contiguous bytes per (32 rows, 128 k), row-major inside
            m_lane = lane * 4; m_kstep = 512;
        }
    }
    // DMA loads lo .. hi - 1 of a stage's LD (compile-time bounds): they are issued one at a time between matrix instructions
    constexpr int LD = A_LD + B_LD + (FP8 ? 2 * M_LD : M_LD);
    auto brings_meta = [](int kt) { return (kt & 3) == 0; };      // MG
    static_assert(LD == C::LOADS, "loads in flight");
    constexpr bool BASED = !blocked && WM == 128;
    auto issue = [&](int kt, int stage, int lo, int hi) {
        const uint32_t sa = ring_lds + stage * C::STAGE, sb = sa + C::A_BYTES, sm = sb + C::B_BYTES;
        // the k position goes into the 32-bit per-lane offset (one vector add per operand); the bases stay put in SGPRs.  Row-major operands have metadata offsets of their own and
        // an index word for every fragment, and the large tile's accumulators and fragments leave them 24 registers: its k position of the metadata, and of A with MG, goes into the bases
        // (with registers in scratch memory / without: T = 8192, N = 8192, K = 2048 150 / 147 us; the 128 tile loses 1 % by it).
        const uint32_t kb = (uint32_t)kt * m_kstep, ko = BASED ? 0 : kb;
        const uint32_t ao = a_lane + (BASED && MG ? 0 : (uint32_t)kt * a_kstep), bo = b_lane + (uint32_t)kt * b_kstep, mo = m_lane + ko;
#pragma unroll
        for (int n = 0; n < A_LD; ++n)
            if (n >= lo && n < hi) dma16(BASED && MG ? a_base[n] + (uint32_t)kt * a_kstep : a_base[n], ao, sa + (wt * A_LD + n) * 1024);
#pragma unroll
        for (int n = 0; n < B_LD; ++n)
            if (A_LD + n >= lo && A_LD + n < hi) dma16(b_base[n], (lineB && (n & 1)) ? bo ^ 64u : bo, sb + (wt * B_LD + n) * 1024);
        if (MG) {
            // 32 bytes of each of 32 rows in one load every four stages, instead of 8 bytes, as many lines, in every stage.  Group g (stages 4 g .. 4 g + 3) arrives
            // with stage 4 g, into the buffer of group g - 2, whose last reads ended with the stage that this refill replaces.  (On blocked operands, whose
            // metadata of a stage are one line a wavefront, it gains nothing: 1840 us for 1821 in eq. (1) at T = D = 8192, F = 28672.)
            if (LD - 1 >= lo && LD - 1 < hi && brings_meta(kt))
                dma16(m_base[0], m_lane + (uint32_t)(kt >> 2) * 32, ring_lds + C::NSTAGE * C::STAGE + ((kt >> 2) & 1) * C::GROUP_BYTES + wt * 1024);
        } else
#pragma unroll
        for (int n = 0; n < M_LD; ++n) {
            if (!FP8) {
                if (A_LD + B_LD + n >= lo && A_LD + B_LD + n < hi) dma4(m_base[n] + (kb - ko), mo, sm + (wt * M_LD + n) * 256);
            } else {
                const int i = A_LD + B_LD + 2 * n;
                if (i >= lo && i < hi) dma4(m_base[n] + (kb - ko), mo, sm + (wt * M_LD + n) * 512);
                // second half of the 32 rows: the next 256 bytes of a blocked unit, or 16 rows further down a row-major array
                if (i + 1 >= lo && i + 1 < hi) dma4(m_base[n] + (blocked ? 0u : kb - ko + (uint32_t)(16 * (Kld / 4))), mo + (blocked ? 256u : 0u), sm + (wt * M_LD + n) * 512 + 256);
            }
        }
    };

    // ---- per-lane LDS offsets of the fragment reads (inside a stage): lane -> row l16 of a fragment, 16-byte chunk lq of 64 bytes; fragments are 16 rows apart ----
    const int a_off = (wm * WM + l16) * 64 + ((lq ^ swz4(l16 >> 2)) << 4);
    // blocked bf16 metadata: the lane's word of unit 32 rows serves both of its fragments; row-major: [row][8 bytes]; fp8: [row][16 bytes]
    const int m_off = MG ? C::NSTAGE * C::STAGE + (wm * WM + l16) * 32 + ((l16 >> 3) << 4) + 2 * lq
                         : C::A_BYTES + C::B_BYTES + (FP8 ? (wm * WM + l16) * 16 + 4 * lq : blocked ? wm * WM * 8 + lane * 4 : (wm * WM + l16) * 8 + 2 * lq);
    // (lineB: a row's 128 bytes are 8 chunks, lq and 4 + lq of them this lane's)
    const int b_off = C::A_BYTES + (lineB ? (wn * WN + l16) * 128 + ((lq ^ (l16 >> 1)) << 4) : (wn * WN + l16) * 64 + ((lq ^ swz4(l16 >> 2)) << 4));

    f32x4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.0f;

    // Fragments of a stage.  B alternates between two sets; an A fragment (and its index bits) is replaced by the next stage's as soon as its row of matrix
    // instructions has been issued.
    struct FragB { Frag16 b16[SPARSE ? FN : 1]; Frag8 b8[SPARSE ? 1 : FN]; };     // SPARSE: 64 k (fp8: 128) a stage, dense: 32
    Frag8 A[FM];
    constexpr bool PAIRED = SPARSE && blocked && !FP8 && !PRUNE;      // an index word for two fragments, low and high half
    int idx[FM];
    FragB B0, B1;
    uint32_t m_kt = 0;          // MG: stage whose fragments are read next
    auto read_a = [&](const unsigned char* st, int a) {
        A[a].u = *reinterpret_cast<const uint4*>(st + a_off + a * 1024);
        if (SPARSE) {
            if (MG) idx[a] = *reinterpret_cast<const uint16_t*>(ring + (m_off ^ ((m_kt & 2) << 3)) + ((m_kt & 4) ? C::GROUP_BYTES : 0) + ((m_kt & 1) << 3) + a * 512);
            else if (FP8) idx[a] = *reinterpret_cast<const uint32_t*>(st + m_off + a * 256);
            else if (!blocked) idx[a] = *reinterpret_cast<const uint16_t*>(st + m_off + a * 128);
            else if (a & 1) idx[a - 1] = *reinterpret_cast<const uint32_t*>(st + m_off + (a >> 1) * 256);
        }
    };
    // piece p of a stage's B fragments: one 16-byte read
    constexpr int BP = SPARSE ? 2 * FN : FN;
    auto read_b = [&](FragB& f, const unsigned char* st, int p) {
        if (!SPARSE) f.b8[p].u = *reinterpret_cast<const uint4*>(st + b_off + p * 1024);
        else if (lineB) f.b16[p >> 1].u[p & 1] = *reinterpret_cast<const uint4*>(st + (b_off ^ (64 * (p & 1))) + (p >> 1) * 2048);
        else f.b16[p >> 1].u[p & 1] = *reinterpret_cast<const uint4*>(st + b_off + (p & 1) * BN * 64 + (p >> 1) * 1024);
    };
    auto mma_row = [&](const FragB& f, int a) {
        const int ix = !SPARSE ? 0 : !PAIRED ? idx[a] : (a & 1) ? (int)((uint32_t)idx[a - 1] >> 16) : idx[a];
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            if (FP8)          acc[a][b] = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(A[a].q, f.b16[b].q, acc[a][b], ix, 0, 0);
            else if (!SPARSE) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[a].v, f.b8[b].v, acc[a][b], 0, 0, 0);
            else              acc[a][b] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(A[a].v, f.b16[b].v, acc[a][b], ix, 0, 0);
        }
    };
#define SB() __builtin_amdgcn_sched_barrier(0)

    // steps of this wavefront: all of them, or (KW > 1) every KW-th one from its own on.  0 for an expert without tokens (weight gradients): zeros
    const int nk = KW == 1 ? K / C::BK : (K / C::BK - kg + KW - 1) / KW;
    auto step_of = [&](int kt) { return KW == 1 ? kt : kg + kt * KW; };
    if constexpr (PRUNE) {
        const uint16_t* const row = a_vals + (int64_t)(i0 + l16) * Kld + 16 * lq;
        uint4 raw[C::NSTAGE][FM][2];
#pragma unroll
        for (int p = 0; p < C::NSTAGE; ++p)
            if (p < nk) issue(step_of(p), p, 0, LD);
#pragma unroll
        for (int p = 0; p < C::NSTAGE; ++p)
            if (p < nk)
#pragma unroll
                for (int a = 0; a < FM; ++a) {
                    const uint4* w = reinterpret_cast<const uint4*>(row + (int64_t)a * 16 * Kld + step_of(p) * 64);
                    raw[p][a][0] = w[0]; raw[p][a][1] = w[1];
                }
        wait_vmcnt<0>();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int p = 0; p < C::NSTAGE; ++p)
            if (p < nk) {
#pragma unroll
                for (int q = 0; q < BP; ++q) read_b(B0, ring + p * C::STAGE, q);
#pragma unroll
                for (int a = 0; a < FM; ++a) {
                    const uint4 w0 = raw[p][a][0], w1 = raw[p][a][1];
                    uint32_t n0, n1, n2, n3;
                    A[a].u.x = select24<PRUNE == 2>(w0.x & 0xFFFFu, w0.x >> 16, w0.y & 0xFFFFu, w0.y >> 16, n0);
                    A[a].u.y = select24<PRUNE == 2>(w0.z & 0xFFFFu, w0.z >> 16, w0.w & 0xFFFFu, w0.w >> 16, n1);
                    A[a].u.z = select24<PRUNE == 2>(w1.x & 0xFFFFu, w1.x >> 16, w1.y & 0xFFFFu, w1.y >> 16, n2);
                    A[a].u.w = select24<PRUNE == 2>(w1.z & 0xFFFFu, w1.z >> 16, w1.w & 0xFFFFu, w1.w >> 16, n3);
                    idx[a] = (int)(n0 | (n1 << 4) | (n2 << 8) | (n3 << 12));
                    mma_row(B0, a);
                }
            }
    } else if (nk > 0) {
    // The ring holds NSTAGE tiles: the one being multiplied, the next one (landed by the middle of the step,
    // when its first fragments are read) and NSTAGE - 2 in flight.  A stage is refilled right after the
    // barrier that ends its last fragment reads, so a tile has almost NSTAGE - 1 steps to arrive.
    // (KW > 1: the ring belongs to one wavefront, whose own waits order its loads and reads.)
#pragma unroll
    for (int p = 0; p < C::NSTAGE; ++p)
        if (p < nk) issue(step_of(p), p, 0, LD);
    if (nk >= C::NSTAGE) wait_vmcnt<(C::NSTAGE - 1) * (C::LOADS - (MG ? 1 : 0))>();
    else wait_vmcnt<0>();
    if (KW == 1) __syncthreads();
    else asm volatile("" ::: "memory");
#pragma unroll
    for (int a = 0; a < FM; ++a) read_a(ring, a);
#pragma unroll
    for (int p = 0; p < BP; ++p) read_b(B0, ring, p);
    int stage = 0;
    // One step = one stage = FM rows of four matrix instructions, on fragments that were read during the step before.  Behind the first row every wavefront has read
    // all of the stage and the next one has landed (barrier): the stage is refilled, and the next one's fragments are read, spread over the step: a CU takes
    // 57 bytes of loads per cycle, and a wavefront that has to wait for its turn cannot issue matrix instructions either.
    // (All loads of a refill right behind the barrier, T = D = 8192, F = 28672: 2045 us for eq. (1); spread: 1930.)  T = F = 8192: 0.81 us a stage of 51,200 bytes, of
    // which the matrix instructions alone take 0.64 at the clock that their power leaves, the loads alone 0.51 - 0.58 (0.70 - 0.83 beside ordinary stores of the outputs); two half stages of 32 x 32 x 32 instructions, their fragments half a stage ahead, took 0.90.
    // full: tiles up to kt + NSTAGE exist.  The last steps load nothing: a repeated tile in their place costs what any other does, and the epilogue waits for it
    // (T = F = 8192, D = 512, 128 tile: 90.7 -> 88.0 us for eq. (1), 74.2 -> 71.7 for eq. (4); 256 tile 0.5 %).
    auto step = [&](auto full, int kt, const FragB& Bc, FragB& Bn) {
        const int next_stage = (stage + 1 == C::NSTAGE) ? 0 : stage + 1;
        const unsigned char* sn = ring + next_stage * C::STAGE;
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            mma_row(Bc, a); SB();
            if (a == 0) {
                // this stage's fragments have arrived, and this wavefront's part of tile kt + 1 has landed
                if (!full.value && kt + C::NSTAGE - 1 >= nk) wait_vmcnt_lgkm0<0>();
                else if constexpr (MG) {
                    if (brings_meta(kt + C::NSTAGE - 1)) wait_vmcnt_lgkm0<(C::NSTAGE - 2) * C::LOADS>();
                    else wait_vmcnt_lgkm0<(C::NSTAGE - 2) * C::LOADS - 1>();
                } else wait_vmcnt_lgkm0<(C::NSTAGE - 2) * C::LOADS>();
                if (KW == 1) __builtin_amdgcn_s_barrier();
                else asm volatile("" ::: "memory");
                SB();
                if (MG) m_kt = (uint32_t)kt + 1;
            }
            if (full.value || kt + C::NSTAGE < nk) issue(step_of(kt + C::NSTAGE), stage, LD * a / FM, LD * (a + 1) / FM);
            SB();
            if (!PAIRED || (a & 1)) {           // (an index word is replaced behind the second of its rows)
                if (PAIRED) read_a(sn, a - 1);
                read_a(sn, a);
            }
            // (B's pieces behind the first five of eight rows: the next step's first row wants all of them)
            constexpr int BS = FM == 8 ? 5 : FM;
#pragma unroll
            for (int p = a < BS ? BP * a / BS : BP; p < (a < BS ? BP * (a + 1) / BS : BP); ++p) read_b(Bn, sn, p);
            SB();
        }
        stage = next_stage;
    };
    int kt = 0;
    for (; kt + 1 + C::NSTAGE < nk; kt += 2) { step(Flag<true>(), kt, B0, B1); step(Flag<true>(), kt + 1, B1, B0); }
    for (; kt + 1 < nk; kt += 2) { step(Flag<false>(), kt, B0, B1); step(Flag<false>(), kt + 1, B1, B0); }
    if (kt < nk) step(Flag<false>(), kt, B0, B1);
#undef SB
    wait_vmcnt<0>();
    }
    __syncthreads();
    // SHARE: the wavefronts of a shared tile share its epilogue too (below)
    constexpr bool SHARE = KW > 1 && (EPI == 1 || EPI == 2);
    constexpr int PART = FM * FN * 4 * 256;
    if (KW > 1 && !SHARE) {       // partial sums -> the first wavefront, in ascending order; the others are done
        static_assert((KW - 1) * PART <= GemmV2Lds<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, TL, MG, PRUNE != 0>::BYTES, "partial sums must fit in the main-loop LDS");
        if (kg > 0) {
            float* p = reinterpret_cast<float*>(smem + (kg - 1) * PART) + lane;
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) p[((a * FN + b) * 4 + r) * 64] = acc[a][b][r];
        }
        __syncthreads();
        if (kg > 0) return;
        for (int g = 1; g < KW; ++g) {
            const float* p = reinterpret_cast<const float*>(smem + (g - 1) * PART) + lane;
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[a][b][r] += p[((a * FN + b) * 4 + r) * 64];
        }
        wave_lds_sync();
    }

    if (OUT_I_CONTIG) {
        // i is the contiguous output axis and a lane owns 4 consecutive i of one j.  Stage the wave's tile
        // through LDS as [j][i] (two halves of 64 i) so that HBM sees 128-byte row segments instead of
        // 16-byte ones; the bias (indexed by i) is added before the single rounding to bf16.
        constexpr int EP = 64 * 2 + 16;
        // EPI: second tile (32 compact rows) for the transposed output
        constexpr int WAVE_LDS = (EPI != 0) ? (WN + 32) * EP : WN * EP;
        static_assert(!SHARE || (KW == 4 && FM == 4 && NH == 1), "four wavefronts, 16 tokens and two sweeps each");
        unsigned char* scratch = smem + (SHARE ? KW * PART : wt * WAVE_LDS);
        static_assert((SHARE ? KW * PART : 0) + TL::NW * WAVE_LDS <= GemmV2Lds<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, TL, MG, PRUNE != 0>::BYTES, "epilogue scratch must fit in the main-loop LDS");
        unsigned char* ttile = scratch + WN * EP;
        // EPI: i = hidden unit f, j = token t; the wave's 64 tokens are exactly one V = 64 block and each half of
        // 64 f holds 8 whole column blocks, so the V:N:M work is wave-local.
        const int t0 = j0 + wn * WN;
        const int nblk = Ra >> 3;
        const int64_t F = Ra;
        uint32_t nib_h0 = 0;                                  // M = 64: the metadata nibble of the first half waits for the second's
        // Of the eight sweeps over a half's tokens (lane = (token, column block)) this wavefront does NSW from it0 on.  On a shared tile the scores are every wavefront's own: one has to
        // add the 64 tokens in order, and the others would wait for it.  (All of the epilogue in the first wavefront: T = 64, D = 2048, F = 8192 a forward call on packed weights 24.2 us, now 23.0; the fp8 step of that size 97.5, 91.9.)
        constexpr int NSW = SHARE ? 2 : 8;
        const int it0 = SHARE ? 2 * kg : 0;
        // The lane's 16 bias values of each half (eq. (4) has none), and (EPI 2) the saved column offsets, metadata and y1 of its 8 sweeps: all fetched here, for
        // both halves.  Loads and stores share one in-order counter, so a load issued after the first half's stores would wait for all of them
        // (and for its own latency) in the middle of the epilogue.
        constexpr bool BIAS = EPI != 2 && EPI != 4 && !GEN_B;
        float4 bb_all[NH][4];
        uint32_t pre_cw[NH], pre_m[NH], pre_y_all[NH][NSW];
        const uint32_t amax_seen = (FP8 && EPI != 0) ? amax_slot_peek(ep.amax) : 0u;
        float vmax_tile = 0.0f;                                 // fp8: largest survivor magnitude of the wave's tile
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int f0 = i0 + wm * WM + h * 64;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                bb_all[h][a] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (BIAS && bias) {
                    int i = f0 + a * 16 + 4 * lq; i = i < Ra ? i : Ra - 4;
                    // EPI 3: compact column i of the expert is hidden unit (i / 4) * M + 4 e + i % 4 (bias already points at 4 e)
                    bb_all[h][a] = *reinterpret_cast<const float4*>(EPI == 3 ? bias + ((int64_t)(i >> 2) << ep.logM) : bias + i);
                }
            }
            pre_cw[h] = 0x03020100u;
            pre_m[h] = 0;
            if (EPI == 2 && t0 < Rb && f0 < Ra) {
                pre_cw[h] = *reinterpret_cast<const uint32_t*>(ep.colidx + ((int64_t)(t0 >> 6) * nblk + (f0 >> 3) + (lane & 7)) * 4);
                // lane -> token lane / 8 + 8 (lane % 8): sweep `it` finds its eight nibbles in lane % 8 = it of its group of 8 lanes
                pre_m[h] = *reinterpret_cast<const uint32_t*>(ep.mcb + (FP8 ? mcb8_off(t0, f0 >> 6, F) : mcb_off(t0, f0 >> 6, F)) + ((lane >> 3) + 8 * (lane & 7)) * (FP8 ? 8 : 4));
                const uint32_t* kp = reinterpret_cast<const uint32_t*>(ep.ykept) + ykept_off(t0, f0 >> 3, F);
#pragma unroll
                for (int it = 0; it < NSW; ++it) pre_y_all[h][it] = kp[lane + (it0 + it) * 64];
            }
        }
        // (the same for the backward epilogue of the wide blocks)
        constexpr int GNB = (GEN_F || GEN_B) ? (64 >> LOGM) : 1;
        uint32_t gpre_cb[NH], gpre_m[NH][GNB], gpre_y[NH][GNB];
        if (GEN_B) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const int f0 = i0 + wm * WM + h * 64;
                gpre_cb[h] = 0x03020100u;
                if (t0 < Rb && f0 < Ra) {
                    const int b = lane & (GNB - 1), r_lane = lane >> (6 - LOGM);
                    const int64_t blk = (f0 >> LOGM) + b;
                    gpre_cb[h] = *reinterpret_cast<const uint32_t*>(ep.colidx + ((int64_t)(t0 >> 6) * (F >> LOGM) + blk) * 4);
                    const uint32_t* kp = reinterpret_cast<const uint32_t*>(ep.ykept) + ((((int64_t)(t0 >> 6) * (F >> 6) + (f0 >> 6)) << 6) + r_lane) * GNB + b;
                    const uint8_t* mp = ep.meta + (int64_t)(t0 + r_lane) * (F >> (LOGM + 1)) + (blk >> 1);
#pragma unroll
                    for (int sw = 0; sw < GNB; ++sw) {
                        gpre_m[h][sw] = mp[(int64_t)sw * (1 << LOGM) * (F >> (LOGM + 1))];
                        gpre_y[h][sw] = kp[sw * (1 << LOGM) * GNB];
                    }
                }
            }
        }
        bool tok_ok[FN];                                       // EPI 3: padding rows of the permuted token order come out as zeros
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            tok_ok[b] = true;
            if (EPI == 3) { int j = t0 + b * 16 + l16; j = j < Rb ? j : Rb - 1; tok_ok[b] = ep.perm[j] >= 0; }
        }
        // Column scores of the half tile: lane = column, strict ascending-row float32 sum of y2.  A transposing read hands every lane four rows of its column.
        // (One 2-byte read per row: 64 reads and 450 vector instructions instead of 16 and 350.)
        auto column_scores = [&]() {
            const unsigned char* p = scratch + ((lane & 15) >> 2) * EP + (lane >> 4) * 32 + (lane & 3) * 8;
            float sc = 0.0f;
#pragma unroll
            for (int r = 0; r < WN; r += 4) {
                const uint2 w = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + r * EP)));
                const uint32_t u = sqrelu2(w.x), v = sqrelu2(w.y);
                sc = sc + __uint_as_float(u << 16);
                sc = sc + __uint_as_float(u & 0xFFFF0000u);
                sc = sc + __uint_as_float(v << 16);
                sc = sc + __uint_as_float(v & 0xFFFF0000u);
            }
            return sc;
        };
        const uint32_t s_off = (uint32_t)(SHARE ? KW * PART : wt * WAVE_LDS);      // the scratch tile as an offset into smem (a multiple of 16, and so are its rows)
        auto lds_u16 = [&](uint32_t off) { return (uint32_t)*reinterpret_cast<const uint16_t*>(smem + off); };
        // EPI 3, 4: the survivors as the dense transposed matrix at[f, t] (row length ep.at_ld), zeros at the dropped positions: the A operand of the
        // experts' weight gradients.  The half tile is turned in place (its rows have been read): two tokens make a word of one of the four rows of
        // the lane's group; the 16-byte chunks of a row are permuted by (row / 16) % 4 so that the 64 words of a store fall into 64 LDS banks.
        // (As a pass of its own over the packed matrix: 15 us at 8192 rows, 2048 columns and 4 experts.)
        auto transposed_out = [&](const uint32_t (&v)[16], const uint32_t (&nib)[2], int f0, bool valid) {
            const int g = lane & 15;
            wave_lds_sync();
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const uint32_t n = nib[p >> 2] >> (8 * (p & 3)), a0 = n & 3u, a1 = (n >> 2) & 3u, b0 = (n >> 4) & 3u, b1 = (n >> 6) & 3u;
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) {
                    const uint32_t lo = c == a0 ? v[2 * p] & 0xFFFFu : c == a1 ? v[2 * p] >> 16 : 0u;
                    const uint32_t hi = c == b0 ? v[2 * p + 1] << 16 : c == b1 ? v[2 * p + 1] & 0xFFFF0000u : 0u;
                    *reinterpret_cast<uint32_t*>(scratch + (4 * g + c) * EP + ((p ^ (g >> 2)) * 4 + (lane >> 4)) * 4) = lo | hi;
                }
            }
            wave_lds_sync();
            store_between(ep.stream, [&](auto store) {
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const int row = p * 8 + (lane >> 3), ch = lane & 7;
                    if (valid) store(ep.at + blk_off(f0 + row, t0 + ch * 8, ep.at_ld / 32), *reinterpret_cast<const uint4*>(scratch + row * EP + (ch ^ ((row >> 4) & 3)) * 16));
                }
            });
        };
        // and as the packed rows.  One branch for all sixteen stores: one in every sweep holds the next sweep's LDS reads back (T = 64, D = 256, F = 1024, M = 8: eq. (1) 14.4 us, so 12.8; eqs. (4),
        // (3) 11.1 and 9.6; the step 53.8 and 50.4).
        auto rows_out = [&](const uint32_t (&v)[16], int f0, bool valid) {
            if (!valid) return;                // (runs of tokens are whole blocks of 64)
            uint16_t* const p = ep.vals + (int64_t)(t0 + 2 * (lane >> 4)) * (F / 2) + (f0 >> 1) + 2 * (lane & 15);
            store_between(ep.stream, [&](auto store) {
#pragma unroll
                for (int it = 0; it < 16; ++it) store(reinterpret_cast<uint32_t*>(p + (int64_t)(8 * (it >> 1) + (it & 1)) * (F / 2)), v[it]);
            });
        };
        const bool stream = !FP8 && ep.stream;
        auto tile_sync = [&]() { if (SHARE) __syncthreads(); else wave_lds_sync(); };
        f32x4 mine[4];                                         // SHARE: the sums, in the order of the shares of the contraction, for the 16 tokens of fragment kg
        if (SHARE) {
            f32x4* p = reinterpret_cast<f32x4*>(smem) + lane;
#pragma unroll
            for (int b = 0; b < FN; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) p[(kg * FN * 4 + b * 4 + a) * 64] = acc[a][b];
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                mine[a] = p[(kg * 4 + a) * 64];
#pragma unroll
                for (int g = 1; g < KW; ++g) mine[a] += p[((g * FN + kg) * 4 + a) * 64];
            }
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int f0 = i0 + wm * WM + h * 64;
            const bool valid = t0 < Rb && f0 < Ra;
            float4 (&bb)[4] = bb_all[h];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < (SHARE ? 1 : FN); ++b) {
                    f32x4 v = SHARE ? mine[a] : acc[4 * h + a][b];
                    const int row = (SHARE ? kg : b) * 16 + l16;
                    const float al = FP8 ? alpha : 1.0f;
                    // (codes were multiplied: the product of the two tensor scales comes first, one rounding, then the bias)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float w = r == 0 ? bb[a].x : r == 1 ? bb[a].y : r == 2 ? bb[a].z : bb[a].w;
                        v[r] = !BIAS ? v[r] * al : FP8 ? v[r] * alpha + w : v[r] + w;
                    }
                    // i = a * 16 + 4 lq .. + 3 inside the 64-wide half
                    *reinterpret_cast<uint2*>(scratch + row * EP + (a * 16 + 4 * lq) * 2) = tok_ok[b] ? make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3])) : make_uint2(0u, 0u);
                }
            if (EPI == 1 || EPI == 2 || GEN_F || GEN_B) {
#pragma unroll
                for (int q = 0; q < (32 * EP / (SHARE ? KW : 1) + 1023) / 1024; ++q) {
                    const int at = (SHARE ? q * 64 * KW + tid : q * 64 + lane) * 16;
                    if (at < 32 * EP) *reinterpret_cast<uint4*>(ttile + at) = make_uint4(0, 0, 0, 0);
                }
            }
            tile_sync();
            auto dense_out = [&](auto store) {
#pragma unroll
                for (int p = 0; p < (EPI == 1 || EPI == 2 ? NSW : WN / 8); ++p) {
                    const int row = (it0 + p) * 8 + (lane >> 3), ch = lane & 7;
                    const int j = t0 + row, i = f0 + ch * 8;
                    if (j < Rb && i < Ra) {
                        const uint4 w = *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16);
                        if (EPI == 0 && grp.map_logM) {     // 8 consecutive compact columns = two groups of four hidden units, M apart
                            uint16_t* o = out + (int64_t)j * ldo + ((int64_t)(i >> 2) << grp.map_logM) + 4 * expert_id;
                            *reinterpret_cast<uint2*>(o) = make_uint2(w.x, w.y);
                            *reinterpret_cast<uint2*>(o + ((int64_t)1 << grp.map_logM)) = make_uint2(w.z, w.w);
                        } else {
                            store(out + (int64_t)j * ldo + i, w);
                        }
                    }
                }
            };
            // (EPI 3: y1 at the experts' hidden units, which eq. (4)'s epilogue reads.  Non-temporal at every size: T = 4096, D = 1024, F = 4096, M = 8 175.8 us the step, so 172.1;
            // T = 10240, D = 576, F = 2560 195.6 and 191.8.)
            if (EPI == 0 || EPI == 3) { if (EPI == 0 || ep.store_dense) store_between(ep.stream, dense_out); }
            else if (ep.store_dense) dense_out([](uint16_t* p, const uint4& w) { store_out(p, w); });      // (for inspection: nothing reads it)
            if (EPI == 3) {
                // lane = (tokens t = 2 (lane / 16) + 8 (it / 2) + it % 2, group of four compact columns g = lane % 16): eq. (2), then the 2:4 rule
                const int g = lane & 15;
                uint32_t vv[16], nn[2] = {0u, 0u};
#pragma unroll
                for (int it = 0; it < 16; ++it) {
                    const int t = 2 * (lane >> 4) + 8 * (it >> 1) + (it & 1);
                    const uint2 w = *reinterpret_cast<const uint2*>(scratch + t * EP + g * 8);
                    uint32_t nib, low, high;
                    const uint32_t v = pick24_pos(sqrelu2(w.x), sqrelu2(w.y), {3u, 2u, 1u, 0u}, low, high);
                    nib = ((low & 3u) | ((high & 3u) << 2)) ^ 0xFu;
                    vv[it] = v; nn[it >> 3] |= nib << (4 * (it & 7));
                    uint32_t mw = nib | (row_shl<1>(nib) << 4);            // metadata of 8 groups -> one 32-bit store from every eighth lane
                    mw |= row_shl<2>(mw) << 8;
                    mw |= row_shl<4>(mw) << 16;
                    if (valid && t0 + t < Rb) {
                        if ((g & 7) == 0) *reinterpret_cast<uint32_t*>(ep.meta + (int64_t)(t0 + t) * (F / 8) + (f0 >> 3) + (g >> 1)) = mw;
                        if (ep.v24) {       // the same packed matrix in the blocked operand layout (A operand of eqs. (3), (7) over the expert's run)
                            *reinterpret_cast<uint32_t*>(ep.v24 + blk_off(t0 + t, (f0 >> 1) + 2 * g, F / 64)) = v;
                            if ((g & 3) == 0) *reinterpret_cast<uint16_t*>(ep.m24 + mblk_off(t0 + t, f0 + 4 * g, F / 64)) = (uint16_t)mw;
                        }
                    }
                }
                rows_out(vv, f0, valid);
                if (ep.at) transposed_out(vv, nn, f0, valid);
            }
            if (EPI == 4) {
                // eq. (6) on the compact tile: lane = (token, group of four compact columns); the two kept positions come from the
                // forward pass's metadata, y1 from the stored compact y1c (ep.ykept); dy2 is the bf16-rounded tile in LDS
                const int g = lane & 15;
                uint2 yv[16];
                uint32_t mb[16], vv[16], nn[2] = {0u, 0u};
#pragma unroll
                for (int it = 0; it < 16; ++it) {
                    const int t = 2 * (lane >> 4) + 8 * (it >> 1) + (it & 1);
                    const bool ok = valid && t0 + t < Rb;
                    yv[it] = ok ? *reinterpret_cast<const uint2*>(ep.ykept + (int64_t)(t0 + t) * F + f0 + 4 * g) : make_uint2(0u, 0u);
                    mb[it] = ok ? ep.meta[(int64_t)(t0 + t) * (F / 8) + (f0 >> 3) + (g >> 1)] : 0x44u;
                }
#pragma unroll
                for (int it = 0; it < 16; ++it) {
                    const int t = 2 * (lane >> 4) + 8 * (it >> 1) + (it & 1);
                    const uint2 w = *reinterpret_cast<const uint2*>(scratch + t * EP + g * 8);
                    const uint32_t nib = (mb[it] >> (4 * (g & 1))) & 0xFu, p0 = nib & 3u, p1 = nib >> 2;
                    const uint32_t d0 = ((p0 >> 1) ? w.y : w.x) >> (16 * (p0 & 1)), d1 = ((p1 >> 1) ? w.y : w.x) >> (16 * (p1 & 1));
                    const uint32_t y0 = ((p0 >> 1) ? yv[it].y : yv[it].x) >> (16 * (p0 & 1)), y1 = ((p1 >> 1) ? yv[it].y : yv[it].x) >> (16 * (p1 & 1));
                    const float ya = bf2f(y0 & 0xFFFFu), yb = bf2f(y1 & 0xFFFFu);
                    const uint32_t v = f2bf2(2.0f * bf2f(d0 & 0xFFFFu) * (ya > 0.0f ? ya : 0.0f), 2.0f * bf2f(d1 & 0xFFFFu) * (yb > 0.0f ? yb : 0.0f));
                    if (valid && t0 + t < Rb) *reinterpret_cast<uint32_t*>(ep.v24 + blk_off(t0 + t, (f0 >> 1) + 2 * g, F / 64)) = v;
                    vv[it] = v; nn[it >> 3] |= nib << (4 * (it & 7));
                }
                rows_out(vv, f0, valid);
                if (ep.at) transposed_out(vv, nn, f0, valid);
            }
            if (GEN_F || GEN_B) {
                // Blocks of M = 16 / 32 / 64 columns (Table 5): the wave's 64 tokens x 64 hidden units hold NB = 64 / M whole blocks.
                // Lane = column for the ordered scores and the ranking inside a block; lane = (token, block) for the per-row 2:4 choice,
                // block = lane % NB in every sweep.  The survivors also go into the compacted transposed tile of the weight-gradient GEMM,
                // in the SAME format as for M = 8 (4 rows per group of 8 hidden units + one kept-column mask byte per group): a block of
                // M columns keeps 4, so none of its M / 8 groups keeps more than 4; row = 4 * group + number of kept units below it.
                constexpr int M = 1 << LOGM, NB = 64 >> LOGM;
                const int64_t nblkM = F >> LOGM, blk0 = f0 >> LOGM;
                const int b = lane & (NB - 1);
                uint32_t cb;                                              // the four kept column offsets of block b
                unsigned long long bmask;                                 // and the same as a bit mask over the block's M columns
                if (GEN_F) {
                    const float sc = column_scores();
                    const int c = lane & (M - 1), base = lane - c;
                    const unsigned long long kept = __ballot(keep4_of<M>(__float_as_uint(sc), lane));
                    unsigned long long bits = (M == 64) ? kept : ((kept >> base) & ((1ull << (M & 63)) - 1ull));
                    const unsigned long long mine = bits;
                    uint32_t cw = 0;
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        cw |= (uint32_t)__builtin_ctzll(bits) << (8 * n);
                        bits &= bits - 1ull;
                    }
                    if (valid && c < (ep.at_kept ? 1 : M / 8)) {          // lane c of a block: its column offsets (c = 0) and the mask byte of its group c of 8 hidden units
                        if (c == 0) *reinterpret_cast<uint32_t*>(ep.colidx + ((int64_t)(t0 >> 6) * nblkM + blk0 + (lane >> LOGM)) * 4) = cw;
                        if (!ep.at_kept) ep.kmask[(int64_t)(t0 >> 6) * (F >> 3) + (f0 >> 3) + (lane >> LOGM) * (M / 8) + c] = (uint8_t)(mine >> (8 * c));
                    }
                    cb = (uint32_t)__shfl((int)cw, b << LOGM, 64);
                    bmask = (unsigned long long)(uint32_t)__shfl((int)(uint32_t)mine, b << LOGM, 64);
                    if (M == 64) bmask |= (unsigned long long)(uint32_t)__shfl((int)(uint32_t)(mine >> 32), b << LOGM, 64) << 32;
                } else {
                    cb = gpre_cb[h];
                    bmask = (1ull << (cb & 0xFFu)) | (1ull << ((cb >> 8) & 0xFFu)) | (1ull << ((cb >> 16) & 0xFFu)) | (1ull << (cb >> 24));
                }
                const uint32_t q0 = (cb & 0xFFu) * 2, q1 = ((cb >> 8) & 0xFFu) * 2, q2 = ((cb >> 16) & 0xFFu) * 2, q3 = (cb >> 24) * 2;
                const uint32_t tag[4] = {0x300u | q0, 0x200u | q1, 0x100u | q2, q3};      // (pick24_pos: position from the end, byte of the column)
                const int r_lane = lane >> (6 - LOGM);                    // token of sweep 0; sweep s adds s * M
                // survivors of (token, block): a pair of bf16, or (fp8 operands) a pair of codes
                uint32_t* vals_p = reinterpret_cast<uint32_t*>(ep.vals) + (int64_t)(t0 + r_lane) * (F >> LOGM) + blk0 + b;
                uint16_t* codes_p = ep.vals + (int64_t)(t0 + r_lane) * (F >> LOGM) + blk0 + b;
                float vmax = 0.0f;                                        // fp8: largest survivor magnitude of this half tile
                uint32_t* kept_p = reinterpret_cast<uint32_t*>(ep.ykept) + ((((int64_t)(t0 >> 6) * (F >> 6) + (f0 >> 6)) << 6) + r_lane) * NB + b;
                uint8_t* meta_p = ep.meta + (int64_t)(t0 + r_lane) * (F >> (LOGM + 1)) + ((blk0 + b) >> 1);
                const uint32_t (&pre_m)[GNB] = gpre_m[h];                 // backward: saved metadata and y1 of the sweeps (fetched above)
                const uint32_t (&pre_y)[GNB] = gpre_y[h];
                if (valid) {
#pragma unroll
                    for (int sw = 0; sw < NB; ++sw) {
                        const int t = r_lane + sw * M;
                        const unsigned char* row = scratch + t * EP + (b << LOGM) * 2;
                        uint32_t v, nib;
                        if (GEN_F) {
                            const uint32_t ro = s_off + t * EP + (b << LOGM) * 2;
                            uint32_t low, high;
                            v = pick24_pos(sqrelu2(lds_u16(ro + q0) | (lds_u16(ro + q1) << 16)), sqrelu2(lds_u16(ro + q2) | (lds_u16(ro + q3) << 16)), tag, low, high);
                            nib = (((low >> 8) & 3u) | (((high >> 8) & 3u) << 2)) ^ 0xFu;
                            const uint32_t k0 = lds_u16(ro + (low & 0xFFu)), k1 = lds_u16(ro + (high & 0xFFu));
                            if (FP8) codes_p[(int64_t)sw * M * (F >> LOGM)] = (uint16_t)fp8_enc2(bf2f(v & 0xFFFFu), bf2f(v >> 16), ep.inv_out);
                            else vals_p[(int64_t)sw * M * (F >> LOGM)] = v;
                            kept_p[sw * M * NB] = k0 | (k1 << 16);
                            // two blocks share a metadata byte: neighbours in the lane order (M = 16, 32) or the two halves of the wave tile (M = 64)
                            if (LOGM == 4) {
                                uint32_t mw = nib | (row_shl<1>(nib) << 4);
                                mw |= row_shl<2>(mw) << 8;
                                if (b == 0) *reinterpret_cast<uint16_t*>(meta_p + (int64_t)sw * M * (F >> (LOGM + 1))) = (uint16_t)mw;
                            } else if (LOGM == 5) {
                                const uint32_t mw = nib | (row_shl<1>(nib) << 4);
                                if (b == 0) meta_p[(int64_t)sw * M * (F >> (LOGM + 1))] = (uint8_t)mw;
                            } else {
                                if (h == 0) nib_h0 = nib;
                                else meta_p[0] = (uint8_t)(nib_h0 | (nib << 4));
                            }
                        } else {
                            const uint32_t yk = pre_y[sw];
                            nib = (pre_m[sw] >> (4 * ((blk0 + b) & 1))) & 0xFu;
                            const uint32_t o0 = (cb >> (8 * (nib & 3u))) & 0xFFu, o1 = (cb >> (8 * (nib >> 2))) & 0xFFu;
                            const float d0 = bf2f(*reinterpret_cast<const uint16_t*>(row + o0 * 2));
                            const float d1 = bf2f(*reinterpret_cast<const uint16_t*>(row + o1 * 2));
                            const float ya = bf2f(yk & 0xFFFFu), yb = bf2f(yk >> 16);
                            v = f2bf2(2.0f * d0 * (ya > 0.0f ? ya : 0.0f), 2.0f * d1 * (yb > 0.0f ? yb : 0.0f));
                            if (FP8) codes_p[(int64_t)sw * M * (F >> LOGM)] = (uint16_t)fp8_enc2(bf2f(v & 0xFFFFu), bf2f(v >> 16), ep.inv_out);
                            else vals_p[(int64_t)sw * M * (F >> LOGM)] = v;
                        }
                        if (FP8) vmax = __builtin_fmaxf(vmax, __builtin_fmaxf(__builtin_fabsf(bf2f(v & 0xFFFFu)), __builtin_fabsf(bf2f(v >> 16))));
                        // compact row of a survivor at column o of the block: group (b M + o) / 8 of the half tile, position = kept columns of
                        // that group below o
                        const uint32_t o0 = (cb >> (8 * (nib & 3u))) & 0xFFu, o1 = (cb >> (8 * (nib >> 2))) & 0xFFu;
                        const uint32_t g0 = (uint32_t)(bmask >> (o0 & ~7u)) & 0xFFu, g1 = (uint32_t)(bmask >> (o1 & ~7u)) & 0xFFu;
                        // (at_kept: the block's four kept rows)
                        const uint32_t r0 = ep.at_kept ? 4 * b + (nib & 3u) : ((b * (M / 8) + (o0 >> 3)) << 2) + __builtin_popcount(g0 & ((1u << (o0 & 7u)) - 1u));
                        const uint32_t r1 = ep.at_kept ? 4 * b + (nib >> 2) : ((b * (M / 8) + (o1 >> 3)) << 2) + __builtin_popcount(g1 & ((1u << (o1 & 7u)) - 1u));
                        *reinterpret_cast<uint16_t*>(ttile + r0 * EP + t * 2) = (uint16_t)(v & 0xFFFFu);
                        *reinterpret_cast<uint16_t*>(ttile + r1 * EP + t * 2) = (uint16_t)(v >> 16);
                    }
                }
                if (FP8) vmax_tile = __builtin_fmaxf(vmax_tile, vmax);
                wave_lds_sync();
                if (!FP8 && ep.at_kept) {       // 4 NB kept rows x 8 chunks of 8 tokens; consecutive lanes take consecutive rows
                    const int64_t R32 = F >> (LOGM + 3);
#pragma unroll
                    for (int q = 0; q < (NB + 1) / 2; ++q) {
                        const int e = q * 64 + lane, rr = e % (4 * NB), c8 = e / (4 * NB);
                        const int64_t R = (f0 >> LOGM) * 4 + rr;
                        if (valid && c8 < 8)
                            *reinterpret_cast<uint4*>(ep.at + kept_off(R, t0 + 8 * c8, R32)) =
                                *reinterpret_cast<const uint4*>(ttile + rr * EP + c8 * 16);
                    }
                } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {          // 2 groups of 16 compact rows x 2 chunks of 32 tokens, 1 KB each
                    const int fr = (q >> 1) * 16 + (lane >> 2), tc = (q & 1) * 32 + (lane & 3) * 8;
                    const uint4 w = *reinterpret_cast<const uint4*>(ttile + fr * EP + tc * 2);
                    if (FP8 && ep.at_fp8) {     // fp8 weight gradients: codes, as in the M = 8 epilogues below
                        if (valid)
                            *reinterpret_cast<uint2*>(ep.at + blk_off(f0 / 2 + fr, (t0 + tc) / 2, tok_ld / 64)) =
                                make_uint2(fp8_enc2(bf2f(w.x & 0xFFFFu), bf2f(w.x >> 16), ep.inv_out) | (fp8_enc2(bf2f(w.y & 0xFFFFu), bf2f(w.y >> 16), ep.inv_out) << 16),
                                           fp8_enc2(bf2f(w.z & 0xFFFFu), bf2f(w.z >> 16), ep.inv_out) | (fp8_enc2(bf2f(w.w & 0xFFFFu), bf2f(w.w >> 16), ep.inv_out) << 16));
                    } else if (valid) {
                        *reinterpret_cast<uint4*>(ep.at + blk_off(f0 / 2 + fr, t0 + tc, tok_ld / 32)) = w;
                    }
                }
                }
            }
            if (EPI == 1 || EPI == 2) {
                const int bl = lane & 7;                                  // column block handled in the per-row pass
                const int64_t blk_g = (f0 >> 3) + bl;
                uint32_t cw;                                              // the four kept column offsets of block bl
                if (EPI == 1) {
                    const unsigned long long kept = __ballot(keep4_of_8(__float_as_uint(column_scores()), lane));
                    const uint32_t bits = (uint32_t)(kept >> (lane & ~7)) & 0xFFu;
                    // kept column number n of the block goes to byte n of the word of all of its lanes
                    uint32_t mine = (bits >> bl) & 1u ? (uint32_t)bl << (8 * __builtin_popcount(bits & ((1u << bl) - 1u))) : 0u;
                    mine = or_of_8(mine);
                    if (valid && bl == 0 && kg == 0)
                    {
                        *reinterpret_cast<uint32_t*>(ep.colidx + ((int64_t)(t0 >> 6) * nblk + (f0 >> 3) + (lane >> 3)) * 4) = mine;
                        ep.kmask[(int64_t)(t0 >> 6) * nblk + (f0 >> 3) + (lane >> 3)] = (uint8_t)bits;
                    }
                    cw = (uint32_t)__shfl((int)mine, bl * 8, 64);
                    if (FP8 && ep.cixt) {       // fp8 form: 16 words per 128 hidden units, word q = (h, p); this half of them (64 hidden units) fills two bytes
                        const int q = lane & 15, hq = q >> 3, pq = q & 7, hf = (f0 >> 6) & 1;
                        const uint32_t b0 = ((uint32_t)__shfl((int)mine, (4 * hq + (pq >> 2)) * 8, 64) >> (8 * (pq & 3))) & 0xFFu;
                        const uint32_t b1 = ((uint32_t)__shfl((int)mine, (4 * hq + 2 + (pq >> 2)) * 8, 64) >> (8 * (pq & 3))) & 0xFFu;
                        if (valid && lane < 16 && kg == 0)
                            *reinterpret_cast<uint16_t*>(ep.cixt + cixt8_off(t0 >> 6, f0 >> 7, tok_ld >> 6) + q * 4 + 2 * hf) = (uint16_t)(b0 | (b1 << 8));
                    }
                    if (!FP8 && ep.cixt) {      // the same offsets regrouped for the transposing reads of gemm_vnm8.hip: word q = (h, r), byte j
                        const int q = lane & 7, hq = q >> 2, rq = q & 3;
                        uint32_t dw = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            dw |= (((uint32_t)__shfl((int)mine, (4 * (j >> 1) + (j & 1) + 2 * hq) * 8, 64) >> (8 * rq)) & 0xFFu) << (8 * j);
                        if (valid && lane < 8 && kg == 0) *reinterpret_cast<uint32_t*>(ep.cixt + cixt_off(t0 >> 6, f0 >> 6, tok_ld >> 6) + q * 4) = dw;
                    }
                } else {
                    cw = pre_cw[h];
                }
                // Per-row pass: lane = (column block bl, token t); 8 tokens per sweep, 8 sweeps.  Every output but the canonical copies is a run of
                // consecutive bytes per sweep: a wave-uniform base, 4 bytes per lane and constant offsets, no address arithmetic.
                // (This pass, the choice and the scores together, T = D = 8192, F = 28672: 1950 -> 1895 us for eq. (1), 1815 -> 1775 for eq. (4); 18 -> 12 us a tile.)
                uint32_t* vals_p = reinterpret_cast<uint32_t*>(ep.vals) + ((int64_t)(t0 + 8 * it0 + (lane >> 3)) * (F / 4) + blk_g * 2) / 2;
                uint32_t* kept_p = reinterpret_cast<uint32_t*>(ep.ykept) + ykept_off(t0, f0 >> 3, F) + it0 * 64;
                // operands of eq. (3) / eq. (7) on the V:2:8 kernel (gemm_vnm8.hip); sweep it: + (it / 4) 32-token groups + 8 (it % 4) tokens
                uint32_t* vcb_p = FP8 ? nullptr : reinterpret_cast<uint32_t*>(ep.vcb + vcb_off(t0, f0 >> 3, F));
                uint8_t* vcb8_p = FP8 ? reinterpret_cast<uint8_t*>(ep.vcb) + vcb8_off(t0 + (lane >> 3), blk_g, F) : nullptr;   // (the lane of block 0 stores its row's 8 pairs of codes)
                const uint32_t c2 = cw * 2;                                 // the four kept columns as byte offsets
                const uint32_t q0 = c2 & 0xFFu, q1 = (c2 >> 8) & 0xFFu, q2 = (c2 >> 16) & 0xFFu, q3 = c2 >> 24;
                const uint32_t tag[4] = {0x30u | q0, 0x20u | q1, 0x10u | q2, q3};
                const uint32_t row0 = s_off + (8 * it0 + (lane >> 3)) * EP + bl * 16;    // (rows and blocks are multiples of 16 bytes: a byte of c2 goes in by OR)
                const uint32_t tt0 = s_off + WN * EP + bl * 4 * EP + (8 * it0 + (lane >> 3)) * 2;
                const uint32_t (&pre_y)[NSW] = pre_y_all[h];
                uint32_t v[NSW], pos[NSW];                                     // of every sweep: the survivors, their positions among the four kept columns
                // (all reads of the tile come first: a sweep that branches or writes LDS waits for its own two LDS latencies before the next one starts)
                if (EPI == 1) {
                    uint32_t low[NSW], high[NSW], mword = 0;                   // mword: the metadata of token lane / 8 + 8 bl
#pragma unroll
                    for (int it = 0; it < NSW; ++it) {
                        const uint32_t r = row0 + it * 8 * EP;
                        v[it] = pick24_pos(sqrelu2(lds_u16(r + q0) | (lds_u16(r + q1) << 16)), sqrelu2(lds_u16(r + q2) | (lds_u16(r + q3) << 16)), tag, low[it], high[it]);
                    }
#pragma unroll
                    for (int it = 0; it < NSW; ++it) {
                        pos[it] = (((low[it] >> 4) & 3u) | ((high[it] >> 2) & 0xCu)) ^ 0xFu;
                        const uint32_t mw = or_of_8(pos[it] << (4 * bl));   // the row's 8 blocks
                        mword = bl == it0 + it ? mw : mword;
                        low[it] = lds_u16(((low[it] & 15u) | row0) + it * 8 * EP) | (lds_u16(((high[it] & 15u) | row0) + it * 8 * EP) << 16);
                    }
                    if (valid) {
                        store_between(stream, [&](auto store) {
#pragma unroll
                            for (int it = 0; it < NSW; ++it) store(kept_p + lane + it * 64, low[it]);
                        });
                        const uint32_t mt = (lane >> 3) + 8 * bl;
                        if (!SHARE || bl >> 1 == kg) *reinterpret_cast<uint32_t*>(ep.meta + (int64_t)t0 * (F / 16) + (f0 >> 4) + mt * (uint32_t)(F / 16)) = mword;
                        if (!SHARE || bl >> 1 == kg) *reinterpret_cast<uint32_t*>(ep.mcb + (FP8 ? mcb8_off(t0, f0 >> 6, F) : mcb_off(t0, f0 >> 6, F)) + mt * (FP8 ? 8 : 4)) = mword;
                    }
                } else {
                    const uint32_t m = pre_m[h];
                    if constexpr (SHARE) {
                        pos[0] = (uint32_t)__shfl((int)m, (lane & 56) + it0, 64); pos[1] = (uint32_t)__shfl((int)m, (lane & 56) + it0 + 1, 64);
                    } else {
                        pos[0] = bcast_of_8<0>(m); pos[1] = bcast_of_8<1>(m); pos[2] = bcast_of_8<2>(m); pos[3] = bcast_of_8<3>(m);
                        pos[4] = bcast_of_8<4>(m); pos[5] = bcast_of_8<5>(m); pos[6] = bcast_of_8<6>(m); pos[7] = bcast_of_8<7>(m);
                    }
#pragma unroll
                    for (int it = 0; it < NSW; ++it) {
                        pos[it] >>= 4 * bl;
                        const float d0 = bf2f(lds_u16(((__builtin_amdgcn_alignbyte(0u, c2, pos[it]) & 15u) | row0) + it * 8 * EP));
                        const float d1 = bf2f(lds_u16(((__builtin_amdgcn_alignbyte(0u, c2, pos[it] >> 2) & 15u) | row0) + it * 8 * EP));
                        const uint32_t yk = pre_y[it];
                        v[it] = f2bf2(2.0f * d0 * relu1(__uint_as_float(yk << 16)), 2.0f * d1 * relu1(__uint_as_float(yk & 0xFFFF0000u)));
                    }
                }
                // transposed tile for the weight-gradient GEMM, compacted to the block's four kept hidden units:
                // row = 4 * block + position among the kept units, column = token
#pragma unroll
                for (int it = 0; it < NSW; ++it) {
                    *reinterpret_cast<uint16_t*>(smem + __umul24(pos[it] & 3u, EP) + tt0 + it * 16) = (uint16_t)(v[it] & 0xFFFFu);
                    *reinterpret_cast<uint16_t*>(smem + __umul24((pos[it] >> 2) & 3u, EP) + tt0 + it * 16) = (uint16_t)(v[it] >> 16);
                }
                if (valid && ep.vals) {    // (lean form: no canonical copy; vcb and the compact transpose carry the values)
#pragma unroll
                    for (int it = 0; it < NSW; ++it) {
                        if (FP8 && EPI == 1)    // canonical values are the survivors' codes [T, F / 4]
                            reinterpret_cast<uint16_t*>(ep.vals)[(int64_t)(t0 + (lane >> 3) + 8 * (it0 + it)) * (F / 8) + blk_g] =
                                (uint16_t)fp8_enc2(bf2f(v[it] & 0xFFFFu), bf2f(v[it] >> 16), ep.inv_out);
                        else vals_p[(int64_t)it * 8 * (F / 8)] = v[it];
                    }
                }
                if (FP8 && valid) {        // the largest survivor magnitude of this half tile
#pragma unroll
                    for (int it = 0; it < NSW; ++it)
                        vmax_tile = __builtin_fmaxf(vmax_tile, __builtin_fmaxf(__builtin_fabsf(bf2f(v[it] & 0xFFFFu)), __builtin_fabsf(bf2f(v[it] >> 16))));
                }
                if (valid && ep.vcb) {
                    if constexpr (!FP8)
                        store_between(stream, [&](auto store) {
#pragma unroll
                            for (int it = 0; it < NSW; ++it) store(vcb_p + (int64_t)((it0 + it) >> 2) * (F >> 6) * 256 + lane + ((it0 + it) & 3) * 64, v[it]);
                        });
                    else
#pragma unroll
                        for (int it = 0; it < NSW; ++it) {             // the survivors' codes: the row's 8 pairs gathered into the lane of block 0, one 16-byte store
                            const int sw = it0 + it;
                            const uint32_t q2w = fp8_enc2(bf2f(v[it] & 0xFFFFu), bf2f(v[it] >> 16), ep.inv_out);
                            const uint32_t w2 = q2w | (row_shl<1>(q2w) << 16);
                            const uint4 w8 = make_uint4(w2, row_shl<2>(w2), row_shl<4>(w2), row_shl<6>(w2));
                            if (bl == 0) *reinterpret_cast<uint4*>(vcb8_p + (int64_t)(sw >> 2) * (F >> 7) * 1024 + (sw & 3) * 256) = w8;
                        }
                }
                tile_sync();
                store_between(stream, [&](auto store) {
#pragma unroll
                    for (int n = 0; n < (SHARE ? 1 : 4); ++n) {          // 2 groups of 16 compact rows x 2 chunks of 32 tokens, 1 KB each
                        const int q = SHARE ? kg : n;
                        const int fr = (q >> 1) * 16 + (lane >> 2), tc = (q & 1) * 32 + (lane & 3) * 8;
                        const uint4 w = *reinterpret_cast<const uint4*>(ttile + fr * EP + tc * 2);
                        if (FP8 && ep.at_fp8) {     // fp8 weight gradients: the compact transposed survivors leave as codes (a 64-token block = one 64-byte chunk)
                            if (valid)
                                *reinterpret_cast<uint2*>(ep.at + blk_off(f0 / 2 + fr, (t0 + tc) / 2, tok_ld / 64)) =
                                    make_uint2(fp8_enc2(bf2f(w.x & 0xFFFFu), bf2f(w.x >> 16), ep.inv_out) | (fp8_enc2(bf2f(w.y & 0xFFFFu), bf2f(w.y >> 16), ep.inv_out) << 16),
                                               fp8_enc2(bf2f(w.z & 0xFFFFu), bf2f(w.z >> 16), ep.inv_out) | (fp8_enc2(bf2f(w.w & 0xFFFFu), bf2f(w.w >> 16), ep.inv_out) << 16));
                        } else if (valid) {
                            store(ep.at + blk_off(f0 / 2 + (q >> 1) * 16, t0 + (q & 1) * 32, tok_ld / 32) + lane * 8, w);
                        }
                    }
                });
            }
            wave_lds_sync();
        }
        if (FP8 && EPI != 0 && ep.amax) note_amax_slots_seen(ep.amax, vmax_tile, amax_seen);
    } else {
        constexpr int EP = WN * 2 + 16;
        constexpr int CH = WN / 8;
        unsigned char* scratch = smem + wt * (32 * EP);
        // destination rows of the lane's 16 stores, looked up before the first store (loads and stores share one in-order counter: a look-up
        // between two stores would wait for the earlier one)
        int32_t io_map[WM / 32][32 * CH / 64];
        if (grp.out_row_map) {
#pragma unroll
            for (int a = 0; a < WM / 32; ++a)
#pragma unroll
                for (int p = 0; p < 32 * CH / 64; ++p) {
                    const int i = i0 + wm * WM + a * 32 + (lane + 64 * p) / CH;
                    io_map[a][p] = i < Ra ? grp.out_row_map[i] : -1;
                }
        }
#pragma unroll
        for (int a = 0; a < WM / 32; ++a) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int b = 0; b < FN; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<uint16_t*>(scratch + (x * 16 + 4 * lq + r) * EP + (b * 16 + l16) * 2) = (uint16_t)f2bf(FP8 ? acc[2 * a + x][b][r] * alpha : acc[2 * a + x][b][r]);
            wave_lds_sync();
            auto rows = [&](auto store) {
#pragma unroll
                for (int p = 0; p < 32 * CH / 64; ++p) {
                    const int e = lane + 64 * p, row = e / CH, ch = e % CH;
                    const int i = i0 + wm * WM + a * 32 + row, j = j0 + wn * WN + ch * 8;
                    if (i < Ra && j < Rb) {
                        int64_t io = grp.map_logM ? ((int64_t)(i >> 2) << grp.map_logM) + 4 * expert_id + (i & 3) : i;
                        if (grp.out_row_map) io = io_map[a][p];
                        if (io >= 0) store(out + io * ldo + j, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
                    }
                }
            };
            if (SPARSE) store_between(ep.stream, rows);
            else rows([](uint16_t* p, const uint4& w) { store_out(p, w); });       // the router's weight gradients
            wave_lds_sync();
        }
    }
}

// Workgroups of a launch: one per BM x BN output tile; grouped: per expert, over its token segment.
inline unsigned grid_tiles(int64_t Ra, int64_t Rb, const GemmGroup& g, int BM, int BN) {
    const int64_t tiles_m = (Ra + BM - 1) / BM, tiles_n = (Rb + BN - 1) / BN;
    if (g.n == 0) return (unsigned)(tiles_m * tiles_n);
    if (g.role == 2) return (unsigned)(g.n * tiles_m * tiles_n);
    const int64_t other = g.role == 0 ? tiles_n : tiles_m, bt = g.role == 0 ? BM : BN;
    if (g.seg_dev) return (unsigned)(((g.cap_rows + bt - 1) / bt + g.n) * other);   // worst case over all run lengths
    int64_t tok_tiles = 0;
    for (int e = 0; e < g.n; ++e) tok_tiles += (g.seg[e + 1] - g.seg[e] + bt - 1) / bt;
    return (unsigned)(tok_tiles * other);
}

// one contraction as a unit that launch_units (launch_mix.hpp) puts into a launch, alone or with others
template <bool SPARSE, bool OUT_I_CONTIG, int EPI, bool BLOCKED, bool FP8, class TL, bool BROW = false, bool MG = false, int PRUNE = 0>
struct GemmV2Unit {
    using Args = GemmV2Args;
    static constexpr int THREADS = TL::THREADS, LDS = GemmV2Lds<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, TL, MG, PRUNE != 0>::BYTES;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        gemm_nt_v2_body<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, TL, BROW, MG, PRUNE>(smem, pid, n_pid, a.a_vals, a.a_meta, a.B, a.bias, a.Ra, a.Rb, a.K, a.out, a.ldo, a.tiles_m, a.tiles_n,
                                                                     a.ep, a.grp, a.alpha);
    }
    static unsigned count(const Args& a) { return grid_tiles(a.Ra, a.Rb, a.grp, TL::BM, TL::BN); }
    static int stages(const Args& a) { return a.K / (SPARSE ? 64 : 32) / TL::KW; }      // of a tile, a wavefront's (K in byte pairs on codes)
    static Args args(Args a) { a.tiles_m = (a.Ra + TL::BM - 1) / TL::BM; a.tiles_n = (a.Rb + TL::BN - 1) / TL::BN; return a; }
};

// the three tiles; blocks of M = 64 columns want 128 hidden units in one wavefront (two blocks share a metadata byte): 256 x 128 in the place of 128 x 128
template <bool SPARSE> using Tile256 = Tile<2, 4, 128, SPARSE ? 3 : 4, 1>;
using TileTall = Tile<2, 2, 128, 2, 1>;       // 256 x 128, four wavefronts, two workgroups a CU (structured-sparse, with an epilogue)
template <bool SPARSE, int EPI> struct TileSel { using T128 = Tile<2, 2, 64, SPARSE ? 3 : 4, 1>; using T64 = Tile<1, 1, 64, 3, 4>; };
template <> struct TileSel<true, 22> { using T128 = TileTall; using T64 = Tile<1, 1, 128, 2, 4>; };
template <> struct TileSel<true, 38> { using T128 = TileTall; using T64 = Tile<1, 1, 128, 2, 4>; };

// tile: 256 / 128 / 64, or 0 to choose here
template <bool SPARSE, bool OUT_I_CONTIG, int EPI, bool BLOCKED, bool FP8>
hipError_t launch_gemm_v2(const GemmV2Args& args, hipStream_t s, int tile = 0) {
    using Sel = TileSel<SPARSE, EPI>;
    GemmV2Args a = args;
    if (EPI == 0 && OUT_I_CONTIG) a.ep.stream = stores_past(2 * (int64_t)a.Ra * a.Rb);
    // (grouped along the contraction, role 2: a tile contracts its own expert's tokens only)
    if (!tile) {
        const int steps = a.K / (SPARSE ? 64 : 32) / (a.grp.n && a.grp.role == 2 ? a.grp.n : 1);
        constexpr int what = EPI == 0 ? kGemmPlain : EPI == 3 || EPI == 4 ? kGemmRouter : EPI == 2 || EPI >= 32 ? kGemmBackward : kGemmForward;
        constexpr int M = Sel::T128::BM == 256 ? 64 : EPI >= 20 ? 16 : 8;
        tile = what == kGemmForward || what == kGemmBackward ? pick_epilogue_tile(a.Ra, a.Rb, steps, a.grp, what, M, FP8)
                                                             : pick_gemm_tile(a.Ra, a.Rb, steps, a.grp, small_round(what, steps), SPARSE, last_round(what, steps));
    }
    // Row-major 2:4 operands, whole groups of 256 k: metadata for four stages at a time (MG).  What bounds the loop is the number of lines a stage touches, 256 of
    // 768 for its metadata: T = 8192, N = 8192, K = 2048 192 -> 164 us; on 128 tiles T = 576, N = 9024, K = 2560 40.7 -> 33; even where few tiles are short.
    if constexpr (SPARSE && !BLOCKED && !FP8)
        if (a.K % 256 == 0) {
            if (tile == 256) return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, Tile256<SPARSE>, false, true>>(s, a);
            if (tile == 128)
                return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, typename Sel::T128, false, true>>(s, a);
        }
    if (tile == 256) return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, Tile256<SPARSE>>>(s, a);
    if (tile == 128) return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, typename Sel::T128>>(s, a);
    // (the dense form has no 64 tile)
    if constexpr (SPARSE) return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, typename Sel::T64>>(s, a);
    else return launch_units<GemmV2Unit<SPARSE, OUT_I_CONTIG, EPI, BLOCKED, FP8, typename Sel::T128>>(s, a);
}

}  // namespace sffn
