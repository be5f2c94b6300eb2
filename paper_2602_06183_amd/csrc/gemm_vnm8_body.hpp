// Eqs. (3), (7) of the paper for V:2:8 activations (V = 64, M = 8: the fused step's own format) without re-expressing the activation as a
// plain 2:4 matrix over all F columns:
//     out[t, n] = sum_k' Ac[t, k'] * Wk[row(t / 64, k'), n],      row(tb, k') = (k' / 4) * 8 + colidx[tb, k' / 4, k' % 4]
// Ac = the packed activation read as a 2:4 matrix of logical width K' = F / 2 (two survivors per four kept columns), Wk = [F, ldw]
// with the contraction index as row (W2.T for eq. (3), W1 as it is for eq. (7)).  The plain-2:4 route of gemm_v2.hip issues one
// structured-sparse matrix instruction per 32 columns of F; this kernel issues one per 64, and fetches half the activation bytes.
//
// Tile: 512 tokens x 128 output columns, a wavefront for each of its 8 token blocks, or 256 x 256 with 4 (token blocks) x 2 (column halves) wavefronts.
// What bounds both is the delivery of their operands to the CU (profiles/tile_kernels_70b_loop_parts.txt), and the first takes 34.25 KB per stage, the second
// 41.25: the slab of Wk weighs four times the rest, and every token block uses half of it.  T = D = 8192, F = 28672: 1222 us, 1307 on 256 x 256; T = 8192,
// D = 2048, F = 8192: 91, 100; on codes 687, 709 (gemm_vnm8.hip chooses).  A 64-row tile (the
// gathered-row kernel of gemm_gather.hip, which fetches only the kept rows) halves the reuse of Wk and is bound by L2 -> LDS delivery at
// M = 8; here the whole [64 f x columns] slab of Wk of a stage goes to LDS once for the tile's token blocks, and each token block picks
// its kept rows when it READS its B fragments: ds_read_b64_tr_b16 takes one address per lane (inside a group of 16 lanes, lane s supplies 4
// consecutive elements of row s / 4, lane l receives element l of those 4 rows), so the 4 rows of a read are the 4 kept hidden units of
// one column block.  The 64-byte pieces of a slab row are XOR-swizzled by f % 8 (128 columns: f % 4): the four rows of a read lie in one group of 8 rows.
//
// Operands as the fused epilogues of eqs. (1), (4) write them (common.hpp: vcb_off, mcb_off, cixt_off):
//   values    [T / 32][F / 64][32 tokens][16 values]   1 KB per (32 tokens, 64 hidden units): one wave-wide LDS-DMA load
//   metadata  [T / 64][F / 64][64 tokens][4 bytes]     the canonical nibbles of the 8 column blocks of a stage
//   offsets   [F / 64][T / 64][8 words]                word (h, r), byte j = kept column r of column block 4 (j / 2) + j % 2 + 2 h of the
//                                                      stage: the four rows that lane (h = lane / 32, r = (lane % 16) / 4) addresses in read j
// A stage = 64 hidden units = 32 k' = one matrix instruction step per fragment pair; 3 stages.
//
// The 64 x 64 tile (few tokens) has one token block, so its stages hold the kept rows only: the loads themselves pick them, half the bytes of the slab from memory and into LDS, and
// two workgroups a CU (77 KB of LDS; with the slab 126 KB), in launches that are shared with other contractions too.  Their addresses need the offsets first: those of the first
// three stages come in front of everything else, the others with the batch three stages ahead.  With the slab / kept rows: T = 64, D = 4096, F = 14336 a forward call on packed weights 40.4 / 32.1 us,
// D = 2048, F = 8192 22.9 / 21.0; steps: T = 512, D = 2624, F = 8000 197 / 160, T = 64, D = 1024, F = 4096 44.3 / 40.4, on codes T = 448, D = 2176, F = 7936 145 / 110.
//
// FP8 (the fp8 step): the same kernel on E4M3 codes with v_smfmac_f32_32x32x64_fp8_fp8, out = bf16(alpha * sum).  A stage is 128 hidden
// units = 64 k' (the instruction's K): the slab is 128 rows x 256 bytes, the survivors' codes fill the same 32 bytes per token and stage,
// the metadata 8 bytes.  The B fragments are read with ds_read_b64_tr_b8 (inside a group of 16 lanes, lane s supplies 8 consecutive bytes of
// row s / 2, lane l receives byte l of those 8 rows), so a read covers the kept rows of TWO column blocks; the offsets unit of a (128 hidden
// units, token block) is 16 words: word (h, p), byte j = kept column p % 4 of column block 8 (j / 2) + 4 h + 2 (j % 2) + p / 4.  The 32-byte
// pieces of a slab row are swizzled by f % 8.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"
#include "split.hpp"

namespace sffn {

// Workgroup tile: WT token blocks (64 tokens) x WH column groups, one wavefront each (64 tokens x 32 FN columns).  KW > 1 (with one wavefront
// per tile): KW wavefronts share the tile, wavefront g contracting stages g, g + KW, ... in a ring of its own; their partial sums meet in LDS.
template <int WT_, int WH_, int FN_, int NST_, int KW_>
struct VTile {
    static constexpr int WT = WT_, WH = WH_, FN = FN_, NST = NST_, KW = KW_;
    static constexpr int NW = WT * WH, BT = 64 * WT, BN = 32 * FN * WH, THREADS = 64 * NW * KW;
    static_assert(KW == 1 || (KW == 4 && NW == 1 && FN == 2), "a shared output tile is 64 x 64 and belongs to four single wavefronts");
    // Tile rows per band of the workgroup -> tile map (see SFFN_TILE_GROUP in common.hpp).  A tile of 256 x 256 fetches four times as many bytes of Wk as of the
    // packed activation, so the 32 tiles that an XCD runs at a time should share few column slabs of Wk: tall bands (T = D = 8192, F = 28672: 1.49 / 1.42 /
    // 1.38 / 1.36 ms per launch with 2 / 4 / 8 / 16 tile rows).  A tile of 512 x 128 fetches about as many of either (8 rows 1222 us, 16 rows 1233; on codes 687, 706).
    static constexpr int BAND = BT == 512 ? 8 : 16;
};
template <bool FP8, class TL>
struct G {
    static constexpr int ES = FP8 ? 1 : 2;               // bytes per element of Wk
    static constexpr int SLAB = FP8 ? 128 : 64;         // hidden units per stage
    static constexpr int ROW = TL::BN * ES;              // bytes of a slab row
    static constexpr bool KEPT = TL::KW > 1;             // the stage holds the kept rows of its one token block only
    static constexpr int kB = (KEPT ? SLAB / 2 : SLAB) * ROW;
    static constexpr int kA = TL::BT * 32;
    static constexpr int kMt = FP8 ? TL::BT * 8 : TL::BT * 4;
    static constexpr int kC = KEPT ? 64 : TL::WT * (FP8 ? 64 : 32) > 256 ? TL::WT * (FP8 ? 64 : 32) : 256;
    static constexpr int C_PARTS = KEPT ? 1 : kC / 256;             // wave-wide loads of the offsets; every wavefront issues one of them
    static constexpr int kStage = kB + kA + kMt + kC;
    static constexpr int B_LD = kB / 1024 / TL::NW, A_LD = kA / 1024 / TL::NW, M_LD = (kMt / 256 + TL::NW - 1) / TL::NW;    // loads per wave and stage
    static constexpr int LOADS = B_LD + A_LD + M_LD + 1;
    static constexpr int PIECE = FP8 ? 32 : 64;          // bytes of a swizzled piece = 32 columns
    static constexpr int NP = ROW / PIECE;               // pieces of a row
    static constexpr int PMASK = (NP < 8 ? NP : 8) - 1;
    static constexpr int BYTES = TL::KW * TL::NST * kStage;
};

// Wk / ldw: bf16 elements, or (FP8) code bytes
template <bool FP8, class TL>
__device__ __forceinline__ void vnm8_gemm_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ vcb, const uint8_t* __restrict__ mcb,
                                               const uint8_t* __restrict__ cixt, const uint8_t* __restrict__ Wk, int ldw,
                                               int Ra, int N, int F, int Ttot, uint16_t* __restrict__ out, int64_t ldo,
                                               int tiles_m, int tiles_n, const GemmGroup& grp, float alpha, const Split& split, bool past) {
    using GG = G<FP8, TL>;
    constexpr int kB = GG::kB, kA = GG::kA, kMt = GG::kMt, kC = GG::kC, kStage = GG::kStage, ES = GG::ES, kStages = TL::NST, kLoads = GG::LOADS, KW = TL::KW, FN = TL::FN;
    constexpr int BT = TL::BT, BN = TL::BN, ROW = GG::ROW, B_LD = GG::B_LD, A_LD = GG::A_LD, M_LD = GG::M_LD, PB = GG::PIECE, PM = GG::PMASK;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int kg = KW > 1 ? wave : 0, wt = KW > 1 ? 0 : wave;       // share of the contraction / place in the tile
    unsigned char* const ring = smem + kg * (kStages * kStage);
    const uint32_t ring_lds = lds_addr(smem) + kg * (kStages * kStage);

    int L = xcd_run(pid, n_pid);
    // Grouped form (role 0): the token tiles of segment e meet expert e's matrix
    int i_base = 0;
    if (grp.n) {
        int e = 0, cnt = 0;
        for (; e < grp.n; ++e) {
            cnt = (grp.seg[e + 1] - grp.seg[e] + BT - 1) / BT * tiles_n;
            if (L < cnt) break;
            L -= cnt;
        }
        if (e == grp.n) return;
        tiles_m = uniform(cnt / tiles_n); i_base = grp.seg[e]; Ra = grp.seg[e + 1];
        Wk += (int64_t)e * grp.b_stride * ES;
    }
    constexpr bool SPLIT = KW == 4;
    const int KS = F / GG::SLAB;                     // stages = slabs of 64 (128) hidden units
    int ks0 = 0, ks1 = KS, sp = 0, tile = 0;         // this workgroup's stages
    if (SPLIT && split.n > 1) {
        const int per = tiles_m * tiles_n;
        sp = uniform(L / per);
        L -= sp * per;
        tile = L;
        ks0 = sp * KS / split.n; ks1 = (sp + 1) * KS / split.n;
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, TL::BAND, tm, tn);
    const int i0 = i_base + tm * BT, n0 = tn * BN;
    const int NTB = Ttot >> 6;

    // ---- DMA sources (wave-uniform 64-bit base + 32-bit per-lane offset).  Token groups past the end of the operand are clamped into it:
    //      they only feed outputs that are never stored. ----------------------------------------------------------------------------------
    // B: a load brings 1024 / ROW slab rows; a lane's 16-byte slot fetches the chunk whose piece (PB bytes = 32 columns) the swizzle puts there:
    // piece p of row f sits at p ^ (f % min(8, pieces)).  Chunks past the right edge of Wk are redirected into the first 64 columns.
    const uint64_t w_base = uniform64(Wk);
    constexpr int LPR = ROW / 16, RPL = 1024 / ROW;         // 16-byte slots per slab row, rows per load
    // KEPT: a load brings the kept rows that the words of the offsets name with one of their bytes, word by word, 128 (FP8: 64) bytes of each: row j RPL + q of the stage is byte j of
    // word q.  That is the order in which the transposing reads want them, so their addresses do not depend on data.  The pieces of a row are exchanged where that puts the rows
    // of a read (4; FP8: 8) on different banks.
    constexpr bool KEPT = GG::KEPT;
    const int kq = lane / LPR, kf = FP8 ? kq >> 2 & 1 : kq >> 1 & 1;
    const uint32_t kept_lane = (uint32_t)(8 * (FP8 ? 4 * (kq >> 3) + (kq >> 2 & 1) : 2 * (kq >> 2))) * (uint32_t)ldw * ES + (uint32_t)n0 * ES + (uint32_t)((lane % LPR) ^ (kf * (PB / 16))) * 16;
    uint32_t b_lane[KEPT ? 1 : B_LD];
    if constexpr (!KEPT)
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        // (the stage goes into the scalar base: a vector instruction less for every load)
        const int row = RPL * (B_LD * wt + i) + lane / LPR, slot = lane % LPR;
        constexpr int SPP = PB / 16;                         // slots per piece
        int c = (((slot / SPP) ^ (row & PM)) * SPP) | (slot & (SPP - 1));
        if (n0 + c * (16 / ES) >= N) c &= (64 * ES / 16) - 1;
        b_lane[i] = ((uint32_t)row * (uint32_t)ldw + (uint32_t)(n0 + c * (16 / ES))) * ES;
    }
    const uint32_t b_kstep = (uint32_t)GG::SLAB * (uint32_t)ldw * ES;
    uint64_t a_base[A_LD], m_base[M_LD], c_base;
    uint32_t a_lane, m_lane, c_lane;
    {
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {                 // 32 tokens of the tile each
            int g32 = (i0 >> 5) + wt * A_LD + i;
            g32 = g32 < (Ttot >> 5) ? g32 : (Ttot >> 5) - 1;
            a_base[i] = uniform64(vcb + (int64_t)g32 * KS * 512);
        }
        const int row = lane >> 1, slot = lane & 1;
        a_lane = (uint32_t)(row * 32 + ((slot ^ ((row >> 3) & 1)) << 4));
#pragma unroll
        for (int i = 0; i < M_LD; ++i) {
            // 256-byte pieces: 64 tokens (bf16) / half of the 512-byte unit of a token block (FP8).  With fewer pieces than wavefronts two fetch the same
            const int mi = (wt * M_LD + i) % (kMt / 256);
            int g64 = (i0 >> 6) + (FP8 ? mi >> 1 : mi);
            g64 = g64 < NTB ? g64 : NTB - 1;
            m_base[i] = uniform64(FP8 ? mcb + (int64_t)g64 * KS * 512 + (mi & 1) * 256 : mcb + (int64_t)g64 * KS * 256);
        }
        m_lane = lane * 4;
        // offsets of the tile's token blocks, 32 (FP8: 64) bytes each: a load brings 256 bytes (slots past the tile's last block repeat it)
        const int words = FP8 ? 16 : 8;
        int tb = KEPT ? 0 : (wt % GG::C_PARTS * 64 + lane) / words;
        tb = (i0 >> 6) + (tb < TL::WT ? tb : TL::WT - 1);
        tb = tb < NTB ? tb : NTB - 1;
        c_base = uniform64(cixt);
        c_lane = (uint32_t)(tb * words * 4 + (lane & (words - 1)) * 4);
    }
    const uint32_t c_kstep = (uint32_t)NTB * (FP8 ? 64u : 32u);
    constexpr uint32_t m_kstep = FP8 ? 512u : 256u;
    // loads lo .. hi - 1 of a stage's kLoads (compile-time bounds).  KEPT: w = the lane's word of the stage's offsets, ahead = the stage whose offsets come with this one's
    auto issue = [&](int kt, int stage, int lo, int hi, uint32_t w = 0, int ahead = 0) {
        const uint32_t sb = ring_lds + stage * kStage, sa = sb + kB, sm = sa + kA, sc = sm + kMt;
#pragma unroll
        for (int i = 0; i < B_LD; ++i)
            if (i >= lo && i < hi) {
                if constexpr (KEPT)
                    dma16(w_base + (uint64_t)((uint32_t)kt * b_kstep + (uint32_t)((FP8 ? 8 * (i >> 1) + 2 * (i & 1) : 4 * (i >> 1) + (i & 1)) * 8) * (uint32_t)ldw * ES),
                          __umul24((w >> (8 * i)) & 0xFFu, (uint32_t)ldw * ES) + kept_lane, sb + i * 1024);
                else dma16(w_base + (uint64_t)((uint32_t)kt * b_kstep), b_lane[i], sb + (B_LD * wt + i) * 1024);
            }
#pragma unroll
        for (int i = 0; i < A_LD; ++i)
            if (B_LD + i >= lo && B_LD + i < hi) dma16(a_base[i], a_lane + (uint32_t)kt * 1024u, sa + (wt * A_LD + i) * 1024);
#pragma unroll
        for (int i = 0; i < M_LD; ++i)
            if (B_LD + A_LD + i >= lo && B_LD + A_LD + i < hi) dma4(m_base[i], m_lane + (uint32_t)kt * m_kstep, sm + ((wt * M_LD + i) % (kMt / 256)) * 256);
        if (kLoads - 1 >= lo && kLoads - 1 < hi) {
            if constexpr (KEPT) { if (lane < kC / 4) dma4(c_base, c_lane + (uint32_t)ahead * c_kstep, sc); }      // (bf16: 8 words, twice)
            else dma4(c_base, c_lane + (uint32_t)kt * c_kstep, sc + wt % GG::C_PARTS * 256);
        }
    };

    // ---- per-lane LDS offsets of the fragment reads (inside a stage).  A wave owns one token block (64 tokens) x 32 FN output columns: the
    //      B fragments it gathers belong to one column selection. ----------------------
    const int tbw = wt / TL::WH, nh = wt % TL::WH;
    // (fragments are 32 tokens apart: 1024 bytes of survivors, 128 (FP8: 256) of metadata)
    const int arow = tbw * 64 + l32;
    const int a_off = kB + arow * 32 + ((lh ^ ((arow >> 3) & 1)) << 4);
    const int m_off = kB + kA + (FP8 ? arow * 8 + 4 * lh : arow * 4 + 2 * lh);
    // bf16: transpose read j of fragment fn: slab row = 8 cb(j) + c with cb(j) = 4 (j / 2) + j % 2 + 2 h and c = byte j of the lane's offsets
    // word; byte address = row * ROW + ((FN nh + fn) ^ (c % pieces)) * 64 + 32 (column half) + 8 (lane % 4)
    // FP8: the lane addresses row p = (lane % 16) / 2 of the read's 8: cb(j) = 8 (j / 2) + 4 h + 2 (j % 2) + p / 4, c = byte j of word (h, p);
    // byte address = row * ROW + ((FN nh + fn) ^ (c % pieces)) * 32 + 16 (column half) + 8 (lane % 2)
    // The part that depends on c is (c * pieces | (c % pieces) ^ FN nh) * PB: a byte of a table of eight, looked up for the four of a word at once (v_perm_b32); the fragments of a
    // row of four differ in two bits of the address.  (Worked out read by read, 30 more vector instructions in a stage of 16 matrix instructions: T = D = 8192, F = 28672 1280 us, now 1200;
    // T = 6400, N = 4096, F = 14336 315, 293; 128 tile, T = 1984, N = 1408, F = 4224 26.8, 25.0, on codes 17.9, 15.8.)
    const int r4 = (lane & 15) >> 2, p8 = (lane & 15) >> 1, g = lane >> 4;
    const int c_off = kB + kA + kMt + (FP8 ? 64 * tbw + (lh * 8 + p8) * 4 : 32 * tbw + (lh * 4 + r4) * 4);
    const uint32_t b_lane0 = FP8 ? (uint32_t)((4 * lh + (p8 >> 2)) * 8 * ROW + ((g & 1) << 4) + ((lane & 1) << 3)) : (uint32_t)(2 * lh * 8 * ROW + ((g & 1) << 5) + ((lane & 3) << 3));
    // KEPT: row q = 4 h + r4 (FP8: 8 h + p8) of each of the four loads, both halves of the columns
    const int rq = FP8 ? lh * 8 + p8 : lh * 4 + r4, rf = FP8 ? rq >> 2 & 1 : rq >> 1 & 1;
    const uint32_t kept_row = (uint32_t)(rq * ROW + (FP8 ? ((g & 1) << 4) + ((lane & 1) << 3) : ((g & 1) << 5) + ((lane & 3) << 3)));
    const uint32_t kept_off[2] = {kept_row + rf * PB, kept_row + (rf ^ 1) * PB};
    const int w_off = kB + kA + kMt + kq * 4;
    constexpr int NP = GG::NP;
    static_assert(NP <= 8, "a byte holds 8 pieces x 8 rows");
    constexpr auto entry = [](uint32_t c) { return c * NP | (c & (NP - 1)); };
    const uint32_t col = 0x01010101u * (uint32_t)(FN * nh);
    const uint32_t tab_lo = (entry(0) | entry(1) << 8 | entry(2) << 16 | entry(3) << 24) ^ col, tab_hi = (entry(4) | entry(5) << 8 | entry(6) << 16 | entry(7) << 24) ^ col;

    f32x16 acc[2][FN];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

    // The stage's fragments in two halves: P = both A fragments, the offsets word and the first HB = FN / 2 B fragments; Q = the others (the A
    // fragments of P stay live until Q's matrix instructions, so A is double-buffered by stage parity)
    constexpr int HB = FN / 2;
    struct BPair { union { s16x4 q[4]; v2i q8[4]; bf16x16 v; i32x8 v8; } b[HB]; };
    struct AFrags { Frag8 a[2]; int idx[2]; uint32_t cw; };
    auto read_a = [&](AFrags& f, const unsigned char* st) {
        if (!KEPT) f.cw = *reinterpret_cast<const uint32_t*>(st + c_off);
#pragma unroll
        for (int a2 = 0; a2 < 2; ++a2) {
            f.a[a2].u = *reinterpret_cast<const uint4*>(st + a_off + a2 * 1024);
            f.idx[a2] = FP8 ? (int)*reinterpret_cast<const uint32_t*>(st + m_off + a2 * 256) : (int)*reinterpret_cast<const uint16_t*>(st + m_off + a2 * 128);
        }
    };
    // the four addresses of a stage's reads, for its first fragment
    struct BAddr { uint32_t j[4]; };
    auto address_b = [&](BAddr& ad, int stage, uint32_t cw) {
        if constexpr (KEPT) { ad.j[0] = ring_lds + (uint32_t)(stage * kStage) + kept_off[0]; ad.j[1] = ring_lds + (uint32_t)(stage * kStage) + kept_off[1]; return; }
        const uint32_t e = __builtin_amdgcn_perm(tab_hi, tab_lo, cw), base = ring_lds + (uint32_t)(stage * kStage) + b_lane0;
#pragma unroll
        for (int j = 0; j < 4; ++j) ad.j[j] = base + ((e >> (8 * j)) & 0xFFu) * (uint32_t)PB;
    };
    auto read_b = [&](BPair& f, const BAddr& ad, int half) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            constexpr int kBlk = 8 * ROW;
            const int cb = FP8 ? 8 * (j >> 1) + 2 * (j & 1) : 4 * (j >> 1) + (j & 1);
#pragma unroll
            for (int q = 0; q < HB; ++q) {
                const uint32_t at = KEPT ? ad.j[half] + (uint32_t)(j * 1024) : (ad.j[j] ^ (uint32_t)((HB * half + q) * PB)) + (uint32_t)(cb * kBlk);
                if (FP8) f.b[q].q8[j] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)at);
                else     f.b[q].q[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
            }
        }
    };
    auto mma_half = [&](const AFrags& fa, const BPair& fb, int half, int a2) {
#pragma unroll
            for (int fn = 0; fn < HB; ++fn)
                if (FP8) acc[a2][HB * half + fn] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(fa.a[a2].q, fb.b[fn].v8, acc[a2][HB * half + fn], fa.idx[a2], 0, 0);
                else     acc[a2][HB * half + fn] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fa.a[a2].v, fb.b[fn].v, acc[a2][HB * half + fn], fa.idx[a2], 0, 0);
    };
#define SB() __builtin_amdgcn_sched_barrier(0)

    const int nk = (ks1 - ks0 - kg + KW - 1) / KW;
    auto step_of = [&](int kt) { return ks0 + kg + kt * KW; };
    // KEPT: the offsets of a tile come with the batch three before it, so they are read from its stage just before the stage is refilled; those of the first three in front
    auto ahead_of = [&](int kt) { return step_of(kt + kStages < nk ? kt + kStages : nk - 1); };
    uint32_t w = 0;
    if (nk > 0) {
    uint32_t first[kStages];
    if constexpr (KEPT) {
        // The offsets of the first three go through LDS too, to where their rows will land, while everything that needs no offsets is on its way: a load that the compiler sees
        // among loads that it does not count makes it wait for all of them, here for one stage after the other.  Four trips to memory / two: forward calls on packed weights T = 64,
        // D = 2048, F = 8192 21.5 / 21.2 us, T = 128, D = 1024, F = 4096 17.8 / 17.1; steps T = 64, D = 1024, F = 4096 38.4 / 37.4, T = 256, D = 512, F = 2048 28.2 / 27.4.
        static_assert(kLoads * 2 / 4 == B_LD, "the last stage's rows are loaded here, the rest in the first step");
#pragma unroll
        for (int p = 0; p < kStages; ++p)
            if (p < nk && lane < kC / 4) dma4(c_base, c_lane + (uint32_t)step_of(p) * c_kstep, ring_lds + p * kStage);
#pragma unroll
        for (int p = 0; p < kStages - 1; ++p)
            if (p < nk) issue(step_of(p), p, B_LD, kLoads, 0, ahead_of(p));
        if (nk >= kStages) wait_vmcnt<(kStages - 1) * (kLoads - B_LD)>();
        else wait_vmcnt<0>();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int p = 0; p < kStages; ++p) first[p] = *reinterpret_cast<const uint32_t*>(ring + p * kStage + kq * 4);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int p = 0; p < kStages; ++p)
            if (p < nk) issue(step_of(p), p, 0, B_LD, first[p]);
        if (nk >= kStages) wait_vmcnt<(kStages - 1) * B_LD>();
        else wait_vmcnt<0>();
    } else {
#pragma unroll
        for (int p = 0; p < kStages; ++p)
            if (p < nk) issue(step_of(p), p, 0, p < kStages - 1 ? kLoads : kLoads * 2 / 4);           // (the rest of the last one's loads are the first step's)
        if (nk >= kStages) wait_vmcnt<(kStages - 2) * kLoads + kLoads * 2 / 4>();
        else wait_vmcnt<0>();
    }
    if (KW == 1) __syncthreads();
    else asm volatile("" ::: "memory");
    AFrags A0, A1;
    BPair P, Q;
    BAddr ad;
    read_a(A0, ring);
    address_b(ad, 0, A0.cw);
    read_b(P, ad, 0);
    int stage = 0;
    if (KEPT) w = first[kStages - 1];
    // two stages per trip so that the A fragment buffers alternate without copies.  The loads of a refill are spread from the barrier that frees its stage
    // to the next one, and the last steps load nothing (gemm_v2_body.hpp says why).  t: the tile that is loaded, s: its stage; full: both of a step's exist.
#define ISSUE(t, s, i) if (full.value || (t) < nk) issue(step_of(t), s, kLoads * (i) / 4, kLoads * ((i) + 1) / 4, w, KEPT ? ahead_of(t) : 0)
    auto step = [&](auto full, int kt, AFrags& cur, AFrags& nxt_a) {
        const int next_stage = (stage + 1 == kStages) ? 0 : stage + 1, last_stage = stage == 0 ? kStages - 1 : stage - 1;
        const unsigned char* sn = ring + next_stage * kStage;
        uint32_t w_next = 0;
        if (KEPT) { w_next = *reinterpret_cast<const uint32_t*>(ring + stage * kStage + w_off); SB(); }
        mma_half(cur, P, 0, 0); SB();
        ISSUE(kt + kStages - 1, last_stage, 2); SB();
        mma_half(cur, P, 0, 1); SB();
        read_b(Q, ad, 1); SB();
        ISSUE(kt + kStages - 1, last_stage, 3); SB();
        w = w_next;
        // Q has arrived and this wave's part of tile kt + 1 has landed; after the barrier every wave is done reading this stage
        if (full.value || kt + kStages - 1 < nk) wait_vmcnt_lgkm0<(kStages - 2) * kLoads>();
        else wait_vmcnt_lgkm0<0>();
        if (KW == 1) __builtin_amdgcn_s_barrier();
        else asm volatile("" ::: "memory");
        SB();
        ISSUE(kt + kStages, stage, 0); SB();
        read_a(nxt_a, sn); SB();
        mma_half(cur, Q, 1, 0); SB();
        ISSUE(kt + kStages, stage, 1); SB();
        mma_half(cur, Q, 1, 1); SB();
        address_b(ad, next_stage, nxt_a.cw);
        read_b(P, ad, 0); SB();
        stage = next_stage;
    };
#undef ISSUE
    int kt = 0;
    for (; kt + 1 + kStages < nk; kt += 2) { step(Flag<true>(), kt, A0, A1); step(Flag<true>(), kt + 1, A1, A0); }
    for (; kt + 1 < nk; kt += 2) { step(Flag<false>(), kt, A0, A1); step(Flag<false>(), kt + 1, A1, A0); }
    if (kt < nk) step(Flag<false>(), kt, A0, A1);
#undef SB
    wait_vmcnt<0>();
    }
    __syncthreads();
    if constexpr (SPLIT) {      // (all four wavefronts store: the first alone 0.3 - 0.7 us more in a launch of 10)
        static_assert(kJoin4 + 4 * 32 * 80 <= GG::BYTES, "sums and their staging must fit in the main-loop LDS");
        float q[16];
        if (split.n == 1) {
            join4(acc, smem, wave, lane, q);
            store_quarter(q, FP8 ? alpha : 1.0f, smem + kJoin4, wave, lane, out, ldo, i0, n0, Ra, N);
        } else if (split_join4(acc, smem, split, tile, sp, wave, lane, q)) {
            store_quarter(q, FP8 ? alpha : 1.0f, smem + kJoin4, wave, lane, out, ldo, i0, n0, Ra, N);
        }
        return;
    }

    // ---- output: the wave's 32 x 64 sub-tiles go through LDS as [t][n] so that HBM sees 128-byte row segments -----------------------------
    constexpr int EP = 64 * 2 + 16;
    unsigned char* scratch = smem + wt * (32 * EP);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int half = 0; half < FN / 2; ++half) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
                    *reinterpret_cast<uint16_t*>(scratch + row * EP + (b * 32 + l32) * 2) = (uint16_t)f2bf(FP8 ? acc[a][2 * half + b][r] * alpha : acc[a][2 * half + b][r]);
                }
            wave_lds_sync();
            store_between(past, [&](auto store) {
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int e = lane + 64 * p, row = e >> 3, ch = e & 7;
                    const int i = i0 + tbw * 64 + a * 32 + row, j = n0 + nh * 32 * FN + half * 64 + ch * 8;
                    if (i < Ra && j < N) store(out + (int64_t)i * ldo + j, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
                }
            });
            wave_lds_sync();
        }
}

inline unsigned vnm8_tiles(int64_t T, int64_t N, const GemmGroup& g, int BT, int BN) {
    const int64_t tiles_n = (N + BN - 1) / BN;
    if (!g.n) return (unsigned)((T + BT - 1) / BT * tiles_n);
    int64_t n = 0;
    for (int e = 0; e < g.n; ++e) n += (g.seg[e + 1] - g.seg[e] + BT - 1) / BT * tiles_n;
    return (unsigned)n;
}
template <bool FP8, class TL>
struct Vnm8Unit {
    using Args = Vnm8Args;
    static constexpr int THREADS = TL::THREADS, LDS = G<FP8, TL>::BYTES;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        vnm8_gemm_body<FP8, TL>(smem, pid, n_pid, a.vcb, a.mcb, a.cixt, a.Wk, a.ldw, a.T, a.N, a.F, a.T, a.out, a.ldo, a.tiles_m, a.tiles_n, a.grp, a.alpha, a.split, a.past != 0);
    }
    static unsigned count(const Args& a) { return vnm8_tiles(a.T, a.N, a.grp, TL::BT, TL::BN) * (unsigned)a.split.n; }
    static int stages(const Args& a) { return a.F / (FP8 ? 128 : 64) / (TL::KW * a.split.n); }      // of a tile, a wavefront's (wgrad_first)
    static Args args(Args a) { a.tiles_m = (a.T + TL::BT - 1) / TL::BT; a.tiles_n = (a.N + TL::BN - 1) / TL::BN; return a; }
};
template <bool FP8> using Vnm8Unit512 = Vnm8Unit<FP8, VTile<8, 1, 4, 3, 1>>;
template <bool FP8> using Vnm8Unit256 = Vnm8Unit<FP8, VTile<4, 2, 4, 3, 1>>;
template <bool FP8> using Vnm8UnitTall = Vnm8Unit<FP8, VTile<4, 1, 4, 3, 1>>;          // 256 tokens x 128 columns
template <bool FP8> using Vnm8Unit128 = Vnm8Unit<FP8, VTile<2, 2, 2, 3, 1>>;
template <bool FP8> using Vnm8Unit64 = Vnm8Unit<FP8, VTile<1, 1, 2, 3, 4>>;

}  // namespace sffn
