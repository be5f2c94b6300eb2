// V:N:M activation x dense matrix with the dense operand's rows gathered per token block (eqs. (3), (7) of the paper
// for blocks of M >= 16 columns, the regime of Table 5; also the stand-alone vnm_spmm at M = 8 when Wk is given as is):
//     out[t, n] = sum_k' Ac[t, k'] * Wk[row(t / 64, k'), n],      row(tb, k') = (k' / 4) * M + colidx[tb, k' / 4, k' % 4]
// Ac = the packed activation read as a plain 2:4 matrix of logical width K' = 4 F / M (vals [T, K' / 2], meta
// [T, K' / 8], both row-major: exactly the canonical V:N:M arrays), Wk = [F, ldw] with the contraction index as row.
// Only the K' selected rows of Wk take part, so the matrix work and the operand traffic shrink with 4 / M; the
// plain-2:4 route of gemm_v2.hip contracts over all F instead.
//
// A workgroup owns one V = 64 token block (the unit that shares a column selection) x 256 output columns; 4 wavefronts,
// 64 x 64 each (or, for outputs of few such tiles, x 64 columns with the contraction shared by the 4 wavefronts: GTile below).  Per 64-k' stage it streams 64 gathered 512-byte row segments of Wk (LDS-DMA, two rows per wave-wide
// load; the per-lane source offset carries the row), the 64 x 32 packed values and their metadata.  The rows arrive
// k-major while v_smfmac_f32_32x32x32_bf16 wants 16 consecutive k per lane, so the B fragments are read with the
// LDS transpose read ds_read_b64_tr_b16: inside each group of 16 lanes, lane s supplies the address of 4 consecutive
// elements of row s / 4 (element chunk s % 4) and lane l receives element l of rows 0..3 (measured with an index
// pattern).  64-byte pieces of a row are XOR-swizzled by k' % 4 so that the four rows of one read hit disjoint banks.
// With 64-row tiles the kernel is bound by L2 -> LDS delivery, not by the matrix cores, and for large M a tile has
// only a few stages, so start-up and drain matter: the ring has 2 stages and the footprint is exactly 80 KB, which
// lets two workgroups share a CU and cover each other's prologue and epilogue (measured faster than one workgroup
// with a 4-stage ring at every M).  Workgroups of one XCD share a column slab of Wk and walk k' together.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"
#include "split.hpp"

namespace sffn {

// NW wavefronts along n, 64 columns each.  KW > 1 (NW = 1): KW wavefronts share the 64 x 64 tile, wavefront g contracting stages g, g + KW, ... in a
// ring of its own; their partial sums meet in LDS.
template <int NW_, int NST_, int KW_>
struct GTile {
    static constexpr int NW = NW_, NST = NST_, KW = KW_, BN = 64 * NW, THREADS = 64 * NW * KW;
    static_assert(KW == 1 || NW == 1, "a shared output tile belongs to single wavefronts");
    static constexpr int ROW = BN * 2, kB = 64 * ROW, kA = 64 * 64, kM = 64 * 8, kStage = kB + kA + kM;      // bytes per gathered row; per stage
    static constexpr int B_LD = kB / 1024 / NW, A_LD = 4 / NW, M_LD = NW == 1 ? 2 : 1, kLoads = B_LD + A_LD + M_LD;     // per wave per stage
    static constexpr int RING = KW * NST * kStage;
};
constexpr int kGStages = 2;                            // fp8 form
constexpr int kGLoads = 8 + 1 + 1;
constexpr int kGMaxKc = 7168;                          // column offsets of one token block kept in LDS (2 stages of the 256-column tile + this = 80 KB)

template <class TL>
__device__ __forceinline__ void vnm_gather_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ a_vals, const uint8_t* __restrict__ a_meta,
                                                             const uint8_t* __restrict__ colidx, const uint16_t* __restrict__ Wk,
                                                             int ldw, int N, int Kc, int logM, int nblk_tok, int tiles_n,
                                                             uint16_t* __restrict__ out, int64_t ldo, const GemmGroup& grp, const Split& split, bool past) {
    constexpr int KW = TL::KW, ROW = TL::ROW, kGB = TL::kB, kGA = TL::kA, kGStage = TL::kStage, kGStages = TL::NST, kGLoads = TL::kLoads;
    unsigned char* const cix = smem + TL::RING;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int kg = KW > 1 ? wave : 0, wt = KW > 1 ? 0 : wave;
    unsigned char* const ring = smem + kg * (kGStages * kGStage);
    const uint32_t ring_lds = lds_addr(smem) + kg * (kGStages * kGStage);

    // Consecutive workgroup ids go to different XCDs; give each XCD a run of consecutive logical ids, and let logical
    // ids walk the token blocks of one column slab, so an XCD's L2 holds one slab of Wk at a time.
    int L = xcd_run(pid, n_pid);
    int ks0 = 0, ks1 = Kc >> 6, sp = 0;                  // this workgroup's stages (split.hpp)
    if (KW > 1 && split.n > 1) {
        const int per = nblk_tok * tiles_n;
        sp = uniform(L / per);
        L -= sp * per;
        ks0 = sp * (Kc >> 6) / split.n; ks1 = (sp + 1) * (Kc >> 6) / split.n;
    }
    const int tn = uniform(L / nblk_tok), tb = L - tn * nblk_tok;
    const int t0 = tb * 64, n0 = tn * TL::BN;
    if (grp.n) {                                         // grouped form: the token block's segment names the expert whose matrix it meets
        int e = 0;
        while (e + 1 < grp.n && t0 >= grp.seg[e + 1]) ++e;
        Wk += e * grp.b_stride;
    }

    // ---- column offsets of this token block -> LDS ------------------------------------------------------------
    {
        const uint4* src = reinterpret_cast<const uint4*>(colidx + (int64_t)tb * Kc);
        for (int i = tid; i < (Kc >> 4); i += 256) reinterpret_cast<uint4*>(cix)[i] = src[i];
    }
    __syncthreads();

    // ---- DMA sources ---------------------------------------------------------------------------------------------
    // B: load i of wave w (i = 0..7) brings rows k' = RPL (8 w + i) + lane / LPR of the stage (RPL rows of LPR 16-byte slots a load); a slot
    // fetches the chunk that the swizzle puts there (64-byte piece ^ (k' % min(4, pieces))).  Chunks past the
    // right edge of Wk are redirected to the first 64 columns of the tile: they only feed outputs that are not stored.
    constexpr int LPR = ROW / 16, RPL = 1024 / ROW, PM = (ROW / 64 < 4 ? ROW / 64 : 4) - 1;
    const uint64_t w_base = uniform64(Wk);
    uint32_t b_col[2];                                   // byte offset of the lane's chunk inside a row, for even / odd load index
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        int c = (lane % LPR) ^ (((par * RPL + lane / LPR) & PM) << 2);
        if (n0 + c * 8 >= N) c &= 7;
        b_col[par] = (uint32_t)(n0 + c * 8) * 2;
    }
    const uint32_t row_bytes = (uint32_t)ldw * 2;
    // A (16 rows x 64 bytes per load, as in gemm_v2_body.hpp) and metadata ([row][8 bytes], 32 rows per load; with four wavefronts, 2 and 3 repeat
    // the loads of 0 and 1 so that every wave has the same number of loads in flight)
    const int lda = Kc >> 1;
    uint64_t a_base[TL::A_LD], m_base[TL::M_LD];
#pragma unroll
    for (int i = 0; i < TL::A_LD; ++i) a_base[i] = uniform64(a_vals + (int64_t)(t0 + 16 * (wt * TL::A_LD + i)) * lda);
#pragma unroll
    for (int i = 0; i < TL::M_LD; ++i) m_base[i] = uniform64(a_meta + (int64_t)(t0 + 32 * ((wt + i) & 1)) * (Kc >> 3));
    uint32_t a_lane, m_lane;
    {
        const int rb = lane >> 2, c = (lane & 3) ^ ((rb >> 2) & 3);
        a_lane = (uint32_t)(rb * lda + c * 8) * 2;
        m_lane = (uint32_t)((lane >> 1) * (Kc >> 3) + (lane & 1) * 4);
    }
    // byte offsets of the gathered rows for the next refill, looked up ahead of the loads that use them
    uint32_t b_row[8];
    auto lookup = [&](int kt) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = kt * 64 + RPL * (8 * wt + i) + lane / LPR;
            b_row[i] = (uint32_t)(((k >> 2) << logM) + cix[k]) * row_bytes;
        }
    };
    auto issue = [&](int kt, int stage) {
        const uint32_t sb = ring_lds + stage * kGStage, sa = sb + kGB, sm = sa + kGA;
#pragma unroll
        for (int i = 0; i < 8; ++i) dma16(w_base, b_row[i] + b_col[i & 1], sb + (8 * wt + i) * 1024);
#pragma unroll
        for (int i = 0; i < TL::A_LD; ++i) dma16(a_base[i], a_lane + (uint32_t)kt * 64, sa + (wt * TL::A_LD + i) * 1024);
#pragma unroll
        for (int i = 0; i < TL::M_LD; ++i) dma4(m_base[i], m_lane + (uint32_t)kt * 8, sm + ((wt + i) & 1) * 256);
    };

    // ---- fragment read offsets inside a stage ----------------------------------------------------------------------
    int a_off[2], m_off[2], b_off[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int row = a * 32 + l32;
        a_off[a] = kGB + row * 64 + ((lh ^ ((row >> 2) & 3)) << 4);
        m_off[a] = kGB + kGA + row * 8 + 2 * lh;
    }
    {
        // transpose read: lane supplies row r = (lane % 16) / 4 and 8-byte piece c = lane % 4 of its 16-lane group's
        // 16 columns; groups 0, 1 are the two column halves of the 32-wide fragment, groups 2, 3 the same for k + 8
        const int r = (lane & 15) >> 2, c = lane & 3, g = lane >> 4;
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
            b_off[fn] = (8 * (g >> 1) + r) * ROW + (((2 * wt + fn) ^ (r & PM)) << 6) + ((g & 1) << 5) + (c << 3);
    }

    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

    struct FragSet {
        Frag8 a[2];
        int idx[2];
        union { s16x4 q[4]; bf16x16 v; } b[2];
    };
    auto read_frags = [&](FragSet& f, const unsigned char* st, int ks) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            f.a[a].u = *reinterpret_cast<const uint4*>(st + (a_off[a] ^ (32 * ks)));
            f.idx[a] = *reinterpret_cast<const uint16_t*>(st + m_off[a] + 4 * ks);
        }
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int j = 0; j < 4; ++j)      // k rows 32 ks + 16 (j / 2) + 4 (j % 2) + (8 h + r): elements 4 j .. 4 j + 3 of the operand
                f.b[fn].q[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_s16x4*)(st + b_off[fn] + (32 * ks + 16 * (j >> 1) + 4 * (j & 1)) * ROW));
    };
    auto mma = [&](const FragSet& f) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int fn = 0; fn < 2; ++fn)
                acc[a][fn] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(f.a[a].v, f.b[fn].v, acc[a][fn], f.idx[a], 0, 0);
    };
#define SB() __builtin_amdgcn_sched_barrier(0)

    const int nk = (ks1 - ks0 - kg + KW - 1) / KW;
    auto step_of = [&](int kt) { return ks0 + kg + kt * KW; };
    if (nk > 0) {
#pragma unroll
    for (int p = 0; p < kGStages; ++p) {
        if (p >= nk) break;
        lookup(step_of(p));
        issue(step_of(p), p);
    }
    if (nk >= kGStages) wait_vmcnt<(kGStages - 1) * kGLoads>();
    else wait_vmcnt<0>();
    if (KW == 1) __syncthreads();
    else asm volatile("" ::: "memory");
    FragSet P, Q;
    read_frags(P, ring, 0);
    int stage = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + kGStages < nk;         // (the last steps load nothing: gemm_v2_body.hpp)
        const int next_stage = (stage + 1 == kGStages) ? 0 : stage + 1;
        const unsigned char* st = ring + stage * kGStage;
        const unsigned char* sn = ring + next_stage * kGStage;
        if (more) lookup(step_of(kt + kGStages));
        SB();
        mma(P); SB();
        read_frags(Q, st, 1); SB();
        // Q has arrived and this wave's part of tile kt + 1 has landed; after the barrier every wave is done reading
        // this stage, which is refilled at once
        if (kt + kGStages - 1 < nk) wait_vmcnt_lgkm0<(kGStages - 2) * kGLoads>();
        else wait_vmcnt_lgkm0<0>();
        if (KW == 1) __builtin_amdgcn_s_barrier();
        else asm volatile("" ::: "memory");
        SB();
        if (more) issue(step_of(kt + kGStages), stage);
        SB();
        mma(Q); SB();
        read_frags(P, sn, 0); SB();
        stage = next_stage;
    }
    wait_vmcnt<0>();
    }
#undef SB
    __syncthreads();
    if constexpr (KW > 1) {
        static_assert(KW == 4 && kJoin4 + 4 * 32 * 80 <= TL::RING, "four wavefronts; sums and their staging must fit in the main-loop LDS");
        float q[16];
        if (split.n == 1) {
            join4(acc, smem, wave, lane, q);
            store_quarter(q, 1.0f, smem + kJoin4, wave, lane, out, ldo, t0, n0, t0 + 64, N);
        } else if (split_join4(acc, smem, split, L, sp, wave, lane, q)) {
            store_quarter(q, 1.0f, smem + kJoin4, wave, lane, out, ldo, t0, n0, t0 + 64, N);
        }
        return;
    }

    // ---- output: the wave's 64 x 64 tile goes through LDS as [t][n] so that HBM sees 128-byte row segments --------
    constexpr int EP = 64 * 2 + 16;
    unsigned char* scratch = smem + wt * (64 * EP);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                // registers r, r + 1 are rows t, t + 1 of the same column: one 16-bit LDS store each
                const int t = a * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                const uint32_t pr = f2bf2(acc[a][fn][r], acc[a][fn][r + 1]);
                *reinterpret_cast<uint16_t*>(scratch + t * EP + (fn * 32 + l32) * 2) = (uint16_t)pr;
                *reinterpret_cast<uint16_t*>(scratch + (t + 1) * EP + (fn * 32 + l32) * 2) = (uint16_t)(pr >> 16);
            }
    wave_lds_sync();
    const int nw = n0 + 64 * wt;
    if (nw < N)
        store_between(past, [&](auto store) {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int row = p * 8 + (lane >> 3), ch = lane & 7;
                store(out + (int64_t)(t0 + row) * ldo + nw + ch * 8, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
            }
        });
}

// The same contraction on E4M3 codes (the fp8 step with blocks of M >= 16 columns): Ac = the survivors' codes [T, K' / 2] + the same
// metadata, Wq = codes [F, ldw bytes] with the contraction index as row, out = bf16(alpha * sum), alpha = the product of the two tensor scales.
// v_smfmac_f32_32x32x64_fp8_fp8 contracts 64 k' per instruction, so a stage holds 128 k' and occupies the same LDS as above: 128 gathered
// 256-byte row segments (four rows per wave-wide load), 64 x 64 bytes of codes, 64 x 16 bytes of metadata.  The B operand wants 16
// consecutive k' per lane and half (lds_dma.hpp); it is read with ds_read_b64_tr_b8: inside a group of 16 lanes, lane s supplies the address
// of 8 consecutive bytes of row s / 2 (piece s % 2) and lane l receives byte l of rows 0..7 (measured with an index pattern).  The 32-byte
// pieces of a row are XOR-swizzled by k' % 8, so the eight rows that the lower or upper 32 lanes read together cover all 64 banks once.
constexpr int kG8Stage = 128 * 256 + 64 * 64 + 64 * 16;
__device__ __forceinline__ void vnm_gather_fp8_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_meta,
                                                                 const uint8_t* __restrict__ colidx, const uint8_t* __restrict__ Wq,
                                                                 int ldw, int N, int Kc, int logM, int nblk_tok, int tiles_n, float alpha,
                                                                 uint16_t* __restrict__ out, int64_t ldo, const GemmGroup& grp, bool past) {
    constexpr int kB = 128 * 256, kA = 64 * 64, kStage = kG8Stage;      // 37888 bytes; two stages = 74 KB: two workgroups per CU

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const uint32_t smem_lds = lds_addr(smem);

    int L = xcd_run(pid, n_pid);
    const int tn = uniform(L / nblk_tok), tb = L - tn * nblk_tok;
    const int t0 = tb * 64, n0 = tn * 256;
    if (grp.n) {
        int e = 0;
        while (e + 1 < grp.n && t0 >= grp.seg[e + 1]) ++e;
        Wq += e * grp.b_stride;
    }
    // column offsets of this token block: a wave's 32 rows of a stage are 8 consecutive blocks = 32 consecutive bytes, read as is (same address
    // in every lane) one stage ahead of the loads that use them
    const uint4* cix = reinterpret_cast<const uint4*>(colidx + (int64_t)tb * Kc + 32 * wave);

    // B: load i of wave w (i = 0..7) brings rows k' = 4 (8 w + i) + lane / 16 of the stage; lane % 16 is the 16-byte slot inside the row and
    // fetches the chunk whose 32-byte piece the swizzle puts there.  Chunks past the right edge of Wq are redirected into the first 64 columns.
    const uint64_t w_base = uniform64(Wq);
    uint32_t b_col[2];
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int slot = lane & 15, k7 = 4 * par + (lane >> 4);
        int c = (((slot >> 1) ^ k7) << 1) | (slot & 1);
        if (n0 + c * 16 >= N) c &= 3;
        b_col[par] = (uint32_t)(n0 + c * 16);
    }
    const uint32_t row_bytes = (uint32_t)ldw;
    const int lda = Kc >> 1;                              // bytes per row of codes
    const uint64_t a_base = uniform64(a_codes + (int64_t)(t0 + 16 * wave) * lda);
    const uint64_t m_base = uniform64(a_meta + (int64_t)(t0 + 16 * wave) * (Kc >> 3));
    uint32_t a_lane, m_lane;
    {
        const int rb = lane >> 2, c = (lane & 3) ^ ((rb >> 2) & 3);
        a_lane = (uint32_t)(rb * lda + c * 16);
        m_lane = (uint32_t)(rb * (Kc >> 3) + (lane & 3) * 4);
    }
    uint4 cw[2];                                         // the 8 blocks' offsets of the stage to be issued next
    auto lookup = [&](int kt) {
        cw[0] = cix[kt * 8];
        cw[1] = cix[kt * 8 + 1];
    };
    const int bsh = (lane >> 4) * 8;                     // the lane's row inside a block of four
    auto issue = [&](int kt, int stage) {
        const uint32_t sb = smem_lds + stage * kStage;
        const uint32_t sa = sb + kB, sm = sa + kA;
        const uint32_t w8[8] = {cw[0].x, cw[0].y, cw[0].z, cw[0].w, cw[1].x, cw[1].y, cw[1].z, cw[1].w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // row k' = 4 (32 kt + 8 w + i) + lane / 16 of the compact operand = row block * M + offset of the dense one
            const uint32_t row = (uint32_t)((kt * 32 + 8 * wave + i) << logM) + ((w8[i] >> bsh) & 0xFFu);
            dma16(w_base, row * row_bytes + b_col[i & 1], sb + (8 * wave + i) * 1024);
        }
        dma16(a_base, a_lane + (uint32_t)kt * 64, sa + wave * 1024);
        dma4(m_base, m_lane + (uint32_t)kt * 16, sm + wave * 256);
    };

    int a_off[2], m_off[2], b_off[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int row = a * 32 + l32;
        a_off[a] = kB + row * 64 + ((lh ^ ((row >> 2) & 3)) << 4);
        m_off[a] = kB + kA + row * 16 + 4 * lh;
    }
    {
        // transpose read: lane supplies row r = (lane % 16) / 2 and 8-byte piece c = lane % 2 of its 16-lane group's 16 columns; groups 0, 1
        // are the two column halves of the 32-wide fragment, groups 2, 3 the same for k' + 16
        const int r = (lane & 15) >> 1, c = lane & 1, g = lane >> 4;
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
            b_off[fn] = (16 * (g >> 1) + r) * 256 + (((2 * wave + fn) ^ r) << 5) + ((g & 1) << 4) + (c << 3);
    }

    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

    struct FragSet {
        Frag8 a[2];
        int idx[2];
        union { v2i q[4]; i32x8 v; } b[2];
    };
    auto read_frags = [&](FragSet& f, const unsigned char* st, int ks) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            f.a[a].u = *reinterpret_cast<const uint4*>(st + (a_off[a] ^ (32 * ks)));
            f.idx[a] = *reinterpret_cast<const uint32_t*>(st + m_off[a] + 8 * ks);
        }
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int j = 0; j < 4; ++j)      // k' rows 64 ks + 32 (j / 2) + 8 (j % 2) + (16 h + r): bytes 8 j .. 8 j + 7 of the operand
                f.b[fn].q[j] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(st + b_off[fn] + (64 * ks + 32 * (j >> 1) + 8 * (j & 1)) * 256));
    };
    auto mma = [&](const FragSet& f) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int fn = 0; fn < 2; ++fn)
                acc[a][fn] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(f.a[a].q, f.b[fn].v, acc[a][fn], f.idx[a], 0, 0);
    };
#define SB() __builtin_amdgcn_sched_barrier(0)

    const int nk = Kc >> 7;
#pragma unroll
    for (int p = 0; p < kGStages; ++p) {
        if (p >= nk) break;
        lookup(p);
        issue(p, p);
    }
    if (nk >= kGStages) wait_vmcnt<(kGStages - 1) * kGLoads>();
    else wait_vmcnt<0>();
    __syncthreads();
    FragSet P, Q;
    read_frags(P, smem, 0);
    int stage = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + kGStages < nk;
        const int next_stage = (stage + 1 == kGStages) ? 0 : stage + 1;
        const unsigned char* st = smem + stage * kStage;
        const unsigned char* sn = smem + next_stage * kStage;
        if (more) lookup(kt + kGStages);
        SB();
        mma(P); SB();
        read_frags(Q, st, 1); SB();
        if (kt + kGStages - 1 < nk) wait_vmcnt_lgkm0<(kGStages - 2) * kGLoads>();
        else wait_vmcnt_lgkm0<0>();
        __builtin_amdgcn_s_barrier();
        SB();
        if (more) issue(kt + kGStages, stage);
        SB();
        mma(Q); SB();
        read_frags(P, sn, 0); SB();
        stage = next_stage;
    }
#undef SB
    wait_vmcnt<0>();
    __syncthreads();

    constexpr int EP = 64 * 2 + 16;
    unsigned char* scratch = smem + wave * (64 * EP);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const int t = a * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                const uint32_t pr = f2bf2(acc[a][fn][r] * alpha, acc[a][fn][r + 1] * alpha);
                *reinterpret_cast<uint16_t*>(scratch + t * EP + (fn * 32 + l32) * 2) = (uint16_t)pr;
                *reinterpret_cast<uint16_t*>(scratch + (t + 1) * EP + (fn * 32 + l32) * 2) = (uint16_t)(pr >> 16);
            }
    wave_lds_sync();
    const int nw = n0 + 64 * wave;
    if (nw < N)
        store_between(past, [&](auto store) {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int row = p * 8 + (lane >> 3), ch = lane & 7;
                store(out + (int64_t)(t0 + row) * ldo + nw + ch * 8, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
            }
        });
}

template <class TL>
struct GatherUnit {
    using Args = GatherArgs;
    static constexpr int THREADS = TL::THREADS, LDS = TL::RING + kGMaxKc;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        vnm_gather_body<TL>(smem, pid, n_pid, (const uint16_t*)a.a_vals, a.a_meta, a.colidx, (const uint16_t*)a.Wk, a.ldw, a.N, a.Kc, a.logM, a.T >> 6, a.tiles_n, a.out, a.ldo, a.grp, a.split, a.past != 0);
    }
    static unsigned count(const Args& a) { return (unsigned)((a.T >> 6) * ((a.N + TL::BN - 1) / TL::BN) * a.split.n); }
    static int stages(const Args& a) { return a.Kc / 64 / (TL::KW * a.split.n); }      // of a tile, a wavefront's (wgrad_first)
    static Args args(Args a) { a.tiles_n = (a.N + TL::BN - 1) / TL::BN; return a; }
};
using GatherUnit256 = GatherUnit<GTile<4, 2, 1>>;      // 64 tokens x 256 columns, two workgroups per CU
using GatherUnit64 = GatherUnit<GTile<1, 3, 4>>;       // 64 x 64
struct GatherFp8Unit {
    using Args = GatherArgs;
    static constexpr int THREADS = 256, LDS = kGStages * kG8Stage;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        vnm_gather_fp8_body(smem, pid, n_pid, (const uint8_t*)a.a_vals, a.a_meta, a.colidx, (const uint8_t*)a.Wk, a.ldw, a.N, a.Kc, a.logM, a.T >> 6, a.tiles_n, a.alpha, a.out, a.ldo, a.grp, a.past != 0);
    }
    static unsigned count(const Args& a) { return (unsigned)((a.T >> 6) * ((a.N + 255) / 256)); }
    static int stages(const Args& a) { return a.Kc / 128; }
    static Args args(Args a) { a.tiles_n = (a.N + 255) / 256; return a; }
};

}  // namespace sffn
