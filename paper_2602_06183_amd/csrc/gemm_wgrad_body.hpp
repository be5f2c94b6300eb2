// Weight-gradient contractions of the fused step, eq. (5) dW2 = y2.T dY and eq. (8) dW1 = dy1.T X (Alg. 2 lines 3, 6):
//   C[f, n] = sum_t A[t, f] * G[t, n],  A = the V:N:M activation (y2 or dy1), G = dY or X, contraction over tokens.
// The 2:4 structure of A lies along the output rows here, so the structured-sparse matrix instruction does not apply;
// what the format still gives is that, inside a block of 64 tokens, only 4 of every 8 hidden units are non-zero.
// The producer (the V:N:M epilogue of gemm_v2.hip) therefore stores the transposed activation compacted to those
// rows ("atc": row 4 g + p of token block tb = hidden unit 8 g + colidx[tb, g, p]; [F / 2 rows, T tokens], blocked
// layout of common.hpp), which halves its bytes in HBM, in L2 and on the way into LDS.  This kernel runs dense
// v_mfma_f32_16x16x32_bf16 on a 256 (hidden) x 256 tile; a lane that needs hidden unit f looks up, once per
// 64-token stage, whether f is one of its group's four kept units (a bit mask per group, written by the producer;
// the position among the kept units is a population count) and reads either that compact row or a row of zeros
// kept at the end of the tile.  Same ring / barrier / LDS-DMA discipline as gemm_v2.hip: 3 stages of 64
// tokens (A 16 KB as two 32-token halves, G 32 KB as two halves, 8 private copies of the tile's 32 mask bytes).
// What bounds it is the power that the matrix instructions take, at 77 % of the pipe's cycles.  The 16 x 16 form does the same products (and sums: same bits) as
// 32 x 32 x 16 for 12 % less of it (registers only, half of the rows zero: 2167 TFLOP/s with 32 x 32 x 16, 2433 with this one): T = N = 8192, F = 28672 2580 -> 2380 us
// at a clock of 1.84 -> 2.01 GHz; T = 8192, N = 2048, F = 8192 220 -> 206.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"

namespace sffn {

// Workgroup tile: WVM x WVN wavefronts of WM hidden units x 64 columns each; KW > 1 (with one wavefront per tile): KW wavefronts share the
// tile, wavefront g contracting token blocks g, g + KW, ... in a ring of its own; their partial sums meet in LDS.
template <int WVM_, int WVN_, int WM_, int NST_, int KW_>
struct WTile {
    static constexpr int WVM = WVM_, WVN = WVN_, WM = WM_, NST = NST_, KW = KW_;
    static constexpr int NW = WVM * WVN, BM = WVM * WM, BN = WVN * 64, THREADS = 64 * NW * KW;
    static_assert(KW == 1 || NW == 1, "a shared output tile belongs to single wavefronts");
    // stage (64 tokens; on codes 128): BM / 2 compact rows x 64 bytes and four rows of zeros, twice; G likewise in two halves; a private copy of the mask bytes per wavefront
    static constexpr int kZero = BM / 2 * 64, kZeros = 256, kAHalf = kZero + kZeros, kABytes = 2 * kAHalf, kBHalf = BN * 64, kBBytes = 2 * kBHalf;
    static constexpr int kStage = kABytes + kBBytes + NW * 256;
    static constexpr int A_LD = BM / 32 / NW, B_LD = kBBytes / 1024 / NW, kLoads = 1 + 2 * A_LD + B_LD;      // LDS-DMA loads per wavefront per stage
    static constexpr int EPI = NW * 64 * (64 * 4 + 16) / 2 > NW * 64 * (64 * 2 + 16) ? NW * 64 * (64 * 4 + 16) / 2 : NW * 64 * (64 * 2 + 16);   // wgrad_store's staging
    static constexpr int BYTES = KW * NST * kStage > EPI ? KW * NST * kStage : EPI;
    // on codes a stage of the shared tile (KW > 1) is one token block, half of everything
    static constexpr int k8A = kAHalf, k8B = kBHalf, k8Stage = k8A + k8B + NW * 256, B8_LD = k8B / 1024 / NW, k8Loads = 1 + A_LD + B8_LD;
    static constexpr int BYTES8 = KW == 1 ? BYTES : KW * NST * k8Stage > EPI ? KW * NST * k8Stage : EPI;
};

// Which of the four rows of zeros a lane reads for a hidden unit that is not kept.  A ds_read_b128 is served in phases of 16 lanes, and a phase is
// lanes 0-3, 12-15, 20-27 of a half-wavefront or its other 16 (measured: two lanes' reads of one bank take longer exactly then): columns 0-3 or 4-7 of each of
// four groups of hidden units.  A group's four kept rows lie in four different quarters of the banks at one 16-byte chunk, its kept columns below 4 from the
// first quarter up, the others up to the last.  So with a unit that is not kept in columns 0-3 the last quarter is free in their phase, with one in columns
// 4-7 the first.  (One row of zeros for all, at another group's chunk: 0.16 ms of 2.5 at T = D = 8192, F = 28672 went into bank conflicts.)
__device__ __forceinline__ int zero_lane(int l32) { return (l32 & 4) ? 0 : 3 * 64; }

// partial sums of KW wavefronts -> the first one, in ascending order; returns false for the wavefronts that are done
template <class TL, class V, int FM, int FN>
__device__ __forceinline__ bool wgrad_join(V (&acc)[FM][FN], unsigned char* smem, int kg, int lane) {
    constexpr int R = sizeof(V) / 4, PART = FM * FN * R * 256;
    static_assert((TL::KW - 1) * PART <= TL::BYTES && (TL::KW - 1) * PART <= TL::BYTES8, "partial sums must fit in the main-loop LDS");
    if (kg > 0) {
        float* p = reinterpret_cast<float*>(smem + (kg - 1) * PART) + lane;
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
#pragma unroll
                for (int r = 0; r < R; ++r) p[((a * FN + b) * R + r) * 64] = acc[a][b][r];
    }
    __syncthreads();
    if (kg > 0) return false;
    for (int g = 1; g < TL::KW; ++g) {
        const float* p = reinterpret_cast<const float*>(smem + (g - 1) * PART) + lane;
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
#pragma unroll
                for (int r = 0; r < R; ++r) acc[a][b][r] += p[((a * FN + b) * R + r) * 64];
    }
    wave_lds_sync();
    return true;
}

// Accumulators of one WM x 64 wave tile (lane: column l % 16, rows 4 (l / 16) .. + 3 of a fragment) -> bf16 output (one rounding; `alpha` = product of the operand scales of
// the fp8 form, 1 otherwise).  ACC32: `out` is a float32 matrix of the same shape that the tile is ADDED to (gradient accumulation over the micro-batches of an
// optimizer step): out32 = out32 + alpha * sum, both in float32.
template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_store(f32x4 (&acc)[TL::WM / 16][4], float alpha, unsigned char* smem, int wave, int lane, int i0, int j0, int F, int N,
                                            uint16_t* __restrict__ out, int64_t ldo) {
    constexpr int WM = TL::WM, WN = 64;
    const int wm = wave / TL::WVN, wn = wave % TL::WVN, l16 = lane & 15, lq = lane >> 4;
    if (ACC32) {
        // rows of 64 float32 of the output: (OUT_I_CONTIG) 32 columns j x 64 hidden units, else 32 hidden units x 64 columns.  The products are rounded to float32 before
        // they are staged, so the addition is never a fused multiply-add
        float* out32 = reinterpret_cast<float*>(out);
        constexpr int EP = 64 * 4 + 16, NQ = OUT_I_CONTIG ? WM / 64 * 2 : WM / 32;
        unsigned char* scratch = smem + wave * (32 * EP);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int row0 = OUT_I_CONTIG ? j0 + wn * WN + (q & 1) * 32 : i0 + wm * WM + q * 32, col0 = OUT_I_CONTIG ? i0 + wm * WM + (q >> 1) * 64 : j0 + wn * WN;
            const int rows = OUT_I_CONTIG ? N : F, cols = OUT_I_CONTIG ? F : N;
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    if (OUT_I_CONTIG) {
                        const f32x4 v = acc[(q >> 1) * 4 + y][(q & 1) * 2 + x];
                        *reinterpret_cast<float4*>(scratch + (x * 16 + l16) * EP + (y * 16 + 4 * lq) * 4) = make_float4(v[0] * alpha, v[1] * alpha, v[2] * alpha, v[3] * alpha);
                    } else {
                        const f32x4 v = acc[q * 2 + x][y];
#pragma unroll
                        for (int r = 0; r < 4; ++r) *reinterpret_cast<float*>(scratch + (x * 16 + 4 * lq + r) * EP + (y * 16 + l16) * 4) = v[r] * alpha;
                    }
                }
            wave_lds_sync();
            // all of the slab's old values are requested before the first sum is stored (a store would otherwise stand between the loads)
            float4 old[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int r = row0 + p * 4 + (lane >> 4), c = col0 + (lane & 15) * 4;
                old[p] = (r < rows && c < cols) ? *reinterpret_cast<const float4*>(out32 + (int64_t)r * ldo + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int r = row0 + p * 4 + (lane >> 4), c = col0 + (lane & 15) * 4;
                if (r < rows && c < cols) {
                    const float4 add = *reinterpret_cast<const float4*>(scratch + (p * 4 + (lane >> 4)) * EP + (lane & 15) * 16);
                    store_out(out32 + (int64_t)r * ldo + c, make_float4(old[p].x + add.x, old[p].y + add.y, old[p].z + add.z, old[p].w + add.w));
                }
            }
            wave_lds_sync();
        }
    } else if (OUT_I_CONTIG) {
        // out[j * ldo + i]: a lane owns 4 consecutive i of one j; stage [j][i] through LDS (two halves of 64 i) so that HBM sees 128-byte row segments
        constexpr int EP = 64 * 2 + 16;
        unsigned char* scratch = smem + wave * (WN * EP);
#pragma unroll
        for (int h = 0; h < WM / 64; ++h) {
            const int f0 = i0 + wm * WM + h * 64, n0 = j0 + wn * WN;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const f32x4 v = acc[4 * h + a][b];
                    *reinterpret_cast<uint2*>(scratch + (b * 16 + l16) * EP + (a * 16 + 4 * lq) * 2) = make_uint2(f2bf2(v[0] * alpha, v[1] * alpha), f2bf2(v[2] * alpha, v[3] * alpha));
                }
            wave_lds_sync();
#pragma unroll
            for (int p = 0; p < WN / 8; ++p) {
                const int row = p * 8 + (lane >> 3), ch = lane & 7;
                const int j = n0 + row, i = f0 + ch * 8;
                if (j < N && i < F)
                    store_out(out + (int64_t)j * ldo + i, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
            }
            wave_lds_sync();
        }
    } else {
        // out[i * ldo + j]: transpose each 32-row slab through LDS for 16-byte row stores
        constexpr int EP = WN * 2 + 16;
        unsigned char* scratch = smem + wave * (32 * EP);
#pragma unroll
        for (int a = 0; a < WM / 32; ++a) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<uint16_t*>(scratch + (x * 16 + 4 * lq + r) * EP + (b * 16 + l16) * 2) = (uint16_t)f2bf(acc[2 * a + x][b][r] * alpha);
            wave_lds_sync();
#pragma unroll
            for (int p = 0; p < 32 * (WN / 8) / 64; ++p) {
                const int e = lane + 64 * p, row = e / (WN / 8), ch = e % (WN / 8);
                const int i = i0 + wm * WM + a * 32 + row, j = j0 + wn * WN + ch * 8;
                if (i < F && j < N)
                    store_out(out + (int64_t)i * ldo + j, *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16));
            }
            wave_lds_sync();
        }
    }
}

template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_vnm_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ atc, const uint8_t* __restrict__ kmask,
                                                       const uint16_t* __restrict__ G, int F, int N, int Ttot,
                                                       uint16_t* __restrict__ out, int64_t ldo, int tiles_m, int tiles_n,
                                                       const GemmGroup& grp) {
    constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = 64, FM = WM / 16, FN = 4, KW = TL::KW;
    constexpr int kStages = TL::NST, kStage = TL::kStage, kAHalf = TL::kAHalf, kABytes = TL::kABytes, kBHalf = TL::kBHalf, kBBytes = TL::kBBytes, kLoads = TL::kLoads;
    constexpr int A_LD = TL::A_LD, B_LD = TL::B_LD;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KW > 1 ? wave : 0, wt = KW > 1 ? 0 : wave;       // share of the contraction / place in the tile
    const int wm = wt / TL::WVN, wn = wt % TL::WVN;
    const int l16 = lane & 15, lq = lane >> 4;
    unsigned char* const ring = smem + kg * (kStages * kStage);
    const uint32_t ring_lds = lds_addr(smem) + kg * (kStages * kStage);

    // workgroup -> tile: an XCD gets a run of consecutive logical ids, which walk bands of 4 tile rows
    int L = xcd_run(pid, n_pid);
    int k_base = 0, K = Ttot;                     // grouped: every expert contracts over its own token segment
    if (grp.n) {
        const int per = tiles_m * tiles_n, e = uniform(L / per);
        L -= e * per;
        k_base = grp.seg[e];
        K = grp.seg[e + 1] - k_base;
        out += e * grp.out_stride * (ACC32 ? 2 : 1);          // (float32 elements are two uint16_t wide)
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, SFFN_TILE_GROUP, tm, tn);
    const int i0 = tm * BM, j0 = tn * BN;
    const int KC = Ttot / 32;                     // 32-token chunks per row of the blocked operands

    // ---- wave-uniform sources of the DMA loads (tile 0 of the k loop) and per-lane offsets.  Rows past the
    //      matrix edge are clamped into it: they only feed outputs that are never stored. ------------------
    uint64_t a_base[A_LD][2], b_base[B_LD], c_base;
    const int rb = lane >> 2;
    const uint32_t blk_lane = (uint32_t)(rb * 32 + ((lane & 3) ^ swz4(rb >> 2)) * 8) * 2;
    {
#pragma unroll
        for (int n = 0; n < A_LD; ++n) {
            int cr = i0 / 2 + (wt * A_LD + n) * 16; cr = cr < F / 2 ? cr : F / 2 - 16;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) a_base[n][kc] = uniform64(atc + (((int64_t)(cr >> 4) * KC + k_base / 32 + kc) << 9));
        }
#pragma unroll
        for (int n = 0; n < B_LD; ++n) {
            const int bk = wt * B_LD + n, h = bk / (BN / 16);
            int gr = j0 + (bk % (BN / 16)) * 16; gr = gr < N ? gr : N - 16;
            b_base[n] = uniform64(G + (((int64_t)(gr >> 4) * KC + k_base / 32 + h) << 9));
        }
        c_base = uniform64(kmask + (int64_t)(k_base / 64) * (F / 8));
    }
    // mask bytes of the tile's 32 groups of 8 hidden units (lanes 0-7 bring 4 each, the others repeat them); every
    // wavefront fetches its own copy
    uint32_t c_lane;
    {
        int g = i0 / 8 + 4 * (lane & 7); g = g < F / 8 ? g : F / 8 - 4;
        c_lane = (uint32_t)g;
    }
    const uint32_t c_kstep = (uint32_t)(F / 8);

    // loads lo .. hi - 1 of a stage's kLoads (compile-time bounds)
    auto issue = [&](int kt, int stage, int lo, int hi) {
        const uint32_t sa = ring_lds + stage * kStage, sb = sa + kABytes, sc = sb + kBBytes;
        const uint32_t o = blk_lane + (uint32_t)kt * 2048;      // k position in the per-lane offset; bases stay in SGPRs
        if (lo <= 0 && hi > 0) dma4(c_base, c_lane + (uint32_t)kt * c_kstep, sc + wt * 256);     // first: the look-up wants it earliest
#pragma unroll
        for (int n = 0; n < 2 * A_LD; ++n)
            if (1 + n >= lo && 1 + n < hi) dma16(a_base[n >> 1][n & 1], o, sa + (n & 1) * kAHalf + (wt * A_LD + (n >> 1)) * 1024);
#pragma unroll
        for (int n = 0; n < B_LD; ++n)
            if (1 + 2 * A_LD + n >= lo && 1 + 2 * A_LD + n < hi) dma16(b_base[n], o, sb + (wt * B_LD + n) * 1024);
    };

    // ---- fragment reads.  Sub-step s (32 tokens) of a stage is its half s; lane -> row l16 of a fragment, 16-byte chunk lq of its 64 bytes. ----
    const int b_off = kABytes + (wn * WN + l16) * 64 + ((lq ^ swz4(l16 >> 2)) << 4);
    // hidden unit of fragment a in this lane: i0 + wm * WM + a * 16 + l16 -> group 2 a + hb of the wavefront's WM / 8, column l16 % 8 of the group.  Its row in a half-tile
    // is 4 groups + the number of kept units below it; a unit that is not kept reads zeros, from the row that its half-group leaves free (zero_lane).
    // a_off[a] = LDS address for fragment a less a * 512, looked up once per stage.
    const int hb = l16 >> 3, col = l16 & 7, g0 = wm * (WM / 8) + hb;
    const uint32_t below[2] = {((1u << col) - 1u) << (8 * hb), ((1u << col) - 1u) << (8 * hb + 16)};      // even / odd a: two groups to a half of a mask word
    const uint32_t bit[2] = {(uint32_t)(8 * hb + col), (uint32_t)(8 * hb + col + 16)};
    const uint32_t lb[2] = {(uint32_t)(g0 * 256 + ((lq ^ swz4(hb)) << 4)), (uint32_t)(g0 * 256 + ((lq ^ swz4(2 + hb)) << 4))};
    const uint32_t no_row = (uint32_t)(TL::kZero / 64 + zero_lane(l16) / 64 - g0 * 4);
    uint32_t a_off[FM], mk[FM / 2];
    auto lookup_read = [&](int stage) {         // the wavefront's mask bytes: the same words in every lane
        const unsigned char* sc = ring + stage * kStage + kABytes + kBBytes + wt * 256 + wm * (WM / 8);
        if constexpr (FM == 8) {
            const uint4 w = *reinterpret_cast<const uint4*>(sc);
            mk[0] = w.x; mk[1] = w.y; mk[FM / 2 - 2] = w.z; mk[FM / 2 - 1] = w.w;
        } else {
            const uint2 w = *reinterpret_cast<const uint2*>(sc);
            mk[0] = w.x; mk[1] = w.y;
        }
    };
    auto lookup = [&](int stage, int a) {
        const uint32_t kept = (uint32_t)__builtin_amdgcn_sbfe((int)mk[a >> 1], bit[a & 1], 1), row = (uint32_t)__builtin_popcount(mk[a >> 1] & below[a & 1]);
        a_off[a] = ((row & kept) | ((no_row - 8 * a) & ~kept)) * 64 + (lb[a & 1] + (uint32_t)(stage * kStage));
    };
    auto read_a = [&](Frag8& f, int s, int a) { f.u = *reinterpret_cast<const uint4*>(ring + a_off[a] + (a * 512 + s * kAHalf)); };
    auto read_b = [&](Frag8& f, const unsigned char* st, int s, int b) { f.u = *reinterpret_cast<const uint4*>(st + b_off + (b * 1024 + s * kBHalf)); };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.0f;
    Frag8 A[4], B[2][FN];
    auto mma_row = [&](int s, int a) {
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[a & 3].v, B[s][b].v, acc[a][b], 0, 0, 0);
    };
#define SB() __builtin_amdgcn_sched_barrier(0)

    // token blocks of this wavefront: all of them, or (KW > 1) every KW-th one from its own on.  0 for an expert without tokens: its gradient is zero
    const int nk = KW == 1 ? K / 64 : (K / 64 - kg + KW - 1) / KW;
    auto step_of = [&](int kt) { return KW == 1 ? kt : kg + kt * KW; };
    // The last steps load nothing (gemm_v2_body.hpp says why), except on the 256 tile, whose last tile is loaded again in their place: a second copy of its step, without loads, runs
    // out of registers (on codes T = N = 8192, F = 28672 1270 -> 1660 us).
    constexpr bool REPEAT = FM == 8;
    auto tile_of = [&](int t) { return step_of(REPEAT && t >= nk ? nk - 1 : t); };
    // (Nothing is in flight here, but the compiler, which does not see the ring's loads, may believe it of other units' loads to the same registers and wait in every step: as the
    // second unit of three, T = 3072, N = 448, F = 1792, the launch took 43 us, 25 without those waits.)
    wait_vmcnt<0>();
    if (nk > 0) {
        // rows of zeros behind both half-tiles of every stage (never touched by the DMA)
        constexpr int ZW = TL::kZeros / 4;
        for (int i = wt * 64 + lane; i < kStages * 2 * ZW; i += TL::NW * 64)
            *reinterpret_cast<uint32_t*>(ring + i / (2 * ZW) * kStage + (i / ZW & 1) * kAHalf + TL::kZero + i % ZW * 4) = 0u;
#pragma unroll
        for (int p = 0; p < kStages; ++p)
            if (REPEAT || p < nk) issue(tile_of(p), p, 0, p < kStages - 1 ? kLoads : kLoads * 2 / 6);           // (the rest of the last one's loads are the first step's)
        if (REPEAT || nk >= kStages) wait_vmcnt<(kStages - 2) * kLoads + kLoads * 2 / 6>();
        else wait_vmcnt<0>();
        if (KW == 1) __syncthreads();
        else { wave_lds_sync(); asm volatile("" ::: "memory"); }
        lookup_read(0);
#pragma unroll
        for (int a = 0; a < FM; ++a) lookup(0, a);
#pragma unroll
        for (int a = 0; a < 4; ++a) read_a(A[a], 0, a);
#pragma unroll
        for (int b = 0; b < FN; ++b) read_b(B[0][b], ring, 0, b);
        constexpr int BAR = FM - 4;
        int stage = 0;
        // One step = one stage = two sub-steps of FM rows of four matrix instructions.  A row's fragment is read four rows ahead, G's fragments one sub-step
        // ahead.  The next stage's mask bytes are the first load of its batch; its rows are looked up as the last reads of this stage are issued, and once every
        // wavefront has issued all of them (barrier, four rows before the step's end) the stage is refilled with the tile three steps ahead.
        // The loads are spread over the step (gemm_v2_body.hpp says why).
        // re_kt, re_stage: the tile that is loaded and its stage; full: both of a step's exist
#define ISSUE(t, i) if (full.value || (t) < nk) issue(re_kt, re_stage, kLoads * (i) / 6, kLoads * ((i) + 1) / 6)
        int re_kt = tile_of(kStages - 1), re_stage = kStages - 1;
        auto step = [&](auto full, int kt) {
            const int next_stage = (stage + 1 == kStages) ? 0 : stage + 1;
            const unsigned char* st = ring + stage * kStage;
            const unsigned char* sn = ring + next_stage * kStage;
#pragma unroll
            for (int a = 0; a < FM; ++a) {
                mma_row(0, a); SB();
                if (a + 4 < FM) read_a(A[a & 3], 0, a + 4);
                else read_a(A[a & 3], 1, a + 4 - FM);
                if (FM == 8) { if (a < FN) read_b(B[1][a], st, 1, a); }
                else if (a < 2) { read_b(B[1][2 * a], st, 1, 2 * a); read_b(B[1][2 * a + 1], st, 1, 2 * a + 1); }
                SB();
                if (FM == 8) { if (a < 4) { ISSUE(kt + kStages - 1, 2 + a); } }
                else if (a < 2) { ISSUE(kt + kStages - 1, 2 + 2 * a); ISSUE(kt + kStages - 1, 3 + 2 * a); }
                if (a == FM - 2) {
                    // all but kLoads - 1 of the next stage's batch and the batch after it may still be in flight
                    if (full.value || kt + kStages - 1 < nk) wait_vmcnt<(kStages - 2) * kLoads + kLoads - 1>();
                    else wait_vmcnt<0>();
                    if (KW > 1) asm volatile("" ::: "memory");
                    lookup_read(next_stage);
                }
                SB();
            }
#pragma unroll
            for (int a = 0; a < FM; ++a) {
                mma_row(1, a); SB();
                if (a + 4 < FM) { read_a(A[a & 3], 1, a + 4); SB(); }
                if (FM == 8 && a < 4) { lookup(next_stage, a); lookup(next_stage, a + FM - 4); SB(); }
                if (FM == 4 && a == 0) {
#pragma unroll
                    for (int r = 0; r < FM; ++r) lookup(next_stage, r);
                    SB();
                }
                if (a == BAR) {
                    // this wavefront's reads of the stage are here, and its part of tile kt + 1
                    if (full.value || kt + kStages - 1 < nk) wait_vmcnt_lgkm0<(kStages - 2) * kLoads>();
                    else wait_vmcnt_lgkm0<0>();
                    if (KW == 1) __builtin_amdgcn_s_barrier();
                    else asm volatile("" ::: "memory");
                    SB();
                    re_kt = tile_of(kt + kStages); re_stage = stage;
#pragma unroll
                    for (int r = 0; r <= BAR - (FM - 4); ++r) read_a(A[r], 0, r);
#pragma unroll
                    for (int b = 0; b < FN; ++b) read_b(B[0][b], sn, 0, b);
                    SB();
                }
                if (a > BAR) { read_a(A[a & 3], 0, a - (FM - 4)); SB(); }
                if (a == FM - 2) { ISSUE(kt + kStages, 0); SB(); }
                if (a == FM - 1) { ISSUE(kt + kStages, 1); SB(); }
            }
            stage = next_stage;
        };
        int kt = 0;
        for (; kt < (REPEAT ? nk : nk - kStages); ++kt) step(Flag<true>(), kt);
        if constexpr (!REPEAT)
            for (; kt < nk; ++kt) step(Flag<false>(), kt);
#undef ISSUE
        wait_vmcnt<0>();
    }
#undef SB
    __syncthreads();
    if (KW > 1 && !wgrad_join<TL>(acc, smem, kg, lane)) return;

    wgrad_store<OUT_I_CONTIG, ACC32, TL>(acc, 1.0f, smem, wt, lane, i0, j0, F, N, out, ldo);
}

// The same contraction on E4M3 codes (the fp8 step with SFFN_FLAG_FP8_WGRAD): atc and G hold one code per element, in the blocked layout
// with a pair of codes per 2-byte element, so one 64-byte chunk of a row is exactly one 64-token block.  v_mfma_scale_f32_16x16x128_f8f6f4 with
// unit scales contracts two such blocks per instruction (measured: lane l supplies k 32 (l / 16) .. + 31 of row / column l % 16 in both operands), so a stage is the bf16
// kernel's with a block for a half: the upper 32 lanes look their rows up in the second block's masks.  A block that is not there (an odd number of them) is one that
// keeps nothing.  A fragment is read two rows ahead.  out = bf16(alpha * sum), alpha = product of the two tensor scales.
// (v_mfma_scale_f32_32x32x64_f8f6f4, one block per instruction, takes 9 % more power for the same products: registers only 3900 TFLOP/s, this one 4240.)
template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_vnm_fp8_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ atc, const uint8_t* __restrict__ kmask,
                                                           const uint16_t* __restrict__ G, int F, int N, int Ttot, float alpha,
                                                           uint16_t* __restrict__ out, int64_t ldo, int tiles_m, int tiles_n, const GemmGroup& grp) {
    constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = 64, FM = WM / 16, FN = 4;
    static_assert(TL::KW == 1, "the shared tile has a kernel of its own");
    constexpr int kStages = TL::NST, kStage = TL::kStage, kAHalf = TL::kAHalf, kABytes = TL::kABytes, kBHalf = TL::kBHalf, kBBytes = TL::kBBytes, kLoads = TL::kLoads;
    constexpr int A_LD = TL::A_LD, B_LD = TL::B_LD;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wt = wave;                          // place in the tile
    const int wm = wt / TL::WVN, wn = wt % TL::WVN;
    const int l16 = lane & 15, lq = lane >> 4, blk = lq >> 1;
    unsigned char* const ring = smem;
    const uint32_t ring_lds = lds_addr(smem);
    int L = xcd_run(pid, n_pid);
    int k_base = 0, K = Ttot;                     // grouped: every expert contracts over its own token segment
    if (grp.n) {
        const int per = tiles_m * tiles_n, e = uniform(L / per);
        L -= e * per;
        k_base = grp.seg[e];
        K = grp.seg[e + 1] - k_base;
        out += e * grp.out_stride * (ACC32 ? 2 : 1);          // (float32 elements are two uint16_t wide)
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, SFFN_TILE_GROUP, tm, tn);
    const int i0 = tm * BM, j0 = tn * BN;
    const int KC = Ttot / 64;                     // 64-token chunks (64 bytes) per row of the blocked operands
    const int nblk = K / 64;

    // chunk c of row group g lies in slot c ^ swz8(g): a lane takes chunks 2 (lq % 2) and the next, and again every phase of a read meets 64 banks (swz4 in lds_dma.hpp)
    auto swz8 = [](int g) { return (g & 3) ^ ((g & 3) >> 1); };
    uint64_t a_base[A_LD], b_base[B_LD], c_base;
    const int rb = lane >> 2;
    const uint32_t blk_lane = (uint32_t)(rb * 32 + ((lane & 3) ^ swz8(rb >> 2)) * 8) * 2;
    {
#pragma unroll
        for (int n = 0; n < A_LD; ++n) {
            int cr = i0 / 2 + (wt * A_LD + n) * 16; cr = cr < F / 2 ? cr : F / 2 - 16;
            a_base[n] = uniform64(atc + (((int64_t)(cr >> 4) * KC + k_base / 64) << 9));
        }
#pragma unroll
        for (int n = 0; n < B_LD; ++n) {
            int gr = j0 + ((wt * B_LD + n) % (BN / 16)) * 16; gr = gr < N ? gr : N - 16;
            b_base[n] = uniform64(G + (((int64_t)(gr >> 4) * KC + k_base / 64) << 9));
        }
        c_base = uniform64(kmask + (int64_t)(k_base / 64) * (F / 8));
    }
    // mask bytes: lanes 0-7 bring the first block's 32, lanes 8-15 the second's, the others repeat them
    uint32_t c_lane;
    {
        int g = i0 / 8 + 4 * (lane & 7); g = g < F / 8 ? g : F / 8 - 4;
        c_lane = (uint32_t)g;
    }
    const uint32_t c_kstep = (uint32_t)(F / 8);
    auto issue = [&](int kt, int stage, int lo, int hi) {
        const uint32_t sa = ring_lds + stage * kStage, sb = sa + kABytes, sc = sb + kBBytes;
        const int second = 2 * kt + 1 < nblk ? 2 * kt + 1 : nblk - 1;           // (clamped into the operand; its rows then keep nothing)
        const uint32_t o[2] = {blk_lane + (uint32_t)kt * 2048, blk_lane + (uint32_t)second * 1024};
        if (lo <= 0 && hi > 0) dma4(c_base, c_lane + (uint32_t)((lane & 8) ? second : 2 * kt) * c_kstep, sc + wt * 256);     // first: the look-up wants it earliest
#pragma unroll
        for (int n = 0; n < 2 * A_LD; ++n)
            if (1 + n >= lo && 1 + n < hi) dma16(a_base[n >> 1], o[n & 1], sa + (n & 1) * kAHalf + (wt * A_LD + (n >> 1)) * 1024);
#pragma unroll
        for (int n = 0; n < B_LD; ++n)
            if (1 + 2 * A_LD + n >= lo && 1 + 2 * A_LD + n < hi) dma16(b_base[n], o[(wt * B_LD + n) / (BN / 16)], sb + (wt * B_LD + n) * 1024);
    };

    const int c0 = 2 * (lq & 1);
    const int b_off = kABytes + blk * kBHalf + (wn * WN + l16) * 64 + ((c0 ^ swz8(l16 >> 2)) << 4);
    // as in the bf16 kernel
    const int hb = l16 >> 3, col = l16 & 7, g0 = wm * (WM / 8) + hb;
    const uint32_t below[2] = {((1u << col) - 1u) << (8 * hb), ((1u << col) - 1u) << (8 * hb + 16)};
    const uint32_t bit[2] = {(uint32_t)(8 * hb + col), (uint32_t)(8 * hb + col + 16)};
    const uint32_t lb[2] = {(uint32_t)(blk * kAHalf + g0 * 256 + ((c0 ^ swz8(hb)) << 4)), (uint32_t)(blk * kAHalf + g0 * 256 + ((c0 ^ swz8(2 + hb)) << 4))};
    const uint32_t no_row = (uint32_t)(TL::kZero / 64 + zero_lane(l16) / 64 - g0 * 4);
    uint32_t a_off[FM], mk[FM / 2];
    auto lookup_read = [&](int stage) {
        const unsigned char* sc = ring + stage * kStage + kABytes + kBBytes + wt * 256 + wm * (WM / 8) + blk * 32;
        if constexpr (FM == 8) {
            const uint4 w = *reinterpret_cast<const uint4*>(sc);
            mk[0] = w.x; mk[1] = w.y; mk[FM / 2 - 2] = w.z; mk[FM / 2 - 1] = w.w;
        } else {
            const uint2 w = *reinterpret_cast<const uint2*>(sc);
            mk[0] = w.x; mk[1] = w.y;
        }
    };
    auto drop_second = [&](int kt) {             // kt: the step whose masks have been read
        if (2 * kt + 1 >= nblk) {
#pragma unroll
            for (int i = 0; i < FM / 2; ++i) mk[i] = blk ? 0u : mk[i];
        }
    };
    auto lookup = [&](int stage, int a) {
        const uint32_t kept = (uint32_t)__builtin_amdgcn_sbfe((int)mk[a >> 1], bit[a & 1], 1), row = (uint32_t)__builtin_popcount(mk[a >> 1] & below[a & 1]);
        a_off[a] = ((row & kept) | ((no_row - 8 * a) & ~kept)) * 64 + (lb[a & 1] + (uint32_t)(stage * kStage));
    };
    auto read_a = [&](Frag16& f, int a) {
        f.u[0] = *reinterpret_cast<const uint4*>(ring + a_off[a] + a * 512);
        f.u[1] = *reinterpret_cast<const uint4*>(ring + (a_off[a] ^ 16) + a * 512);
    };
    auto read_b = [&](Frag16& f, const unsigned char* st, int b) {
        f.u[0] = *reinterpret_cast<const uint4*>(st + b_off + b * 1024);
        f.u[1] = *reinterpret_cast<const uint4*>(st + (b_off ^ 16) + b * 1024);
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.0f;
    Frag16 A[2], B[FN];
    auto mma = [&](int a, int b) {
        acc[a][b] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[a & 1].q, B[b].q, acc[a][b], 0, 0, 0, 0x7F, 0, 0x7F);   // fp8 x fp8, scales 2^0
    };
#define SB() __builtin_amdgcn_sched_barrier(0)
    const int nk = (nblk + 1) / 2;                // 0 for an expert without tokens: its gradient is zero
    // The last steps load nothing (gemm_v2_body.hpp says why), except on the 256 tile, whose last tile is loaded again in their place: a second copy of its step, without loads, runs
    // out of registers (on codes T = N = 8192, F = 28672 1270 -> 1660 us).
    constexpr bool REPEAT = FM == 8;
    auto tile_of = [&](int t) { return REPEAT && t >= nk ? nk - 1 : t; };
    // (Nothing is in flight here, but the compiler, which does not see the ring's loads, may believe it of other units' loads to the same registers and wait in every step: as the
    // second unit of three, T = 3072, N = 448, F = 1792, the launch took 43 us, 25 without those waits.)
    wait_vmcnt<0>();
    if (nk > 0) {
        constexpr int ZW = TL::kZeros / 4;
        for (int i = wt * 64 + lane; i < kStages * 2 * ZW; i += TL::NW * 64)
            *reinterpret_cast<uint32_t*>(ring + i / (2 * ZW) * kStage + (i / ZW & 1) * kAHalf + TL::kZero + i % ZW * 4) = 0u;
#pragma unroll
        for (int p = 0; p < kStages; ++p)
            if (REPEAT || p < nk) issue(tile_of(p), p, 0, p < kStages - 1 ? kLoads : kLoads * 2 / 4);           // (the rest of the last one's loads are the first step's)
        if (REPEAT || nk >= kStages) wait_vmcnt<(kStages - 2) * kLoads + kLoads * 2 / 4>();
        else wait_vmcnt<0>();
        __syncthreads();
        lookup_read(0);
        drop_second(0);
#pragma unroll
        for (int a = 0; a < FM; ++a) lookup(0, a);
        read_a(A[0], 0);
        read_a(A[1], 1);
#pragma unroll
        for (int b = 0; b < FN; ++b) read_b(B[b], ring, b);
        int stage = 0;
        // One step = one stage = FM rows of four matrix instructions.  Behind the last but one the last reads of the stage have arrived (barrier): it is refilled, and the next one's
        // first fragments are read, G's each in the place of the one whose last instruction has been issued.  Its rows are looked up as the last ones of this stage have been read.
#define ISSUE(t, i) if (full.value || (t) < nk) issue(re_kt, re_stage, kLoads * (i) / 4, kLoads * ((i) + 1) / 4)
        int re_kt = tile_of(kStages - 1), re_stage = kStages - 1;
        auto step = [&](auto full, int kt) {
            const int next_stage = (stage + 1 == kStages) ? 0 : stage + 1;
            const unsigned char* sn = ring + next_stage * kStage;
#pragma unroll
            for (int a = 0; a < FM; ++a) {
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    mma(a, b);
                    if (a == FM - 1) { SB(); read_b(B[b], sn, b); SB(); }
                }
                SB();
                if (a + 2 < FM) { read_a(A[a & 1], a + 2); SB(); }
                if (a == 0) { ISSUE(kt + kStages - 1, 2); if (FM == 4) { ISSUE(kt + kStages - 1, 3); } SB(); }
                if (FM == 8 && a == 1) { ISSUE(kt + kStages - 1, 3); SB(); }
                if (a == FM - 4) {
                    // the next stage's masks were the first load of its batch: all but kLoads - 1 of that batch and the batch after it may still be in flight
                    if (full.value || kt + kStages - 1 < nk) wait_vmcnt<(kStages - 2) * kLoads + kLoads - 1>();
                    else wait_vmcnt<0>();
                    lookup_read(next_stage); SB();
                }
                if (a == FM - 3) {
                    drop_second(kt + 1);
#pragma unroll
                    for (int r = 0; r < FM; ++r) lookup(next_stage, r);
                    SB();
                }
                if (a == FM - 2) {
                    // this wavefront's reads of the stage are here, and its part of tile kt + 1
                    if (full.value || kt + kStages - 1 < nk) wait_vmcnt_lgkm0<(kStages - 2) * kLoads>();
                    else wait_vmcnt_lgkm0<0>();
                    __builtin_amdgcn_s_barrier();
                    SB();
                    re_kt = tile_of(kt + kStages); re_stage = stage;
                    read_a(A[0], 0); SB();
                    ISSUE(kt + kStages, 0); SB();
                }
                if (a == FM - 1) { read_a(A[1], 1); SB(); ISSUE(kt + kStages, 1); SB(); }
            }
            stage = next_stage;
        };
        int kt = 0;
        for (; kt < (REPEAT ? nk : nk - kStages); ++kt) step(Flag<true>(), kt);
        if constexpr (!REPEAT)
            for (; kt < nk; ++kt) step(Flag<false>(), kt);
#undef ISSUE
        wait_vmcnt<0>();
    }
#undef SB
    __syncthreads();
    wgrad_store<OUT_I_CONTIG, ACC32, TL>(acc, alpha, smem, wt, lane, i0, j0, F, N, out, ldo);
}

// The 64 tile on codes: one token block a stage and an instruction (v_mfma_scale_f32_32x32x64_f8f6f4, lane l: k 32 (l / 32) .. + 31 of row / column l % 32).  Few tiles and long
// contractions are bound by the chain of a step, not by power, and with two blocks a stage (156,672 bytes for 79,872) launches that hold such tiles run one workgroup a CU: fp8
// steps T = 3968, D = 384, F = 1152 50 us for 46.5, T = 13952, D = 512, F = 1792 154 for 143.  (One block a stage on the 16 x 16 x 128 instruction, half of it zeros: T = 4224,
// D = 256, F = 768 46 for 41.)  A's fragments are read one row ahead, G's one step ahead.
template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_vnm_fp8_shared_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ atc, const uint8_t* __restrict__ kmask,
                                                           const uint16_t* __restrict__ G, int F, int N, int Ttot, float alpha,
                                                           uint16_t* __restrict__ out, int64_t ldo, int tiles_m, int tiles_n, const GemmGroup& grp) {
    constexpr int BM = TL::BM, BN = TL::BN, FM = 2, FN = 2, KW = TL::KW;
    static_assert(KW == 4 && BM == 64 && BN == 64, "a 64 x 64 tile of four wavefronts");
    constexpr int kStages = TL::NST, kStage = TL::k8Stage, k8A = TL::k8A, k8B = TL::k8B, kLoads = TL::k8Loads, A_LD = TL::A_LD, B_LD = TL::B8_LD;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave;                          // share of the contraction
    const int l32 = lane & 31, lh = lane >> 5;
    unsigned char* const ring = smem + kg * (kStages * kStage);
    const uint32_t ring_lds = lds_addr(smem) + kg * (kStages * kStage);
    int L = xcd_run(pid, n_pid);
    int k_base = 0, K = Ttot;                     // grouped: every expert contracts over its own token segment
    if (grp.n) {
        const int per = tiles_m * tiles_n, e = uniform(L / per);
        L -= e * per;
        k_base = grp.seg[e];
        K = grp.seg[e + 1] - k_base;
        out += e * grp.out_stride * (ACC32 ? 2 : 1);          // (float32 elements are two uint16_t wide)
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, SFFN_TILE_GROUP, tm, tn);
    const int i0 = tm * BM, j0 = tn * BN;
    const int KC = Ttot / 64;                     // 64-token chunks (64 bytes) per row of the blocked operands

    uint64_t a_base[A_LD], b_base[B_LD], c_base;
    const int rb = lane >> 2;
    const uint32_t blk_lane = (uint32_t)(rb * 32 + ((lane & 3) ^ ((rb >> 2) & 3)) * 8) * 2;   // chunk swizzle, as in the bf16 kernel
    {
#pragma unroll
        for (int n = 0; n < A_LD; ++n) {
            int cr = i0 / 2 + n * 16; cr = cr < F / 2 ? cr : F / 2 - 16;
            a_base[n] = uniform64(atc + (((int64_t)(cr >> 4) * KC + k_base / 64) << 9));
        }
#pragma unroll
        for (int n = 0; n < B_LD; ++n) {
            int gr = j0 + n * 16; gr = gr < N ? gr : N - 16;
            b_base[n] = uniform64(G + (((int64_t)(gr >> 4) * KC + k_base / 64) << 9));
        }
        c_base = uniform64(kmask + (int64_t)(k_base / 64) * (F / 8));
    }
    uint32_t c_lane;
    {
        int g = i0 / 8 + 4 * (lane & 7); g = g < F / 8 ? g : F / 8 - 4;
        c_lane = (uint32_t)g;
    }
    const uint32_t c_kstep = (uint32_t)(F / 8);
    auto issue = [&](int kt, int stage, int lo, int hi) {
        const uint32_t sa = ring_lds + stage * kStage;
        const uint32_t o = blk_lane + (uint32_t)kt * 1024;
        if (lo <= 0 && hi > 0) dma4(c_base, c_lane + (uint32_t)kt * c_kstep, sa + k8A + k8B);     // first: the look-up wants it earliest
#pragma unroll
        for (int n = 0; n < A_LD; ++n)
            if (1 + n >= lo && 1 + n < hi) dma16(a_base[n], o, sa + n * 1024);
#pragma unroll
        for (int n = 0; n < B_LD; ++n)
            if (1 + A_LD + n >= lo && 1 + A_LD + n < hi) dma16(b_base[n], o, sa + k8A + n * 1024);
    };

    // fragment reads: a lane wants the 32 bytes k 32 lh .. + 31 of its row = 16-byte chunks 2 lh, 2 lh + 1 (slot = chunk ^ ((row >> 2) & 3))
    int b_off[FN];
#pragma unroll
    for (int b = 0; b < FN; ++b) {
        const int row = b * 32 + l32;
        b_off[b] = k8A + row * 64 + (((2 * lh) ^ ((row >> 2) & 3)) << 4);
    }
    int a_off[FM], a_next[FM];
    const uint32_t col = l32 & 7, below = (1u << col) - 1u;
    const int zero_row = TL::kZero + zero_lane(l32) + (((2 * lh) ^ (l32 >> 3)) << 4);
    uint32_t mk[FM];
    auto lookup_read = [&](int stage) {
        const unsigned char* sc = ring + stage * kStage + k8A + k8B;
#pragma unroll
        for (int a = 0; a < FM; ++a) mk[a] = sc[a * 4 + (l32 >> 3)];
    };
    auto lookup = [&](int stage) {
        const int sa = stage * kStage;
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            const int gl = a * 4 + (l32 >> 3);
            const int row = gl * 4 + __builtin_popcount(mk[a] & below);                   // (row >> 2) & 3 == l32 >> 3
            a_next[a] = sa + (((mk[a] >> col) & 1u) ? row * 64 + (((2 * lh) ^ (l32 >> 3)) << 4) : zero_row);
        }
    };
    auto read_a = [&](Frag16& f, int off) {
        f.u[0] = *reinterpret_cast<const uint4*>(ring + off);
        f.u[1] = *reinterpret_cast<const uint4*>(ring + (off ^ 16));
    };
    auto read_b = [&](Frag16& f, const unsigned char* st, int b) {
        f.u[0] = *reinterpret_cast<const uint4*>(st + b_off[b]);
        f.u[1] = *reinterpret_cast<const uint4*>(st + (b_off[b] ^ 16));
    };
    f32x16 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    auto mma_row = [&](const Frag16& fa, const Frag16 (&fb)[FN], int a) {
#pragma unroll
        for (int b = 0; b < FN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa.q, fb[b].q, acc[a][b], 0, 0, 0, 0x7F, 0, 0x7F);   // fp8 x fp8, scales 2^0
    };
#define SB() __builtin_amdgcn_sched_barrier(0)
    const int nk = (K / 64 - kg + KW - 1) / KW;                // 0 for an expert without tokens: its gradient is zero
    auto step_of = [&](int kt) { return kg + kt * KW; };
    wait_vmcnt<0>();                              // (see the bf16 kernel)
    if (nk > 0) {
        constexpr int ZW = TL::kZeros / 4;
        for (int i = lane; i < kStages * ZW; i += 64) *reinterpret_cast<uint32_t*>(ring + i / ZW * kStage + TL::kZero + i % ZW * 4) = 0u;   // the rows of zeros
#pragma unroll
        for (int p = 0; p < kStages; ++p) issue(step_of(p < nk ? p : nk - 1), p, 0, kLoads);
        wait_vmcnt<(kStages - 1) * kLoads>();
        wave_lds_sync();
        asm volatile("" ::: "memory");
        Frag16 A0, A1, B0[FN], B1[FN];
        lookup_read(0);
        lookup(0);
#pragma unroll
        for (int a = 0; a < FM; ++a) a_off[a] = a_next[a];
        read_a(A0, a_off[0]);
#pragma unroll
        for (int b = 0; b < FN; ++b) read_b(B0[b], ring, b);
        int stage = 0;
        // One step = one token block; two steps per loop trip so that the two G fragment sets alternate by name.
        int re_kt = step_of(kStages - 1 < nk ? kStages - 1 : nk - 1), re_stage = kStages - 1;
#define ISSUE(i) issue(re_kt, re_stage, kLoads * (i) / 2, kLoads * ((i) + 1) / 2)
        auto step = [&](int kt, Frag16 (&Bc)[FN], Frag16 (&Bn)[FN]) {
            const int next_stage = (stage + 1 == kStages) ? 0 : stage + 1;
            const unsigned char* sn = ring + next_stage * kStage;
            read_a(A1, a_off[1]); SB();
            // the next block's mask bytes were the first load of its batch
            wait_vmcnt<(kStages - 2) * kLoads + kLoads - 1>();
            asm volatile("" ::: "memory");
            lookup_read(next_stage); SB();
            mma_row(A0, Bc, 0); SB();
            wait_vmcnt_lgkm0<(kStages - 2) * kLoads>();      // my reads of this stage are done, block kt + 1 has landed (this wavefront's part)
            asm volatile("" ::: "memory");
            SB();
            re_kt = step_of((kt + kStages < nk) ? kt + kStages : nk - 1); re_stage = stage;
            ISSUE(0); SB();
            lookup(next_stage); SB();
#pragma unroll
            for (int a = 0; a < FM; ++a) a_off[a] = a_next[a];
            read_a(A0, a_off[0]);
#pragma unroll
            for (int b = 0; b < FN; ++b) read_b(Bn[b], sn, b);
            SB();
            mma_row(A1, Bc, 1); SB();
            ISSUE(1); SB();
            stage = next_stage;
        };
        int kt = 0;
        for (; kt + 1 < nk; kt += 2) { step(kt, B0, B1); step(kt + 1, B1, B0); }
        if (kt < nk) step(kt, B0, B1);
#undef ISSUE
        wait_vmcnt<0>();
    }
#undef SB
    __syncthreads();
    if (!wgrad_join<TL>(acc, smem, kg, lane)) return;
    // four rows of a column at a time to the lanes that wgrad_store expects them in
    f32x4* const quad = reinterpret_cast<f32x4*>(smem);          // [row / 4][column]
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                quad[(8 * a + 2 * g + lh) * 64 + 32 * b + l32] = f32x4{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
    wave_lds_sync();
    f32x4 sum[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) sum[a][b] = quad[(4 * a + (lane >> 4)) * 64 + 16 * b + (lane & 15)];
    wave_lds_sync();
    wgrad_store<OUT_I_CONTIG, ACC32, TL>(sum, alpha, smem, 0, lane, i0, j0, F, N, out, ldo);
}

template <bool FP8, bool OUT_I_CONTIG, bool ACC32, class TL>
struct WgradUnit {
    using Args = WgradArgs;
    static constexpr int THREADS = TL::THREADS, LDS = FP8 ? TL::BYTES8 : TL::BYTES;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        if constexpr (FP8 && TL::KW > 1) wgrad_vnm_fp8_shared_body<OUT_I_CONTIG, ACC32, TL>(smem, pid, n_pid, a.atc, a.kmask, a.G, a.F, a.N, a.T, a.alpha, a.out, a.ldo, a.tiles_m, a.tiles_n, a.grp);
        else if constexpr (FP8) wgrad_vnm_fp8_body<OUT_I_CONTIG, ACC32, TL>(smem, pid, n_pid, a.atc, a.kmask, a.G, a.F, a.N, a.T, a.alpha, a.out, a.ldo, a.tiles_m, a.tiles_n, a.grp);
        else               wgrad_vnm_body<OUT_I_CONTIG, ACC32, TL>(smem, pid, n_pid, a.atc, a.kmask, a.G, a.F, a.N, a.T, a.out, a.ldo, a.tiles_m, a.tiles_n, a.grp);
    }
    static unsigned count(const Args& a) { return (unsigned)((a.F + TL::BM - 1) / TL::BM * ((a.N + TL::BN - 1) / TL::BN) * (a.grp.n ? a.grp.n : 1)); }
    static int stages(const Args& a) { return a.T / (FP8 && TL::KW == 1 ? 128 : 64) / (TL::KW * (a.grp.n ? a.grp.n : 1)); }      // of a tile, a wavefront's, on average (wgrad_first)
    static Args args(Args a) { a.tiles_m = (a.F + TL::BM - 1) / TL::BM; a.tiles_n = (a.N + TL::BN - 1) / TL::BN; return a; }
};
template <bool FP8, bool OUT_I_CONTIG, bool ACC32> using WgradUnit256 = WgradUnit<FP8, OUT_I_CONTIG, ACC32, WTile<2, 4, 128, 3, 1>>;
template <bool FP8, bool OUT_I_CONTIG, bool ACC32> using WgradUnitTall = WgradUnit<FP8, OUT_I_CONTIG, ACC32, WTile<2, 2, 128, 2, 1>>;      // 256 hidden units x 128 columns
template <bool FP8, bool OUT_I_CONTIG, bool ACC32> using WgradUnit128 = WgradUnit<FP8, OUT_I_CONTIG, ACC32, WTile<2, 2, 64, 3, 1>>;
template <bool FP8, bool OUT_I_CONTIG, bool ACC32> using WgradUnit64 = WgradUnit<FP8, OUT_I_CONTIG, ACC32, WTile<1, 1, 64, 3, 4>>;

}  // namespace sffn
