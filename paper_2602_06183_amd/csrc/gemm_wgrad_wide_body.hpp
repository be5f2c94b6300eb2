// Weight-gradient contractions for blocks of M = 32, 64 columns (Table 5): C[f, n] = sum_t A[t, f] * G[t, n] as in gemm_wgrad_body.hpp, but a
// block of M hidden units keeps only 4 of them in a 64-token block, so the 256-row tile of that kernel multiplies mostly rows of zeros: at
// T = F = 16384, N = 4096, M = 32 it issued 8 times the products the format has.
//
// Here the matrix instructions run on the kept rows only, 32 of them (8 blocks x 4) at a time, and which hidden units these are changes with every
// token block.  The output tile therefore lives in LDS as float32: for every token block a wavefront reads the tile rows of its 32 kept hidden units
// into the accumulator of four v_mfma_f32_32x32x16_bf16 (64 tokens), and writes the result back.  Every element is still summed over the tokens in
// ascending order in one float32 chain, exactly as when the rows of zeros are multiplied too.  The operands go straight from L2 to registers, four
// token blocks ahead (no wavefront reads what another one has loaded into LDS, so LDS would only be a detour).
//   Bound: the chain load - multiply - write - read of one wavefront per SIMD and the vector loads (1 KB each, 16 clocks of the CU's 64 bytes per clock: 576
//   of about 830 clocks per token block at M = 32); 128 KB of LDS is all the tile there can be.  T = F = 16384, N = 4096: 1390 us with the
//   rows of zeros, 815 us at M = 32.  The next token block's LDS addresses are worked out between the matrix instructions of this one: M = 64 (two wavefronts)
//   690 -> 606 us; T = 4096, N = 2048, F = 8192 58 -> 51; M = 32, bound by the loads, 817 -> 815.
//   Kept rows through an LDS ring on 256 x 128 tiles (20 KB of loads per token block instead of 32): 8 % slower, every token block then has a barrier; loads
//   between the matrix instructions: M = 64 6 % slower; 6 or 8 token blocks ahead: the same.
//   At M = 16 the same form took 1300 us, and 103 instead of 94 at T = 4096, N = 2048, F = 8192 (twice the kept rows, the same bytes from L2 as the dense
//   form), so M = 16 stays with gemm_wgrad_body.hpp.
//
// A comes from the V:N:M epilogues (gemm_v2_body.hpp, VnmEpilogue::at_kept) in the order of the instruction's lanes:
//   [T / 64][R / 32][4 steps of 16 tokens][64 lanes][8 tokens], R = 4 F / M kept rows, lane = 32 (token / 8 % 2) + row % 32
// cixl = the kept column offsets as the lanes want them: [T / 64][F / (8 M)][2][4] words, word (h, g) = the four offsets of block 2 g + h of 8.
// G is the transposed operand [N, T] in the same order ([T / 64][N / 32][4][64][8], lane_off in common.hpp): every load of a wavefront is 1 KB
// of consecutive bytes.  (From the blocked layout, whose 16-byte pieces lie 64 bytes apart, the loads alone took 1240 clocks per token block.)
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"

namespace sffn {

// BF hidden units x BN columns; WR x WN wavefronts, each 32 kept rows x 32 columns
template <int LOGM_, int BF_, int BN_>
struct WideTile {
    static constexpr int LOGM = LOGM_, M = 1 << LOGM, BF = BF_, BN = BN_;
    static constexpr int WR = 4 * BF / M / 32, WN = BN / 32, NW = WR * WN, THREADS = 64 * NW;
    static constexpr int PITCH = BN + 1;                 // floats; odd, so that columns can be read as well as rows
    static constexpr int LDS = BF * PITCH * 4;
    static_assert(4 * BF / M % 32 == 0 && BN % 32 == 0, "whole pieces");
};

template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_wide_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ at, const uint8_t* __restrict__ cixl,
                                                const uint16_t* __restrict__ G, int F, int N, int Ttot, uint16_t* __restrict__ out, int64_t ldo, int tiles_m, int tiles_n,
                                                const GemmGroup& grp) {
    constexpr int M = TL::M, LOGM = TL::LOGM, BF = TL::BF, BN = TL::BN, PITCH = TL::PITCH, DEPTH = 4;
    float* const tile = reinterpret_cast<float*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / TL::WN, wn = wave % TL::WN;
    const int l32 = lane & 31, lh = lane >> 5;

    int L = xcd_run(pid, n_pid);
    int tb0 = 0, nk = Ttot / 64;                  // grouped: every expert contracts over its own token segment
    if (grp.n) {
        const int per = tiles_m * tiles_n, e = uniform(L / per);
        L -= e * per;
        tb0 = grp.seg[e] / 64;
        nk = grp.seg[e + 1] / 64 - tb0;
        out += e * grp.out_stride * (ACC32 ? 2 : 1);
    }
    int tm, tn;
    band_tile(L, tiles_m, tiles_n, 4, tm, tn);
    const int i0 = tm * BF, j0 = tn * BN;

    static_assert(BF * PITCH % 4 == 0, "cleared in 16-byte pieces");
    for (int i = tid; i < BF * PITCH / 4; i += TL::THREADS) reinterpret_cast<float4*>(tile)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();

    // ---- operands of this wavefront.  Pieces past the matrix edge are clamped into it: they only feed outputs that are not stored. -------------
    const int R32 = F >> (LOGM + 3);              // groups of 32 kept rows = of 8 blocks
    int rg = i0 / (8 * M) + wr;
    rg = rg < R32 ? rg : R32 - 1;
    // (wave-uniform bases: 4 KB per token block and piece, 32 bytes of offsets; the lane's part is 16 bytes of each KB)
    const uint64_t a_base = uniform64(at + ((int64_t)tb0 * R32 + rg) * 2048);
    const int N32 = N / 32;
    int ng = j0 / 32 + wn;
    ng = ng < N32 ? ng : N32 - 1;
    const uint64_t b_base = uniform64(G + ((int64_t)tb0 * N32 + ng) * 2048);
    const uint64_t c_base = uniform64(cixl + ((int64_t)tb0 * R32 + rg) * 32);
    const uint64_t a_step = (uint64_t)R32 * 4096, b_step = (uint64_t)N32 * 4096, c_step = (uint64_t)R32 * 32;
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) u4 glb_u4;
    auto to_uint4 = [](u4 v) { return make_uint4(v.x, v.y, v.z, v.w); };
    struct Stage { Frag8 a[4], b[4]; uint4 c; };
    auto load = [&](Stage& st, int kt) {
        const uint64_t k = (uint64_t)(kt < nk ? kt : nk - 1);
        st.c = to_uint4(((const glb_u4*)(c_base + k * c_step))[lh]);
        const glb_u4* pa = (const glb_u4*)(a_base + k * a_step);
#pragma unroll
        for (int s = 0; s < 4; ++s) st.a[s].u = to_uint4(pa[lane + s * 64]);
        const glb_u4* pb = (const glb_u4*)(b_base + k * b_step);
#pragma unroll
        for (int s = 0; s < 4; ++s) st.b[s].u = to_uint4(pb[lane + s * 64]);
    };

    // LDS byte address of accumulator register r: kept row 8 (r / 4) + 4 lh + r % 4 = column offset r % 4 of block 2 (r / 4) + lh
    const uint32_t base = (uint32_t)((wr * 8 + lh) * M * PITCH + wn * 32 + l32) * 4;
    // (of two token blocks: the next one's are worked out while the matrix instructions of this one run)
    uint32_t addr[2][16];
    auto look_up = [&](uint32_t (&to)[16], const Stage& st, int g) {
        const uint32_t c = g == 0 ? st.c.x : g == 1 ? st.c.y : g == 2 ? st.c.z : st.c.w;
#pragma unroll
        for (int r = 0; r < 4; ++r) to[4 * g + r] = __umul24((c >> (8 * r)) & 0xFFu, PITCH * 4) + (base + g * (2 * M * PITCH * 4));
    };
    f32x16 acc;
    auto rd = [&](const uint32_t (&at_)[16]) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = *reinterpret_cast<float*>(smem + at_[r]);
    };
    auto wrb = [&](const uint32_t (&at_)[16]) {
#pragma unroll
        for (int r = 0; r < 16; ++r) *reinterpret_cast<float*>(smem + at_[r]) = acc[r];
    };
#define SB() __builtin_amdgcn_sched_barrier(0)
    if (nk > 0) {
        Stage st[DEPTH];
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) load(st[p], p);
#pragma unroll
        for (int g = 0; g < 4; ++g) look_up(addr[0], st[0], g);
        rd(addr[0]);
        auto block = [&](int kt, Stage& cur, Stage& nxt, uint32_t (&here)[16], uint32_t (&next)[16]) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[s].v, cur.b[s].v, acc, 0, 0, 0); SB();
                look_up(next, nxt, s); SB();           // (past the last block: the rows of a block that is loaded again, read and not used)
            }
            wrb(here); SB();
            rd(next); SB();
            load(cur, kt + DEPTH); SB();
        };
        int kt = 0;
        static_assert(DEPTH % 2 == 0, "the two sets of addresses alternate");
        for (; kt + DEPTH <= nk; kt += DEPTH) {
#pragma unroll
            for (int p = 0; p < DEPTH; ++p) block(kt + p, st[p], st[(p + 1) % DEPTH], addr[p & 1], addr[(p + 1) & 1]);
        }
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p)
            if (kt + p < nk) block(kt + p, st[p], st[(p + 1) % DEPTH], addr[p & 1], addr[(p + 1) & 1]);
    }
#undef SB
    __syncthreads();

    // ---- output: 16 bytes per lane, rows of the contiguous axis ------------------------------------------------------------------------------
    constexpr int EPL = ACC32 ? 4 : 8;            // elements per lane and store
    constexpr int C = (OUT_I_CONTIG ? BF : BN) / EPL, RWS = OUT_I_CONTIG ? BN : BF;
    // four chunks at a time: with one or two wavefronts per CU the LDS reads of a single one would be waited for each time
    static_assert(C * RWS % (4 * TL::THREADS) == 0, "whole rounds");
    for (int i0c = tid; i0c < C * RWS; i0c += 4 * TL::THREADS) {
        float v[4][EPL];
        float4 old[4];
        int64_t o[4];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // contiguous along f: 8 lanes cover 8 chunks of a column and the next ones the next columns, 64 different LDS banks
            const int i = i0c + u * TL::THREADS, j = i >> 6;
            const int c = OUT_I_CONTIG ? (j % (C / 8) * 8 + (i & 7)) * EPL : (i % C) * EPL;
            const int r = OUT_I_CONTIG ? j / (C / 8) * 8 + (i >> 3) % 8 : i / C;
            const int f = i0 + (OUT_I_CONTIG ? c : r), n = j0 + (OUT_I_CONTIG ? r : c);
            ok[u] = f < F && n < N;               // (F, N and the chunks are multiples of 8: whole chunks)
            o[u] = OUT_I_CONTIG ? (int64_t)n * ldo + f : (int64_t)f * ldo + n;
#pragma unroll
            for (int q = 0; q < EPL; ++q) v[u][q] = OUT_I_CONTIG ? tile[(c + q) * PITCH + r] : tile[r * PITCH + c + q];
            if (ACC32 && ok[u]) old[u] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(out) + o[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!ok[u]) continue;
            if constexpr (ACC32)
                *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + o[u]) = make_float4(old[u].x + v[u][0], old[u].y + v[u][1], old[u].z + v[u][2], old[u].w + v[u][3]);
            else
                *reinterpret_cast<uint4*>(out + o[u]) = make_uint4(f2bf2(v[u][0], v[u][1]), f2bf2(v[u][2], v[u][3]), f2bf2(v[u][4], v[u][5]), f2bf2(v[u][6], v[u][7]));
        }
    }
}

template <bool OUT_I_CONTIG, bool ACC32, class TL>
struct WgradWideUnit {
    using Args = WgradArgs;
    static constexpr int THREADS = TL::THREADS, LDS = TL::LDS;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int n_pid, const Args& a) {
        wgrad_wide_body<OUT_I_CONTIG, ACC32, TL>(smem, pid, n_pid, a.atc, a.kmask, a.G, a.F, a.N, a.T, a.out, a.ldo, a.tiles_m, a.tiles_n, a.grp);
    }
    static unsigned count(const Args& a) { return (unsigned)((a.F + TL::BF - 1) / TL::BF * ((a.N + TL::BN - 1) / TL::BN) * (a.grp.n ? a.grp.n : 1)); }
    static Args args(Args a) { a.tiles_m = (a.F + TL::BF - 1) / TL::BF; a.tiles_n = (a.N + TL::BN - 1) / TL::BN; return a; }
};

}  // namespace sffn
