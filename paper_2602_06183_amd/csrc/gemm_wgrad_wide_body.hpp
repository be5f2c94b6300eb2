// Weight-gradient contractions for blocks of M = 32, 64 columns (Table 5): C[f, n] = sum_t A[t, f] * G[t, n] as in gemm_wgrad_body.hpp, but a
// block of M hidden units keeps only 4 of them in a 64-token block, so the 256-row tile of that kernel multiplies mostly rows of zeros: at
// T = F = 16384, N = 4096, M = 32 it issued 8 times the products the format has.
//
// Here the matrix instructions run on the kept rows only, 32 of them (8 blocks x 4) at a time, and which hidden units these are changes with every
// token block.  The output tile therefore lives in LDS as float32: for every token block a wavefront reads the tile rows of its 32 kept hidden units
// into the accumulator of four v_mfma_f32_32x32x16_bf16 (64 tokens), and writes the result back.  Every element is still summed over the tokens in
// ascending order in one float32 chain, exactly as when the rows of zeros are multiplied too.  The operands go straight from L2 to registers, four to six
// token blocks ahead (no wavefront reads what another one has loaded into LDS, so LDS would only be a detour).
//   The columns of G are the rows of the instruction and the kept hidden units its columns: a lane then owns one hidden unit and 4 times 4 neighbouring
//   columns, four 16-byte LDS accesses and one kept offset per token block.  (The other way round it owned 16 hidden units: 32 LDS instructions of 4 bytes and
//   32 instructions for their addresses, all issued by one wavefront per SIMD.)  With that, loads of 32 columns more per wavefront at M = 32, and more
//   wavefronts than the main loop has work for, which clear the tile and store it: T = F = 16384, N = 4096: M = 32 830 -> 675 us, M = 64 600 -> 450;
//   T = 4096, N = 2048, F = 8192 60 -> 48 and 53 -> 38; 64 tokens 12 - 19 -> 7.
//   Bound now: M = 64, two wavefronts: the chain load - multiply - write - read (its last instruction, 4 + 4 LDS instructions and 9 loads of 1 KB, 16 clocks
//   each, come after one another); M = 32: the loads, 24 KB per token block at 64 bytes per clock and CU = 400 of about 700 clocks, and what two wavefronts can issue.
//   M = 32 with 32 columns per wavefront (four of them, 32 KB of loads): 775 us; M = 64 with 64 columns (one wavefront): 500.  Four token blocks ahead at M = 32: 7 % slower,
//   eight: the same; M = 64, six: the same.  Loads between the matrix instructions: M = 64 up to 6 % slower, M = 32 (64 columns) 4 % faster.  A barrier per token block, so
//   that wavefronts meet the same lines in L1: 15 % slower.  Kept rows through an LDS ring on 256 x 128 tiles (20 KB of loads per token block): slower, every
//   token block then has a barrier.  Kept rows at the lanes 8 (block / 2) + ... (128 bytes of `at` per 8 lanes): 785 and 530 us, 8 lanes of an LDS write then meet in 2 blocks' banks.
//   At M = 16 this form took 1150 us and 73 at T = 4096, N = 2048, F = 8192 (gemm_wgrad_body.hpp 1330 and 82): not built.
//
// A comes from the V:N:M epilogues (gemm_v2_body.hpp, VnmEpilogue::at_kept) in the order of the instruction's lanes:
//   [T / 64][R / 32][4 steps of 16 tokens][64 lanes][8 tokens], R = 4 F / M kept rows, lane = 32 (token / 8 % 2) + kept_lane(row) (kept_off in common.hpp)
// colidx = the kept column offsets of the packed activation, [T / 64][F / M][4] bytes: a lane's is one of them.
// G is the transposed operand [N, T] in the same order ([T / 64][N / 32][4][64][8], lane_off in common.hpp): every load of a wavefront is 1 KB
// of consecutive bytes.  (From the blocked layout, whose 16-byte pieces lie 64 bytes apart, the loads alone took 1240 clocks per token block.)
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "lds_dma.hpp"

namespace sffn {

template <int N> struct Num { static constexpr int value = N; };
// BF hidden units x BN columns; WR x WN wavefronts, each 32 kept rows x 32 NC columns, in the main loop, DEPTH token blocks ahead; the others of the
// workgroup's four only clear the tile and store it
template <int LOGM_, int BF_, int BN_, int NC_, int DEPTH_>
struct WideTile {
    static constexpr int LOGM = LOGM_, M = 1 << LOGM, BF = BF_, BN = BN_, NC = NC_, DEPTH = DEPTH_;
    static constexpr int WR = 4 * BF / M / 32, WN = BN / 32 / NC, NW = WR * WN, THREADS = 256;
    static constexpr int LDS = BF * BN * 4, LINE = BN * 32;        // bytes of one row of each of 8 blocks
    static_assert(4 * BF / M % 32 == 0 && (BN == 64 || BN == 32) && BN % (32 * NC) == 0 && NW <= 4 && DEPTH % 2 == 0, "whole pieces; two sets of addresses alternate");
    // Byte address of (hidden unit, column): 8 columns (a chunk) of the same row of 8 neighbouring blocks make 256 bytes, all 64 banks, so kept rows of different
    // blocks never meet.  The blocks' order changes with the chunk, so that the chunks of one row do not meet either when the tile is stored.
    static __device__ __forceinline__ int slot(int block, int chunk) { return chunk * 256 + ((block ^ chunk) & 7) * 32; }
    static __device__ __forceinline__ int at(int row, int col) {
        return (row >> (LOGM + 3)) * (M * LINE) + (row & (M - 1)) * LINE + slot(row >> LOGM, col >> 3) + (col & 7) * 4;
    }
};

template <bool OUT_I_CONTIG, bool ACC32, class TL>
__device__ __forceinline__ void wgrad_wide_body(unsigned char* __restrict__ smem, int pid, int n_pid, const uint16_t* __restrict__ at, const uint8_t* __restrict__ colidx,
                                                const uint16_t* __restrict__ G, int F, int N, int Ttot, uint16_t* __restrict__ out, int64_t ldo, int tiles_m, int tiles_n,
                                                const GemmGroup& grp) {
    constexpr int M = TL::M, LOGM = TL::LOGM, BF = TL::BF, BN = TL::BN, NC = TL::NC, DEPTH = TL::DEPTH;
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

    // ---- operands of this wavefront.  Pieces past the matrix edge are clamped into it: they only feed outputs that are not stored. -------------
    const int R32 = F >> (LOGM + 3);              // groups of 32 kept rows = of 8 blocks
    int rg = i0 / (8 * M) + wr;
    rg = rg < R32 ? rg : R32 - 1;
    // (wave-uniform bases: 4 KB per token block and piece, 32 bytes of offsets; the lane's part is 16 bytes of each KB)
    const uint64_t a_base = uniform64(at + ((int64_t)tb0 * R32 + rg) * 2048);
    const int N32 = N / 32;
    uint64_t b_base[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int ng = j0 / 32 + wn * NC + c;
        b_base[c] = uniform64(G + ((int64_t)tb0 * N32 + (ng < N32 ? ng : N32 - 1)) * 2048);
    }
    const uint64_t c_base = uniform64(colidx + ((int64_t)tb0 * R32 + rg) * 32);
    const uint32_t a_step = (uint32_t)R32 * 4096, b_step = (uint32_t)N32 * 4096, c_step = (uint32_t)R32 * 32;
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) u4 glb_u4;
    auto to_uint4 = [](u4 v) { return make_uint4(v.x, v.y, v.z, v.w); };
    struct Stage { Frag8 a[4], b[NC][4]; uint32_t c; };
    const int block = l32 & 7;                    // the lane's kept hidden unit (kept_lane): block and, l32 / 8, position among its four
    const uint32_t c_lane = block * 4 + (l32 >> 3);
    auto at_block = [&](uint64_t base, int kt, uint32_t step) { return base + (uint64_t)(uint32_t)(kt < nk ? kt : nk - 1) * step; };
    auto load_a = [&](Stage& st, int kt) {
        const glb_u4* p = (const glb_u4*)at_block(a_base, kt, a_step);
#pragma unroll
        for (int s = 0; s < 4; ++s) st.a[s].u = to_uint4(p[lane + s * 64]);
    };
    auto load_b = [&](Stage& st, int kt, int c) {
        const glb_u4* p = (const glb_u4*)at_block(b_base[c], kt, b_step);
#pragma unroll
        for (int s = 0; s < 4; ++s) st.b[c][s].u = to_uint4(p[lane + s * 64]);
    };
    auto load_c = [&](Stage& st, int kt) { st.c = ((const __attribute__((address_space(1))) uint8_t*)at_block(c_base, kt, c_step))[c_lane]; };

    // LDS address of the lane's accumulator registers 4 g .. 4 g + 3: columns 8 g + 4 lh + 0..3 of its hidden unit
    uint32_t base[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) base[c][g] = lds_addr(smem) + wr * (M * TL::LINE) + TL::slot(block, (wn * NC + c) * 4 + g) + lh * 16;
    // (of two token blocks: the next one's are worked out while the matrix instructions of this one run)
    struct Addr { uint32_t p[NC][4]; } addr[2];
    auto look_up = [&](Addr& to, const Stage& st) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g) to.p[c][g] = st.c * TL::LINE + base[c][g];
    };
    f32x16 acc[NC];
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) f4 lds_f4;
    auto rd = [&](int c, const Addr& ad) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f4 v = *(const lds_f4*)ad.p[c][g];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[c][4 * g + r] = v[r];
        }
    };
    auto wrb = [&](int c, const Addr& ad) {
#pragma unroll
        for (int g = 0; g < 4; ++g) *(lds_f4*)ad.p[c][g] = (f4){acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
    };
#define SB() __builtin_amdgcn_sched_barrier(0)
#define MM(c, s) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.b[c][s].v, cur.a[s].v, acc[c], 0, 0, 0); SB()
    auto clear = [&]() {
        for (int i = tid; i < BF * BN / 4; i += TL::THREADS) reinterpret_cast<float4*>(smem)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the first loads stay in flight)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if (nk > 0 && wave < TL::NW) {
        Stage st[DEPTH];
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) {
            load_c(st[p], p);
            load_b(st[p], p, 0);
            if (NC == 1 || p < DEPTH - 1) {
                load_a(st[p], p);
                if (NC == 2) load_b(st[p], p, NC - 1);
            }
        }
        clear();
        look_up(addr[0], st[0]);
        look_up(addr[1], st[0]);
#pragma unroll
        for (int c = 0; c < NC; ++c) rd(c, addr[0]);
        // (past the last block: the rows of a block that is loaded again, read and not used)
        auto block_of = [&](int kt, Stage& prv, Stage& cur, Stage& nxt, Addr& here, Addr& next) {
            if constexpr (NC == 1) {
                MM(0, 0);
                look_up(next, nxt); SB();
                MM(0, 1); MM(0, 2); MM(0, 3);
                wrb(0, here); SB();
                rd(0, next); SB();
                load_c(cur, kt + DEPTH); load_a(cur, kt + DEPTH); load_b(cur, kt + DEPTH, 0); SB();
            } else {
                // the two halves take turns: while one is multiplied the other's result goes back and its next rows come.  `next` still holds the
                // addresses of the token block before (at the first one, the same as `here`).  The stage that the token block before has
                // used is refilled in this one, but for what its second half did not read.
                MM(0, 0);
                wrb(NC - 1, next); SB();
                MM(0, 1);
                rd(NC - 1, here); SB();
                MM(0, 2);
                load_a(prv, kt + DEPTH - 1); SB();
                MM(0, 3);
                load_b(prv, kt + DEPTH - 1, NC - 1); SB();
                look_up(next, nxt); SB();
                MM(NC - 1, 0);
                wrb(0, here); SB();
                MM(NC - 1, 1);
                rd(0, next); SB();
                MM(NC - 1, 2);
                load_b(cur, kt + DEPTH, 0); SB();
                MM(NC - 1, 3);
                load_c(cur, kt + DEPTH); SB();
            }
        };
        int kt = 0;
        for (; kt + DEPTH <= nk; kt += DEPTH) {
#pragma unroll
            for (int p = 0; p < DEPTH; ++p) block_of(kt + p, st[(p + DEPTH - 1) % DEPTH], st[p], st[(p + 1) % DEPTH], addr[p & 1], addr[(p + 1) & 1]);
        }
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p)
            if (kt + p < nk) block_of(kt + p, st[(p + DEPTH - 1) % DEPTH], st[p], st[(p + 1) % DEPTH], addr[p & 1], addr[(p + 1) & 1]);
        if constexpr (NC == 2) {
            if (nk & 1) wrb(1, addr[0]);
            else wrb(1, addr[1]);
        }
    } else clear();
#undef MM
#undef SB
    __syncthreads();

    // ---- output: 16 bytes per lane, rows of the contiguous axis ------------------------------------------------------------------------------
    constexpr int EPL = ACC32 ? 4 : 8;            // elements per lane and store
    // NS runs of EPL elements; float32 sums: what they are added to is read first
    auto put = [&](int64_t o, int64_t step, auto& v, auto ns) {
        constexpr int NS = decltype(ns)::value;
        if constexpr (ACC32) {
            float4* p[NS];
            float4 old[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j) { p[j] = reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + o + j * step); old[j] = *p[j]; }
#pragma unroll
            for (int j = 0; j < NS; ++j) store_out(p[j], make_float4(old[j].x + v[j][0], old[j].y + v[j][1], old[j].z + v[j][2], old[j].w + v[j][3]));
        } else
#pragma unroll
            for (int j = 0; j < NS; ++j)
                store_out(out + o + j * step, make_uint4(f2bf2(v[j][0], v[j][1]), f2bf2(v[j][2], v[j][3]), f2bf2(v[j][4], v[j][5]), f2bf2(v[j][6], v[j][7])));
    };
    auto get4 = [&](int row, int col) { return *reinterpret_cast<const float4*>(smem + TL::at(row, col)); };
    if constexpr (OUT_I_CONTIG) {
        // a lane: EPL hidden units x 4 columns, eight lanes 8 chunks of columns
        constexpr int CH = BN / 8, FC = BF / EPL;
        static_assert(BF * BN % (4 * EPL * TL::THREADS) == 0, "whole rounds");
        for (int i = tid; i < BF * BN / (4 * EPL); i += TL::THREADS) {
            const int ch = i % CH, fc = i / CH % FC, half = i / (CH * FC);
            const int f = fc * EPL, n = ch * 8 + half * 4;
            float v[4][EPL];
#pragma unroll
            for (int q = 0; q < EPL; ++q) {
                const float4 x = get4(f + q, n);
                v[0][q] = x.x; v[1][q] = x.y; v[2][q] = x.z; v[3][q] = x.w;
            }
            if (i0 + f < F && j0 + n < N) put((int64_t)(j0 + n) * ldo + i0 + f, ldo, v, Num<4>());
        }
    } else {
        constexpr int C = BN / EPL;
        constexpr int RW = TL::THREADS / C;       // rows of one round; a lane takes four of them
        static_assert(TL::THREADS % C == 0 && BF % (4 * RW) == 0, "whole rounds");
        for (int f = tid / C; f < BF; f += 4 * RW) {
            const int n = tid % C * EPL;
            if (j0 + n >= N) break;
            float v[4][EPL];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < EPL; q += 4) {
                    const float4 x = get4(f + j * RW, n + q);
                    v[j][q] = x.x; v[j][q + 1] = x.y; v[j][q + 2] = x.z; v[j][q + 3] = x.w;
                }
            if (i0 + f + 3 * RW < F) put((int64_t)(i0 + f) * ldo + j0 + n, (int64_t)RW * ldo, v, Num<4>());
            else
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i0 + f + j * RW < F) {
                        float w[1][EPL];
#pragma unroll
                        for (int q = 0; q < EPL; ++q) w[0][q] = v[j][q];
                        put((int64_t)(i0 + f + j * RW) * ldo + j0 + n, 0, w, Num<1>());
                    }
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
