// Neuron-level router of Section 3.3 / Alg. 3, steps 1 and 2 of the conversion listed in Section 3.4, and the small
// data-movement kernels of step 3:
//   route:   s[t, e] = x[t] . mean[e] (float32, fixed summation order), expert[t] = argmax_e (ties to the lower e)
//   permute: stable grouping of the tokens by expert, every run padded to 64 rows (perm, row_of_token, seg)
//   gather:  X rows in permuted order, written in the blocked operand layout; colidx of the V:N:M result
// HBM-bound: the route kernel reads X once (16 bytes per lane), the others move indices and one copy of X.
#include "common.hpp"
#include "kernels.hpp"
#include "scans.hpp"

namespace sffn {

// One wavefront scores TOK tokens against all E experts.  Summation order (part of the parity contract, the argmax
// depends on it): the products are cut into chunks of 8 consecutive d; lane l accumulates chunks l, l + 64, ... in
// ascending d, then the 64 partial sums are folded by 32, 16, 8, 4, 2, 1.  A bf16 x bf16 product is exact in
// float32, so fmaf rounds exactly like the separate add.
template <int E, int TOK>
__global__ void __launch_bounds__(256) venom_route_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ means, int T, int D,
                                                         int32_t* __restrict__ expert, float* __restrict__ scores) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * 4 + wave) * TOK;
    if (t0 >= T) return;
    float acc[TOK][E];
#pragma unroll
    for (int q = 0; q < TOK; ++q)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[q][e] = 0.0f;
    for (int d = lane * 8; d < D; d += 512) {
        uint4 mv[E];
#pragma unroll
        for (int e = 0; e < E; ++e) mv[e] = *reinterpret_cast<const uint4*>(means + (int64_t)e * D + d);
#pragma unroll
        for (int q = 0; q < TOK; ++q) {
            const int t = t0 + q < T ? t0 + q : T - 1;
            const uint4 xv = *reinterpret_cast<const uint4*>(X + (int64_t)t * D + d);
            const uint32_t xw[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t mw[4] = {mv[e].x, mv[e].y, mv[e].z, mv[e].w};
                float a = acc[q][e];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    a = __builtin_fmaf(bf2f(xw[k] & 0xFFFFu), bf2f(mw[k] & 0xFFFFu), a);
                    a = __builtin_fmaf(bf2f(xw[k] >> 16), bf2f(mw[k] >> 16), a);
                }
                acc[q][e] = a;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < TOK; ++q) {
        float best = 0.0f;
        int arg = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float s = acc[q][e];
#pragma unroll
            for (int w = 32; w >= 1; w >>= 1) s = s + __shfl_xor(s, w, 64);     // both partners add the same two numbers
            if (e == 0 || s > best) { best = s; arg = e; }
            if (scores && lane == 0 && t0 + q < T) scores[(int64_t)(t0 + q) * E + e] = s;
        }
        if (lane == 0 && t0 + q < T) expert[t0 + q] = arg;
    }
}

// ---- stable grouping by expert ------------------------------------------------------------------------------------
// Up to 32768 tokens: one launch.  Every workgroup places 1024 tokens and counts, by ballots, all tokens of each expert and those before its own, so that
// no workgroup waits for another (at most 128 KB from L2 each).  Three passes over blocks of 1024 tokens took 14 us for 8192 tokens, nearly all of
// it launches; this takes 5.
constexpr int kGroupThreads = 1024, kGroupMost = 32768;
template <int E>
__global__ void __launch_bounds__(kGroupThreads) venom_group_kernel(const int32_t* __restrict__ expert, int T, int cap, int32_t* __restrict__ seg,
                                                                   int32_t* __restrict__ perm, int32_t* __restrict__ row_of_token) {
    constexpr int NW = kGroupThreads / 64, U = 4;
    __shared__ int w_all[NW][E], w_before[NW][E], w_own[NW][E], all[E], before[E];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, base = blockIdx.x * kGroupThreads;
    int n_all[E], n_before[E];
#pragma unroll
    for (int e = 0; e < E; ++e) n_all[e] = n_before[e] = 0;
    for (int c = wave * 64; c < T; c += U * kGroupThreads) {
        int v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { const int t = c + u * kGroupThreads + lane; v[u] = t < T ? expert[t] : -1; }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int n = __popcll(__ballot(v[u] == e));
                n_all[e] += n;
                n_before[e] += c + u * kGroupThreads < base ? n : 0;
            }
    }
    const int t = base + tid, mine = t < T ? expert[t] : -1;
    int rank = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long m = __ballot(mine == e);
        if (mine == e) rank = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) { w_all[wave][e] = n_all[e]; w_before[wave][e] = n_before[e]; w_own[wave][e] = __popcll(m); }
    }
    __syncthreads();
    if (tid < E) {
        int x = 0, y = 0;
        for (int w = 0; w < NW; ++w) { x += w_all[w][tid]; y += w_before[w][tid]; }
        all[tid] = x; before[tid] = y;
    }
    __syncthreads();
    int row = 0, off = 0;
    for (int e = 0; e < E; ++e) {
        if (mine == e) row = off + before[e] + rank;
        const int end = off + all[e], next = (end + 63) & ~63;
        if (blockIdx.x == 0) {                 // the run offsets, and the padding of the runs and past the last one
            if (tid == 0) seg[e] = off;
            if (end + tid < next) perm[end + tid] = -1;
        }
        off = next;
    }
    if (blockIdx.x == 0) {
        if (tid == 0) seg[E] = off;
        for (int r = off + tid; r < cap; r += kGroupThreads) perm[r] = -1;
    }
    if (mine >= 0) {
        for (int w = 0; w < wave; ++w) row += w_own[w][mine];
        perm[row] = t;
        row_of_token[t] = row;
    }
}

// More tokens: three passes.
// Pass 1: per block of 1024 tokens, how many go to each expert; also clears perm to -1 (padding).
__global__ void __launch_bounds__(256) venom_count_kernel(const int32_t* __restrict__ expert, int T, int E, int cap,
                                                         int32_t* __restrict__ blockcnt, int32_t* __restrict__ perm) {
    __shared__ int cnt[16];
    if (threadIdx.x < 16) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * 1024;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int t = base + k * 256 + threadIdx.x;
        if (t < cap) perm[t] = -1;
        if (t < T) atomicAdd(&cnt[expert[t]], 1);            // integer counts: the result does not depend on the order
    }
    __syncthreads();
    if ((int)threadIdx.x < E) blockcnt[blockIdx.x * E + threadIdx.x] = cnt[threadIdx.x];
}

// Pass 2 (one workgroup): first row of every (block, expert) and the 64-row padded run offsets.
__global__ void __launch_bounds__(64) venom_scan_kernel(int32_t* __restrict__ blockcnt, int nblk, int E, int32_t* __restrict__ seg) {
    __shared__ int total[16];
    const int e = threadIdx.x;
    if (e < E) {
        int run = 0;
        for (int b = 0; b < nblk; ++b) {
            const int c = blockcnt[b * E + e];
            blockcnt[b * E + e] = run;                        // becomes: tokens of expert e in earlier blocks
            run += c;
        }
        total[e] = run;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int off = 0;
        seg[0] = 0;
        for (int q = 0; q < E; ++q) { off += (total[q] + 63) & ~63; seg[q + 1] = off; }
    }
}

// Pass 3: every token's row = seg[e] + tokens of e in earlier blocks + rank among the block's earlier tokens of e.
__global__ void __launch_bounds__(256) venom_scatter_kernel(const int32_t* __restrict__ expert, int T, int E,
                                                           const int32_t* __restrict__ blockbase, const int32_t* __restrict__ seg,
                                                           int32_t* __restrict__ perm, int32_t* __restrict__ row_of_token) {
    __shared__ int run[16];
    __shared__ int wcnt[4][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)threadIdx.x < E) run[threadIdx.x] = seg[threadIdx.x] + blockbase[blockIdx.x * E + threadIdx.x];
    __syncthreads();
    const int base = blockIdx.x * 1024;
    for (int k = 0; k < 4; ++k) {
        const int t = base + k * 256 + threadIdx.x;
        const int e = t < T ? expert[t] : -1;
        int rank = 0;
        for (int q = 0; q < E; ++q) {                         // E <= 16 ballots: rank among the wave's earlier lanes of the same expert
            const unsigned long long m = __ballot(e == q);
            if (e == q) rank = __popcll(m & ((1ull << lane) - 1ull));
            if (lane == 0) wcnt[wave][q] = __popcll(m);
        }
        __syncthreads();
        if (e >= 0) {
            int r = run[e] + rank;
            for (int w = 0; w < wave; ++w) r += wcnt[w][e];
            perm[r] = t;
            row_of_token[t] = r;
        }
        __syncthreads();
        if ((int)threadIdx.x < E) run[threadIdx.x] += wcnt[0][threadIdx.x] + wcnt[1][threadIdx.x] + wcnt[2][threadIdx.x] + wcnt[3][threadIdx.x];
        __syncthreads();
    }
}

// X rows in permuted order (zero rows for padding), blocked operand layout: one thread per 16 bytes.
__global__ void __launch_bounds__(256) venom_gather_x_kernel(const uint16_t* __restrict__ X, const int32_t* __restrict__ perm, int cap, int D,
                                                            uint16_t* __restrict__ xb) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int cpr = D >> 3;
    const int64_t r = idx / cpr;
    const int c = (int)(idx - r * cpr);
    if (r >= cap) return;
    const int t = perm[r];
    uint4 v = make_uint4(0, 0, 0, 0);
    if (t >= 0) v = *reinterpret_cast<const uint4*>(X + (int64_t)t * D + c * 8);
    *reinterpret_cast<uint4*>(xb + blk_off(r, c * 8, D >> 5)) = v;
}

// colidx[tb, g, :] = (4e, 4e + 1, 4e + 2, 4e + 3) for the 64-row blocks of expert e's run; blocks past the last run: e = 0.
__device__ __forceinline__ void venom_colidx_word(const GemmGroup& g, int64_t idx, int groups, uint32_t* __restrict__ colidx) {
    const int tb = (int)(idx / groups);
    int e = 0;
    for (int q = 0; q < g.n; ++q)
        if (tb * 64 >= (g.seg_dev ? g.seg_dev[q] : g.seg[q]) && tb * 64 < (g.seg_dev ? g.seg_dev[q + 1] : g.seg[q + 1])) e = q;
    colidx[idx] = 0x03020100u + 0x04040404u * (uint32_t)e;
}
__global__ void __launch_bounds__(256) venom_colidx_kernel(GemmGroup g, int nblocks, int groups, uint32_t* __restrict__ colidx) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx < (int64_t)nblocks * groups) venom_colidx_word(g, idx, groups, colidx);
}

// Padding rows past the last run: rows first .. rows - 1 of up to five [rows, row_words] arrays <- their fill words, in one launch.
__global__ void __launch_bounds__(256) fill_tail_rows_kernel(TailFill f, int64_t first, int64_t rows) {
    const int a = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x + first * f.row_words[a];
    if (i < rows * f.row_words[a]) f.p[a][i] = f.v[a];
}
hipError_t launch_fill_tail_rows(const TailFill& f, int64_t first, int64_t rows, hipStream_t s) {
    int64_t widest = 0;
    for (int a = 0; a < f.n; ++a) widest = f.row_words[a] > widest ? f.row_words[a] : widest;
    const int64_t n = (rows - first) * widest;
    if (n == 0 || f.n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_tail_rows_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)f.n), dim3(256), 0, s, f, first, rows);
    return hipGetLastError();
}

// ---- the step's preparing passes ------------------------------------------------------------------------------------
// Weights.  Expert e owns hidden units 4 e .. 4 e + 3 of every M; compact column j of its slice is unit (j / 4) M + 4 e + j % 4.  A workgroup takes 8 M
// hidden units (32 compact columns of every expert: whole 64-byte rows of the blocked layout) x TD of d_model through LDS, reads them once and writes
// the pruned expert-major rows and the experts' unpruned [D, Kc] slices.  (Before: W2 -> W2.T -> slices and pruned rows, W1 twice, with a second,
// unread copy of the packed rows: five passes, 80 us at D = 2048, F = 8192.)
template <int LOGM>
struct RouterTile {
    static constexpr int M = 1 << LOGM, E = M / 4, TF = 8 * M, TD = LOGM == 6 ? 32 : 64;       // (M = 64: half the depth, to leave room for several workgroups)
    static constexpr int Q = TD / 16, ITEMS = TF * Q, P2 = TF + 2, P1 = TD + 2;
    static constexpr int LDS = TD * P2 > TF * P1 ? TD * P2 * 2 : TF * P1 * 2;
};
template <int LOGM, bool SOFT>
__device__ __forceinline__ void router_w2_body(void* smem, int bx, int by, const RouterPrologueArgs& a) {
    using R = RouterTile<LOGM>;
    constexpr int M = R::M, TF = R::TF, TD = R::TD, P = R::P2, Q = R::Q;
    uint16_t* const tile = reinterpret_cast<uint16_t*>(smem);
    uint32_t* const tile32 = reinterpret_cast<uint32_t*>(smem);
    const int tid = threadIdx.x, D = a.D, Kc = a.F >> (LOGM - 2);
    const int f0 = bx * TF, d0 = by * TD, j0 = bx * 32;
#pragma unroll
    for (int i = 0; i < TD * TF / 8 / 256; ++i) {
        const int e = tid + 256 * i, kk = e / (TF / 8), sg = e % (TF / 8);
        const uint4 w = *reinterpret_cast<const uint4*>(a.W2 + (int64_t)(d0 + kk) * a.F + f0 + sg * 8);
        uint32_t* p = tile32 + (kk * P) / 2 + sg * 4;
        p[0] = w.x; p[1] = w.y; p[2] = w.z; p[3] = w.w;
    }
    __syncthreads();
    // pruned rows: item = (expert, 16 rows, row, 16 of d_model); a wavefront writes whole 1 KB blocks
#pragma unroll
    for (int i = 0; i < (R::ITEMS + 255) / 256; ++i) {
        const int idx = tid + 256 * i, q = idx % Q, u = idx / (16 * Q), jl = (u & 1) * 16 + (idx / Q) % 16, e = u >> 1;
        if (R::ITEMS % 256 != 0 && idx >= R::ITEMS) break;
        const uint16_t* p = tile + 16 * q * P + ((jl >> 2) << LOGM) + 4 * e + (jl & 3);
        uint32_t ov[8], mb = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t nib;
            ov[g] = select24<SOFT>(p[4 * g * P], p[(4 * g + 1) * P], p[(4 * g + 2) * P], p[(4 * g + 3) * P], nib);
            mb |= nib << (4 * g);
        }
        const int64_t r = (int64_t)e * Kc + j0 + jl;
        *reinterpret_cast<uint4*>(a.w2vb + blk_off(r, (d0 + 16 * q) / 2, D / 64)) = make_uint4(ov[0], ov[1], ov[2], ov[3]);
        *reinterpret_cast<uint16_t*>(a.w2mb + mblk_off(r, d0 + 16 * q, D / 64)) = (uint16_t)mb;
    }
    // slices: item = (expert, row d, 8 compact columns = two groups of four hidden units)
#pragma unroll
    for (int i = 0; i < R::E * TD * 4 / 256; ++i) {
        const int idx = tid + 256 * i, c = idx & 3, dl = (idx >> 2) % TD, e = idx / (4 * TD);
        const uint32_t* p = tile32 + (dl * P + ((2 * c) << LOGM) + 4 * e) / 2;
        *reinterpret_cast<uint4*>(a.w2e + (int64_t)e * D * Kc + blk_off(d0 + dl, j0 + 8 * c, Kc / 32)) = make_uint4(p[0], p[1], p[M / 2], p[M / 2 + 1]);
    }
}
template <int LOGM, bool SOFT>
__device__ __forceinline__ void router_w1_body(void* smem, int bx, int by, const RouterPrologueArgs& a) {
    using R = RouterTile<LOGM>;
    constexpr int TF = R::TF, TD = R::TD, P = R::P1, Q = R::Q;
    uint16_t* const tile = reinterpret_cast<uint16_t*>(smem);        // [expert, compact column][d]
    uint32_t* const tile32 = reinterpret_cast<uint32_t*>(smem);
    const int tid = threadIdx.x, D = a.D, Kc = a.F >> (LOGM - 2);
    const int f0 = bx * TF, d0 = by * TD, j0 = bx * 32;
#pragma unroll
    for (int i = 0; i < (R::ITEMS + 255) / 256; ++i) {
        const int idx = tid + 256 * i, q = idx % Q, u = idx / (16 * Q), jl = (u & 1) * 16 + (idx / Q) % 16, e = u >> 1;
        if (R::ITEMS % 256 != 0 && idx >= R::ITEMS) break;
        const uint16_t* src = a.W1 + (int64_t)(f0 + ((jl >> 2) << LOGM) + 4 * e + (jl & 3)) * D + d0 + 16 * q;
        const uint4 w0 = *reinterpret_cast<const uint4*>(src), w1 = *reinterpret_cast<const uint4*>(src + 8);
        uint32_t* p = tile32 + ((e * 32 + jl) * P + 16 * q) / 2;
        p[0] = w0.x; p[1] = w0.y; p[2] = w0.z; p[3] = w0.w; p[4] = w1.x; p[5] = w1.y; p[6] = w1.z; p[7] = w1.w;
        uint32_t n0, n1, n2, n3;
        const uint32_t o0 = select24<SOFT>(w0.x & 0xFFFFu, w0.x >> 16, w0.y & 0xFFFFu, w0.y >> 16, n0), o1 = select24<SOFT>(w0.z & 0xFFFFu, w0.z >> 16, w0.w & 0xFFFFu, w0.w >> 16, n1);
        const uint32_t o2 = select24<SOFT>(w1.x & 0xFFFFu, w1.x >> 16, w1.y & 0xFFFFu, w1.y >> 16, n2), o3 = select24<SOFT>(w1.z & 0xFFFFu, w1.z >> 16, w1.w & 0xFFFFu, w1.w >> 16, n3);
        const int64_t r = (int64_t)e * Kc + j0 + jl;
        *reinterpret_cast<uint4*>(a.w1vb + blk_off(r, (d0 + 16 * q) / 2, D / 64)) = make_uint4(o0, o1, o2, o3);
        *reinterpret_cast<uint16_t*>(a.w1mb + mblk_off(r, d0 + 16 * q, D / 64)) = (uint16_t)(n0 | (n1 << 4) | (n2 << 8) | (n3 << 12));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R::E * TD * 4 / 256; ++i) {
        const int idx = tid + 256 * i, c = idx & 3, dl = (idx >> 2) % TD, e = idx / (4 * TD);
        const uint16_t* p = tile + (e * 32 + 8 * c) * P + dl;
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = p[2 * k * P] | ((uint32_t)p[(2 * k + 1) * P] << 16);
        *reinterpret_cast<uint4*>(a.w1t + (int64_t)e * D * Kc + blk_off(d0 + dl, j0 + 8 * c, Kc / 32)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// n_w: workgroups of each weight; n_x: of X and of dY; n_c: of colidx (1024 words each); then n_t for each array of the tail
template <int LOGM, bool SOFT>
__global__ void __launch_bounds__(256) router_prologue_kernel(RouterPrologueArgs a, int n_w2, int n_w1, int n_x, int n_dy, int n_c, int n_t) {
    using R = RouterTile<LOGM>;
    __shared__ __attribute__((aligned(16))) unsigned char smem[R::LDS > kTransposeLds ? R::LDS : kTransposeLds];
    int b = blockIdx.x;
    const int gw = a.F / R::TF, gx = a.D / 64;
    if (b < n_w2) { router_w2_body<LOGM, SOFT>(smem, b % gw, b / gw, a); return; }
    b -= n_w2;
    if (b < n_w1) { router_w1_body<LOGM, SOFT>(smem, b % gw, b / gw, a); return; }
    b -= n_w1;
    if (b < n_x) { transpose_bf16_body(smem, b % gx, b / gx, a.X, a.rows, a.D, a.D, a.xt, 0, a.xb, a.perm); return; }
    b -= n_x;
    if (b < n_dy) { transpose_bf16_body(smem, b % gx, b / gx, a.dY, a.rows, a.D, a.D, a.dyt, 0, a.dyb, a.perm); return; }
    b -= n_dy;
    if (b < n_c) {
        const int groups = a.F >> LOGM;
        for (int64_t i = (int64_t)b * 1024 + threadIdx.x, k = 0; k < 4; ++k, i += 256)
            if (i < (int64_t)(a.rows / 64) * groups) venom_colidx_word(a.seg, i, groups, reinterpret_cast<uint32_t*>(a.colidx));
        return;
    }
    b -= n_c;
    const int arr = b / n_t;
    const int64_t words = a.tail.row_words[arr], first = a.seg.seg_dev ? a.seg.seg_dev[a.seg.n] : a.seg.seg[a.seg.n];
    int64_t i = first * words + (int64_t)(b - arr * n_t) * 1024 + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k, i += 256)
        if (i < a.rows * words) a.tail.p[arr][i] = a.tail.v[arr];
}

template <int LOGM>
static hipError_t launch_router_prologue_m(const RouterPrologueArgs& a, hipStream_t s) {
    using R = RouterTile<LOGM>;
    const int n_w = a.F / R::TF * (a.D / R::TD), n_tr = a.rows / 64 * (a.D / 64);
    int64_t widest = 0;
    for (int k = 0; k < a.tail.n; ++k) widest = a.tail.row_words[k] > widest ? a.tail.row_words[k] : widest;
    const int64_t colidx_words = (int64_t)(a.rows / 64) * (a.F >> LOGM);
    const int n_w2 = a.W2 ? n_w : 0, n_w1 = a.W1 ? n_w : 0, n_x = a.X ? n_tr : 0, n_dy = a.dY ? n_tr : 0, n_c = a.colidx ? (int)((colidx_words + 1023) / 1024) : 0;
    const int n_t = (int)((a.max_tail * widest + 1023) / 1024);
    const int64_t n = (int64_t)n_w2 + n_w1 + n_x + n_dy + n_c + (int64_t)n_t * a.tail.n;
    if (n == 0) return hipSuccess;
    if (n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if (a.mode == 0) hipLaunchKernelGGL((router_prologue_kernel<LOGM, false>), dim3((unsigned)n), dim3(256), 0, s, a, n_w2, n_w1, n_x, n_dy, n_c, n_t > 0 ? n_t : 1);
    else             hipLaunchKernelGGL((router_prologue_kernel<LOGM, true>), dim3((unsigned)n), dim3(256), 0, s, a, n_w2, n_w1, n_x, n_dy, n_c, n_t > 0 ? n_t : 1);
    return hipGetLastError();
}
hipError_t launch_router_prologue(const RouterPrologueArgs& a, hipStream_t s) {
    if (a.rows % 64 || a.D % 64 || a.F % (16 << a.logM)) return hipErrorInvalidValue;
    switch (a.logM) {
        case 3: return launch_router_prologue_m<3>(a, s);
        case 4: return launch_router_prologue_m<4>(a, s);
        case 5: return launch_router_prologue_m<5>(a, s);
        case 6: return launch_router_prologue_m<6>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_venom_route(const uint16_t* X, const uint16_t* means, int64_t T, int64_t D, int E, int32_t* expert, float* scores,
                              hipStream_t s) {
    if (T == 0) return hipSuccess;
    // two tokens per wavefront: enough wavefronts in flight to hide the load latency (8 tokens per wavefront: 1.2-2.2 TB/s of X)
    constexpr int TOK = 2;
    dim3 grid((unsigned)((T + 4 * TOK - 1) / (4 * TOK)));
    switch (E) {
        case 2:  hipLaunchKernelGGL((venom_route_kernel<2, TOK>), grid, dim3(256), 0, s, X, means, (int)T, (int)D, expert, scores); break;
        case 4:  hipLaunchKernelGGL((venom_route_kernel<4, TOK>), grid, dim3(256), 0, s, X, means, (int)T, (int)D, expert, scores); break;
        case 8:  hipLaunchKernelGGL((venom_route_kernel<8, TOK>), grid, dim3(256), 0, s, X, means, (int)T, (int)D, expert, scores); break;
        case 16: hipLaunchKernelGGL((venom_route_kernel<16, 4>), dim3((unsigned)((T + 15) / 16)), dim3(256), 0, s, X, means, (int)T, (int)D, expert, scores); break;   // 16 experts: the means' L2 traffic weighs more
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_venom_permute(const int32_t* expert, int64_t T, int E, int64_t cap, int32_t* blockcnt, int32_t* seg, int32_t* perm,
                                int32_t* row_of_token, hipStream_t s) {
    if (T <= kGroupMost) {
        const dim3 grid((unsigned)((T + kGroupThreads - 1) / kGroupThreads)), threads(kGroupThreads);
        switch (E) {
            case 2:  hipLaunchKernelGGL(venom_group_kernel<2>, grid, threads, 0, s, expert, (int)T, (int)cap, seg, perm, row_of_token); break;
            case 4:  hipLaunchKernelGGL(venom_group_kernel<4>, grid, threads, 0, s, expert, (int)T, (int)cap, seg, perm, row_of_token); break;
            case 8:  hipLaunchKernelGGL(venom_group_kernel<8>, grid, threads, 0, s, expert, (int)T, (int)cap, seg, perm, row_of_token); break;
            case 16: hipLaunchKernelGGL(venom_group_kernel<16>, grid, threads, 0, s, expert, (int)T, (int)cap, seg, perm, row_of_token); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const int nblk = (int)((cap + 1023) / 1024);
    hipLaunchKernelGGL(venom_count_kernel, dim3(nblk), dim3(256), 0, s, expert, (int)T, E, (int)cap, blockcnt, perm);
    hipLaunchKernelGGL(venom_scan_kernel, dim3(1), dim3(64), 0, s, blockcnt, nblk, E, seg);
    hipLaunchKernelGGL(venom_scatter_kernel, dim3(nblk), dim3(256), 0, s, expert, (int)T, E, blockcnt, seg, perm, row_of_token);
    return hipGetLastError();
}

hipError_t launch_venom_gather_x(const uint16_t* X, const int32_t* perm, int64_t cap, int64_t D, uint16_t* xb, hipStream_t s) {
    const int64_t n = cap * (D / 8);
    hipLaunchKernelGGL(venom_gather_x_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, perm, (int)cap, (int)D, xb);
    return hipGetLastError();
}

hipError_t launch_venom_colidx(const GemmGroup& g, int64_t cap, int64_t groups, uint8_t* colidx, hipStream_t s) {
    const int64_t n = (cap / 64) * groups;
    hipLaunchKernelGGL(venom_colidx_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, (int)(cap / 64), (int)groups,
                       reinterpret_cast<uint32_t*>(colidx));
    return hipGetLastError();
}

}  // namespace sffn
