// The preparing passes of the router's step as a unit (launch_mix.hpp): a launch of their own (router.hip), or workgroups behind the tiles of eq. (1)
// (router_mix.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "scans.hpp"

namespace sffn {

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

// colidx[tb, g, :] = (4e, 4e + 1, 4e + 2, 4e + 3) for the 64-row blocks of expert e's run; blocks past the last run: e = 0.
__device__ __forceinline__ void venom_colidx_word(const GemmGroup& g, int64_t idx, int groups, uint32_t* __restrict__ colidx) {
    const int tb = (int)(idx / groups);
    int e = 0;
    for (int q = 0; q < g.n; ++q)
        if (tb * 64 >= (g.seg_dev ? g.seg_dev[q] : g.seg[q]) && tb * 64 < (g.seg_dev ? g.seg_dev[q + 1] : g.seg[q + 1])) e = q;
    colidx[idx] = 0x03020100u + 0x04040404u * (uint32_t)e;
}

// counts: workgroups of each weight; of X and of dY; of colidx (1024 words each); of each array of the tail
template <int LOGM, bool SOFT>
struct RouterPrologueUnit {
    using R = RouterTile<LOGM>;
    struct Args { RouterPrologueArgs a; int n_w2, n_w1, n_x, n_dy, n_c, n_t; };
    static constexpr int THREADS = 256, LDS = R::LDS > kTransposeLds ? R::LDS : kTransposeLds;
    static __device__ __forceinline__ void run(unsigned char* smem, int b, int, const Args& u) {
        const RouterPrologueArgs& a = u.a;
        const int gw = a.F / R::TF, gx = a.D / 64;
        if (b < u.n_w2) { router_w2_body<LOGM, SOFT>(smem, b % gw, b / gw, a); return; }
        b -= u.n_w2;
        if (b < u.n_w1) { router_w1_body<LOGM, SOFT>(smem, b % gw, b / gw, a); return; }
        b -= u.n_w1;
        if (b < u.n_x) { transpose_bf16_body(smem, b % gx, b / gx, a.X, a.rows, a.D, a.D, a.xt, 1, a.xb, a.perm); return; }
        b -= u.n_x;
        if (b < u.n_dy) { transpose_bf16_body(smem, b % gx, b / gx, a.dY, a.rows, a.D, a.D, a.dyt, 1, a.dyb, a.perm); return; }
        b -= u.n_dy;
        if (b < u.n_c) {
            const int groups = a.F >> LOGM;
            for (int64_t i = (int64_t)b * 1024 + threadIdx.x, k = 0; k < 4; ++k, i += 256)
                if (i < (int64_t)(a.rows / 64) * groups) venom_colidx_word(a.seg, i, groups, reinterpret_cast<uint32_t*>(a.colidx));
            return;
        }
        b -= u.n_c;
        const int arr = b / u.n_t;
        const int64_t words = a.tail.row_words[arr], first = a.seg.seg_dev ? a.seg.seg_dev[a.seg.n] : a.seg.seg[a.seg.n];
        int64_t i = first * words + (int64_t)(b - arr * u.n_t) * 1024 + threadIdx.x;
#pragma unroll
        for (int k = 0; k < 4; ++k, i += 256)
            if (i < a.rows * words) a.tail.p[arr][i] = a.tail.v[arr];
    }
    static Args make(const RouterPrologueArgs& a) {
        const int n_w = a.F / R::TF * (a.D / R::TD), n_tr = a.rows / 64 * (a.D / 64);
        int64_t widest = 0;
        for (int k = 0; k < a.tail.n; ++k) widest = a.tail.row_words[k] > widest ? a.tail.row_words[k] : widest;
        const int64_t colidx_words = (int64_t)(a.rows / 64) * (a.F >> LOGM), n_t = (a.max_tail * widest + 1023) / 1024;
        return {a, a.W2 ? n_w : 0, a.W1 ? n_w : 0, a.X ? n_tr : 0, a.dY ? n_tr : 0, a.colidx ? (int)((colidx_words + 1023) / 1024) : 0, n_t > 0 ? (int)n_t : 1};
    }
    static int64_t total(const Args& u) { return (int64_t)u.n_w2 + u.n_w1 + u.n_x + u.n_dy + u.n_c + (u.a.max_tail > 0 ? (int64_t)u.n_t * u.a.tail.n : 0); }
    static bool fits(const Args& u) { return total(u) < ((int64_t)1 << 31); }
    static unsigned count(const Args& u) { return (unsigned)total(u); }
    static Args args(const Args& u) { return u; }
};

}  // namespace sffn
