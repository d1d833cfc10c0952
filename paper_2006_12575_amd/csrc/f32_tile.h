// Tiles of output voxels of the fp32 convolutions, and fp32 values as sums of three bf16 ones.
#pragma once
#include "internal.h"

namespace lamp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// A tile of output voxels, each side a power of two (log2), and the tiles a sample needs.
struct TileGeo {
    int ld, lh, lw;      // log2 of the tile's sides
    int nd, nh, nw;      // tiles along each axis
};
// All sides' products equal `vox` (a power of two), w side at least 4, halo at most `halo` voxels: the fewest tiles, then the
// smallest halo.
inline TileGeo pick_tile(int D, int H, int W, int vox, int halo) {
    TileGeo best{0, 0, 2, 0, 0, 0};
    int64_t bt = -1;
    int bh = 0, lv = 0;
    while ((1 << lv) < vox) ++lv;
    for (int lw = 2; lw <= 5 && lw <= lv; ++lw)
        for (int lh = 0; lh + lw <= lv && lh <= 4; ++lh) {
            const int ld = lv - lw - lh;
            const int hv = ((1 << ld) + 2) * ((1 << lh) + 2) * ((1 << lw) + 2);
            if (ld > 4 || hv > halo) continue;
            const int nd = cdiv(D, 1 << ld), nh = cdiv(H, 1 << lh), nw = cdiv(W, 1 << lw);
            const int64_t t = (int64_t)nd * nh * nw;
            if (bt < 0 || t < bt || (t == bt && hv < bh)) {
                bt = t;
                bh = hv;
                best = TileGeo{ld, lh, lw, nd, nh, nw};
            }
        }
    return best;
}

// sum over the 16 lanes of a row
__device__ __forceinline__ float row_sum16(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, true));
    return v;
}

// the largest of the lanes of a row of 16 whose numbers are the same modulo Q
template <int Q> __device__ __forceinline__ float row_most(float v) {
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true)));
    if (Q <= 4) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, true)));
    if (Q <= 2) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, true)));
    return v;
}

// v = h + m + l exactly, each of them bf16: h the value cut to 8 significant bits (so that an infinity stays one and the largest values
// do not become one), m the rest rounded to 8 bits, l what is left, which fits.  Of an infinity or NaN m and l are NaN.
__device__ __forceinline__ void split3(const f32x4& v, uint2 (&o)[3]) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    uint32_t p[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t a = __float_as_uint(v[2 * i]), b = __float_as_uint(v[2 * i + 1]);
        p[0][i] = __builtin_amdgcn_perm(b, a, 0x07060302);
        const float ra = v[2 * i] - __uint_as_float(a & 0xFFFF0000u), rb = v[2 * i + 1] - __uint_as_float(b & 0xFFFF0000u);
        const bf16x2 m = {(__bf16)ra, (__bf16)rb};
        p[1][i] = __builtin_bit_cast(uint32_t, m);
        const float la = ra - __uint_as_float(p[1][i] << 16), lb = rb - __uint_as_float(p[1][i] & 0xFFFF0000u);
        p[2][i] = __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) o[k] = make_uint2(p[k][0], p[k][1]);
}

// The same with h and m in whole steps of grids that the elements of a column share: M = 1.5 * 2^23 steps of a grid whose 2^8 steps reach
// past every |v| (grid_of), so that adding and taking it away rounds to the grid; the rest goes to a grid 2^9 finer, what is left rounds to
// bf16 (2^-26 of the column's largest value).  The matrix unit cuts products to 24 bits below the largest of a group, towards zero, which
// shifts a long sum whose small terms are mostly of one sign; the products of pieces on grids have 16 bits and are added up whole.
__device__ __forceinline__ void split3_grid(const f32x4& v, const f32x4& M, const f32x4& M2, uint2 (&o)[3]) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    uint32_t p[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float h[2], m[2], l[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = 2 * i + j;
            h[j] = (v[k] + M[k]) - M[k];
            const float r = v[k] - h[j];
            m[j] = (r + M2[k]) - M2[k];
            l[j] = r - m[j];
        }
        p[0][i] = __builtin_amdgcn_perm(__float_as_uint(h[1]), __float_as_uint(h[0]), 0x07060302);
        p[1][i] = __builtin_amdgcn_perm(__float_as_uint(m[1]), __float_as_uint(m[0]), 0x07060302);
        const bf16x2 q = {(__bf16)l[0], (__bf16)l[1]};
        p[2][i] = __builtin_bit_cast(uint32_t, q);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) o[k] = make_uint2(p[k][0], p[k][1]);
}
constexpr float GRID_MOST = 0x1p110f;   // from here on M would overflow
__device__ __forceinline__ void grid_of(const f32x4& most, f32x4& M, f32x4& M2) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t e = (__float_as_uint(most[k]) & 0x7F800000u) + (16u << 23 | 0x400000u);
        M[k] = __uint_as_float(e);
        M2[k] = __uint_as_float(e - (9u << 23));
    }
}

// Sum of the h * h products and of the others: where the first is not finite the second may be NaN for no other reason than that
// infinities have no rest.
__device__ __forceinline__ float join_hl(float hh, float rest) { return __builtin_fabsf(hh) < __builtin_inff() ? hh + rest : hh; }

}  // namespace lamp
