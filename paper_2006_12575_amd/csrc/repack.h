// Weight repacking for the matrix-core 3x3x3 convolution kernels, one element per thread: shared by
// the per-call repack kernels and the batched one the network entry points use.
#pragma once
#include "internal.h"

namespace lamp {

// Output channels a workgroup of the tiled kernel covers: 64 where the 32-channel blocks pair up, else 32.
__host__ __device__ inline int conv_wrows(int Cout) { return ((Cout + 31) / 32) % 2 == 0 ? 64 : 32; }
// Elements of the repacked weights: input channels in whole chunks of 16, output channels in whole blocks.
__host__ __device__ inline int64_t repack_elems(int Cout, int Cin) {
    const int r = conv_wrows(Cout);
    return (int64_t)27 * ((Cin + 15) / 16 * 16) * ((Cout + r - 1) / r * r);
}

// One thread moves one granule of 8 consecutive input channels (16 bytes) of the repacked layout.
// Forward: the granule is contiguous in W as well (one 16-byte load).  Data gradient: its 8 elements
// come from 8 rows of W; the threads are numbered with the output channel fastest, which is the
// contiguous dimension of W in that direction, so each of the 8 loads is coalesced across the wave.
__device__ __forceinline__ uint4 repack_gather8(const bf16_t* __restrict__ p, int64_t stride) {
    uint32_t r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (uint32_t)p[(2 * e) * stride] | ((uint32_t)p[(2 * e + 1) * stride] << 16);
    return make_uint4(r[0], r[1], r[2], r[3]);
}

// Tiled kernel: the repacked weights are the kernel's LDS image,
//   wp[co block][chunk][group g][tap9 t9][plane][row][8],  oc = block*wrows + row, ic = chunk*16 + plane*8 + e,
// so that every 1 KB global -> LDS copy of the kernel reads consecutive memory (with [tap][oc][ic] a copy
// gathered 64 pieces of 16 bytes from 64 rows, and for many input channels those rows no longer stayed in
// L2).  Tap of (g, t9): kd = g, (kh, kw) = (t9/3, t9%3); bykh (8-deep tile, taps walked kh-major): kh = g,
// (kd, kw) = (t9/3, t9%3).  Values: forward W[oc][tap][ic], data gradient W[ic][26-tap][oc].
// Channel counts that do not fill the last chunk or block are padded with zeros there.
// 16 zero bytes behind the weights are the source of the zero padding.
// g: granule index in the order of the lanes.  Data gradient: output channels fastest, as in W.  Forward: the two planes, up to four
// chunks, then output channels, so that a wave reads 64 to 128 bytes in a row of W and writes 128 in a row of wp (with output channels
// fastest every lane read 16 bytes of a row of its own: all forward weights of the 5-level base-32 net 34 us, two chunks 24, four 21;
// one layer's, 4 to 5 us, are launch latency either way).  Divisions in 32 bits where the index fits.
struct RepackPos { int row, plane, t9, grp, chunk, blk; };
template <typename I>
__device__ __forceinline__ RepackPos repack_pos(I u, int wrows, int nchunks, int dgrad) {
    RepackPos p;
    const int lr = wrows == 64 ? 6 : 5, cb = dgrad || (nchunks & 1) ? 0 : (nchunks & 3) ? 1 : 2;
    int c = 0;
    if (!dgrad) { p.plane = (int)(u & 1); c = (int)(u >> 1) & ((1 << cb) - 1); u >>= 1 + cb; }
    p.row = (int)u & (wrows - 1); u >>= lr;
    if (dgrad) { p.plane = (int)(u & 1); u >>= 1; }
    const I t = u / 27;
    const int k = (int)(u - t * 27);
    p.grp = k / 9; p.t9 = k - p.grp * 9;
    const I nc = (I)(nchunks >> cb), b = t / nc;
    p.chunk = ((int)(t - b * nc) << cb) | c;
    p.blk = (int)b;
    return p;
}
__device__ __forceinline__ void repack_tile_gran(const bf16_t* __restrict__ w, bf16_t* __restrict__ wp, int64_t g, int Cout,
                                                 int Cin, int wrows, int dgrad, int bykh) {
    const int64_t total = repack_elems(Cout, Cin);
    if (g == 0) *reinterpret_cast<uint4*>(wp + total) = make_uint4(0, 0, 0, 0);
    if (g >= total / 8) return;
    const int nchunks = (Cin + 15) >> 4;
    const RepackPos p = total / 8 < 0x7FFFFFFF ? repack_pos((uint32_t)g, wrows, nchunks, dgrad) : repack_pos((uint64_t)g, wrows, nchunks, dgrad);
    const int oc = p.blk * wrows + p.row, ic0 = p.chunk * 16 + p.plane * 8;
    const int t = bykh ? (p.t9 / 3) * 9 + p.grp * 3 + (p.t9 % 3) : p.grp * 9 + p.t9;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (oc >= Cout || ic0 >= Cin) {
    } else if (ic0 + 8 > Cin || (!dgrad && Cin % 8)) {   // a granule cut short, or rows without 16-byte alignment
        uint32_t q[4] = {0, 0, 0, 0};
        for (int e = 0; e < 8 && ic0 + e < Cin; ++e)
            q[e >> 1] |= (uint32_t)(dgrad ? w[((int64_t)(ic0 + e) * 27 + (26 - t)) * Cout + oc] : w[((int64_t)oc * 27 + t) * Cin + ic0 + e]) << (16 * (e & 1));
        v = make_uint4(q[0], q[1], q[2], q[3]);
    } else if (!dgrad) v = *reinterpret_cast<const uint4*>(w + ((int64_t)oc * 27 + t) * Cin + ic0);
    else v = repack_gather8(w + ((int64_t)ic0 * 27 + (26 - t)) * Cout + oc, (int64_t)27 * Cout);
    const int64_t o = ((((int64_t)p.blk * nchunks + p.chunk) * 27 + p.grp * 9 + p.t9) * 2 + p.plane) * wrows + p.row;
    *reinterpret_cast<uint4*>(wp + o * 8) = v;
}

}  // namespace lamp
