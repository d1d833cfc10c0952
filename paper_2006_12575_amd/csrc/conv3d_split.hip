// Data and weight gradient of the 3x3x3 convolution of fp32 tensors on the bf16 matrix instructions.
//
// Each operand is the exact sum of three bf16 pieces h + m + l, and of the nine products of pieces the six that matter at 24 bits are
// formed: h h in one accumulator, m h, h m, l h, h l, m m in a second one, which is 2^-8 of the first, so that its five roundings an
// instruction do not count.  (The three left out are 2^-25 of a product.)  v_mfma_f32_16x16x32_bf16 rounds a few times for 32 products
// where v_mfma_f32_16x16x4_f32 rounds every one, so the results are nearer to 64 bits than those of fp32 products: relative error of the
// data gradient 32->32 on 41 x 56 x 47 5.2e-7 -> 1.9e-7, 128->256 on 25 x 28 x 16 1.4e-6 -> 5.1e-7, 8->8 on 2 x 64 x 48 x 80 2.6e-7 -> 1.0e-7.
// (All six in one accumulator: 4.2e-7 where fp32 products have 3.7e-7, 864 of them with one operand non-negative; the three largest alone:
// 4.4e-6.)  Six bf16 products at 1.75 PFLOP/s are 290 TFLOP/s against 154 of the fp32 instructions.
// The forward pass stays with fp32 products: other last bits put pre-activations on the other side of zero, which moves elements of the
// gradients by their full size.
#include "f32_tile.h"

namespace lamp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// ---- data gradient --------------------------------------------------------------------------------
// Bound: the matrix rate of the six products.  D[co][voxel] += W[co][k] * X[k][voxel], k = 4 taps x 8 channels of dz an instruction (7 of
// them for 27 taps of a chunk of 8 channels), A = weights, B = voxels, so that a lane ends with 4 consecutive outputs of a voxel.  A
// workgroup of 4 waves walks tiles of 64 VB voxels x 16 CB outputs: halo and weights of a chunk go through registers, where they are
// split, to LDS (the next chunk's loads in flight during the multiplies).  Weights come in their own layout, so no launch stands in front.
// PACK: up to 8 outputs fill half a block; its other rows take the weights' m pieces, 4 instructions instead of 6.
// A voxel's 8 channels lie in LDS as 48 bytes (h, m, l): 16 voxels in a row are on different banks.  Per step of 4 taps 3 CB + 3 VB reads
// of 16 bytes a lane feed 6 CB VB instructions; with 16 outputs (CB 1) the reads take as long as the products.
// us, fp32 products -> this: 32->32 on 41 x 56 x 47 68 -> 41 (of these about 22 are products at the clock they run at, 11 launch, first loads
// and last stores: a CU gets one or two tiles), 256->128 on 25 x 28 x 16 247 -> 133, 64->48 on 53 x 64 x 29 227 -> 123, 16->16 on
// 2 x 64 x 48 x 80 75 -> 46, 8->8 42 -> 22.5.
// Not better: the second workgroup of a CU started half a chunk later or at another wave priority (within 1 %); three workgroups a CU for
// 16 outputs with single fragment sets (46 -> 50).
struct SplitConvArgs {
    const float* x; const float* w; float* z;   // gradient of the output, weights [x's channels][27][z's], gradient of the input
    int ldx, ldz, D, H, W, Ci, Co;              // Ci, Co: channels of x and z
    TileGeo t;
    int ntiles, per;                   // tiles of all samples; tiles per workgroup
    int zvec;                          // 16-byte stores possible
    int sw2, sw3;                      // bits of a voxel's number in its tile that change places with bits 2 and 3 (split_swap)
    uint32_t mHW, mHH;                 // division of less than 2^11 by the halo's sides: * m >> 16
    uint32_t mT, mNw, mNh; int sT, sNw, sNh;   // by the tiles of a sample, along w, along h
};

// Number of a voxel in its tile from its place in the order of waves, blocks and lanes.
__device__ __forceinline__ int split_swap(int i, int sw2, int sw3) {
    int x = (i >> 2 ^ i >> sw2) & 1;
    i ^= x << 2 | x << sw2;
    x = (i >> 3 ^ i >> sw3) & 1;
    return i ^ (x << 3 | x << sw3);
}
constexpr int SPLIT_EB = 48;   // bytes of a halo voxel: 8 channels, three pieces
__host__ __device__ constexpr int split_wbytes(int cb, bool pack) { return 7 * (pack ? 2 : 3 * cb) * 1024; }
__host__ __device__ constexpr int split_maxk(int vb) { return (2 * (vb == 4 ? 648 : vb == 2 ? 432 : 256) + 255) / 256; }

template <int CB, int VB, bool PACK>
__global__ __launch_bounds__(256, CB == 1 && VB < 4 ? 3 : 2) void conv3d_split_dgrad_kernel(SplitConvArgs a) {
    extern __shared__ __attribute__((aligned(16))) char split_lds[];
    static_assert(!PACK || CB == 1, "up to 8 outputs are half a block");
    constexpr int MAXK = split_maxk(VB), NP = PACK ? 2 : 3, G = CB == 1 && VB > 1 ? 2 : 1, VG = VB / G;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int TD = 1 << a.t.ld, TH = 1 << a.t.lh, TW = 1 << a.t.lw;
    const int HH = TH + 2, HW = TW + 2, HV = (TD + 2) * HH * HW;
    const int tiles = a.t.nd * a.t.nh * a.t.nw, nchunks = a.Ci >> 3;
    const int co0 = blockIdx.y * (16 * CB);
    char* ws = split_lds;                              // [7 tap quads][NP][CB][4 taps][16 outputs][8 inputs]
    char* xs = ws + split_wbytes(CB, PACK);            // [HV] voxels, then 48 zero bytes

    // Loads and stores by buffer instructions: a lane's offset from the tile's first voxel stays for the whole walk, chunks and taps are
    // scalar offsets, and an offset past the end (SKIP) loads zeros and stores nothing.  With 64-bit addresses worked out per piece and
    // chunk the staging took 740 vector instructions of a wave a chunk.
    constexpr int SKIP = (int)0x80000000u, END = 0x7FFFFFF0;
    const int quad = tid & 1;
    int hc[MAXK], vo[MAXK], xo[MAXK];   // halo pieces: coordinates; offset in the halo's frame; the same or SKIP for this tile
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        const uint32_t e = (uint32_t)(tid + 256 * k) >> 1;
        const uint32_t row = e * a.mHW >> 16, hw = e - row * HW, hd = row * a.mHH >> 16, hh = row - hd * HH;
        hc[k] = (int)e < HV ? (int)(hd << 20 | hh << 10 | hw) : -1;
        vo[k] = (((int)(hd * a.H + hh) * a.W + (int)hw) * a.ldx + 4 * quad) * 4;
    }
    f32x4 px[MAXK], pw[4 * CB];
    int dv = 0, hv = 0, wv = 0;         // the tile's first voxel
    const float* xt = a.x;
    auto locate = [&](int tile, int& n, int& d0, int& h0, int& w0) __attribute__((always_inline)) {
        n = (int)((uint64_t)(uint32_t)tile * a.mT >> a.sT);
        const uint32_t r0 = (uint32_t)(tile - n * tiles), r1 = (uint32_t)((uint64_t)r0 * a.mNw >> a.sNw);
        const uint32_t r2 = (uint32_t)((uint64_t)r1 * a.mNh >> a.sNh);
        d0 = (int)(r2 << a.t.ld);
        h0 = (int)((r1 - r2 * a.t.nh) << a.t.lh);
        w0 = (int)((r0 - r1 * a.t.nw) << a.t.lw);
    };
    auto to_tile = [&](int tile) __attribute__((always_inline)) {
        int n;
        locate(tile, n, dv, hv, wv);
        xt = a.x + ((((int64_t)n * a.D + dv - 1) * a.H + hv - 1) * a.W + wv - 1) * a.ldx;
#pragma unroll
        for (int k = 0; k < MAXK; ++k) {
            asm volatile("" : "+v"(hc[k]));   // its parts are not worth registers of their own across the walk
            const int hd = hc[k] >> 20, hh = hc[k] >> 10 & 1023, hw = hc[k] & 1023;
            const bool in = hc[k] >= 0 && (unsigned)(dv - 1 + hd) < (unsigned)a.D && (unsigned)(hv - 1 + hh) < (unsigned)a.H &&
                            (unsigned)(wv - 1 + hw) < (unsigned)a.W;
            xo[k] = in ? vo[k] : SKIP;
        }
    };
    auto fetch_x = [&](int c0) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xt), 0, END, 0x00020000);
#pragma unroll
        for (int k = 0; k < MAXK; ++k) px[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, xo[k], 4 * c0, 0));
    };
    char* const xst = xs + (tid >> 1) * SPLIT_EB + 8 * quad;
    auto stage_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (hc[k] >= 0) {
                uint2 p[3];
                split3(px[k], p);
#pragma unroll
                for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(xst + k * (128 * SPLIT_EB) + 16 * i) = p[i];
            }
    };
    // Weight pieces: 4 inputs (rows of W) of 4 outputs and a tap, W[ci][26 - t][co..], transposed in registers; a thread's pieces differ in the
    // block of outputs.  Rows past the last output hold other weights or zeros and are not stored.
    constexpr int OQ = PACK ? 2 : 4, STEP = (PACK ? 2 : 3 * CB) * 1024;
    const int kq = tid / OQ & 1, wt = tid / (2 * OQ), wr = 4 * (tid % OQ);
    const int wo = 4 * ((4 * kq * 27 + 26 - min(wt, 26)) * a.Co + co0 + wr);
    char* const wst = ws + (wt >> 2) * STEP + (wt & 3) * 256 + kq * 8;
    auto put_w = [&](char* o, int row, const f32x4& v) __attribute__((always_inline)) {
        uint2 p[3];
        split3(v, p);
        const int tg = wt & 3;   // (rows swapped by tap: the lanes that transpose write to different banks)
        if constexpr (PACK) {   // rows 0-7: h, rows 8-15: m; the second piece's rows 0-7: l
            *reinterpret_cast<uint2*>(o + ((row ^ tg) << 4)) = p[0];
            *reinterpret_cast<uint2*>(o + (((row ^ tg) + 8) << 4)) = p[1];
            *reinterpret_cast<uint2*>(o + 1024 + ((row ^ tg) << 4)) = p[2];
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(o + i * CB * 1024 + ((row ^ tg) << 4)) = p[i];
        }
    };
    auto fetch_w = [&](int c0) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w), 0, 108 * a.Ci * a.Co, 0x00020000);
#pragma unroll
        for (int u = 0; u < 4 * CB; ++u)
            pw[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, wo, 4 * ((c0 + u % 4) * 27 * a.Co + u / 4 * 16), 0));
    };
    auto stage_w = [&]() __attribute__((always_inline)) {
        if (wt >= 27) return;
#pragma unroll
        for (int u = 0; u < CB; ++u)
#pragma unroll
            for (int o = 0; o < 4; ++o)
                put_w(wst + u * 1024, wr + o, f32x4{pw[4 * u][o], pw[4 * u + 1][o], pw[4 * u + 2][o], pw[4 * u + 3][o]});
    };

    int base[VB], zo[VB], ko[7];   // the lane's voxels: in the halo, in z
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        const int p = split_swap((wid * VB + vb) * 16 + l16, a.sw2, a.sw3);
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        base[vb] = ((d * HH + h) * HW + w) * SPLIT_EB;
        zo[vb] = (((d * a.H + h) * a.W + w) * a.ldz + co0 + 4 * g) * 4;
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = 4 * i + g;
        ko[i] = ((t / 9 * HH + t / 3 % 3) * HW + t % 3) * SPLIT_EB;
    }
    const char* wl = ws + (g * 16 + (l16 ^ g)) * 16;
    f32x4 acc[CB][VB], rest[CB][VB];   // products of the h pieces, the others

    // tap 27 (weights and voxel), the rows that PACK leaves empty
    if (PACK)
        for (int i = tid; i < split_wbytes(CB, PACK) / 16; i += 256) reinterpret_cast<uint4*>(ws)[i] = make_uint4(0, 0, 0, 0);
    else
        for (int i = tid; i < 3 * CB * 16; i += 256)
            *reinterpret_cast<uint4*>(ws + (6 * 3 * CB + i / 16) * 1024 + 768 + i % 16 * 16) = make_uint4(0, 0, 0, 0);
    if (tid < 3) *reinterpret_cast<uint4*>(xs + HV * SPLIT_EB + tid * 16) = make_uint4(0, 0, 0, 0);
    if (PACK) __syncthreads();

    const int t0 = blockIdx.x * a.per;
    int t1 = t0 + a.per;
    if (t1 > a.ntiles) t1 = a.ntiles;
    if (t0 >= t1) return;
    to_tile(t0);
    fetch_w(0);
    fetch_x(0);
    for (int tile = t0; tile < t1; ++tile) {
        int n, d0, h0, w0;
        locate(tile, n, d0, h0, w0);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) acc[cb][vb] = rest[cb][vb] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int ch = 0; ch < nchunks; ++ch) {
            if (ch || tile > t0) __syncthreads();   // every wave is done with the previous chunk
            stage_x();
            if (nchunks > 1 || tile == t0) stage_w();
            __syncthreads();
            const bool last = ch + 1 == nchunks;
            if (last && tile + 1 < t1) to_tile(tile + 1);
            if (!last || tile + 1 < t1) {   // (one call of each: the results of two meet behind a wait for the loads)
                fetch_x(last ? 0 : (ch + 1) * 8);
                if (nchunks > 1) fetch_w(last ? 0 : (ch + 1) * 8);
            }
            __builtin_amdgcn_sched_barrier(0);
            // steps of 4 taps of 8 channels; a unit is G voxel blocks of a step, its fragments read one unit ahead
            bf16x8 wf[2][NP][CB], b[2][G][3];
            auto wfrags = [&](int i) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) wf[i & 1][p][cb] = *reinterpret_cast<const bf16x8*>(wl + ((i * NP + p) * CB + cb) * 1024);
            };
            auto xfrags = [&](int u) __attribute__((always_inline)) {
                const int i = u / VG;
#pragma unroll
                for (int v = 0; v < G; ++v) {
                    int o = base[u % VG * G + v] + ko[i];
                    if (i == 6) o = g == 3 ? HV * SPLIT_EB : o;
#pragma unroll
                    for (int p = 0; p < 3; ++p) b[u & 1][v][p] = *reinterpret_cast<const bf16x8*>(xs + o + 16 * p);
                }
            };
            wfrags(0);
            xfrags(0);
#pragma unroll
            for (int u = 0; u < 7 * VG; ++u) {
                const int i = u / VG;
                if (u + 1 < 7 * VG) xfrags(u + 1);
                if (u % VG == 0 && i + 1 < 7) wfrags(i + 1);
                // the smallest first: m m, l h, h l, m h, h m into `rest`, h h into `acc`
                constexpr int PW[6] = {1, 2, 0, 1, 0, 0}, PX[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < (PACK ? 4 : 6); ++q)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int v = 0; v < G; ++v) {
                            const int vb = u % VG * G + v;
                            // PACK: (h, m) x l, l x h, (h, m) x m, (h, m) x h
                            const int pw_ = PACK ? (q == 1 ? 1 : 0) : PW[q], px_ = PACK ? (q == 0 ? 2 : q == 2 ? 1 : 0) : PX[q];
                            f32x4& c = q == (PACK ? 3 : 5) ? acc[cb][vb] : rest[cb][vb];
                            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i & 1][pw_][cb], b[u & 1][v][px_], c, 0, 0, 0);
                        }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        int lo = l16;
        asm volatile("" : "+v"(lo));
        float* const zt = a.z + (((int64_t)n * a.D + d0) * a.H + h0) * (int64_t)a.W * a.ldz + (int64_t)w0 * a.ldz;
        const auto rz = __builtin_amdgcn_make_buffer_rsrc(zt, 0, END, 0x00020000);
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            if constexpr (PACK) {   // outputs c + 8 hold the products of the weights' m pieces; they lie 32 lanes further on
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float t = acc[0][vb][r] + rest[0][vb][r];
                    rest[0][vb][r] += __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false)[1]);
                }
            }
            const int p = split_swap((wid * VB + vb) * 16 + lo, a.sw2, a.sw3);
            const bool in = w0 + (p & (TW - 1)) < a.W && h0 + ((p >> a.t.lw) & (TH - 1)) < a.H && d0 + (p >> (a.t.lw + a.t.lh)) < a.D;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int co = co0 + 16 * cb + 4 * g;
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = join_hl(acc[cb][vb][r], rest[cb][vb][r]);
                if (a.zvec)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rz, in && co < a.Co ? zo[vb] : SKIP, 64 * cb, 0);
                else
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r]), rz, in && co + r < a.Co ? zo[vb] + 4 * r : SKIP, 64 * cb, 0);
            }
        }
    }
}

// The fewest tiles, then the smallest halo, then the longest rows along w.
static TileGeo split_tile(int D, int H, int W, int vox, int halo) {
    TileGeo best{0, 0, 2, 0, 0, 0};
    int64_t bt = -1;
    int bh = 0, lv = 0;
    while ((1 << lv) < vox) ++lv;
    for (int lw = 5; lw >= 2; --lw)
        for (int lh = lv - lw < 4 ? lv - lw : 4; lh >= 0; --lh) {
            const int ld = lv - lw - lh;
            const int hv = ((1 << ld) + 2) * ((1 << lh) + 2) * ((1 << lw) + 2);
            if (ld < 0 || ld > 4 || hv > halo) continue;
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
// The 16 voxels of a fragment read lie 16-byte pieces 3 * (their place in the halo) apart, modulo the 16 pieces of the LDS banks: rows of
// fewer than 16 voxels take the bits of the tile that spread them best (rows 4 apart for tiles of 8 x 8 along h and w).
static void split_swaps(const TileGeo& t, int* sw2, int* sw3) {
    const int lv = t.ld + t.lh + t.lw, HW = (1 << t.lw) + 2, HH = (1 << t.lh) + 2;
    int least = 17;
    *sw2 = 2;
    *sw3 = 3;
    for (int a = 2; a < (t.lw == 2 ? lv : 3); ++a)
        for (int b = 3; b < (t.lw <= 3 ? lv : 4); ++b) {
            if (b == a || a == 3) continue;
            int n[16] = {}, most = 0;
            for (int i = 0; i < 16; ++i) {
                const int p = (i & 3) | (i >> 2 & 1) << a | (i >> 3 & 1) << b;
                const int w = p & ((1 << t.lw) - 1), h = p >> t.lw & ((1 << t.lh) - 1), d = p >> (t.lw + t.lh);
                const int k = ++n[((d * HH + h) * HW + w) * 3 & 15];
                most = k > most ? k : most;
            }
            if (most < least) {
                least = most;
                *sw2 = a;
                *sw3 = b;
            }
        }
}
// 256 voxels a workgroup where that gives every CU one, else 128, else 64, and then 16 outputs (sweep over 24 shapes: within 6 % of the
// best of the six choices but for 256->128 on 25 x 28 x 16, 133 against 124 us).
struct SplitPlan { int vb, cb; bool pack; TileGeo t; };
__host__ constexpr int split_halo(int vb) { return vb == 4 ? 648 : vb == 2 ? 432 : 256; }
static SplitPlan split_plan(const lamp_tensor_desc* zd) {
    SplitPlan p;
    p.pack = zd->c <= 8;
    p.cb = zd->c > 16 ? 2 : 1;
    const int64_t v = (int64_t)zd->d * zd->h * zd->w;
    auto blocks = [&](int vox) { return (int64_t)zd->n * ((v + vox - 1) / vox) * cdiv(zd->c, 16 * p.cb); };
    p.vb = blocks(256) >= 256 ? 4 : blocks(128) >= 256 ? 2 : 1;
    if (p.vb == 1 && p.cb == 2 && blocks(64) < 256) p.cb = 1;
    p.t = split_tile(zd->d, zd->h, zd->w, p.vb * 64, split_halo(p.vb));
    return p;
}
// Whole 16-byte pieces and whole chunks of 8 channels of dz, offsets within 32 bits.  With one or two chunks it pays from about 350 thousand
// elements of dz on (us, fp32 products / this: 8->8 on 32^3 7.3 / 7.5, on 48^3 13.3 / 8.7; 16->16 on 16^3 7.4 / 7.8, on 40^3 13.0 / 10.1);
// with three or more everywhere (32->32 on 8^3 10.0 / 8.4).
bool split_dgrad_takes(const lamp_tensor_desc* xd, const void* x, const lamp_tensor_desc* zd, const void* w) {
    if (xd->dtype != LAMP_F32 || xd->c % 8 || xd->ldc % 4 || !aligned16(x) || !aligned16(w) || zd->c % 4) return false;
    if (xd->c < 24 && nvox(xd) * xd->c < 350000) return false;
    const SplitPlan p = split_plan(zd);
    return (int64_t)p.t.nd * p.t.nh * p.t.nw * zd->n < ((int64_t)1 << 31) && cdiv(zd->c, 16) <= 65535 &&
           (int64_t)zd->h * zd->w * 18 * (xd->ldc > zd->ldc ? xd->ldc : zd->ldc) < ((int64_t)1 << 29) &&   // byte offsets in a tile, in w
           (int64_t)xd->c * zd->c < ((int64_t)1 << 24);
}

template <int CB, int VB, bool PACK>
static lamp_status split_launch(const SplitPlan& p, dim3 grid, hipStream_t s, const SplitConvArgs& a) {
    const int hv = ((1 << p.t.ld) + 2) * ((1 << p.t.lh) + 2) * ((1 << p.t.lw) + 2);
    constexpr int most = split_wbytes(CB, PACK) + (split_halo(VB) + 1) * SPLIT_EB;
    if (most > 65536 && ensure_dyn_lds((const void*)conv3d_split_dgrad_kernel<CB, VB, PACK>, most) != LAMP_OK) return LAMP_ERR_HIP;
    hipLaunchKernelGGL((conv3d_split_dgrad_kernel<CB, VB, PACK>), grid, dim3(256), split_wbytes(CB, PACK) + (hv + 1) * SPLIT_EB, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

lamp_status split_dgrad(const lamp_tensor_desc* xd, const float* x, const float* w, const lamp_tensor_desc* zd, float* z, hipStream_t s) {
    const SplitPlan p = split_plan(zd);
    const int tiles = p.t.nd * p.t.nh * p.t.nw, cols = cdiv(zd->c, 16 * p.cb);
    SplitConvArgs a;
    a.x = x; a.w = w; a.z = z;
    a.ldx = xd->ldc; a.ldz = zd->ldc;
    a.D = zd->d; a.H = zd->h; a.W = zd->w; a.Ci = xd->c; a.Co = zd->c;
    a.t = p.t;
    a.zvec = aligned16(z) && zd->ldc % 4 == 0;
    split_swaps(p.t, &a.sw2, &a.sw3);
    a.mHW = (65536 + (1 << p.t.lw) + 1) / ((1 << p.t.lw) + 2);
    a.mHH = (65536 + (1 << p.t.lh) + 1) / ((1 << p.t.lh) + 2);
    div_magic(tiles, &a.mT, &a.sT);
    div_magic(p.t.nw, &a.mNw, &a.sNw);
    div_magic(p.t.nh, &a.mNh, &a.sNh);
    // tiles per workgroup: as in f32_conv
    a.ntiles = tiles * zd->n;
    a.per = 1;
    int64_t best = -1;
    for (int per = 1; per <= 16 && (per == 1 || (int64_t)cdiv(a.ntiles, per) * cols > 256); ++per) {
        const int64_t load = (int64_t)per * (((int64_t)cdiv(a.ntiles, per) * cols + 255) / 256);
        if (best < 0 || load <= best) {
            best = load;
            a.per = per;
        }
    }
    const dim3 grid((unsigned)((a.ntiles + a.per - 1) / a.per), cols);
    if (p.pack) return p.vb == 4 ? split_launch<1, 4, true>(p, grid, s, a) : p.vb == 2 ? split_launch<1, 2, true>(p, grid, s, a) : split_launch<1, 1, true>(p, grid, s, a);
    if (p.cb == 1) return p.vb == 4 ? split_launch<1, 4, false>(p, grid, s, a) : p.vb == 2 ? split_launch<1, 2, false>(p, grid, s, a) : split_launch<1, 1, false>(p, grid, s, a);
    return p.vb == 4 ? split_launch<2, 4, false>(p, grid, s, a) : p.vb == 2 ? split_launch<2, 2, false>(p, grid, s, a) : split_launch<2, 1, false>(p, grid, s, a);
}

// ---- weight gradient ------------------------------------------------------------------------------
// Bound: the matrix rate of the six products.  dW[co][column] += dz[voxel][co] * x[voxel + tap][ci], 32 voxels an instruction, column =
// (tap, ci) of a slab of CIC input channels in blocks of 16.  A workgroup of 4 waves walks tiles of 128 (256) voxels; x halo and dz go
// through registers, where they are split, to LDS, one plane a piece, and transposing reads give each lane 8 voxels of its channel.  CG waves
// share out the column blocks, 7 each, 4 / CG the voxels; each of the latter has a partial of its own, added up in a fixed order by
// reduce_partials_kernel; after SPLITW_CHAIN tiles (128 instructions' roundings) the sums go to the partial.
// The pieces lie on grids (split3_grid): with those of split3, sums over 10^5 voxels of a dz that is more often negative than positive were
// shifted by the products that the matrix unit cuts off (32->32 on 41 x 56 x 47, dz from an InstanceNorm backward: relative error 1.8e-7
// with fp32 products in chains of 128, 8.5e-7 with split3, 1.4e-7 with grids of single threads, 6.5e-8 so; 8->8 on 2 x 64 x 48 x 80 1.8e-7 ->
// 5.8e-8, 256->256 on 3 x 28 x 27 x 26 2.9e-7 -> 1.0e-7).
// With the reduction, us, fp32 products -> this: 32->32 on 41 x 56 x 47 81 -> 54, 8->8 on 2 x 64 x 48 x 80 53 -> 28, 16->16 91 -> 51,
// 128->256 on 25 x 28 x 16 214 -> 115, 48->64 on 53 x 64 x 29 198 -> 110.  256 / 384 / 512 / 768 workgroups: 61 / 62 / 58 / 75 us, 71 / 67 /
// 52 / 55 us (the first and the third of these shapes).
struct SplitWgradArgs {
    const float* x; const float* dz; float* part;   // part [splits * VG][Co][27][Ci]
    NormIn nm;
    int ldx, lddz, N, D, H, W, Ci, Co;
    TileGeo t;
    int ntiles, per, flush;                         // tiles of all samples; per split; per chain of additions
    int cochunks;
    uint32_t mHW, mHH;
    uint32_t mT, mNw, mNh; int sT, sNw, sNh;
};
template <int CIC, int CBO> struct SplitWg {
    static constexpr int VOX = CIC == 8 && CBO == 1 ? 256 : 128, HALO = VOX == 256 ? 648 : 432;
    static constexpr int CG = CIC == 16 ? 4 : 2, VG = 4 / CG, NB = 7;   // waves along the columns, along the voxels; blocks of 16 columns a wave
    static constexpr int XP = HALO * CIC * 2;                           // bytes of a piece of the halo
};

template <int CIC, int CBO, bool PACK>
__global__ __launch_bounds__(256, 2) void conv3d_split_wgrad_kernel(SplitWgradArgs a) {
    extern __shared__ __attribute__((aligned(16))) char splitw_lds[];
    static_assert(!PACK || CBO == 1, "up to 8 outputs are half a block");
    typedef SplitWg<CIC, CBO> P;
    constexpr int VOX = P::VOX, HALO = P::HALO, CG = P::CG, VG = P::VG, NB = P::NB, XP = P::XP, NK = VOX / 32 / VG;
    constexpr int QE = CIC / 4, MX = (HALO * QE + 255) / 256, QZ = PACK ? 2 : 4 * CBO, MZ = VOX * QZ / 256;
    constexpr int NP = PACK ? 2 : 3, NBUF = CBO == 2 ? 2 : 3;
    constexpr int SKIP = (int)0x80000000u, END = 0x7FFFFFF0;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int cg = __builtin_amdgcn_readfirstlane(wid % CG), vg = __builtin_amdgcn_readfirstlane(wid / CG);
    const int ci0 = (blockIdx.y / a.cochunks) * CIC, co0 = (blockIdx.y % a.cochunks) * (16 * CBO);
    const int TD = 1 << a.t.ld, TH = 1 << a.t.lh, TW = 1 << a.t.lw;
    const int HH = TH + 2, HW = TW + 2, HV = (TD + 2) * HH * HW;
    const int tiles = a.t.nd * a.t.nh * a.t.nw;
    char* xs = splitw_lds;             // [3][HALO][CIC] bf16
    char* zs = splitw_lds + 3 * XP;    // [3][CBO][VOX][16]; PACK [VOX][h, m, l, zeros][8]

    const int xq = tid & (QE - 1);
    int hc[MX];
    uint32_t pin = 0;   // halo pieces inside the volume
#pragma unroll
    for (int k = 0; k < MX; ++k) {
        const uint32_t e = (uint32_t)(tid + 256 * k) / QE;
        const uint32_t row = e * a.mHW >> 16, hw = e - row * HW, hd = row * a.mHH >> 16, hh = row - hd * HH;
        hc[k] = (int)e < HV ? (int)(hd << 20 | hh << 10 | hw) : -1;
    }
    const int zq = tid % QZ;
    int zc[MZ];
#pragma unroll
    for (int k = 0; k < MZ; ++k) {
        const int p = (tid + 256 * k) / QZ;
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        zc[k] = d << 20 | h << 10 | w;
    }
    f32x4 px[MX], pz[MZ];
    int pn = 0;                        // sample of the tile in flight
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        const int n = (int)((uint64_t)(uint32_t)tile * a.mT >> a.sT);
        const uint32_t r0 = (uint32_t)(tile - n * tiles), r1 = (uint32_t)((uint64_t)r0 * a.mNw >> a.sNw);
        const uint32_t r2 = (uint32_t)((uint64_t)r1 * a.mNh >> a.sNh);
        const int d0 = (int)(r2 << a.t.ld), h0 = (int)((r1 - r2 * a.t.nh) << a.t.lh), w0 = (int)((r0 - r1 * a.t.nw) << a.t.lw);
        pn = n;
        pin = 0;
        const int64_t org = (((int64_t)n * a.D + d0) * a.H + h0) * a.W + w0;
        const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x + (org - ((int64_t)a.H + 1) * a.W - 1) * a.ldx), 0, END, 0x00020000);
        const auto rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.dz + org * a.lddz), 0, END, 0x00020000);
#pragma unroll
        for (int k = 0; k < MX; ++k) {
            asm volatile("" : "+v"(hc[k]));
            const int hd = hc[k] >> 20, hh = hc[k] >> 10 & 1023, hw = hc[k] & 1023;
            const bool in = hc[k] >= 0 && ci0 + 4 * xq < a.Ci && (unsigned)(d0 - 1 + hd) < (unsigned)a.D && (unsigned)(h0 - 1 + hh) < (unsigned)a.H &&
                            (unsigned)(w0 - 1 + hw) < (unsigned)a.W;
            if (in) pin |= 1u << k;
            px[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rx, in ? (((hd * a.H + hh) * a.W + hw) * a.ldx + ci0 + 4 * xq) * 4 : SKIP, 0, 0));
        }
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
            asm volatile("" : "+v"(zc[k]));
            const int d = zc[k] >> 20, h = zc[k] >> 10 & 1023, w = zc[k] & 1023;
            const bool in = co0 + 4 * zq < a.Co && d0 + d < a.D && h0 + h < a.H && w0 + w < a.W;
            pz[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rz, in ? (((d * a.H + h) * a.W + w) * a.lddz + co0 + 4 * zq) * 4 : SKIP, 0, 0));
        }
    };
    char* const xst = xs + tid / QE * (2 * CIC) + 8 * xq;
    char* const zst = PACK ? zs + tid / 2 * 64 + 8 * zq : zs + (zq >> 2) * (VOX * 32) + tid / QZ * 32 + (zq & 3) * 8;
    auto stage = [&]() __attribute__((always_inline)) {
        if (a.nm.mean_rstd) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = ci0 + 4 * xq + j;
                if (c >= a.nm.c_norm) continue;
                float na, nb;
                norm_coeffs(a.nm, pn, c, na, nb);
#pragma unroll
                for (int k = 0; k < MX; ++k)
                    if (pin >> k & 1) {   // the padding is zero behind the normalisation
                        const float u = norm_u(px[k][j], na, nb);
                        px[k][j] = !a.nm.relu || u > 0.f ? u : 0.f;
                    }
            }
        }
        // A thread's pieces are of the same four channels: the largest of its own values and of those that the lanes of its row hold of these
        // channels sets their grid, near enough to the other rows' (a product's 16 bits leave the matrix unit 8).
        auto most = [](const f32x4& m, const f32x4& v) __attribute__((always_inline)) {
            f32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = fmaxf(m[j], __builtin_fabsf(v[j]));
            return o;
        };
        f32x4 mx = {0.f, 0.f, 0.f, 0.f}, mz = mx, gx, gx2, gz, gz2;
#pragma unroll
        for (int k = 0; k < MX; ++k) mx = most(mx, px[k]);
#pragma unroll
        for (int k = 0; k < MZ; ++k) mz = most(mz, pz[k]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            mx[j] = row_most<QE>(mx[j]);
            mz[j] = row_most<QZ>(mz[j]);
        }
        const f32x4 mm = most(mx, mz);
        const bool wide = __any(fmaxf(fmaxf(mm[0], mm[1]), fmaxf(mm[2], mm[3])) >= GRID_MOST);
        grid_of(mx, gx, gx2);
        grid_of(mz, gz, gz2);
        auto put = [&](auto cut_x, auto cut_z) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < MX; ++k)
                if (hc[k] >= 0) {
                    uint2 p[3];
                    cut_x(px[k], p);
#pragma unroll
                    for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(xst + k * (512 / QE * CIC) + i * XP) = p[i];
                }
#pragma unroll
            for (int k = 0; k < MZ; ++k) {
                uint2 p[3];
                cut_z(pz[k], p);
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    *reinterpret_cast<uint2*>(PACK ? zst + k * (128 * 64) + i * 16 : zst + k * (256 / QZ * 32) + i * (CBO * VOX * 32)) = p[i];
            }
        };
        if (__builtin_expect(wide, 0)) {   // infinities and values that large
            auto cut = [](const f32x4& v, uint2 (&p)[3]) __attribute__((always_inline)) { split3(v, p); };
            put(cut, cut);
        } else
            put([&](const f32x4& v, uint2 (&p)[3]) __attribute__((always_inline)) { split3_grid(v, gx, gx2, p); },
                [&](const f32x4& v, uint2 (&p)[3]) __attribute__((always_inline)) { split3_grid(v, gz, gz2, p); });
    };
    if constexpr (PACK) {
        for (int i = tid; i < VOX; i += 256) *reinterpret_cast<uint4*>(zs + i * 64 + 48) = make_uint4(0, 0, 0, 0);
    }

    // Fragments by transposing reads: of 16 lanes, lane s gives the address of 4 channels (s % 4) of a voxel (s / 4), and each gets 4
    // voxels of channel l16.  A k-step is 32 voxels, in the order that both operands share: first 4 g + 0..3, then 16 + 4 g + 0..3, so
    // that half a wave reads 8 voxels in a row.  A column is (tap, channel) of the slab.
    auto vox_off = [&](int p) __attribute__((always_inline)) {
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        return ((d * HH + h) * HW + w) * (2 * CIC);
    };
    int col[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int c = (cg * NB + i) * 16 + 4 * (l16 & 3);
        int t = c / CIC;
        t = t < 27 ? t : 26;   // columns past the end are computed and not written
        col[i] = vox_off(4 * g + (l16 >> 2)) + ((t / 9 * HH + t / 3 % 3) * HW + t % 3) * (2 * CIC) + c % CIC * 2;
    }
    int ko[NK];                        // k-steps of this wave: offset in the halo
#pragma unroll
    for (int k = 0; k < NK; ++k) ko[k] = __builtin_amdgcn_readfirstlane(vox_off((k * VG + vg) * 32));
    const int half = __builtin_amdgcn_readfirstlane(vox_off(16));
    const char* const za = PACK ? zs + (vg * 32 + 4 * g + (l16 >> 2)) * 64 + (l16 & 3) * 8 : zs + (vg * 32 + 4 * g + (l16 >> 2)) * 32 + (l16 & 3) * 8;

    typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    auto tr = [](const char* lo, const char* hi) __attribute__((always_inline)) {
        const s16x4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)lo), v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)hi);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(u, v, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    f32x4 acc[CBO][NB], rest[CBO][NB];   // products of the h pieces, the others
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < CBO; ++cb)
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[cb][i] = rest[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    float* const pb = a.part + ((int64_t)blockIdx.x * VG + vg) * a.Co * 27 * a.Ci;
    // Buffer accesses: a lane's output and channel in its offset, block, tap and row in scalars (a branch and a 64-bit address to every value
    // were 1100 instructions a wave and dump).
    auto dump = [&](bool add) __attribute__((always_inline)) {
        const auto rp = __builtin_amdgcn_make_buffer_rsrc(pb, 0, END, 0x00020000);
        const int tl = CIC == 16 ? 0 : l16 >> 3, ci = ci0 + l16 % CIC;
        int vo[CBO];
#pragma unroll
        for (int cb = 0; cb < CBO; ++cb) vo[cb] = ci < a.Ci && co0 + 16 * cb + 4 * g < a.Co ? ((4 * g * 27 + tl) * a.Ci + ci) * 4 : SKIP;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int t = (cg * NB + i) * (16 / CIC);   // the block's (first) tap
            if (t >= 27) continue;
#pragma unroll
            for (int cb = 0; cb < CBO; ++cb) {
                const int o = CIC < 16 && t + tl >= 27 ? SKIP : vo[cb];
                float old[4] = {0.f, 0.f, 0.f, 0.f};
                if (add)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        old[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, o, ((co0 + 16 * cb + r) * 27 + t) * a.Ci * 4, 0));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float q = rest[cb][i][r];
                    if constexpr (PACK) {   // rows c + 8 hold the products of dz's m pieces; they lie 32 lanes further on
                        const float u = acc[cb][i][r] + q;
                        q += __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(u), false, false)[1]);
                    }
                    const float v = join_hl(acc[cb][i][r], q);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(add ? old[r] + v : v), rp, o, ((co0 + 16 * cb + r) * 27 + t) * a.Ci * 4, 0);
                }
            }
        }
    };

    const int t0 = blockIdx.x * a.per;
    int t1 = t0 + a.per;
    if (t1 > a.ntiles) t1 = a.ntiles;
    fetch(t0);   // (no workgroup is without a tile)
    int chain = 0;
    bool more = false;
    for (int tile = t0; tile < t1; ++tile) {
        if (tile > t0) __syncthreads();
        stage();
        __syncthreads();
        if (tile + 1 < t1) fetch(tile + 1);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int ZB = CBO == 2 ? 1 : 2;   // (a second set of 24 registers spills)
        bf16x8 af[ZB][NP][CBO], b[NBUF][3];
        auto zfrags = [&](int k) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int cb = 0; cb < CBO; ++cb) {
                    const char* q = PACK ? za + k * VG * 2048 + p * 32 : za + k * VG * 1024 + (p * CBO + cb) * (VOX * 32);
                    af[k % ZB][p][cb] = tr(q, q + (PACK ? 1024 : 512));
                }
        };
        auto xfrags = [&](int u) __attribute__((always_inline)) {
            int c = col[u % NB];
            asm volatile("" : "+v"(c));   // sums with the k-steps' offsets are not worth registers of their own
            const char *q = xs + (c + ko[u / NB]), *r = q + half;
#pragma unroll
            for (int p = 0; p < 3; ++p) b[u % NBUF][p] = tr(q + p * XP, r + p * XP);
        };
        zfrags(0);
#pragma unroll
        for (int u = 0; u < NBUF - 1; ++u) xfrags(u);
#pragma unroll
        for (int u = 0; u < NK * NB; ++u) {
            const int k = u / NB, i = u % NB;
            if (u + NBUF - 1 < NK * NB) xfrags(u + NBUF - 1);
            if (ZB == 2 && i == 0 && k + 1 < NK) zfrags(k + 1);
            constexpr int PZ[6] = {1, 2, 0, 1, 0, 0}, PX[6] = {1, 0, 2, 0, 1, 0};   // as in the forward pass
#pragma unroll
            for (int q = 0; q < (PACK ? 4 : 6); ++q)
#pragma unroll
                for (int cb = 0; cb < CBO; ++cb) {
                    const int pz_ = PACK ? (q == 1 ? 1 : 0) : PZ[q], px_ = PACK ? (q == 0 ? 2 : q == 2 ? 1 : 0) : PX[q];
                    f32x4& c = q == (PACK ? 3 : 5) ? acc[cb][i] : rest[cb][i];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[k % ZB][pz_][cb], b[u % NBUF][px_], c, 0, 0, 0);
                }
            if (ZB == 1 && i == NB - 1 && k + 1 < NK) zfrags(k + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (++chain == a.flush || tile + 1 == t1) {
            dump(more);
            clear();
            chain = 0;
            more = true;
        }
    }
}

constexpr int SPLITW_CHAIN = 32;
struct SplitWgradPlan { int cic, cbo, cichunks, cochunks, splits, per, vg; bool pack; int64_t ntiles; TileGeo t; };
static SplitWgradPlan split_wgrad_plan(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    SplitWgradPlan p;
    p.cic = xd->c > 8 ? 16 : 8;
    p.cbo = dzd->c > 16 ? 2 : 1;
    p.pack = dzd->c <= 8;
    p.cichunks = cdiv(xd->c, p.cic);
    p.cochunks = cdiv(dzd->c, 16 * p.cbo);
    p.vg = p.cic == 16 ? 1 : 2;
    const bool big = p.cic == 8 && p.cbo == 1;
    p.t = split_tile(xd->d, xd->h, xd->w, big ? 256 : 128, big ? 648 : 432);
    p.ntiles = (int64_t)xd->n * p.t.nd * p.t.nh * p.t.nw;
    // two workgroups fit a CU; the walks share the tiles evenly, and the partials stay under 64 MB
    int64_t s = 512 / ((int64_t)p.cichunks * p.cochunks);
    const int64_t cap = (int64_t)(16u << 20) / ((int64_t)p.vg * dzd->c * 27 * xd->c);
    if (s > cap) s = cap;
    if (s < 1) s = 1;
    if (s > p.ntiles) s = p.ntiles;
    p.per = (int)((p.ntiles + s - 1) / s);
    p.splits = (int)((p.ntiles + p.per - 1) / p.per);
    return p;
}
// Whole 16-byte pieces, offsets within 32 bits, and enough workgroups: with 16 inputs x 32 outputs two a CU (32->32 on 20^3 22.8 us with
// fp32 products, 24.4 here, on 30^3 36.1 and 35.9; 64->64 on 24^3 47.8 and 39.0), else 32 tiles (8->8 on 16^3 11.2 and 12.1 us, on
// 26 x 18 x 21 12.6 and 11.9).
bool split_wgrad_takes(const lamp_tensor_desc* xd, const void* x, const lamp_tensor_desc* dzd, const void* dz) {
    if (xd->dtype != LAMP_F32 || xd->c < 8 || xd->c % 4 || dzd->c % 4 || xd->ldc % 4 || dzd->ldc % 4 || !aligned16(x) || !aligned16(dz)) return false;
    const SplitWgradPlan p = split_wgrad_plan(xd, dzd);
    if (p.cic * p.cbo == 32 ? p.ntiles * p.cichunks * p.cochunks < 512 : p.ntiles < 32) return false;
    return p.ntiles < ((int64_t)1 << 31) && (int64_t)p.cichunks * p.cochunks <= 65535 &&
           (int64_t)xd->h * xd->w * 18 * (xd->ldc > dzd->ldc ? xd->ldc : dzd->ldc) < ((int64_t)1 << 29) &&   // byte offsets in a tile, in dw
           (int64_t)xd->c * dzd->c < ((int64_t)1 << 24);
}
size_t split_wgrad_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    if (xd->dtype != LAMP_F32) return 0;
    const SplitWgradPlan p = split_wgrad_plan(xd, dzd);
    return align_up((size_t)p.splits * p.vg * dzd->c * 27 * xd->c * sizeof(float));
}

template <int CIC, int CBO, bool PACK>
static lamp_status split_wgrad_launch(const SplitWgradPlan& p, hipStream_t s, const SplitWgradArgs& a) {
    typedef SplitWg<CIC, CBO> G;
    constexpr int lds = 3 * G::XP + (PACK ? G::VOX * 64 : 3 * CBO * G::VOX * 32);
    if (lds > 65536 && ensure_dyn_lds((const void*)conv3d_split_wgrad_kernel<CIC, CBO, PACK>, lds) != LAMP_OK) return LAMP_ERR_HIP;
    hipLaunchKernelGGL((conv3d_split_wgrad_kernel<CIC, CBO, PACK>), dim3(p.splits, p.cichunks * p.cochunks), dim3(256), lds, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

lamp_status split_wgrad(const lamp_tensor_desc* xd, const float* x, const NormIn& nm, const lamp_tensor_desc* dzd, const float* dz,
                        float* dw, float beta, void* ws, size_t ws_bytes, hipStream_t s) {
    const SplitWgradPlan p = split_wgrad_plan(xd, dzd);
    if (!ws || ws_bytes < split_wgrad_ws_bytes(xd, dzd)) return LAMP_ERR_WORKSPACE;
    SplitWgradArgs a;
    a.x = x; a.dz = dz; a.part = (float*)ws; a.nm = nm;
    a.ldx = xd->ldc; a.lddz = dzd->ldc;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = dzd->c;
    a.t = p.t; a.ntiles = (int)p.ntiles; a.per = p.per; a.cochunks = p.cochunks;
    a.flush = SPLITW_CHAIN;
    a.mHW = (65536 + (1 << p.t.lw) + 1) / ((1 << p.t.lw) + 2);
    a.mHH = (65536 + (1 << p.t.lh) + 1) / ((1 << p.t.lh) + 2);
    div_magic(p.t.nd * p.t.nh * p.t.nw, &a.mT, &a.sT);
    div_magic(p.t.nw, &a.mNw, &a.sNw);
    div_magic(p.t.nh, &a.mNh, &a.sNh);
    lamp_status st;
    if (p.cic == 16) st = p.pack ? split_wgrad_launch<16, 1, true>(p, s, a) : p.cbo == 1 ? split_wgrad_launch<16, 1, false>(p, s, a)
                                                                                        : split_wgrad_launch<16, 2, false>(p, s, a);
    else st = p.pack ? split_wgrad_launch<8, 1, true>(p, s, a) : p.cbo == 1 ? split_wgrad_launch<8, 1, false>(p, s, a)
                                                                           : split_wgrad_launch<8, 2, false>(p, s, a);
    if (st != LAMP_OK) return st;
    return launch_reduce_partials((const float*)ws, p.splits * p.vg, (int64_t)dzd->c * 27 * xd->c, dw, beta, s);
}

}  // namespace lamp
