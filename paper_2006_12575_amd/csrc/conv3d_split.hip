// Data gradient of the 3x3x3 convolution of fp32 tensors on the bf16 matrix instructions.
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

}  // namespace lamp
