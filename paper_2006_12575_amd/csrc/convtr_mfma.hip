// Matrix-core kernels for the 2x2x2 stride-2 transposed convolution (bf16, fp32 accumulate).
//
// Every output voxel depends on one input voxel and one tap, so forward and data gradient are plain
// GEMMs over voxels with a gather / scatter to the 2x2x2 sub-positions:
//   forward : Y[(tap,co)][v] = sum_ci  Wt'[(tap,co)][ci] * X[v][ci]        -> y[up(v,tap)][co]
//   dgrad   : DX[ci][v]      = sum_{(tap,co)} Wt[ci][(tap,co)] * DY[up(v,tap)][co]
// Operands are read straight from global memory into MFMA fragments (16 contiguous bytes per lane:
// the weights are small and cache-resident, the activations are streamed once); the op is bound by
// writing / reading the fine-resolution tensor, not by the matrix cores.
// The weight gradient has voxels as its reduction dimension and reads both operands through LDS with
// the transposing load, like the 3x3x3 weight gradient.
#include <stdlib.h>
#include "internal.h"
#include "vec.h"

namespace lamp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

struct CtArgs {
    const bf16_t* a;      // row-major A[rows][K]
    const bf16_t* b;      // activations (x for forward, dy for dgrad)
    bf16_t* out;
    const float* bias;    // forward only, [Co] or nullptr
    int rows, K;
    int N, D, H, W;       // coarse (input-resolution) dims
    int Ci, Co;
    int ldb, ldo;         // channel strides of b and out
    uint32_t mW, mH, mD;  // v / d == (v * m) >> s for v < 2^31 (div_magic)
    int sW, sH, sD;
};

// wt'[(tap*Co + co)][ci] = wt[ci][tap][co]
__global__ __launch_bounds__(256) void convtr_repack_kernel(const bf16_t* __restrict__ wt, bf16_t* __restrict__ wp, int Ci,
                                                            int Co) {
    const int64_t total = (int64_t)Ci * 8 * Co;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int ci = (int)(i % Ci);
    const int r = (int)(i / Ci);  // tap*Co + co
    wp[i] = wt[(int64_t)ci * 8 * Co + r];
}

__device__ __forceinline__ bf16x8 gfrag(const bf16_t* p, bool ok) {
    uint4 q = make_uint4(0, 0, 0, 0);
    if (ok) q = *reinterpret_cast<const uint4*>(p);
    return __builtin_bit_cast(bf16x8, q);
}

// MODE 0: forward, MODE 1: data gradient.  One wave = 64 coarse voxels x up to 128 rows.
template <int MODE>
__global__ __launch_bounds__(256) void convtr_gemm_kernel(CtArgs a) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int64_t nvox = (int64_t)a.N * a.D * a.H * a.W;
    const int64_t v0 = ((int64_t)blockIdx.x * 4 + wv) * 64;
    if (v0 >= nvox) return;
    const int r0 = blockIdx.y * 128;
    const int nrb = min(4, (a.rows - r0 + 31) / 32);

    // the lane's two voxels (column j of voxel blocks 0 and 1) and their fine-resolution origin
    int64_t vq[2], fine[2];
    bool vok[2];
#pragma unroll
    for (int vb = 0; vb < 2; ++vb) {
        const int64_t v = v0 + vb * 32 + l32;
        vok[vb] = v < nvox;
        const int64_t vc = vok[vb] ? v : 0;
        const int w = (int)(vc % a.W);
        int64_t r = vc / a.W;
        const int h = (int)(r % a.H);
        r /= a.H;
        const int d = (int)(r % a.D);
        const int n = (int)(r / a.D);
        vq[vb] = vc;
        fine[vb] = (((int64_t)n * 2 * a.D + 2 * d) * 2 * a.H + 2 * h) * 2 * a.W + 2 * w;  // voxel (2d,2h,2w)
    }
    auto tap_off = [&](int tap) -> int64_t {
        const int i = tap >> 2, j = (tap >> 1) & 1, k = tap & 1;
        return ((int64_t)i * 2 * a.H + j) * 2 * a.W + k;
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int vb = 0; vb < 2; ++vb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][vb][r] = 0.f;

    for (int k0 = 0; k0 < a.K; k0 += 16) {
        const int k = k0 + 8 * half;
        bf16x8 bf[2], af[4];
        if (MODE == 0) {
#pragma unroll
            for (int vb = 0; vb < 2; ++vb) bf[vb] = gfrag(a.b + vq[vb] * a.ldb + k, vok[vb]);
        } else {
            const int tap = k / a.Co, co = k - tap * a.Co;
            const int64_t to = tap_off(tap);
#pragma unroll
            for (int vb = 0; vb < 2; ++vb) bf[vb] = gfrag(a.b + (fine[vb] + to) * a.ldb + co, vok[vb]);
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const int row = r0 + rb * 32 + l32;
            af[rb] = gfrag(a.a + (int64_t)row * a.K + k, rb < nrb && row < a.rows);
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int vb = 0; vb < 2; ++vb)
                if (rb < nrb) acc[rb][vb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb], bf[vb], acc[rb][vb], 0, 0, 0);
    }

    // lane holds, for its voxel of each block, rows r0 + rb*32 + 8*(r/4) + 4*half + (r%4)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
        if (rb >= nrb) continue;
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const int row = r0 + rb * 32 + rg * 8 + half * 4;
            if (row >= a.rows) continue;
#pragma unroll
            for (int vb = 0; vb < 2; ++vb) {
                if (!vok[vb]) continue;
                uint32_t pk[2];
                if (MODE == 0) {
                    const int tap = row / a.Co, co = row - tap * a.Co;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float b0 = a.bias ? a.bias[co + 2 * e] : 0.f, b1 = a.bias ? a.bias[co + 2 * e + 1] : 0.f;
                        pk[e] = f2bf2(acc[rb][vb][rg * 4 + 2 * e] + b0, acc[rb][vb][rg * 4 + 2 * e + 1] + b1);
                    }
                    *reinterpret_cast<uint2*>(a.out + (fine[vb] + tap_off(tap)) * a.ldo + co) = make_uint2(pk[0], pk[1]);
                } else {
#pragma unroll
                    for (int e = 0; e < 2; ++e) pk[e] = f2bf2(acc[rb][vb][rg * 4 + 2 * e], acc[rb][vb][rg * 4 + 2 * e + 1]);
                    *reinterpret_cast<uint2*>(a.out + vq[vb] * a.ldo + row) = make_uint2(pk[0], pk[1]);
                }
            }
        }
    }
}


// ------------------------------------------------------------------------------------------------
// Kernels for channel counts that are multiples of 32: the fine-resolution tensor is written
// (forward) and read (data gradient) in whole 64-byte pieces -- 32 channels of one fine voxel, four
// lanes of 16 bytes side by side -- instead of one 8-byte piece per lane.  A per-wave LDS buffer
// transposes between that memory order and the matrix-core fragment order; only the owning wave
// touches its buffer, so no workgroup barrier is needed.

static constexpr int CT_ROW = 80;  // bytes per voxel row in the transposing buffer: 64 of data, padded

// fine-resolution voxel (2d,2h,2w) of coarse voxel v (v < 2^31)
__device__ __forceinline__ uint32_t ct_div(uint32_t v, uint32_t m, int sh) { return (uint32_t)(((uint64_t)v * m) >> sh); }
__device__ __forceinline__ int64_t ct_fine_origin(const CtArgs& a, int64_t v) {
    const uint32_t vi = (uint32_t)v;
    uint32_t r = ct_div(vi, a.mW, a.sW);
    const uint32_t w = vi - r * (uint32_t)a.W;
    uint32_t r2 = ct_div(r, a.mH, a.sH);
    const uint32_t h = r - r2 * (uint32_t)a.H;
    const uint32_t n = ct_div(r2, a.mD, a.sD);
    const uint32_t d = r2 - n * (uint32_t)a.D;
    return (((int64_t)n * 2 * a.D + 2 * d) * 2 * a.H + 2 * h) * 2 * a.W + 2 * w;
}
__device__ __forceinline__ int64_t ct_tap_off(const CtArgs& a, int tap) {
    return ((int64_t)(tap >> 2) * 2 * a.H + ((tap >> 1) & 1)) * 2 * a.W + (tap & 1);
}

// Forward.  One wave = VB*32 coarse voxels x one block of RB units (a unit is (tap, 32 output
// channels) = 32 rows of the repacked weight).  For the input channel counts and the weights off 16 bytes that the
// kernel with the weights in LDS does not take.  Every load of a wave is issued before its first store:
// loads and stores complete in one queue, so a load behind a store would wait for the store; the
// bias therefore sits in LDS.  Requires Co % 32 == 0, Co <= 256 * 4, Ci % 16 == 0, < 2^31 voxels.
template <int RB, int VB>
__global__ __launch_bounds__(256) void convtr_fwd32_kernel(CtArgs a) {
    constexpr int VW = 32 * VB;  // voxels per wave
    __shared__ __attribute__((aligned(16))) char tb[4][VW * CT_ROW];
    __shared__ __attribute__((aligned(16))) float bsh[4][1024];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int64_t nvox = (int64_t)a.N * a.D * a.H * a.W;
    const int K = a.K;
    // workgroup id -> (voxel group, row block): ids are dealt round-robin to the 8 XCDs, so the row
    // blocks of one voxel group take consecutive slots of ONE XCD and share its L2 for x
    const int nblocks = a.rows / (32 * RB);
    const uint32_t xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
    const int yb = (int)(slot % (uint32_t)nblocks);
    const int64_t vg = (int64_t)(slot / (uint32_t)nblocks) * 8 + xcd;
    const int64_t v0 = (vg * 4 + wv) * VW;
    if (v0 >= nvox) return;
    const int r0 = yb * (32 * RB);

    const bf16_t* xrow[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        int64_t v = v0 + vb * 32 + l32;  // columns past the end repeat the last voxel and are never stored
        if (v >= nvox) v = nvox - 1;
        xrow[vb] = a.b + v * a.ldb + 8 * half;
    }
    const bf16_t* arow = a.a + (int64_t)(r0 + l32) * K + 8 * half;
    // bias -> this wave's LDS copy
    for (int c = lane * 4; c < a.Co; c += 256) {
        float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.bias) bv = make_float4(a.bias[c], a.bias[c + 1], a.bias[c + 2], a.bias[c + 3]);
        *reinterpret_cast<float4*>(&bsh[wv][c]) = bv;
    }
    // the voxels this lane stores: 16 per pass, four lanes per voxel
    int64_t fs[2 * VB];
#pragma unroll
    for (int it = 0; it < 2 * VB; ++it) {
        const int64_t v = v0 + it * 16 + (lane >> 2);
        fs[it] = v < nvox ? ct_fine_origin(a, v) : -1;
    }

    f32x16 acc[RB][VB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int vb = 0; vb < VB; ++vb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][vb][r] = 0.f;

    // streaming reduction, operands fetched one step ahead
    bf16x8 bfn[VB], afn[RB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) bfn[vb] = *reinterpret_cast<const bf16x8*>(xrow[vb]);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) afn[rb] = *reinterpret_cast<const bf16x8*>(arow + (int64_t)rb * 32 * K);
    for (int k0 = 0; k0 < K; k0 += 16) {
        bf16x8 bf[VB], af[RB];
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) bf[vb] = bfn[vb];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) af[rb] = afn[rb];
        if (k0 + 16 < K) {
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) bfn[vb] = *reinterpret_cast<const bf16x8*>(xrow[vb] + k0 + 16);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) afn[rb] = *reinterpret_cast<const bf16x8*>(arow + (int64_t)rb * 32 * K + k0 + 16);
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int vb = 0; vb < VB; ++vb)
                acc[rb][vb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb], bf[vb], acc[rb][vb], 0, 0, 0);
    }

    // lane holds, for voxel l32 of block vb, rows 8*(r/4) + 4*half + (r%4) of the unit
    char* mine = tb[wv];
    const int cpt = a.Co >> 5;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int unit = (r0 >> 5) + rb;
        const int tap = unit / cpt, co0 = (unit - tap * cpt) << 5;
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const int c = rg * 8 + half * 4;
            const float4 bv = *reinterpret_cast<const float4*>(&bsh[wv][co0 + c]);
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) {
                const uint2 pk = make_uint2(f2bf2(acc[rb][vb][rg * 4 + 0] + bv.x, acc[rb][vb][rg * 4 + 1] + bv.y),
                                            f2bf2(acc[rb][vb][rg * 4 + 2] + bv.z, acc[rb][vb][rg * 4 + 3] + bv.w));
                *reinterpret_cast<uint2*>(mine + (vb * 32 + l32) * CT_ROW + c * 2) = pk;
            }
        }
        __builtin_amdgcn_wave_barrier();
        const int64_t to = ct_tap_off(a, tap);
#pragma unroll
        for (int it = 0; it < 2 * VB; ++it) {
            const uint4 q = *reinterpret_cast<const uint4*>(mine + (it * 16 + (lane >> 2)) * CT_ROW + (lane & 3) * 16);
            if (fs[it] >= 0) *reinterpret_cast<uint4*>(a.out + (fs[it] + to) * a.ldo + co0 + (lane & 3) * 8) = q;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Forward with the weights in LDS, for 16, 32, 64 and 128 input channels.  The rows (tap, output channel) are cut into pairs of 32-row
// units; a workgroup keeps up to four pairs (K = 16 * KS deep, transposed from the public layout on the way in) and its 8 waves walk
// groups of 32 coarse voxels, the next group's x in flight during the current one's multiplies and stores.  A pair is 64 consecutive
// rows, 128 bytes of output a voxel: with 32 output channels the two taps of a w pair, which lie side by side in memory, so a store
// instruction covers 1 KB of consecutive bytes where a unit at a time wrote every other 64 bytes.
// Bound: HBM.  64->32 on 2 x 64^3 (67 MB in, 268 MB out): 106 us with a wave per 32 voxels x 8 units, weights from the caches,
// and a repacking launch in front -> 58 us.  Same products in the same order as convtr_fwd32_kernel.
// Requires Co % 8 == 0, whole 16-byte pieces everywhere, tap offsets in 32 bits, fine voxels in 32 bits.
static constexpr int CT_PROW = 144;                        // patch: 128 bytes a voxel, padded
static constexpr int CT_PATCH = 32 * CT_PROW + 128;        // and the 32 voxels' fine origins
static size_t ct_fwd_lds(int pb, int ks) { return (size_t)pb * (2 * ks * 1024 + 256 + 32) + 8 * CT_PATCH; }

template <int KS, bool NT>
__global__ __launch_bounds__(512, KS <= 4 ? 4 : 2) void convtr_fwd_lds_kernel(CtArgs a) {
    extern __shared__ __attribute__((aligned(16))) char ctl[];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, half = lane >> 5;
    const int pairs = a.rows >> 6, nblocks = (pairs + 3) >> 2;
    // row blocks of the same voxel groups take consecutive slots of one XCD and share its L2 for x
    const int slot = (int)blockIdx.x >> 3, yb = slot % nblocks, walker = slot / nblocks * 8 + ((int)blockIdx.x & 7);
    const int walkers = (int)gridDim.x / nblocks;
    const int p0 = yb * 4, pb = min(4, pairs - p0);
    char* const wl = ctl;                                                  // [unit][ks][half][32 rows][8 channels]
    float* const bl = reinterpret_cast<float*>(ctl + pb * (2 * KS * 1024));  // bias of every row
    int* const po = reinterpret_cast<int*>(bl + pb * 64);                  // output offset of every 8-row piece
    char* const patch = reinterpret_cast<char*>(po + pb * 8) + wv * CT_PATCH;
    uint32_t* const org = reinterpret_cast<uint32_t*>(patch + 32 * CT_PROW);

    const uint32_t nvox = (uint32_t)((int64_t)a.N * a.D * a.H * a.W), ngroups = (nvox + 31) >> 5, step = (uint32_t)walkers * 8;
    uint32_t g = (uint32_t)walker * 8 + wv;
    auto voxel = [&](uint32_t grp) { return min(grp * 32 + l32, nvox - 1); };   // lanes past the end repeat the last voxel, same value
    bf16x8 nx[KS];
    auto fetch = [&](uint32_t grp) __attribute__((always_inline)) {
        const bf16_t* p = a.b + (int64_t)voxel(grp) * a.ldb + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) nx[ks] = *reinterpret_cast<const bf16x8*>(p + ks * 16);
    };
    if (g < ngroups) fetch(g);

    // weights: eight pieces of 8 rows, one per input channel, to eight pieces of 8 input channels
    for (int i = tid; i < pb * 8 * 2 * KS; i += 512) {
        const int rp = i % (pb * 8), kb = i / (pb * 8);
        const bf16_t* src = a.a + (int64_t)(kb * 8) * a.rows + p0 * 64 + rp * 8;
        vec_u32x4 q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = *reinterpret_cast<const vec_u32x4*>(src + (int64_t)e * a.rows);
        char* dst = wl + (((rp >> 2) * KS + (kb >> 1)) * 2 + (kb & 1)) * 512 + (rp & 3) * 128;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            vec_u32x4 o;
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = __builtin_amdgcn_perm(q[2 * d + 1][j >> 1], q[2 * d][j >> 1], j & 1 ? 0x07060302u : 0x05040100u);
            *reinterpret_cast<vec_u32x4*>(dst + j * 16) = o;
        }
    }
    for (int i = tid; i < pb * 64; i += 512) bl[i] = a.bias ? a.bias[(p0 * 64 + i) % a.Co] : 0.f;
    for (int i = tid; i < pb * 8; i += 512) {
        const int row = (p0 * 8 + i) * 8, tap = row / a.Co, co = row - tap * a.Co;
        po[i] = (int)ct_tap_off(a, tap) * a.ldo + co;
    }
    __syncthreads();

    for (; g < ngroups; g += step) {
        bf16x8 cx[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) cx[ks] = nx[ks];
        fetch(g + step < ngroups ? g + step : g);
        if (lane < 32) org[l32] = (uint32_t)ct_fine_origin(a, voxel(g));
        __builtin_amdgcn_wave_barrier();
        bf16_t* op[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) op[it] = a.out + (int64_t)org[it * 8 + (lane >> 3)] * a.ldo;
        for (int m = 0; m < pb; ++m) {
            f32x16 acc[2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
            const char* wp = wl + m * (2 * KS * 1024) + half * 512 + l32 * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(wp + (u * KS + ks) * 1024), cx[ks],
                                                                     acc[u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const int c = u * 32 + rg * 8 + half * 4;
                    const float4 bv = *reinterpret_cast<const float4*>(bl + m * 64 + c);
                    *reinterpret_cast<uint2*>(patch + l32 * CT_PROW + c * 2) =
                        make_uint2(f2bf2(acc[u][rg * 4 + 0] + bv.x, acc[u][rg * 4 + 1] + bv.y),
                                   f2bf2(acc[u][rg * 4 + 2] + bv.z, acc[u][rg * 4 + 3] + bv.w));
                }
            __builtin_amdgcn_wave_barrier();
            const int off = po[m * 8 + (lane & 7)];
#pragma unroll
            for (int it = 0; it < 4; ++it)
                st16<NT>(op[it] + off, *reinterpret_cast<const vec_u32x4*>(patch + (it * 8 + (lane >> 3)) * CT_PROW + (lane & 7) * 16));
            __builtin_amdgcn_wave_barrier();
        }
    }
}
template <int KS>
static lamp_status ct_fwd_lds_launch(const CtArgs& a, int64_t nv, hipStream_t s) {
    const int pairs = a.rows / 64, nblocks = (pairs + 3) / 4, pb = pairs < 4 ? pairs : 4;
    const size_t lds = ct_fwd_lds(pb, KS);
    // as many workgroups as are resident at a time, fewer where the volume has fewer groups
    const int per_cu = KS <= 4 ? 2 : 1;
    int64_t walkers = 256 * per_cu / nblocks;   // 0 where the row blocks alone are more than are resident
    if (walkers > cdiv(nv, 256)) walkers = cdiv(nv, 256);
    if (walkers < 1) walkers = 1;
    walkers = (walkers + 7) / 8 * 8;
    const dim3 grid((unsigned)(walkers * nblocks));
    const bool nt = beyond_cache(nv * (a.Ci + 8 * (int64_t)a.Co) * 2);
    if (nt) {
        if (ensure_dyn_lds((const void*)convtr_fwd_lds_kernel<KS, true>, (int)ct_fwd_lds(4, KS)) != LAMP_OK) return LAMP_ERR_HIP;
        hipLaunchKernelGGL((convtr_fwd_lds_kernel<KS, true>), grid, dim3(512), lds, s, a);
    } else {
        if (ensure_dyn_lds((const void*)convtr_fwd_lds_kernel<KS, false>, (int)ct_fwd_lds(4, KS)) != LAMP_OK) return LAMP_ERR_HIP;
        hipLaunchKernelGGL((convtr_fwd_lds_kernel<KS, false>), grid, dim3(512), lds, s, a);
    }
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

// Data gradient.  One wave = 64 coarse voxels x RB blocks of 32 input channels; the reduction runs
// over units of (tap, 32 output channels), in this order whatever RB is.  The 64-byte pieces of dy are gathered PF units ahead
// into registers and handed to the matrix-core fragment order through the wave's double buffer.
// PF = 4, RB = 1, a wave to a workgroup: for small volumes, which have few voxel groups and, deep in the net, many units, whose gathers
// one unit ahead were one chain of memory latencies (512->256 on 2 x 8^3, forward and backward: 138 -> 77 us with the forward's part of it;
// 256->128 on 2 x 16^3 96 -> 78).  Four waves with a quarter of the units each were no faster (75 and 86 us) and rounded some elements
// of dx the other way, which the bf16 layers below amplified: 4e-3 in the deepest weight gradients of the 5-level base-32 net.
// Requires Co % 32 == 0, Ci % 32 == 0.
template <int RB, int PF = 1>
__global__ __launch_bounds__(PF > 1 ? 64 : 256) void convtr_dgrad32_kernel(CtArgs a) {
    constexpr int WV = PF > 1 ? 1 : 4;
    __shared__ __attribute__((aligned(16))) char tb[WV][2][64 * CT_ROW];
    const int lane = threadIdx.x & 63, wv = WV > 1 ? threadIdx.x >> 6 : 0;
    const int l32 = lane & 31, half = lane >> 5;
    const int64_t nvox = (int64_t)a.N * a.D * a.H * a.W;
    const int64_t v0 = ((int64_t)blockIdx.x * WV + wv) * 64;
    if (v0 >= nvox) return;
    const int r0 = blockIdx.y * (32 * RB);
    const int nrb = min(RB, (a.rows - r0) >> 5);

    int64_t fs[4], vs[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        vs[it] = v0 + it * 16 + (lane >> 2);
        fs[it] = ct_fine_origin(a, vs[it] < nvox ? vs[it] : nvox - 1);   // past the end: the last voxel again, not stored
    }
    const bf16_t* arow = a.a + (int64_t)(r0 + l32) * a.K + 8 * half;
    const int cpt = a.Co >> 5, units = 8 * cpt;

    f32x16 acc[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int vb = 0; vb < 2; ++vb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][vb][r] = 0.f;

    auto multiply = [&](const char* cur, const bf16x8 (&af)[RB], int ks) __attribute__((always_inline)) {
        bf16x8 bf[2];
#pragma unroll
        for (int vb = 0; vb < 2; ++vb)
            bf[vb] = *reinterpret_cast<const bf16x8*>(cur + (vb * 32 + l32) * CT_ROW + ks * 32 + half * 16);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int vb = 0; vb < 2; ++vb)
                acc[rb][vb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb], bf[vb], acc[rb][vb], 0, 0, 0);
    };
    if constexpr (PF > 1) {
        static_assert(RB == 1 && 8 % PF == 0, "the units are a multiple of 8");
        vec_u32x4 q[PF][4];   // (vectors, and loads without a branch: nothing is taken apart behind a wait)
        bf16x8 af[PF][2][1];
        const bf16_t* src[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) src[it] = a.b + fs[it] * a.ldb + (lane & 3) * 8;
        auto fetch = [&](int u, int p) __attribute__((always_inline)) {
            const int tap = u / cpt;
            const int64_t o = ct_tap_off(a, tap) * a.ldb + ((u - tap * cpt) << 5);
#pragma unroll
            for (int it = 0; it < 4; ++it) q[p][it] = *reinterpret_cast<const vec_u32x4*>(src[it] + o);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) af[p][ks][0] = *reinterpret_cast<const bf16x8*>(arow + u * 32 + ks * 16);
        };
#pragma unroll
        for (int p = 0; p < PF; ++p) fetch(p, p);
#pragma unroll 1
        for (int u = 0; u < units; u += PF)
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                char* cur = tb[wv][p & 1];
#pragma unroll
                for (int it = 0; it < 4; ++it)
                    *reinterpret_cast<vec_u32x4*>(cur + (it * 16 + (lane >> 2)) * CT_ROW + (lane & 3) * 16) = q[p][it];
                __builtin_amdgcn_wave_barrier();
                multiply(cur, af[p][0], 0);
                multiply(cur, af[p][1], 1);
                fetch(u + p + PF < units ? u + p + PF : u + p, p);   // the last ones again: no branch
                __builtin_amdgcn_wave_barrier();
            }
    } else {
        auto gather = [&](int u, vec_u32x4 (&q)[4]) __attribute__((always_inline)) {
            const int tap = u / cpt, c0 = (u - tap * cpt) << 5;
            const int64_t to = ct_tap_off(a, tap);
#pragma unroll
            for (int it = 0; it < 4; ++it) q[it] = *reinterpret_cast<const vec_u32x4*>(a.b + (fs[it] + to) * a.ldb + c0 + (lane & 3) * 8);
        };
        auto put = [&](char* buf, const vec_u32x4 (&q)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int it = 0; it < 4; ++it) *reinterpret_cast<vec_u32x4*>(buf + (it * 16 + (lane >> 2)) * CT_ROW + (lane & 3) * 16) = q[it];
        };
        vec_u32x4 q[4];
        gather(0, q);
        put(tb[wv][0], q);
        __builtin_amdgcn_wave_barrier();
        // No branch in the loop, which would make every wait one for all loads: past the last unit the last one again, past the last block
        // of rows its weights again, whose products are not stored.
        for (int u = 0; u < units; ++u) {
            // the unit's weights in front of the next unit's dy: loads return in order, and a weight behind dy would wait for it
            bf16x8 af[2][RB];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) af[ks][rb] = *reinterpret_cast<const bf16x8*>(arow + (int64_t)min(rb, nrb - 1) * 32 * a.K + u * 32 + ks * 16);
            __builtin_amdgcn_sched_barrier(0);
            gather(u + 1 < units ? u + 1 : u, q);
            __builtin_amdgcn_sched_barrier(0);
            const char* cur = tb[wv][u & 1];
            multiply(cur, af[0], 0);
            multiply(cur, af[1], 1);
            put(tb[wv][(u + 1) & 1], q);
            __builtin_amdgcn_wave_barrier();
        }
    }

    char* mine = tb[wv][0];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (rb >= nrb) break;
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
            for (int vb = 0; vb < 2; ++vb) {
                const uint2 pk = make_uint2(f2bf2(acc[rb][vb][rg * 4 + 0], acc[rb][vb][rg * 4 + 1]),
                                            f2bf2(acc[rb][vb][rg * 4 + 2], acc[rb][vb][rg * 4 + 3]));
                *reinterpret_cast<uint2*>(mine + (vb * 32 + l32) * CT_ROW + (rg * 8 + half * 4) * 2) = pk;
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const uint4 o = *reinterpret_cast<const uint4*>(mine + (it * 16 + (lane >> 2)) * CT_ROW + (lane & 3) * 16);
            if (vs[it] < nvox) *reinterpret_cast<uint4*>(a.out + vs[it] * a.ldo + r0 + rb * 32 + (lane & 3) * 8) = o;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

static void ct_set_magic(CtArgs& a) {
    div_magic(a.W, &a.mW, &a.sW);
    div_magic(a.H, &a.mH, &a.sH);
    div_magic(a.D, &a.mD, &a.sD);
}

// 32 rows per wave when the volume is small (more workgroups), up to 128 otherwise (measured: from 32768
// voxels on the fewer re-reads of dy win)
static constexpr int64_t CT_SMALL = 32768;
static int ct_row_blocks(int64_t nv, int rows) {
    if (nv < CT_SMALL) return 1;
    return rows >= 128 ? 4 : (rows >= 64 ? 2 : 1);
}

bool mfma_convtr_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* yd, const lamp_norm_in* xnorm) {
    if (xd->dtype != LAMP_BF16) return false;
    if (xnorm && xnorm->mean_rstd && xnorm->c_norm > 0) return false;
    if (xd->c % 16 || yd->c % 8 || xd->ldc % 8 || yd->ldc % 4) return false;
    return true;
}

size_t mfma_convtr_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* yd) {
    if (!mfma_convtr_supported(xd, yd, nullptr)) return 0;
    return align_up((size_t)xd->c * 8 * yd->c * 2);
}

lamp_status mfma_convtr_fwd(const lamp_tensor_desc* xd, const void* x, const void* wt, const float* bias,
                            const lamp_tensor_desc* yd, void* y, void* ws, size_t ws_bytes, hipStream_t s) {
    if ((((uintptr_t)x) & 15u) || (((uintptr_t)y) & 7u) || (((uintptr_t)ws) & 15u)) return LAMP_ERR_ALIGN;
    if (ws_bytes < mfma_convtr_ws_bytes(xd, yd)) return LAMP_ERR_WORKSPACE;
    const int Ci = xd->c, Co = yd->c;
    if ((Ci == 16 || Ci == 32 || Ci == 64 || Ci == 128) && yd->ldc % 8 == 0 && aligned16(y) && aligned16(wt) &&
        nvox(xd) < ((int64_t)1 << 29) && ((int64_t)2 * yd->h * yd->w + 2 * yd->w) * yd->ldc < ((int64_t)1 << 31)) {
        CtArgs a;
        a.a = (const bf16_t*)wt; a.b = (const bf16_t*)x; a.out = (bf16_t*)y; a.bias = bias; a.rows = 8 * Co; a.K = Ci;
        a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = Ci; a.Co = Co; a.ldb = xd->ldc; a.ldo = yd->ldc;
        ct_set_magic(a);
        const int64_t nv = nvox(xd);
        return Ci == 16 ? ct_fwd_lds_launch<1>(a, nv, s) : Ci == 32 ? ct_fwd_lds_launch<2>(a, nv, s) : Ci == 64 ? ct_fwd_lds_launch<4>(a, nv, s)
                        : ct_fwd_lds_launch<8>(a, nv, s);
    }
    bf16_t* wp = (bf16_t*)ws;
    hipLaunchKernelGGL(convtr_repack_kernel, dim3(cdiv((int64_t)Ci * 8 * Co, 256)), dim3(256), 0, s, (const bf16_t*)wt, wp, Ci, Co);
    LAMP_CHECK_LAUNCH();
    CtArgs a;
    a.a = wp; a.b = (const bf16_t*)x; a.out = (bf16_t*)y; a.bias = bias; a.rows = 8 * Co; a.K = Ci;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = Ci; a.Co = Co; a.ldb = xd->ldc; a.ldo = yd->ldc;
    if (Co % 32 == 0 && Co <= 1024 && yd->ldc % 8 == 0 && ((((uintptr_t)y) & 15u) == 0) && nvox(xd) < ((int64_t)1 << 31)) {
        const int64_t nv = nvox(xd);
        ct_set_magic(a);
        if (Ci >= 256 && (int64_t)cdiv(nv, 256) * (a.rows / 256) >= 128) {
            // many input channels and enough voxels for a workgroup to every other CU (512->256 on 75 x 4^3, 152 workgroups, forward and
            // backward: 170 us so, 194 with a unit a wave; on 2 x 8^3, 32 workgroups: 98 and 78): a wave takes 64 voxels x 8 units (16 accumulator tiles), so that every weight
            // fragment fetched from the cache feeds two matrix-core instructions and the row blocks re-read x less
            dim3 grid((unsigned)(cdiv(cdiv(nv, 256), 8) * 8 * (a.rows / 256)));
            hipLaunchKernelGGL((convtr_fwd32_kernel<8, 2>), grid, dim3(256), 0, s, a);
        } else if (nv >= 65536) {
            // a wave = 32 voxels x 8 units: for Co = 32 it writes all eight taps of its voxels
            const int64_t groups8 = cdiv(cdiv(nv, 128), 8) * 8;  // voxel groups, padded to whole XCD rounds
            dim3 grid((unsigned)(groups8 * (a.rows / 256)));
            hipLaunchKernelGGL((convtr_fwd32_kernel<8, 1>), grid, dim3(256), 0, s, a);
        } else {
            const int64_t groups8 = cdiv(cdiv(nv, 256), 8) * 8;
            dim3 grid((unsigned)(groups8 * (a.rows / 32)));
            hipLaunchKernelGGL((convtr_fwd32_kernel<1, 2>), grid, dim3(256), 0, s, a);
        }
        LAMP_CHECK_LAUNCH();
        return LAMP_OK;
    }
    dim3 grid(cdiv(nvox(xd), 256), cdiv(a.rows, 128));
    hipLaunchKernelGGL((convtr_gemm_kernel<0>), grid, dim3(256), 0, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

bool mfma_convtr_dgrad_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd, const lamp_tensor_desc* dxd) {
    if (xd->dtype != LAMP_BF16) return false;
    if (xd->c % 4 || dyd->c % 8 || dyd->ldc % 8 || dxd->ldc % 4) return false;
    return true;
}

lamp_status mfma_convtr_dgrad(const lamp_tensor_desc* xd, const void* wt, const lamp_tensor_desc* dyd, const void* dy,
                              const lamp_tensor_desc* dxd, void* dx, hipStream_t s) {
    if ((((uintptr_t)dy) & 15u) || (((uintptr_t)dx) & 7u) || (((uintptr_t)wt) & 15u)) return LAMP_ERR_ALIGN;
    CtArgs a;
    a.a = (const bf16_t*)wt; a.b = (const bf16_t*)dy; a.out = (bf16_t*)dx; a.bias = nullptr; a.rows = xd->c; a.K = 8 * dyd->c;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = dyd->c; a.ldb = dyd->ldc; a.ldo = dxd->ldc;
    if (a.Co % 32 == 0 && a.Ci % 32 == 0 && dyd->ldc % 8 == 0 && dxd->ldc % 8 == 0 && ((((uintptr_t)dx) & 15u) == 0) &&
        nvox(xd) < ((int64_t)1 << 31)) {
        ct_set_magic(a);
        const int rb = ct_row_blocks(nvox(xd), a.rows);
        dim3 grid(cdiv(nvox(xd), 256), cdiv(a.rows, 32 * rb));
        if (nvox(xd) < CT_SMALL) hipLaunchKernelGGL((convtr_dgrad32_kernel<1, 4>), dim3(cdiv(nvox(xd), 64), grid.y), dim3(64), 0, s, a);
        else if (rb == 4) hipLaunchKernelGGL((convtr_dgrad32_kernel<4>), grid, dim3(256), 0, s, a);
        else if (rb == 2) hipLaunchKernelGGL((convtr_dgrad32_kernel<2>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((convtr_dgrad32_kernel<1>), grid, dim3(256), 0, s, a);
        LAMP_CHECK_LAUNCH();
        return LAMP_OK;
    }
    dim3 grid(cdiv(nvox(xd), 256), cdiv(a.rows, 128));
    hipLaunchKernelGGL((convtr_gemm_kernel<1>), grid, dim3(256), 0, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

// ------------------------------------------------------------------------------------------------
// Weight gradient  dWt[ci][tap][co] = sum_v x[v][ci] * dy[up(v,tap)][co]   (K = coarse voxels).
// Workgroup = 4 waves on (split s, 64-wide ci block, 32-wide co block); wave w owns taps 2w, 2w+1.  Channels past the end of the
// last block come from the zero source.  Bound: HBM (dy is read once).  The bias gradient is a product of the same dy fragments
// with a row of ones (2 more matrix instructions per 4), taken by the first ci block: a pass of its own over dy cost 48 of the 351 us
// of 64->32 on 2 x 64^3, forward and backward.  Its chain ends with every chunk (432 products in a row on 2 x 96^3 round more than
// that pass did: 7.7e-8 against 6.3e-8; now 3.4e-8).
// FOLD (channel counts outside the multiples of 32): sums are cut into chains, chains added to a second set of registers, and
// partials leave the split where that would round too much, so that dWt is no further off than with the thread per weight that served
// these counts before (128 voxels a chain where 32 MB of partials allow it): 16->8 on 2 x 64^3 5.6e-8 a thread per weight, 1.4e-7 one
// chain per split (75 us), 5.8e-8 so (82 us); 32->16 on 2 x 96^3 1.5e-7, 3.0e-7 (219 us), 1.1e-7 (222 us).
// Chunks of 64 coarse voxels are staged in LDS (x rows of 128 bytes, dy rows of 64 bytes per tap,
// double buffered, register-free copies) and read with the transposing LDS load.
// (inline assembly, so that the compiler's wait-count bookkeeping does not see the copies and keeps
// partial waits for the fragment reads; completion is tracked by hand)
__device__ __forceinline__ void g2lds16_ct(const void* g, char* lds_base) {
    const uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_base);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m), "v"(g) : "memory", "m0");
}
template <int ROWB> __device__ __forceinline__ bf16x8 frag_tr(const char* p) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * ROWB));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

struct CtWArgs {
    const bf16_t* x; int ldx;
    const bf16_t* dy; int ldy;
    float* part;              // [S][Ci][8][Co]
    float* bpart;             // [S][4][Co] partial column sums of dy (one row per wave: two taps each); may be nullptr
    const bf16_t* zero16;
    int N, D, H, W, Ci, Co;
    int chunks_per_split;     // 64-voxel chunks per split
    int fold, dump, parts_per_split;   // FOLD: chunks per chain, chunks per partial, partials per split
};

static constexpr int CTW_X = 64 * 128;            // x tile bytes
static constexpr int CTW_DY = 8 * 64 * 64;        // dy tile bytes (8 taps)
static constexpr int CTW_STAGE = CTW_X + CTW_DY;  // 40960

__device__ __forceinline__ void ctw_stage(const CtWArgs& a, char* __restrict__ st, int64_t v0, int64_t nvox, int ci0,
                                          int co0, int wv, int lane) {
    // x: copy q = wv*2 + i covers voxels 8q..8q+7, 8 pieces of 16 bytes each
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = wv * 2 + i;
        const int64_t v = v0 + q * 8 + (lane >> 3);
        const int pc = lane & 7;
        const bool ok = v < nvox && ci0 + pc * 8 < a.Ci;
        g2lds16_ct(ok ? a.x + v * a.ldx + ci0 + pc * 8 : a.zero16, st + q * 1024);
    }
    // dy: copy q = wv*8 + i: tap q/4, voxels 16*(q%4) .. +15, 4 pieces each
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int q = wv * 8 + i;
        const int tap = q >> 2;
        const int64_t v = v0 + (q & 3) * 16 + (lane >> 2);
        const int pc = lane & 3;
        const bf16_t* src = a.zero16;
        if (v < nvox && co0 + pc * 8 < a.Co) {
            const int vi = (int)v;  // host guarantees nvox < 2^31
            const int w = vi % a.W;
            int r = vi / a.W;
            const int h = r % a.H;
            r /= a.H;
            const int d = r % a.D, n = r / a.D;
            const int64_t ov = (((int64_t)n * 2 * a.D + 2 * d + (tap >> 2)) * 2 * a.H + 2 * h + ((tap >> 1) & 1)) * 2 * a.W + 2 * w + (tap & 1);
            src = a.dy + ov * a.ldy + co0 + pc * 8;
        }
        g2lds16_ct(src, st + CTW_X + q * 1024);
    }
}

template <bool BIAS>
__device__ __forceinline__ void ctw_compute(f32x16 (&acc)[2][2], double& bsum, const char* __restrict__ st, int wv, int lane) {
    const int b16 = lane >> 4, s16 = lane & 15;
    const uint32_t lx = (uint32_t)((8 * (b16 >> 1) + (s16 >> 2)) * 128 + 32 * (b16 & 1) + 8 * (s16 & 3));
    const uint32_t ly = (uint32_t)((8 * (b16 >> 1) + (s16 >> 2)) * 64 + 32 * (b16 & 1) + 8 * (s16 & 3));
    f32x16 bacc;
    if constexpr (BIAS)
#pragma unroll
        for (int r = 0; r < 16; ++r) bacc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        bf16x8 af[2], bf[2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) af[rb] = frag_tr<128>(st + ks * 16 * 128 + rb * 64 + lx);
#pragma unroll
        for (int t = 0; t < 2; ++t) bf[t] = frag_tr<64>(st + CTW_X + ((wv * 2 + t) * 64 + ks * 16) * 64 + ly);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[rb][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb], bf[t], acc[rb][t], 0, 0, 0);
        if constexpr (BIAS) {
            const uint4 one = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
#pragma unroll
            for (int t = 0; t < 2; ++t) bacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, one), bf[t], bacc, 0, 0, 0);
        }
    }
    if constexpr (BIAS) bsum += (double)bacc[0];   // every row is the sum
}

template <bool FOLD>
__global__ __launch_bounds__(256, 2) void convtr_wgrad_mfma_kernel(CtWArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ci0 = blockIdx.y * 64, co0 = blockIdx.z * 32;
    const int64_t nvox = (int64_t)a.N * a.D * a.H * a.W;
    const int64_t nchunks = (nvox + 63) / 64;
    const int64_t c_lo = (int64_t)blockIdx.x * a.chunks_per_split;
    int64_t c_hi = c_lo + a.chunks_per_split;
    if (c_hi > nchunks) c_hi = nchunks;
    f32x16 acc[2][2], sum[FOLD ? 2 : 1][2];   // sum: the chains of the partial that are done
    auto clear = [](f32x16& v) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = 0.f;
    };
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            clear(acc[rb][t]);
            if constexpr (FOLD) clear(sum[rb][t]);
        }
    // part[slot][ci][tap][co]; input channels exist in whole groups of 8
    auto write_partial = [&](int64_t slot, const f32x16 (&v)[2][2]) __attribute__((always_inline)) {
        int ln = lane;
        if constexpr (FOLD) asm volatile("" : "+v"(ln));   // the address is not worth registers of its own across the split
        const int co = co0 + (ln & 31), wvu = __builtin_amdgcn_readfirstlane(wv);
        if (co >= a.Co) return;
        float* pb = a.part + ((slot * a.Ci + ci0 + 4 * (ln >> 5)) * 8 + wvu * 2) * a.Co + co;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
                if (ci0 + rb * 32 + 8 * rg < a.Ci)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) pb[(int64_t)((rb * 32 + 8 * rg + r) * 8 + t) * a.Co] = v[rb][t][4 * rg + r];
    };
    double bsum = 0.0;
    const bool bias = a.bpart && blockIdx.y == 0;
    if (c_lo < c_hi) ctw_stage(a, lds, c_lo * 64, nvox, ci0, co0, wv, lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int par = 0, in_chain = 0, in_part = 0;
    int64_t part = (int64_t)blockIdx.x * a.parts_per_split;
    for (int64_t c = c_lo; c < c_hi; ++c, par ^= 1) {
        if (c + 1 < c_hi) ctw_stage(a, lds + (par ^ 1) * CTW_STAGE, (c + 1) * 64, nvox, ci0, co0, wv, lane);
        __builtin_amdgcn_sched_barrier(0);
        if (bias) ctw_compute<true>(acc, bsum, lds + par * CTW_STAGE, wv, lane);
        else ctw_compute<false>(acc, bsum, lds + par * CTW_STAGE, wv, lane);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (FOLD) {
            const bool out = c + 1 == c_hi || ++in_part == a.dump;
            if (out || ++in_chain == a.fold) {
                in_chain = 0;
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        sum[rb][t] += acc[rb][t];
                        clear(acc[rb][t]);
                    }
                if (out) {
                    in_part = 0;
                    write_partial(part++, sum);
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                        for (int t = 0; t < 2; ++t) clear(sum[rb][t]);
                }
            }
        }
    }
    if constexpr (!FOLD) write_partial(blockIdx.x, acc);
    const int co = co0 + (lane & 31);
    if (bias && lane < 32 && co < a.Co) a.bpart[((int64_t)blockIdx.x * 4 + wv) * a.Co + co] = (float)bsum;
}

static int ctw_splits(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    const int64_t chunks = (nvox(xd) + 63) / 64;
    const int types = ((xd->c + 63) / 64) * ((dyd->c + 31) / 32);
    int64_t s = 512 / types;  // about two workgroups per CU; more only enlarges the partial sums
    if (s < 1) s = 1;
    if (s > chunks) s = chunks;
    return (int)s;
}

// Splits, chunks per split; FOLD: chunks per chain (0: one chain per split) and per partial; number of partials.
struct CtwPlan { int splits, per, fold, dump, parts_per_split, parts; };
static CtwPlan ctw_plan(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    const int64_t chunks = (nvox(xd) + 63) / 64;
    CtwPlan p;
    p.splits = p.parts = ctw_splits(xd, dyd);
    p.per = p.dump = (int)((chunks + p.splits - 1) / p.splits);
    p.fold = 0;
    p.parts_per_split = 1;
    if (xd->c % 32 || dyd->c % 32) {
        // A chain of matrix instructions (4 a chunk) rounds like the scalar chain of 15 times as many voxels, measured; `room` of them
        // stand for the thread-per-weight kernel's chain.  F chunks a chain and room - 4 F chains a partial cover most where F is an
        // eighth of it.
        const double f = (double)nvox(xd) / convtr_splits(nvox(xd), (int64_t)xd->c * 8 * dyd->c);
        const int room = f < 128.0 ? 8 : (int)(f / 15.0);
        p.fold = room < 16 ? 1 : room / 8;
        if (p.fold > p.per) p.fold = p.per;
        int64_t dump = (int64_t)(room - 4 * p.fold) * p.fold;
        if (dump > p.per) dump = p.per;
        const int cuts = (int)((p.per + dump - 1) / dump);
        p.dump = (p.per + cuts - 1) / cuts;
        p.parts_per_split = (p.per + p.dump - 1) / p.dump;
        const int64_t walks = (chunks + p.per - 1) / p.per, last = chunks - (walks - 1) * p.per;
        p.parts = (int)((walks - 1) * p.parts_per_split + (last + p.dump - 1) / p.dump);
    }
    return p;
}

bool mfma_convtr_wgrad_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd, const lamp_norm_in* xnorm) {
    if (xd->dtype != LAMP_BF16) return false;
    if (xnorm && xnorm->mean_rstd && xnorm->c_norm > 0) return false;
    if (xd->c % 8 || dyd->c % 8 || xd->ldc % 8 || dyd->ldc % 8) return false;
    if (nvox(xd) >= ((int64_t)1 << 31)) return false;
    return true;
}

size_t mfma_convtr_wgrad_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    if (!mfma_convtr_wgrad_supported(xd, dyd, nullptr)) return 0;
    const CtwPlan p = ctw_plan(xd, dyd);
    return align_up((size_t)p.parts * xd->c * 8 * dyd->c * sizeof(float)) + align_up((size_t)p.splits * 4 * dyd->c * sizeof(float));
}

lamp_status mfma_convtr_wgrad(const lamp_tensor_desc* xd, const void* x, const lamp_tensor_desc* dyd, const void* dy,
                              float* dwt, float* dbias, float beta, void* ws, size_t ws_bytes, hipStream_t s) {
    if ((((uintptr_t)x) & 15u) || (((uintptr_t)dy) & 15u) || (((uintptr_t)ws) & 15u)) return LAMP_ERR_ALIGN;
    if (ws_bytes < mfma_convtr_wgrad_ws_bytes(xd, dyd)) return LAMP_ERR_WORKSPACE;
    const CtwPlan p = ctw_plan(xd, dyd);
    const int64_t O = (int64_t)xd->c * 8 * dyd->c;
    CtWArgs a;
    a.x = (const bf16_t*)x; a.ldx = xd->ldc; a.dy = (const bf16_t*)dy; a.ldy = dyd->ldc; a.part = (float*)ws;
    const bool direct = p.parts == 1 && beta == 0.f;   // the only partial is the result: written in place
    if (direct) a.part = dwt;
    a.bpart = dbias ? (float*)((char*)ws + align_up((size_t)p.parts * O * sizeof(float))) : nullptr;
    a.zero16 = device_zero16(s);
    if (!a.zero16) return LAMP_ERR_HIP;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = dyd->c;
    a.chunks_per_split = p.per;
    a.fold = p.fold; a.dump = p.dump; a.parts_per_split = p.parts_per_split;
    const dim3 grid(p.splits, (xd->c + 63) / 64, (dyd->c + 31) / 32);
    if (p.fold) {
        if (ensure_dyn_lds((const void*)convtr_wgrad_mfma_kernel<true>, 2 * CTW_STAGE) != LAMP_OK) return LAMP_ERR_HIP;
        hipLaunchKernelGGL(convtr_wgrad_mfma_kernel<true>, grid, dim3(256), 2 * CTW_STAGE, s, a);
    } else {
        if (ensure_dyn_lds((const void*)convtr_wgrad_mfma_kernel<false>, 2 * CTW_STAGE) != LAMP_OK) return LAMP_ERR_HIP;
        hipLaunchKernelGGL(convtr_wgrad_mfma_kernel<false>, grid, dim3(256), 2 * CTW_STAGE, s, a);
    }
    LAMP_CHECK_LAUNCH();
    if (dbias) {
        const lamp_status st = launch_reduce_partials(a.bpart, p.splits * 4, a.Co, dbias, beta, s);
        if (st != LAMP_OK) return st;
    }
    if (direct) return LAMP_OK;
    return launch_reduce_partials((const float*)ws, p.parts, O, dwt, beta, s);
}

// ------------------------------------------------------------------------------------------------
// Data gradient and weight gradient (with the bias gradient) in one pass over dy, for 32 or 64 input and 16 or 32 output channels: the
// last levels of a decoder, where the volume is.  (Wider ones: 64 x 8 x 32 sums and the chain's registers behind them are what eight
// waves hold; 128->64 has four times as many.  Narrower ones leave the 32 rows of a product half empty.)
// A workgroup (8 waves) walks chunks of 64 coarse voxels, three stages of x and dy (20 to 40 KB each) in LDS, so that two chunks are in
// flight while one is multiplied; waves 0-3 (0-1 for 32 inputs) take a quadrant (32 input channels x 32 voxels) of the data gradient
// each, its weight fragments in registers for the whole walk, waves 4-7 two taps of the weight gradient each, a w pair, whose 2 * Co
// columns lie side by side.
// LDS rows are the channels of x, and both voxels of a w pair of dy (consecutive bytes of memory, so a copy instruction fetches 1 KB in
// a row), 64 or 128 bytes, their 16-byte pieces in an order that turns with the voxel pair, so that neither the plain reads (16 voxels
// side by side) nor the transposing ones (4 voxels x 32 bytes) meet in a bank.
// Sums of the weight gradient: chains of `fold` chunks, added in S; a partial per workgroup.  Relative error against the separate
// kernel's: 64->32 on 2 x 64^3 9.0e-8 and 1.4e-7, on 2 x 32^3 4.9e-8 and 5.3e-8; 32->16 on 2 x 64^3 4.8e-8 and 7.7e-8.
// Bound: HBM.  Data, weight and bias gradient with all launches, against separate kernels (dy read twice): 64->32 on 2 x 64^3 (402 MB)
// 162 -> 83 us, on 2 x 32^3 40 -> 23; 32->16 on 2 x 64^3 146 -> 37, on 2 x 16^3 22 -> 10; 32->32 on 2 x 64^3 144 -> 67, 64->16 165 -> 51.
struct CtBArgs {
    const bf16_t* x; const bf16_t* wt; const bf16_t* dy; bf16_t* dx;
    const bf16_t* zero16;
    float* part;          // [workgroup][CI][8][CO], then [2][CO] bias sums (in two floats each) where `bias`
    int slab;             // floats of a workgroup's partial
    int ldx, lddx, bias, fold;
    CtArgs g;             // geometry: dims and reciprocals, ldb = channel stride of dy
};
static constexpr int CTB_PATCH = 32 * CT_ROW;
__host__ __device__ constexpr int ctb_stage(int ci, int co) { return 64 * ci * 2 + 4 * 64 * co * 4; }
__host__ __device__ constexpr int ctb_lds(int ci, int co) { return 3 * ctb_stage(ci, co) + 4 * CTB_PATCH; }
__host__ __device__ constexpr int ctb_per_cu(int ci, int co) { return ci * co <= 512 ? 2 : 1; }   // workgroups: LDS and registers
__device__ __forceinline__ int ctb_turn(int v, int pieces) { return (v >> 1) & (pieces - 1); }

template <int CI, int CO, typename S>
__global__ __launch_bounds__(512, 2 * ctb_per_cu(CI, CO)) void convtr_bwd_kernel(CtBArgs a) {
    extern __shared__ __attribute__((aligned(16))) char ctl[];
    constexpr int XROW = CI * 2, DROW = CO * 4, PX = XROW / 16, PD = DROW / 16;   // bytes and 16-byte pieces of a row
    constexpr int XB = 64 * XROW, STAGE = ctb_stage(CI, CO), VI = 64 / PD, ND = 32 / VI;   // voxels a copy of dy, copies of a wave
    constexpr int NKS = CO / 2, KP = CO / 8, RB = CI / 32, TB = CO / 16;   // 16-deep steps of the data gradient, of a w pair; blocks of 32
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, half = lane >> 5;
    const int nvox = a.g.N * a.g.D * a.g.H * a.g.W, nchunks = (nvox + 63) >> 6;
    const int first = blockIdx.x, wgs = gridDim.x, mine = (nchunks - first + wgs - 1) / wgs;

    // copies of a wave: 8 voxels of x, 32 voxels of one (i, j) row pair of dy
    const int cij = wv >> 1, csub = wv & 1;
    const int64_t cijoff = ct_tap_off(a.g, cij * 2);
    auto stage = [&](int chunk, int buf) __attribute__((always_inline)) {
        const int v0 = chunk * 64;
        char* st = ctl + buf * STAGE;
        if (lane < 8 * PX) {
            const int lv = wv * 8 + lane / PX, v = v0 + lv, pc = (lane & (PX - 1)) ^ ctb_turn(lv, PX);
            g2lds16_ct(v < nvox ? a.x + (int64_t)v * a.ldx + pc * 8 : a.zero16, st + wv * 8 * XROW);
        }
        const uint32_t fo = (uint32_t)ct_fine_origin(a.g, min(v0 + lane, nvox - 1));
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int lv = (csub * ND + i) * VI + lane / PD, pc = (lane & (PD - 1)) ^ ctb_turn(lv, PD);
            const uint32_t f = (uint32_t)__builtin_amdgcn_ds_bpermute(lv * 4, (int)fo);
            const bf16_t* src = a.dy + ((int64_t)f + cijoff + pc / KP) * a.g.ldb + (pc & (KP - 1)) * 8;
            g2lds16_ct(v0 + lv < nvox ? src : a.zero16, st + XB + (cij * 64 + (csub * ND + i) * VI) * DROW);
        }
    };
    // transposing reads: voxel rows rr (and rr + 4), 32 channels (64 bytes) of a row
    const int b16 = lane >> 4, s16 = lane & 15, rr = 8 * (b16 >> 1) + (s16 >> 2), pc0 = 2 * (b16 & 1) + ((s16 & 3) >> 1);
    auto toff = [&](int r, int row, int pieces) { return (uint32_t)(r * row + ((pc0 ^ ctb_turn(r, pieces)) << 4) + (s16 & 1) * 8); };
    const uint32_t xlo = toff(rr, XROW, PX), xhi = toff(rr + 4, XROW, PX), dlo = toff(rr, DROW, PD), dhi = toff(rr + 4, DROW, PD);
    auto frag2 = [&](const char* p, uint32_t tlo, uint32_t thi, uint32_t h64) __attribute__((always_inline)) {
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + (tlo ^ h64)));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + (thi ^ h64)));
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
        const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    };
    auto zero = [](f32x16& v) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = 0.f;
    };
    // Entering chunk k of the walk: its copies have landed for every wave (the 1 + ND youngest of a wave are the next chunk's; what a wave
    // has stored since only makes it wait longer), every wave is done with chunk k - 1, whose buffer takes chunk k + 2.
    auto enter = [&](int k) __attribute__((always_inline)) {
        if (k + 1 < mine) {
            if constexpr (ND == 4) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
        } else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        static_assert(ND == 4 || ND == 2, "the waits above");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (k + 2 < mine) stage(first + (k + 2) * wgs, (k + 2) % 3);
        __builtin_amdgcn_sched_barrier(0);
    };

    if (wv < 4) {
        const int cb = wv & (RB - 1), vb = wv / RB & 1, row = vb * 32 + l32;
        const bool on = wv < 2 * RB;   // (wave-uniform; the others copy only)
        bf16x8 wf[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) wf[ks] = *reinterpret_cast<const bf16x8*>(a.wt + (cb * 32 + l32) * (8 * CO) + ks * 16 + half * 8);
        const uint32_t ro = row * DROW + ((half ^ ctb_turn(row, PD)) << 4);
        char* const patch = ctl + 3 * STAGE + wv * CTB_PATCH;
        stage(first, 0);
        if (mine > 1) stage(first + wgs, 1);
        for (int k = 0; k < mine; ++k) {
            enter(k);
            if (!on) continue;
            const char* st = ctl + (k % 3) * STAGE + XB;
            f32x16 acc;
            zero(acc);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)   // (tap, channel) in order, 16 of them
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    wf[ks], *reinterpret_cast<const bf16x8*>(st + ks / KP * (64 * DROW) + (ro ^ (uint32_t)((ks & (KP - 1)) << 5))), acc, 0, 0, 0);
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
                *reinterpret_cast<uint2*>(patch + l32 * CT_ROW + (rg * 8 + half * 4) * 2) =
                    make_uint2(f2bf2(acc[rg * 4 + 0], acc[rg * 4 + 1]), f2bf2(acc[rg * 4 + 2], acc[rg * 4 + 3]));
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int lv = it * 16 + (lane >> 2), v = (first + k * wgs) * 64 + vb * 32 + lv;
                const uint4 o = *reinterpret_cast<const uint4*>(patch + lv * CT_ROW + (lane & 3) * 16);
                if (v < nvox) *reinterpret_cast<uint4*>(a.dx + (int64_t)v * a.lddx + cb * 32 + (lane & 3) * 8) = o;
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (a.bias) __syncthreads();
    } else {
        const int ij = wv - 4;
        f32x16 acc[RB][TB];
        S sum[RB][TB][16];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                zero(acc[rb][t]);
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[rb][t][r] = 0;
            }
        int chain = 0;
        double bsum = 0.0;
        constexpr bool APART = sizeof(S) == 8 && RB * TB == 4;   // no registers left for the bias products beside the others
        auto bias_add = [&](const bf16x8& d) __attribute__((always_inline)) {   // column sums of dy: a row of ones times dy, every row of which is the sum
            const uint4 one = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
            f32x16 z;
            zero(z);
            bsum += (double)__builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, one), d, z, 0, 0, 0)[0];
        };
        stage(first, 0);
        if (mine > 1) stage(first + wgs, 1);
        for (int k = 0; k < mine; ++k) {
            enter(k);
            const char* st = ctl + (k % 3) * STAGE;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                bf16x8 af[RB], bf[TB];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) af[rb] = frag2(st + ks * (16 * XROW), xlo, xhi, rb * 64);
#pragma unroll
                for (int t = 0; t < TB; ++t) bf[t] = frag2(st + XB + ij * (64 * DROW) + ks * (16 * DROW), dlo, dhi, t * 64);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int t = 0; t < TB; ++t) acc[rb][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb], bf[t], acc[rb][t], 0, 0, 0);
                if (!APART && a.bias)
#pragma unroll
                    for (int t = 0; t < TB; ++t) bias_add(bf[t]);
            }
            if (++chain == a.fold || k + 1 == mine) {
                chain = 0;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int t = 0; t < TB; ++t) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum[rb][t][r] += (S)acc[rb][t][r];
                        zero(acc[rb][t]);
                    }
            }
            if (APART && a.bias) {
                __builtin_amdgcn_sched_barrier(0);   // (the fragments are read again: kept, they spill)
#pragma unroll 1
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int t = 0; t < TB; ++t) bias_add(frag2(st + XB + ij * (64 * DROW) + ks * (16 * DROW), dlo, dhi, t * 64));
            }
        }
        float* pb = a.part + (int64_t)blockIdx.x * a.slab + (4 * half * 8 + ij * 2) * CO + l32;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int t = 0; t < TB; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) pb[(rb * 32 + 8 * rg + r) * (8 * CO) + t * 32] = (float)sum[rb][t][4 * rg + r];
        if (a.bias) {
            double* bs = reinterpret_cast<double*>(ctl + 3 * STAGE + 2 * CTB_PATCH);   // where waves 2 and 3 have their patches
            __syncthreads();
            if (half == 0) bs[ij * 32 + l32] = bsum;
        }
    }
    if (a.bias) {   // columns l32 of the four row pairs; with 16 channels the pair's second voxel behind the first's
        __syncthreads();
        const double* bs = reinterpret_cast<const double*>(ctl + 3 * STAGE + 2 * CTB_PATCH);
        if (tid < CO) {
            double t = ((bs[tid] + bs[32 + tid]) + bs[64 + tid]) + bs[96 + tid];
            if (CO == 16) t += ((bs[16 + tid] + bs[48 + tid]) + bs[80 + tid]) + bs[112 + tid];
            float* o = a.part + (int64_t)blockIdx.x * a.slab + CI * 8 * CO + tid;
            o[0] = (float)t;
            o[CO] = (float)(t - (double)(float)t);
        }
    }
}

static bool ctb_channels(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    return (xd->c == 32 || xd->c == 64) && (dyd->c == 16 || dyd->c == 32);
}
bool mfma_convtr_bwd_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd, const lamp_tensor_desc* dxd, const lamp_norm_in* xnorm) {
    return mfma_convtr_wgrad_supported(xd, dyd, xnorm) && ctb_channels(xd, dyd) && dxd && dxd->ldc % 8 == 0 && nvox(xd) < ((int64_t)1 << 29);
}
static int ctb_wgs(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    const int64_t chunks = (nvox(xd) + 63) / 64, fit = 256 * ctb_per_cu(xd->c, dyd->c);
    return (int)(chunks < fit ? chunks : fit);
}
size_t mfma_convtr_bwd_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    if (!mfma_convtr_wgrad_supported(xd, dyd, nullptr) || !ctb_channels(xd, dyd)) return 0;
    return align_up((size_t)ctb_wgs(xd, dyd) * (xd->c * 8 * dyd->c + 2 * dyd->c) * sizeof(float));
}
template <int CI, int CO, typename S = double>
static lamp_status ctb_launch(const CtBArgs& a, int wgs, hipStream_t s) {
    if (ensure_dyn_lds((const void*)convtr_bwd_kernel<CI, CO, S>, ctb_lds(CI, CO)) != LAMP_OK) return LAMP_ERR_HIP;
    hipLaunchKernelGGL((convtr_bwd_kernel<CI, CO, S>), dim3(wgs), dim3(512), ctb_lds(CI, CO), s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}
lamp_status mfma_convtr_bwd(const lamp_tensor_desc* xd, const void* x, const void* wt, const lamp_tensor_desc* dyd, const void* dy,
                            const lamp_tensor_desc* dxd, void* dx, float* dwt, float* dbias, float beta, void* ws, size_t ws_bytes,
                            hipStream_t s) {
    if (ws_bytes < mfma_convtr_bwd_ws_bytes(xd, dyd)) return LAMP_ERR_WORKSPACE;
    const int Ci = xd->c, Co = dyd->c;
    CtBArgs a;
    a.x = (const bf16_t*)x; a.wt = (const bf16_t*)wt; a.dy = (const bf16_t*)dy; a.dx = (bf16_t*)dx; a.part = (float*)ws;
    a.ldx = xd->ldc; a.lddx = dxd->ldc; a.bias = dbias ? 1 : 0;
    a.slab = Ci * 8 * Co + (dbias ? 2 * Co : 0);
    // 64->32 pays for its fp64 sums, which leave no registers for the bias products beside the others: in long walks chains of four chunks
    // and fp32 sums (2 x 64^3, forward and backward: 145.8 us, 147.3 with fp64 sums; relative error 9.0e-8 and 7.5e-8, separate kernels
    // 1.4e-7; on 2 x 96^3 1.2e-7 and 2.9e-7).  Short walks have few partials to hide this behind (2 x 32^3: 4.9e-8 so, 7.0e-8 with chains
    // of four, separate kernels 5.3e-8).
    a.fold = Ci * Co == 2048 && (nvox(xd) + 63) / 64 > 8 * 256 ? 4 : 1;
    a.zero16 = device_zero16(s);
    if (!a.zero16) return LAMP_ERR_HIP;
    a.g = CtArgs{};
    a.g.N = xd->n; a.g.D = xd->d; a.g.H = xd->h; a.g.W = xd->w; a.g.Ci = Ci; a.g.Co = Co; a.g.ldb = dyd->ldc;
    ct_set_magic(a.g);
    const int wgs = ctb_wgs(xd, dyd);
    const lamp_status st = Ci == 64 ? (Co == 32 ? (a.fold > 1 ? ctb_launch<64, 32, float>(a, wgs, s) : ctb_launch<64, 32>(a, wgs, s)) : ctb_launch<64, 16>(a, wgs, s))
                                    : (Co == 32 ? ctb_launch<32, 32>(a, wgs, s) : ctb_launch<32, 16>(a, wgs, s));
    if (st != LAMP_OK) return st;
    return launch_reduce_partials((const float*)ws, wgs, Ci * 8 * Co + (dbias ? Co : 0), dwt, beta, s, dbias, Ci * 8 * Co);
}

}  // namespace lamp
