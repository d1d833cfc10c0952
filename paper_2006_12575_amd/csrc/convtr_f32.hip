// 2x2x2 stride-2 transposed convolution of fp32 tensors on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums).
// Every output voxel depends on one input voxel and one tap, so all three passes are plain products over voxels:
//   forward         : Y[(tap,co)][v] = sum_ci Wt[ci][(tap,co)] * X[ci][v]          -> y[up(v,tap)][co]
//   data gradient   : DX[ci][v]      = sum_{(tap,co)} Wt[ci][(tap,co)] * DY[(tap,co)][v]
//   weight gradient : DWt[ci][(tap,co)] = sum_v X[v][ci] * DY[v][(tap,co)]
// Operands go straight from global memory to fragments, in the weights' own layout; a 16x16x4 product keeps a SIMD busy for 32
// cycles, which is more than its operands take to arrive from the caches.  Bound: HBM for few channels (the fine tensor), else the
// matrix rate.  In the training step of the 3-level base-8 net on 2 x 64 x 48 x 80 (16->8 and 32->16): forward 55 -> 17 us, data
// gradient 180 -> 14, weight and bias gradient 160 -> 45, against a thread per output with scalar multiply-adds.
#include "internal.h"

namespace lamp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

struct CtF32Args {
    const float* x; const float* w; const float* bias; const float* dy;
    float* out;           // y, dx, or the weight gradient's partials [slabs][Ci][8][Co]
    float* bpart;         // weight gradient: partial sums of dy, [slabs / 4][8][Co]; may be nullptr
    int ldx, ldy, ldo;    // channel strides of x, of the fine tensor, of out
    int D, H, W, Ci, Co;  // coarse dims
    int nvox;             // of all samples
    int per;              // weight gradient: steps of 4 voxels per slab
    uint32_t mW, mH, mD, mC;
    int sW, sH, sD, sC;
};
__device__ __forceinline__ uint32_t ctf_div(uint32_t v, uint32_t m, int sh) { return (uint32_t)(((uint64_t)v * m) >> sh); }
__device__ __forceinline__ int64_t ctf_fine(const CtF32Args& a, int v) {   // fine voxel (2d,2h,2w) of coarse voxel v
    const uint32_t r = ctf_div((uint32_t)v, a.mW, a.sW), w = (uint32_t)v - r * (uint32_t)a.W;
    const uint32_t r2 = ctf_div(r, a.mH, a.sH), h = r - r2 * (uint32_t)a.H;
    const uint32_t n = ctf_div(r2, a.mD, a.sD), d = r2 - n * (uint32_t)a.D;
    return (((int64_t)n * 2 * a.D + 2 * d) * 2 * a.H + 2 * h) * 2 * a.W + 2 * w;
}
__device__ __forceinline__ int ctf_tap(const CtF32Args& a, int tap) { return ((tap >> 2) * 2 * a.H + ((tap >> 1) & 1)) * 2 * a.W + (tap & 1); }
__device__ __forceinline__ float4 ctf_ld4(const float* p, bool ok) {
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ok) q = *reinterpret_cast<const float4*>(p);
    return q;
}

// Forward (FWD) and data gradient.  One wave = VB blocks of 16 coarse voxels x RB blocks of 16 rows; operands are loaded
// one step of 16 reduction indices ahead.  Forward: product j of a step contracts channels 4j .. 4j + 3 one after the other, so a sum
// starts from the bias and takes the channels in order.  Data gradient: a lane's 4 indices are consecutive, both operands arrive 16
// bytes at a time.
template <bool FWD, int VB, int RB>
__global__ __launch_bounds__(256) void convtr_f32_kernel(CtF32Args a) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int v0 = (blockIdx.x * 4 + wid) * (16 * VB), r0 = blockIdx.y * (16 * RB);
    if (v0 >= a.nvox) return;
    const int rows = FWD ? 8 * a.Co : a.Ci, K = FWD ? a.Ci : 8 * a.Co, ldw = 8 * a.Co;
    int v[VB];
    bool ok[VB];
    int64_t fine[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        v[vb] = v0 + 16 * vb + l16;
        ok[vb] = v[vb] < a.nvox;
        fine[vb] = ok[vb] ? ctf_fine(a, v[vb]) : 0;
    }
    int row[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = r0 + 16 * rb + l16;
        row[rb] = r < rows ? r : rows - 1;   // rows past the end are computed and not stored
    }
    f32x4 acc[RB][VB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        float bs[4] = {0.f, 0.f, 0.f, 0.f};
        const int r = r0 + 16 * rb + 4 * g;   // Co % 4 == 0: 4 rows of one tap
        if (FWD && a.bias && r < rows) {
            const int co = r - (int)ctf_div((uint32_t)r, a.mC, a.sC) * a.Co;
#pragma unroll
            for (int i = 0; i < 4; ++i) bs[i] = a.bias[co + i];
        }
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) acc[rb][vb] = f32x4{bs[0], bs[1], bs[2], bs[3]};
    }
    auto load = [&](int k0, float (&fa)[RB][4], float4 (&fb)[VB]) __attribute__((always_inline)) {
        if constexpr (FWD) {
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) {
                const float* p = a.x + (int64_t)v[vb] * a.ldx + k0 + g;
                fb[vb] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (ok[vb]) {                    // K is a multiple of 4
                    fb[vb].x = p[0];
                    if (k0 + 4 < K) fb[vb].y = p[4];
                    if (k0 + 8 < K) fb[vb].z = p[8];
                    if (k0 + 12 < K) fb[vb].w = p[12];
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int j = 0; j < 4; ++j) fa[rb][j] = k0 + 4 * j < K ? a.w[(int64_t)(k0 + 4 * j + g) * ldw + row[rb]] : 0.f;
        } else {
            const int k = k0 + 4 * g;
            const bool in = k < K;               // K is a multiple of 4
            const int tap = (int)ctf_div((uint32_t)k, a.mC, a.sC), co = k - tap * a.Co;
            const int to = ctf_tap(a, tap);
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) fb[vb] = ctf_ld4(a.dy + (fine[vb] + to) * a.ldy + co, ok[vb] && in);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float4 q = ctf_ld4(a.w + (int64_t)row[rb] * ldw + k, in);
                fa[rb][0] = q.x; fa[rb][1] = q.y; fa[rb][2] = q.z; fa[rb][3] = q.w;
            }
        }
    };
    auto mul = [&](const float (&fa)[RB][4], const float4 (&fb)[VB]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) {
                const float b = j == 0 ? fb[vb].x : j == 1 ? fb[vb].y : j == 2 ? fb[vb].z : fb[vb].w;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[rb][vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[rb][j], b, acc[rb][vb], 0, 0, 0);
            }
    };
    float fa[RB][4], ga[RB][4];
    float4 fb[VB], gb[VB];
    load(0, fa, fb);
    for (int k0 = 0; k0 < K; k0 += 32) {
        if (k0 + 16 < K) load(k0 + 16, ga, gb);
        mul(fa, fb);
        if (k0 + 32 < K) load(k0 + 32, fa, fb);
        if (k0 + 16 < K) mul(ga, gb);
    }
    // a lane holds 4 consecutive rows of its voxels: output channels of one tap, or input channels
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = r0 + 16 * rb + 4 * g;
        if (r >= rows) continue;
        int64_t off = r;
        if (FWD) {
            const int tap = (int)ctf_div((uint32_t)r, a.mC, a.sC), co = r - tap * a.Co;
            off = (int64_t)ctf_tap(a, tap) * a.ldo + co;
        }
#pragma unroll
        for (int vb = 0; vb < VB; ++vb)
            if (ok[vb])
                *reinterpret_cast<float4*>(a.out + (FWD ? fine[vb] : (int64_t)v[vb]) * a.ldo + off) =
                    make_float4(acc[rb][vb][0], acc[rb][vb][1], acc[rb][vb][2], acc[rb][vb][3]);
    }
}

// Weight gradient, voxels as the reduction dimension (4 per product).  One wave = RB blocks of 16 input channels x 8 blocks of 16
// columns (tap, co) over a contiguous range of voxels, its own partial; a fragment is one 4-byte load, 16 channels of 4 voxels, two
// steps loaded ahead.  The waves of the first channel block also add up dy per column for the bias gradient.  Every 64 voxels go to a
// second set of sums: one chain over a slab that grows with the volume rounds more than the thread per weight did (16->8 on
// 2 x 64^3: 1.4e-7 a thread per weight, 2.1e-7 in one chain (62 us), 1.2e-7 so (65 us); 64->32: 4.1e-7, 4.1e-7, 1.3e-7).
template <int RB>
__global__ __launch_bounds__(256, 2) void convtr_wgrad_f32_kernel(CtF32Args a) {
    constexpr int NB = 8, U = 2;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int slab = blockIdx.x * 4 + wid, r0 = blockIdx.y * (16 * RB), c0 = blockIdx.z * (16 * NB);
    const int cols = 8 * a.Co;
    int coff[NB];
    bool con[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int c = c0 + 16 * i + l16;
        con[i] = c < cols;
        const int tap = con[i] ? (int)ctf_div((uint32_t)c, a.mC, a.sC) : 0;
        coff[i] = con[i] ? ctf_tap(a, tap) * a.ldy + (c - tap * a.Co) : 0;
    }
    f32x4 acc[RB][NB], sum[RB][NB];   // the last 64 voxels, all before them
    float bacc[NB], bsum[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        bacc[i] = bsum[i] = 0.f;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[rb][i] = sum[rb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int steps = (a.nvox + 3) >> 2;
    const int s0 = slab * a.per < steps ? slab * a.per : steps, s1 = s0 + a.per < steps ? s0 + a.per : steps;
    auto load = [&](int s, float (&fa)[U][RB], float (&fb)[U][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = 4 * (s + u) + g;
            const bool ok = s + u < s1 && v < a.nvox;
            const float* xp = a.x + (int64_t)(ok ? v : 0) * a.ldx + r0 + l16;
            const float* yp = a.dy + (ok ? ctf_fine(a, v) : 0) * a.ldy;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) fa[u][rb] = ok && r0 + 16 * rb + l16 < a.Ci ? xp[16 * rb] : 0.f;
#pragma unroll
            for (int i = 0; i < NB; ++i) fb[u][i] = ok && con[i] ? yp[coff[i]] : 0.f;
        }
    };
    auto mul = [&](const float (&fa)[U][RB], const float (&fb)[U][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                bacc[i] += fb[u][i];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[rb][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][rb], fb[u][i], acc[rb][i], 0, 0, 0);
            }
    };
    float fa[U][RB], fb[U][NB], ga[U][RB], gb[U][NB];
    load(s0, fa, fb);
    for (int s = s0; s < s1; s += 2 * U) {
        load(s + U, ga, gb);
        mul(fa, fb);
        load(s + 2 * U, fa, fb);
        mul(ga, gb);
        if (((s - s0) & 15) == 16 - 2 * U)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                bsum[i] += bacc[i];
                bacc[i] = 0.f;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    sum[rb][i] += acc[rb][i];
                    acc[rb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
    }
    float* pb = a.out + (int64_t)slab * a.Ci * cols;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int c = c0 + 16 * i + l16;
        if (!con[i]) continue;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ci = r0 + 16 * rb + 4 * g + r;
                if (ci < a.Ci) pb[(int64_t)ci * cols + c] = sum[rb][i][r] + acc[rb][i][r];
            }
    }
    if (!a.bpart || blockIdx.y) return;
    __shared__ float bs[4][16 * NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        float t = bsum[i] + bacc[i];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (g == 0) bs[wid][16 * i + l16] = t;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 16 * NB && c0 + c < cols) a.bpart[(int64_t)blockIdx.x * cols + c0 + c] = bs[0][c] + bs[1][c] + bs[2][c] + bs[3][c];
}

static CtF32Args ctf_args(const lamp_tensor_desc* xd, const lamp_tensor_desc* yd) {
    CtF32Args a = {};
    a.ldx = xd->ldc; a.ldy = yd->ldc;
    a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = yd->c;
    a.nvox = (int)nvox(xd);
    div_magic(a.W, &a.mW, &a.sW);
    div_magic(a.H, &a.mH, &a.sH);
    div_magic(a.D, &a.mD, &a.sD);
    div_magic(a.Co, &a.mC, &a.sC);
    return a;
}

// Channels, strides and pointers in whole 16-byte pieces, 32-bit voxel indices and tap offsets.
bool f32_convtr_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* yd, const lamp_norm_in* xnorm) {
    if (xd->dtype != LAMP_F32 || (xnorm && xnorm->mean_rstd && xnorm->c_norm > 0)) return false;
    if (xd->c % 4 || yd->c % 4 || xd->ldc % 4 || yd->ldc % 4) return false;
    return nvox(xd) < ((int64_t)1 << 30) && cdiv(yd->c, 2) <= 65535 && cdiv(xd->c, 16) <= 65535 &&
           (2 * (int64_t)yd->h + 2) * yd->w * yd->ldc < ((int64_t)1 << 31);
}

lamp_status f32_convtr_fwd(const lamp_tensor_desc* xd, const float* x, const float* wt, const float* bias, const lamp_tensor_desc* yd,
                           float* y, hipStream_t s) {
    CtF32Args a = ctf_args(xd, yd);
    a.x = x; a.w = wt; a.bias = bias; a.out = y; a.ldo = yd->ldc;
    // 64 voxels x 64 rows a wave where that gives every CU a workgroup, else 16 x 32
    if ((int64_t)cdiv(a.nvox, 256) * cdiv(8 * a.Co, 64) >= 256)
        hipLaunchKernelGGL((convtr_f32_kernel<true, 4, 4>), dim3(cdiv(a.nvox, 256), cdiv(8 * a.Co, 64)), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((convtr_f32_kernel<true, 1, 2>), dim3(cdiv(a.nvox, 64), cdiv(8 * a.Co, 32)), dim3(256), 0, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

lamp_status f32_convtr_dgrad(const lamp_tensor_desc* xd, const float* wt, const lamp_tensor_desc* dyd, const float* dy,
                             const lamp_tensor_desc* dxd, float* dx, hipStream_t s) {
    CtF32Args a = ctf_args(xd, dyd);
    a.w = wt; a.dy = dy; a.out = dx; a.ldo = dxd->ldc;
    // 64 voxels x 32 rows a wave where that gives every CU a workgroup, else 16 x 16
    if ((int64_t)cdiv(a.nvox, 256) * cdiv(a.Ci, 32) >= 256)
        hipLaunchKernelGGL((convtr_f32_kernel<false, 4, 2>), dim3(cdiv(a.nvox, 256), cdiv(a.Ci, 32)), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((convtr_f32_kernel<false, 1, 1>), dim3(cdiv(a.nvox, 64), cdiv(a.Ci, 16)), dim3(256), 0, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

// Slabs (waves along the voxels, a multiple of 4): 2048 waves fill every SIMD twice; at least 8 steps each, partials under 32 MB.
static int ctf_slabs(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    const int64_t types = (int64_t)cdiv(xd->c, xd->c > 16 ? 32 : 16) * cdiv(dyd->c, 16), steps = (nvox(xd) + 3) / 4;
    int64_t s = 2048 / types;
    const int64_t cap = ((int64_t)8 << 20) / ((int64_t)xd->c * 8 * dyd->c);
    if (s > cap) s = cap;
    if (s > steps / 8) s = steps / 8;
    s = s / 4 * 4;
    return (int)(s < 4 ? 4 : s);
}
size_t f32_convtr_wgrad_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* dyd) {
    if (!f32_convtr_supported(xd, dyd, nullptr)) return 0;
    const size_t s = (size_t)ctf_slabs(xd, dyd);
    return align_up(s * xd->c * 8 * dyd->c * sizeof(float)) + align_up(s * 2 * dyd->c * sizeof(float));
}
lamp_status f32_convtr_wgrad(const lamp_tensor_desc* xd, const float* x, const lamp_tensor_desc* dyd, const float* dy, float* dwt,
                             float* dbias, float beta, void* ws, size_t ws_bytes, hipStream_t s) {
    if (!ws || ws_bytes < f32_convtr_wgrad_ws_bytes(xd, dyd)) return LAMP_ERR_WORKSPACE;
    const int slabs = ctf_slabs(xd, dyd);
    const int64_t O = (int64_t)xd->c * 8 * dyd->c;
    CtF32Args a = ctf_args(xd, dyd);
    a.x = x; a.dy = dy; a.out = (float*)ws;
    a.bpart = dbias ? (float*)((char*)ws + align_up((size_t)slabs * O * sizeof(float))) : nullptr;
    a.per = cdiv(cdiv(a.nvox, 4), slabs);
    const int zc = cdiv(a.Co, 16);
    if (a.Ci > 16) hipLaunchKernelGGL((convtr_wgrad_f32_kernel<2>), dim3(slabs / 4, cdiv(a.Ci, 32), zc), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((convtr_wgrad_f32_kernel<1>), dim3(slabs / 4, 1, zc), dim3(256), 0, s, a);
    LAMP_CHECK_LAUNCH();
    lamp_status st = launch_reduce_partials((const float*)ws, slabs, O, dwt, beta, s);
    if (st != LAMP_OK || !dbias) return st;
    return launch_reduce_partials(a.bpart, slabs * 2, a.Co, dbias, beta, s);
}

}  // namespace lamp
