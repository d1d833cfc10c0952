// 3x3x3 convolution of fp32 tensors on the matrix cores: forward, data gradient and weight gradient, any channel counts.
// Products and sums stay fp32 (v_mfma_f32_16x16x4_f32, 256 flops per cycle and CU, twice the vector units' rate).
#include "internal.h"
#include "vec.h"

namespace lamp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// A tile of output voxels, each side a power of two (log2), and the tiles a sample needs.
struct TileGeo {
    int ld, lh, lw;      // log2 of the tile's sides
    int nd, nh, nw;      // tiles along each axis
};
// All sides' products equal `vox` (a power of two), w side at least 4, halo at most `halo` voxels: the fewest tiles, then the
// smallest halo.
static TileGeo pick_tile(int D, int H, int W, int vox, int halo) {
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

// ---- forward and data gradient --------------------------------------------------------------------
// Bound: the fp32 matrix rate (157 TFLOP/s; 32 input channels are 432 flops a byte).  D[co][voxel] += W[co][ci] * X[ci][voxel + tap]
// with A = weights, B = voxels, so that a lane ends with 4 consecutive output channels of one voxel (a 16-byte store).  A
// workgroup of 4 waves owns one tile of output voxels; its halo is staged KC channels at a time in LDS (through registers, the next
// chunk's loads in flight during the multiplies), the weights come straight from the caches in their own layout (a 16x16x4 product
// keeps a SIMD busy for 32 cycles: per 16 channels and tap a wave needs CB + VB 16-byte fragments for 4 * CB * VB products, and no
// repacking launch stands in front of the call).  A lane's KC / 4 channels are consecutive, and product j of a chunk contracts the
// j-th channel of every lane group: the order inside a sum is free, operands agree on it.  LDS entries are padded (80, 48, 16 bytes)
// so that the 16 voxels a fragment read serves at a time fall on different banks.  32->32 on 41 x 56 x 47: 430 -> 82 us with the
// statistics (73 TFLOP/s), data gradient 385 -> 98 us, against scalar multiply-adds and a separate statistics pass.
// MAXK: halo pieces (4 channels of a voxel) a thread stages at most.  PT: taps whose weights are fetched together, one group ahead.
struct F32ConvArgs {
    const float* x; const float* w; const float* bias; float* z;
    float* partial; int32_t* counts;   // [N][tiles][Co][2], [tiles]; nullptr: no statistics
    NormIn nm;
    int ldx, ldz, N, D, H, W, Ci, Co;
    TileGeo t;
    int lvg;                           // log2 of the waves that share out the voxels; the others take further output channels
    int xvec, zvec;                    // 16-byte accesses possible
};

template <int KC> struct Frag;         // a lane's KC / 4 channels
template <> struct Frag<16> { static constexpr int EST = 20; float v[4]; };
template <> struct Frag<8> { static constexpr int EST = 12; float v[2]; };
template <> struct Frag<4> { static constexpr int EST = 4; float v[1]; };
template <int KC> __device__ __forceinline__ Frag<KC> frag_lds(const float* p) {
    Frag<KC> f;
    if constexpr (KC == 16) { const float4 q = *reinterpret_cast<const float4*>(p); f.v[0] = q.x; f.v[1] = q.y; f.v[2] = q.z; f.v[3] = q.w; }
    else if constexpr (KC == 8) { const float2 q = *reinterpret_cast<const float2*>(p); f.v[0] = q.x; f.v[1] = q.y; }
    else f.v[0] = *p;
    return f;
}

template <int KC, int CB, int VB, int MAXK, int PT, bool DGRAD>
__global__ __launch_bounds__(256, 2) void conv3d_f32_kernel(F32ConvArgs a) {
    extern __shared__ __attribute__((aligned(16))) float f32_lds[];
    constexpr int EST = Frag<KC>::EST, KL = KC / 4, QE = KC / 4, NG = 27 / PT;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int vg = wid & ((1 << a.lvg) - 1), cgrp = wid >> a.lvg;
    const int TD = 1 << a.t.ld, TH = 1 << a.t.lh, TW = 1 << a.t.lw;
    const int HH = TH + 2, HW = TW + 2, HV = (TD + 2) * HH * HW;
    int tile = blockIdx.x;
    const int tiles = a.t.nd * a.t.nh * a.t.nw;
    const int n = tile / tiles;
    tile -= n * tiles;
    const int iw = tile % a.t.nw, r1 = tile / a.t.nw, ih = r1 % a.t.nh, idd = r1 / a.t.nh;
    const int d0 = idd << a.t.ld, h0 = ih << a.t.lh, w0 = iw << a.t.lw;
    const int co0 = (blockIdx.y * (4 >> a.lvg) + cgrp) * (16 * CB);

    // the halo pieces this thread stages: voxel offset from the tile's origin, or none
    constexpr int NONE = (int)0x80000000;
    const int quad = tid & (QE - 1);
    int vo[MAXK];
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        const int e = (tid + 256 * k) / QE;
        const int row = e / HW, hw = e - row * HW, hd = row / HH, hh = row - hd * HH;
        const bool in = e < HV && (unsigned)(d0 - 1 + hd) < (unsigned)a.D && (unsigned)(h0 - 1 + hh) < (unsigned)a.H &&
                        (unsigned)(w0 - 1 + hw) < (unsigned)a.W;
        vo[k] = in ? ((hd - 1) * a.H + (hh - 1)) * a.W + (hw - 1) : NONE;
    }
    const float* xt = a.x + ((((int64_t)n * a.D + d0) * a.H + h0) * a.W + w0) * a.ldx;

    float4 pre[MAXK];
    auto fetch = [&](int c0) __attribute__((always_inline)) {
        const int c = c0 + 4 * quad;
#pragma unroll
        for (int k = 0; k < MAXK; ++k) {
            float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
            if (vo[k] != NONE) {
                const float* p = xt + (int64_t)vo[k] * a.ldx + c;
                if (a.xvec) {
                    if (c < a.Ci) q = *reinterpret_cast<const float4*>(p);
                } else {
                    if (c < a.Ci) q.x = p[0];
                    if (c + 1 < a.Ci) q.y = p[1];
                    if (c + 2 < a.Ci) q.z = p[2];
                    if (c + 3 < a.Ci) q.w = p[3];
                }
            }
            pre[k] = q;
        }
    };
    auto stage = [&](int c0) __attribute__((always_inline)) {
        float na[4] = {1.f, 1.f, 1.f, 1.f}, nb[4] = {0.f, 0.f, 0.f, 0.f};
        bool on[4] = {false, false, false, false};
        if (a.nm.mean_rstd) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = c0 + 4 * quad + i;
                on[i] = c < a.nm.c_norm;
                if (on[i]) norm_coeffs(a.nm, n, c, na[i], nb[i]);
            }
        }
#pragma unroll
        for (int k = 0; k < MAXK; ++k) {
            const int i = tid + 256 * k, e = i / QE;
            if (e >= HV) continue;
            float v[4] = {pre[k].x, pre[k].y, pre[k].z, pre[k].w};
            if (a.nm.mean_rstd && vo[k] != NONE) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (on[j]) {
                        const float u = norm_u(v[j], na[j], nb[j]);
                        v[j] = !a.nm.relu || u > 0.f ? u : 0.f;
                    }
            }
            *reinterpret_cast<float4*>(f32_lds + e * EST + 4 * quad) = make_float4(v[0], v[1], v[2], v[3]);
        }
    };

    // weights of tap group gi of chunk c0: forward W[co][t][ci], data gradient W[ci][26 - t][co]; a lane's byte offset stays, the
    // rest of the address is the same for all lanes.  KC == 16 takes whole chunks only, elsewhere missing channels give zeros.
    const int nchunks = (a.Ci + KC - 1) / KC;
    uint32_t wl[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        int co = co0 + 16 * cb + l16;
        co = co < a.Co ? co : a.Co - 1;   // rows past the end are computed and not stored
        wl[cb] = DGRAD ? (uint32_t)co * 4u : (uint32_t)co * (27u * 4u) * (uint32_t)a.Ci;
        if (KC == 16) wl[cb] += DGRAD ? (uint32_t)(g * KL) * (27u * 4u) * (uint32_t)a.Co : (uint32_t)(g * KL) * 4u;
    }
    auto wload = [&](int c0, int gi, Frag<KC> (&f)[PT][CB]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int t = gi * PT + p;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                if constexpr (KC == 16 && !DGRAD) {
                    f[p][cb] = frag_lds<16>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.w + ((int64_t)t * a.Ci + c0)) + wl[cb]));
                } else if constexpr (KC == 16) {
#pragma unroll
                    for (int j = 0; j < KL; ++j)
                        f[p][cb].v[j] = *reinterpret_cast<const float*>(
                            reinterpret_cast<const char*>(a.w + ((int64_t)(c0 + j) * 27 + (26 - t)) * a.Co) + wl[cb]);
                } else {
#pragma unroll
                    for (int j = 0; j < KL; ++j) {
                        const int ic = c0 + g * KL + j;
                        const uint32_t icc = (uint32_t)(ic < a.Ci ? ic : a.Ci - 1);
                        const uint32_t o = wl[cb] + (DGRAD ? icc * (27u * 4u) * (uint32_t)a.Co : icc * 4u);
                        const float v = *reinterpret_cast<const float*>(
                            reinterpret_cast<const char*>(a.w + (int64_t)(DGRAD ? (26 - t) * a.Co : t * a.Ci)) + o);
                        f[p][cb].v[j] = ic < a.Ci ? v : 0.f;
                    }
                }
            }
        }
    };

    int base[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        const int p = (vg * VB + vb) * 16 + l16;
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        base[vb] = ((d * HH + h) * HW + w) * EST + g * KL;
    }
    f32x4 acc[CB][VB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) acc[cb][vb] = f32x4{0.f, 0.f, 0.f, 0.f};

    Frag<KC> wf[2][PT][CB];
    fetch(0);
    wload(0, 0, wf[0]);
    for (int ch = 0; ch < nchunks; ++ch) {
        if (ch) __syncthreads();   // every wave is done with the previous chunk
        stage(ch * KC);
        __syncthreads();
        if (ch + 1 < nchunks) fetch((ch + 1) * KC);
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            // NG is odd: the last group fetches into slot 0 what the next chunk starts with, behind its own use of it
            if (gi + 1 < NG) wload(ch * KC, gi + 1, wf[(gi + 1) & 1]);
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const int t = gi * PT + p;
                const int toff = ((t / 9 * HH + t / 3 % 3) * HW + t % 3) * EST;
                Frag<KC> b[VB];
#pragma unroll
                for (int vb = 0; vb < VB; ++vb) b[vb] = frag_lds<KC>(f32_lds + base[vb] + toff);
#pragma unroll
                for (int j = 0; j < KL; ++j)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int vb = 0; vb < VB; ++vb)
                            acc[cb][vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[gi & 1][p][cb].v[j], b[vb].v[j], acc[cb][vb], 0, 0, 0);
            }
            if (gi + 1 == NG && ch + 1 < nchunks) wload((ch + 1) * KC, 0, wf[0]);
        }
    }

    float bs[CB][4], s[CB][4], q[CB][4];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = co0 + 16 * cb + 4 * g + r;
            bs[cb][r] = a.bias && co < a.Co ? a.bias[co] : 0.f;
            s[cb][r] = q[cb][r] = 0.f;
        }
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        const int p = (vg * VB + vb) * 16 + l16;
        const int w = w0 + (p & (TW - 1)), h = h0 + ((p >> a.t.lw) & (TH - 1)), d = d0 + (p >> (a.t.lw + a.t.lh));
        if (w >= a.W || h >= a.H || d >= a.D) continue;
        float* zp = a.z + ((((int64_t)n * a.D + d) * a.H + h) * a.W + w) * a.ldz;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int co = co0 + 16 * cb + 4 * g;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = acc[cb][vb][r] + bs[cb][r];
                s[cb][r] += v[r];
                q[cb][r] = fmaf(v[r], v[r], q[cb][r]);
            }
            if (a.zvec && co + 4 <= a.Co) *reinterpret_cast<float4*>(zp + co) = make_float4(v[0], v[1], v[2], v[3]);
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (co + r < a.Co) zp[co + r] = v[r];
        }
    }
    if (!a.partial) return;
    // sums of the tile per channel: 16 voxel lanes, then the waves that share the channels, in order
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                s[cb][r] += __shfl_xor(s[cb][r], o);
                q[cb][r] += __shfl_xor(q[cb][r], o);
            }
    __syncthreads();
    if (l16 == 0)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* o = f32_lds + ((wid * CB + cb) * 16 + 4 * g + r) * 2;
                o[0] = s[cb][r];
                o[1] = q[cb][r];
            }
    __syncthreads();
    const int groups = 4 >> a.lvg;
    if (tid < groups * CB * 16) {
        const int cg = tid / (CB * 16), c = tid - cg * (CB * 16);
        const int co = (blockIdx.y * groups + cg) * (16 * CB) + c;
        float ss = 0.f, qq = 0.f;
        for (int v = 0; v < (1 << a.lvg); ++v) {
            const float* o = f32_lds + (((cg << a.lvg) + v) * CB * 16 + c) * 2;
            ss += o[0];
            qq += o[1];
        }
        if (co < a.Co) *reinterpret_cast<float2*>(a.partial + (((int64_t)n * tiles + tile) * a.Co + co) * 2) = make_float2(ss, qq);
    }
    if (n == 0 && blockIdx.y == 0 && tid == 0) {
        const int cd = a.D - d0 < TD ? a.D - d0 : TD, chh = a.H - h0 < TH ? a.H - h0 : TH, cw = a.W - w0 < TW ? a.W - w0 : TW;
        a.counts[tile] = cd * chh * cw;
    }
}

// Voxel blocks per wave (4, 2, 1) and how the four waves share out voxels and channels.
struct F32Plan { int vb, cb, lvg; TileGeo t; };
static F32Plan f32_plan(const lamp_tensor_desc* zd) {
    F32Plan p;
    p.cb = zd->c > 16 ? 2 : 1;
    p.lvg = 2;
    const int64_t v = (int64_t)zd->d * zd->h * zd->w;
    const int64_t cols = cdiv(zd->c, 16 * p.cb);
    // 256 voxels a workgroup where that gives every CU one, else 128, else 64
    auto blocks = [&](int vox) { return (int64_t)zd->n * ((v + vox - 1) / vox) * cols; };
    p.vb = blocks(256) >= 256 ? 4 : blocks(128) >= 256 ? 2 : 1;
    if (p.vb == 1 && p.cb == 2 && blocks(64) < 256) { p.cb = 1; p.lvg = 1; }   // 32 voxels x 32 channels
    const int vox = p.vb * 16 << p.lvg;
    p.t = pick_tile(zd->d, zd->h, zd->w, vox, p.vb == 4 ? 648 : p.vb == 2 ? 432 : 256);
    return p;
}
static size_t f32_partial_bytes(const lamp_tensor_desc* zd, const TileGeo& t) {
    return align_up((size_t)zd->n * t.nd * t.nh * t.nw * zd->c * 2 * sizeof(float));
}
size_t f32_conv_ws_bytes(const lamp_tensor_desc* zd, int want_stats) {
    if (zd->dtype != LAMP_F32 || !want_stats) return 0;
    const TileGeo t = f32_plan(zd).t;
    return f32_partial_bytes(zd, t) + align_up((size_t)t.nd * t.nh * t.nw * sizeof(int32_t));
}

// The grid's limits, and 32-bit offsets inside the weights and the halo of a tile.
bool f32_conv_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd) {
    if (xd->dtype != LAMP_F32) return false;
    const F32Plan p = f32_plan(zd);
    return (int64_t)p.t.nd * p.t.nh * p.t.nw * zd->n < ((int64_t)1 << 31) && cdiv(zd->c, 16) <= 65535 &&
           (int64_t)xd->c * zd->c * 27 * 4 < ((int64_t)1 << 32) && (int64_t)zd->h * zd->w * 18 < ((int64_t)1 << 31);
}

template <int KC, bool DGRAD>
static void f32_launch(const F32Plan& p, dim3 grid, hipStream_t s, const F32ConvArgs& a) {
    constexpr int Q = KC / 4;
    const int hv = ((1 << p.t.ld) + 2) * ((1 << p.t.lh) + 2) * ((1 << p.t.lw) + 2);
    size_t lds = (size_t)hv * Frag<KC>::EST * sizeof(float);
    if (lds < 1024) lds = 1024;   // the statistics' 4 x 32 pairs
#define LAMP_F32(CB, VB, MK, PT) hipLaunchKernelGGL((conv3d_f32_kernel<KC, CB, VB, MK, PT, DGRAD>), grid, dim3(256), lds, s, a)
    constexpr int M4 = (648 * Q + 255) / 256, M2 = (432 * Q + 255) / 256, M1 = (256 * Q + 255) / 256;
    if (p.cb == 2) {
        if (p.vb == 4) LAMP_F32(2, 4, M4, 3);
        else if (p.vb == 2) LAMP_F32(2, 2, M2, 3);
        else LAMP_F32(2, 1, M1, 9);
    } else {
        if (p.vb == 4) LAMP_F32(1, 4, M4, 3);
        else if (p.vb == 2) LAMP_F32(1, 2, M2, 9);
        else LAMP_F32(1, 1, M1, 9);
    }
#undef LAMP_F32
}

lamp_status f32_conv(const lamp_tensor_desc* xd, const float* x, const NormIn& nm, const float* w, const float* bias, bool dgrad,
                     const lamp_tensor_desc* zd, float* z, float* stats_out, float eps, void* ws, size_t ws_bytes, hipStream_t s) {
    const F32Plan p = f32_plan(zd);
    const int64_t tiles = (int64_t)p.t.nd * p.t.nh * p.t.nw;
    const int cols = cdiv(zd->c, 16 * p.cb * (4 >> p.lvg));
    if (!f32_conv_supported(xd, zd)) return LAMP_ERR_UNSUPPORTED;
    F32ConvArgs a;
    a.x = x; a.w = w; a.bias = bias; a.z = z; a.nm = nm;
    a.ldx = xd->ldc; a.ldz = zd->ldc;
    a.N = zd->n; a.D = zd->d; a.H = zd->h; a.W = zd->w; a.Ci = xd->c; a.Co = zd->c;
    a.t = p.t; a.lvg = p.lvg;
    a.xvec = aligned16(x) && xd->c % 4 == 0 && xd->ldc % 4 == 0;
    a.zvec = aligned16(z) && zd->ldc % 4 == 0;
    // input channels per pass: 16, or 8 / 4 where those fill their chunks better
    const int kc = xd->c <= 4 ? 4 : xd->c % 16 == 0 && aligned16(w) ? 16 : 8;
    a.partial = nullptr; a.counts = nullptr;
    if (stats_out) {
        if (!ws || ws_bytes < f32_conv_ws_bytes(zd, 1)) return LAMP_ERR_WORKSPACE;
        a.partial = (float*)ws;
        a.counts = (int32_t*)((char*)ws + f32_partial_bytes(zd, p.t));
    }
    const dim3 grid((unsigned)(tiles * zd->n), cols);
    if (dgrad) {
        if (kc == 16) f32_launch<16, true>(p, grid, s, a);
        else if (kc == 8) f32_launch<8, true>(p, grid, s, a);
        else f32_launch<4, true>(p, grid, s, a);
    } else {
        if (kc == 16) f32_launch<16, false>(p, grid, s, a);
        else if (kc == 8) f32_launch<8, false>(p, grid, s, a);
        else f32_launch<4, false>(p, grid, s, a);
    }
    LAMP_CHECK_LAUNCH();
    if (stats_out) return launch_stats_finalize(a.partial, a.counts, (int)tiles, zd->n, zd->c, eps, stats_out, s);
    return LAMP_OK;
}

// ---- weight gradient ------------------------------------------------------------------------------
// Bound: the fp32 matrix rate.  dW[co][column] += dz[voxel][co] * x[voxel + tap][ci], column = (tap, ci) of a slab of CIC input
// channels, voxels as the reduction dimension (4 per product).  The 27 * CIC columns are cut into blocks of 16 whatever CIC is, so
// an image of one or two channels fills the product's columns with taps.  A workgroup walks a contiguous range of 128-voxel tiles:
// x halo and dz tile go through registers to LDS (the next tile's loads in flight during the multiplies), where one 4-byte read per
// fragment gives 16 channels of 4 voxels, 64 consecutive floats.  CG waves share out the column blocks, 4 / CG the voxels; each
// writes its own partial [Co][27][Ci], added up in a fixed order by reduce_partials_kernel.  32->32 on 41 x 56 x 47: 2450 -> 93 us
// (64 TFLOP/s) against a thread per weight; 16->8 on 2 x 64 x 48 x 80: 108 us.
struct F32WgradArgs {
    const float* x; const float* dz; float* part;   // part [splits * VG][Co][27][Ci]
    NormIn nm;
    int ldx, lddz, N, D, H, W, Ci, Co;
    TileGeo t;
    int ntiles, per;                                // tiles of all samples; tiles per split
    int cochunks;
    int xvec, zvec;
};
constexpr int F32W_VOX = 128, F32W_HALO = 432;

template <int CIC> struct WgradCols {
    static constexpr int NB = (27 * CIC + 15) / 16, CG = CIC == 16 ? 4 : CIC == 8 ? 2 : 1, VG = 4 / CG, NBW = (NB + CG - 1) / CG;
};

template <int CIC, int CBO>
__global__ __launch_bounds__(256, 2) void conv3d_wgrad_f32_kernel(F32WgradArgs a) {
    extern __shared__ __attribute__((aligned(16))) float f32w_lds[];
    constexpr int CS = CIC < 4 ? 4 : CIC, QE = CS / 4, CG = WgradCols<CIC>::CG, VG = WgradCols<CIC>::VG, NBW = WgradCols<CIC>::NBW;
    constexpr int MX = (F32W_HALO * QE + 255) / 256, MZ = F32W_VOX * CBO * 4 / 256;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int cg = wid % CG, vg = wid / CG;
    const int ci0 = (blockIdx.y / a.cochunks) * CIC, co0 = (blockIdx.y % a.cochunks) * (16 * CBO);
    const int TH = 1 << a.t.lh, TW = 1 << a.t.lw, TD = 1 << a.t.ld;
    const int HH = TH + 2, HW = TW + 2, HV = (TD + 2) * HH * HW;
    float* xs = f32w_lds;                 // [HV][CS]
    float* zs = f32w_lds + HV * CS;       // [CBO][128][16]

    // halo pieces (4 channels of a voxel) and dz pieces of this thread: coordinates in the tile, voxel offset from its origin
    const int xq = 4 * (tid & (QE - 1));
    int xc[MX], xo[MX], zc[MZ], zo[MZ];
#pragma unroll
    for (int k = 0; k < MX; ++k) {
        const int e = (tid + 256 * k) / QE;
        const int row = e / HW, hw = e - row * HW, hd = row / HH, hh = row - hd * HH;
        xc[k] = e < HV ? (hd << 20 | hh << 10 | hw) : 1 << 30;
        xo[k] = ((hd - 1) * a.H + (hh - 1)) * a.W + (hw - 1);
    }
#pragma unroll
    for (int k = 0; k < MZ; ++k) {
        const int i = tid + 256 * k, p = i / (CBO * 4);
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        zc[k] = d << 20 | h << 10 | w;
        zo[k] = (d * a.H + h) * a.W + w;
    }
    const int zq = 4 * (tid % (CBO * 4));
    // columns of this wave's blocks: LDS offset of (tap, ci), 4 consecutive voxels over the lane groups
    int col[NBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        int c = (cg * NBW + i) * 16 + l16;
        c = c < 27 * CIC ? c : 27 * CIC - 1;   // columns past the end are computed and not written
        const int t = c / CIC;
        col[i] = ((t / 9 * HH + t / 3 % 3) * HW + t % 3 + g) * CS + (c - t * CIC);
    }
    f32x4 acc[CBO][NBW];
#pragma unroll
    for (int cb = 0; cb < CBO; ++cb)
#pragma unroll
        for (int i = 0; i < NBW; ++i) acc[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    float4 px[MX], pz[MZ];
    uint32_t pin = 0;   // halo pieces inside the volume (the padding is zero behind the normalisation)
    int pn = 0;         // their sample
    const int tiles = a.t.nd * a.t.nh * a.t.nw;
    auto fetch = [&](int t) __attribute__((always_inline)) {
        const int n = t / tiles;
        t -= n * tiles;
        const int iw = t % a.t.nw, r1 = t / a.t.nw, ih = r1 % a.t.nh, idd = r1 / a.t.nh;
        const int d0 = idd << a.t.ld, h0 = ih << a.t.lh, w0 = iw << a.t.lw;
        const int64_t org = (((int64_t)n * a.D + d0) * a.H + h0) * a.W + w0;
        pin = 0;
        pn = n;
#pragma unroll
        for (int k = 0; k < MX; ++k) {
            float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
            const int c = ci0 + xq;
            if (xc[k] < 1 << 30 && (unsigned)(d0 - 1 + (xc[k] >> 20)) < (unsigned)a.D &&
                (unsigned)(h0 - 1 + (xc[k] >> 10 & 1023)) < (unsigned)a.H && (unsigned)(w0 - 1 + (xc[k] & 1023)) < (unsigned)a.W) {
                pin |= 1u << k;
                const float* p = a.x + (org + xo[k]) * a.ldx + c;
                if (a.xvec) {
                    if (c < a.Ci) q = *reinterpret_cast<const float4*>(p);
                } else {
                    if (c < a.Ci) q.x = p[0];
                    if (xq + 1 < CIC && c + 1 < a.Ci) q.y = p[1];
                    if (xq + 2 < CIC && c + 2 < a.Ci) q.z = p[2];
                    if (xq + 3 < CIC && c + 3 < a.Ci) q.w = p[3];
                }
            }
            px[k] = q;
        }
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
            float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
            const int c = co0 + zq;
            if (d0 + (zc[k] >> 20) < a.D && h0 + (zc[k] >> 10 & 1023) < a.H && w0 + (zc[k] & 1023) < a.W) {
                const float* p = a.dz + (org + zo[k]) * a.lddz + c;
                if (a.zvec) {
                    if (c < a.Co) q = *reinterpret_cast<const float4*>(p);
                } else {
                    if (c < a.Co) q.x = p[0];
                    if (c + 1 < a.Co) q.y = p[1];
                    if (c + 2 < a.Co) q.z = p[2];
                    if (c + 3 < a.Co) q.w = p[3];
                }
            }
            pz[k] = q;
        }
    };
    auto stage = [&]() __attribute__((always_inline)) {
        if (a.nm.mean_rstd) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = ci0 + xq + j;
                if (c >= a.nm.c_norm || xq + j >= CIC) continue;
                float na, nb;
                norm_coeffs(a.nm, pn, c, na, nb);
#pragma unroll
                for (int k = 0; k < MX; ++k)
                    if (pin >> k & 1) {
                        float& v = j == 0 ? px[k].x : j == 1 ? px[k].y : j == 2 ? px[k].z : px[k].w;
                        const float u = norm_u(v, na, nb);
                        v = !a.nm.relu || u > 0.f ? u : 0.f;
                    }
            }
        }
#pragma unroll
        for (int k = 0; k < MX; ++k)
            if (xc[k] < 1 << 30) *reinterpret_cast<float4*>(xs + (tid + 256 * k) / QE * CS + xq) = px[k];
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
            const int p = (tid + 256 * k) / (CBO * 4);
            *reinterpret_cast<float4*>(zs + ((zq >> 4) * F32W_VOX + p) * 16 + (zq & 15)) = pz[k];
        }
    };

    const int t0 = blockIdx.x * a.per;
    int t1 = t0 + a.per;
    if (t1 > a.ntiles) t1 = a.ntiles;
    if (t0 < t1) fetch(t0);
    for (int t = t0; t < t1; ++t) {
        if (t > t0) __syncthreads();
        stage();
        __syncthreads();
        if (t + 1 < t1) fetch(t + 1);
        auto frags = [&](int ks, float (&fa)[CBO], float (&fb)[NBW]) __attribute__((always_inline)) {
            const int p = 4 * ks;
            const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
            const int off = ((d * HH + h) * HW + w) * CS;
#pragma unroll
            for (int cb = 0; cb < CBO; ++cb) fa[cb] = zs[cb * (F32W_VOX * 16) + p * 16 + lane];
#pragma unroll
            for (int i = 0; i < NBW; ++i) fb[i] = xs[col[i] + off];
        };
        float fa[CBO], fb[NBW];
        frags(vg, fa, fb);
        for (int ks = vg; ks < F32W_VOX / 4; ks += VG) {
            float ga[CBO], gb[NBW];
            const int nx = ks + VG < F32W_VOX / 4 ? ks + VG : ks;   // the last step reads its own again
            frags(nx, ga, gb);
#pragma unroll
            for (int i = 0; i < NBW; ++i)
#pragma unroll
                for (int cb = 0; cb < CBO; ++cb) acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[cb], fb[i], acc[cb][i], 0, 0, 0);
#pragma unroll
            for (int cb = 0; cb < CBO; ++cb) fa[cb] = ga[cb];
#pragma unroll
            for (int i = 0; i < NBW; ++i) fb[i] = gb[i];
        }
    }
    float* pb = a.part + ((int64_t)blockIdx.x * VG + vg) * a.Co * 27 * a.Ci;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        const int c = (cg * NBW + i) * 16 + l16, t = c / CIC, ci = ci0 + c - t * CIC;
        if (c >= 27 * CIC || ci >= a.Ci) continue;
#pragma unroll
        for (int cb = 0; cb < CBO; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = co0 + 16 * cb + 4 * g + r;
                if (co < a.Co) pb[((int64_t)co * 27 + t) * a.Ci + ci] = acc[cb][i][r];
            }
    }
}

struct F32WPlan { int cic, cbo, cichunks, cochunks, splits, per; int64_t ntiles; TileGeo t; int vgs; };
static F32WPlan f32w_plan(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    F32WPlan p;
    p.cic = xd->c >= 9 ? 16 : xd->c >= 5 ? 8 : xd->c >= 3 ? 4 : xd->c;
    p.cbo = dzd->c > 16 ? 2 : 1;
    p.cichunks = cdiv(xd->c, p.cic);
    p.cochunks = cdiv(dzd->c, 16 * p.cbo);
    p.vgs = p.cic == 16 ? 1 : p.cic == 8 ? 2 : 4;
    p.t = pick_tile(xd->d, xd->h, xd->w, F32W_VOX, F32W_HALO);
    p.ntiles = (int64_t)xd->n * p.t.nd * p.t.nh * p.t.nw;
    // two workgroups fit a CU; the walks share the tiles evenly, and the partials stay under 64 MB
    const int64_t yz = (int64_t)p.cichunks * p.cochunks;
    int64_t s = 512 / yz;
    const int64_t cap = (int64_t)(16u << 20) / ((int64_t)p.vgs * dzd->c * 27 * xd->c);
    if (s > cap) s = cap;
    if (s < 1) s = 1;
    if (s > p.ntiles) s = p.ntiles;
    p.per = (int)((p.ntiles + s - 1) / s);
    p.splits = (int)((p.ntiles + p.per - 1) / p.per);
    return p;
}
size_t f32_wgrad_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    if (xd->dtype != LAMP_F32) return 0;
    const F32WPlan p = f32w_plan(xd, dzd);
    return align_up((size_t)p.splits * p.vgs * dzd->c * 27 * xd->c * sizeof(float));
}

bool f32_wgrad_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    if (xd->dtype != LAMP_F32) return false;
    const F32WPlan p = f32w_plan(xd, dzd);
    return p.ntiles < ((int64_t)1 << 31) && (int64_t)p.cichunks * p.cochunks <= 65535 &&
           (int64_t)xd->h * xd->w * 18 < ((int64_t)1 << 31);
}

template <int CIC>
static void f32w_launch(const F32WPlan& p, hipStream_t s, const F32WgradArgs& a) {
    const int hv = ((1 << p.t.ld) + 2) * ((1 << p.t.lh) + 2) * ((1 << p.t.lw) + 2);
    const size_t lds = ((size_t)hv * (CIC < 4 ? 4 : CIC) + (size_t)p.cbo * F32W_VOX * 16) * sizeof(float);
    const dim3 grid(p.splits, p.cichunks * p.cochunks);
    if (p.cbo == 2) hipLaunchKernelGGL((conv3d_wgrad_f32_kernel<CIC, 2>), grid, dim3(256), lds, s, a);
    else hipLaunchKernelGGL((conv3d_wgrad_f32_kernel<CIC, 1>), grid, dim3(256), lds, s, a);
}

lamp_status f32_wgrad(const lamp_tensor_desc* xd, const float* x, const NormIn& nm, const lamp_tensor_desc* dzd, const float* dz,
                      float* dw, float beta, void* ws, size_t ws_bytes, hipStream_t s) {
    const F32WPlan p = f32w_plan(xd, dzd);
    if (!ws || ws_bytes < f32_wgrad_ws_bytes(xd, dzd)) return LAMP_ERR_WORKSPACE;
    if (!f32_wgrad_supported(xd, dzd)) return LAMP_ERR_UNSUPPORTED;
    F32WgradArgs a;
    a.x = x; a.dz = dz; a.part = (float*)ws; a.nm = nm;
    a.ldx = xd->ldc; a.lddz = dzd->ldc;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = dzd->c;
    a.t = p.t; a.ntiles = (int)p.ntiles; a.per = p.per; a.cochunks = p.cochunks;
    a.xvec = aligned16(x) && xd->c % 4 == 0 && xd->ldc % 4 == 0;
    a.zvec = aligned16(dz) && dzd->c % 4 == 0 && dzd->ldc % 4 == 0;
    if (p.cic == 16) f32w_launch<16>(p, s, a);
    else if (p.cic == 8) f32w_launch<8>(p, s, a);
    else if (p.cic == 4) f32w_launch<4>(p, s, a);
    else if (p.cic == 2) f32w_launch<2>(p, s, a);
    else f32w_launch<1>(p, s, a);
    LAMP_CHECK_LAUNCH();
    return launch_reduce_partials((const float*)ws, p.splits * p.vgs, (int64_t)dzd->c * 27 * xd->c, dw, beta, s);
}

}  // namespace lamp
