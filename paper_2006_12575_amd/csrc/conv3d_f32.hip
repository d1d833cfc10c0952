// 3x3x3 convolution of fp32 tensors (and the forward pass of narrow bf16 inputs) on the fp32 matrix instruction: forward, data gradient and weight gradient, any channel counts.
// Products and sums stay fp32 (v_mfma_f32_16x16x4_f32, 256 flops per cycle and CU, twice the vector units' rate).
#include "f32_tile.h"
#include "vec.h"

namespace lamp {

// ---- forward and data gradient --------------------------------------------------------------------
// Bound: the fp32 matrix rate (157 TFLOP/s; 32 input channels are 432 flops a byte).  D[co][voxel] += W[co][ci] * X[ci][voxel + tap]
// with A = weights, B = voxels, so that a lane ends with 4 consecutive output channels of one voxel (a 16-byte store).  A
// workgroup of 4 waves walks a contiguous range of tiles; halo and weights of KC input channels go through registers to LDS (the next
// chunk's or tile's loads in flight during the multiplies; the weights stay where one chunk holds all channels).  Weights come in
// their own layout, so no repacking launch stands in front of the call; read as fragments straight from the caches they cost every
// wave 16 lines an instruction (16->8 on 2 x 64 x 48 x 80: 96 us, through LDS 85).  Product j of a chunk contracts channels 4j .. 4j + 3, one per lane group,
// and the matrix unit adds its four products one after the other, each rounded: channels in chunks of 8, in a chunk the taps, in a tap
// the channels -- bit for bit the sums of a thread that does so with fused multiply-adds (a chunk of 16 is walked as two of 8).
// LDS voxel entries are padded (80, 48, 16 bytes) so that the 64 words of a fragment read fall on different banks.  32->32 on
// 41 x 56 x 47 with the statistics: 430 -> 73 us (82 TFLOP/s; of 462 tiles a CU gets one or two, which alone is 12 %), data gradient
// 385 -> 73 us, against scalar multiply-adds and a separate statistics pass; 8->8 on 2 x 64 x 48 x 80: 46 us.
// MAXK: halo pieces (4 channels of a voxel) a thread stages at most.
// CF: 1 to 3 input channels, forward: a product contracts 4 consecutive (tap, channel) pairs, whatever tap they belong to -- the same
// order, ceil(27 CF / 4) products instead of 27 with the channels padded to 4.  A lane's pair differs from product to product by more
// than an immediate, so the offsets sit in registers.  2->16 bf16 on 2 x 64 x 80 x 96: 50 -> 38 us, with loads by buffer instructions (no
// branch to a channel of a voxel, both channels at once) 35.6 -> 32.5 of the launch alone; 3->32 on 83 x 61 x 97 52.5 -> 46.8.
// FAST: fp32 with whole 16-byte pieces and whole chunks of input channels.  Loads without a branch: a piece outside the volume comes
// from 16 zero bytes, weights past the last output channel from the last ones (their rows are not stored).  A branch to every piece is
// most of what a workgroup with one wave a SIMD does between two chunks (32->96 on 9 x 9 x 22, data gradient: 27 -> 22 us; one or two
// chunks 10.0 -> 9.5).
struct F32ConvArgs {
    const void* x; const void* w; const float* bias; void* z;   // storage type of the instantiation
    const void* zero16;                // 16 zero bytes (FAST)
    float* partial; int32_t* counts;   // [N][tiles][Co][2], [tiles]; nullptr: no statistics
    NormIn nm;
    int ldx, ldz, N, D, H, W, Ci, Co;
    TileGeo t;
    int ntiles, per;                   // tiles of all samples; tiles per workgroup
    int xvec, wvec, zvec;              // 16-byte accesses possible (xvec, CF 2: both channels of a voxel in one load)
    uint32_t mHW, mHH, mT, mNw, mNh;   // division by the halo's sides, by the tiles of a sample, along w, along h
    uint8_t sHW, sHH, sT, sNw, sNh;
};

__host__ __device__ constexpr int f32_flat(int cf) { return (27 * cf + 3) / 4; }
__host__ __device__ constexpr int f32_est(int kc) { return kc == 16 ? 20 : kc == 8 ? 12 : 4; }

template <typename T, int KC, int CB, int VB, int MAXK, bool DGRAD, int CF = 0, bool FAST = false>
__global__ __launch_bounds__(256, CB == 1 ? 3 : 2) void conv3d_f32_kernel(F32ConvArgs a) {
    extern __shared__ __attribute__((aligned(16))) float f32_lds[];
    static_assert(!CF || (KC == 4 && !DGRAD), "the forward pass of narrow inputs");
    constexpr int NJ = CF ? f32_flat(CF) : 27;   // products of a quad of channels
    constexpr int EST = CF ? CF : f32_est(KC), QE = KC / 4, KL = QE < 2 ? QE : 2, MAXW = (NJ * QE * 16 * CB + 255) / 256;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int TD = 1 << a.t.ld, TH = 1 << a.t.lh, TW = 1 << a.t.lw;
    const int HH = TH + 2, HW = TW + 2, HV = (TD + 2) * HH * HW;
    const int tiles = a.t.nd * a.t.nh * a.t.nw, nchunks = (a.Ci + KC - 1) / KC;
    const int co0 = blockIdx.y * (16 * CB);
    float* st = f32_lds;                // [4][16 * CB][2]
    float* ws = f32_lds + 128 * CB;     // [27][CB][QE][16 channels out][4 channels in]
    float* xs = ws + NJ * CB * 64 * QE; // [HV][EST]

    // the halo pieces this thread stages: coordinates in the halo
    const int quad = tid & (QE - 1);
    int hc[MAXK];
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        const uint32_t e = (uint32_t)(tid + 256 * k) / QE;
        const uint32_t row = (uint32_t)(((uint64_t)e * a.mHW) >> a.sHW), hw = e - row * HW;
        const uint32_t hd = (uint32_t)(((uint64_t)row * a.mHH) >> a.sHH), hh = row - hd * HH;
        hc[k] = (int)e < HV ? (int)(hd << 20 | hh << 10 | hw) : 1 << 30;
    }
    f32x4 px[MAXK], pw[MAXW];   // (vectors: a float4 is taken apart and put together again behind a wait for every load;
                                      // 32->32 on 41 x 56 x 47, whole kernel: 80 -> 74 us)
    uint32_t pin = 0;   // pieces inside the volume (the padding is zero behind the normalisation)
    // once per tile: which pieces lie inside the volume, and where.  CF, and FAST with two blocks of outputs (one has no registers for it):
    // by buffer loads, a lane's byte offset from the halo's first voxel, which stays for the walk, or SKIP, past the end, which loads zeros;
    // else voxel offsets.
    constexpr bool BUF = CF || (FAST && CB == 2);
    constexpr int SKIP = (int)0x80000000u, END = 0x7FFFFFF0;
    int vo[MAXK], xo[BUF ? MAXK : 1];
    if constexpr (BUF)
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            vo[k] = ((((hc[k] >> 20) * a.H + (hc[k] >> 10 & 1023)) * a.W + (hc[k] & 1023)) * a.ldx + 4 * quad) * (int)sizeof(T);
    const T* const ax = static_cast<const T*>(a.x);
    const T* const aw = static_cast<const T*>(a.w);
    const T* xt = ax;
    // sample and first voxel of a tile (by division where one tile a workgroup is the rule and its constants would come late)
    auto where = [&](int tile, int& n, int& d0, int& h0, int& w0) __attribute__((always_inline)) {
        if constexpr (BUF) {
            n = (int)((uint64_t)(uint32_t)tile * a.mT >> a.sT);
            const uint32_t r0 = (uint32_t)(tile - n * tiles), r1 = (uint32_t)((uint64_t)r0 * a.mNw >> a.sNw);
            const uint32_t r2 = (uint32_t)((uint64_t)r1 * a.mNh >> a.sNh);
            d0 = (int)(r2 << a.t.ld);
            h0 = (int)((r1 - r2 * a.t.nh) << a.t.lh);
            w0 = (int)((r0 - r1 * a.t.nw) << a.t.lw);
        } else {
            n = tile / tiles;
            tile -= n * tiles;
            const int iw = tile % a.t.nw, r1 = tile / a.t.nw, ih = r1 % a.t.nh, idd = r1 / a.t.nh;
            d0 = idd << a.t.ld;
            h0 = ih << a.t.lh;
            w0 = iw << a.t.lw;
        }
    };
    auto locate = [&](int tile) __attribute__((always_inline)) {
        int n, d0, h0, w0;
        where(tile, n, d0, h0, w0);
        --d0, --h0, --w0;
        xt = ax + ((((int64_t)n * a.D + d0) * a.H + h0) * a.W + w0) * a.ldx + (BUF ? 0 : 4 * quad);
        pin = 0;
#pragma unroll
        for (int k = 0; k < MAXK; ++k) {
            asm volatile("" : "+v"(hc[k]));   // its parts are not worth registers of their own across the walk
            const int hd = hc[k] >> 20, hh = hc[k] >> 10 & 1023, hw = hc[k] & 1023;
            const bool in = hc[k] < 1 << 30 && (unsigned)(d0 + hd) < (unsigned)a.D && (unsigned)(h0 + hh) < (unsigned)a.H &&
                            (unsigned)(w0 + hw) < (unsigned)a.W;
            if constexpr (BUF) xo[k] = in ? vo[k] : SKIP;
            else {
                vo[k] = (hd * a.H + hh) * a.W + hw;
                if (in) pin |= 1u << k;
            }
        }
    };
    auto inside = [&](int k) __attribute__((always_inline)) { return BUF ? xo[BUF ? k : 0] != SKIP : (pin >> k & 1) != 0; };
    auto fetch_x = [&](int c0) __attribute__((always_inline)) {
        const int left = a.Ci - c0 - 4 * quad;
        const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(xt), 0, END, 0x00020000);
#pragma unroll
        for (int k = 0; k < MAXK; ++k) {
            f32x4 q = {0.f, 0.f, 0.f, 0.f};
            if constexpr (FAST && BUF) {
                q = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, xo[k], 4 * c0, 0));
            } else if constexpr (FAST) {
                const T* p = xt + ((int64_t)vo[k] * a.ldx + c0);
                p = pin >> k & 1 ? p : reinterpret_cast<const T*>(a.zero16);
                q = *reinterpret_cast<const f32x4*>(p);
            } else if constexpr (CF) {
                if (CF == 2 && a.xvec) {
                    if constexpr (sizeof(T) == 4) {
                        typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
                        const f32x2 u = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rx, xo[k], 0, 0));
                        q[0] = u[0];
                        q[1] = u[1];
                    } else {
                        const uint32_t u = __builtin_amdgcn_raw_buffer_load_b32(rx, xo[k], 0, 0);
                        q[0] = __uint_as_float(u << 16);
                        q[1] = __uint_as_float(u & 0xFFFF0000u);
                    }
                } else
#pragma unroll
                    for (int j = 0; j < CF; ++j) {
                        if constexpr (sizeof(T) == 4) q[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, xo[k], 4 * j, 0));
                        else q[j] = __uint_as_float((uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rx, xo[k], 2 * j, 0) << 16);
                    }
            } else if (pin >> k & 1) {
                const T* p = xt + ((int64_t)vo[k] * a.ldx + c0);
                if (sizeof(T) == 4 && a.xvec) {
                    if (left > 0) q = *reinterpret_cast<const f32x4*>(p);
                } else {
                    if (left > 0) q[0] = io<T>::ld(p);
                    if (left > 1) q[1] = io<T>::ld(p + 1);
                    if (left > 2) q[2] = io<T>::ld(p + 2);
                    if (left > 3) q[3] = io<T>::ld(p + 3);
                }
            }
            px[k] = q;
        }
    };
    auto stage_x = [&](int n, int c0) __attribute__((always_inline)) {
        if (a.nm.mean_rstd) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = c0 + 4 * quad + j;
                if (c >= a.nm.c_norm) continue;
                float na, nb;
                norm_coeffs(a.nm, n, c, na, nb);
#pragma unroll
                for (int k = 0; k < MAXK; ++k)
                    if (inside(k)) {
                        const float u = norm_u(px[k][j], na, nb);
                        px[k][j] = io<T>::rnd(!a.nm.relu || u > 0.f ? u : 0.f);
                    }
            }
        }
        int ti = tid;
        asm volatile("" : "+v"(ti));
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (hc[k] < 1 << 30) {
                float* o = xs + (ti + 256 * k) / QE * EST + 4 * quad;
                if constexpr (CF) {
                    o[0] = px[k][0];
                    if constexpr (CF > 1) o[1] = px[k][1];
                    if constexpr (CF > 2) o[2] = px[k][2];
                } else *reinterpret_cast<f32x4*>(o) = px[k];
            }
    };
    // Weight pieces of 4 floats along the contiguous index, the other channel fastest over the lanes (whole LDS rows, and 16 or more
    // lanes of a line): forward W[co][t][ci..], data gradient W[ci][26 - t][co..].  A thread's pieces differ in the tap only, by TS.
    constexpr int TS = 256 / (16 * QE * CB);
    const int wk = DGRAD ? tid % KC : tid / 16 % QE * 4, wc = DGRAD ? tid / KC % (4 * CB) * 4 : tid % 16 + tid / (16 * QE) % CB * 16;
    const int wt0 = tid / (16 * QE * CB);
    const T* wp = DGRAD ? aw + ((int64_t)wk * 27 + (26 - wt0)) * a.Co + co0 + wc : aw + ((int64_t)(co0 + wc) * 27 + wt0) * a.Ci + wk;
    const T* const wf0 = DGRAD ? aw + ((int64_t)wk * 27 + (26 - wt0)) * a.Co + min(co0 + wc, a.Co - 4)
                               : aw + ((int64_t)min(co0 + wc, a.Co - 1) * 27 + wt0) * a.Ci + wk;   // FAST
    auto fetch_w = [&](int c0) __attribute__((always_inline)) {
        if constexpr (CF) {   // W[co][27 * CF]: four consecutive pairs of a row
#pragma unroll
            for (int u = 0; u < MAXW; ++u) {
                const int e = tid + 256 * u, co = co0 + e % (16 * CB), k = e / (16 * CB) * 4, left = co < a.Co ? 27 * CF - k : 0;
                const T* p = aw + (int64_t)co * (27 * CF) + k;
                f32x4 q = {0.f, 0.f, 0.f, 0.f};
                if (left > 0) q[0] = io<T>::ld(p);
                if (left > 1) q[1] = io<T>::ld(p + 1);
                if (left > 2) q[2] = io<T>::ld(p + 2);
                if (left > 3) q[3] = io<T>::ld(p + 3);
                pw[u] = q;
            }
            return;
        }
        if constexpr (FAST) {
            const T* p = wf0 + (DGRAD ? (int64_t)c0 * 27 * a.Co : (int64_t)c0);
#pragma unroll
            for (int u = 0; u < MAXW; ++u) {
                const int dt = u < MAXW - 1 || wt0 + u * TS < 27 ? u * TS : 0;
                pw[u] = *reinterpret_cast<const f32x4*>(p + (DGRAD ? -(int64_t)dt * a.Co : (int64_t)dt * a.Ci));
            }
            return;
        }
        const int left = DGRAD ? a.Co - co0 - wc : a.Ci - c0 - wk;   // elements of the row from the piece's first on
        const bool on = left > 0 && (DGRAD ? c0 + wk < a.Ci : co0 + wc < a.Co);
        const T* p = wp + (DGRAD ? (int64_t)c0 * 27 * a.Co : (int64_t)c0);
        const int64_t step = DGRAD ? -(int64_t)TS * a.Co : (int64_t)TS * a.Ci;
#pragma unroll
        for (int u = 0; u < MAXW; ++u) {
            f32x4 q = {0.f, 0.f, 0.f, 0.f};
            if (on && wt0 + u * TS < 27) {
                if (sizeof(T) == 4 && a.wvec) q = *reinterpret_cast<const f32x4*>(p + u * step);
                else {
                    q[0] = io<T>::ld(p + u * step);
                    if (left > 1) q[1] = io<T>::ld(p + u * step + 1);
                    if (left > 2) q[2] = io<T>::ld(p + u * step + 2);
                    if (left > 3) q[3] = io<T>::ld(p + u * step + 3);
                }
            }
            pw[u] = q;
        }
    };
    auto stage_w = [&]() __attribute__((always_inline)) {
        if constexpr (CF) {
#pragma unroll
            for (int u = 0; u < MAXW; ++u)
                if (tid + 256 * u < NJ * 16 * CB) reinterpret_cast<f32x4*>(ws)[tid + 256 * u] = pw[u];
            return;
        }
        float* o0 = ws + ((wt0 * CB + wc / 16) * QE + wk / 4) * 64 + wc % 16 * 4 + wk % 4;
#pragma unroll
        for (int u = 0; u < MAXW; ++u) {
            if (wt0 + u * TS >= 27) continue;
            float* o = o0 + u * (TS * CB * QE * 64);
            if constexpr (DGRAD) {
                o[0] = pw[u][0];
                o[4] = pw[u][1];
                o[8] = pw[u][2];
                o[12] = pw[u][3];
            } else {
                *reinterpret_cast<f32x4*>(o) = pw[u];
            }
        }
    };

    int base[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        const int p = (wid * VB + vb) * 16 + l16;
        const int w = p & (TW - 1), h = (p >> a.t.lw) & (TH - 1), d = p >> (a.t.lw + a.t.lh);
        base[vb] = ((d * HH + h) * HW + w) * EST + (CF ? 0 : g);
    }
    int ko[CF ? NJ : 1];   // where the lane's pair of every product lies
    if constexpr (CF) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            int k = 4 * j + g;
            k = k < 27 * CF ? k : 27 * CF - 1;
            const int t = k / CF;
            ko[j] = ((t / 9 * HH + t / 3 % 3) * HW + t % 3) * EST + k - t * CF;
        }
    }
    const float* wl = ws + l16 * 4 + g;
    f32x4 acc[CB][VB];

    const int t0 = blockIdx.x * a.per;
    int t1 = t0 + a.per;
    if (t1 > a.ntiles) t1 = a.ntiles;
    if (t0 >= t1) return;
    locate(t0);
    fetch_x(0);
    fetch_w(0);
    for (int tile = t0; tile < t1; ++tile) {
        const int n = BUF ? (int)((uint64_t)(uint32_t)tile * a.mT >> a.sT) : tile / tiles, tl = tile - n * tiles;
        float bs[CB][4];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = co0 + 16 * cb + 4 * g + r;
                bs[cb][r] = a.bias && co < a.Co ? a.bias[co] : 0.f;
            }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) acc[cb][vb] = f32x4{bs[cb][0], bs[cb][1], bs[cb][2], bs[cb][3]};
        for (int ch = 0; ch < nchunks; ++ch) {
            if (ch || tile > t0) __syncthreads();   // every wave is done with the previous chunk
            stage_x(n, ch * KC);
            if (nchunks > 1 || tile == t0) stage_w();
            __syncthreads();
            const bool last = ch + 1 == nchunks;
            if (last && tile + 1 < t1) locate(tile + 1);
            if (!last || tile + 1 < t1) {   // (one call of each: the results of two meet behind a wait for the loads)
                fetch_x(last ? 0 : (ch + 1) * KC);
                if (nchunks > 1) fetch_w(last ? 0 : (ch + 1) * KC);
            }
            __builtin_amdgcn_sched_barrier(0);
            // every step's fragments are read one step ahead; a step is a tap of 8 (4) channels
            constexpr int STEPS = NJ * QE / KL;
            float wf[2][CB][KL], b[2][VB][KL];
            auto frags = [&](int i) __attribute__((always_inline)) {
                if constexpr (CF) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) wf[i & 1][cb][0] = wl[(i * CB + cb) * 64];
#pragma unroll
                    for (int vb = 0; vb < VB; ++vb) {
                        const float v = xs[base[vb] + ko[i]];
                        b[i & 1][vb][0] = i + 1 < NJ || g < 27 * CF - 4 * (NJ - 1) ? v : 0.f;   // pairs past the last are zero
                    }
                    return;
                }
                const int t = i % 27, q0 = i / 27 * KL;
                const int toff = ((t / 9 * HH + t / 3 % 3) * HW + t % 3) * EST + q0 * 4;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int j = 0; j < KL; ++j) wf[i & 1][cb][j] = wl[((t * CB + cb) * QE + q0 + j) * 64];
#pragma unroll
                for (int vb = 0; vb < VB; ++vb)
#pragma unroll
                    for (int j = 0; j < KL; ++j) b[i & 1][vb][j] = xs[base[vb] + toff + 4 * j];
            };
            frags(0);
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                if (i + 1 < STEPS) frags(i + 1);
#pragma unroll
                for (int j = 0; j < KL; ++j)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int vb = 0; vb < VB; ++vb)
                            acc[cb][vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[i & 1][cb][j], b[i & 1][vb][j], acc[cb][vb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        int nn, d0, h0, w0;
        where(tile, nn, d0, h0, w0);
        float s[CB][4], q[CB][4];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) s[cb][r] = q[cb][r] = 0.f;
        int lo = l16;
        asm volatile("" : "+v"(lo));
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            const int p = (wid * VB + vb) * 16 + lo;
            const int w = w0 + (p & (TW - 1)), h = h0 + ((p >> a.t.lw) & (TH - 1)), d = d0 + (p >> (a.t.lw + a.t.lh));
            if (w >= a.W || h >= a.H || d >= a.D) continue;
            T* zp = static_cast<T*>(a.z) + ((((int64_t)n * a.D + d) * a.H + h) * a.W + w) * a.ldz;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int co = co0 + 16 * cb + 4 * g;
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = io<T>::rnd(acc[cb][vb][r]);
                    s[cb][r] += v[r];
                    q[cb][r] = fmaf(v[r], v[r], q[cb][r]);
                }
                if (a.zvec && co + 4 <= a.Co) {
                    if constexpr (sizeof(T) == 4) *reinterpret_cast<float4*>(zp + co) = make_float4(v[0], v[1], v[2], v[3]);
                    else
                        *reinterpret_cast<uint2*>(zp + co) = make_uint2(__float_as_uint(v[0]) >> 16 | (__float_as_uint(v[1]) & 0xFFFF0000u),
                                                                        __float_as_uint(v[2]) >> 16 | (__float_as_uint(v[3]) & 0xFFFF0000u));
                } else
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (co + r < a.Co) io<T>::st(zp + co + r, v[r]);
            }
        }
        if (!a.partial) continue;
        // sums of the tile per channel: 16 voxel lanes, then the waves that share the channels, in order
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[cb][r] = row_sum16(s[cb][r]);
                q[cb][r] = row_sum16(q[cb][r]);
            }
        if (l16 == 0)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<float2*>(st + ((wid * CB + cb) * 16 + 4 * g + r) * 2) = make_float2(s[cb][r], q[cb][r]);
        __syncthreads();
        if (tid < CB * 16) {
            const int co = co0 + tid;
            float ss = 0.f, qq = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float2 o = *reinterpret_cast<const float2*>(st + (v * CB * 16 + tid) * 2);
                ss += o.x;
                qq += o.y;
            }
            if (co < a.Co) *reinterpret_cast<float2*>(a.partial + (((int64_t)n * tiles + tl) * a.Co + co) * 2) = make_float2(ss, qq);
        }
        if (n == 0 && blockIdx.y == 0 && tid == 0) {
            const int cd = a.D - d0 < TD ? a.D - d0 : TD, chh = a.H - h0 < TH ? a.H - h0 : TH, cw = a.W - w0 < TW ? a.W - w0 : TW;
            a.counts[tl] = cd * chh * cw;
        }
    }
}

// Input channels per chunk (4, 8, 16), voxel blocks per wave (4, 2, 1), blocks of 16 output channels per workgroup (2, 1).
struct F32Plan { int kc, vb, cb, cf; TileGeo t; };   // cf: CF of the forward pass
static F32Plan f32_plan(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd) {
    F32Plan p;
    p.cb = zd->c > 16 ? 2 : 1;
    const int64_t v = (int64_t)zd->d * zd->h * zd->w;
    const int64_t cols = cdiv(zd->c, 16 * p.cb);
    // 256 voxels a workgroup where that gives every CU one, else 128, else 64
    auto blocks = [&](int vox) { return (int64_t)zd->n * ((v + vox - 1) / vox) * cols; };
    p.vb = blocks(256) >= 256 ? 4 : blocks(128) >= 256 ? 2 : 1;
    if (p.vb == 1 && p.cb == 2 && blocks(64) < 256) p.cb = 1;
    // chunks of 16 where they are filled and registers and LDS hold them beside the weights
    p.kc = xd->c <= 4 ? 4 : p.cb == 1 && p.vb < 4 && xd->c % 16 == 0 ? 16 : 8;
    p.cf = xd->c < 4 ? xd->c : 0;
    const int vox = p.vb * 64;
    p.t = pick_tile(zd->d, zd->h, zd->w, vox, p.vb == 4 ? 648 : p.vb == 2 ? 432 : 256);
    return p;
}
static size_t f32_partial_bytes(const lamp_tensor_desc* zd, const TileGeo& t) {
    return align_up((size_t)zd->n * t.nd * t.nh * t.nw * zd->c * 2 * sizeof(float));
}
size_t f32_conv_ws_bytes(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd, int want_stats) {
    if (!want_stats) return 0;
    const TileGeo t = f32_plan(xd, zd).t;
    return f32_partial_bytes(zd, t) + align_up((size_t)t.nd * t.nh * t.nw * sizeof(int32_t));
}
// The grid's limits, and 32-bit voxel offsets inside the halo of a tile.
bool f32_conv_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd) {
    // bf16: the forward pass of two to four input channels, in the order of the scalar kernel (whole unit 2->16: 716 -> 151 us,
    // 111 with CF here and conv3d_narrow_wgrad_kernel in its backward)
    if (xd->dtype != LAMP_F32 && (xd->c < 2 || xd->c > 4 || zd->ldc % 4)) return false;
    const F32Plan p = f32_plan(xd, zd);
    return (int64_t)p.t.nd * p.t.nh * p.t.nw * zd->n < ((int64_t)1 << 31) && cdiv(zd->c, 16) <= 65535 &&
           (int64_t)zd->h * zd->w * 18 < ((int64_t)1 << 31);
}

static size_t f32_lds_bytes(const F32Plan& p, bool flat) {
    const int hv = ((1 << p.t.ld) + 2) * ((1 << p.t.lh) + 2) * ((1 << p.t.lw) + 2);
    if (flat) return ((size_t)hv * p.cf + (size_t)f32_flat(p.cf) * p.cb * 64 + 128 * p.cb) * sizeof(float);
    return ((size_t)hv * f32_est(p.kc) + (size_t)27 * p.cb * 16 * p.kc + 128 * p.cb) * sizeof(float);
}
template <typename T, int KC, bool DGRAD, int CF = 0, bool FAST = false>
static void f32_launch(const F32Plan& p, dim3 grid, hipStream_t s, const F32ConvArgs& a) {
    constexpr int Q = KC / 4;
    const size_t lds = f32_lds_bytes(p, CF != 0);
#define LAMP_F32(CB, VB, MK) hipLaunchKernelGGL((conv3d_f32_kernel<T, KC, CB, VB, MK, DGRAD, CF, FAST>), grid, dim3(256), lds, s, a)
    constexpr int M4 = (648 * Q + 255) / 256, M2 = (432 * Q + 255) / 256, M1 = (256 * Q + 255) / 256;
    if constexpr (KC < 16)
        if (p.cb == 2) {
            if (p.vb == 4) LAMP_F32(2, 4, M4);
            else if (p.vb == 2) LAMP_F32(2, 2, M2);
            else LAMP_F32(2, 1, M1);
            return;
        }
    if constexpr (KC < 16)
        if (p.vb == 4) {
            LAMP_F32(1, 4, M4);
            return;
        }
    if (p.vb == 2) LAMP_F32(1, 2, M2);
    else LAMP_F32(1, 1, M1);
#undef LAMP_F32
}

// More than 64 output channels: each channel of a voxel feeds 64 outputs of a wave, and both operands go straight from the caches to
// fragments -- a wave = VB blocks of 16 consecutive voxels x CB of 16 output channels, no LDS, no barrier, operands DEPTH - 1
// steps ahead.  Taps
// outermost, in a tap the channels in order, one fused multiply-add after the other: bit for bit the sums of conv3d_direct_kernel.
// Product j contracts channels 4j .. 4j + 3 of a step, one per lane group; a lane loads 4 consecutive ones, and a 4 x 4 transpose
// between registers and lane groups (4 permlane swaps) hands each to its lane.  VEC: 16-byte loads possible, else 4-byte ones.
// Bound: the fp32 matrix rate (154 TFLOP/s from registers), and the latency of a step's loads where few waves are in flight: 128->256 on
// 20 x 28 x 36 55 TFLOP/s, 32->128 on 30 x 29 x 22 109 us; the whole conv unit of that size, forward and backward, 9.30 ms -> 251 us
// against a thread per output or weight.
__device__ __forceinline__ void lanes_transpose(float (&v)[4]) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[r]), __float_as_uint(v[r + 2]), false, false);
        v[r] = __uint_as_float(q[0]);
        v[r + 2] = __uint_as_float(q[1]);
    }
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[r]), __float_as_uint(v[r + 1]), false, false);
        v[r] = __uint_as_float(q[0]);
        v[r + 1] = __uint_as_float(q[1]);
    }
}
struct F32WideArgs {
    const float* x; const float* w; const float* bias; float* z;
    int ldx, ldz, D, H, W, Ci, Co;
    int nvox;                          // of all samples
    int zvec;
    uint32_t mW, mH, mD; int sW, sH, sD;
};
template <bool VEC, int VB, int CB, int DEPTH>
__global__ __launch_bounds__(256, 2) void conv3d_f32_wide_kernel(F32WideArgs a) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int v0 = (blockIdx.x * 4 + wid) * (16 * VB), co0 = blockIdx.y * (16 * CB);
    if (v0 >= a.nvox) return;
    int64_t xo[VB];                    // element offset of the lane's voxels
    int pos[VB];                       // which neighbours lie inside: bits d-1, d+1, h-1, h+1, w-1, w+1, voxel itself
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        const uint32_t v = (uint32_t)(v0 + 16 * vb + l16);
        const uint32_t r = (uint32_t)(((uint64_t)v * a.mW) >> a.sW), w = v - r * (uint32_t)a.W;
        const uint32_t r2 = (uint32_t)(((uint64_t)r * a.mH) >> a.sH), h = r - r2 * (uint32_t)a.H;
        const uint32_t n = (uint32_t)(((uint64_t)r2 * a.mD) >> a.sD), d = r2 - n * (uint32_t)a.D;
        const bool ok = (int)v < a.nvox;
        xo[vb] = (int64_t)v * a.ldx;
        pos[vb] = ok ? (d > 0 ? 1 : 0) | ((int)d < a.D - 1 ? 2 : 0) | (h > 0 ? 4 : 0) | ((int)h < a.H - 1 ? 8 : 0) | (w > 0 ? 16 : 0) |
                           ((int)w < a.W - 1 ? 32 : 0) | 64 : 0;
    }
    uint32_t wl[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        int co = co0 + 16 * cb + l16;
        co = co < a.Co ? co : a.Co - 1;   // rows past the end are computed and not stored
        wl[cb] = (uint32_t)co * 27u * (uint32_t)a.Ci;
    }
    f32x4 acc[CB][VB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        float bs[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = co0 + 16 * cb + 4 * g + r;
            bs[r] = a.bias && co < a.Co ? a.bias[co] : 0.f;
        }
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) acc[cb][vb] = f32x4{bs[0], bs[1], bs[2], bs[3]};
    }
    auto get = [&](const float* p, int k0, bool on, float (&f)[4]) __attribute__((always_inline)) {   // channels k0 .. k0 + 15 of p
        f[0] = f[1] = f[2] = f[3] = 0.f;
        if constexpr (VEC) {
            if (on && k0 + 4 * g < a.Ci) {
                const float4 q = *reinterpret_cast<const float4*>(p + k0 + 4 * g);
                f[0] = q.x; f[1] = q.y; f[2] = q.z; f[3] = q.w;
            }
        } else if (on) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + 4 * j + g < a.Ci) f[j] = p[k0 + 4 * j + g];
        }
    };
    int t = 0, k0 = 0;
    auto load = [&](float (&fa)[CB][4], float (&fb)[VB][4]) __attribute__((always_inline)) {
        const int kd = t / 9, kh = t / 3 - kd * 3, kw = t % 3;
        const int need = (kd == 0 ? 1 : kd == 2 ? 2 : 0) | (kh == 0 ? 4 : kh == 2 ? 8 : 0) | (kw == 0 ? 16 : kw == 2 ? 32 : 0) | 64;
        const int64_t off = (((int64_t)(kd - 1) * a.H + (kh - 1)) * a.W + (kw - 1)) * a.ldx;
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) get(a.x + (xo[vb] + off), k0, (pos[vb] & need) == need, fb[vb]);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) get(a.w + (int64_t)t * a.Ci + wl[cb], k0, true, fa[cb]);
        k0 += 16;
        if (k0 >= a.Ci) { k0 = 0; ++t; }
    };
    auto mul = [&](float (&fa)[CB][4], float (&fb)[VB][4]) __attribute__((always_inline)) {
        if constexpr (VEC) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) lanes_transpose(fa[cb]);
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) lanes_transpose(fb[vb]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int vb = 0; vb < VB; ++vb)
                    acc[cb][vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[cb][j], fb[vb][j], acc[cb][vb], 0, 0, 0);
    };
    float fa[DEPTH][CB][4], fb[DEPTH][VB][4];
#pragma unroll
    for (int u = 0; u < DEPTH - 1; ++u)
        if (t < 27) load(fa[u], fb[u]);
    const int steps = 27 * ((a.Ci + 15) / 16);
    for (int i = 0; i < steps; i += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (t < 27) load(fa[(u + DEPTH - 1) % DEPTH], fb[(u + DEPTH - 1) % DEPTH]);
            if (i + u < steps) mul(fa[u], fb[u]);
        }
    }
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
        if (!pos[vb]) continue;
        float* zp = a.z + (int64_t)(v0 + 16 * vb + l16) * a.ldz;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int co = co0 + 16 * cb + 4 * g;
            if (a.zvec && co + 4 <= a.Co) *reinterpret_cast<float4*>(zp + co) = make_float4(acc[cb][vb][0], acc[cb][vb][1], acc[cb][vb][2], acc[cb][vb][3]);
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (co + r < a.Co) zp[co + r] = acc[cb][vb][r];
        }
    }
}
// Not with normalise-on-load, whose coefficients every tap would fetch anew (128->256 on 2 x 16^3: 855 us, the tiled kernel 154): above
// 64 outputs a call with it takes the tiled kernel's order of sums and a call without it this one's.
static bool f32_wide(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd, const NormIn& nm, bool dgrad) {
    return !dgrad && !nm.mean_rstd && zd->c > 64 && nvox(zd) < ((int64_t)1 << 30) && (int64_t)27 * xd->c * zd->c < ((int64_t)1 << 32) &&
           cdiv(zd->c, 16) <= 65535;
}
bool f32_norm_on_load(const lamp_tensor_desc* xd, const lamp_tensor_desc* zd) {
    return xd->dtype == LAMP_F32 && f32_conv_supported(xd, zd) && !f32_wide(xd, zd, make_norm(nullptr), false);
}
static void f32_wide_launch(const lamp_tensor_desc* xd, const float* x, const float* w, const float* bias, const lamp_tensor_desc* zd,
                            float* z, hipStream_t s) {
    F32WideArgs a;
    a.x = x; a.w = w; a.bias = bias; a.z = z;
    a.ldx = xd->ldc; a.ldz = zd->ldc;
    a.D = zd->d; a.H = zd->h; a.W = zd->w; a.Ci = xd->c; a.Co = zd->c;
    a.nvox = (int)nvox(zd);
    a.zvec = aligned16(z) && zd->ldc % 4 == 0;
    div_magic(a.W, &a.mW, &a.sW);
    div_magic(a.H, &a.mH, &a.sH);
    div_magic(a.D, &a.mD, &a.sD);
    const bool vec = aligned16(x) && aligned16(w) && xd->c % 4 == 0 && xd->ldc % 4 == 0;
    // 64 voxels x 64 channels a wave where that gives every CU half a workgroup at least, else 16 x 16 with more steps in flight
    const bool big = (int64_t)cdiv(a.nvox, 256) * cdiv(a.Co, 64) >= 128;
    const dim3 grid(cdiv(a.nvox, big ? 256 : 64), cdiv(a.Co, big ? 64 : 16));
    if (big) {
        if (vec) hipLaunchKernelGGL((conv3d_f32_wide_kernel<true, 4, 4, 2>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((conv3d_f32_wide_kernel<false, 4, 4, 2>), grid, dim3(256), 0, s, a);
    } else {
        if (vec) hipLaunchKernelGGL((conv3d_f32_wide_kernel<true, 1, 1, 8>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((conv3d_f32_wide_kernel<false, 1, 1, 8>), grid, dim3(256), 0, s, a);
    }
}

lamp_status f32_conv(const lamp_tensor_desc* xd, const void* x, const NormIn& nm, const void* w, const float* bias, bool dgrad,
                     const lamp_tensor_desc* zd, void* z, float* stats_out, float eps, void* ws, size_t ws_bytes, hipStream_t s) {
    if (!f32_conv_supported(xd, zd)) return LAMP_ERR_UNSUPPORTED;
    if (dgrad && split_dgrad_takes(xd, x, zd, w)) return split_dgrad(xd, (const float*)x, (const float*)w, zd, (float*)z, s);
    if (xd->dtype == LAMP_F32 && f32_wide(xd, zd, nm, dgrad)) {
        f32_wide_launch(xd, (const float*)x, (const float*)w, bias, zd, (float*)z, s);
        LAMP_CHECK_LAUNCH();
        return stats_out ? launch_stats(zd, z, eps, stats_out, ws, ws_bytes, s) : LAMP_OK;
    }
    const F32Plan p = f32_plan(xd, zd);
    const int tiles = p.t.nd * p.t.nh * p.t.nw;
    const int cols = cdiv(zd->c, 16 * p.cb);
    F32ConvArgs a;
    a.x = x; a.w = w; a.bias = bias; a.z = z; a.nm = nm;
    a.ldx = xd->ldc; a.ldz = zd->ldc;
    a.N = zd->n; a.D = zd->d; a.H = zd->h; a.W = zd->w; a.Ci = xd->c; a.Co = zd->c;
    a.t = p.t;
    a.xvec = aligned16(x) && xd->c % 4 == 0 && xd->ldc % 4 == 0;
    a.zvec = aligned16(z) && zd->ldc % 4 == 0;
    a.wvec = aligned16(w) && (dgrad ? zd->c : xd->c) % 4 == 0;
    auto magic = [](int d, uint32_t* m, uint8_t* sh) {
        int k;
        div_magic(d, m, &k);
        *sh = (uint8_t)k;
    };
    magic((1 << p.t.lw) + 2, &a.mHW, &a.sHW);
    magic((1 << p.t.lh) + 2, &a.mHH, &a.sHH);
    magic(tiles, &a.mT, &a.sT);
    magic(p.t.nw, &a.mNw, &a.sNw);
    magic(p.t.nh, &a.mNh, &a.sNh);
    a.partial = nullptr; a.counts = nullptr;
    if (stats_out) {
        if (!ws || ws_bytes < f32_conv_ws_bytes(xd, zd, 1)) return LAMP_ERR_WORKSPACE;
        a.partial = (float*)ws;
        a.counts = (int32_t*)((char*)ws + f32_partial_bytes(zd, p.t));
    }
    // Tiles per workgroup: the CUs multiply at the same rate however many workgroups share one, so the longest CU's tiles count;
    // of equals the longest walk (it keeps the weights of a single chunk and loads a tile ahead), two workgroups a CU at least.
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
    // (buffer loads: a tile's byte offsets in 32 bits)
    const bool near = (int64_t)xd->h * xd->w * 18 * xd->ldc * (int64_t)esize(xd->dtype) < ((int64_t)1 << 31);
    const int cf = near ? p.cf : 0;
    if (cf == 2) a.xvec = xd->ldc % 2 == 0 && ((uintptr_t)x & (xd->dtype == LAMP_F32 ? 7u : 3u)) == 0;
    const bool fast = near && xd->dtype == LAMP_F32 && p.kc > 4 && a.xvec && a.wvec && xd->c % p.kc == 0 && zd->c >= 4;
    a.zero16 = fast ? device_zero16(s) : nullptr;
    if (fast && !a.zero16) return LAMP_ERR_HIP;
    if (fast) {
        if (dgrad) {
            if (p.kc == 16) f32_launch<float, 16, true, 0, true>(p, grid, s, a);
            else f32_launch<float, 8, true, 0, true>(p, grid, s, a);
        } else if (p.kc == 16) f32_launch<float, 16, false, 0, true>(p, grid, s, a);
        else f32_launch<float, 8, false, 0, true>(p, grid, s, a);
    } else if (dgrad) {
        if (p.kc == 16) f32_launch<float, 16, true>(p, grid, s, a);
        else if (p.kc == 8) f32_launch<float, 8, true>(p, grid, s, a);
        else f32_launch<float, 4, true>(p, grid, s, a);
    } else {
        if (p.kc == 16) f32_launch<float, 16, false>(p, grid, s, a);
        else if (p.kc == 8) f32_launch<float, 8, false>(p, grid, s, a);
        else if (xd->dtype == LAMP_F32) {
            if (cf == 1) f32_launch<float, 4, false, 1>(p, grid, s, a);
            else if (cf == 2) f32_launch<float, 4, false, 2>(p, grid, s, a);
            else if (cf == 3) f32_launch<float, 4, false, 3>(p, grid, s, a);
            else f32_launch<float, 4, false>(p, grid, s, a);
        } else if (cf == 2) f32_launch<bf16_t, 4, false, 2>(p, grid, s, a);
        else if (cf == 3) f32_launch<bf16_t, 4, false, 3>(p, grid, s, a);
        else f32_launch<bf16_t, 4, false>(p, grid, s, a);
    }
    LAMP_CHECK_LAUNCH();
    if (stats_out) return launch_stats_finalize(a.partial, a.counts, tiles, zd->n, zd->c, eps, stats_out, s);
    return LAMP_OK;
}

// ---- weight gradient ------------------------------------------------------------------------------
// Bound: the fp32 matrix rate.  dW[co][column] += dz[voxel][co] * x[voxel + tap][ci], column = (tap, ci) of a slab of CIC input
// channels, voxels as the reduction dimension (4 per product).  The 27 * CIC columns are cut into blocks of 16 whatever CIC is, so
// an image of one or two channels fills the product's columns with taps.  A workgroup walks a contiguous range of 128-voxel tiles:
// x halo and dz tile go through registers to LDS (the next tile's loads in flight during the multiplies), where one 4-byte read per
// fragment gives 16 channels of 4 voxels, 64 consecutive floats.  CG waves share out the column blocks, 4 / CG the voxels; each
// writes its own partial [Co][27][Ci], added up in a fixed order by reduce_partials_kernel.  A wave adds up 128 voxels and puts them
// to the sum of those before them: the walks grow with the volume, and a single chain over them would round like sqrt(walk) (8->8 on
// 2 x 128^3, walks of 4096 voxels: relative error 8.9e-7 in one chain, 1.9e-7 so, 3.8e-7 with a thread per weight over 864 voxels).
// 16-channel slabs of 32 outputs keep half of these sums in LDS, where each thread has its own slots: all of them in registers spill
// (32->32 on 41 x 56 x 47: 98 -> 106 us, with the slots 100).  With the reduction 32->32 on 41 x 56 x 47: 2450 -> 87 us against a
// thread per weight; 8->8 on 2 x 64 x 48 x 80: 50 us.
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
    constexpr bool LS = CIC * CBO == 32;   // half of the sums in LDS
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int cg = wid % CG, vg = wid / CG, vgu = __builtin_amdgcn_readfirstlane(vg);
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
    f32x4 acc[CBO][NBW], sum[LS ? 1 : CBO][NBW];   // the last 128 voxels of the wave, all before them
    f32x4* const ls = reinterpret_cast<f32x4*>(zs + CBO * F32W_VOX * 16) + tid;   // LS: sum[1], [NBW][256]
#pragma unroll
    for (int cb = 0; cb < CBO; ++cb)
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            acc[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (LS && cb) ls[i * 256] = acc[cb][i];
            else sum[cb][i] = acc[cb][i];
        }

    f32x4 px[MX], pz[MZ];
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
            f32x4 q = {0.f, 0.f, 0.f, 0.f};
            const int c = ci0 + xq;
            if (xc[k] < 1 << 30 && (unsigned)(d0 - 1 + (xc[k] >> 20)) < (unsigned)a.D &&
                (unsigned)(h0 - 1 + (xc[k] >> 10 & 1023)) < (unsigned)a.H && (unsigned)(w0 - 1 + (xc[k] & 1023)) < (unsigned)a.W) {
                pin |= 1u << k;
                const float* p = a.x + (org + xo[k]) * a.ldx + c;
                if (a.xvec) {
                    if (c < a.Ci) q = *reinterpret_cast<const f32x4*>(p);
                } else {
                    if (c < a.Ci) q[0] = p[0];
                    if (xq + 1 < CIC && c + 1 < a.Ci) q[1] = p[1];
                    if (xq + 2 < CIC && c + 2 < a.Ci) q[2] = p[2];
                    if (xq + 3 < CIC && c + 3 < a.Ci) q[3] = p[3];
                }
            }
            px[k] = q;
        }
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
            f32x4 q = {0.f, 0.f, 0.f, 0.f};
            const int c = co0 + zq;
            if (d0 + (zc[k] >> 20) < a.D && h0 + (zc[k] >> 10 & 1023) < a.H && w0 + (zc[k] & 1023) < a.W) {
                const float* p = a.dz + (org + zo[k]) * a.lddz + c;
                if (a.zvec) {
                    if (c < a.Co) q = *reinterpret_cast<const f32x4*>(p);
                } else {
                    if (c < a.Co) q[0] = p[0];
                    if (c + 1 < a.Co) q[1] = p[1];
                    if (c + 2 < a.Co) q[2] = p[2];
                    if (c + 3 < a.Co) q[3] = p[3];
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
                        const float u = norm_u(px[k][j], na, nb);
                        px[k][j] = !a.nm.relu || u > 0.f ? u : 0.f;
                    }
            }
        }
#pragma unroll
        for (int k = 0; k < MX; ++k)
            if (xc[k] < 1 << 30) *reinterpret_cast<f32x4*>(xs + (tid + 256 * k) / QE * CS + xq) = px[k];
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
            const int p = (tid + 256 * k) / (CBO * 4);
            *reinterpret_cast<f32x4*>(zs + ((zq >> 4) * F32W_VOX + p) * 16 + (zq & 15)) = pz[k];
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
        // two register sets by turns, reads in front of the multiplies they do not belong to: with one set and copies, each copy waited
        // for its read between the multiplies (32->32 on 41 x 56 x 47: 94 -> 81 us; 8->8 on 2 x 64 x 48 x 80: 59 -> 50)
        constexpr int NK = F32W_VOX / 4 / VG;
        float fa[2][CBO], fb[2][NBW];
        auto mul = [&](const float (&fa)[CBO], const float (&fb)[NBW]) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NBW; ++i)
#pragma unroll
                for (int cb = 0; cb < CBO; ++cb) acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[cb], fb[i], acc[cb][i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        frags(vgu, fa[0], fb[0]);
#pragma unroll 1
        for (int k = 0; k < NK; k += 2) {
            frags(vgu + (k + 1) * VG, fa[1], fb[1]);
            mul(fa[0], fb[0]);
            if (k + 2 < NK) frags(vgu + (k + 2) * VG, fa[0], fb[0]);
            mul(fa[1], fb[1]);
        }
        if (((t - t0) & (VG - 1)) == VG - 1 && t + 1 < t1) {
#pragma unroll
            for (int cb = 0; cb < CBO; ++cb)
#pragma unroll
                for (int i = 0; i < NBW; ++i) {
                    if (LS && cb) ls[i * 256] += acc[cb][i];
                    else sum[cb][i] += acc[cb][i];
                    acc[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    }
    float* pb = a.part + ((int64_t)blockIdx.x * VG + vg) * a.Co * 27 * a.Ci;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        const int c = (cg * NBW + i) * 16 + l16, t = c / CIC, ci = ci0 + c - t * CIC;
        if (c >= 27 * CIC || ci >= a.Ci) continue;
#pragma unroll
        for (int cb = 0; cb < CBO; ++cb) {
            const f32x4 all = (LS && cb ? ls[i * 256] : sum[LS ? 0 : cb][i]) + acc[cb][i];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = co0 + 16 * cb + 4 * g + r;
                if (co < a.Co) pb[((int64_t)co * 27 + t) * a.Ci + ci] = all[r];
            }
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
    const size_t b = align_up((size_t)p.splits * p.vgs * dzd->c * 27 * xd->c * sizeof(float)), c = split_wgrad_ws_bytes(xd, dzd);
    return b > c ? b : c;
}

bool f32_wgrad_supported(const lamp_tensor_desc* xd, const lamp_tensor_desc* dzd) {
    if (xd->dtype != LAMP_F32) return false;
    const F32WPlan p = f32w_plan(xd, dzd);
    return p.ntiles < ((int64_t)1 << 31) && (int64_t)p.cichunks * p.cochunks <= 65535 &&
           (int64_t)xd->h * xd->w * 18 < ((int64_t)1 << 31);
}

template <int CIC>
static lamp_status f32w_launch(const F32WPlan& p, hipStream_t s, const F32WgradArgs& a) {
    const int hv = ((1 << p.t.ld) + 2) * ((1 << p.t.lh) + 2) * ((1 << p.t.lw) + 2);
    size_t lds = ((size_t)hv * (CIC < 4 ? 4 : CIC) + (size_t)p.cbo * F32W_VOX * 16) * sizeof(float);
    const dim3 grid(p.splits, p.cichunks * p.cochunks);
    if (CIC * p.cbo == 32) {
        const size_t ls = (size_t)WgradCols<CIC>::NBW * 256 * 16;
        lds += ls;
        const size_t most = ((size_t)F32W_HALO * CIC + 2 * F32W_VOX * 16) * sizeof(float) + ls;
        if (ensure_dyn_lds((const void*)conv3d_wgrad_f32_kernel<CIC, 2>, (int)most) != LAMP_OK) return LAMP_ERR_HIP;
    }
    if (p.cbo == 2) hipLaunchKernelGGL((conv3d_wgrad_f32_kernel<CIC, 2>), grid, dim3(256), lds, s, a);
    else hipLaunchKernelGGL((conv3d_wgrad_f32_kernel<CIC, 1>), grid, dim3(256), lds, s, a);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

lamp_status f32_wgrad(const lamp_tensor_desc* xd, const float* x, const NormIn& nm, const lamp_tensor_desc* dzd, const float* dz,
                      float* dw, float beta, void* ws, size_t ws_bytes, hipStream_t s) {
    const F32WPlan p = f32w_plan(xd, dzd);
    if (!ws || ws_bytes < f32_wgrad_ws_bytes(xd, dzd)) return LAMP_ERR_WORKSPACE;
    if (!f32_wgrad_supported(xd, dzd)) return LAMP_ERR_UNSUPPORTED;
    if (split_wgrad_takes(xd, x, dzd, dz)) return split_wgrad(xd, x, nm, dzd, dz, dw, beta, ws, ws_bytes, s);
    F32WgradArgs a;
    a.x = x; a.dz = dz; a.part = (float*)ws; a.nm = nm;
    a.ldx = xd->ldc; a.lddz = dzd->ldc;
    a.N = xd->n; a.D = xd->d; a.H = xd->h; a.W = xd->w; a.Ci = xd->c; a.Co = dzd->c;
    a.t = p.t; a.ntiles = (int)p.ntiles; a.per = p.per; a.cochunks = p.cochunks;
    a.xvec = aligned16(x) && xd->c % 4 == 0 && xd->ldc % 4 == 0;
    a.zvec = aligned16(dz) && dzd->c % 4 == 0 && dzd->ldc % 4 == 0;
    const lamp_status st = p.cic == 16  ? f32w_launch<16>(p, s, a)
                           : p.cic == 8 ? f32w_launch<8>(p, s, a)
                           : p.cic == 4 ? f32w_launch<4>(p, s, a)
                           : p.cic == 2 ? f32w_launch<2>(p, s, a)
                                        : f32w_launch<1>(p, s, a);
    if (st != LAMP_OK) return st;
    return launch_reduce_partials((const float*)ws, p.splits * p.vgs, (int64_t)dzd->c * 27 * xd->c, dw, beta, s);
}

}  // namespace lamp
