// InstanceNorm + ReLU: statistics (two-stage, deterministic), apply, and backward.
// Bandwidth-bound kernels on NDHWC tensors; fp32 arithmetic, fp64 merging of partial moments.
#include <initializer_list>
#include <mutex>
#include "internal.h"
#include "vec.h"

// Scratch of the allocation-free entry point (lamp_inorm_relu_noalloc): partial moments and per-chunk counts of
// the statistics pass (LAMP_NOALLOC_SCRATCH_BYTES of the public header).  One copy per GPU, held until the process
// ends; every call on a GPU shares it.
static __device__ __align__(256) unsigned char scratch[LAMP_NOALLOC_SCRATCH_BYTES];

namespace lamp {

// Device address of `scratch` on the current device.  In host code the array's name is only a stand-in for
// the symbol, never an address a kernel may get: the address is looked up once per device, with that device
// current, and kept.
static lamp_status noalloc_scratch(void** out) {
    static std::mutex mu;
    static void* cache[64] = {nullptr};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LAMP_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!cache[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return LAMP_ERR_HIP;
        cache[dev] = p;
    }
    *out = cache[dev];
    return LAMP_OK;
}


// Rows of one partial sum: about 2048 chunks per sample so that small volumes still fill the chip,
// never fewer than 32 rows.
static int rows_per_chunk(int64_t v) {
    const int64_t r = (v + 2047) / 2048;
    return (int)(r < 32 ? 32 : r);
}

int stats_chunks(int64_t v) {
    const int r = rows_per_chunk(v);
    return (int)((v + r - 1) / r);
}

// Rows of one partial sum of the two-tensor reductions (backward sums, squeeze).  1024 chunks are four blocks to a CU, which is what
// their registers allow; 2048 at three to a CU left a third round two thirds full (64 channels at 128^3: squeeze 77 -> 65 us, gate's
// backward 126 -> 118).  fp32: at least four rows to every row lane, which are in flight together (training step of the 3-level base-8
// net on 2 x 64 x 48 x 80: 1297 -> 1273 us), and a thread's sums in fp64, without which they round more than over 32 rows (dgamma and
// dbeta of 8 channels on 24 x 32 x 40, relative to the square root of the rows: 5.9e-8 and 3.9e-8 over 32 rows, 6.5e-8 and 5.4e-8 in
// fp32, 5.0e-8 and 3.9e-8 so; the time is the same).  bf16: the same chunks whatever the width; other chunks are other roundings of the sums, and
// the layers below amplify these (four rows to every row lane moved weight gradients of a 4-level base-16 net by 3e-3; where it pays
// most, 16 channels on 3 x 28 x 43 x 39, forward and backward 86 -> 76 us).
static int bwd_rows(int64_t v, int C, int dtype) {
    int64_t r = (v + 1023) / 1024;
    if (r < 32) r = 32;
    if (dtype == LAMP_F32) {
        const int rl = C % 4 ? 8 : make_rowmap(C, 4).rl;
        if (r < 4 * rl) r = 4 * rl;
    }
    return (int)r;
}
int bwd_chunks(int64_t v, int C, int dtype) {
    const int r = bwd_rows(v, C, dtype);
    return (int)((v + r - 1) / r);
}

size_t stats_ws_bytes(const lamp_tensor_desc* zd) {
    int64_t V = (int64_t)zd->d * zd->h * zd->w;
    int ch = stats_chunks(V);
    return align_up((size_t)zd->n * ch * zd->c * 2 * sizeof(float)) + align_up((size_t)ch * sizeof(int32_t));
}

// ---- forward statistics ---------------------------------------------------------------------
// partial[((n*chunks + chunk)*C + c)*2] = (sum, sum of squares) over the chunk's rows.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void stats_partial_kernel(const T* __restrict__ z, int ld, int64_t V, int C,
                                                            int cthreads, int rl, int rows_per_chunk,
                                                            float* __restrict__ partial, int32_t* __restrict__ counts) {
    __shared__ float red[2 * 256 * VEC], part[256];
    const int tid = threadIdx.x;
    const int cl = tid % cthreads, r0 = tid / cthreads;
    const int cv = blockIdx.z * 256 + cl;
    const int chunk = blockIdx.x, n = blockIdx.y, chunks = gridDim.x;
    const int64_t rbeg = (int64_t)chunk * rows_per_chunk;
    int64_t rend = rbeg + rows_per_chunk;
    if (rend > V) rend = V;
    float sq[2][VEC];
    auto &s = sq[0], &q = sq[1];
#pragma unroll
    for (int i = 0; i < VEC; ++i) { s[i] = 0.f; q[i] = 0.f; }
    const bool active = r0 < rl && cv * VEC < C;
    if (active) {
        const T* base = z + ((int64_t)n * V) * ld + (int64_t)cv * VEC;
        int64_t r = rbeg + r0;
        // four rows in flight; the additions keep the row order
        for (; r + 3 * (int64_t)rl < rend; r += 4 * (int64_t)rl) {
            float v[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) Vec<T, VEC>::load(base + (r + u * (int64_t)rl) * ld, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < VEC; ++i) { s[i] += v[u][i]; q[i] = fmaf(v[u][i], v[u][i], q[i]); }
        }
        for (; r < rend; r += rl) {
            float v[VEC];
            Vec<T, VEC>::load(base + r * ld, v);
#pragma unroll
            for (int i = 0; i < VEC; ++i) { s[i] += v[i]; q[i] = fmaf(v[i], v[i], q[i]); }
        }
    }
    block_fold(sq, cthreads, rl, red, part, [&](int k, int e, float t) {
        const int c = blockIdx.z * 256 * VEC + e;
        if (c < C) partial[(((size_t)n * chunks + chunk) * C + c) * 2 + k] = t;
    });
    if (counts && n == 0 && blockIdx.z == 0 && tid == 0) counts[chunk] = (int32_t)(rend - rbeg);
}

// One 256-thread block per (n,c).  The parts carry (sum, sum of squares, count); they are added in
// fp64 in a fixed order (strided per thread, four parts in flight, then a fixed tree over lanes and
// waves), and mean / variance follow from the totals in fp64: with fp32 part sums as the input this
// loses nothing against merging per-part means and second moments.
// NT threads per (sample, channel): 256, or 1024 where there are thousands of parts (the loop over them is a chain of
// strided loads: its length, not the bytes, is what the kernel takes).  Every part's loads are in flight at once up to 4 NT parts, and the
// lanes fold by permlane swaps and DPP (shuffles of doubles were 36 trips through the LDS pipe in a row): the 27-launch forward of the
// 3-level base-8 net 134.3 -> 131.7 us with its ten launches of this.
template <int NT>
__global__ __launch_bounds__(NT) void stats_finalize_kernel(const float* __restrict__ partial,
                                                            const int32_t* __restrict__ counts, int parts, int C,
                                                            float eps, float* __restrict__ stats, int counts_per_sample) {
    __shared__ double sh[NT / 64][3];
    const int c = blockIdx.x, n = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t* cnt = counts + (counts_per_sample ? (size_t)n * parts : (size_t)0);
    const float2* pp = reinterpret_cast<const float2*>(partial) + (size_t)n * parts * C + c;
    double k = 0.0, sm = 0.0, sq = 0.0;
    for (int p = tid; p < parts; p += 4 * NT) {
        float2 v[4];
        int32_t kk[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = min(p + NT * u, parts - 1);
            v[u] = pp[(size_t)q * C];
            kk[u] = p + NT * u < parts ? cnt[q] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (kk[u] > 0) { k += (double)kk[u]; sm += (double)v[u].x; sq += (double)v[u].y; }
    }
    k = wave_fold(k);
    sm = wave_fold(sm);
    sq = wave_fold(sq);
    if (lane == 0) { sh[wv][0] = k; sh[wv][1] = sm; sh[wv][2] = sq; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < NT / 64; ++w) { k += sh[w][0]; sm += sh[w][1]; sq += sh[w][2]; }
        double mean = 0.0, var = 0.0;
        if (k > 0.0) {
            mean = sm / k;
            var = sq / k - mean * mean;
            if (var < 0.0) var = 0.0;
        }
        stats[((size_t)n * C + c) * 2 + 0] = (float)mean;
        stats[((size_t)n * C + c) * 2 + 1] = (float)(1.0 / sqrt(var + (double)eps));
    }
}

lamp_status launch_stats_finalize(const float* partials, const int32_t* counts, int parts, int N, int C,
                                  float eps, float* stats, hipStream_t s, bool counts_per_sample) {
    if (parts >= 4096)
        hipLaunchKernelGGL(stats_finalize_kernel<1024>, dim3(C, N), dim3(1024), 0, s, partials, counts, parts, C, eps, stats,
                           counts_per_sample ? 1 : 0);
    else
        hipLaunchKernelGGL(stats_finalize_kernel<256>, dim3(C, N), dim3(256), 0, s, partials, counts, parts, C, eps, stats,
                           counts_per_sample ? 1 : 0);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

lamp_status launch_stats(const lamp_tensor_desc* zd, const void* z, float eps, float* stats,
                         void* ws, size_t ws_bytes, hipStream_t s) {
    const int64_t V = (int64_t)zd->d * zd->h * zd->w;
    const int chunks = stats_chunks(V);
    if (!ws || ws_bytes < stats_ws_bytes(zd)) return LAMP_ERR_WORKSPACE;
    float* partial = (float*)ws;
    int32_t* counts = (int32_t*)((char*)ws + align_up((size_t)zd->n * chunks * zd->c * 2 * sizeof(float)));
    const int vec = pick_vec(zd->dtype, zd->c, {zd->ldc}, {z});
    LAMP_DISPATCH_TV(zd->dtype, vec, {
        RowMap m = make_rowmap(zd->c, VEC);
        hipLaunchKernelGGL((stats_partial_kernel<T, VEC>), dim3(chunks, zd->n, m.ctiles), dim3(256), 0, s,
                           (const T*)z, zd->ldc, V, zd->c, m.cthreads, m.rl, rows_per_chunk(V), partial, counts);
    });
    LAMP_CHECK_LAUNCH();
    return launch_stats_finalize(partial, counts, chunks, zd->n, zd->c, eps, stats, s);
}

// ---- sum of split-reduction partials -------------------------------------------------------
// z[v][c] = bf16( sum_s zpart[s][v][c] ), splits added in order.  C % 8 == 0.
__device__ __forceinline__ uint4 splitk_sum(const float* src, int S, int64_t split_stride) {
    float4 a0 = *reinterpret_cast<const float4*>(src), a1 = *reinterpret_cast<const float4*>(src + 4);
    auto add = [&](const float4& b0, const float4& b1) {
        a0.x += b0.x; a0.y += b0.y; a0.z += b0.z; a0.w += b0.w;
        a1.x += b1.x; a1.y += b1.y; a1.z += b1.z; a1.w += b1.w;
    };
    int sp = 1;
    for (; sp + 3 < S; sp += 4) {   // four splits in flight
        float4 b0[4], b1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            b0[u] = *reinterpret_cast<const float4*>(src + (sp + u) * split_stride);
            b1[u] = *reinterpret_cast<const float4*>(src + (sp + u) * split_stride + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) add(b0[u], b1[u]);
    }
    for (; sp < S; ++sp) add(*reinterpret_cast<const float4*>(src + sp * split_stride), *reinterpret_cast<const float4*>(src + sp * split_stride + 4));
    const float v[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    return Vec<bf16_t, 8>::pack(v);
}
struct SplitkArgs {
    const float* zpart; int S; int64_t split_stride;
    bf16_t* z; int ldz; bf16_t* z2; int ldz2, zsplit;   // channels from zsplit on belong to the second output tensor
    int64_t V; int C, cthreads, rl, rows_per_chunk;
    float* partial; int32_t* counts;
};
__device__ __forceinline__ void splitk_store(const SplitkArgs& a, int64_t row, int cv, const uint4& q) {
    bf16_t* dst = cv * 8 < a.zsplit ? a.z + row * a.ldz + (int64_t)cv * 8 : a.z2 + row * a.ldz2 + ((int64_t)cv * 8 - a.zsplit);
    *reinterpret_cast<uint4*>(dst) = q;
}
// Without statistics (data gradients): one thread per 8 channels of a voxel (512 channels on 2 x 8^3: 21.3 -> 4.9 us against chunks of 32 rows).
__global__ __launch_bounds__(256) void splitk_reduce_kernel(SplitkArgs a, int64_t pieces) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= pieces) return;
    const int gpv = a.C / 8;
    const int64_t row = i / gpv;
    const int cv = (int)(i - row * gpv);
    splitk_store(a, row, cv, splitk_sum(a.zpart + row * a.C + cv * 8, a.S, a.split_stride));
}
// With the statistics: the (sum, sum of squares) of the rounded values, in the order of stats_partial_kernel.  All 1024 threads add up
// splits and hand the rounded values over in LDS to the 256 that sum, which keeps the order of the sums, and with it every bit of the
// net behind them, while a chunk's loads are in flight together (512 channels on 2 x 8^3, 256 threads that did both: 21.3 us,
// so 10.8).
__global__ __launch_bounds__(1024) void splitk_stats_kernel(SplitkArgs a) {
    __shared__ uint4 val[2048];
    __shared__ float red[2 * 256 * 8], part[256];
    const int tid = threadIdx.x, cl = tid % a.cthreads, r0 = tid / a.cthreads;   // (of the summing threads)
    const int chunk = blockIdx.x, n = blockIdx.y, chunks = gridDim.x, cv0 = blockIdx.z * 256;
    const int64_t rbeg = (int64_t)chunk * a.rows_per_chunk;
    int64_t rend = rbeg + a.rows_per_chunk;
    if (rend > a.V) rend = a.V;
    float sq[2][8];
    auto &s = sq[0], &q = sq[1];
#pragma unroll
    for (int i = 0; i < 8; ++i) { s[i] = 0.f; q[i] = 0.f; }
    const int batch = 2048 / a.cthreads / a.rl * a.rl;   // rows handed over at a time, whole rounds of the row lanes
    for (int64_t rb = rbeg; rb < rend; rb += batch) {
        const int rows = (int)(rend - rb < batch ? rend - rb : batch);
        for (int p = tid; p < rows * a.cthreads; p += 1024) {
            const int row = p / a.cthreads, cv = cv0 + p - row * a.cthreads;
            if (cv * 8 >= a.C) continue;
            const int64_t gr = (int64_t)n * a.V + rb + row;
            const uint4 v = splitk_sum(a.zpart + gr * a.C + cv * 8, a.S, a.split_stride);
            splitk_store(a, gr, cv, v);
            val[p] = v;
        }
        __syncthreads();
        if (tid < 256 && r0 < a.rl && (cv0 + cl) * 8 < a.C)
            for (int r = r0; r < rows; r += a.rl) {
                float v[8];
                Vec<bf16_t, 8>::unpack(val[r * a.cthreads + cl], v);
#pragma unroll
                for (int i = 0; i < 8; ++i) { s[i] += v[i]; q[i] = fmaf(v[i], v[i], q[i]); }
            }
        __syncthreads();
    }
    block_fold<float, 1024>(sq, a.cthreads, a.rl, red, part, [&](int k, int e, float t) {
        const int c = blockIdx.z * 256 * 8 + e;
        if (c < a.C) a.partial[(((size_t)n * chunks + chunk) * a.C + c) * 2 + k] = t;
    });
    if (n == 0 && blockIdx.z == 0 && tid == 0) a.counts[chunk] = (int32_t)(rend - rbeg);
}

lamp_status launch_splitk_reduce(const float* zpart, int S, const lamp_tensor_desc* zd, void* z, float eps, float* stats,
                                 void* ws, size_t ws_bytes, hipStream_t s, void* z2, int ldz2, int zsplit) {
    const RowMap m = make_rowmap(zd->c, 8);
    SplitkArgs a;
    a.zpart = zpart; a.S = S; a.split_stride = nvox(zd) * zd->c;
    a.z = (bf16_t*)z; a.ldz = zd->ldc; a.z2 = (bf16_t*)z2; a.ldz2 = ldz2; a.zsplit = z2 ? zsplit : 0x7fffffff;
    a.V = (int64_t)zd->d * zd->h * zd->w; a.C = zd->c; a.cthreads = m.cthreads; a.rl = m.rl; a.rows_per_chunk = rows_per_chunk(a.V);
    a.partial = nullptr; a.counts = nullptr;
    if (!stats) {
        const int64_t pieces = nvox(zd) * (zd->c / 8);
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(cdiv(pieces, 256)), dim3(256), 0, s, a, pieces);
        LAMP_CHECK_LAUNCH();
        return LAMP_OK;
    }
    const int chunks = stats_chunks(a.V);
    if (!ws || ws_bytes < stats_ws_bytes(zd)) return LAMP_ERR_WORKSPACE;
    a.partial = (float*)ws;
    a.counts = (int32_t*)((char*)ws + align_up((size_t)zd->n * chunks * zd->c * 2 * sizeof(float)));
    hipLaunchKernelGGL(splitk_stats_kernel, dim3(chunks, zd->n, m.ctiles), dim3(1024), 0, s, a);
    LAMP_CHECK_LAUNCH();
    return launch_stats_finalize(a.partial, a.counts, chunks, zd->n, zd->c, eps, stats, s);
}

// ---- apply ----------------------------------------------------------------------------------
// Bound: HBM.  64 channels at 128^3 (537 MB): 103 -> 83 us.
template <typename T, int VEC, bool NT>
__global__ __launch_bounds__(256) void inorm_apply_kernel(const T* __restrict__ z, int ldz, T* __restrict__ y, int ldy,
                                                          int64_t V, int C, int cthreads, int rl,
                                                          const float* __restrict__ stats,
                                                          const float* __restrict__ gamma, const float* __restrict__ beta) {
    const int tid = threadIdx.x;
    const int cl = tid % cthreads, r0 = tid / cthreads;
    const int cv = blockIdx.z * 256 + cl;
    const int n = blockIdx.y;
    if (r0 >= rl || cv * VEC >= C) return;
    NormIn nm{stats, gamma, beta, C, 1};
    float a[VEC], b[VEC];
    norm_coeffs_vec<VEC>(nm, n, cv * VEC, a, b);
    const T* zb = z + ((int64_t)n * V) * ldz + (int64_t)cv * VEC;
    T* yb = y + ((int64_t)n * V) * ldy + (int64_t)cv * VEC;
    block_rows(V, rl, r0, [&](int64_t r, bool second) {
        typename Vec<T, VEC>::raw q[2];
        q[0] = Vec<T, VEC>::raw_load(zb + r * ldz);
        if (second) q[1] = Vec<T, VEC>::raw_load(zb + (r + rl) * ldz);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !second) break;
            float v[VEC];
            Vec<T, VEC>::unpack(q[k], v);
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                float u = norm_u(v[i], a[i], b[i]);
                v[i] = u > 0.f ? u : 0.f;
            }
            Vec<T, VEC>::template store<NT>(yb + (r + k * rl) * ldy, v);
        }
    });
}

// ---- backward -------------------------------------------------------------------------------
// partial[((n*chunks+chunk)*C + c)*2] = (sum g, sum g*zh) over the chunk's rows.
// NT: z is read past the caches, so that what they hold at the end is dy for the apply pass.
template <typename T, int VEC, bool NT>
__global__ __launch_bounds__(256, 4) void inorm_bwd_partial_kernel(const T* __restrict__ dy, int ldg, const T* __restrict__ z,
                                                                int ldz, int64_t V, int C, int cthreads, int rl,
                                                                int rows_per_chunk, const float* __restrict__ stats,
                                                                const float* __restrict__ gamma,
                                                                const float* __restrict__ beta,
                                                                float* __restrict__ partial) {
    typedef typename SumOf<T>::type S;
    __shared__ S red[2 * 256 * VEC], part[256];
    const int tid = threadIdx.x;
    const int cl = tid % cthreads, r0 = tid / cthreads;
    const int cv = blockIdx.z * 256 + cl;
    const int chunk = blockIdx.x, n = blockIdx.y, chunks = gridDim.x;
    const int64_t rbeg = (int64_t)chunk * rows_per_chunk;
    int64_t rend = rbeg + rows_per_chunk;
    if (rend > V) rend = V;
    S sq[2][VEC];
    auto &s = sq[0], &q = sq[1];
#pragma unroll
    for (int i = 0; i < VEC; ++i) { s[i] = 0; q[i] = 0; }
    if (r0 < rl && cv * VEC < C) {
        NormIn nm{stats, gamma, beta, C, 1};
        float a[VEC], b[VEC], mean[VEC], rstd[VEC];
        norm_coeffs_vec<VEC>(nm, n, cv * VEC, a, b, mean, rstd);
        const T* zb = z + ((int64_t)n * V) * ldz + (int64_t)cv * VEC;
        const T* gb = dy + ((int64_t)n * V) * ldg + (int64_t)cv * VEC;
        auto add_row = [&](const float (&v)[VEC], const float (&g)[VEC]) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                float u = norm_u(v[i], a[i], b[i]);
                float gg = u > 0.f ? g[i] : 0.f;
                float zh = (v[i] - mean[i]) * rstd[i];
                s[i] += (S)gg;
                q[i] = sum_fma(gg, zh, q[i]);
            }
        };
        int64_t r = rbeg + r0;
        // Four rows in flight; the additions keep the row order.  The first half of the rows leaves its sums in the thread's own slots
        // of `red`, so that a chain is no longer than with twice as many chunks (128 channels on 96^3: relative error of dgamma 1.1e-7 with
        // 2048 chunks, 1.5e-7 with 1024 in one chain, 1.0e-7 so).  fp64 sums need no cut.
        const bool halves = sizeof(S) == 4 && rows_per_chunk >= 16 * rl;   // a chain worth cutting
#pragma unroll 1
        for (int half = halves ? 0 : 1; half < 2; ++half) {
            const int64_t stop = half ? rend : half_rows(rbeg, rows_per_chunk, rl, rend);
            for (; r + 3 * (int64_t)rl < stop; r += 4 * (int64_t)rl) {
                typename Vec<T, VEC>::raw vr[4], gr[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    vr[u] = Vec<T, VEC>::template raw_load<NT>(zb + (r + u * (int64_t)rl) * ldz);
                    gr[u] = Vec<T, VEC>::raw_load(gb + (r + u * (int64_t)rl) * ldg);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    float v[VEC], g[VEC];
                    Vec<T, VEC>::unpack(vr[u], v);
                    Vec<T, VEC>::unpack(gr[u], g);
                    add_row(v, g);
                }
            }
            if constexpr (sizeof(S) == 4)
                if (half == 0) stash(sq, red);
        }
        for (; r < rend; r += rl) {
            float v[VEC], g[VEC];
            Vec<T, VEC>::load(zb + r * ldz, v);
            Vec<T, VEC>::load(gb + r * ldg, g);
            add_row(v, g);
        }
        if constexpr (sizeof(S) == 4)
            if (halves) unstash(sq, red);
    }
    block_fold<double>(sq, cthreads, rl, red, part, [&](int k, int e, float t) {
        const int c = blockIdx.z * 256 * VEC + e;
        if (c < C) partial[(((size_t)n * chunks + chunk) * C + c) * 2 + k] = t;
    });
}

// sums[n][c][2] = (sum g, sum g*zh) over all parts, fp64, fixed order (strided per thread with four
// parts in flight, then a fixed tree over lanes and waves).
// zstats != nullptr: the second partial sum is over g*z (raw z, from the data-gradient epilogue) and is turned into
// the sum over g*zhat here, in fp64: rstd * (sum g*z - mean * sum g).
__global__ __launch_bounds__(256) void inorm_bwd_finalize_kernel(const float* __restrict__ partial, int parts, int C,
                                                                 float* __restrict__ sums, const float* __restrict__ zstats) {
    __shared__ double sh[4][2];
    const int c = blockIdx.x, n = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float2* pp = reinterpret_cast<const float2*>(partial) + (size_t)n * parts * C + c;
    double s = 0.0, q = 0.0;
    for (int p = tid; p < parts; p += 1024) {
        float2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = pp[(size_t)min(p + 256 * u, parts - 1) * C];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (p + 256 * u < parts) { s += (double)v[u].x; q += (double)v[u].y; }
    }
    s = wave_fold(s);
    q = wave_fold(q);
    if (lane == 0) { sh[wv][0] = s; sh[wv][1] = q; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) { s += sh[w][0]; q += sh[w][1]; }
        if (zstats) q = (double)zstats[((size_t)n * C + c) * 2 + 1] * (q - (double)zstats[((size_t)n * C + c) * 2 + 0] * s);
        sums[((size_t)n * C + c) * 2 + 0] = (float)s;
        sums[((size_t)n * C + c) * 2 + 1] = (float)q;
    }
}

// The sums of one sample from its partials, by every block of the apply pass for itself: tot[2 * C], fp64, a fixed order.  zstats as in
// inorm_bwd_finalize_kernel.  Three barriers a 256 outputs; every thread of the block calls it.
__device__ __forceinline__ void fold_parts(const float* __restrict__ partial, int parts, int n, int C, const float* __restrict__ zstats,
                                           double* sh, float* tot) {
    const int tid = threadIdx.x, nout = 2 * C;
    const float* pp = partial + (size_t)n * parts * nout;
    for (int o0 = 0; o0 < nout; o0 += 256) {
        const int w = min(256, nout - o0), lanes = 256 / w, o = tid % w, p = tid / w;
        double t = 0.0;
        if (p < lanes) {
            const float* q = pp + o0 + o;
            for (int k = p; k < parts; k += 8 * lanes) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = q[(size_t)min(k + u * lanes, parts - 1) * nout];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k + u * lanes < parts) t += (double)v[u];
            }
        }
        sh[tid] = t;
        __syncthreads();
        if (tid < w) {
            for (int k = 1; k < lanes; ++k) t += sh[k * w + tid];
            sh[tid] = t;
        }
        __syncthreads();
        if (tid < w) {
            const int c = (o0 + tid) >> 1;
            if (zstats && (tid & 1)) t = (double)zstats[((size_t)n * C + c) * 2 + 1] * (t - (double)zstats[((size_t)n * C + c) * 2] * sh[tid - 1]);
            tot[o0 + tid] = (float)t;
        }
        __syncthreads();
    }
}
// Where every block of the apply pass folds the partials itself: at most 7 loads a thread (68 channels, 7 partials), which are in flight
// together, in place of a launch (sums and apply of bf16, folded and with the launch: 64 channels on 4^3 7.8 and 9.7 us, 32 on 8^3 8.7 and
// 10.3, 64 on 3 x 6 x 7 x 5 without gradients 8.4 and 9.7, 48 on 6 x 7 x 8 no difference).  Not where several samples' gradients are
// wanted: the block that writes these would fold all samples.
static constexpr int FOLD_C = 512;
static bool fold_in_apply(int parts, int N, int C, int vec, bool grads) {
    return vec > 1 && C <= FOLD_C && (int64_t)parts * C <= 512 && (N == 1 || !grads);
}

// Bound: HBM.  64 channels at 128^3, sums and apply (1.34 GB): 262 -> 214 us with non-temporal accesses (loads too: both inputs are
// read for the last time here).
// FOLD: `sums` holds partials ([N][parts][C][2]), see fold_parts.
template <typename T, int VEC, bool NT, bool FOLD>
__global__ __launch_bounds__(256) void inorm_bwd_apply_kernel(const T* __restrict__ dy, int ldg, const T* __restrict__ z,
                                                              int ldz, T* __restrict__ dz, int ldo, int64_t V, int C,
                                                              int cthreads, int rl, const float* __restrict__ stats,
                                                              const float* __restrict__ gamma,
                                                              const float* __restrict__ beta,
                                                              const float* __restrict__ sums, float* __restrict__ dgamma,
                                                              float* __restrict__ dbeta, float beta_acc, int parts,
                                                              const float* __restrict__ zstats) {
    __shared__ double fsh[FOLD ? 256 : 1];
    __shared__ float tot[FOLD ? 2 * FOLD_C : 1];
    const int tid = threadIdx.x;
    const int cl = tid % cthreads, r0 = tid / cthreads;
    const int cv = blockIdx.z * 256 + cl;
    const int n = blockIdx.y;
    if constexpr (FOLD) {
        fold_parts(sums, parts, n, C, zstats, fsh, tot);
    }
    // (FOLD with gradients is for one sample: `tot` holds no other)
    if (n == 0) affine_grads(FOLD ? tot : sums, FOLD ? 1 : gridDim.y, C, blockIdx.z * 256 * VEC, min(C - (int)blockIdx.z * 256 * VEC, 256 * VEC), dgamma, dbeta, beta_acc);
    if (r0 >= rl || cv * VEC >= C) return;
    NormIn nm{stats, gamma, beta, C, 1};
    float a[VEC], b[VEC], mean[VEC], rstd[VEC], c1[VEC], c2[VEC];
    const float invV = 1.0f / (float)V;
    float sm[2 * VEC];
    if constexpr (FOLD)
#pragma unroll
        for (int i = 0; i < 2 * VEC; ++i) sm[i] = tot[cv * VEC * 2 + i];
    else ld_floats<2 * VEC>(sums + ((size_t)n * C + cv * VEC) * 2, sm);
    norm_coeffs_vec<VEC>(nm, n, cv * VEC, a, b, mean, rstd);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        c1[i] = sm[2 * i] * invV;
        c2[i] = sm[2 * i + 1] * invV;
    }
    const T* zb = z + ((int64_t)n * V) * ldz + (int64_t)cv * VEC;
    const T* gb = dy + ((int64_t)n * V) * ldg + (int64_t)cv * VEC;
    T* ob = dz + ((int64_t)n * V) * ldo + (int64_t)cv * VEC;
    block_rows(V, rl, r0, [&](int64_t r, bool second) {
        typename Vec<T, VEC>::raw q[2], p[2];
        q[0] = Vec<T, VEC>::template raw_load<NT>(zb + r * ldz);
        p[0] = Vec<T, VEC>::template raw_load<NT>(gb + r * ldg);
        if (second) {
            q[1] = Vec<T, VEC>::template raw_load<NT>(zb + (r + rl) * ldz);
            p[1] = Vec<T, VEC>::template raw_load<NT>(gb + (r + rl) * ldg);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !second) break;
            float v[VEC], g[VEC];
            Vec<T, VEC>::unpack(q[k], v);
            Vec<T, VEC>::unpack(p[k], g);
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                float u = norm_u(v[i], a[i], b[i]);
                float gg = u > 0.f ? g[i] : 0.f;
                float zh = (v[i] - mean[i]) * rstd[i];
                v[i] = a[i] * (gg - c1[i] - zh * c2[i]);
            }
            Vec<T, VEC>::template store<NT>(ob + (r + k * rl) * ldo, v);
        }
    });
}

static int apply_blocks(int64_t V, int rl) {
    int64_t b = (V + rl - 1) / rl;
    int64_t cap = 256 * 16;
    b = (b + 3) / 4;  // a few rows per thread
    if (b < 1) b = 1;
    return (int)(b > cap ? cap : b);
}

}  // namespace lamp

using namespace lamp;

extern "C" size_t lamp_inorm_relu_workspace_bytes(const lamp_tensor_desc* zd) {
    if (!desc_ok(zd)) return 0;
    return stats_ws_bytes(zd);
}

extern "C" lamp_status lamp_inorm_relu(const lamp_tensor_desc* zd, const void* z, const float* gamma,
                                       const float* beta, float eps, const lamp_tensor_desc* yd, void* y,
                                       float* stats, int stats_given, void* ws, size_t ws_bytes, void* stream) {
    if (!zd || !yd || !z || !y || !stats) return LAMP_ERR_NULL;
    if (!desc_ok(zd) || !desc_ok(yd) || !same_space(zd, yd) || zd->c != yd->c) return LAMP_ERR_SHAPE;
    if (zd->dtype != yd->dtype) return LAMP_ERR_DTYPE;
    if (!(eps >= 0.f)) return LAMP_ERR_SHAPE;
    hipStream_t s = (hipStream_t)stream;
    if (!stats_given) {
        if (!ws || ws_bytes < stats_ws_bytes(zd)) return LAMP_ERR_WORKSPACE;
        lamp_status st = launch_stats(zd, z, eps, stats, ws, ws_bytes, s);
        if (st != LAMP_OK) return st;
    }
    const int64_t V = (int64_t)zd->d * zd->h * zd->w;
    const int vec = pick_vec(zd->dtype, zd->c, {zd->ldc, yd->ldc}, {z, y});
    const bool nt = beyond_cache(2 * nvox(zd) * zd->c * (int64_t)esize(zd->dtype));
    LAMP_DISPATCH_TV(zd->dtype, vec, {
        RowMap m = make_rowmap(zd->c, VEC, true);
        if (nt) {
            hipLaunchKernelGGL((inorm_apply_kernel<T, VEC, true>), dim3(apply_blocks(V, m.rl), zd->n, m.ctiles), dim3(256), 0, s,
                           (const T*)z, zd->ldc, (T*)y, yd->ldc, V, zd->c, m.cthreads, m.rl, stats, gamma, beta);
        } else {
            hipLaunchKernelGGL((inorm_apply_kernel<T, VEC, false>), dim3(apply_blocks(V, m.rl), zd->n, m.ctiles), dim3(256), 0, s,
                           (const T*)z, zd->ldc, (T*)y, yd->ldc, V, zd->c, m.cthreads, m.rl, stats, gamma, beta);
        }
    });
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

extern "C" lamp_status lamp_inorm_relu_noalloc(const lamp_tensor_desc* zd, const void* z, const float* gamma,
                                               const float* beta, float eps, const lamp_tensor_desc* yd, void* y,
                                               float* stats, void* stream) {
    if (!zd || !yd || !z || !y || !stats) return LAMP_ERR_NULL;
    if (!desc_ok(zd) || !desc_ok(yd)) return LAMP_ERR_SHAPE;
    if (stats_ws_bytes(zd) > (size_t)LAMP_NOALLOC_SCRATCH_BYTES) return LAMP_ERR_WORKSPACE;   // beyond the fixed scratch
    void* ptr = nullptr;
    lamp_status st = noalloc_scratch(&ptr);
    if (st != LAMP_OK) return st;
    // Nothing in the scratch has to start at zero: the statistics pass writes every partial and every count
    // that its second stage reads, so what the previous call left there is never seen.
    return lamp_inorm_relu(zd, z, gamma, beta, eps, yd, y, stats, 0, ptr, (size_t)LAMP_NOALLOC_SCRATCH_BYTES, stream);
}

extern "C" size_t lamp_inorm_relu_bwd_workspace_bytes(const lamp_tensor_desc* zd) {
    if (!desc_ok(zd)) return 0;
    int64_t V = (int64_t)zd->d * zd->h * zd->w;
    int ch = bwd_chunks(V, zd->c, zd->dtype);
    return align_up((size_t)zd->n * ch * zd->c * 2 * sizeof(float)) + align_up((size_t)zd->n * zd->c * 2 * sizeof(float));
}

extern "C" lamp_status lamp_inorm_relu_bwd(const lamp_tensor_desc* dyd, const void* dy, const lamp_tensor_desc* zd,
                                           const void* z, const float* stats, const float* gamma, const float* beta,
                                           const lamp_tensor_desc* dzd, void* dz, float* dgamma, float* dbeta,
                                           float beta_acc, void* ws, size_t ws_bytes, void* stream) {
    if (!dyd || !zd || !dzd || !dy || !z || !stats || !dz) return LAMP_ERR_NULL;
    if (!desc_ok(dyd) || !desc_ok(zd) || !desc_ok(dzd) || !same_space(zd, dyd) || !same_space(zd, dzd) ||
        zd->c != dyd->c || zd->c != dzd->c)
        return LAMP_ERR_SHAPE;
    if (zd->dtype != dyd->dtype || zd->dtype != dzd->dtype) return LAMP_ERR_DTYPE;
    if (beta_acc != 0.f && beta_acc != 1.f) return LAMP_ERR_SHAPE;
    if (!ws || ws_bytes < lamp_inorm_relu_bwd_workspace_bytes(zd)) return LAMP_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const int64_t V = (int64_t)zd->d * zd->h * zd->w;
    const int chunks = bwd_chunks(V, zd->c, zd->dtype);
    float* partial = (float*)ws;
    float* sums = (float*)((char*)ws + align_up((size_t)zd->n * chunks * zd->c * 2 * sizeof(float)));
    const int vec = pick_vec(zd->dtype, zd->c, {zd->ldc, dyd->ldc, dzd->ldc}, {z, dy, dz});
    const bool nt = beyond_cache(2 * nvox(zd) * zd->c * (int64_t)esize(zd->dtype));
    LAMP_DISPATCH_TV(zd->dtype, vec, {
        RowMap m = make_rowmap(zd->c, VEC);
        if (nt) {
            hipLaunchKernelGGL((inorm_bwd_partial_kernel<T, VEC, true>), dim3(chunks, zd->n, m.ctiles), dim3(256), 0, s,
                           (const T*)dy, dyd->ldc, (const T*)z, zd->ldc, V, zd->c, m.cthreads, m.rl, bwd_rows(V, zd->c, zd->dtype),
                           stats, gamma, beta, partial);
        } else {
            hipLaunchKernelGGL((inorm_bwd_partial_kernel<T, VEC, false>), dim3(chunks, zd->n, m.ctiles), dim3(256), 0, s,
                           (const T*)dy, dyd->ldc, (const T*)z, zd->ldc, V, zd->c, m.cthreads, m.rl, bwd_rows(V, zd->c, zd->dtype),
                           stats, gamma, beta, partial);
        }
    });
    LAMP_CHECK_LAUNCH();
    return launch_inorm_bwd_apply(dyd, dy, zd, z, stats, gamma, beta, partial, chunks, nullptr, sums, dzd, dz, dgamma, dbeta, beta_acc, s);
}

lamp_status lamp::launch_inorm_bwd_apply(const lamp_tensor_desc* dyd, const void* dy, const lamp_tensor_desc* zd, const void* z,
                                   const float* stats, const float* gamma, const float* beta, const float* partial, int parts,
                                   const float* zstats, float* sums, const lamp_tensor_desc* dzd, void* dz, float* dgamma, float* dbeta,
                                   float beta_acc, hipStream_t s) {
    const int64_t V = (int64_t)zd->d * zd->h * zd->w;
    const int vec = pick_vec(zd->dtype, zd->c, {zd->ldc, dyd->ldc, dzd->ldc}, {z, dy, dz});
    const bool nt = beyond_cache(3 * nvox(zd) * zd->c * (int64_t)esize(zd->dtype));
    const bool fold = !nt && fold_in_apply(parts, zd->n, zd->c, vec, dgamma || dbeta);
    if (!fold) {
        hipLaunchKernelGGL(inorm_bwd_finalize_kernel, dim3(zd->c, zd->n), dim3(256), 0, s, partial, parts, zd->c, sums, zstats);
        LAMP_CHECK_LAUNCH();
    }
#define LAMP_APPLY(NT, FOLD) \
    hipLaunchKernelGGL((inorm_bwd_apply_kernel<T, VEC, NT, FOLD>), dim3(apply_blocks(V, m.rl), zd->n, m.ctiles), dim3(256), 0, s, \
                       (const T*)dy, dyd->ldc, (const T*)z, zd->ldc, (T*)dz, dzd->ldc, V, zd->c, m.cthreads, m.rl, stats, gamma, beta, \
                       fold ? partial : sums, dgamma, dbeta, beta_acc, parts, zstats)
    LAMP_DISPATCH_TV(zd->dtype, vec, {
        RowMap m = make_rowmap(zd->c, VEC, true);
        if (nt) LAMP_APPLY(true, false);
        else if (VEC > 1 && fold) LAMP_APPLY(false, (VEC > 1));
        else LAMP_APPLY(false, false);
    });
#undef LAMP_APPLY
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}
