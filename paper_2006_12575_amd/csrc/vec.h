// Vector load/store helpers and the (channel-vector, row-lane) thread mapping used by the
// bandwidth-bound NDHWC kernels.
#pragma once
#include <initializer_list>
#include "common.h"

namespace lamp {

template <typename T, int VEC> struct Vec;

// Non-temporal accesses: lines that no later pass will find in the caches are not kept there.
typedef __attribute__((__vector_size__(16))) uint32_t vec_u32x4;
template <bool NT, typename R> __device__ __forceinline__ R ld16(const void* p) {
    static_assert(sizeof(R) == 16, "one 16-byte piece");
    const vec_u32x4* q = reinterpret_cast<const vec_u32x4*>(p);
    return __builtin_bit_cast(R, NT ? __builtin_nontemporal_load(q) : *q);
}
template <bool NT, typename R> __device__ __forceinline__ void st16(void* p, const R& v) {
    static_assert(sizeof(R) == 16, "one 16-byte piece");
    vec_u32x4* q = reinterpret_cast<vec_u32x4*>(p);
    if (NT) __builtin_nontemporal_store(__builtin_bit_cast(vec_u32x4, v), q);
    else *q = __builtin_bit_cast(vec_u32x4, v);
}

// load = raw_load + unpack: kernels with several rows in flight hold them packed.
template <> struct Vec<bf16_t, 8> {
    typedef uint4 raw;
    template <bool NT = false> static __device__ __forceinline__ raw raw_load(const bf16_t* p) { return ld16<NT, raw>(p); }
    static __device__ __forceinline__ void unpack(const raw& q, float (&v)[8]) {
        const uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(r[i] << 16);
            v[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) {
        unpack(raw_load(p), v);
    }
    static __device__ __forceinline__ raw pack(const float (&v)[8]) {
        uint32_t r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = f2bf2(v[2 * i], v[2 * i + 1]);
        return make_uint4(r[0], r[1], r[2], r[3]);
    }
    template <bool NT = false> static __device__ __forceinline__ void raw_store(bf16_t* p, const raw& q) { st16<NT>(p, q); }
    template <bool NT = false> static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) { st16<NT>(p, pack(v)); }
};
template <> struct Vec<float, 4> {
    typedef float4 raw;
    template <bool NT = false> static __device__ __forceinline__ raw raw_load(const float* p) { return ld16<NT, raw>(p); }
    static __device__ __forceinline__ void unpack(const raw& q, float (&v)[4]) { v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w; }
    static __device__ __forceinline__ void load(const float* p, float (&v)[4]) { unpack(raw_load(p), v); }
    static __device__ __forceinline__ raw pack(const float (&v)[4]) { return make_float4(v[0], v[1], v[2], v[3]); }
    template <bool NT = false> static __device__ __forceinline__ void raw_store(float* p, const raw& q) { st16<NT>(p, q); }
    template <bool NT = false> static __device__ __forceinline__ void store(float* p, const float (&v)[4]) { st16<NT>(p, pack(v)); }
};
template <typename T> struct Vec<T, 1> {
    typedef float raw;
    template <bool NT = false> static __device__ __forceinline__ raw raw_load(const T* p) { return io<T>::ld(p); }
    static __device__ __forceinline__ void unpack(const raw& q, float (&v)[1]) { v[0] = q; }
    static __device__ __forceinline__ void load(const T* p, float (&v)[1]) { v[0] = io<T>::ld(p); }
    static __device__ __forceinline__ raw pack(const float (&v)[1]) { return v[0]; }
    template <bool NT = false> static __device__ __forceinline__ void raw_store(T* p, const raw& q) { io<T>::st(p, q); }
    template <bool NT = false> static __device__ __forceinline__ void store(T* p, const float (&v)[1]) { io<T>::st(p, v[0]); }
};

// VEC consecutive floats, 4-byte aligned.
template <int VEC> __device__ __forceinline__ void ld_floats(const float* p, float (&v)[VEC]) { __builtin_memcpy(v, p, sizeof(v)); }

// norm_coeffs of VEC consecutive channels, and (mean, rstd) themselves.  Whole pieces, one branch per optional parameter: channel by
// channel every gamma and beta was a branch and a wait of its own, a chain of sixteen memory latencies in front of a block's first row
// (apply pass with gamma and beta, 64 channels on 83 x 61 x 97: 28.4 us where it took 21.9 without them).
template <int VEC> __device__ __forceinline__ void norm_coeffs_vec(const NormIn& nm, int n, int c0, float (&a)[VEC], float (&b)[VEC],
                                                                   float (&mean)[VEC], float (&rstd)[VEC]) {
    float st[2 * VEC], g[VEC], bt[VEC];
    ld_floats<2 * VEC>(nm.mean_rstd + ((size_t)n * nm.c_norm + c0) * 2, st);
#pragma unroll
    for (int i = 0; i < VEC; ++i) { g[i] = 1.f; bt[i] = 0.f; }
    if (nm.gamma) ld_floats<VEC>(nm.gamma + c0, g);
    if (nm.beta) ld_floats<VEC>(nm.beta + c0, bt);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        mean[i] = st[2 * i];
        rstd[i] = st[2 * i + 1];
        a[i] = g[i] * rstd[i];
        b[i] = bt[i] - mean[i] * a[i];
    }
}
template <int VEC> __device__ __forceinline__ void norm_coeffs_vec(const NormIn& nm, int n, int c0, float (&a)[VEC], float (&b)[VEC]) {
    float mean[VEC], rstd[VEC];
    norm_coeffs_vec<VEC>(nm, n, c0, a, b, mean, rstd);
}

// dgamma, dbeta of channels [c0, c0 + nc): the backward sums over the samples, fp64, in order, by the threads of the apply pass's blocks
// of the first sample, a thread to a channel and sum, the sums of eight samples in flight (a launch of its own took 1.2 to 5 us; one
// thread with eight channels one after the other waited 8 N times in front of its first row).  Called by whole blocks; nothing is read
// where neither is wanted.
__device__ __forceinline__ void affine_grads(const float* sums, int N, int C, int c0, int nc, float* dgamma, float* dbeta, float beta_acc) {
    if (!dgamma && !dbeta) return;
    for (int o = blockIdx.x * 256 + threadIdx.x; o < 2 * nc; o += gridDim.x * 256) {
        const float* p = sums + 2 * c0 + o;
        double t = 0.0;
        for (int n = 0; n < N; n += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(n + u, N - 1) * C * 2];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (n + u < N) t += (double)v[u];
        }
        float* out = o & 1 ? dgamma : dbeta;
        const int c = c0 + (o >> 1);
        if (out) out[c] = (beta_acc != 0.f ? beta_acc * out[c] : 0.f) + (float)t;
    }
}

// Thread mapping inside a 256-thread block: cthreads threads side by side cover the channel
// vectors of one row, rl rows are in flight per block.  Channel-vector tiles beyond 256 go to
// blockIdx.z.
struct RowMap {
    int cthreads, rl, ctiles;
};
inline RowMap make_rowmap(int C, int VEC, bool lines = false) {
    RowMap m;
    int cv = C / VEC;
    m.cthreads = cv < 256 ? cv : 256;
    m.rl = 256 / m.cthreads;
    // whole 128-byte lines to a round of rows where that idles a sixteenth of the threads at most (not in sums, whose order it would change)
    if (lines && VEC > 1)
        for (int r = m.rl; r * 16 >= m.rl * 15; --r)
            if (r * m.cthreads % 8 == 0) { m.rl = r; break; }
    m.ctiles = (cv + 255) / 256;
    return m;
}
// Rows [beg, end) of a block in the elementwise passes: contiguous, in whole row rounds.  fn(r, second) handles row r and, where
// `second`, row r + rl, both loads in flight before the first store.  With the rows of a block strided over the whole tensor and one
// row at a time the apply pass ran at 5.2 TB/s (64 channels at 128^3), contiguous pairs with non-temporal stores at 6.4.
template <typename F> __device__ __forceinline__ void block_rows(int64_t V, int rl, int r0, F fn) {
    const int64_t rounds = (V + rl - 1) / rl, per = (rounds + gridDim.x - 1) / gridDim.x * rl;
    const int64_t beg = blockIdx.x * per;
    int64_t end = beg + per;
    if (end > V) end = V;
    for (int64_t r = beg + r0; r < end; r += 2 * rl) fn(r, r + rl < end);
}
// Passes over more bytes than the memory-side cache holds (256 MB) use non-temporal accesses: nothing of them would be found there.
inline bool beyond_cache(int64_t bytes) { return bytes > ((int64_t)256 << 20); }
// Vector width usable for a tensor set: all channel counts / strides divisible and pointers aligned.
inline int pick_vec(int dtype, int C, std::initializer_list<int> lds, std::initializer_list<const void*> ptrs) {
    int v = dtype == LAMP_BF16 ? 8 : 4;
    if (C % v) return 1;
    for (int l : lds) if (l % v) return 1;
    for (const void* p : ptrs) if (p && (((uintptr_t)p) & 15u)) return 1;
    return v;
}

// Vector load with the optional normalise+ReLU-on-load transform.
template <typename T, int VEC>
__device__ __forceinline__ void load_norm_vec(const T* p, const NormIn& nm, int n, int c0, float (&v)[VEC]) {
    Vec<T, VEC>::load(p, v);
    if (nm.mean_rstd) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            int c = c0 + i;
            if (c < nm.c_norm) {
                float a, b;
                norm_coeffs(nm, n, c, a, b);
                float u = norm_u(v[i], a, b);
                if (nm.relu) u = u > 0.f ? u : 0.f;
                v[i] = io<T>::rnd(u);
            }
        }
    }
}

// The value OFF lanes further on, for the lanes below OFF (of a wave for 32 and 16, of each row of 16 below that): permlane swaps and DPP,
// where a shuffle of a double is two trips through the LDS pipe.
template <int OFF> __device__ __forceinline__ double lanes_down(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint32_t w[2] = {(uint32_t)b, (uint32_t)(b >> 32)};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (OFF == 32) w[i] = __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false)[1];
        else if constexpr (OFF == 16) w[i] = __builtin_amdgcn_permlane16_swap(w[i], w[i], false, false)[1];
        else w[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[i], 0x100 + OFF, 0xf, 0xf, true);
    }
    return __builtin_bit_cast(double, (uint64_t)w[1] << 32 | w[0]);
}
// Lane 0: the sum over the wave, halves folded onto each other.
__device__ __forceinline__ double wave_fold(double v) {
    v += lanes_down<32>(v);
    v += lanes_down<16>(v);
    v += lanes_down<8>(v);
    v += lanes_down<4>(v);
    v += lanes_down<2>(v);
    v += lanes_down<1>(v);
    return v;
}

// The first half of a chunk's rows, in whole groups of four row rounds; a thread's sums over it wait in its own slots of block_fold's
// buffer (no barrier: nobody else touches them before the fold).
__device__ __forceinline__ int64_t half_rows(int64_t rbeg, int rows, int rl, int64_t rend) {
    const int64_t e = rbeg + (rows / 2 + 4 * rl - 1) / (4 * rl) * (4 * rl);
    return e < rend ? e : rend;
}
template <int NV, int VEC> __device__ __forceinline__ void stash(float (&v)[NV][VEC], float* red) {
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            red[k * (256 * VEC) + threadIdx.x * VEC + i] = v[k][i];
            v[k][i] = 0.f;
        }
}
template <int NV, int VEC> __device__ __forceinline__ void unstash(float (&v)[NV][VEC], const float* red) {
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[k][i] += red[k * (256 * VEC) + threadIdx.x * VEC + i];
}

// Type of a thread's backward sums: fp64 for fp32 tensors, whose chunks have several rows to a thread, fp32 for bf16 (bwd_rows, norm.hip).
template <typename T> struct SumOf { typedef float type; };
template <> struct SumOf<float> { typedef double type; };
__device__ __forceinline__ float sum_fma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double sum_fma(float a, float b, double c) { return fma((double)a, (double)b, c); }

// Sums NV sets of VEC values per thread over the row lanes of a block (thread = row lane * cthreads + channel-vector lane) and
// hands each to put(set, channel of the block, sum).  All 256 threads add: with only the first row lane's cthreads threads at
// work, a 16-channel bf16 tensor left 2 threads a serial chain of 2048 LDS reads, which was 45 of the 60 us of its backward sums
// (2 x 64 x 80 x 96 voxels).  `red`: NV * 256 * VEC floats, `part`: 256 floats.  A fixed order for a given cthreads.  A: double in the
// backward sums, whose chunks are the longest: these are the largest addends of a partial and round most.  NT: threads of the block, of which the first 256 have sums.
// V: type of the threads' sums, `red` and `part`.
template <typename A = float, int NT = 256, int NV, int VEC, typename V, typename F>
__device__ __forceinline__ void block_fold(const V (&v)[NV][VEC], int cthreads, int rl, V* red, V* part, F put) {
    const int tid = threadIdx.x, nc = cthreads * VEC, nout = NV * nc;
    const bool on = NT == 256 || tid < 256;
    if (on)
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int i = 0; i < VEC; ++i) red[k * (256 * VEC) + tid * VEC + i] = v[k][i];
    __syncthreads();
    if (nout <= 128) {   // several threads per sum, each a share of the rows, then the shares in order
        const int P = 256 / nout, o = tid % nout, p = tid / nout, k = o / nc, e = o - k * nc;
        A t = 0;
        if (on && p < P)
            for (int r = p; r < rl; r += P) t += (A)red[k * (256 * VEC) + r * nc + e];
        if (on) part[tid] = (V)t;
        __syncthreads();
        if (tid < nout) {
            t = (A)part[tid];
            for (int q = 1; q < P; ++q) t += (A)part[q * nout + tid];
            put(k, e, (float)t);
        }
    } else {
        for (int o = on ? tid : nout; o < nout; o += 256) {
            const int k = o / nc, e = o - k * nc;
            A t = 0;
            for (int r = 0; r < rl; ++r) t += (A)red[k * (256 * VEC) + r * nc + e];
            put(k, e, (float)t);
        }
    }
}

}  // namespace lamp

// Expands BODY with T / VEC bound to the storage type and vector width.
#define LAMP_DISPATCH_TV(dtype, vec, BODY)                                          \
    do {                                                                            \
        if ((dtype) == LAMP_BF16) {                                                 \
            if ((vec) == 8) { typedef bf16_t T; constexpr int VEC = 8; BODY }        \
            else { typedef bf16_t T; constexpr int VEC = 1; BODY }                   \
        } else {                                                                    \
            if ((vec) == 4) { typedef float T; constexpr int VEC = 4; BODY }         \
            else { typedef float T; constexpr int VEC = 1; BODY }                    \
        }                                                                           \
    } while (0)
