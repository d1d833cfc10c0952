// 2x2x2 max pooling (stride 2), forward and backward.  Bandwidth-bound; one thread per
// (output voxel, channel vector).
#include <initializer_list>
#include "internal.h"
#include "vec.h"

namespace lamp {

// The optional normalise+ReLU-on-load of VEC channels from c0 on, coefficients fetched once.
template <typename T, int VEC> struct NormVec {
    float a[VEC], b[VEC];
    int left;    // channels of the vector that are normalised
    int relu;
    __device__ __forceinline__ NormVec(const NormIn& nm, int n, int c0) : left(nm.mean_rstd ? nm.c_norm - c0 : 0), relu(nm.relu) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            a[i] = 1.f;
            b[i] = 0.f;
        }
        if (left >= VEC) norm_coeffs_vec<VEC>(nm, n, c0, a, b);
        else
#pragma unroll
            for (int i = 0; i < VEC; ++i)
                if (i < left) norm_coeffs(nm, n, c0 + i, a[i], b[i]);
    }
    __device__ __forceinline__ void apply(float (&v)[VEC]) const {
        if (left <= 0) return;
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            if (i < left) {
                float u = norm_u(v[i], a[i], b[i]);
                if (relu) u = u > 0.f ? u : 0.f;
                v[i] = io<T>::rnd(u);
            }
    }
};
// Work item = (pooled voxel, channel vector), 64 consecutive ones to a wave.
// PAIR: the two voxels of a w pair lie side by side in memory, so the lower 32 lanes fetch the first voxel of 32 items, the upper 32
// the second: an instruction covers a contiguous run (with both voxels on one lane it touches every other 64 bytes at 32 channels),
// and a swap of register halves between the lanes of two such fetches gives every lane both voxels of its own item; stores of the
// full-resolution tensor go back the same way.  For passes beyond the memory-side cache, where it pairs with non-temporal accesses:
// backward of 2 x 128^3 x 32 with the skip's gradient (840 MB) 195 -> 146 us; on 2 x 64^3 x 64, which the cache holds, the second
// item's index arithmetic costs more than it gives (33 -> 40 us).
struct PoolItem { int cv, n; int64_t ov, iv; bool ok; };   // channel vector, sample, pooled voxel, input voxel (2d, 2h, 2w)
template <typename I> __device__ __forceinline__ PoolItem pool_item_t(I i, I total, int Do, int Ho, int Wo, int CV) {
    PoolItem p;
    p.ok = i < total;
    if (!p.ok) i = 0;
    const I ov = i / (I)CV, r = ov / (I)Wo, r2 = r / (I)Ho, n = r2 / (I)Do;
    const int w = (int)(ov - r * (I)Wo), h = (int)(r - r2 * (I)Ho), d = (int)(r2 - n * (I)Do);
    p.cv = (int)(i - ov * (I)CV);
    p.n = (int)n;
    p.ov = (int64_t)ov;
    p.iv = (((int64_t)n * 2 * Do + 2 * d) * 2 * Ho + 2 * h) * 2 * Wo + 2 * w;
    return p;
}
__device__ __forceinline__ PoolItem pool_item(int64_t i, int64_t total, int Do, int Ho, int Wo, int CV) {
    if (total <= (int64_t)0x7FFFFFFF - 64) return pool_item_t<uint32_t>((uint32_t)i, (uint32_t)total, Do, Ho, Wo, CV);
    return pool_item_t<int64_t>(i, total, Do, Ho, Wo, CV);
}
// Swaps the upper lanes of a with the lower lanes of b, dword by dword; applied twice it changes nothing.
template <typename R> __device__ __forceinline__ void pair_swap(R& a, R& b) {
    if constexpr (sizeof(R) == 16) {
        vec_u32x4 u = __builtin_bit_cast(vec_u32x4, a), v = __builtin_bit_cast(vec_u32x4, b);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto q = __builtin_amdgcn_permlane32_swap(u[i], v[i], false, false);
            u[i] = q[0];
            v[i] = q[1];
        }
        a = __builtin_bit_cast(R, u);
        b = __builtin_bit_cast(R, v);
    } else {
        const auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
        a = __builtin_bit_cast(R, (uint32_t)q[0]);
        b = __builtin_bit_cast(R, (uint32_t)q[1]);
    }
}
// PAIR: the wave's two fetches (items j and j + 32) and this lane's own item; else the own item only.
struct PoolWave { PoolItem f0, f1, own; int par; };
template <bool PAIR> __device__ __forceinline__ PoolWave pool_wave(int64_t total, int Do, int Ho, int Wo, int CV) {
    const int lane = threadIdx.x & 63;
    if constexpr (!PAIR) {
        const PoolItem o = pool_item((int64_t)blockIdx.x * 256 + threadIdx.x, total, Do, Ho, Wo, CV);
        return PoolWave{o, o, o, 0};
    }
    const int64_t j = (int64_t)blockIdx.x * 256 + (threadIdx.x & ~63) + (lane & 31);
    PoolWave w;
    w.par = lane >> 5;
    w.f0 = pool_item(j, total, Do, Ho, Wo, CV);
    w.f1 = pool_item(j + 32, total, Do, Ho, Wo, CV);
    w.own = PoolItem{w.par ? w.f1.cv : w.f0.cv, w.par ? w.f1.n : w.f0.n, w.par ? w.f1.ov : w.f0.ov, 0, w.par ? w.f1.ok : w.f0.ok};
    return w;
}
// Both voxels of the own item in row pair (i, j): q0 the first, q1 the second of the w pair.
template <typename T, int VEC, bool NT>
__device__ __forceinline__ void pool_load(const T* x, int ld, const PoolWave& w, int64_t off, typename Vec<T, VEC>::raw& q0,
                                          typename Vec<T, VEC>::raw& q1) {
    q0 = q1 = typename Vec<T, VEC>::raw{};
    if constexpr (!NT) {
        if (!w.own.ok) return;
        q0 = Vec<T, VEC>::raw_load(x + (w.own.iv + off) * ld + w.own.cv * VEC);
        q1 = Vec<T, VEC>::raw_load(x + (w.own.iv + off + 1) * ld + w.own.cv * VEC);
        return;
    }
    if (w.f0.ok) q0 = Vec<T, VEC>::template raw_load<NT>(x + (w.f0.iv + off + w.par) * ld + w.f0.cv * VEC);
    if (w.f1.ok) q1 = Vec<T, VEC>::template raw_load<NT>(x + (w.f1.iv + off + w.par) * ld + w.f1.cv * VEC);
    pair_swap(q0, q1);
}
template <typename T, int VEC, bool NT>
__device__ __forceinline__ void pool_store(T* y, int ld, const PoolWave& w, int64_t off, const float (&v0)[VEC], const float (&v1)[VEC]) {
    typename Vec<T, VEC>::raw q0 = Vec<T, VEC>::pack(v0), q1 = Vec<T, VEC>::pack(v1);
    if constexpr (!NT) {
        if (!w.own.ok) return;
        Vec<T, VEC>::raw_store(y + (w.own.iv + off) * ld + w.own.cv * VEC, q0);
        Vec<T, VEC>::raw_store(y + (w.own.iv + off + 1) * ld + w.own.cv * VEC, q1);
        return;
    }
    pair_swap(q0, q1);
    if (w.f0.ok) Vec<T, VEC>::template raw_store<NT>(y + (w.f0.iv + off + w.par) * ld + w.f0.cv * VEC, q0);
    if (w.f1.ok) Vec<T, VEC>::template raw_store<NT>(y + (w.f1.iv + off + w.par) * ld + w.f1.cv * VEC, q1);
}

// Forward (paired fetches and non-temporal accesses cost here: 2 x 128^3 x 32 with the activated tensor written 105 -> 120 us).
template <typename T, int VEC>
__global__ __launch_bounds__(256) void maxpool2_fwd_kernel(const T* __restrict__ x, int ldx, NormIn nm, T* __restrict__ y,
                                                           int ldy, int N, int Do, int Ho, int Wo, int C,
                                                           T* __restrict__ yfull = nullptr, int ldyf = 0) {
    const int CV = C / VEC;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = (int64_t)N * Do * Ho * Wo * CV;
    if (idx >= total) return;
    const int cv = (int)(idx % CV);
    int64_t ov = idx / CV;
    const int w = (int)(ov % Wo);
    int64_t r = ov / Wo;
    const int h = (int)(r % Ho);
    r /= Ho;
    const int d = (int)(r % Do);
    const int n = (int)(r / Do);
    const int H = 2 * Ho, W = 2 * Wo, D = 2 * Do;
    float m[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) m[i] = -INFINITY;
    if (yfull) {
        // also write the activated input: all channels normalised, the coefficients of this thread's channels
        // fetched once, the two voxels of a w pair stored back to back
        float a[VEC], b[VEC];
        norm_coeffs_vec<VEC>(nm, n, cv * VEC, a, b);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int i = t >> 1, j = t & 1;
            const int64_t iv = (((int64_t)n * D + 2 * d + i) * H + 2 * h + j) * W + 2 * w;
            float v0[VEC], v1[VEC];
            Vec<T, VEC>::load(x + iv * ldx + cv * VEC, v0);
            Vec<T, VEC>::load(x + (iv + 1) * ldx + cv * VEC, v1);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                float u0 = norm_u(v0[e], a[e], b[e]), u1 = norm_u(v1[e], a[e], b[e]);
                if (nm.relu) { u0 = u0 > 0.f ? u0 : 0.f; u1 = u1 > 0.f ? u1 : 0.f; }
                v0[e] = io<T>::rnd(u0); v1[e] = io<T>::rnd(u1);
                const float mm = v0[e] > v1[e] ? v0[e] : v1[e];
                m[e] = mm > m[e] ? mm : m[e];
            }
            Vec<T, VEC>::store(yfull + iv * ldyf + cv * VEC, v0);
            Vec<T, VEC>::store(yfull + (iv + 1) * ldyf + cv * VEC, v1);
        }
        Vec<T, VEC>::store(y + ov * ldy + cv * VEC, m);
        return;
    }
    for (int t = 0; t < 8; ++t) {
        int i = t >> 2, j = (t >> 1) & 1, k = t & 1;
        const T* p = x + ((((int64_t)n * D + 2 * d + i) * H + 2 * h + j) * W + 2 * w + k) * ldx + cv * VEC;
        float v[VEC];
        load_norm_vec<T, VEC>(p, nm, n, cv * VEC, v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) m[e] = v[e] > m[e] ? v[e] : m[e];
    }
    Vec<T, VEC>::store(y + ov * ldy + cv * VEC, m);
}

// Forward with the activated tensor, bf16, a power of two up to 32 channel vectors: a thread per (w, channel vector) of the four rows of a
// pooled row, so that every access of a wave is 1 KB in a row (a thread per pooled voxel touched every other 64 bytes at 32 channels);
// the other voxel of the pair sits CV lanes away.  W is even, so pairs never part.  Bound: HBM: 2 x 128^3 x 32 105 -> 91 us,
// 75 x 64^3 x 32 602 -> 515 us, past the caches (570 with plain accesses).
template <bool NT>
__global__ __launch_bounds__(256) void inorm_pool_rows_kernel(const bf16_t* __restrict__ x, int ldx, NormIn nm, bf16_t* __restrict__ y, int ldy,
                                                              int Do, int Ho, int W, int lcv, int64_t total, bf16_t* __restrict__ yfull, int ldyf) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;   // (whole pairs: total is a multiple of 2 * CV)
    const int cv = (int)idx & ((1 << lcv) - 1);
    const int64_t v = idx >> lcv;
    int w, h, d, n;
    if (total < (int64_t)0x7FFFFFFF) {
        const uint32_t u = (uint32_t)v, r = u / (uint32_t)W, r2 = r / (uint32_t)Ho, r3 = r2 / (uint32_t)Do;
        w = (int)(u - r * (uint32_t)W); h = (int)(r - r2 * (uint32_t)Ho); d = (int)(r2 - r3 * (uint32_t)Do); n = (int)r3;
    } else {
        const int64_t r = v / W, r2 = r / Ho, r3 = r2 / Do;
        w = (int)(v - r * W); h = (int)(r - r2 * Ho); d = (int)(r2 - r3 * Do); n = (int)r3;
    }
    int64_t iv[4];
    uint4 q[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        iv[t] = ((((int64_t)n * Do + d) * 2 + (t >> 1)) * 2 * Ho + 2 * h + (t & 1)) * W + w;
        q[t] = Vec<bf16_t, 8>::template raw_load<NT>(x + iv[t] * ldx + cv * 8);
    }
    float a[8], b[8], m[8];
    norm_coeffs_vec<8>(nm, n, cv * 8, a, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float f[8], o[8];
        Vec<bf16_t, 8>::unpack(q[t], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            f[e] = norm_u(f[e], a[e], b[e]);
            if (nm.relu) f[e] = f[e] > 0.f ? f[e] : 0.f;
        }
        const uint4 k = Vec<bf16_t, 8>::pack(f);
        Vec<bf16_t, 8>::template raw_store<NT>(yfull + iv[t] * ldyf + cv * 8, k);
        const uint4 kp = make_uint4(__shfl_xor(k.x, 1 << lcv), __shfl_xor(k.y, 1 << lcv), __shfl_xor(k.z, 1 << lcv), __shfl_xor(k.w, 1 << lcv));
        Vec<bf16_t, 8>::unpack(k, f);
        Vec<bf16_t, 8>::unpack(kp, o);
#pragma unroll
        for (int e = 0; e < 8; ++e) {   // of an even w: the voxel itself, then its neighbour, as in raster order (a NaN never wins)
            m[e] = f[e] > m[e] ? f[e] : m[e];
            m[e] = o[e] > m[e] ? o[e] : m[e];
        }
    }
    if (!(w & 1)) Vec<bf16_t, 8>::store(y + ((((int64_t)n * Do + d) * Ho + h) * (W / 2) + (w >> 1)) * ldy + cv * 8, m);
}

// Bound: HBM.  NT (passes beyond the memory-side cache): PAIR, and full-resolution tensors are read and written past the caches.
template <typename T, int VEC, bool NT>
__global__ __launch_bounds__(256) void maxpool2_bwd_kernel(const T* __restrict__ x, int ldx, NormIn nm,
                                                           const T* __restrict__ dy, int ldg, const T* __restrict__ add,
                                                           int lda, T* __restrict__ dx, int ldo, int N, int Do, int Ho,
                                                           int Wo, int C) {
    const int CV = C / VEC;
    const int64_t total = (int64_t)N * Do * Ho * Wo * CV;
    const PoolWave w = pool_wave<NT>(total, Do, Ho, Wo, CV);
    typename Vec<T, VEC>::raw q[8], qa[8];
    int64_t off[4];
    auto gr = typename Vec<T, VEC>::raw{};
    if (w.own.ok) gr = Vec<T, VEC>::raw_load(dy + w.own.ov * ldg + w.own.cv * VEC);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        off[t] = ((int64_t)(t >> 1) * 2 * Ho + (t & 1)) * 2 * Wo;
        pool_load<T, VEC, NT>(x, ldx, w, off[t], q[2 * t], q[2 * t + 1]);
        if (add) pool_load<T, VEC, NT>(add, lda, w, off[t], qa[2 * t], qa[2 * t + 1]);
    }
    NormVec<T, VEC> nv(nm, w.own.n, w.own.cv * VEC);
    float m[VEC];
    int arg[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) { m[i] = -INFINITY; arg[i] = 0; }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        float v[VEC];
        Vec<T, VEC>::unpack(q[t], v);
        nv.apply(v);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if (v[e] > m[e]) { m[e] = v[e]; arg[e] = t; }
    }
    float g[VEC];
    Vec<T, VEC>::unpack(gr, g);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float o[2][VEC];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (add) Vec<T, VEC>::unpack(qa[2 * t + k], o[k]);
            else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) o[k][e] = 0.f;
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) o[k][e] += (arg[e] == 2 * t + k) ? g[e] : 0.f;
        }
        pool_store<T, VEC, NT>(dx, ldo, w, off[t], o[0], o[1]);
    }
}

}  // namespace lamp

using namespace lamp;


static lamp_status pool_shapes(const lamp_tensor_desc* xd, const lamp_tensor_desc* yd) {
    if (!desc_ok(xd) || !desc_ok(yd)) return LAMP_ERR_SHAPE;
    if ((xd->d & 1) || (xd->h & 1) || (xd->w & 1)) return LAMP_ERR_SHAPE;
    if (yd->n != xd->n || yd->d * 2 != xd->d || yd->h * 2 != xd->h || yd->w * 2 != xd->w || yd->c != xd->c)
        return LAMP_ERR_SHAPE;
    if (xd->dtype != yd->dtype) return LAMP_ERR_DTYPE;
    return LAMP_OK;
}

// InstanceNorm + ReLU of a raw conv output and the max-pool of the result in one pass: writes the activated
// tensor (yfull, channel stride ldyf) and its pooled version.  Same arithmetic and rounding as the two
// separate passes; one read of the full-resolution tensor less.
lamp_status lamp::inorm_relu_maxpool2(const lamp_tensor_desc* xd, const void* z, const lamp_norm_in* xnorm, void* yfull, int ldyf,
                                      const lamp_tensor_desc* yd, void* y, hipStream_t s) {
    if (!xd || !yd || !z || !y || !yfull || !xnorm || !xnorm->mean_rstd) return LAMP_ERR_NULL;
    lamp_status st = pool_shapes(xd, yd);
    if (st != LAMP_OK) return st;
    if ((st = norm_ok(xnorm, xd)) != LAMP_OK) return st;
    if (xnorm->c_norm != xd->c) return LAMP_ERR_SHAPE;
    const int vec = pick_vec(xd->dtype, xd->c, {xd->ldc, yd->ldc, ldyf}, {z, y, yfull});
    NormIn nm = make_norm(xnorm);
    const int cv = xd->c / 8;
    if (xd->dtype == LAMP_BF16 && vec == 8 && cv <= 32 && (cv & (cv - 1)) == 0) {
        int lcv = 0;
        while ((1 << lcv) < cv) ++lcv;
        const int64_t total = nvox(yd) * 2 * cv;
        if (beyond_cache(2 * nvox(xd) * xd->c * 2))
            hipLaunchKernelGGL((inorm_pool_rows_kernel<true>), dim3(cdiv(total, 256)), dim3(256), 0, s, (const bf16_t*)z, xd->ldc, nm, (bf16_t*)y,
                               yd->ldc, yd->d, yd->h, xd->w, lcv, total, (bf16_t*)yfull, ldyf);
        else
            hipLaunchKernelGGL((inorm_pool_rows_kernel<false>), dim3(cdiv(total, 256)), dim3(256), 0, s, (const bf16_t*)z, xd->ldc, nm, (bf16_t*)y,
                               yd->ldc, yd->d, yd->h, xd->w, lcv, total, (bf16_t*)yfull, ldyf);
        LAMP_CHECK_LAUNCH();
        return LAMP_OK;
    }
    LAMP_DISPATCH_TV(xd->dtype, vec, {
        int64_t total = nvox(yd) * (xd->c / VEC);
        hipLaunchKernelGGL((maxpool2_fwd_kernel<T, VEC>), dim3(cdiv(total, 256)), dim3(256), 0, s, (const T*)z, xd->ldc, nm,
                       (T*)y, yd->ldc, yd->n, yd->d, yd->h, yd->w, xd->c, (T*)yfull, ldyf);
    });
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

extern "C" lamp_status lamp_maxpool2_fwd(const lamp_tensor_desc* xd, const void* x, const lamp_norm_in* xnorm,
                                         const lamp_tensor_desc* yd, void* y, void* stream) {
    if (!xd || !yd || !x || !y) return LAMP_ERR_NULL;
    lamp_status st = pool_shapes(xd, yd);
    if (st != LAMP_OK) return st;
    if ((st = norm_ok(xnorm, xd)) != LAMP_OK) return st;
    const int vec = pick_vec(xd->dtype, xd->c, {xd->ldc, yd->ldc}, {x, y});
    NormIn nm = make_norm(xnorm);
    LAMP_DISPATCH_TV(xd->dtype, vec, {
        int64_t total = nvox(yd) * (xd->c / VEC);
        hipLaunchKernelGGL((maxpool2_fwd_kernel<T, VEC>), dim3(cdiv(total, 256)), dim3(256), 0, (hipStream_t)stream,
                       (const T*)x, xd->ldc, nm, (T*)y, yd->ldc, yd->n, yd->d, yd->h, yd->w, xd->c);
    });
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

extern "C" lamp_status lamp_maxpool2_bwd(const lamp_tensor_desc* xd, const void* x, const lamp_norm_in* xnorm,
                                         const lamp_tensor_desc* dyd, const void* dy, const lamp_tensor_desc* addd,
                                         const void* add, const lamp_tensor_desc* dxd, void* dx, void* stream) {
    if (!xd || !dyd || !dxd || !x || !dy || !dx) return LAMP_ERR_NULL;
    lamp_status st = pool_shapes(xd, dyd);
    if (st != LAMP_OK) return st;
    if (!desc_ok(dxd) || !same_space(xd, dxd) || dxd->c != xd->c) return LAMP_ERR_SHAPE;
    if (dxd->dtype != xd->dtype) return LAMP_ERR_DTYPE;
    int lda = 0;
    if (add) {
        if (!addd) return LAMP_ERR_NULL;
        if (!desc_ok(addd) || !same_space(xd, addd) || addd->c != xd->c) return LAMP_ERR_SHAPE;
        if (addd->dtype != xd->dtype) return LAMP_ERR_DTYPE;
        lda = addd->ldc;
    }
    if ((st = norm_ok(xnorm, xd)) != LAMP_OK) return st;
    const int vec = pick_vec(xd->dtype, xd->c, {xd->ldc, dyd->ldc, dxd->ldc, add ? lda : xd->ldc}, {x, dy, dx, add});
    NormIn nm = make_norm(xnorm);
    const bool nt = beyond_cache(2 * nvox(xd) * xd->c * (int64_t)esize(xd->dtype));
    LAMP_DISPATCH_TV(xd->dtype, vec, {
        int64_t total = nvox(dyd) * (xd->c / VEC);
        if (nt) {
            hipLaunchKernelGGL((maxpool2_bwd_kernel<T, VEC, true>), dim3(cdiv(total, 256)), dim3(256), 0, (hipStream_t)stream,
                           (const T*)x, xd->ldc, nm, (const T*)dy, dyd->ldc, (const T*)add, lda, (T*)dx, dxd->ldc,
                           dyd->n, dyd->d, dyd->h, dyd->w, xd->c);
        } else {
            hipLaunchKernelGGL((maxpool2_bwd_kernel<T, VEC, false>), dim3(cdiv(total, 256)), dim3(256), 0, (hipStream_t)stream,
                           (const T*)x, xd->ldc, nm, (const T*)dy, dyd->ldc, (const T*)add, lda, (T*)dx, dxd->ldc,
                           dyd->n, dyd->d, dyd->h, dyd->w, xd->c);
        }
    });
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}
