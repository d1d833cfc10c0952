// Deterministic second-stage reductions shared by the weight-gradient paths.
#include <mutex>
#include "internal.h"
#include "vec.h"

namespace lamp {

// 16 zero bytes in device memory: the source of the zero padding for the register-free global -> LDS
// copies.  A statically initialised device array that no kernel writes; `used` keeps it in the device
// code object although no kernel names it (a const array would have internal linkage and be dropped
// there, and the lookup below would then fail).  Its address is looked up once per device and checked
// (device memory, reads back as zeros) before any kernel gets it; a first call inside a graph capture on `s` goes without the
// read-back, which a capture does not allow.
__device__ __attribute__((used, aligned(16))) uint32_t lamp_zero16_storage[4] = {0u, 0u, 0u, 0u};
const bf16_t* device_zero16(hipStream_t s) {
    static const bf16_t* cache[64] = {nullptr};
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!cache[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(lamp_zero16_storage)) != hipSuccess || !p) return nullptr;
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice) return nullptr;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) return nullptr;
        if (cap == hipStreamCaptureStatusNone) {
            uint32_t back[4] = {1u, 1u, 1u, 1u};
            if (hipMemcpy(back, p, sizeof(back), hipMemcpyDeviceToHost) != hipSuccess) return nullptr;
            if (back[0] | back[1] | back[2] | back[3]) return nullptr;
        }
        cache[dev] = (const bf16_t*)p;
    }
    return cache[dev];
}

// Block = 256 / SL groups of VO consecutive outputs x SL lanes over the parts; every lane adds its strided parts in order, then
// the lanes are folded by halves: a fixed summation tree, fp64, with one barrier (one for every halving took 5.2 where this takes 4.9 us,
// 512 parts of 27 * 64 outputs).
// Bound: HBM (the parts are read once).  VO = 4 makes a part's row a run of whole 64-byte pieces also where SL lanes leave a block
// few outputs (64->32 transposed conv, 512 parts of 16384: 37 -> 12 us, with the right number of lanes less), and gives a thread
// enough in flight where there are few parts of many outputs (256->256 conv weights, 4 parts of 1.8 M: 21.6 -> 10.6 us).
// LO: the outputs from O1 on come in two floats a part, high parts and, as many outputs behind them, what these leave of the sum.
template <int SL, int VO, bool LO>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ part, int S, int64_t O,
                                                              float* __restrict__ out, float beta, float* __restrict__ out2, int64_t O1) {
    constexpr int GPB = 256 / SL;
    __shared__ double sh[SL > 1 ? 256 * VO : 1];
    const int gl = threadIdx.x % GPB, sl = threadIdx.x / GPB;
    const int64_t o = ((int64_t)blockIdx.x * GPB + gl) * VO;
    typedef typename Vec<float, VO>::raw raw;
    double acc[VO];
#pragma unroll
    for (int i = 0; i < VO; ++i) acc[i] = 0.0;
    auto add = [&](const raw& q) {
        float v[VO];
        Vec<float, VO>::unpack(q, v);
#pragma unroll
        for (int i = 0; i < VO; ++i) acc[i] += (double)v[i];
    };
    const int64_t ld = LO ? 2 * O - O1 : O;
    // eight loads in flight, added in the order of the parts: a loop of load-then-add is a chain of memory latencies
    auto walk = [&](const float* p) __attribute__((always_inline)) {
        int s = sl;
        for (; s + 7 * SL < S; s += 8 * SL) {
            raw v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = Vec<float, VO>::raw_load(p + (int64_t)(s + u * SL) * ld);
#pragma unroll
            for (int u = 0; u < 8; ++u) add(v[u]);
        }
        for (; s + SL < S; s += 2 * SL) {
            const raw v0 = Vec<float, VO>::raw_load(p + (int64_t)s * ld), v1 = Vec<float, VO>::raw_load(p + (int64_t)(s + SL) * ld);
            add(v0);
            add(v1);
        }
        if (s < S) add(Vec<float, VO>::raw_load(p + (int64_t)s * ld));
    };
    if (o < O) {
        walk(part + o);
        if (LO && o >= O1) walk(part + o + (O - O1));
    }
    if constexpr (SL > 1) {
#pragma unroll
        for (int i = 0; i < VO; ++i) sh[i * 256 + threadIdx.x] = acc[i];
        // halves onto each other: across the waves in one trip through LDS, within the first wave by lane moves
        __syncthreads();
        constexpr int KEEP = GPB > 64 ? GPB : 64;
        if (threadIdx.x >= KEEP) return;
#pragma unroll
        for (int i = 0; i < VO; ++i) {
            const double* q = sh + i * 256 + threadIdx.x;
            if constexpr (GPB == 128) acc[i] += q[128];
            else acc[i] = (acc[i] + q[128]) + (q[64] + q[192]);
            if constexpr (GPB <= 32) acc[i] += lanes_down<32>(acc[i]);
            if constexpr (GPB <= 16) acc[i] += lanes_down<16>(acc[i]);
            if constexpr (GPB <= 8) acc[i] += lanes_down<8>(acc[i]);
            if constexpr (GPB <= 4) acc[i] += lanes_down<4>(acc[i]);
        }
    }
    if (sl == 0 && o < O) {
        if (o >= O1) out = out2 - O1;
        float v[VO];
        if (beta != 0.f) {
            Vec<float, VO>::load(out + o, v);
#pragma unroll
            for (int i = 0; i < VO; ++i) v[i] = beta * v[i] + (float)acc[i];
        } else {
#pragma unroll
            for (int i = 0; i < VO; ++i) v[i] = (float)acc[i];
        }
        Vec<float, VO>::store(out + o, v);
    }
}

// Lanes over the parts: as many as leave fewer than 1024 blocks (four a CU), never more than there are parts.  From 1024 blocks on the
// short blocks of many lanes take turns, and their many small reads of every part's row cost more than a longer loop over the parts
// (27648 outputs, 256 parts: 64 lanes 11.0 us, 32 to 8 lanes 3.7, one lane 14.8; 16384 x 512: 12.3, 4.3 with 32).  64 lanes pay for
// a few outputs only (32 x 4096: 4.4 us, with 32 lanes 6.0; 864 x 3000: 6.9 and 5.4).
template <int VO, bool LO>
static void reduce_launch(const float* part, int S, int64_t O, float* out, float beta, hipStream_t s, float* out2, int64_t O1) {
    const int64_t g = O / VO;
    int sl = 1;
    while (2 * sl <= (O <= 256 ? 64 : 32) && 2 * sl <= S && (g * 2 * sl + 255) / 256 < 1024) sl *= 2;
#define LAMP_REDUCE(SL) \
    case SL: hipLaunchKernelGGL((reduce_partials_kernel<SL, VO, LO>), dim3(cdiv(g, 256 / SL)), dim3(256), 0, s, part, S, O, out, beta, out2, O1); break
    switch (sl) {
        LAMP_REDUCE(1);
        LAMP_REDUCE(2);
        LAMP_REDUCE(4);
        LAMP_REDUCE(8);
        LAMP_REDUCE(16);
        LAMP_REDUCE(32);
        LAMP_REDUCE(64);
    }
#undef LAMP_REDUCE
}

lamp_status launch_reduce_partials(const float* part, int S, int64_t O, float* out, float beta, hipStream_t s, float* out2, int64_t O1) {
    const bool lo = out2 != nullptr;
    if (!lo) O1 = O;
    const bool vec = O % 4 == 0 && O1 % 4 == 0 && aligned16(part) && aligned16(out) && aligned16(out2);
    if (vec && lo) reduce_launch<4, true>(part, S, O, out, beta, s, out2, O1);
    else if (vec) reduce_launch<4, false>(part, S, O, out, beta, s, out2, O1);
    else if (lo) reduce_launch<1, true>(part, S, O, out, beta, s, out2, O1);
    else reduce_launch<1, false>(part, S, O, out, beta, s, out2, O1);
    LAMP_CHECK_LAUNCH();
    return LAMP_OK;
}

// rows per chunk: about 2048 chunks, at least 32 rows each
static int col_rows(int64_t rows) {
    int64_t r = (rows + 2047) / 2048;
    return (int)(r < 32 ? 32 : r);
}

// Threads side by side cover the channel vectors of one row; the row lanes are added in order.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const T* __restrict__ t, int64_t rows, int C, int ld,
                                                             int rows_per_chunk, float* __restrict__ part, RowMap m) {
    __shared__ float red[256 * VEC], fold[256];
    const int tid = threadIdx.x, cl = tid % m.cthreads, r0 = tid / m.cthreads;
    const int c0 = (blockIdx.y * 256 + cl) * VEC;
    int64_t rbeg = (int64_t)blockIdx.x * rows_per_chunk, rend = rbeg + rows_per_chunk;
    if (rend > rows) rend = rows;
    float sv[1][VEC];
    auto& s = sv[0];
#pragma unroll
    for (int i = 0; i < VEC; ++i) s[i] = 0.f;
    if (r0 < m.rl && c0 < C)
        for (int64_t r = rbeg + r0; r < rend; r += m.rl) {
            float v[VEC];
            Vec<T, VEC>::load(t + r * ld + c0, v);
#pragma unroll
            for (int i = 0; i < VEC; ++i) s[i] += v[i];
        }
    block_fold(sv, m.cthreads, m.rl, red, fold, [&](int, int e, float t) {
        const int c = blockIdx.y * 256 * VEC + e;
        if (c < C) part[(int64_t)blockIdx.x * C + c] = t;
    });
}

size_t colsum_ws_bytes(int64_t rows, int C) {
    const int cr = col_rows(rows);
    int64_t chunks = (rows + cr - 1) / cr;
    return align_up((size_t)chunks * C * sizeof(float));
}

lamp_status launch_colsum(const void* t, int dtype, int64_t rows, int C, int ld, float* out, float beta, void* ws,
                          size_t ws_bytes, hipStream_t s) {
    const int cr = col_rows(rows);
    int chunks = (int)((rows + cr - 1) / cr);
    if (!ws || ws_bytes < colsum_ws_bytes(rows, C)) return LAMP_ERR_WORKSPACE;
    float* part = (float*)ws;
    const int vec = pick_vec(dtype, C, {ld}, {t});
    const RowMap m = make_rowmap(C, vec);
    dim3 grid(chunks, m.ctiles);
    LAMP_DISPATCH_TV(dtype, vec, {
        hipLaunchKernelGGL((colsum_partial_kernel<T, VEC>), grid, dim3(256), 0, s, (const T*)t, rows, C, ld, cr, part, m);
    });
    LAMP_CHECK_LAUNCH();
    return launch_reduce_partials(part, chunks, C, out, beta, s);
}

}  // namespace lamp
