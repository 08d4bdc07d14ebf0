// Row kernels of the prefill decoder stack, for gfx950: what stands between
// the library GEMMs and the attention kernels of a layer (RMSNorm with the
// residual add, the per-head norm + rotary embedding + head split of Q, K, V,
// and the SwiGLU product).
//
// All of them are bound by memory: each activation is read once and written
// once, 16 bytes per lane, where a chain of one-operation
// kernels moves it some ten times and pays a launch each.  Arithmetic is fp32
// and every value is rounded to bf16 exactly where the operator-by-operator
// form rounds it (after the residual add, after each norm, after the rotary
// embedding, after silu and after the product); contraction into fma is off
// for the same reason.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/bf1.h"
#include "bf1_device.h"

#pragma clang fp contract(off)

namespace bf1 {
namespace {

constexpr int ROW_THREADS = 256;

__device__ __forceinline__ void unpack8(u32x4 w, float* f) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = __uint_as_float(w[k] << 16);
        f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
}

__device__ __forceinline__ u32x4 pack8(const float* f) {
    bf16x8 b;
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k] = (__bf16)f[k];
    return __builtin_bit_cast(u32x4, b);
}

// ---------------------------------------------------------------------------
// RMSNorm of rows, optionally of h + r with the sum written back to h
// ---------------------------------------------------------------------------
// One wave per row, the row in registers (NC chunks of 8 elements per lane:
// cols <= 512 NC), so it is read once.  RES = 1: x = bf16(h + r) is stored to
// h first and the norm is that of the rounded sum.  8192 x 1024: 12.4 us for
// 67 MB (5.4 TB/s; a large copy reaches 4.9), one operator at a time some 70.
template <int NC, bool RES>
__global__ __launch_bounds__(ROW_THREADS) void rms_kernel(__bf16* __restrict__ h, const __bf16* __restrict__ r,
                                                          const __bf16* __restrict__ gain, __bf16* __restrict__ out,
                                                          int64_t rows, int32_t cols, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (ROW_THREADS / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int nch = cols / 8;
    u32x4* hp = reinterpret_cast<u32x4*>(h + row * cols);
    float x[NC][8];
    u32x4 hw[NC], rw[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        hw[i] = c < nch ? hp[c] : u32x4{0u, 0u, 0u, 0u};
        if (RES) rw[i] = c < nch ? reinterpret_cast<const u32x4*>(r + row * cols)[c] : u32x4{0u, 0u, 0u, 0u};
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        unpack8(hw[i], x[i]);
        if (RES) {
            float y[8];
            unpack8(rw[i], y);
#pragma unroll
            for (int k = 0; k < 8; ++k) x[i][k] += y[k];
            const u32x4 w = pack8(x[i]);
            unpack8(w, x[i]);
            if (lane + 64 * i < nch) hp[lane + 64 * i] = w;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) s += x[i][k] * x[i][k];
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
    const float rs = 1.0f / sqrtf(s / (float)cols + eps);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) {
            float g[8], y[8];
            unpack8(reinterpret_cast<const u32x4*>(gain)[c], g);
#pragma unroll
            for (int k = 0; k < 8; ++k) y[k] = x[i][k] * rs * g[k];
            reinterpret_cast<u32x4*>(out + row * cols)[c] = pack8(y);
        }
    }
}

// ---------------------------------------------------------------------------
// Heads of Q, K and V from the projections
// ---------------------------------------------------------------------------
// q [n, H D], k and v [n, Hkv D] (row strides ldq, ldk, ldv) into head-major
// Q [H, n, D], K, V [Hkv, n, D]; Q and K rows get their RMSNorm and rotary
// embedding on the way (cos, sin: fp32 [n, D], their two halves equal).  D / 16
// lanes per (token, head) row; a lane owns 8 elements of the lower half of the
// row and the 8 they are rotated with, so the rotation stays in the lane.
// 8192 tokens of 16 + 2 * 8 heads of 128: 26 us for 142 MB (5.5 TB/s; 32 us with
// 8-byte loads and D / 8 lanes per row), some 420 as single operators (norms,
// rotations and three transposed copies).
template <int D>
__global__ __launch_bounds__(ROW_THREADS) void heads_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v, int64_t ldq,
    int64_t ldk, int64_t ldv, const __bf16* __restrict__ qgain, const __bf16* __restrict__ kgain,
    const float* __restrict__ cosv, const float* __restrict__ sinv, __bf16* __restrict__ Q, __bf16* __restrict__ K,
    __bf16* __restrict__ V, int32_t n, int32_t H, int32_t Hkv, float eps) {
    constexpr int LPR = D / 16;
    constexpr int RPB = ROW_THREADS / LPR;
    const int32_t heads = H + 2 * Hkv;
    const int64_t p = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
    const int l = threadIdx.x % LPR;
    const bool live = p < (int64_t)n * heads;
    const int32_t tok = live ? (int32_t)(p / heads) : 0;
    const int32_t hd = live ? (int32_t)(p - (int64_t)tok * heads) : 0;
    const __bf16* src;
    __bf16* dst;
    const __bf16* gain;
    if (hd < H) {
        src = q + tok * ldq + (int64_t)hd * D;
        dst = Q + ((int64_t)hd * n + tok) * D;
        gain = qgain;
    } else if (hd < H + Hkv) {
        src = k + tok * ldk + (int64_t)(hd - H) * D;
        dst = K + ((int64_t)(hd - H) * n + tok) * D;
        gain = kgain;
    } else {
        src = v + tok * ldv + (int64_t)(hd - H - Hkv) * D;
        dst = V + ((int64_t)(hd - H - Hkv) * n + tok) * D;
        gain = nullptr;
    }
    u32x4 lo = reinterpret_cast<const u32x4*>(src)[l];
    u32x4 hi = reinterpret_cast<const u32x4*>(src + D / 2)[l];
    float a[8], b[8], s = 0.f;
    unpack8(lo, a);
    unpack8(hi, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) s += a[e] * a[e] + b[e] * b[e];
#pragma unroll
    for (int m = LPR / 2; m > 0; m >>= 1) s += __shfl_xor(s, m);
    if (!live) return;
    if (gain != nullptr) {
        const float rs = 1.0f / sqrtf(s / (float)D + eps);
        float ga[8], gb[8];
        unpack8(reinterpret_cast<const u32x4*>(gain)[l], ga);
        unpack8(reinterpret_cast<const u32x4*>(gain + D / 2)[l], gb);
        const f32x4* cp = reinterpret_cast<const f32x4*>(cosv + (int64_t)tok * D) + 2 * l;
        const f32x4* tp = reinterpret_cast<const f32x4*>(sinv + (int64_t)tok * D) + 2 * l;
        const f32x4 c[2] = {cp[0], cp[1]}, t[2] = {tp[0], tp[1]};
        float ya[8], yb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float na = (float)(__bf16)(a[e] * rs * ga[e]), nb = (float)(__bf16)(b[e] * rs * gb[e]);
            ya[e] = na * c[e >> 2][e & 3] - nb * t[e >> 2][e & 3];
            yb[e] = nb * c[e >> 2][e & 3] + na * t[e >> 2][e & 3];
        }
        lo = pack8(ya);
        hi = pack8(yb);
    }
    reinterpret_cast<u32x4*>(dst)[l] = lo;
    reinterpret_cast<u32x4*>(dst + D / 2)[l] = hi;
}

// ---------------------------------------------------------------------------
// silu(g) * u over [rows, cols] (row strides ldg, ldu), out contiguous
// ---------------------------------------------------------------------------
// 8192 x 3072: 28 us for 151 MB (5.3 TB/s), 46 as two operators.
__global__ __launch_bounds__(ROW_THREADS) void swiglu_kernel(const __bf16* __restrict__ g, const __bf16* __restrict__ u,
                                                             int64_t ldg, int64_t ldu, __bf16* __restrict__ out,
                                                             int64_t rows, int32_t nch) {
    const int64_t x = (int64_t)blockIdx.x * ROW_THREADS + threadIdx.x;
    const int64_t row = x / nch;
    const int32_t c = (int32_t)(x - row * nch);
    if (row >= rows) return;
    float a[8], b[8];
    unpack8(reinterpret_cast<const u32x4*>(g + row * ldg)[c], a);
    unpack8(reinterpret_cast<const u32x4*>(u + row * ldu)[c], b);
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = (float)(__bf16)(a[k] / (1.0f + expf(-a[k]))) * b[k];
    reinterpret_cast<u32x4*>(out)[x] = pack8(a);
}

bool aligned16(const void* p) { return p != nullptr && reinterpret_cast<uintptr_t>(p) % 16 == 0; }

int status_of(hipError_t e) { return e == hipSuccess ? BF1_OK : BF1_ERR_HIP; }

// A launch has fewer than 2^32 threads.
bool launchable(int64_t blocks) { return blocks < (int64_t(1) << 32) / ROW_THREADS; }

template <int NC>
hipError_t launch_rms_nc(void* h, const void* r, const void* gain, void* out, int64_t rows, int32_t cols, float eps,
                         hipStream_t s) {
    const dim3 grid((unsigned)((rows + 3) / 4));
    if (r != nullptr)
        hipLaunchKernelGGL((rms_kernel<NC, true>), grid, dim3(ROW_THREADS), 0, s, (__bf16*)h, (const __bf16*)r,
                           (const __bf16*)gain, (__bf16*)out, rows, cols, eps);
    else
        hipLaunchKernelGGL((rms_kernel<NC, false>), grid, dim3(ROW_THREADS), 0, s, (__bf16*)h, (const __bf16*)nullptr,
                           (const __bf16*)gain, (__bf16*)out, rows, cols, eps);
    return hipGetLastError();
}

}  // namespace
}  // namespace bf1

extern "C" {

int bf1_stack_rms(void* h, const void* r, const void* gain, void* out, int64_t rows, int32_t cols, float eps,
                  void* stream) {
    if (rows < 0 || rows >= (int64_t(1) << 32) || cols < 1) return BF1_ERR_INVALID_ARG;
    if (cols % 8 != 0 || cols > 4096 || !bf1::launchable((rows + 3) / 4)) return BF1_ERR_UNSUPPORTED;
    if (rows == 0) return BF1_OK;
    if (!bf1::aligned16(h) || !bf1::aligned16(gain) || !bf1::aligned16(out) || (r && !bf1::aligned16(r)))
        return BF1_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    // registers hold the whole row: 2, 4 or 8 chunks of 8 elements per lane
    if (cols <= 1024) return bf1::status_of(bf1::launch_rms_nc<2>(h, r, gain, out, rows, cols, eps, s));
    if (cols <= 2048) return bf1::status_of(bf1::launch_rms_nc<4>(h, r, gain, out, rows, cols, eps, s));
    return bf1::status_of(bf1::launch_rms_nc<8>(h, r, gain, out, rows, cols, eps, s));
}

int bf1_stack_heads(const void* q, const void* k, const void* v, int64_t ldq, int64_t ldk, int64_t ldv,
                    const void* qgain, const void* kgain, const float* cosv, const float* sinv, void* Q, void* K,
                    void* V, int64_t n, int32_t H, int32_t Hkv, int32_t head_dim, float eps, void* stream) {
    if (n < 0 || H < 1 || Hkv < 1) return BF1_ERR_INVALID_ARG;
    if (head_dim != 64 && head_dim != 128) return BF1_ERR_UNSUPPORTED;
    if (n >= (int64_t(1) << 24) || H > 4096 || Hkv > 4096) return BF1_ERR_UNSUPPORTED;
    if (n == 0) return BF1_OK;
    for (const void* p : {q, k, v, qgain, kgain, (const void*)cosv, (const void*)sinv,
                          (const void*)Q, (const void*)K, (const void*)V})
        if (!bf1::aligned16(p)) return BF1_ERR_INVALID_ARG;
    if (ldq < (int64_t)H * head_dim || ldk < (int64_t)Hkv * head_dim || ldv < (int64_t)Hkv * head_dim || ldq % 8 ||
        ldk % 8 || ldv % 8)
        return BF1_ERR_INVALID_ARG;
    const int64_t rows = n * (H + 2 * (int64_t)Hkv);
    const int rpb = bf1::ROW_THREADS / (head_dim / 16);
    const int64_t grid = (rows + rpb - 1) / rpb;
    if (!bf1::launchable(grid)) return BF1_ERR_UNSUPPORTED;
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(bf1::ROW_THREADS), 0, (hipStream_t)stream,
                           (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, ldq, ldk, ldv, (const __bf16*)qgain,
                           (const __bf16*)kgain, cosv, sinv, (__bf16*)Q, (__bf16*)K, (__bf16*)V, (int32_t)n, H, Hkv, eps);
        return bf1::status_of(hipGetLastError());
    };
    return head_dim == 64 ? launch(bf1::heads_kernel<64>) : launch(bf1::heads_kernel<128>);
}

int bf1_stack_swiglu(const void* g, const void* u, int64_t ldg, int64_t ldu, void* out, int64_t rows, int32_t cols,
                     void* stream) {
    if (rows < 0 || cols < 1 || rows >= (int64_t(1) << 32)) return BF1_ERR_INVALID_ARG;
    if (cols % 8 != 0) return BF1_ERR_UNSUPPORTED;
    if (rows == 0) return BF1_OK;
    if (!bf1::aligned16(g) || !bf1::aligned16(u) || !bf1::aligned16(out) || ldg < cols || ldu < cols || ldg % 8 ||
        ldu % 8)
        return BF1_ERR_INVALID_ARG;
    const int32_t nch = cols / 8;
    const int64_t grid = (rows * nch + bf1::ROW_THREADS - 1) / bf1::ROW_THREADS;
    if (!bf1::launchable(grid)) return BF1_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(bf1::swiglu_kernel, dim3((unsigned)grid), dim3(bf1::ROW_THREADS), 0, (hipStream_t)stream,
                       (const __bf16*)g, (const __bf16*)u, ldg, ldu, (__bf16*)out, rows, nch);
    return bf1::status_of(hipGetLastError());
}

}  // extern "C"
