// 4-bit form of the offline weight fold for gfx950: the W4A4 setting of the paper's latency table (Sec. 6.4).
// Codes are clipped to +-7 (Sec. 2.3: +-(2^(b-1) - 1)) and stored two per byte, the even index in the low
// nibble, two's complement (the packing of App. B.1 "Quantization": the odd index fills the high nibble).
//   ptq4vm_fold_smoothing_w4   W' = W diag(m), s_w = max|W'| / 7, codes packed [N, K / 2]
#include <hip/hip_fp16.h>

#include "common.hpp"
#include "quant_device.hpp"

namespace {

using ptq4vm::cvt_i32_f32;

constexpr int kThreads = 256;

// Blocks [0, N) quantize one output channel each; blocks [N, N + ceil(K/256)) write 1/m.
__global__ __launch_bounds__(kThreads) void fold_smoothing_w4_rows(const __half *__restrict__ w,
                                                                   const float *__restrict__ m,
                                                                   uint8_t *__restrict__ wq4, float *__restrict__ s_w,
                                                                   float *__restrict__ inv_m, int64_t N, int64_t K,
                                                                   int64_t ldw, int64_t ldwq) {
    const int64_t o = blockIdx.x;
    if (o >= N) {
        const int64_t k = (o - N) * kThreads + threadIdx.x;
        if (k < K) inv_m[k] = 1.0f / m[k];
        return;
    }
    __shared__ float red[kThreads / 64];
    const __half *wrow = w + o * ldw;
    float amax = 0.0f;
    for (int64_t k = threadIdx.x; k < K; k += kThreads) amax = fmaxf(amax, fabsf(__half2float(wrow[k]) * m[k]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
    __syncthreads();
    amax = red[0];
#pragma unroll
    for (int i = 1; i < kThreads / 64; i++) amax = fmaxf(amax, red[i]);
    const float step = (amax == 0.0f) ? 1.0f : amax / 7.0f;
    if (threadIdx.x == 0) s_w[o] = step;
    uint8_t *qrow = wq4 + o * ldwq;
    for (int64_t j = threadIdx.x; j < K / 2; j += kThreads) {
        int q[2];
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const float wf = __half2float(wrow[2 * j + e]) * m[2 * j + e];
            q[e] = min(max(cvt_i32_f32(__builtin_rintf(wf / step)), -7), 7);
        }
        qrow[j] = (uint8_t)(((q[1] & 15) << 4) | (q[0] & 15));
    }
}

}  // namespace

extern "C" int ptq4vm_fold_smoothing_w4(const void *w_f16, const float *m, uint8_t *wq4, float *s_w, float *inv_m,
                                        int64_t N, int64_t K, int64_t ldw, int64_t ldwq, void *stream_) {
    if (!w_f16 || !m || !wq4 || !s_w || !inv_m) return PTQ4VM_ERR_NULL;
    if (N < 0 || K <= 0 || K % 2 != 0) return PTQ4VM_ERR_SHAPE;
    if (ldw < K || ldwq < K / 2) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(w_f16, 16) || !ptq4vm::aligned_to(wq4, 16) || !ptq4vm::aligned_to(m, 4) ||
        !ptq4vm::aligned_to(s_w, 4) || !ptq4vm::aligned_to(inv_m, 4))
        return PTQ4VM_ERR_ALIGN;
    const int64_t blocks = N + ptq4vm::ceil_div(K, kThreads);
    if (blocks > 0x7fffffffLL) return PTQ4VM_ERR_SHAPE;
    fold_smoothing_w4_rows<<<dim3((unsigned)blocks), dim3(kThreads), 0, static_cast<hipStream_t>(stream_)>>>(
        static_cast<const __half *>(w_f16), m, wq4, s_w, inv_m, N, K, ldw, ldwq);
    return ptq4vm::check_launch("fold_smoothing_w4_rows");
}
