// Per-Token Static activation quantizer for gfx950 (Sec. 5.1; App. B.1 smoothing + quantization
// fused):  xq[r,k] = clip(rne((f32(x[r,k]) * inv_m[k]) * (1 / s_tok[r mod L])), -127, 127).
// and its 4-bit form (codes clipped to +-7, two per byte) and zero-offset form.
//
// The kernel is a pure stream (2 B read + 1 B, or half a byte, written per element), so everything is arranged
// for HBM: 128-bit loads, consecutive lanes on consecutive addresses, several loads in flight
// per lane, and no per-element index arithmetic.  The grid is a fixed, small number of
// workgroups per CU that stride over the rows together.  The total thread count is a multiple of the
// chunks per row, so a thread keeps ONE column chunk (8 channels) for its whole life: the
// smoothing factors sit in registers and the row index advances by a constant, the token position
// without a modulo.
#include <hip/hip_fp16.h>

#include "common.hpp"
#include "quant_device.hpp"

namespace {

using ptq4vm::cvt_i32_f32;
using ptq4vm::pack4;

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));  // (float vectors are 4-byte aligned at the boundary)

constexpr int kMaxThreads = 256;
constexpr int kMaxLdsTokens = 16384;  // reciprocal-step table of up to 64 KiB; longer sequences divide per row

enum class Form { kInt8, kOffset, kBits4 };

// kOffset: per-token zero offset (Sec. 5.1 names it; quantizer form of Sec. 2.3 with the code range shifted
// into int8): the offset is added to the rounded value and the clip range is [-128, 127].
// kBits4: codes clipped to +-7 (Sec. 2.3 with b = 4).
template <Form FORM>
__device__ __forceinline__ int quantize_one(float x, float inv_m, float inv_s, int z) {
    float v = x * inv_m;  // smoothing first (two separate fp32 multiplies, never fused or reordered)
    v = v * inv_s;
    int q = cvt_i32_f32(__builtin_rintf(v));  // round half to even, then NaN -> 0, Inf -> +-INT_MAX
    if constexpr (FORM == Form::kOffset) {
        q = min(max(q, -(1 << 20)), 1 << 20);  // room for the offset without integer overflow
        return min(max(q + z, -128), 127);
    }
    return FORM == Form::kBits4 ? min(max(q, -7), 7) : min(max(q, -127), 127);
}

template <Form FORM>
struct CodesOf {
    using Out = u32x2;  // 8 x int8
};
template <>
struct CodesOf<Form::kBits4> {
    using Out = uint32_t;  // 8 x 4 bits, the even index in the low nibble (the packing of App. B.1)
};

template <Form FORM>
__device__ __forceinline__ typename CodesOf<FORM>::Out quantize_chunk(u32x4 in, const float (&im)[8], float inv_s, int z) {
    int q[8];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const uint32_t word = in[e];
        const __half2 h = __builtin_bit_cast(__half2, word);
        q[2 * e] = quantize_one<FORM>(__low2float(h), im[2 * e], inv_s, z);
        q[2 * e + 1] = quantize_one<FORM>(__high2float(h), im[2 * e + 1], inv_s, z);
    }
    if constexpr (FORM == Form::kBits4) {
        uint32_t r = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) r |= ((uint32_t)q[i] & 15u) << (4 * i);
        return r;
    } else {
        return u32x2{pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7])};
    }
}

// Column-stationary grid-stride stream.  gridDim.x * 256 is a multiple of `chunks` (= K / 8, rounded up),
// so thread g owns column chunk g mod chunks and rows g / chunks + i * row_step, i = 0, 1, ...
// TABLE: reciprocal steps (and offsets) of all token positions in LDS; without it each row divides for itself.
// ALIGNED: chunks are aligned to their size on both sides.  Otherwise any pitch and any K >= 8: the last chunk of a row
// starts at K - 8 and overlaps its neighbour (both write the same codes there).
template <Form FORM, bool HAS_M, bool TABLE, bool ALIGNED>
__global__ __launch_bounds__(kMaxThreads) void quantize_pts_stream(
    const __half *__restrict__ x, const float *__restrict__ inv_m, const float *__restrict__ s_tok,
    const int32_t *__restrict__ z_tok, uint8_t *__restrict__ xq, int64_t M, int L, int K, int chunks, int64_t ldx,
    int64_t ldxq, int64_t row_step) {
    using Out = typename CodesOf<FORM>::Out;
    typedef u32x4 InAny __attribute__((aligned(2)));
    typedef Out OutAny __attribute__((aligned(1)));
    constexpr bool kOffset = FORM == Form::kOffset;
    extern __shared__ float inv_s_lds[];  // [L] reciprocal steps, then (kOffset) [L] offsets
    int *const z_lds = reinterpret_cast<int *>(inv_s_lds + L);

    const uint32_t gtid = blockIdx.x * kMaxThreads + threadIdx.x;  // (fewer than 2^31 threads)
    const uint32_t row32 = gtid / (uint32_t)chunks;
    const int chunk8 = (int)(gtid - row32 * (uint32_t)chunks) * 8;
    const int col = ALIGNED ? chunk8 : min(chunk8, K - 8);
    int64_t row = row32;
    uint32_t t = row32 % (uint32_t)L;  // (unsigned: t + t_step passes 2^31 for the longest sequences)
    const uint32_t t_step = (uint32_t)(row_step % L);
    const __half *xp = x + row * ldx + col;
    uint8_t *qp = xq + row * ldxq + (FORM == Form::kBits4 ? col / 2 : col);
    const int64_t x_step = row_step * ldx, q_step = row_step * ldxq;
    auto load = [&](const __half *ptr) {
        if constexpr (ALIGNED)
            return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(ptr));
        else
            return (u32x4)*reinterpret_cast<const InAny *>(ptr);
    };
    auto store = [&](uint8_t *ptr, Out codes) {
        if constexpr (ALIGNED)
            ptq4vm::store_for_next_kernel(reinterpret_cast<Out *>(ptr), codes);
        else
            *reinterpret_cast<OutAny *>(ptr) = codes;
    };

    constexpr int UNROLL = 2;
    u32x4 v[UNROLL];
    float is[UNROLL], im[8];
    int zs[UNROLL];
    auto fetch = [&]() {  // the rows row, row + row_step of this thread
#pragma unroll
        for (int u = 0; u < UNROLL; u++)
            if (row + u * row_step < M) v[u] = load(xp + u * x_step);
    };
    auto fetch_factors = [&]() {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            f32x4 four = {1.0f, 1.0f, 1.0f, 1.0f};
            if constexpr (HAS_M) four = *reinterpret_cast<const f32x4 *>(inv_m + col + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; e++) im[4 * h + e] = four[e];
        }
    };
    auto steps = [&]() {
#pragma unroll
        for (int u = 0; u < UNROLL; u++) {
            is[u] = TABLE ? inv_s_lds[t] : 1.0f / s_tok[t];
            zs[u] = kOffset ? (TABLE ? z_lds[t] : z_tok[t]) : 0;
            t += t_step;
            if (t >= (uint32_t)L) t -= (uint32_t)L;
        }
    };
    auto finish = [&]() {
#pragma unroll
        for (int u = 0; u < UNROLL; u++)
            if (row + u * row_step < M) store(qp + u * q_step, quantize_chunk<FORM>(v[u], im, is[u], zs[u]));
        row += UNROLL * row_step;
        xp += UNROLL * x_step;
        qp += UNROLL * q_step;
    };

    if constexpr (TABLE) {
        for (int i = threadIdx.x; i < L; i += kMaxThreads) {
            inv_s_lds[i] = 1.0f / s_tok[i];  // IEEE-correct division (compiled without fast-math)
            if constexpr (kOffset) z_lds[i] = z_tok[i];
        }
        __syncthreads();
        fetch_factors();
        while (row < M) {
            fetch();
            steps();
            finish();
        }
    } else {
        // few rows per thread: the first ones are requested ahead of everything else
        fetch();
        fetch_factors();
        while (row < M) {
            steps();
            finish();
            fetch();
        }
    }
}

// Rows of fewer than 8 elements (or absurdly many): one byte of codes per thread-iteration, index arithmetic per element.
template <Form FORM>
__global__ __launch_bounds__(kMaxThreads) void quantize_pts_any(
    const __half *__restrict__ x, const float *__restrict__ inv_m, const float *__restrict__ s_tok,
    const int32_t *__restrict__ z_tok, uint8_t *__restrict__ xq, int64_t M, int64_t L, int64_t K, int64_t ldx,
    int64_t ldxq) {
    constexpr int PER = FORM == Form::kBits4 ? 2 : 1;  // codes per byte
    const int64_t per_row = K / PER, total = M * per_row;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = e / per_row;
        const int64_t j = e - r * per_row;
        const float inv_s = 1.0f / s_tok[r % L];
        const int z = FORM == Form::kOffset ? z_tok[r % L] : 0;
        int byte = 0;
#pragma unroll
        for (int h = 0; h < PER; h++) {
            const int64_t k = j * PER + h;
            const int q = quantize_one<FORM>(__half2float(x[r * ldx + k]), inv_m ? inv_m[k] : 1.0f, inv_s, z);
            byte |= PER == 1 ? q : (q & 15) << (4 * h);
        }
        xq[r * ldxq + j] = (uint8_t)byte;
    }
}

int64_t gcd64(int64_t a, int64_t b) {
    while (b) {
        int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

template <Form FORM>
int launch(const __half *x, const float *inv_m, const float *s_tok, const int32_t *z_tok, uint8_t *xq, int64_t M, int64_t L,
           int64_t K, int64_t ldx, int64_t ldxq, hipStream_t stream) {
    const dim3 block(kMaxThreads);
    const int64_t chunks = ptq4vm::ceil_div(K, 8);
    // Grid: a multiple of `unit` workgroups (so that threads % chunks == 0), fewer than needed when the threads can walk
    // over several rows: about 3 per CU of the 256-CU part for long walks, 6 for short ones (us, 3 / 6 per CU: one Vim-S
    // block over 128 x 197 rows 96.3 / 97.5, but the quantizer alone at 12608 x 384 5.3 / 4.9).
    const int64_t unit = chunks / gcd64(chunks, kMaxThreads);
    int64_t want = M * chunks > 8 * 768 * kMaxThreads ? 768 : 1536;
    const int64_t needed = ptq4vm::ceil_div(M * chunks, kMaxThreads);
    if (want > needed) want = needed;
    const int64_t blocks = ptq4vm::ceil_div(want, unit) * unit;
    if (K < 8 || blocks > 0x7fffffLL) {  // (2^31 threads: rows of tens of millions of elements)
        int64_t any = ptq4vm::ceil_div(M * K, kMaxThreads);
        if (any > 65536) any = 65536;
        quantize_pts_any<FORM><<<dim3((unsigned)any), block, 0, stream>>>(x, inv_m, s_tok, z_tok, xq, M, L, K, ldx, ldxq);
        return ptq4vm::check_launch("quantize_pts_any");
    }
    const int64_t row_step = blocks * kMaxThreads / chunks;
    const bool offset = FORM == Form::kOffset, bits4 = FORM == Form::kBits4;
    // A table of reciprocal steps is a serial start (load, divide, barrier) that pays from about five rows per thread
    // (us, table / each row for itself: 12608 x 1536 [6 rows] 11.5 / 11.9, 3152 x 768 [1] 4.0 / 3.6, 197 x 384 2.3 / 2.0).
    // (K that is no multiple of 8 used to take an element-wise kernel: 12608 x 334 13.4 us, now 5.4; packed codes of
    // 12608 x 1000 21.9 us, now 9.0.)
    const bool table = M > 4 * row_step && L <= (offset ? kMaxLdsTokens / 2 : kMaxLdsTokens);
    const size_t lds = table ? (size_t)L * sizeof(float) * (offset ? 2 : 1) : 0;
    const bool aligned = K % 8 == 0 && ldx % 8 == 0 && ldxq % (bits4 ? 4 : 8) == 0;
    using Kernel = void (*)(const __half *, const float *, const float *, const int32_t *, uint8_t *, int64_t, int, int, int, int64_t, int64_t, int64_t);
    static const Kernel kernels[2][2][2] = {  // [smoothing][table][aligned]
        {{quantize_pts_stream<FORM, false, false, false>, quantize_pts_stream<FORM, false, false, true>},
         {quantize_pts_stream<FORM, false, true, false>, quantize_pts_stream<FORM, false, true, true>}},
        {{quantize_pts_stream<FORM, true, false, false>, quantize_pts_stream<FORM, true, false, true>},
         {quantize_pts_stream<FORM, true, true, false>, quantize_pts_stream<FORM, true, true, true>}}};
    kernels[inv_m ? 1 : 0][table ? 1 : 0][aligned ? 1 : 0]<<<dim3((unsigned)blocks), block, lds, stream>>>(
        x, inv_m, s_tok, z_tok, xq, M, (int)L, (int)K, (int)chunks, ldx, ldxq, row_step);
    return ptq4vm::check_launch("quantize_pts_stream");
}

template <Form FORM>
int quantize_entry(const void *x_f16, const float *inv_m, const float *s_tok, const int32_t *z_tok, void *xq, int64_t B,
                   int64_t L, int64_t K, int64_t ldx, int64_t ldxq, void *stream_) {
    constexpr int PER = FORM == Form::kBits4 ? 2 : 1;  // codes per byte
    if (B < 0 || L <= 0 || K <= 0 || K % PER != 0) return PTQ4VM_ERR_SHAPE;
    if (L > 0x7fffffffLL || K > 0x7fffffffLL || (B > 0 && L > INT64_MAX / B)) return PTQ4VM_ERR_SHAPE;
    if (ldx < K || ldxq < K / PER) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(x_f16, 16) || !ptq4vm::aligned_to(xq, 16) || !ptq4vm::aligned_to(s_tok, 4) ||
        !ptq4vm::aligned_to(z_tok, 4) || (inv_m && !ptq4vm::aligned_to(inv_m, 4)))
        return PTQ4VM_ERR_ALIGN;
    const int64_t M = B * L;
    if (M == 0) return PTQ4VM_OK;
    return launch<FORM>(static_cast<const __half *>(x_f16), inv_m, s_tok, z_tok, static_cast<uint8_t *>(xq), M, L, K, ldx, ldxq,
                        static_cast<hipStream_t>(stream_));
}

}  // namespace

extern "C" int ptq4vm_quantize_pts(const void *x_f16, const float *inv_m, const float *s_tok, int8_t *xq,
                                   int64_t B, int64_t L, int64_t K, int64_t ldx, int64_t ldxq, void *stream_) {
    if (!x_f16 || !s_tok || !xq) return PTQ4VM_ERR_NULL;
    return quantize_entry<Form::kInt8>(x_f16, inv_m, s_tok, nullptr, xq, B, L, K, ldx, ldxq, stream_);
}

extern "C" int ptq4vm_quantize_pts_offset(const void *x_f16, const float *inv_m, const float *s_tok,
                                          const int32_t *z_tok, int8_t *xq, int64_t B, int64_t L, int64_t K,
                                          int64_t ldx, int64_t ldxq, void *stream_) {
    if (!x_f16 || !s_tok || !z_tok || !xq) return PTQ4VM_ERR_NULL;
    return quantize_entry<Form::kOffset>(x_f16, inv_m, s_tok, z_tok, xq, B, L, K, ldx, ldxq, stream_);
}

extern "C" int ptq4vm_quantize_pts_a4(const void *x_f16, const float *inv_m, const float *s_tok, uint8_t *xq4, int64_t B,
                                      int64_t L, int64_t K, int64_t ldx, int64_t ldxq, void *stream_) {
    if (!x_f16 || !s_tok || !xq4) return PTQ4VM_ERR_NULL;
    return quantize_entry<Form::kBits4>(x_f16, inv_m, s_tok, nullptr, xq4, B, L, K, ldx, ldxq, stream_);
}
