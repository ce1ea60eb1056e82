// Fused activation quantizer + linear with a split reduction, included by pts_linear_fused.hip.
#pragma once
#include "gemm_tile.hpp"
#include "quant_device.hpp"

namespace ptq4vm {
namespace mfma {

// Form of a fused launch: 8-bit codes, 4-bit codes (packed weight), or 8-bit codes with a per-token zero offset.
enum class Form { kInt8 = 0, kBits4 = 1, kOffset = 2 };

// One PTS code (Sec. 5.1): smoothing multiply, step multiply, round half to even, clip.  Two
// separate fp32 multiplies in this order: the codes must equal the stand-alone quantizer's.
// BITS4: clip to +-7 (Sec. 2.3 with b = 4) instead of +-127.
// OFFSET: per-token zero offset z (Sec. 5.1; the quantizer of Sec. 2.3 with its code range shifted into int8):
// clip(q + z, -128, 127), formed as clip(q, -128 - z, 127 - z) + z so that a saturated q cannot overflow.
template <bool BITS4, bool OFFSET>
__device__ __forceinline__ int clip_code(int q, int z) {
    if constexpr (OFFSET) return min(max(q, -128 - z), 127 - z) + z;
    return BITS4 ? min(max(q, -7), 7) : min(max(q, -127), 127);
}

// Four int8 bytes holding 4-bit codes -> the same codes times 16 (what the int8 MFMA is fed on the 4-bit path:
// the accumulator is then 256 times the sum, undone exactly in the channel steps).
__device__ __forceinline__ uint32_t times16(uint32_t packed_codes) { return (packed_codes << 4) & 0xF0F0F0F0u; }

// Eight packed 4-bit codes (even index in the low nibble) -> eight int8 bytes, codes times 16, in index order.
__device__ __forceinline__ u32x2 expand_nibbles_in_order(uint32_t p) {
    const uint32_t even = (p << 4) & 0xF0F0F0F0u, odd = p & 0xF0F0F0F0u;  // codes 0, 2, 4, 6 / 1, 3, 5, 7 of the dword, times 16
    return u32x2{__builtin_amdgcn_perm(odd, even, 0x05010400u),   // even.b0, odd.b0, even.b1, odd.b1
                 __builtin_amdgcn_perm(odd, even, 0x07030602u)};  // even.b2, odd.b2, even.b3, odd.b3
}

// f32(fp16 half of `pair`) * m in one instruction: v_fma_mix_f32 converts the selected half exactly,
// multiplies and rounds once to fp32 - the same value as a conversion followed by v_mul_f32.
template <bool HIGH>
__device__ __forceinline__ float half_times(int pair, float m) {
    float d;
    if constexpr (HIGH)
        asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(m));
    else
        asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(m));
    return d;
}

template <bool BITS4, bool OFFSET>
__device__ __forceinline__ int code_of_smoothed(float v, float inv_s, int z) {
    return clip_code<BITS4, OFFSET>(cvt_i32_f32(__builtin_rintf(v * inv_s)), z);
}

// Eight fp16 values (one 16-byte load) -> eight int8 codes (BITS4: 4-bit codes times 16).
template <bool BITS4, bool OFFSET>
__device__ __forceinline__ u32x2 quantize_8(v4i raw, const float (&im)[8], float inv_s, int z) {
    int q[8];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int word = raw[e];  // (a bit_cast applied directly to a vector element reads element 0 with this compiler)
        q[2 * e] = code_of_smoothed<BITS4, OFFSET>(half_times<false>(word, im[2 * e]), inv_s, z);
        q[2 * e + 1] = code_of_smoothed<BITS4, OFFSET>(half_times<true>(word, im[2 * e + 1]), inv_s, z);
    }
    u32x2 out = {pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7])};
    if constexpr (BITS4) out = u32x2{times16(out[0]), times16(out[1])};
    return out;
}

template <Form FORM>
struct FusedPath;
template <>
struct FusedPath<Form::kInt8> {
    using Path = Int8Path;
};
template <>
struct FusedPath<Form::kBits4> {
    using Path = Int4Path;  // operands times 16, the accumulator shifted back in the epilogue
};
template <>
struct FusedPath<Form::kOffset> {
    using Path = Int8OffsetPath;
};

// ------------------------------------------------------------------------------------------
// A workgroup of W wavefronts owns 16 RB token rows x 16 NB channels; wavefront w takes the MFMA steps (64 codes, one
// 128-byte line of fp16 per row) w, w + W, ...  It fetches the rows' lines with whole-line loads (lane s: row 8 i + s / 8,
// 16-byte piece s mod 8), the smoothing factors and the weight operands, turns each eight fp16 into
// eight codes, passes them through a private LDS tile into MFMA operand layout, and the partial sums meet in LDS at the
// end.  No barrier before that: where the weight-resident kernel gives a wavefront the whole reduction of its rows, this
// one spreads it over the workgroup, so that a few thousand rows fill the chip.  The price is the weight read once per
// 16 RB rows (from L2, through the CU's one 64-byte-per-clock load path, which is what bounds long reductions) instead of
// once per CU (us, this / weight-resident: 4137 x 1536 -> 80 14.1 / 10.3, 25216 x 768 -> 56 19.4 / 12.4), so it serves what
// that kernel cannot: fewer rows than fill its CUs, any alignment, tables beyond the LDS.
// kAligned: K % 64 == 0, 16-byte aligned rows of x and of the weight.  Otherwise any K and pitch: weight bytes beyond K
// read as zero, so the codes there do not matter.  (Six blocks of 32 rows: a third wavefront per SIMD is worth a small spill, 37575 x 136 -> 91
// 22.4 / 19.9 us; at three, four and seven blocks a bound that spills loses.)
// ------------------------------------------------------------------------------------------
template <Form FORM, int NB, int RB, int W, Rows ROWS>
__global__ __launch_bounds__(64 * W, (ROWS == Rows::kAny && NB == 6 && RB == 2 ? 3 : 1)) void pts_linear_split(const LinearArgs p) {
    using Path = typename FusedPath<FORM>::Path;
    constexpr bool BITS4 = FORM == Form::kBits4, OFFSET = FORM == Form::kOffset;
    constexpr bool ALIGNED = ROWS == Rows::kAligned;
    static_assert(ALIGNED || FORM == Form::kInt8, "the other forms exist for the shapes of the resident kernel only");
    constexpr int NL = 2 * RB;  // loads of 8 rows per step
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int LDS_BYTES = W * RB * NB * 1024;  // partial sums; before that the wavefronts' code tiles (RB KiB each)
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];

    int tile_r, tile_o;
    if (!tile_of_block(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * 16 * RB, o0 = (int64_t)tile_o * 16 * NB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;  // MFMA operand position: row, 16-code chunk
    const int rr = lane >> 3, pc = lane & 7;    // load position: row within a group of 8, 16-byte piece
    const int64_t K = p.k_bytes;
    const int n_steps = (int)((K + 63) / 64);
    char *const tile = lds + wave * RB * 1024;
    // Code tile: row pitch 64 bytes, 16-byte chunk c of row r at chunk position c ^ (((r >> 1) ^ (r >> 2)) & 3)
    uint32_t tile_wr[NL];
#pragma unroll
    for (int i = 0; i < NL; i++) {
        const int row = i * 8 + rr;
        tile_wr[i] = row * 64 + (((pc >> 1) ^ swizzle(row)) << 4) + (pc & 1) * 8;
    }
    const uint32_t tile_rd = l16 * 64 + ((lq ^ swizzle(l16)) << 4);  // + 1024 per row block

    const char *xrow[NL], *wrow[NB];
    float inv_s[NL];
    int zq[NL];
#pragma unroll
    for (int i = 0; i < NL; i++) {
        const int64_t r = min(r0 + i * 8 + rr, p.M - 1);  // clamped rows are never stored
        xrow[i] = p.x + r * p.ldx_bytes;
        const uint32_t t = token_of(p, r);
        inv_s[i] = p.s_tok[t];
        zq[i] = OFFSET ? p.z_tok[t] : 0;
    }
#pragma unroll
    for (int i = 0; i < NB; i++) wrow[i] = p.w + min(o0 + i * 16 + l16, p.N - 1) * p.ldw_bytes;
    const char *const x_end = p.x + ((p.M - 1) * p.ldx_bytes + K * 2);
    const char *const w_end = p.w + ((p.N - 1) * p.ldw_bytes + K);

    v4i acc[NB][RB];
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < RB; j++) acc[i][j] = v4i{0, 0, 0, 0};

    struct Step {
        v4i x[NL];
        v4f im[2];
        v4i w[BITS4 ? 1 : NB];
        u32x2 w4[BITS4 ? NB : 1];
    };
    auto whole = [&](int s) { return ALIGNED || (int64_t)(s + 1) * 64 <= K; };  // uniform
    auto fetch = [&](Step &f, int s) {
        const int64_t k0 = (int64_t)s * 64;
        if (!whole(s)) {
            auto load_last = [&](const char *at, const char *end) {
                if constexpr (ROWS == Rows::kTiny)
                    return load_bytes(at, end);
                else
                    return load_within(at, end);
            };
#pragma unroll
            for (int i = 0; i < NL; i++) f.x[i] = load_last(xrow[i] + k0 * 2 + pc * 16, x_end);
            f.im[0] = f.im[1] = v4f{1.0f, 1.0f, 1.0f, 1.0f};
            if (p.inv_m) {
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int e = 0; e < 4; e++) f.im[h][e] = p.inv_m[min(k0 + pc * 8 + 4 * h + e, K - 1)];
            }
            if constexpr (!BITS4) {
#pragma unroll
                for (int i = 0; i < NB; i++) f.w[i] = load_last(wrow[i] + k0 + lq * 16, w_end);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; i++)
            f.x[i] = ALIGNED ? __builtin_nontemporal_load(reinterpret_cast<const v4i *>(xrow[i] + k0 * 2 + pc * 16))
                             : *reinterpret_cast<const v4i_unaligned *>(xrow[i] + k0 * 2 + pc * 16);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            f.im[h] = v4f{1.0f, 1.0f, 1.0f, 1.0f};
            if (p.inv_m) f.im[h] = *reinterpret_cast<const f32x4_any *>(p.inv_m + k0 + pc * 8 + 4 * h);
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if constexpr (BITS4) {
                f.w4[i] = *reinterpret_cast<const u32x2 *>(wrow[i] + k0 / 2 + lq * 8);
            } else {
                f.w[i] = ALIGNED ? *reinterpret_cast<const v4i *>(wrow[i] + k0 + lq * 16)
                                 : *reinterpret_cast<const v4i_unaligned *>(wrow[i] + k0 + lq * 16);
            }
        }
    };
    auto compute = [&](Step &f, int s) {
        const int64_t k0 = (int64_t)s * 64;
        if (!whole(s)) {  // (codes beyond K meet weights of zero)
            if (ROWS == Rows::kAny && K % 8 != 0) {
#pragma unroll
                for (int i = 0; i < NL; i++) f.x[i] = place_within(f.x[i], xrow[i] + k0 * 2 + pc * 16, x_end);
            }
            if constexpr (!BITS4) {
                if (ROWS == Rows::kAny && K % 16 != 0) {
#pragma unroll
                    for (int i = 0; i < NB; i++) f.w[i] = place_within(f.w[i], wrow[i] + k0 + lq * 16, w_end);
                }
                const v4i mask = mask_within(k0 + lq * 16, K);
#pragma unroll
                for (int i = 0; i < NB; i++) f.w[i] &= mask;
            }
        }
        float im[8];
#pragma unroll
        for (int e = 0; e < 8; e++) im[e] = f.im[e >> 2][e & 3];
#pragma unroll
        for (int i = 0; i < NL; i++) {
            const u32x2 codes = quantize_8<BITS4, OFFSET>(f.x[i], im, inv_s[i], zq[i]);
            *reinterpret_cast<u32x2 *>(tile + tile_wr[i]) = codes;
            if (p.xq_out && tile_o == 0) {  // parity aid: the codes that the MFMA will see (4-bit form: one code per byte)
                const int64_t r = r0 + i * 8 + rr;
#pragma unroll
                for (int b = 0; b < 8; b++) {
                    const int8_t fed = (int8_t)(codes[b >> 2] >> (8 * (b & 3)));
                    const int64_t k = k0 + pc * 8 + b;
                    if (r < p.M && k < K) p.xq_out[r * p.ldxq_out + k] = BITS4 ? (int8_t)(fed >> 4) : fed;
                }
            }
        }
        asm volatile("" ::: "memory");  // wavefront-private tile: LDS runs a wavefront's accesses in order
        v4i fx[RB];
#pragma unroll
        for (int j = 0; j < RB; j++) fx[j] = *reinterpret_cast<const v4i *>(tile + tile_rd + j * 1024);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < NB; i++) {
            v4i w;
            if constexpr (BITS4) {
                const u32x2 lo = expand_nibbles_in_order(f.w4[i][0]), hi = expand_nibbles_in_order(f.w4[i][1]);
                w = v4i{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
            } else {
                w = f.w[i];
            }
#pragma unroll
            for (int j = 0; j < RB; j++) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, fx[j], acc[i][j], 0, 0, 0);
        }
    };
    Step f;
    if (wave < n_steps) fetch(f, wave);
#pragma unroll
    for (int i = 0; i < NL; i++) inv_s[i] = 1.0f / inv_s[i];  // IEEE division
    for (int s = wave; s < n_steps; s += W) {
        compute(f, s);
        if (s + W < n_steps) fetch(f, s + W);  // (a second step in flight gains nothing: the other wavefronts cover the wait)
    }
    __syncthreads();  // the code tiles are done with
    finish_split<Path, RB, NB, W>(acc, p, lds, r0, o0);
}

}  // namespace mfma
}  // namespace ptq4vm
