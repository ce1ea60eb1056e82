// Tile kernels of the MFMA linears for problems that do not fill the chip with 256 x 256 tiles
// (small and medium row counts, narrow outputs): included by gemm_tile.hip, which holds their dispatch.
//
//   linear_mfma_tile    BR x BO tiles, one workgroup each, both operands copied global -> LDS directly
//   linear_mfma_splitk  a few hundred tiles or fewer: the wavefronts of a workgroup share one small tile
//                       and split the reduction, operands go from memory straight into registers
#pragma once
#include <type_traits>

#include "mfma_linear.hpp"

namespace ptq4vm {
namespace mfma {

// Token position of row r (a 64-bit remainder is some 150 instructions; hardly any problem needs it).
__device__ __forceinline__ uint32_t token_of(const LinearArgs &p, int64_t r) {
    return p.M <= 0x7fffffffLL ? (uint32_t)r % (uint32_t)p.L : (uint32_t)(r % p.L);
}

// 16-byte accesses at any byte address and 8- / 16-byte ones at any even address: gfx950 takes unaligned vector accesses
typedef int v4i_unaligned __attribute__((ext_vector_type(4), aligned(1)));
typedef float v4f_unaligned __attribute__((ext_vector_type(4), aligned(2)));
typedef float v2f_unaligned __attribute__((ext_vector_type(2), aligned(2)));

// Dequantization and fp16 rounding of four neighbouring channels of one row; the result is the four fp16 as raw words.
template <class Path>
__device__ __forceinline__ v2f finish_four(const typename Path::Acc16 acc, float rs, int rz, const v4f cs, const v4i cz,
                                           const v2f bias4) {
    float a[4], s[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if constexpr (Path::kElemBytes == 1 && std::is_same_v<typename Path::Acc16, v4f>) {  // integers carried in fp32 (E2M3)
            a[c] = acc[c];
            s[c] = rs * cs[c];
        } else if constexpr (Path::kElemBytes == 1) {
            int v = acc[c];
            if constexpr (Path::kPacked4) v >>= 8;              // operands were codes times 16: exact
            if constexpr (Path::kOffset) v -= __mul24(rz, cz[c]);  // |z| < 2^8, |rowsum| < 2^23
            a[c] = (float)v;
            s[c] = rs * cs[c];
        } else {
            a[c] = acc[c];
            s[c] = 1.0f;
        }
    }
    const float b01 = bias4.x, b23 = bias4.y;
    return v2f{dequantize_pair_f16(a[0], s[0], a[1], s[1], b01), dequantize_pair_f16(a[2], s[2], a[3], s[3], b23)};
}

// One MFMA step (64 bytes of K) of an FO x FR block of 16 x 16 tiles.
template <class Path, int FO, int FR>
__device__ __forceinline__ void mfma_step(typename Path::Acc16 (&acc)[FO][FR], const v4i (&fw)[FO], const v4i (&fx)[FR]) {
    if constexpr (Path::kPacked4) {
#pragma unroll
        for (int half = 0; half < 2; half++) {
            v4i ew[FO], ex[FR];
#pragma unroll
            for (int i = 0; i < FO; i++) ew[i] = half ? Path::odd_codes(fw[i]) : Path::even_codes(fw[i]);
#pragma unroll
            for (int j = 0; j < FR; j++) ex[j] = half ? Path::odd_codes(fx[j]) : Path::even_codes(fx[j]);
#pragma unroll
            for (int j = 0; j < FR; j++)
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(ew[i], ex[j], acc[i][j]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < FR; j++)
#pragma unroll
            for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(fw[i], fx[j], acc[i][j]);
    }
}

// Eight fp16 results of a row, n_valid of them inside the matrix; rows may start at any even address.  Through the caches:
// with non-temporal stores instead the blocks of all sizes take the same time (a Vim-S block over 64 x 785 rows 149.8 / 149.3 us,
// the offset block of Vim-B over 64 x 197 rows 121.1 / 121.4, a fp16 Vim-S block over 128 x 197 rows 101.7 / 101.5), and lines that
// two stores share have to meet in the L2 (15614 x 128 -> 2310, 4620-byte rows: 29 - 48 us non-temporal, 22 us through it).
__device__ __forceinline__ void store_eight(char *dst, v4f data, int n_valid) {
    if (n_valid >= 8) {
        *reinterpret_cast<v4f_unaligned *>(dst) = data;
        return;
    }
    const float w[4] = {data.x, data.y, data.z, data.w};
#pragma unroll
    for (int e = 0; e < 7; e++)
        if (e < n_valid)
            reinterpret_cast<uint16_t *>(dst)[e] = (uint16_t)(__builtin_bit_cast(uint32_t, w[e >> 1]) >> (16 * (e & 1)));
}

// 16 bytes of a row at byte kb, bytes at or beyond k_bytes read as 0; `end` is the end of the matrix.
__device__ __forceinline__ v4i load_any(const char *row, int64_t kb, int64_t k_bytes, const char *end) {
    v4i out = {0, 0, 0, 0};
    const int64_t valid = k_bytes - kb;
    if (valid <= 0) return out;
    if (row + kb + 16 <= end) {
        out = *reinterpret_cast<const v4i_unaligned *>(row + kb);
        if (valid < 16) {
#pragma unroll
            for (int j = 0; j < 4; j++) out[j] = (int)keep_low_bytes((uint32_t)out[j], (int)valid - 4 * j);
        }
        return out;
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; b++)
            if (4 * j + b < valid) v |= (uint32_t) * reinterpret_cast<const uint8_t *>(row + kb + 4 * j + b) << (8 * b);
        out[j] = (int)v;
    }
    return out;
}

// The step, bias and offset vectors of a BR x BO tile, in LDS behind the ring.  fetch() loads one element per thread
// (before the first operand copies, so that it returns ahead of them), park() writes them to LDS.  Channels and rows
// beyond the matrix are clamped; they are never stored.
template <class Path, int BR, int BO, int THREADS>
struct TileVectors {
    static_assert(BO <= THREADS && BR <= THREADS, "one thread per channel and per row");
    static constexpr bool kInt8 = Path::kElemBytes == 1;
    float *cs;     // s_w of the tile's channels
    int *cz;       // their weight row sums
    float *rs;     // s_tok of the tile's rows
    int *rz;       // their zero offsets
    uint16_t *cb;  // bias of the channels, raw fp16
    float col_s = 1.0f, row_s = 1.0f;
    int col_z = 0, row_z = 0;
    uint16_t col_b = 0;

    __device__ __forceinline__ explicit TileVectors(char *lds)
        : cs(reinterpret_cast<float *>(lds)), cz(reinterpret_cast<int *>(cs + BO)), rs(reinterpret_cast<float *>(cz + BO)),
          rz(reinterpret_cast<int *>(rs + BR)), cb(reinterpret_cast<uint16_t *>(rz + BR)) {}
    __device__ __forceinline__ void fetch(const LinearArgs &p, int tid, int64_t r0, int64_t o0, int rows_valid, int cols_valid) {
        if (tid < BO) {
            const int64_t o = o0 + min(tid, cols_valid - 1);
            if constexpr (kInt8) col_s = p.s_w[o];
            if constexpr (Path::kOffset) col_z = p.rowsum[o];
            if (p.bias) col_b = reinterpret_cast<const uint16_t *>(p.bias)[o];
        }
        if constexpr (kInt8) {
            if (tid < BR) {
                const uint32_t t = ((uint32_t)(r0 % p.L) + (uint32_t)min(tid, rows_valid - 1)) % (uint32_t)p.L;
                row_s = p.s_tok[t];
                if constexpr (Path::kOffset) row_z = p.z_tok[t];
            }
        }
    }
    __device__ __forceinline__ void park(int tid) {
        if (tid < BO) {
            cs[tid] = col_s;
            cb[tid] = col_b;
            if constexpr (Path::kOffset) cz[tid] = col_z;
        }
        if (tid < BR) {
            rs[tid] = row_s;
            if constexpr (Path::kOffset) rz[tid] = row_z;
        }
    }
};
template <int BR, int BO>
constexpr int tile_vector_bytes() {
    return BO * (4 + 2 + 4) + BR * (4 + 4);
}

// Epilogue of a workgroup: every wavefront dequantizes its (BR / WR) x (BO / WO) accumulators, transposes them through
// its own patch of the ring (RING_BYTES, free by now) and stores whole row segments.
template <class Path, int BR, int BO, int WR, int WO, int RING_BYTES, int FO, int FR, class Vectors>
__device__ __forceinline__ void store_tile(const typename Path::Acc16 (&acc)[FO][FR], const LinearArgs &p, char *ring, const Vectors &vec,
                                           int64_t r0, int64_t o0, int rows_valid, int cols_valid) {
    constexpr bool kInt8 = Path::kElemBytes == 1;
    constexpr int NW = WR * WO, WAVE_R = BR / WR, WAVE_O = BO / WO;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;

    // Accumulator register v of block (i, j): token row 16 j + l16, channel 16 i + 4 lq + v.
    if constexpr (kInt8) {
        if (p.acc_out) {
#pragma unroll
            for (int i = 0; i < FO; i++)
#pragma unroll
                for (int j = 0; j < FR; j++)
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        const int r = wave_r + j * 16 + l16, o = wave_o + i * 16 + lq * 4 + c;
                        if (r < rows_valid && o < cols_valid)
                            p.acc_out[(r0 + r) * p.N + o0 + o] = Path::kPacked4 ? (int)acc[i][j][c] >> 8 : (int)acc[i][j][c];
                    }
        }
    }

    constexpr int CPR = WAVE_O / 8, RPS = 64 / CPR;  // 16-byte chunks per patch row, rows per store instruction
    constexpr int FIT = RING_BYTES / NW / (16 * WAVE_O * 2);
    constexpr int JB = FIT >= FR ? FR : (FIT >= 2 && FR % 2 == 0 ? 2 : 1);  // 16-row blocks per round
    static_assert(FIT >= 1 && RPS <= 16 * JB, "patches fit the ring");
    char *const patch = ring + wave * (JB * 16 * WAVE_O * 2);
    auto patch_chunk = [&](int row, int chunk) {
        const int sw = CPR >= 8 ? (row & 7) : ((row / (8 / CPR)) & (CPR - 1));
        return row * (WAVE_O * 2) + ((chunk ^ sw) << 4);
    };
    char *const y_tile = reinterpret_cast<char *>(p.y + r0 * p.ldy + o0);
#pragma unroll
    for (int jb = 0; jb < FR; jb += JB) {
#pragma unroll
        for (int jj = 0; jj < JB; jj++) {
            const int j = jb + jj;
            const float rs = vec.rs[wave_r + j * 16 + l16];
            const int rz = Path::kOffset ? vec.rz[wave_r + j * 16 + l16] : 0;
#pragma unroll
            for (int i = 0; i < FO; i++) {
                const int col = wave_o + i * 16 + lq * 4;
                const v4f cs = *reinterpret_cast<const v4f *>(vec.cs + col);
                const v2f cb = *reinterpret_cast<const v2f *>(vec.cb + col);
                v4i cz = {0, 0, 0, 0};
                if constexpr (Path::kOffset) cz = *reinterpret_cast<const v4i *>(vec.cz + col);
                *reinterpret_cast<v2f *>(patch + patch_chunk(jj * 16 + l16, 2 * i + (lq >> 1)) + (lq & 1) * 8) =
                    finish_four<Path>(acc[i][j], rs, rz, cs, cz, cb);
            }
        }
        asm volatile("" ::: "memory");  // wavefront-private patch: LDS runs a wavefront's accesses in order
#pragma unroll
        for (int s = 0; s < JB * 16 / RPS; s++) {
            const int prow = s * RPS + lane / CPR, chunk = lane % CPR;
            const v4f data = *reinterpret_cast<const v4f *>(patch + patch_chunk(prow, chunk));
            const int r = wave_r + jb * 16 + prow, o = wave_o + chunk * 8;
            if (r < rows_valid && o < cols_valid)
                store_eight(y_tile + (int64_t)r * p.ldy * 2 + o * 2, data, cols_valid - o);
        }
        asm volatile("" ::: "memory");
    }
}

// ------------------------------------------------------------------------------------------
// One BR x BO tile per workgroup.  K is walked in slabs of SLAB bytes per row through a ring of STAGES LDS stages; what
// bounds a workgroup is the latency of its copies and of its stores, so the shape of the kernel is small: few registers
// and 33 - 76 KiB of LDS (17 - 66 with the slabs through registers) let 2 - 4 (2 - 8) workgroups share a CU, and one's
// epilogue runs under the others' MFMAs without any pipelining inside the workgroup.  The step, bias and offset vectors
// are fetched before the first copy and wait in LDS, and results cross a wavefront-private patch into 16-byte stores of whole row segments (25216 x 768 -> 384: 15.6 us
// = 2.5 TB/s, 22.3 us with the tile kernel before, whose epilogue loaded each scale where it was used).
// COPY kDirect: 16-byte aligned bases and pitches, k_bytes % 64 == 0; slabs are copied global -> LDS directly.  Otherwise any
// pitch, alignment and K: slabs pass through registers, one in flight, bytes beyond K zeroed (two stages).  Only the last
// slab reaches beyond K; the loads of the others carry no tests (16236 x 1584 -> 760 fp16 106.7 -> 62.8 us, 24104 x 830 -> 760
// 45.7 -> 36.1, 3184 x 1000 -> 500 12.3 -> 10.3, each with the larger tiles that this pays for; 69.1, 43.4 and 12.3 with the
// tiles alone).  A reduction of one slab keeps the tested loads alone (kOneSlab): the second form costs it 2 %.
// Requirements (host-checked): L < 2^31, BR * ldx_bytes and BO * ldw_bytes below 2^31.
// ------------------------------------------------------------------------------------------
template <int BR, int BO, int SLAB, int STAGES>
constexpr int tile_lds_bytes() {
    return STAGES * (BR + BO) * SLAB + tile_vector_bytes<BR, BO>();
}

enum class Copy { kDirect, kRegisters, kOneSlab };

template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES, Copy COPY>
__global__ __launch_bounds__(64 * WR * WO) void linear_mfma_tile(const LinearArgs p) {
    constexpr bool ALIGNED = COPY == Copy::kDirect;
    constexpr int NW = WR * WO, THREADS = 64 * NW;
    constexpr int WAVE_R = BR / WR, WAVE_O = BO / WO, FR = WAVE_R / 16, FO = WAVE_O / 16;
    constexpr int CHUNKS = SLAB / 16, ROWS_PER_COPY = 64 / CHUNKS, COPIES = (BR + BO) / ROWS_PER_COPY / NW;
    constexpr int STAGE_BYTES = (BR + BO) * SLAB;
    static_assert(SLAB == 64 || SLAB == 128, "LDS rows hold 64 or 128 bytes of K");
    static_assert(WAVE_R % 16 == 0 && WAVE_O % 16 == 0, "wave tile must be whole MFMA blocks");
    static_assert(ALIGNED || STAGES == 2, "the register-staged form is double buffered");
    static_assert((BR + BO) % (ROWS_PER_COPY * NW) == 0 && BR % ROWS_PER_COPY == 0, "every wavefront issues the same number of copies");
    static_assert(STAGES >= 2 && (STAGES - 2) * COPIES <= 63, "vmcnt is a 6-bit counter");
    using Acc = typename Path::Acc16;

    int tile_r, tile_o;
    if (!tile_of_block(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;
    const int rows_valid = (int)min((int64_t)BR, p.M - r0), cols_valid = (int)min((int64_t)BO, p.N - o0);
    auto chunk_of = [&](int row, int chunk) { return chunk ^ (SLAB == 64 ? swizzle(row) : (row & 7)); };

    char *const ring = lds_dyn;
    TileVectors<Path, BR, BO, THREADS> vec(lds_dyn + STAGES * STAGE_BYTES);
    vec.fetch(p, tid, r0, o0, rows_valid, cols_valid);

    // Copies: 1 KiB per wavefront and instruction, linear on the LDS side, so the swizzle is applied by choosing
    // which global chunk a lane fetches.  Copy c covers LDS rows ROWS_PER_COPY c ..: activation rows, then weights.
    // The register-staged form writes the same LDS places from registers.
    uint32_t off[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; i++) {
        const int row = (wave + NW * i) * ROWS_PER_COPY + lane / CHUNKS;
        const int chunk = chunk_of(row, lane % CHUNKS);  // (BR is a multiple of 16: a weight row swizzles like row - BR)
        const bool is_x = row < BR;
        const int src_row = is_x ? min(row, rows_valid - 1) : min(row - BR, cols_valid - 1);
        off[i] = (uint32_t)src_row * (uint32_t)(is_x ? p.ldx_bytes : p.ldw_bytes) + (ALIGNED ? chunk * 16 : 0);
    }
    const char *gx = p.x + r0 * p.ldx_bytes, *gw = p.w + o0 * p.ldw_bytes;
    v4i staged[ALIGNED ? 1 : COPIES];
    auto issue = [&](int slab, int stage) {  // ALIGNED: copy a slab into a ring stage; otherwise fetch it into registers
#pragma unroll
        for (int i = 0; i < COPIES; i++) {
            const int c = wave + NW * i;  // scalar
            const char *src = c * ROWS_PER_COPY < BR ? gx : gw;
            if constexpr (ALIGNED) {
                // the last slab of a K that ends in half a slab: the far chunks re-read the near ones, nobody uses them
                if (SLAB == 128 && (int64_t)(slab + 1) * SLAB > p.k_bytes) src -= chunk_of(c * ROWS_PER_COPY + lane / CHUNKS, lane % CHUNKS) & 4 ? 64 : 0;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (int64_t)slab * SLAB + off[i]),
                                                 (__attribute__((address_space(3))) void *)(ring + stage * STAGE_BYTES + c * 1024), 16, 0, 0);
            } else {
                const int chunk = chunk_of(c * ROWS_PER_COPY + lane / CHUNKS, lane % CHUNKS);
                if (COPY == Copy::kRegisters && (int64_t)(slab + 1) * SLAB <= p.k_bytes) {  // a slab inside the rows
                    staged[i] = *reinterpret_cast<const v4i_unaligned *>(src + off[i] + (int64_t)slab * SLAB + chunk * 16);
                    continue;
                }
                const char *end = c * ROWS_PER_COPY < BR ? p.x + ((p.M - 1) * p.ldx_bytes + p.k_bytes) : p.w + ((p.N - 1) * p.ldw_bytes + p.k_bytes);
                staged[i] = load_any(src + off[i], (int64_t)slab * SLAB + chunk * 16, p.k_bytes, end);
            }
        }
    };
    auto commit = [&](int stage) {
#pragma unroll
        for (int i = 0; i < COPIES; i++)
            *reinterpret_cast<v4i *>(ring + stage * STAGE_BYTES + (wave + NW * i) * 1024 + lane * 16) = staged[i];
    };

    Acc acc[FO][FR];
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++)
#pragma unroll
            for (int v = 0; v < 4; v++) acc[i][j][v] = 0;

    const int n_slabs = (int)((p.k_bytes + SLAB - 1) / SLAB);
#pragma unroll
    for (int s = 0; s < STAGES - 1; s++)
        if (s < n_slabs) issue(s, s);
    vec.park(tid);
    if constexpr (!ALIGNED) commit(0);

    int stage = 0;
    for (int it = 0; it < n_slabs; it++) {
        constexpr int KEEP = (STAGES - 2) * COPIES;  // younger slabs that may stay in flight
        if constexpr (!ALIGNED) {
            __syncthreads();
        } else {
            if (it + STAGES - 2 < n_slabs)
                wait_vmcnt_at_most<KEEP>();
            else
                wait_vmcnt_at_most<0>();
            if (it == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the scale vectors are in LDS
            __builtin_amdgcn_s_barrier();  // everyone's copies of slab `it` are visible; slab it-1 is fully consumed
        }
        int refill = stage + STAGES - 1;
        if (refill >= STAGES) refill -= STAGES;
        if (it + STAGES - 1 < n_slabs) issue(it + STAGES - 1, refill);
        const char *sx = ring + stage * STAGE_BYTES + wave_r * SLAB, *sw = ring + stage * STAGE_BYTES + (BR + wave_o) * SLAB;
#pragma unroll
        for (int ks = 0; ks < SLAB / 64; ks++) {
            if (ks > 0 && (int64_t)it * SLAB + ks * 64 >= p.k_bytes) break;
            v4i fw[FO], fx[FR];
#pragma unroll
            for (int i = 0; i < FO; i++) {
                const int row = i * 16 + l16;
                fw[i] = *reinterpret_cast<const v4i *>(sw + row * SLAB + (chunk_of(row, 4 * ks + lq) << 4));
            }
#pragma unroll
            for (int j = 0; j < FR; j++) {
                const int row = j * 16 + l16;
                fx[j] = *reinterpret_cast<const v4i *>(sx + row * SLAB + (chunk_of(row, 4 * ks + lq) << 4));
            }
            mfma_step<Path, FO, FR>(acc, fw, fx);
        }
        if constexpr (!ALIGNED) {
            if (it + 1 < n_slabs) commit(refill);
        }
        if (++stage == STAGES) stage = 0;
    }
    __syncthreads();  // the ring becomes the wavefronts' transposition patches

    store_tile<Path, BR, BO, WR, WO, STAGES * STAGE_BYTES>(acc, p, ring, vec, r0, o0, rows_valid, cols_valid);
}

// The partial sums of a workgroup's SK wavefronts meet in LDS (SK FR FO KiB) and wavefront b finishes block b.
template <class Path, int FR, int FO, int SK>
__device__ __forceinline__ void finish_split(const typename Path::Acc16 (&acc)[FO][FR], const LinearArgs &p, char *partial, int64_t r0, int64_t o0) {
    constexpr bool kInt8 = Path::kElemBytes == 1;
    constexpr int NB = FR * FO;
    using Acc = typename Path::Acc16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    // Partial sums: [wavefront][block][lane] 16-byte pieces.
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++)
            *reinterpret_cast<Acc *>(partial + ((wave * NB + i * FR + j) * 64 + lane) * 16) = acc[i][j];
    __syncthreads();
    for (int b = wave; b < NB; b += SK) {
        Acc sum = *reinterpret_cast<const Acc *>(partial + (b * 64 + lane) * 16);
#pragma unroll
        for (int w = 1; w < SK; w++) {
            const Acc part = *reinterpret_cast<const Acc *>(partial + ((w * NB + b) * 64 + lane) * 16);
#pragma unroll
            for (int v = 0; v < 4; v++) sum[v] += part[v];
        }
        const int i = b / FR, j = b - i * FR;
        const int64_t r = r0 + j * 16 + l16, o = o0 + i * 16 + lq * 4;
        if (r >= p.M || o >= p.N) continue;
        float rs = 1.0f;
        int rz = 0;
        v4f cs = {1.0f, 1.0f, 1.0f, 1.0f};
        v4i cz = {0, 0, 0, 0};
        uint32_t bias_word[2] = {0, 0};
        if constexpr (kInt8) {
            const uint32_t t = token_of(p, r);
            rs = p.s_tok[t];
            if constexpr (Path::kOffset) rz = p.z_tok[t];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int64_t oc = min(o + c, p.N - 1);
            if constexpr (kInt8) cs[c] = p.s_w[oc];
            if constexpr (Path::kOffset) cz[c] = p.rowsum[oc];
            if (p.bias) bias_word[c >> 1] |= (uint32_t) reinterpret_cast<const uint16_t *>(p.bias)[oc] << (16 * (c & 1));
            if constexpr (kInt8) {
                if (p.acc_out && o + c < p.N) p.acc_out[r * p.N + o + c] = Path::kPacked4 ? (int)sum[c] >> 8 : (int)sum[c];
            }
        }
        const v2f out = finish_four<Path>(sum, rs, rz, cs, cz, v2f{__builtin_bit_cast(float, bias_word[0]), __builtin_bit_cast(float, bias_word[1])});
        __half *dst = p.y + r * p.ldy + o;
        if (o + 4 <= p.N) {
            *reinterpret_cast<v2f_unaligned *>(dst) = out;
        } else {
            const float w[2] = {out.x, out.y};
#pragma unroll
            for (int c = 0; c < 4; c++)
                if (o + c < p.N)
                    reinterpret_cast<uint16_t *>(dst)[c] = (uint16_t)(__builtin_bit_cast(uint32_t, w[c >> 1]) >> (16 * (c & 1)));
        }
    }
}

// ------------------------------------------------------------------------------------------
// Split reduction, for problems of so few tiles that one wavefront's chain of loads is the whole run time.  A workgroup
// of SK wavefronts owns one tile of 16 FR rows x 16 FO channels; wavefront w takes
// the MFMA steps w, w + SK, ... (64 bytes of K each, so that neighbouring wavefronts read neighbouring bytes),
// with U steps of operands in flight in registers, then the partial sums meet in LDS and wavefront b finishes
// block b.  ALIGNED: 16-byte aligned bases and pitches and k_bytes a multiple of 64; otherwise any pitch,
// alignment and K: loads of 16 bytes wherever they fall, bytes beyond K zeroed.
// ------------------------------------------------------------------------------------------
template <class Path, int FR, int FO, int SK, int U, bool ALIGNED>
__global__ __launch_bounds__(64 * SK) void linear_mfma_splitk(const LinearArgs p) {
    constexpr int BR = 16 * FR, BO = 16 * FO;
    using Acc = typename Path::Acc16;
    __shared__ __attribute__((aligned(16))) char partial[SK * FR * FO * 1024];

    int tile_r, tile_o;
    if (!tile_of_block(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const char *xrow[FR], *wrow[FO];
#pragma unroll
    for (int j = 0; j < FR; j++) xrow[j] = p.x + min(r0 + j * 16 + l16, p.M - 1) * p.ldx_bytes + lq * 16;
#pragma unroll
    for (int i = 0; i < FO; i++) wrow[i] = p.w + min(o0 + i * 16 + l16, p.N - 1) * p.ldw_bytes + lq * 16;
    const char *const x_end = p.x + ((p.M - 1) * p.ldx_bytes + p.k_bytes), *const w_end = p.w + ((p.N - 1) * p.ldw_bytes + p.k_bytes);

    Acc acc[FO][FR];
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++)
#pragma unroll
            for (int v = 0; v < 4; v++) acc[i][j][v] = 0;

    const int n_steps = (int)((p.k_bytes + 63) / 64);
    for (int s0 = wave; s0 < n_steps; s0 += SK * U) {
        v4i fw[U][FO], fx[U][FR];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int s = s0 + u * SK;
            if (s < n_steps) {
#pragma unroll
                for (int i = 0; i < FO; i++)
                    fw[u][i] = ALIGNED ? *reinterpret_cast<const v4i *>(wrow[i] + (int64_t)s * 64)
                                       : load_any(wrow[i] - lq * 16, (int64_t)s * 64 + lq * 16, p.k_bytes, w_end);
#pragma unroll
                for (int j = 0; j < FR; j++)
                    fx[u][j] = ALIGNED ? *reinterpret_cast<const v4i *>(xrow[j] + (int64_t)s * 64)
                                       : load_any(xrow[j] - lq * 16, (int64_t)s * 64 + lq * 16, p.k_bytes, x_end);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (s0 + u * SK < n_steps) mfma_step<Path, FO, FR>(acc, fw[u], fx[u]);
    }

    finish_split<Path, FR, FO, SK>(acc, p, partial, r0, o0);
}

}  // namespace mfma
}  // namespace ptq4vm
