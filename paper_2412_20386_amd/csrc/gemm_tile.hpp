// Tile kernels of the MFMA linears for problems that fill the chip with 256 x 256 tiles once or not at all
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

// Operands of any pitch, alignment and K.  Only the last MFMA step (or slab) of a reduction reaches beyond K; every other one loads its 16-byte
// pieces without tests.  The last one's are requested by load_within and put right by place_within where they are used, so that
// nothing between a request and the next one depends on loaded data: with the correction behind each load (and its branches, whose joins wait
// for the load) the requests ran one after another (us, so / as now: 33 x 1648 -> 49 5.3 / 3.5, fp16 76 x 1818 -> 2020 13.9 / 9.7, fused
// 362 x 288 -> 893 6.9 / 6.1).
//
// A matrix of fewer than 16 bytes is loaded byte by byte (host-checked: the other forms never meet one): kTiny both, kTinyWeight the
// weight alone, whose activations may be many rows (50432 x 4 -> 3 5.2 us with both, 4.4 so, 4.8 before these forms came in).
enum class Rows { kAligned, kAny, kTiny, kTinyWeight };
inline bool is_tiny(int64_t rows, int64_t pitch_bytes, int64_t k_bytes) {
    return k_bytes < 16 && (rows == 1 || (rows < 16 && pitch_bytes < 16 && (rows - 1) * pitch_bytes + k_bytes < 16));
}

// The 16 bytes at `at`; where these would pass the end of the matrix, its last 16.
__device__ __forceinline__ v4i load_within(const char *at, const char *end) {
    const char *const last = end - 16;
    return *reinterpret_cast<const v4i_unaligned *>(at < last ? at : last);
}
// What load_within returned, moved to where it would lie in the 16 bytes at `at`; what enters from above lies beyond K.  (Where K is a multiple of
// 16 bytes, no piece of a row passes the end.)
__device__ __forceinline__ v4i place_within(v4i v, const char *at, const char *end) {
    const int over = (int)max((int64_t)0, min((int64_t)16, (int64_t)(at + 16 - end)));  // (the end may lie gigabytes away)
    if (over > 0) {
        if (over & 8) v = v4i{v[2], v[3], 0, 0};
        if (over & 4) v = v4i{v[1], v[2], v[3], 0};
        const int b = over & 3;
        v = v4i{(int)__builtin_amdgcn_alignbyte(v[1], v[0], b), (int)__builtin_amdgcn_alignbyte(v[2], v[1], b),
                (int)__builtin_amdgcn_alignbyte(v[3], v[2], b), (int)__builtin_amdgcn_alignbyte(0, v[3], b)};
    }
    return v;
}
// The 16 bytes at `at`, those from `end` on repeating the last one before it (no branches: all 16 in flight).
__device__ __forceinline__ v4i load_bytes(const char *at, const char *end) {
    v4i out;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const char *const byte = at + 4 * j + b;
            word |= (uint32_t) * reinterpret_cast<const uint8_t *>(byte < end ? byte : end - 1) << (8 * b);
        }
        out[j] = (int)word;
    }
    return out;
}
// The bytes of a row's 16 at byte kb that lie before k_bytes, as a mask.  Integer products need it on one operand only.
__device__ __forceinline__ v4i mask_within(int64_t kb, int64_t k_bytes) {
    const int valid = (int)max((int64_t)0, min((int64_t)16, k_bytes - kb));
    v4i m;
#pragma unroll
    for (int j = 0; j < 4; j++) m[j] = (int)keep_low_bytes(0xffffffffu, valid - 4 * j);
    return m;
}

// n / d for n < 2^31 and a divisor known on the host, 1 <= d < 2^31: with 2^(shift-1) < d <= 2^shift and mul = floor(2^32 (2^shift -
// d) / d) + 1, (mulhi(n, mul) + n) >> shift is the quotient (Granlund and Montgomery, division by invariant integers).
struct FastDiv {
    uint32_t mul, shift, d;
};
inline FastDiv fast_div(uint32_t d) {
    uint32_t shift = 0;
    while ((1ULL << shift) < d) shift++;
    return {(uint32_t)(((1ULL << 32) * ((1ULL << shift) - d)) / d + 1), shift, d};
}
__device__ __forceinline__ uint32_t quotient(const FastDiv &f, uint32_t n) { return (__umulhi(n, f.mul) + n) >> f.shift; }
__device__ __forceinline__ uint32_t remainder_of(const FastDiv &f, uint32_t n) { return n - quotient(f, n) * f.d; }

// What a tile kernel reads of LinearArgs, with the divisions of its set-up prepared on the host: a workgroup's set-up is a serial chain
// that nothing hides in small problems (64-bit remainders and divisions by tiles_o took 0.35 us of 1.4).
struct TileArgs {
    const char *x, *w;
    int64_t M, N, ldx_bytes, ldw_bytes, k_bytes;
    uint32_t per_xcd, xcd_extra;  // 8 per_xcd + xcd_extra tiles
    FastDiv inner, tok;           // tiles along the dimension walked first; L
    uint32_t rows_first;          // which dimension that is
    uint32_t stores;              // Stores
    const float *s_tok, *s_w;
    const __half *bias;
    __half *y;
    int64_t ldy, L;
    const int32_t *z_tok, *rowsum;
    int32_t *acc_out;
};
// How results leave: kAny any address and channel count; the others whole 16-byte pieces at 16-byte aligned addresses (y, its
// pitch and N multiples of 8 elements): kThrough at device scope, kPast non-temporal, kCached ordinary ones.
enum Stores : uint32_t { kAny = 0, kThrough = 1, kPast = 2, kCached = 3 };
// Device-scope stores leave no dirty lines in the L2 for the end of the launch to write back, but push the operands of this and the
// next launches out of the memory-side cache (us, kThrough / kPast / ordinary stores: 12608 x 384 -> 384 6.1 / 6.8 / 7.8, 6304 x 384 -> 1536
// 9.4 / 10.1 / 11.0, 25216 x 768 -> 384 13.4 / 13.7 / 14.5, 50240 x 768 -> 384 30.0 / 24.7 / 32.4; whole Vim-S blocks over 128 x 197 rows, results of
// 9.7 M elements, 88.2 / 86.9, and over 64 x 785 rows 155.5 / 152.3).  Rows that are no whole 128-byte lines share lines between tiles; in large
// results these have to meet in the L2 (12608 x 384 -> 1000 16.7 / 18.5 / 14.2, 24104 x 830 -> 760 43 kPast, 38 ordinary; small ones gain all
// the same: 12608 x 384 -> 328 6.5 / 7.0 / 7.2).
constexpr int64_t kThroughElements = 6LL << 20;  // results up to this many are stored kThrough

// Tiles of BR x BO for `a`; false if there are too many.  Neighbouring workgroups of an XCD walk the dimension with the
// smaller operand behind it first, so that an XCD reads its share of the larger operand once (197 x 768 -> 3072: 4.3 us with the
// rows first, 4.8 with the channels first; 197 x 1536 -> 768 5.0 / 5.4).
template <int BR, int BO>
inline bool tile_args(const LinearArgs &a, TileArgs &t, dim3 &grid) {
    const int64_t tiles_r = ptq4vm::ceil_div(a.M, BR), tiles_o = ptq4vm::ceil_div(a.N, BO);
    if (tiles_r * tiles_o > 0x3fffffffLL) return false;
    t.x = a.x, t.w = a.w, t.s_tok = a.s_tok, t.s_w = a.s_w, t.bias = a.bias, t.y = a.y, t.z_tok = a.z_tok, t.rowsum = a.rowsum, t.acc_out = a.acc_out;
    t.M = a.M, t.N = a.N, t.ldx_bytes = a.ldx_bytes, t.ldw_bytes = a.ldw_bytes, t.k_bytes = a.k_bytes, t.ldy = a.ldy, t.L = a.L;
    t.per_xcd = (uint32_t)(tiles_r * tiles_o / kXcds);
    t.xcd_extra = (uint32_t)(tiles_r * tiles_o % kXcds);
    t.rows_first = a.M < a.N;
    t.inner = fast_div((uint32_t)(t.rows_first ? tiles_r : tiles_o));
    t.tok = fast_div((uint32_t)a.L);
    const bool wide = a.N % 8 == 0 && a.ldy % 8 == 0 && ptq4vm::aligned_to(a.y, 16) && a.ldy * 2 * BR < (1LL << 31);
    const bool whole_lines = a.ldy % 64 == 0 && ptq4vm::aligned_to(a.y, 128);
    t.stores = !wide ? kAny : a.M * a.N <= kThroughElements ? kThrough : whole_lines ? kPast : kCached;
    grid = grid_of_tiles(tiles_r * tiles_o);
    return true;
}

// The workgroup's tile: workgroup ids go round-robin over the 8 XCDs, each XCD gets a contiguous range of tiles.
__device__ __forceinline__ bool locate_tile(const TileArgs &p, uint32_t &tile_r, uint32_t &tile_o) {
    // What the set-up needs is wanted here, so that it is loaded with one wait instead of one behind every branch
    asm volatile("" ::"s"(p.x), "s"(p.w), "s"(p.M), "s"(p.N), "s"(p.ldx_bytes), "s"(p.ldw_bytes), "s"(p.k_bytes), "s"(p.tok.mul), "s"(p.tok.shift),
                 "s"(p.tok.d), "s"(p.s_tok), "s"(p.s_w), "s"(p.bias));
    const uint32_t block = blockIdx.x + (blockIdx.y << kGridRowLog2), xcd = block % kXcds;  // (grid_of_tiles)
    const uint32_t i = block / kXcds;
    if (i >= p.per_xcd + (xcd < p.xcd_extra)) return false;
    const uint32_t tile = xcd * p.per_xcd + min(xcd, p.xcd_extra) + i;
    const uint32_t outer = quotient(p.inner, tile), first = tile - outer * p.inner.d;
    tile_r = p.rows_first ? first : outer;
    tile_o = p.rows_first ? outer : first;
    return true;
}

// The channel of a 32-channel group that LDS row `row` of the weight (0 .. 31) holds: MFMA block h = row / 16, operand row a = row mod
// 16 carries channel 8 (a / 4) + 4 h + a mod 4, so that a lane's results of two blocks are eight neighbouring channels.
__device__ __forceinline__ int channel_of_row(int row) { return (row & ~31) + 8 * ((row >> 2) & 3) + 4 * ((row >> 4) & 1) + (row & 3); }

// The step, bias and offset vectors of a BR x BO tile, in LDS behind the ring.  fetch() loads one element per thread into
// registers (behind the first operand copies), park() writes them to LDS after the reduction, before a barrier.  Channels and
// rows beyond the matrix are clamped; they are never stored.  Every thread loads, without a branch: a load that only some
// paths have issued makes the compiler wait for everything in flight at the next use of a register.
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
    __device__ __forceinline__ void fetch(const TileArgs &p, int tid, int64_t r0, int64_t o0, int rows_valid, int cols_valid) {
        const int64_t o = o0 + min(tid, cols_valid - 1);
        if constexpr (kInt8) {
            const bool small = p.M <= 0x7fffffffLL;
            const uint32_t t0 = small ? remainder_of(p.tok, (uint32_t)r0) : (uint32_t)(r0 % p.L);
            const uint32_t n = t0 + (uint32_t)min(tid, rows_valid - 1);
            const uint32_t t = small ? remainder_of(p.tok, n) : n % (uint32_t)p.L;
            row_s = p.s_tok[t];
            if constexpr (Path::kOffset) row_z = p.z_tok[t];
            col_s = p.s_w[o];
            if constexpr (Path::kOffset) col_z = p.rowsum[o];
        }
        // without a bias any readable address of N elements stands in
        const uint16_t *bias = reinterpret_cast<const uint16_t *>(p.bias ? static_cast<const void *>(p.bias) : kInt8 ? static_cast<const void *>(p.s_w) : p.w);
        col_b = bias[o];
    }
    __device__ __forceinline__ void park(const TileArgs &p, int tid) {
        if (tid < BO) {
            cs[tid] = col_s;
            cb[tid] = p.bias ? col_b : (uint16_t)0;
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
// its own patch of the ring (RING_BYTES, free by now) and stores whole row segments.  The weight rows lie in LDS in the order
// of channel_of_row, so a lane's results are 16-byte pieces of its row.  Whole pieces leave as buffer stores, whose range
// check drops the rows beyond the matrix.
template <class Path, int BR, int BO, int WR, int WO, int RING_BYTES, bool DUMP, int FO, int FR, class Vectors>
__device__ __forceinline__ void store_tile(const typename Path::Acc16 (&acc)[FO][FR], const TileArgs &p, char *ring, const Vectors &vec,
                                           int64_t r0, int64_t o0, int rows_valid, int cols_valid) {
    constexpr int NW = WR * WO, WAVE_R = BR / WR, WAVE_O = BO / WO;
    static_assert(FO % 2 == 0, "pairs of MFMA blocks");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;

    // Accumulator register v of block (i, j): token row 16 j + l16, channel 32 (i / 2) + 8 lq + 4 (i mod 2) + v.
    if constexpr (DUMP) {
#pragma unroll
        for (int i = 0; i < FO; i++)
#pragma unroll
            for (int j = 0; j < FR; j++)
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    const int r = wave_r + j * 16 + l16, o = wave_o + (i >> 1) * 32 + 8 * lq + 4 * (i & 1) + c;
                    if (r < rows_valid && o < cols_valid)
                        p.acc_out[(r0 + r) * p.N + o0 + o] = Path::kPacked4 ? (int)acc[i][j][c] >> 8 : (int)acc[i][j][c];
                }
    }

    // Patch rows of 16 (CPR + 2) bytes: measured in a read loop, 16-byte accesses of 16 rows run at 241 bytes per clock and CU
    // when the pitch is 2 mod 4 pieces and at 128 when it is odd.
    constexpr int CPR = WAVE_O / 8, RPS = 64 / CPR, PITCH = CPR * 16 + 32;  // 16-byte chunks per patch row, rows per store instruction
    constexpr int FIT = RING_BYTES / NW / (16 * PITCH);
    constexpr int JB = FIT >= FR ? FR : (FIT >= 2 && FR % 2 == 0 ? 2 : 1);  // 16-row blocks per round
    static_assert(FIT >= 1 && RPS <= 16 * JB && 64 % CPR == 0, "patches fit the ring");
    char *const patch = ring + wave * (JB * 16 * PITCH);

    v4f cs[FO / 2][2], cb[FO / 2];
    v4i cz[FO / 2][2];
#pragma unroll
    for (int g = 0; g < FO / 2; g++) {
        const int col = wave_o + 32 * g + 8 * lq;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            cs[g][h] = *reinterpret_cast<const v4f *>(vec.cs + col + 4 * h);
            cz[g][h] = Path::kOffset ? *reinterpret_cast<const v4i *>(vec.cz + col + 4 * h) : v4i{0, 0, 0, 0};
        }
        cb[g] = *reinterpret_cast<const v4f *>(vec.cb + col);
    }
    const int srow = lane / CPR, schunk = lane % CPR;
    const int first_row = wave_r + srow, col = wave_o + schunk * 8;
    char *const y_tile = reinterpret_cast<char *>(p.y + r0 * p.ldy + o0);
    // (the span of a tile; with kAny stores, whose pitch may be anything, the descriptor is not used)
    const __amdgpu_buffer_rsrc_t y_rows = __builtin_amdgcn_make_buffer_rsrc(y_tile, 0, (int)(((int64_t)(rows_valid - 1) * p.ldy + cols_valid) * 2), 0x00020000);
    const uint32_t ldy_bytes = (uint32_t)p.ldy * 2, y_off = (uint32_t)first_row * ldy_bytes + (uint32_t)col * 2;
#pragma unroll
    for (int jb = 0; jb < FR; jb += JB) {
#pragma unroll
        for (int jj = 0; jj < JB; jj++) {
            const int j = jb + jj;
            const float rs = vec.rs[wave_r + j * 16 + l16];
            const int rz = Path::kOffset ? vec.rz[wave_r + j * 16 + l16] : 0;
#pragma unroll
            for (int g = 0; g < FO / 2; g++) {
                const v2f lo = finish_four<Path>(acc[2 * g][j], rs, rz, cs[g][0], cz[g][0], v2f{cb[g].x, cb[g].y});
                const v2f hi = finish_four<Path>(acc[2 * g + 1][j], rs, rz, cs[g][1], cz[g][1], v2f{cb[g].z, cb[g].w});
                *reinterpret_cast<v4f *>(patch + (jj * 16 + l16) * PITCH + (4 * g + lq) * 16) = v4f{lo.x, lo.y, hi.x, hi.y};
            }
        }
        asm volatile("" ::: "memory");  // wavefront-private patch: LDS runs a wavefront's accesses in order
        constexpr int S = JB * 16 / RPS;
        v4f data[S];
#pragma unroll
        for (int s = 0; s < S; s++) data[s] = *reinterpret_cast<const v4f *>(patch + (s * RPS + srow) * PITCH + schunk * 16);
        if (p.stores == kAny) {
#pragma unroll
            for (int s = 0; s < S; s++) {
                const int r = first_row + jb * 16 + s * RPS;
                if (r < rows_valid && col < cols_valid) store_eight(y_tile + (int64_t)r * p.ldy * 2 + col * 2, data[s], cols_valid - col);
            }
        } else if (col < cols_valid) {
            typedef unsigned int v4u __attribute__((ext_vector_type(4)));
            auto store = [&](auto policy) {
#pragma unroll
                for (int s = 0; s < S; s++)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, data[s]), y_rows, (int)(y_off + (uint32_t)(jb * 16 + s * RPS) * ldy_bytes), 0,
                                                           decltype(policy)::value);
            };
            // cache policy of the store: 16 is sc1 (device scope), 2 is nt
            if (p.stores == kThrough)
                store(std::integral_constant<int, 16>{});
            else if (p.stores == kPast)
                store(std::integral_constant<int, 2>{});
            else
                store(std::integral_constant<int, 0>{});
        }
        asm volatile("" ::: "memory");
    }
}

// How a direct tile holds its fragments: those of the next step too (kDoubled), the weight's only (kTight), one step's (kSingle).
enum class Fragments { kDoubled, kTight, kSingle };
// How linear_mfma_tile gets its operands: copied to LDS directly, to LDS through registers, or (reductions of one slab) as fragments or, VIA_LDS,
// through registers too.
enum class Copy { kDirect, kRegisters, kOneSlab };

template <int BR, int BO, int SLAB, int STAGES>
constexpr int tile_lds_bytes() {
    return STAGES * (BR + BO) * SLAB + tile_vector_bytes<BR, BO>();
}

// ------------------------------------------------------------------------------------------
// One BR x BO tile per workgroup, operands copied global -> LDS directly, K walked in slabs of SLAB bytes per row (SLAB 96: one
// 128-code block of the E2M3 container) through a ring of STAGES stages.  The fragments of the next MFMA step are fetched from LDS
// while the present step's MFMAs run, each into the registers that its predecessor has just left (the weight's are doubled).
// A slab's end - its last fragments in registers, the next slab landed, one barrier, the refill of its stage - stands between the
// MFMAs of its last step.  What bounds it now (12608 x 1536 -> 768 in 256 x 192 tiles, 18.8 us of which 2 are the launch): MFMAs 8.8 us
// at the 2.0 GHz that the chip holds, operand reads and copies that do not hide 5, set-up and epilogue 3.  Before, with fragments
// fetched and used step by step and a set-up that waited for the scale vectors: 23.7 us; 197 x 768 -> 3072 5.8 -> 4.3,
// 3152 x 384 -> 1536 8.0 -> 5.9, 25216 x 768 -> 384 16.5 -> 12.6.
// Requirements (host-checked): 16-byte aligned bases and pitches, k_bytes a multiple of 64 (E2M3: of 96), L < 2^31, 256 pitches
// below 2^31.
// ------------------------------------------------------------------------------------------
template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES, bool DUMP, Fragments HELD>
__device__ __forceinline__ void direct_tile(const TileArgs &p) {
    constexpr int NW = WR * WO, THREADS = 64 * NW;
    constexpr int WAVE_R = BR / WR, WAVE_O = BO / WO, FR = WAVE_R / 16, FO = WAVE_O / 16;
    constexpr bool E2M3 = Path::kE2m3, TIGHT = HELD == Fragments::kTight;
    constexpr int KS = E2M3 ? 1 : SLAB / 64;  // MFMA steps per slab
    static_assert(HELD != Fragments::kSingle || KS == 1, "one step per slab");
    constexpr int CHUNKS = SLAB / 16;
    constexpr int STAGE_BYTES = (BR + BO) * SLAB, X_COPIES = BR * SLAB / 1024, ALL_COPIES = STAGE_BYTES / 1024;
    constexpr int COPIES = (ALL_COPIES + NW - 1) / NW;     // 1 KiB each; those beyond the last repeat it
    constexpr int KEEP = (STAGES - 2) * COPIES;            // copies of younger slabs that may stay in flight
    using Frag = typename Path::Frag;
    using Acc = typename Path::Acc16;
    static_assert(SLAB == (E2M3 ? 96 : SLAB >= 128 ? 128 : 64), "LDS rows hold 64 or 128 bytes of K or one E2M3 block");
    static_assert(WAVE_R % 16 == 0 && WAVE_O % 32 == 0 && BR * SLAB % 1024 == 0 && STAGE_BYTES % 1024 == 0, "whole MFMA blocks and copies");
    static_assert(STAGES >= 2 && KEEP <= 63, "vmcnt is a 6-bit counter");

    uint32_t tile_r, tile_o;
    if (!locate_tile(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;
    const int rows_valid = (int)min((int64_t)BR, p.M - r0), cols_valid = (int)min((int64_t)BO, p.N - o0);
    // Which 16-byte chunk of its row lies at position c of LDS row `row` (bank conflicts: 241 bytes per clock and CU in a read loop)
    auto chunk_at = [](int row, int c) {
        if constexpr (E2M3) return c < 4 ? c : 4 + ((c - 4) ^ ((row >> 3) & 1));
        return c ^ (SLAB == 64 ? swizzle(row) : (row & 7));
    };
    char *const ring = lds_dyn;

    // Copies: linear on the LDS side, so order of the rows and swizzle are applied by choosing which global chunk a lane fetches.
    // Rows beyond the matrix repeat its last one.
    uint32_t off[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; i++) {
        const int c = min(wave + NW * i, ALL_COPIES - 1);  // scalar
        const bool is_x = c < X_COPIES;
        const int piece = (is_x ? c : c - X_COPIES) * 64 + lane, row = piece / CHUNKS;
        const int src = min(is_x ? row : channel_of_row(row), (is_x ? rows_valid : cols_valid) - 1);
        off[i] = (uint32_t)src * (uint32_t)(E2M3 ? SLAB : is_x ? p.ldx_bytes : p.ldw_bytes) + chunk_at(row, piece - row * CHUNKS) * 16;
    }
    const char *const gx = p.x + r0 * (E2M3 ? SLAB : p.ldx_bytes), *const gw = p.w + o0 * (E2M3 ? SLAB : p.ldw_bytes);
    const uint32_t k_bytes = (uint32_t)p.k_bytes;
    auto issue = [&](int slab, int stage) {
#pragma unroll
        for (int i = 0; i < COPIES; i++) {
            const int c = min(wave + NW * i, ALL_COPIES - 1);
            const bool is_x = c < X_COPIES;
            const char *src = (is_x ? gx : gw) + (E2M3 ? slab * (is_x ? p.ldx_bytes : p.ldw_bytes) : (int64_t)(uint32_t)slab * SLAB);
            uint32_t o = off[i];
            // the last slab of a K that ends in half a slab: the far chunks re-read the near ones, nobody uses them
            if (SLAB == 128 && (uint32_t)(slab + 1) * SLAB > k_bytes) {
                const int piece = (is_x ? c : c - X_COPIES) * 64 + lane, row = piece / CHUNKS;
                o -= chunk_at(row, piece - row * CHUNKS) & 4 ? 64 : 0;
            }
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + o),
                                             (__attribute__((address_space(3))) void *)(ring + stage * STAGE_BYTES + c * 1024), 16, 0, 0);
        }
    };
    const int n_slabs = (int)((k_bytes + SLAB - 1) / SLAB);
    issue(0, 0);
    TileVectors<Path, BR, BO, THREADS> vec(lds_dyn + STAGES * STAGE_BYTES);
    vec.fetch(p, tid, r0, o0, rows_valid, cols_valid);  // under the first slab's latency
#pragma unroll
    for (int s = 1; s < STAGES - 1; s++)
        if (s < n_slabs) issue(s, s);

    Acc acc[FO][FR];
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++)
#pragma unroll
            for (int v = 0; v < 4; v++) acc[i][j][v] = 0;

    uint32_t frag[KS];  // where row l16 of a block has the lane's operand
#pragma unroll
    for (int ks = 0; ks < KS; ks++) frag[ks] = (uint32_t)l16 * SLAB + (E2M3 ? lq * 16 : chunk_at(l16, 4 * ks + lq) << 4);
    const uint32_t frag_high = (uint32_t)l16 * SLAB + 64 + ((lq * 8) ^ ((l16 & 8) << 1));  // E2M3: high parts, swapped as copied
    auto fragment = [&](const char *rows, int ks) {
        if constexpr (E2M3)
            return Path::make_fragment(*reinterpret_cast<const v4i *>(rows + frag[0]), *reinterpret_cast<const v2i *>(rows + frag_high));
        else
            return *reinterpret_cast<const v4i *>(rows + frag[ks]);
    };
    // Both operands' fragments are doubled; in a TIGHT kernel the activations' are not: each is fetched again as soon as its MFMAs
    // have been issued, and the other wavefronts of the SIMD hide what is left of that latency.
    constexpr int BUFFERS = HELD == Fragments::kSingle ? 1 : 2;
    Frag fw[BUFFERS][FO], fx[HELD == Fragments::kDoubled ? 2 : 1][FR];
    auto load_fw = [&](int buf, const char *st, int ks) {
#pragma unroll
        for (int i = 0; i < FO; i++) fw[buf][i] = fragment(st + (BR + wave_o + i * 16) * SLAB, ks);
    };
    auto load_fx = [&](int buf, int j, const char *st, int ks) { fx[HELD == Fragments::kDoubled ? buf : 0][j] = fragment(st + (wave_r + j * 16) * SLAB, ks); };
    // The products of buffer `buf`, `fetch(j)` behind those of row block j
    auto products = [&](int buf, auto fetch) {
        Frag we[FO], wo[FO];
#pragma unroll
        for (int i = 0; i < FO; i++) {
            if constexpr (Path::kPacked4)
                we[i] = Path::even_codes(fw[buf][i]), wo[i] = Path::odd_codes(fw[buf][i]);
            else
                we[i] = fw[buf][i];
        }
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const Frag x = fx[HELD == Fragments::kDoubled ? buf : 0][j];
            if constexpr (Path::kPacked4) {
                const v4i xe = Path::even_codes(x), xo = Path::odd_codes(x);
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(we[i], xe, acc[i][j]);
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(wo[i], xo, acc[i][j]);
            } else {
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(we[i], x, acc[i][j]);
            }
            fetch(j);
        }
    };
    auto wait_slab = [&](int slab) {  // this wavefront's copies of it have landed
        if (KEEP == 0 || slab + STAGES - 2 >= n_slabs)
            wait_vmcnt_at_most<0>();
        else
            wait_vmcnt_at_most<KEEP>();
    };
    int stage = 0;
    if constexpr (HELD == Fragments::kSingle) {  // the other workgroups of the CU hide the latency of the fragments
#pragma unroll 1
        for (int it = 0; it < n_slabs; it++) {
            wait_slab(it);
            wait_lgkmcnt_0();
            __builtin_amdgcn_s_barrier();  // everyone's copies of slab `it` are visible; slab it - 1 is in registers and used
            if (it + STAGES - 1 < n_slabs) issue(it + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
            const char *const now = ring + stage * STAGE_BYTES;
            load_fw(0, now, 0);
#pragma unroll
            for (int j = 0; j < FR; j++) load_fx(0, j, now, 0);
            products(0, [](int) {});
            if (++stage == STAGES) stage = 0;
        }
    } else {
        wait_slab(0);
        __builtin_amdgcn_s_barrier();
        if (STAGES - 1 < n_slabs) issue(STAGES - 1, STAGES - 1);
        load_fw(0, ring, 0);
#pragma unroll
        for (int j = 0; j < FR; j++) load_fx(0, j, ring, 0);

        // One MFMA step on the fragments of buffer `cur`; the next step's, step `nks` of its slab, are fetched meanwhile.  Where a slab
        // ends (over) every wavefront holds its last fragments, so one barrier makes the next slab visible and frees this one's stage.
        // What the very last step fetches nobody uses.
        auto step = [&](int cur, int nks, bool over, int slab) {
            wait_lgkmcnt_0();  // (known to the compiler, so that no MFMA waits for the fetches that follow)
            if (over) {
                if (slab + 1 < n_slabs) {
                    wait_slab(slab + 1);
                    __builtin_amdgcn_s_barrier();
                    if (slab + STAGES < n_slabs) issue(slab + STAGES, stage);
                }
                if (++stage == STAGES) stage = 0;
            }
            const char *const next = ring + stage * STAGE_BYTES;
            load_fw(cur ^ 1, next, nks);
            if constexpr (TIGHT) {
                products(cur, [&](int j) {
                    load_fx(0, j, next, nks);
                    __builtin_amdgcn_sched_barrier(0);  // keep a fetch behind the MFMAs that free its registers
                });
            } else {
#pragma unroll
                for (int j = 0; j < FR; j++) load_fx(cur ^ 1, j, next, nks);
                __builtin_amdgcn_sched_barrier(0);  // fetch first, then multiply
                products(cur, [](int) {});
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (KS == 2) {
            const int whole = (int)(k_bytes / SLAB);
#pragma unroll 1
            for (int it = 0; it < whole; it++) {
                step(0, 1, false, it);
                step(1, 0, true, it);
            }
            if (whole < n_slabs) step(0, 0, false, whole);
        } else {
#pragma unroll 1
            for (int it = 0; it + 2 <= n_slabs; it += 2) {
                step(0, 0, true, it);
                step(1, 0, true, it + 1);
            }
            if (n_slabs & 1) step(0, 0, true, n_slabs - 1);
        }
    }
    vec.park(p, tid);
    __syncthreads();  // the vectors are visible, the ring becomes the wavefronts' transposition patches
    store_tile<Path, BR, BO, WR, WO, STAGES * STAGE_BYTES, DUMP>(acc, p, ring, vec, r0, o0, rows_valid, cols_valid);
}

// The same tile for any pitch, alignment and K: slabs pass through registers, one in flight, bytes beyond K zeroed (two stages).  (Two in
// flight cost a quarter to a half more registers, which packed operands in 64 x 64 tiles spilled: 6854 x 704 -> 512 9.8 us with one,
// 11.7 with two; over 1500 shapes one is 1 % faster, 3 % with 128-byte slabs.)
// Only the last slab reaches beyond K; the loads of the others carry no tests (16236 x 1584 -> 760 fp16 106.7 -> 62.8 us, 24104 x 830 -> 760
// 45.7 -> 36.1).
// Requirements (host-checked): L < 2^31, BR * ldx_bytes and BO * ldw_bytes below 2^31.
template <class Path, int BR, int BO, int WR, int WO, int SLAB, bool DUMP>
__device__ __forceinline__ void staged_tile(const TileArgs &p) {
    constexpr int NW = WR * WO, THREADS = 64 * NW;
    constexpr int WAVE_R = BR / WR, WAVE_O = BO / WO, FR = WAVE_R / 16, FO = WAVE_O / 16;
    constexpr int CHUNKS = SLAB / 16, ROWS_PER_COPY = 64 / CHUNKS, COPIES = (BR + BO) / ROWS_PER_COPY / NW;
    constexpr int STAGE_BYTES = (BR + BO) * SLAB;
    static_assert(SLAB == 64 || SLAB == 128, "LDS rows hold 64 or 128 bytes of K");
    static_assert(WAVE_R % 16 == 0 && WAVE_O % 32 == 0, "wave tile must be whole MFMA blocks");
    static_assert((BR + BO) % (ROWS_PER_COPY * NW) == 0 && BR % ROWS_PER_COPY == 0, "every wavefront brings the same number of pieces");
    using Acc = typename Path::Acc16;

    uint32_t tile_r, tile_o;
    if (!locate_tile(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;
    const int rows_valid = (int)min((int64_t)BR, p.M - r0), cols_valid = (int)min((int64_t)BO, p.N - o0);
    auto chunk_of = [](int row, int chunk) { return chunk ^ (SLAB == 64 ? swizzle(row) : (row & 7)); };
    char *const ring = lds_dyn;

    uint32_t off[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; i++) {
        const int row = (wave + NW * i) * ROWS_PER_COPY + lane / CHUNKS;
        const bool is_x = (wave + NW * i) * ROWS_PER_COPY < BR;
        const int src_row = is_x ? min(row, rows_valid - 1) : min(channel_of_row(row - BR), cols_valid - 1);
        off[i] = (uint32_t)src_row * (uint32_t)(is_x ? p.ldx_bytes : p.ldw_bytes);
    }
    const char *gx = p.x + r0 * p.ldx_bytes, *gw = p.w + o0 * p.ldw_bytes;
    const int64_t k_bytes = p.k_bytes;
    const char *const x_end = p.x + ((p.M - 1) * p.ldx_bytes + k_bytes), *const w_end = p.w + ((p.N - 1) * p.ldw_bytes + k_bytes);
    v4i staged[COPIES];
    auto fetch = [&](int slab) {
        const bool inside = (int64_t)(slab + 1) * SLAB <= k_bytes;  // uniform
#pragma unroll
        for (int i = 0; i < COPIES; i++) {
            const int c = wave + NW * i;  // scalar
            const bool is_x = c * ROWS_PER_COPY < BR;
            const char *src = is_x ? gx : gw;
            const int chunk = chunk_of(c * ROWS_PER_COPY + lane / CHUNKS, lane % CHUNKS);  // (BR is a multiple of 16: a weight row swizzles like row - BR)
            if (inside) {
                staged[i] = *reinterpret_cast<const v4i_unaligned *>(src + (int64_t)slab * SLAB + (off[i] + chunk * 16));
            } else {
                staged[i] = load_within(src + (int64_t)slab * SLAB + (off[i] + chunk * 16), is_x ? x_end : w_end);
            }
        }
    };
    auto commit = [&](int slab, int stage) {
        if ((int64_t)(slab + 1) * SLAB > k_bytes) {  // uniform
#pragma unroll
            for (int i = 0; i < COPIES; i++) {
                const int c = wave + NW * i;
                const bool is_x = c * ROWS_PER_COPY < BR;
                const int64_t kb = (int64_t)slab * SLAB + chunk_of(c * ROWS_PER_COPY + lane / CHUNKS, lane % CHUNKS) * 16;
                if (k_bytes % 16 != 0) staged[i] = place_within(staged[i], (is_x ? gx : gw) + off[i] + kb, is_x ? x_end : w_end);
                staged[i] &= mask_within(kb, k_bytes);
            }
        }
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

    const int n_slabs = (int)((k_bytes + SLAB - 1) / SLAB);
    fetch(0);
    TileVectors<Path, BR, BO, THREADS> vec(lds_dyn + 2 * STAGE_BYTES);
    vec.fetch(p, tid, r0, o0, rows_valid, cols_valid);
    commit(0, 0);
#pragma unroll 1
    for (int it = 0; it < n_slabs; it++) {
        const int stage = it & 1;
        __syncthreads();
        if (it + 1 < n_slabs) fetch(it + 1);
        const char *sx = ring + stage * STAGE_BYTES + wave_r * SLAB, *sw = ring + stage * STAGE_BYTES + (BR + wave_o) * SLAB;
#pragma unroll
        for (int ks = 0; ks < SLAB / 64; ks++) {
            if (ks > 0 && (int64_t)it * SLAB + ks * 64 >= k_bytes) break;
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
        if (it + 1 < n_slabs) commit(it + 1, stage ^ 1);
    }
    vec.park(p, tid);
    __syncthreads();  // the vectors are visible, the ring becomes the wavefronts' transposition patches
    store_tile<Path, BR, BO, WR, WO, 2 * STAGE_BYTES, DUMP>(acc, p, ring, vec, r0, o0, rows_valid, cols_valid);
}

// The same tile for a reduction of one slab at any pitch and alignment: every wavefront loads its operands as MFMA fragments, 16 rows x 64
// bytes at a time; nothing is shared but through the caches, and nothing waits for anybody before the epilogue.  What bounds it is
// that chain of latencies and the output stream (12608 x 12 -> 384 7.1 us through LDS, 5.6 now; 6304 x 24 -> 768 6.7 / 5.7).
template <class Path, int BR, int BO, int WR, int WO, int SLAB, bool DUMP>
__device__ __forceinline__ void one_slab_tile(const TileArgs &p) {
    constexpr int NW = WR * WO, THREADS = 64 * NW;
    constexpr int WAVE_R = BR / WR, WAVE_O = BO / WO, FR = WAVE_R / 16, FO = WAVE_O / 16, KS = SLAB / 64;
    using Acc = typename Path::Acc16;

    uint32_t tile_r, tile_o;
    if (!locate_tile(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;
    const int rows_valid = (int)min((int64_t)BR, p.M - r0), cols_valid = (int)min((int64_t)BO, p.N - o0);
    const char *const gx = p.x + r0 * p.ldx_bytes, *const gw = p.w + o0 * p.ldw_bytes;
    const char *const x_end = p.x + ((p.M - 1) * p.ldx_bytes + p.k_bytes), *const w_end = p.w + ((p.N - 1) * p.ldw_bytes + p.k_bytes);
    v4i fw[KS][FO], fx[KS][FR];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
        if (ks > 0 && ks * 64 >= p.k_bytes) break;  // (uniform)
#pragma unroll
        for (int i = 0; i < FO; i++) {
            const int row = min(wave_o + channel_of_row(i * 16 + l16), cols_valid - 1);
            fw[ks][i] = load_within(gw + ((uint32_t)row * (uint32_t)p.ldw_bytes + ks * 64 + lq * 16), w_end);
        }
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const int row = min(wave_r + j * 16 + l16, rows_valid - 1);
            fx[ks][j] = load_within(gx + ((uint32_t)row * (uint32_t)p.ldx_bytes + ks * 64 + lq * 16), x_end);
        }
    }
    TileVectors<Path, BR, BO, THREADS> vec(lds_dyn + 2 * (BR + BO) * SLAB);
    vec.fetch(p, tid, r0, o0, rows_valid, cols_valid);
    Acc acc[FO][FR];
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++)
#pragma unroll
            for (int v = 0; v < 4; v++) acc[i][j][v] = 0;
    // uniform: a row of the tile whose 16-byte pieces may pass the end of the matrix
    const bool pieces = p.k_bytes % 16 != 0;
    const bool w_edge = pieces && gw + ((int64_t)(cols_valid - 1) * p.ldw_bytes + KS * 64) > w_end, x_edge = pieces && gx + ((int64_t)(rows_valid - 1) * p.ldx_bytes + KS * 64) > x_end;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
        if (ks > 0 && ks * 64 >= p.k_bytes) break;
        if (w_edge) {
#pragma unroll
            for (int i = 0; i < FO; i++) {
                const int row = min(wave_o + channel_of_row(i * 16 + l16), cols_valid - 1);
                fw[ks][i] = place_within(fw[ks][i], gw + ((uint32_t)row * (uint32_t)p.ldw_bytes + ks * 64 + lq * 16), w_end);
            }
        }
        if (x_edge) {
#pragma unroll
            for (int j = 0; j < FR; j++) {
                const int row = min(wave_r + j * 16 + l16, rows_valid - 1);
                fx[ks][j] = place_within(fx[ks][j], gx + ((uint32_t)row * (uint32_t)p.ldx_bytes + ks * 64 + lq * 16), x_end);
            }
        }
        const v4i mask = mask_within(ks * 64 + lq * 16, p.k_bytes);
#pragma unroll
        for (int i = 0; i < FO; i++) fw[ks][i] &= mask;
        if constexpr (Path::kElemBytes == 2) {  // (infinities and NaN beyond K)
#pragma unroll
            for (int j = 0; j < FR; j++) fx[ks][j] &= mask;
        }
        mfma_step<Path, FO, FR>(acc, fw[ks], fx[ks]);
    }
    vec.park(p, tid);
    __syncthreads();
    store_tile<Path, BR, BO, WR, WO, 2 * (BR + BO) * SLAB, DUMP>(acc, p, lds_dyn, vec, r0, o0, rows_valid, cols_valid);
}

// Registers of a direct tile: results, the fragments that it holds, some for everything else.
template <class Path, int FR, int FO>
constexpr int tile_registers(Fragments held) {
    constexpr int frag = sizeof(typename Path::Frag) / 4;
    const int frags = held == Fragments::kDoubled ? 2 * FO + 2 * FR : held == Fragments::kTight ? 2 * FO + FR : FO + 1;
    return FR * FO * 4 + frags * frag + (Path::kPacked4 ? (FO + 2) * frag : 0) + (Path::kE2m3 ? 24 : 16);
}
// Wavefronts per SIMD that a direct tile is compiled for: those of as many workgroups as the LDS of a CU holds, as far as the registers
// go round.  (A bound also keeps results in plain registers; moving them from accumulation registers costs an instruction each.)
template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES>
constexpr int tile_waves_by_lds() {
    constexpr int waves = 160 * 1024 / tile_lds_bytes<BR, BO, SLAB, STAGES>() * WR * WO / 4;
    return waves < 1 ? 1 : (waves > 8 ? 8 : waves);
}
// E2M3 fragments are twice as large: where holding those of two steps would cost a quarter of the CU's workgroups or more, whose epilogues
// run under the others' products, one step's do (us, kTight / kSingle: 22663 x 1024 -> 1972 in 128 x 256 tiles 81.5 / 53.5, 42321 x 128
// -> 861 29.7 / 23.6; over 500 shapes 128 x 256 0.86 of the time, 128 x 128 0.92, 64 x 128 0.96).  64 x 64 tiles, five workgroups for six,
// keep two steps (reductions from 640 codes on 0.96 of the time).
template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES>
constexpr Fragments tile_fragments() {
    constexpr int by_lds = tile_waves_by_lds<Path, BR, BO, WR, WO, SLAB, STAGES>(), FR = BR / WR / 16, FO = BO / WO / 16;
    constexpr int by_registers = 512 / tile_registers<Path, FR, FO>(Fragments::kTight), waves = by_lds < by_registers ? by_lds : by_registers;
    if (Path::kE2m3 && waves * 4 <= by_lds * 3) return Fragments::kSingle;
    return tile_registers<Path, FR, FO>(Fragments::kDoubled) > 512 / waves / 8 * 8 ? Fragments::kTight : Fragments::kDoubled;
}
template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES>
constexpr int tile_waves() {
    constexpr int by_lds = tile_waves_by_lds<Path, BR, BO, WR, WO, SLAB, STAGES>();
    constexpr Fragments held = tile_fragments<Path, BR, BO, WR, WO, SLAB, STAGES>();
    constexpr int by_registers = 512 / tile_registers<Path, BR / WR / 16, BO / WO / 16>(held == Fragments::kSingle ? held : Fragments::kTight);
    constexpr int waves = by_lds < by_registers ? by_lds : by_registers;
    return waves < 1 ? 1 : waves;
}

template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES, bool DUMP, bool VIA_LDS, Copy COPY>
__global__ __launch_bounds__(64 * WR * WO, (COPY == Copy::kDirect ? tile_waves<Path, BR, BO, WR, WO, SLAB, STAGES>() : WR * WO == 8 && SLAB == 64 && !Path::kPacked4 ? 6 : 4)) void linear_mfma_tile(const TileArgs p) {
    static_assert(COPY == Copy::kDirect || STAGES == 2, "the register-staged form is double buffered");
    if constexpr (COPY == Copy::kDirect)
        direct_tile<Path, BR, BO, WR, WO, SLAB, STAGES, DUMP, tile_fragments<Path, BR, BO, WR, WO, SLAB, STAGES>()>(p);
    else if constexpr (COPY == Copy::kRegisters || VIA_LDS)
        staged_tile<Path, BR, BO, WR, WO, SLAB, DUMP>(p);
    else
        one_slab_tile<Path, BR, BO, WR, WO, SLAB, DUMP>(p);
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
// block b.  kAligned: 16-byte aligned bases and pitches and k_bytes a multiple of 64; otherwise any pitch,
// alignment and K: loads of 16 bytes wherever they fall, bytes beyond K zeroed.  Four workgroups to a CU, or the up to 1000 tiles of
// 32 x 32 become two rounds (packed 826 x 650 -> 1068 11.5 us at three, 9.1 at four).
// ------------------------------------------------------------------------------------------
template <class Path, int FR, int FO, int SK, int U, Rows ROWS>
__global__ __launch_bounds__(64 * SK, 4) void linear_mfma_splitk(const LinearArgs p) {
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

    const int n_whole = (int)(p.k_bytes / 64);
    // The step that reaches beyond K, requested first and used last
    const bool last = ROWS != Rows::kAligned && p.k_bytes % 64 != 0 && wave == n_whole % SK;
    constexpr bool W_BYTES = ROWS == Rows::kTiny || ROWS == Rows::kTinyWeight, X_BYTES = ROWS == Rows::kTiny;
    v4i lw[FO], lx[FR];
    if (last) {
#pragma unroll
        for (int i = 0; i < FO; i++) {
            const char *const at = wrow[i] + (int64_t)n_whole * 64;
            lw[i] = W_BYTES ? load_bytes(at, w_end) : load_within(at, w_end);
        }
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const char *const at = xrow[j] + (int64_t)n_whole * 64;
            lx[j] = X_BYTES ? load_bytes(at, x_end) : load_within(at, x_end);
        }
    }
    using Load = std::conditional_t<ROWS == Rows::kAligned, v4i, v4i_unaligned>;
    for (int s0 = wave; s0 < n_whole; s0 += SK * U) {
        v4i fw[U][FO], fx[U][FR];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int s = s0 + u * SK;
            if (s < n_whole) {
#pragma unroll
                for (int i = 0; i < FO; i++) fw[u][i] = *reinterpret_cast<const Load *>(wrow[i] + (int64_t)s * 64);
#pragma unroll
                for (int j = 0; j < FR; j++) fx[u][j] = *reinterpret_cast<const Load *>(xrow[j] + (int64_t)s * 64);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (s0 + u * SK < n_whole) mfma_step<Path, FO, FR>(acc, fw[u], fx[u]);
    }
    if (last) {
        if (p.k_bytes % 16 != 0) {
#pragma unroll
            for (int i = 0; i < FO; i++)
                if (!W_BYTES) lw[i] = place_within(lw[i], wrow[i] + (int64_t)n_whole * 64, w_end);
#pragma unroll
            for (int j = 0; j < FR; j++)
                if (!X_BYTES) lx[j] = place_within(lx[j], xrow[j] + (int64_t)n_whole * 64, x_end);
        }
        const v4i mask = mask_within((int64_t)n_whole * 64 + lq * 16, p.k_bytes);
#pragma unroll
        for (int i = 0; i < FO; i++) lw[i] &= mask;
        if constexpr (Path::kElemBytes == 2) {  // (infinities and NaN beyond K)
#pragma unroll
            for (int j = 0; j < FR; j++) lx[j] &= mask;
        }
        mfma_step<Path, FO, FR>(acc, lw, lx);
    }

    finish_split<Path, FR, FO, SK>(acc, p, partial, r0, o0);
}

}  // namespace mfma
}  // namespace ptq4vm
