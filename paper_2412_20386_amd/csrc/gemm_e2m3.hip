// W4A4 linear for gfx950 on FP6 (E2M3) containers: the integer product of App. B.1 "INT GEMM" carried by
// v_mfma_f32_16x16x128_f8f6f4 (128 codes per instruction, twice the rate of the int8 MFMA), with the PTS
// dequantization fused behind it (PTS equation of Sec. 5.1; App. B.1 "Dequantization").  The 4-bit codes
// -7..7 (Sec. 2.3; the W4A4 setting of the latency table, Sec. 6.4) are exactly representable in E2M3, their
// products and partial sums are integers below 2^24, so the fp32 accumulators hold sum_k xq wq exactly.
//
// Operand layout of the instruction (checked against integer dot products on the device): lane l feeds row
// (l mod 16) of its matrix with the 32 codes of group (l / 16) of the current 128-code block, as 6 dwords;
// accumulator register v of lane l is (first-operand row 4 (l / 16) + v) x (second-operand row l mod 16).
// The weight is the first operand: a lane's four results are four consecutive channels of one token row.
//
// Kernels:
//   linear_e2m3_persistent  one workgroup of 8 wavefronts per CU walks 256 x 256 tiles (wave tile 128 token rows x
//                           64 channels); a ring of 3 stages, each one 128-code block of the tile's 256 + 256
//                           rows, is filled by direct global -> LDS copies that run two stages ahead.
//   linear_e2m3_tile        one tile of 32 x 64 .. 128 x 256 per workgroup, every other shape and any alignment of y
//   linear_e2m3_splitk      a few hundred blocks of 16 x 16 or fewer: the wavefronts of a workgroup split the reduction
#include "gemm_tile.hpp"

namespace ptq4vm {
namespace mfma {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));

constexpr int kBlockBytes = 96;  // one row's 128 codes: 4 x 16 bytes (groups' low parts), 4 x 8 bytes (high parts)

__device__ __forceinline__ v4f mfma_e2m3(const v8i &w, const v8i &x, const v4f &c) {
    // cbsz = blgp = 2: both operands are FP6 E2M3; no block scales
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w, x, c, 2, 2, 0, 0, 0, 0);
}
__device__ __forceinline__ v8i make_fragment(const v4i &lo, const v2i &hi) {
    return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
}

// What the shared pieces of gemm_tile.hpp need to know: 4-bit codes, sums carried exactly in fp32.
struct E2m3Path {
    static constexpr int kElemBytes = 1;
    static constexpr bool kOffset = false;
    static constexpr bool kPacked4 = false;
    static constexpr bool kE2m3 = true;
    using Acc16 = v4f;
    using Frag = v8i;
    static __device__ __forceinline__ Acc16 mfma16(const Frag &w, const Frag &x, const Acc16 &c) { return mfma_e2m3(w, x, c); }
    static __device__ __forceinline__ Frag make_fragment(const v4i &lo, const v2i &hi) { return mfma::make_fragment(lo, hi); }
};

// ------------------------------------------------------------------------------------------
// One BR x BO tile per workgroup: direct_tile of gemm_tile.hpp with ring stages of one 128-code block.  A block of the tile's rows is
// one contiguous span of the container; a stage row is the 96-byte block as in memory, except that rows whose bit 3 is set keep
// their two high-part chunks swapped (bank conflicts, see the persistent kernel).
// ------------------------------------------------------------------------------------------
template <int BR, int BO, int WR, int WO, int STAGES, bool DUMP>
__global__ __launch_bounds__(64 * WR * WO, (tile_waves<E2m3Path, BR, BO, WR, WO, kBlockBytes, STAGES>())) void linear_e2m3_tile(const TileArgs p) {
    direct_tile<E2m3Path, BR, BO, WR, WO, kBlockBytes, STAGES, DUMP, tile_fragments<E2m3Path, BR, BO, WR, WO, kBlockBytes, STAGES>()>(p);
}

// Split reduction (see linear_mfma_splitk): wavefront w takes the 128-code blocks w, w + SK, ... with U blocks of operands
// in flight in registers.
template <int FR, int FO, int SK, int U>
__global__ __launch_bounds__(64 * SK) void linear_e2m3_splitk(const LinearArgs p) {
    __shared__ __attribute__((aligned(16))) char partial[SK * FR * FO * 1024];
    int tile_r, tile_o;
    if (!tile_of_block(p, tile_r, tile_o)) return;
    const int64_t r0 = (int64_t)tile_r * 16 * FR, o0 = (int64_t)tile_o * 16 * FO;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const char *xrow[FR], *wrow[FO];
#pragma unroll
    for (int j = 0; j < FR; j++) xrow[j] = p.x + min(r0 + j * 16 + l16, p.M - 1) * kBlockBytes;
#pragma unroll
    for (int i = 0; i < FO; i++) wrow[i] = p.w + min(o0 + i * 16 + l16, p.N - 1) * kBlockBytes;
    auto fragment = [&](const char *row) {
        return make_fragment(*reinterpret_cast<const v4i *>(row + lq * 16), *reinterpret_cast<const v2i *>(row + 64 + lq * 8));
    };

    v4f acc[FO][FR];
#pragma unroll
    for (int i = 0; i < FO; i++)
#pragma unroll
        for (int j = 0; j < FR; j++) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const int n_blocks = (int)(p.k_bytes / kBlockBytes);
    for (int b0 = wave; b0 < n_blocks; b0 += SK * U) {
        v8i fw[U][FO], fx[U][FR];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t b = b0 + u * SK;
            if (b < n_blocks) {
#pragma unroll
                for (int i = 0; i < FO; i++) fw[u][i] = fragment(wrow[i] + b * p.ldw_bytes);
#pragma unroll
                for (int j = 0; j < FR; j++) fx[u][j] = fragment(xrow[j] + b * p.ldx_bytes);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (b0 + u * SK < n_blocks) {
#pragma unroll
                for (int i = 0; i < FO; i++)
#pragma unroll
                    for (int j = 0; j < FR; j++) acc[i][j] = mfma_e2m3(fw[u][i], fx[u][j], acc[i][j]);
            }
    }
    finish_split<E2m3Path, FR, FO, SK>(acc, p, partial, r0, o0);
}

// ------------------------------------------------------------------------------------------
// Persistent kernel.  LDS: ring of kStages stages, each (256 token rows + 256 channels) x 96 bytes, then two
// buffers of per-tile scale vectors and the wavefronts' patches.  The containers are block-major, so what a stage receives is two contiguous
// 24 KiB spans of memory.  A stage row is the 96-byte block as in memory, except that rows with bit 3 set keep
// their last two 16-byte chunks (the groups' 8-byte high parts) swapped.  Measured with a stand-alone read loop
// (bytes per clock and CU, 16-byte low-part reads / 8-byte high-part reads / both): rows as in memory 228 / 118 /
// 168, high chunks swapped by row bit 3: 245 / 174 / 203, all chunk pairs swapped by row bit 3: 127 / 170 / 141.
// Weight rows sit in the order of channel_of_row, so that a lane's results are 16-byte pieces of its row.
// Ring discipline: barrier B(g) sits before the MFMAs of block g - 1, after its fragments have arrived in
// registers.  Passing it means every wavefront's copies of block g have landed and nobody reads block g - 1's
// stage again, so that stage is refilled at once with block g + 2, after a tile's last block too: the results cross
// patches of their own, and the stores queue behind the copies of the next tile's first two blocks, so that only
// the third of them waits for the stores.  With the results crossing the ring, that refill came behind the stores and
// the next tile's first block waited for them all (us, before -> now: 50432 x 768 -> 3072 116.8 -> 108.4,
// 50432 x 1536 -> 768 54.0 -> 51.6, 25216 x 384 -> 1536 28.1 -> 26.0; rows that are not whole lines, stored past the L2
// before, 50240 x 384 -> 1000 44.9 -> 34.8).
// Requirements (host-checked): K a multiple of 128 and at least 256 codes, 16-byte aligned operand rows,
// N a multiple of 8, y rows 16-byte aligned, 4-byte aligned bias, 256 row pitches below 2^31, L < 2^31.
// ------------------------------------------------------------------------------------------
// Tile geometry: 256 token rows x 256 channels; 4 wavefronts side by side along the channels per 128 rows.
// Which 16-byte chunk of a row's block goes to chunk position c of its stage row.
__device__ __forceinline__ int stage_chunk_source(int row, int c) { return c < 4 ? c : 4 + ((c - 4) ^ ((row >> 3) & 1)); }

constexpr int kTile = 256;                 // channels per tile
constexpr int kTileRows = 256;             // token rows per tile
constexpr int kStages = 3;
constexpr int kWavesPerWg = 8;             // one workgroup per CU
constexpr int kStageBytes = (kTileRows + kTile) * kBlockBytes;
constexpr int kScaleBytes = kTile * 4 + kTileRows * 4 + kTile * 2;
constexpr int kPatchPitch = 160, kPatchBytes = 8 * kPatchPitch;  // a wavefront's patch: 8 rows of 64 fp16 (2 mod 4 pieces of 16 bytes: no bank conflicts)
constexpr int kPersistentLds = kStages * kStageBytes + 2 * kScaleBytes + kWavesPerWg * kPatchBytes;

template <bool HAS_BIAS, bool DUMP_ACC>
__global__ __launch_bounds__(kWavesPerWg * 64, 2) void linear_e2m3_persistent(const LinearArgs p) {
    constexpr int NW = kWavesPerWg, FR = 8, FO = 4, WAVE_R = 128, WAVE_O = 64;
    constexpr int X_COPIES = kTileRows * 6 / 64 / NW;  // 1 KiB copies per wavefront and stage: 3 of token rows,
    constexpr int W_COPIES = kTile * 6 / 64 / NW;      // 3 of weight rows
    constexpr int LOADS_PER_BLOCK = X_COPIES + W_COPIES;
    constexpr int KEEP = (kStages - 2) * LOADS_PER_BLOCK;  // copies allowed in flight when a block is needed
    constexpr int TILE_STORES = 2 * FR;                    // a wavefront's store instructions per tile

    char *const ring = lds_dyn;
    char *const scales = lds_dyn + kStages * kStageBytes;
    char *const patch = scales + 2 * kScaleBytes + (threadIdx.x >> 6) * kPatchBytes;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_r = (wave >> 2) * WAVE_R, wave_o = (wave & 3) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;
    const int swap = (l16 >> 3) & 1;
    // byte offsets of this lane's fragment parts inside a stage row block of 16 rows
    const int frag_lo = l16 * kBlockBytes + (lq << 4);
    const int frag_hi = l16 * kBlockBytes + ((4 + ((lq >> 1) ^ swap)) << 4) + (lq & 1) * 8;

    // work split: XCD x owns a contiguous range of tiles (channel tiles fastest), its workgroups interleave in it
    const int total_tiles = p.tiles_o * p.tiles_r;
    const int per_xcd = (total_tiles + kXcds - 1) / kXcds;
    const int wpx = (int)gridDim.x / kXcds, xcd = (int)(blockIdx.x % kXcds), wj = (int)(blockIdx.x / kXcds);
    const int lo_tile = xcd * per_xcd, hi_tile = min(lo_tile + per_xcd, total_tiles);
    const int n_range = max(hi_tile - lo_tile, 0);
    const int n_my = n_range / wpx + (wj < n_range % wpx ? 1 : 0);
    const int first = lo_tile + wj, last = first + n_my * wpx;

    const int n_blocks = (int)(p.k_bytes / kBlockBytes);
    const int total_blocks = n_my * n_blocks;
    if (total_blocks == 0) return;  // the whole workgroup: no barrier has been executed yet

    // ---- producer: the next block to copy, possibly of a later tile than the one being computed
    int pf_tile = first, pf_block = 0, pf_stage = 0, issued = 0;
    const char *pf_x = nullptr, *pf_w = nullptr;
    uint32_t x_off[X_COPIES], w_off[W_COPIES];
    auto pf_setup = [&]() {
        const int to = pf_tile % p.tiles_o, tr = pf_tile / p.tiles_o;
        const int64_t r0 = (int64_t)tr * kTileRows, o0 = (int64_t)to * kTile;
        pf_x = p.x + r0 * kBlockBytes;  // in plane 0; block b is b plane pitches further
        pf_w = p.w + o0 * kBlockBytes;
        const int rows_x = (int)min((int64_t)kTileRows, p.M - r0), rows_w = (int)min((int64_t)kTile, p.N - o0);
        // 16-byte chunk q of a stage half: row q / 6, chunk q mod 6; rows with bit 3 set keep chunks 4 and 5 swapped.
        // Rows beyond the matrix are clamped: their results are never stored.
#pragma unroll
        for (int i = 0; i < X_COPIES; i++) {
            const int q = (wave + NW * i) * 64 + lane;
            const int row = q / 6, c = q - row * 6;
            x_off[i] = (uint32_t)min(row, rows_x - 1) * kBlockBytes + stage_chunk_source(row, c) * 16;
        }
#pragma unroll
        for (int i = 0; i < W_COPIES; i++) {
            const int q = (wave + NW * i) * 64 + lane;
            const int row = q / 6, c = q - row * 6;
            w_off[i] = (uint32_t)min(channel_of_row(row), rows_w - 1) * kBlockBytes + stage_chunk_source(row, c) * 16;
        }
    };
    auto issue = [&]() {  // copy the producer's block into ring stage pf_stage, then advance
        char *sx = ring + pf_stage * kStageBytes;
        char *sw = sx + kTileRows * kBlockBytes;
        const char *gx = pf_x + (int64_t)pf_block * p.ldx_bytes;
        const char *gw = pf_w + (int64_t)pf_block * p.ldw_bytes;
#pragma unroll
        for (int i = 0; i < X_COPIES; i++)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gx + x_off[i]),
                                             (__attribute__((address_space(3))) void *)(sx + (wave + NW * i) * 1024),
                                             16, 0, 0);
#pragma unroll
        for (int i = 0; i < W_COPIES; i++)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gw + w_off[i]),
                                             (__attribute__((address_space(3))) void *)(sw + (wave + NW * i) * 1024),
                                             16, 0, 0);
        issued++;
        if (++pf_stage == kStages) pf_stage = 0;
        if (++pf_block == n_blocks) {
            pf_block = 0;
            pf_tile += wpx;
            if (pf_tile < last) pf_setup();
        }
    };
    // Block g has landed for this wavefront.  after_tile: one of the two blocks that were copied ahead of the last tile's
    // stores, which may stay in flight (loads and stores retire in the order of their issue).
    auto wait_block = [&](int g, bool after_tile) {
        if (g + kStages - 2 >= total_blocks)
            wait_vmcnt_at_most<0>();
        else if (after_tile)
            wait_vmcnt_at_most<KEEP + TILE_STORES>();
        else
            wait_vmcnt_at_most<KEEP>();
    };

    pf_setup();
    while (issued < kStages - 1 && issued < total_blocks) issue();
    wait_block(0, false);
    __builtin_amdgcn_s_barrier();  // B(0)
    if (issued < total_blocks) issue();

    int stage = 0, g = 0, parity = 0;  // consumer: ring stage, running block number, scale buffer
    for (int tile = first; tile < last; tile += wpx, parity ^= 1) {
        const int tile_o = tile % p.tiles_o, tile_r = tile / p.tiles_o;
        const int64_t r0 = (int64_t)tile_r * kTileRows, o0 = (int64_t)tile_o * kTile;
        const int rows_valid = (int)min((int64_t)kTileRows, p.M - r0), cols_valid = (int)min((int64_t)kTile, p.N - o0);
        float *const cs_lds = reinterpret_cast<float *>(scales + parity * kScaleBytes);  // s_w of the tile's channels
        float *const rs_lds = cs_lds + kTile;                                           // s_tok of the tile's rows
        uint32_t *const cb_lds = reinterpret_cast<uint32_t *>(rs_lds + kTileRows);      // bias, two fp16 per word

        // Scale vectors of this tile, one 4-byte element per lane, straight into LDS (indices beyond the
        // matrix are clamped; those rows / channels are never stored).  Tasks 0-3: s_w, then s_tok (64 rows each), then 2 of bias.
        constexpr int kRowTasks = kTileRows / 64;
#pragma unroll
        for (int task = 0; task < 4 + kRowTasks + 2; task++) {
            if (task % NW != wave) continue;
            if (task < 4) {
                const int c = min(task * 64 + lane, cols_valid - 1);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p.s_w + o0 + c),
                                                 (__attribute__((address_space(3))) void *)(cs_lds + task * 64), 4, 0, 0);
            } else if (task < 4 + kRowTasks) {
                const int blk = task - 4;
                const int r = min(blk * 64 + lane, rows_valid - 1);
                const uint32_t t = ((uint32_t)(r0 % p.L) + (uint32_t)r) % (uint32_t)p.L;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p.s_tok + t),
                                                 (__attribute__((address_space(3))) void *)(rs_lds + blk * 64), 4, 0, 0);
            } else if constexpr (HAS_BIAS) {
                const int blk = task - 4 - kRowTasks;
                const int c2 = min(blk * 64 + lane, cols_valid / 2 - 1);
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(reinterpret_cast<const uint32_t *>(p.bias + o0) + c2),
                    (__attribute__((address_space(3))) void *)(cb_lds + blk * 64), 4, 0, 0);
            }
        }
        int loads_after_scales = 0;

        v4f acc[FO][FR];
#pragma unroll
        for (int i = 0; i < FO; i++)
#pragma unroll
            for (int j = 0; j < FR; j++) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

        // An operand is dead after its last MFMA of a block and is fetched again at once for the next block.
        v8i fw[FO], fx[FR];
        auto load_fw = [&](int i, int stg) {
            const char *sw = ring + stg * kStageBytes + (kTileRows + wave_o + i * 16) * kBlockBytes;
            fw[i] = make_fragment(*reinterpret_cast<const v4i *>(sw + frag_lo), *reinterpret_cast<const v2i *>(sw + frag_hi));
        };
        auto load_fx = [&](int j, int stg) {
            const char *sx = ring + stg * kStageBytes + (wave_r + j * 16) * kBlockBytes;
            fx[j] = make_fragment(*reinterpret_cast<const v4i *>(sx + frag_lo), *reinterpret_cast<const v2i *>(sx + frag_hi));
        };

        // B(g) for the tile's first block was passed during the previous tile (or before the loop)
#pragma unroll
        for (int i = 0; i < FO; i++) load_fw(i, stage);
#pragma unroll
        for (int j = 0; j < FR; j++) load_fx(j, stage);

        for (int s = 0; s < n_blocks; s++, g++) {
            int next_stage = stage + 1;
            if (next_stage == kStages) next_stage = 0;
            bool has_next = false;
            if (g + 1 < total_blocks) {
                // B(g+1): this wavefront holds the fragments of block g in registers and its copies of block g+1 have landed
                wait_lgkmcnt_0();
                wait_block(g + 1, s < kStages - 1 && tile != first);
                __builtin_amdgcn_s_barrier();
                if (issued < total_blocks) {
                    issue();  // refills the stage of block g
                    loads_after_scales += LOADS_PER_BLOCK;
                }
                has_next = s + 1 < n_blocks;
            }
#pragma unroll
            for (int j = 0; j < FR; j++) {
#pragma unroll
                for (int i = 0; i < FO; i++) {
                    acc[i][j] = mfma_e2m3(fw[i], fx[j], acc[i][j]);
                    if (j == FR - 1 && has_next) load_fw(i, next_stage);
                }
                if (has_next) load_fx(j, next_stage);
            }
            stage = next_stage;
        }

        // ---- epilogue, under the copies of the next tile's first two blocks.  The scale vectors were copied ahead of the
        // blocks counted in loads_after_scales.
        if (loads_after_scales >= 2 * KEEP)
            wait_vmcnt_at_most<2 * KEEP>();
        else
            wait_vmcnt_at_most<0>();
        __builtin_amdgcn_s_barrier();  // scale vectors are visible to every wavefront
        asm volatile("" ::: "memory");

        // Accumulator register v of block (i, j): token row 16 j + l16, channel 32 (i / 2) + 8 lq + 4 (i mod 2) + v: two pieces of 16
        // bytes per lane and 16-row block.  The lanes of rows 0..7 hand their second piece to those of rows 8..15 for their
        // first, so that each half of the block crosses the wavefront's patch by itself, into stores of eight whole 128-byte
        // row segments; a block's stores are issued behind the conversion of the next one.
        v4f cs[FO], cb[FO / 2];
#pragma unroll
        for (int h = 0; h < FO / 2; h++) {
            const int col = wave_o + 32 * h + 8 * lq;
            cs[2 * h] = *reinterpret_cast<const v4f *>(cs_lds + col), cs[2 * h + 1] = *reinterpret_cast<const v4f *>(cs_lds + col + 4);
            cb[h] = HAS_BIAS ? *reinterpret_cast<const v4f *>(cb_lds + col / 2) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
        const uint32_t ldy_bytes = (uint32_t)p.ldy * 2;
        const bool whole_lines = p.ldy % 64 == 0;
        const int srow = lane >> 3, scol = wave_o + (lane & 7) * 8;
        const uint32_t beyond = 0x80000000u;  // past every tile's span
        const uint32_t y_off = scol < cols_valid ? (uint32_t)(wave_r + srow) * ldy_bytes + (uint32_t)scol * 2 : beyond;
        const __amdgpu_buffer_rsrc_t y_rows =
            __builtin_amdgcn_make_buffer_rsrc(p.y + r0 * p.ldy + o0, 0, (int)(((int64_t)(rows_valid - 1) * p.ldy + cols_valid) * 2), 0x00020000);
        v4f data[2];
        auto store_block = [&](int j) {
            typedef unsigned int v4u __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int off = (int)(y_off + (uint32_t)(j * 16 + h * 8) * ldy_bytes);
                if (whole_lines)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, data[h]), y_rows, off, 0, 2);  // non-temporal
                else  // lines shared between tiles meet in the L2
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, data[h]), y_rows, off, 0, 0);
            }
        };
        constexpr int kRowRotate8 = 0x128;  // DPP: every 16 lanes rotated by 8; bank masks 0xc, 0x3: lanes 8..15, 0..7 are written
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const float rs = rs_lds[wave_r + j * 16 + l16];
            v4f piece[2];
#pragma unroll
            for (int i = 0; i < FO; i++) {
                if constexpr (DUMP_ACC) {
                    const int64_t r = r0 + wave_r + j * 16 + l16;
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        const int64_t o = o0 + wave_o + 32 * (i >> 1) + 8 * lq + 4 * (i & 1) + c;
                        if (r < p.M && o < p.N) p.acc_out[r * p.N + o] = (int)acc[i][j][c];
                    }
                }
                const int e = 2 * (i & 1);  // two fp16 biases a word
                piece[i >> 1][e] = dequantize_pair_f16(acc[i][j][0], rs * cs[i][0], acc[i][j][1], rs * cs[i][1], cb[i >> 1][e]);
                piece[i >> 1][e + 1] = dequantize_pair_f16(acc[i][j][2], rs * cs[i][2], acc[i][j][3], rs * cs[i][3], cb[i >> 1][e + 1]);
            }
            const v4i near = __builtin_bit_cast(v4i, piece[0]), far = __builtin_bit_cast(v4i, piece[1]);
            v4i half[2];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                half[0][c] = __builtin_amdgcn_update_dpp(near[c], far[c], kRowRotate8, 0xf, 0xc, false);
                half[1][c] = __builtin_amdgcn_update_dpp(far[c], near[c], kRowRotate8, 0xf, 0x3, false);
            }
            if (j > 0) store_block(j - 1);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                asm volatile("" ::: "memory");  // wavefront-private patch: LDS runs a wavefront's accesses in order
                *reinterpret_cast<v4i *>(patch + (l16 & 7) * kPatchPitch + ((l16 >> 3) * 4 + lq) * 16) = half[h];
                asm volatile("" ::: "memory");
                data[h] = *reinterpret_cast<const v4f *>(patch + srow * kPatchPitch + (lane & 7) * 16);
            }
        }
        store_block(FR - 1);
    }
}

int launch_persistent(LinearArgs a, hipStream_t stream) {
    int device = 0, cus = 0;
    hipError_t err = hipGetDevice(&device);
    if (err == hipSuccess) err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (err != hipSuccess) return ptq4vm::record_hip_error(err, "hipDeviceGetAttribute(multiprocessor count)");
    const int64_t tiles_r = ptq4vm::ceil_div(a.M, kTileRows), tiles_o = ptq4vm::ceil_div(a.N, kTile);
    a.tiles_r = (int)tiles_r;
    a.tiles_o = (int)tiles_o;
    const unsigned wgs = (unsigned)max(1, cus / kXcds) * kXcds;  // one workgroup per CU, a multiple of the XCD count
    using Kernel = void (*)(const LinearArgs);
    static const Kernel kernels[2][2] = {{linear_e2m3_persistent<false, false>, linear_e2m3_persistent<false, true>},
                                         {linear_e2m3_persistent<true, false>, linear_e2m3_persistent<true, true>}};
    const Kernel kernel = kernels[a.bias ? 1 : 0][a.acc_out ? 1 : 0];
    if (int rc = ptq4vm::set_lds_limit(reinterpret_cast<const void *>(kernel), kPersistentLds, "hipFuncSetAttribute(linear_e2m3_persistent)")) return rc;
    kernel<<<dim3(wgs), dim3(kWavesPerWg * 64), kPersistentLds, stream>>>(a);
    return ptq4vm::check_launch("linear_e2m3_persistent");
}

template <int BR, int BO, int WR, int WO, int STAGES>
int launch_tile(const LinearArgs &a, hipStream_t stream) {
    TileArgs t;
    dim3 grid;
    if (!tile_args<BR, BO>(a, t, grid)) return PTQ4VM_ERR_SHAPE;
    constexpr int lds_bytes = tile_lds_bytes<BR, BO, kBlockBytes, STAGES>();
    auto kernel = a.acc_out ? linear_e2m3_tile<BR, BO, WR, WO, STAGES, true> : linear_e2m3_tile<BR, BO, WR, WO, STAGES, false>;
    if constexpr (lds_bytes > 64 * 1024) {
        if (int rc = ptq4vm::set_lds_limit(reinterpret_cast<const void *>(kernel), lds_bytes, "hipFuncSetAttribute(linear_e2m3_tile)")) return rc;
    }
    kernel<<<grid, dim3(64 * WR * WO), lds_bytes, stream>>>(t);
    return ptq4vm::check_launch("linear_e2m3_tile");
}

template <int FR, int FO, int SK, int U>
int launch_splitk(LinearArgs a, hipStream_t stream) {
    dim3 grid;
    if (!set_grid<16 * FR, 16 * FO>(a, grid)) return PTQ4VM_ERR_SHAPE;
    linear_e2m3_splitk<FR, FO, SK, U><<<grid, dim3(64 * SK), 0, stream>>>(a);
    return ptq4vm::check_launch("linear_e2m3_splitk");
}
}  // namespace
}  // namespace mfma
}  // namespace ptq4vm

extern "C" int ptq4vm_w4a4_linear_e2m3(const uint8_t *xq6, const uint8_t *wq6, const float *s_tok, const float *s_w,
                                       const void *bias_f16, void *y_f16, int32_t *acc_out, int64_t B, int64_t L,
                                       int64_t K, int64_t N, int64_t ldxq, int64_t ldwq, int64_t ldy, void *stream_) {
    using namespace ptq4vm::mfma;
    if (!xq6 || !wq6 || !s_tok || !s_w || !y_f16) return PTQ4VM_ERR_NULL;
    if (B < 0 || N < 0 || L <= 0 || K <= 0 || K > PTQ4VM_MAX_K_E2M3) return PTQ4VM_ERR_SHAPE;
    if (B > 0 && L > INT64_MAX / B) return PTQ4VM_ERR_SHAPE;
    const int64_t row_bytes = PTQ4VM_E2M3_BLOCKS(K) * kBlockBytes;
    // ldxq / ldwq: plane pitches of the block-major containers
    if ((B > 0 && ldxq / kBlockBytes < B * L) || ldwq / kBlockBytes < N || ldxq % 16 != 0 || ldwq % 16 != 0 || ldy < N)
        return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(xq6, 16) || !ptq4vm::aligned_to(wq6, 16) || !ptq4vm::aligned_to(y_f16, 2) ||
        !ptq4vm::aligned_to(s_tok, 4) || !ptq4vm::aligned_to(s_w, 4) || !ptq4vm::aligned_to(bias_f16, 2) ||
        !ptq4vm::aligned_to(acc_out, 4))
        return PTQ4VM_ERR_ALIGN;
    const int64_t M = B * L;
    if (M == 0 || N == 0) return PTQ4VM_OK;
    LinearArgs a{};
    a.x = reinterpret_cast<const char *>(xq6);
    a.w = reinterpret_cast<const char *>(wq6);
    a.s_tok = s_tok;
    a.s_w = s_w;
    a.bias = static_cast<const __half *>(bias_f16);
    a.y = static_cast<__half *>(y_f16);
    a.acc_out = acc_out;
    a.M = M;
    a.N = N;
    a.k_bytes = row_bytes;
    a.ldx_bytes = ldxq;
    a.ldw_bytes = ldwq;
    a.ldy = ldy;
    a.L = L;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    auto tiles = [&](int br, int bo) { return ptq4vm::ceil_div(M, br) * ptq4vm::ceil_div(N, bo); };
    // 256 x 256 tiles from two rounds of them that are filled to 80 % (us, persistent / tiles: 50432 x 384 -> 1536 [1182 tiles] 43.9 / 46.6,
    // 36906 x 256 -> 1120 [725] 23.1 / 30.0, 21704 x 1280 -> 2072 [765] 50.4 / 62.3, but 50432 x 1536 -> 768 [591] 52.3 / 47.5, 12608 x 768 -> 3072 [600]
    // 33.9 / 29.1, 25216 x 1536 -> 768 [297] 34.7 / 27.1; over 600 shapes tiles take 0.90 .. 0.96 of the time below 80 %, 0.98 .. 1.01 to 90 % and
    // 1.04 .. 1.08 beyond), unless they pad the channels by more than a quarter.  Also within one round, where the
    // 128 x 128 tiles, three to a CU, would need a second one (14148 x 1152 -> 832 [224] 15.3 / 17.4, 9030 x 1280 -> 1344 [216]
    // 16.0 / 18.7, 20860 x 1920 -> 576 [246] 20.9 / 25.8), for shorter reductions just beyond that line only (K <= 1024 from 832 small tiles on).
    const int64_t big_tiles = tiles(256, kTile), small_tiles = tiles(128, 128);
    const bool one_round = big_tiles <= 256 && small_tiles > 768 && (K > 1024 || small_tiles < 832);
    const bool full_rounds = big_tiles >= 512 && big_tiles * 100 >= ptq4vm::ceil_div(big_tiles, 256) * 256 * 80;
    const bool little_padding = ptq4vm::ceil_div(N, kTile) * kTile * 4 <= N * 5;
    const bool persistent_ok = K % 128 == 0 && K >= 256 && N % 8 == 0 && ptq4vm::aligned_to(y_f16, 16) && ldy % 8 == 0 &&
                               ptq4vm::aligned_to(bias_f16, 4) &&
                               ldy * 2 * kTile < (1LL << 31) && L < (1LL << 31) && ((full_rounds && little_padding) || one_round) && big_tiles <= 0x3fffffffLL;
    if (persistent_ok) return launch_persistent(a, stream);
    // The largest tile that leaves the CUs a few workgroups each, as in gemm_tile.hip; measured (us, tiles in brackets):
    //   split reduction / 32 x 64:  197 x 1536 -> 80 [65 blocks] 3.3 / 4.6, 392 x 1152 -> 200 [325] 3.6 / 4.1, 60 x 384 -> 2281 [572] 3.6 / 3.0
    //   32 x 64 / 64 x 64:          788 x 1536 -> 768 [156] 5.4 / 5.8, 197 x 768 -> 3072 [192] 4.1 / 4.1
    //   64 x 64 / 64 x 128:         6304 x 768 -> 384 [297] 5.4 / 5.9, 3192 x 896 -> 1047 [450] 7.6 / 7.6
    //   64 x 128 / 128 x 128:       3152 x 384 -> 1536 [300] 5.7 / 6.5, 6304 x 384 -> 1536 [600] 8.5 / 8.1
    //   128 x 128 / 128 x 256:      25216 x 768 -> 384 [394] 11.5 / 12.8, 12608 x 768 -> 3072 [1188] 34.4 / 30.5
    // (over 500 shapes the best of these forms takes 0.99 of the time of the rule's)
    if (L >= (1LL << 31) || tiles(16, 16) <= (K >= 896 ? 600 : 256)) return launch_splitk<1, 1, 4, 3>(a, stream);
    const int64_t most = tiles(32, 64) * 32 * 64 * 4 / 3;  // padded size that a tile may have
    if (tiles(128, 256) >= 800 && tiles(128, 256) * 128 * 256 <= most) return launch_tile<128, 256, 2, 4, 2>(a, stream);
    if (tiles(128, 128) >= 500 && tiles(128, 128) * 128 * 128 <= most) return launch_tile<128, 128, 2, 4, 2>(a, stream);
    if (tiles(64, 128) >= 400 && tiles(64, 128) * 64 * 128 <= most) return launch_tile<64, 128, 2, 2, 2>(a, stream);
    if (tiles(64, 64) >= 190) return launch_tile<64, 64, 2, 2, 2>(a, stream);
    return launch_tile<32, 64, 2, 2, 3>(a, stream);
}
