// MFMA linear layers for gfx950.
//
//   ptq4vm_w8a8_linear  int8 x int8 -> int32 GEMM with the PTS dequantization fused into the
//                       epilogue (PTS equation of Sec. 5.1: diag(Delta_W)(W-bar X-bar)diag(Delta_X);
//                       App. B.1 "INT GEMM" + "Dequantization" without the materialised
//                       step-size outer product).
//   ptq4vm_f16_linear   the unquantized FP16 linear the paper's latency table compares with,
//                       on the same tiling skeleton.
//
// Both operands are K-contiguous (X[M,K], W[N,K]), which is exactly what the CDNA4 MFMA wants:
// a lane feeds 16 consecutive bytes of K per instruction (16 int8 for v_mfma_i32_32x32x32_i8,
// 8 fp16 for v_mfma_f32_32x32x16_f16), so one 128-bit load from either matrix is one operand.
// The weight is the MFMA "A" operand and the activation the "B" operand: the accumulator of a
// lane then holds one token row r and runs of four consecutive output channels, and the
// per-token step s_tok[r mod L] is one scalar per lane.
//
// Kernels: linear_mfma_persistent here (many 256 x 256 tiles), linear_mfma_smallk here (fp16, reductions of at most 128
// bytes), the row-streaming kernel of pts_linear_fused.hip (very short reductions over many rows), and the tile kernels of
// gemm_tile.hip for everything else.
#include "gemm_tile.hpp"

namespace {

using namespace ptq4vm::mfma;

// ------------------------------------------------------------------------------------------
// Large-problem path: persistent workgroups, one per CU, 8 wavefronts on a 256 x 256 tile
// (wave tile 128 token rows x 64 channels), LDS ring of two 128-byte slabs fed by direct global -> LDS copies.
// Compared with the one-tile-per-workgroup kernels of gemm_tile.hpp the stream of slabs never drains: the copies of the
// next tile's first two slabs are issued at the ends of this tile's last two and land under its epilogue, whose patches
// have LDS of their own.  As there
//   * the MFMA is v_mfma_i32_16x16x64_i8 (v_mfma_f32_16x16x32_f16 on the fp16 path): with random operand bytes it sustains ~18 % more
//     than the 32x32x32 form on this part (the matrix pipes are clock/power limited once operands toggle);
//   * both operands' fragments are double buffered in registers, fetched ahead of the MFMAs of the step before theirs, and the
//     waits for them are known to the compiler;
//   * a slab's end is one barrier: every wavefront holds its last fragments and its copies of the next slab have landed.
// Loads and stores of a wavefront retire in the order of their issue, so a wait that leaves the youngest operations in flight leaves the
// epilogue's stores alone: at the end of a tile's first slab, whose successor was requested before them, they may all still be on
// their way (kStores).  They are buffer stores whose range check drops rows and channels beyond the matrix, so that every wavefront
// issues the same number whatever its tile.
// The per-tile scale vectors (s_w, bias, s_tok[r mod L]) are copied into LDS at the start of a tile (double buffered).
// Requirements (host-checked): 16-byte aligned bases and pitches, 256 * pitch below 2^31, k_bytes % SLAB == 0,
// k_bytes >= 2 SLAB, N % 8 == 0, 16-byte aligned y pitch, 4-byte aligned bias, 256 * ldy * 2 < 2^31, L < 2^31.
// ------------------------------------------------------------------------------------------
constexpr int kTileCols = 256, kSlab = 128, kPatchPitch = 160;  // (16 rows of 64 fp16; 2 mod 4 pieces of 16 bytes: no bank conflicts)
template <class Path>
constexpr int persistent_scale_bytes() {
    return kTileCols * 4 + 256 * 4 + kTileCols * 2 + (Path::kOffset ? kTileCols * 4 + 256 * 4 : 0);
}
template <class Path>
constexpr int persistent_lds_bytes() {
    return 2 * (256 + kTileCols) * kSlab + 2 * persistent_scale_bytes<Path>() + 8 * 16 * kPatchPitch;
}

// The tiles `first`, `first + stride`, ... (n_my of them) of the grid of (32 FR)-row x 256-channel
// tiles, channel tiles fastest, processed by the whole workgroup.  FR = 8: 256-row tiles; FR = 4:
// 128-row half tiles (used to spread a last, partial round of tiles over idle workgroups).
template <class Path, bool HAS_BIAS, bool DUMP_ACC, int FR>
__device__ __forceinline__ void persistent_tiles(const LinearArgs &p, const int first, const int stride, const int n_my) {
    constexpr int BR = 32 * FR, BO = kTileCols, SLAB = kSlab, NW = 8, WO = 4, WAVE_R = 16 * FR, WAVE_O = 64, FO = WAVE_O / 16;
    constexpr int CHUNKS = SLAB / 16, ROWS_PER_COPY = 64 / CHUNKS;  // rows in one wavefront-wide 1 KiB copy
    constexpr int X_COPIES = BR / ROWS_PER_COPY / NW, W_COPIES = BO / ROWS_PER_COPY / NW;
    constexpr int STAGE_BYTES = (BR + BO) * SLAB, SCALE_BYTES = persistent_scale_bytes<Path>();
    constexpr int kStores = 2 * FR;  // of a wavefront and tile
    constexpr bool kInt8 = Path::kElemBytes == 1;
    using Acc = typename Path::Acc16;

    char *const ring = lds_dyn;
    char *const scales = lds_dyn + 2 * (256 + BO) * SLAB;  // per-tile scale vectors, double buffered by tile parity
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *const patch = scales + 2 * SCALE_BYTES + wave * (16 * kPatchPitch);
    const int wave_r = (wave / WO) * WAVE_R, wave_o = (wave % WO) * WAVE_O;
    const int l16 = lane & 15, lq = lane >> 4;

    const int last = first + n_my * stride;
    const int n_slabs = (int)(p.k_bytes / SLAB);
    const int total_slabs = n_my * n_slabs;
    if (total_slabs == 0) return;
    // The lane by way of a zero that the compiler cannot see through: addresses built on it are computed where they are used instead
    // of being hoisted out of the tile loop into scratch memory, whose loads would wait for every copy and store in flight.
    auto lane_now = [&]() {
        uint32_t zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        return (int)((threadIdx.x + zero) & 63);
    };

    // ---- producer: the next slab to copy, possibly of a later tile than the one being computed
    int pf_tile = first, pf_slab = 0, issued = 0;
    const char *pf_x = nullptr, *pf_w = nullptr;
    int pf_rows = 0, pf_cols = 0;
    auto pf_setup = [&]() {
        const int tr = pf_tile / p.tiles_o, to = pf_tile - tr * p.tiles_o;
        const int64_t r0 = (int64_t)tr * BR, o0 = (int64_t)to * BO;
        pf_x = p.x + r0 * p.ldx_bytes;
        pf_w = p.w + o0 * p.ldw_bytes;
        pf_rows = (int)min((int64_t)BR, p.M - r0), pf_cols = (int)min((int64_t)BO, p.N - o0);
    };
    const int copy_row = wave * ROWS_PER_COPY + lane / CHUNKS;  // (rows of later copies differ by multiples of 64: same swizzle, same order)
    const int copy_channel = channel_of_row(copy_row);
    const uint32_t copy_chunk = (uint32_t)((lane % CHUNKS) ^ (copy_row & 7)) * 16;
    auto issue = [&](int stage) {  // copy the producer's slab into a ring stage, then advance
        char *const sx = ring + stage * STAGE_BYTES, *const sw = sx + BR * SLAB;
        const char *const gx = pf_x + (int64_t)pf_slab * SLAB, *const gw = pf_w + (int64_t)pf_slab * SLAB;
#pragma unroll
        for (int i = 0; i < X_COPIES; i++) {  // (pitches are below 2^23)
            const uint32_t off = __umul24((uint32_t)min(copy_row + NW * ROWS_PER_COPY * i, pf_rows - 1), (uint32_t)p.ldx_bytes) + copy_chunk;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gx + off),
                                             (__attribute__((address_space(3))) void *)(sx + (wave + NW * i) * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < W_COPIES; i++) {
            const uint32_t off = __umul24((uint32_t)min(copy_channel + NW * ROWS_PER_COPY * i, pf_cols - 1), (uint32_t)p.ldw_bytes) + copy_chunk;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gw + off),
                                             (__attribute__((address_space(3))) void *)(sw + (wave + NW * i) * 1024), 16, 0, 0);
        }
        issued++;
        if (++pf_slab == n_slabs) {
            pf_slab = 0;
            pf_tile += stride;
            if (pf_tile < last) pf_setup();
        }
    };

    Acc acc[FO][FR];
    // The activations' fragments are doubled in half tiles only: beside 128 result registers each is fetched again as soon as its MFMAs have
    // been issued.
    constexpr bool TIGHT = FR == 8;
    v4i fw[2][FO], fx[TIGHT ? 1 : 2][FR];
    uint32_t frag[2];  // where row l16 of a block has the lane's operand
#pragma unroll
    for (int ks = 0; ks < 2; ks++) frag[ks] = (uint32_t)l16 * SLAB + (((4 * ks + lq) ^ (l16 & 7)) << 4);
    auto load_fw = [&](int buf, int stage, int ks) {
        const char *const sw = ring + stage * STAGE_BYTES + (BR + wave_o) * SLAB + frag[ks];
#pragma unroll
        for (int i = 0; i < FO; i++) fw[buf][i] = *reinterpret_cast<const v4i *>(sw + i * 16 * SLAB);
    };
    auto load_fx = [&](int buf, int j, int stage, int ks) {
        fx[TIGHT ? 0 : buf][j] = *reinterpret_cast<const v4i *>(ring + stage * STAGE_BYTES + wave_r * SLAB + frag[ks] + j * 16 * SLAB);
    };
    auto load_fragments = [&](int buf, int stage, int ks) {
        load_fw(buf, stage, ks);
#pragma unroll
        for (int j = 0; j < FR; j++) load_fx(buf, j, stage, ks);
    };
    auto products = [&](int buf, bool fresh, auto fetch) {  // fresh: the tile's first step; fetch(j) behind the MFMAs of row block j
        const Acc zero = {0, 0, 0, 0};
        v4i we[FO], wo[FO];
#pragma unroll
        for (int i = 0; i < FO; i++) {
            // a packed 16-byte fragment is two MFMA operands: even and odd reduction indices
            if constexpr (Path::kPacked4)
                we[i] = Path::even_codes(fw[buf][i]), wo[i] = Path::odd_codes(fw[buf][i]);
            else
                we[i] = fw[buf][i];
        }
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const v4i x = fx[TIGHT ? 0 : buf][j];
            if constexpr (Path::kPacked4) {
                const v4i xe = Path::even_codes(x), xo = Path::odd_codes(x);
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(we[i], xe, fresh ? zero : acc[i][j]);
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(wo[i], xo, acc[i][j]);
            } else {
#pragma unroll
                for (int i = 0; i < FO; i++) acc[i][j] = Path::mfma16(we[i], x, fresh ? zero : acc[i][j]);
            }
            fetch(j);
        }
    };
    // The products of buffer `buf` while the fragments of step `ks` of ring stage `stg` arrive for buffer buf ^ 1
    auto products_and_fetch = [&](int buf, bool fresh, int stg, int ks) {
        if constexpr (TIGHT) {
            load_fw(buf ^ 1, stg, ks);
            products(buf, fresh, [&](int j) {
                load_fx(0, j, stg, ks);
                __builtin_amdgcn_sched_barrier(0);  // keep a fetch behind the MFMAs that free its registers
            });
        } else {
            load_fragments(buf ^ 1, stg, ks);
            __builtin_amdgcn_sched_barrier(0);  // fetch first, then multiply
            products(buf, fresh, [](int) {});
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    pf_setup();
    issue(0);
    issue(1);  // (a tile has two slabs at least)
    wait_vmcnt_at_most<X_COPIES + W_COPIES>();
    __builtin_amdgcn_s_barrier();
    wait_lgkmcnt_0();
    load_fragments(0, 0, 0);

    int stage = 0, parity = 0;  // consumer: ring stage, scale buffer
    for (int tile = first; tile < last; tile += stride, parity ^= 1) {
        const int tile_r = tile / p.tiles_o, tile_o = tile - tile_r * p.tiles_o;
        const int64_t r0 = (int64_t)tile_r * BR, o0 = (int64_t)tile_o * BO;
        const int rows_valid = (int)min((int64_t)BR, p.M - r0), cols_valid = (int)min((int64_t)BO, p.N - o0);
        float *const cs_lds = reinterpret_cast<float *>(scales + parity * SCALE_BYTES);  // s_w of the tile's channels
        float *const rs_lds = cs_lds + BO;                                              // s_tok of the tile's rows
        uint32_t *const cb_lds = reinterpret_cast<uint32_t *>(rs_lds + 256);            // bias, two fp16 per word
        int *const cz_lds = reinterpret_cast<int *>(cb_lds + BO / 2);                   // rowsum of the tile's channels
        int *const rz_lds = cz_lds + BO;                                                // z_tok of the tile's rows

        // Scale vectors of this tile, 64 elements of 4 bytes a task, straight into LDS.  Indices beyond the matrix are clamped; those
        // rows / channels are never stored.  The tasks are dealt round-robin to the wavefronts.
        constexpr int kColTasks = BO / 64, kRowTasks = BR / 64, kBiasTasks = BO / 128;
        constexpr int kScaleTasks = kColTasks + kRowTasks + kBiasTasks, kOffsetTasks = Path::kOffset ? kColTasks + kRowTasks : 0;
        auto copy_element = [&](const void *src, void *dst) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
        };
        const int ln = lane_now();
        auto token = [&](int block) {
            const uint32_t t0 = p.M <= 0x7fffffffLL ? (uint32_t)r0 % (uint32_t)p.L : (uint32_t)(r0 % p.L);
            return (t0 + (uint32_t)min(block * 64 + ln, rows_valid - 1)) % (uint32_t)p.L;
        };
#pragma unroll
        for (int task = 0; task < kScaleTasks + kOffsetTasks; task++) {
            if (task % NW != wave) continue;
            if (task < kColTasks) {
                if constexpr (kInt8) copy_element(p.s_w + o0 + min(task * 64 + ln, cols_valid - 1), cs_lds + task * 64);
            } else if (task < kColTasks + kRowTasks) {
                if constexpr (kInt8) copy_element(p.s_tok + token(task - kColTasks), rs_lds + (task - kColTasks) * 64);
            } else if (task < kScaleTasks) {
                const int blk = task - kColTasks - kRowTasks;
                if constexpr (HAS_BIAS) copy_element(reinterpret_cast<const uint32_t *>(p.bias + o0) + min(blk * 64 + ln, cols_valid / 2 - 1), cb_lds + blk * 64);
            } else if constexpr (Path::kOffset) {
                const int blk = task - kScaleTasks;
                if (blk < kColTasks)
                    copy_element(p.rowsum + o0 + min(blk * 64 + ln, cols_valid - 1), cz_lds + blk * 64);
                else
                    copy_element(p.z_tok + token(blk - kColTasks), rz_lds + (blk - kColTasks) * 64);
            }
        }

        // One step inside a slab, one at its end (s: its number in the tile), where everyone holds the slab's last fragments
        auto step_inside = [&](bool fresh) {
            wait_lgkmcnt_0();
            products_and_fetch(0, fresh, stage, 1);
        };
        auto slab_end = [&](bool stores_younger) {  // the next slab landed and everyone here: it is visible, this one's stage is free
            wait_lgkmcnt_0();
            if (stores_younger)
                wait_vmcnt_at_most<kStores>();
            else
                wait_vmcnt_at_most<0>();
            __builtin_amdgcn_s_barrier();
            if (issued < total_slabs) issue(stage);
            stage ^= 1;
        };
        auto step_over = [&](bool stores_younger) {
            slab_end(stores_younger);
            products_and_fetch(1, false, stage, 0);
        };
        step_inside(true);
        step_over(tile != first && !DUMP_ACC);
#pragma unroll 1
        for (int s = 1; s + 1 < n_slabs; s++) {
            step_inside(false);
            step_over(false);
        }
        step_inside(false);
        slab_end(false);  // (also: the tile's scale vectors are visible)
        products(1, false, [](int) {});
        __builtin_amdgcn_sched_barrier(0);

        // ---- epilogue.  Accumulator register v of block (i, j): token row 16 j + l16, channel 32 (i / 2) + 8 lq + 4 (i mod 2) + v.
        // Each 16-row block crosses the wavefront's patch into stores of eight whole 128-byte row segments; a block's stores are issued
        // behind the conversion of the next one, so that its way through LDS costs no wait.
        const int le = lane_now(), e16 = le & 15, eq = le >> 4;
        v4f cs[FO / 2][2], cb[FO / 2];
        v4i cz[FO / 2][2];
#pragma unroll
        for (int g = 0; g < FO / 2; g++) {
            const int col = wave_o + 32 * g + 8 * eq;
#pragma unroll
            for (int h = 0; h < 2; h++) {
                cs[g][h] = *reinterpret_cast<const v4f *>(cs_lds + col + 4 * h);
                cz[g][h] = Path::kOffset ? *reinterpret_cast<const v4i *>(cz_lds + col + 4 * h) : v4i{0, 0, 0, 0};
            }
            cb[g] = HAS_BIAS ? *reinterpret_cast<const v4f *>(cb_lds + col / 2) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
        const uint32_t ldy_bytes = (uint32_t)p.ldy * 2;
        const bool whole_lines = p.ldy % 64 == 0;
        const int srow = le >> 3, scol = wave_o + (le & 7) * 8;
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
                if (whole_lines)  // non-temporal: measured 4-8 % faster than ordinary stores here
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, data[h]), y_rows, off, 0, 2);
                else  // lines shared between tiles meet in the L2
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, data[h]), y_rows, off, 0, 0);
            }
        };
#pragma unroll
        for (int j = 0; j < FR; j++) {
            const float rs = kInt8 ? rs_lds[wave_r + j * 16 + e16] : 1.0f;
            const int rz = Path::kOffset ? rz_lds[wave_r + j * 16 + e16] : 0;
            v4f out[FO / 2];
#pragma unroll
            for (int g = 0; g < FO / 2; g++) {
                const v2f lo = finish_four<Path>(acc[2 * g][j], rs, rz, cs[g][0], cz[g][0], v2f{cb[g].x, cb[g].y});
                const v2f hi = finish_four<Path>(acc[2 * g + 1][j], rs, rz, cs[g][1], cz[g][1], v2f{cb[g].z, cb[g].w});
                out[g] = v4f{lo.x, lo.y, hi.x, hi.y};
                if constexpr (DUMP_ACC) {
#pragma unroll
                    for (int c = 0; c < 8; c++) {
                        const int64_t r = r0 + wave_r + j * 16 + e16, o = o0 + wave_o + 32 * g + 8 * eq + c;
                        const int a = (int)acc[2 * g + (c >> 2)][j][c & 3];
                        if (r < p.M && o < p.N) p.acc_out[r * p.N + o] = Path::kPacked4 ? a >> 8 : a;
                    }
                }
            }
            if (j > 0) store_block(j - 1);
            asm volatile("" ::: "memory");  // wavefront-private patch: LDS runs a wavefront's accesses in order
#pragma unroll
            for (int g = 0; g < FO / 2; g++) *reinterpret_cast<v4f *>(patch + e16 * kPatchPitch + (4 * g + eq) * 16) = out[g];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int h = 0; h < 2; h++) data[h] = *reinterpret_cast<const v4f *>(patch + (h * 8 + srow) * kPatchPitch + (le & 7) * 16);
        }
        store_block(FR - 1);
        load_fragments(0, stage, 0);  // the next tile's first (behind the last tile: what is left in the ring, unused)
    }
}

// Work split.  Workgroup ids go round-robin over the XCDs; XCD x owns a contiguous range of tiles
// (channel tiles fastest, so tiles sharing an activation strip share one L2) and its workgroups
// interleave in it.  FRM = 8: 256-row tiles.  A range is whole rounds of tiles plus a partial last
// round; when that round has at most half as many tiles as the XCD has workgroups, its tiles are cut
// into two 128-row halves, which twice as many workgroups take BEFORE their whole tiles (Vim-B
// out_proj: 2.31 rounds -> 1/2 + 2 instead of 3, measured 81 -> 70 us).  A half-tile pass costs ~0.7
// of a tile (its own slab pipeline, more LDS traffic per MAC); doing it first also moves those
// workgroups' epilogues out of step with the others' (in_proj, 9.23 rounds: 149.4 -> 146.9 us; with
// the halves last it gained nothing there).  FRM = 4: every tile has 128 rows (packed 4-bit operands,
// whose expanded fragments would not fit the register file next to a 256-row tile's accumulators).
template <class Path, bool HAS_BIAS, bool DUMP_ACC, int FRM>
__global__ __launch_bounds__(512, 2) void linear_mfma_persistent(const LinearArgs p) {
    const int total_tiles = p.tiles_o * p.tiles_r;
    const int per_xcd = (total_tiles + kXcds - 1) / kXcds;
    const int wpx = (int)gridDim.x / kXcds, xcd = (int)(blockIdx.x % kXcds), j = (int)(blockIdx.x / kXcds);
    const int lo = xcd * per_xcd, hi = min(lo + per_xcd, total_tiles);
    const int n = max(hi - lo, 0);
    const int rounds = n / wpx, tail = n - rounds * wpx;
    if constexpr (FRM == 8) {
        const bool halves = tail > 0 && 2 * tail <= wpx;
        const int n_full = rounds + ((!halves && j < tail) ? 1 : 0);
        if (halves && j < 2 * tail) {
            const int tile = lo + rounds * wpx + (j >> 1);
            const int half_tile = ((tile / p.tiles_o) * 2 + (j & 1)) * p.tiles_o + tile % p.tiles_o;  // in the 128-row grid
            if ((int64_t)(half_tile / p.tiles_o) * 128 < p.M) {
                persistent_tiles<Path, HAS_BIAS, DUMP_ACC, 4>(p, half_tile, 1, 1);
                __syncthreads();  // the ring and the scale buffers change layout
            }
        }
        persistent_tiles<Path, HAS_BIAS, DUMP_ACC, 8>(p, lo + j, wpx, n_full);
    } else {
        persistent_tiles<Path, HAS_BIAS, DUMP_ACC, 4>(p, lo + j, wpx, rounds + (j < tail ? 1 : 0));
    }
}

// ------------------------------------------------------------------------------------------
// Small-K fp16 path (K bytes < 128, large results in whole lines, e.g. dt_proj with K = dt_rank): the whole reduction is 1-4 MFMA
// k-steps, so the kernel is a stream of output rows bound by the fp16 stores.  A wavefront owns
// 64 output channels for its whole life and keeps their weight fragments and biases in
// registers; it walks over 32-row blocks, fetching the activation fragments straight from
// global memory (no LDS staging of operands), and transposes results through a private LDS
// patch so that every store instruction writes eight whole 128-byte row segments.
// LOAD_ALIGN 16: pitches and bases are multiples of 16 bytes; 4: multiples of 4 bytes.  N and the pitch of y are multiples of 64,
// y is 128-byte aligned.
// ------------------------------------------------------------------------------------------
template <int LOAD_ALIGN>
__device__ __forceinline__ v4i load_fragment_chunk(const char *row_ptr, int kb, int k_bytes) {
    v4i out = {0, 0, 0, 0};
    if (kb >= k_bytes) return out;
    const int valid = min(16, k_bytes - kb);
    if constexpr (LOAD_ALIGN == 16) {
        out = *reinterpret_cast<const v4i *>(row_ptr + kb);
    } else {
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (4 * j < valid) out[j] = *reinterpret_cast<const int *>(row_ptr + kb + 4 * j);
    }
    if (valid < 16) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int nb = valid - 4 * j;
            out[j] = nb >= 4 ? out[j] : (nb <= 0 ? 0 : (out[j] & ((1 << (8 * nb)) - 1)));
        }
    }
    return out;
}

template <int KSTEPS, int LOAD_ALIGN, bool HAS_BIAS>
__global__ __launch_bounds__(kThreads) void linear_mfma_smallk(const LinearArgs p) {
    using Path = Half16Path;
    using Acc = typename Path::Acc;
    __shared__ __attribute__((aligned(16))) char patches[kWaves][32 * 64 * 2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lhalf = lane >> 5;
    const int k_bytes = (int)p.k_bytes;
    const int64_t o_base = ((int64_t)blockIdx.y * kWaves + wave) * 64;
    if (o_base >= p.N) return;  // whole wavefront out of range; no barriers are used below

    // weight fragments of the strip's 64 channels: block i covers channels 32 i .. 32 i + 31
    v4i fw[2][KSTEPS];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const char *wrow = p.w + (o_base + i * 32 + l32) * p.ldw_bytes;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ks++) fw[i][ks] = load_fragment_chunk<LOAD_ALIGN>(wrow, (2 * ks + lhalf) * 16, k_bytes);
    }
    // biases of this lane's channels: o_base + 32 i + 8 g + 4 lhalf + c
    float cb[2][4][4];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int g = 0; g < 4; g++)
#pragma unroll
            for (int c = 0; c < 4; c++) {
                cb[i][g][c] = 0.0f;
                if constexpr (HAS_BIAS) cb[i][g][c] = __half2float(p.bias[o_base + i * 32 + g * 8 + lhalf * 4 + c]);
            }

    const int64_t n_blocks = (p.M + 31) / 32;
    int64_t rb = blockIdx.x;
    auto load_x = [&](int64_t block, v4i (&fx)[KSTEPS]) {
        const int64_t row = min(block * 32 + l32, p.M - 1);
        const char *xrow = p.x + row * p.ldx_bytes;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ks++) fx[ks] = load_fragment_chunk<LOAD_ALIGN>(xrow, (2 * ks + lhalf) * 16, k_bytes);
    };
    char *patch = patches[wave];
    auto patch_chunk = [&](int row, int chunk) { return row * 128 + ((chunk ^ (row & 7)) << 4); };

    v4i fx[KSTEPS], fx_next[KSTEPS];
    if (rb < n_blocks) load_x(rb, fx);
    for (; rb < n_blocks; rb += gridDim.x) {
        const int64_t nb = rb + gridDim.x;
        if (nb < n_blocks) load_x(nb, fx_next);  // in flight while this block is computed and stored
        Acc acc[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][v] = 0;
        }
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ks++) acc[i] = Path::mfma(fw[i][ks], fx[ks], acc[i]);
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                float out[4];
#pragma unroll
                for (int c = 0; c < 4; c++) out[c] = acc[i][g * 4 + c] + cb[i][g][c];
                __half2 lo = __floats2half2_rn(out[0], out[1]);
                __half2 hi = __floats2half2_rn(out[2], out[3]);
                u32x2 packed = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                *reinterpret_cast<u32x2 *>(patch + patch_chunk(l32, i * 4 + g) + lhalf * 8) = packed;
            }
        asm volatile("" ::: "memory");  // wavefront-private patch: LDS runs a wavefront's accesses in order
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int row = q * 8 + (lane >> 3), chunk = lane & 7;
            const v4i data = *reinterpret_cast<const v4i *>(patch + patch_chunk(row, chunk));
            const int64_t rr = rb * 32 + row;
            if (rr < p.M) __builtin_nontemporal_store(data, reinterpret_cast<v4i *>(p.y + rr * p.ldy + o_base + chunk * 8));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ks++) fx[ks] = fx_next[ks];
    }
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------
template <class Path>
int launch_persistent(LinearArgs a, hipStream_t stream) {
    constexpr int FRM = Path::kPacked4 ? 4 : 8;  // tile rows / 32
    dim3 grid;
    if (!set_grid<32 * FRM, kTileCols>(a, grid)) return PTQ4VM_ERR_SHAPE;
    // One 8-wavefront workgroup per CU (all that LDS allows), a multiple of the XCD count.
    int device = 0, cus = 0;
    hipError_t err = hipGetDevice(&device);
    if (err == hipSuccess) err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (err != hipSuccess) return ptq4vm::record_hip_error(err, "hipDeviceGetAttribute(multiprocessor count)");
    unsigned wgs = (unsigned)(cus / kXcds * kXcds);
    if (wgs == 0) wgs = kXcds;
    if (wgs > grid.x) wgs = grid.x;  // grid.x is the tile count rounded up to a multiple of kXcds
    constexpr int lds_bytes = persistent_lds_bytes<Path>();
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
    using Kernel = void (*)(const LinearArgs);
    // [has bias][also write the int32 accumulators]
    static const Kernel kernels[2][2] = {{linear_mfma_persistent<Path, false, false, FRM>, linear_mfma_persistent<Path, false, true, FRM>},
                                         {linear_mfma_persistent<Path, true, false, FRM>, linear_mfma_persistent<Path, true, true, FRM>}};
    const Kernel kernel = kernels[a.bias ? 1 : 0][a.acc_out ? 1 : 0];
    if (int rc = ptq4vm::set_lds_limit(reinterpret_cast<const void *>(kernel), lds_bytes, "hipFuncSetAttribute(linear_mfma_persistent)")) return rc;
    kernel<<<dim3(wgs), dim3(512), lds_bytes, stream>>>(a);
    return ptq4vm::check_launch("linear_mfma_persistent");
}

template <int KSTEPS, int LOAD_ALIGN>
int launch_smallk(const LinearArgs &a, hipStream_t stream) {
    const int64_t strips = ptq4vm::ceil_div(a.N, 64 * kWaves), blocks = ptq4vm::ceil_div(a.M, 32);
    if (strips > 65535) return PTQ4VM_ERR_SHAPE;
    // about 8 workgroups per CU in total, each walking over row blocks
    int64_t gx = ptq4vm::ceil_div(2048, strips);
    if (gx > blocks) gx = blocks;
    dim3 grid((unsigned)gx, (unsigned)strips), block(kThreads);
    if (a.bias)
        linear_mfma_smallk<KSTEPS, LOAD_ALIGN, true><<<grid, block, 0, stream>>>(a);
    else
        linear_mfma_smallk<KSTEPS, LOAD_ALIGN, false><<<grid, block, 0, stream>>>(a);
    return ptq4vm::check_launch("linear_mfma_smallk");
}

template <int LOAD_ALIGN>
int launch_smallk_ksteps(const LinearArgs &a, hipStream_t stream) {
    const int ksteps = (int)ptq4vm::ceil_div(a.k_bytes, 32);
    if (ksteps == 1) return launch_smallk<1, LOAD_ALIGN>(a, stream);
    if constexpr (LOAD_ALIGN == 16) {
        if (ksteps == 3) return launch_smallk<3, LOAD_ALIGN>(a, stream);
        if (ksteps == 4) return launch_smallk<4, LOAD_ALIGN>(a, stream);
    }
    return launch_smallk<2, LOAD_ALIGN>(a, stream);
}

// Widest load granularity that base pointers and pitches allow for both operands.
int pick_load_align(const LinearArgs &a) {
    auto ok = [&](uintptr_t g) {
        return ptq4vm::aligned_to(a.x, g) && ptq4vm::aligned_to(a.w, g) && a.ldx_bytes % g == 0 &&
               a.ldw_bytes % g == 0;
    };
    return ok(16) ? 16 : (ok(4) ? 4 : 0);
}

template <class Path>
int dispatch(LinearArgs a, hipStream_t stream) {
    const int la = pick_load_align(a);
    a.y_vec = (a.ldy % 8 == 0 && ptq4vm::aligned_to(a.y, 16)) ? 8
              : ((a.ldy % 4 == 0 && ptq4vm::aligned_to(a.y, 8)) ? 4 : 1);
    if constexpr (Path::kElemBytes == 1) {
        // One MFMA step of K and results of 24 M elements and more in whole lines: whole rows of y streamed out by one wavefront each.  (us,
        // streamed / tiles: 39246 x 24 -> 768 [30 M] 14.0 / 18.2, 50432 x 48 -> 1536 [77 M] 34.0 / 43.0, over 160 such shapes tiles take 1.15
        // of the time, packed and offset alike, but 25216 x 24 -> 768 [19 M] 10.3 / 9.2, 29083 x 12 -> 512 [15 M] 10.3 / 9.0.  Rows of y that are
        // not whole lines, 46384 x 32 -> 712 37.6 / 16.9, 49570 x 48 -> 171 21.4 / 11.2; operands at any alignment 0.36 .. 0.7 for the
        // tiles; operands that the tiles copy directly, K a multiple of 64 bytes, 0.86 .. 0.97; two steps of K 0.82 of the time below 24 M
        // elements and as long above.)
        const int64_t codes = Path::kPacked4 ? 2 * a.k_bytes : a.k_bytes;
        const bool direct = la == 16 && a.k_bytes % 64 == 0;
        const bool whole_lines = a.N % 64 == 0 && a.ldy % 64 == 0 && ptq4vm::aligned_to(a.y, 128);
        if (codes <= 64 && la >= 4 && !direct && whole_lines && a.M * a.N >= (24LL << 20)) {
            const int rc = launch_stream_smallk(a, false, stream, Path::kPacked4, Path::kOffset);
            if (rc <= 0) return rc;
        }
    } else {
        // Results of 24 M elements and more in whole lines.  (us, channel strips / tiles: 39238 x 24 -> 768 [30 M] 15.0 / 17.8, 27273 x 14 ->
        // 1024 [28 M] 11.5 / 16.5, 39184 x 48 -> 1536 [60 M] 26.4 / 34.1, over 90 such shapes tiles take 1.19 of the time, but 25146 x 24 -> 768
        // [19 M] 11.1 / 9.5, 5852 x 12 -> 384 4.3 / 3.4, over 130 of 8 .. 24 M 0.78.  Other rows of y, 28912 x 12 -> 300 9.5 / 7.9, 13647 x 22 -> 1288
        // 20.3 / 11.3; rows of operands that start between 16-byte boundaries up to 48 bytes of K only, 39130 x 12 -> 1472 alike 1.2, but 34005 x 60
        // -> 2880 89.6 / 51.4; whole MFMA steps of K, which the tiles copy directly, 25216 x 64 -> 768 20.6 / 12.6.)
        const bool whole_lines = a.N % 64 == 0 && a.ldy % 64 == 0 && ptq4vm::aligned_to(a.y, 128);
        if (a.k_bytes <= 128 && a.k_bytes % 64 != 0 && whole_lines && a.M * a.N >= (24LL << 20)) {
            if (la == 16) return launch_smallk_ksteps<16>(a, stream);
            if (la == 4 && a.k_bytes <= 48) return launch_smallk_ksteps<4>(a, stream);
        }
    }
    // 256 x 256 tiles on one 8-wavefront workgroup per CU from a round of them on (over 400 shapes the tile kernels take 1.05 of the time of one to
    // two rounds, 1.08 .. 1.17 beyond), unless they pad the channels by more than a quarter (50240 x 768 -> 384 26.1 us against 25.0 on 256 x
    // 192 tiles; over 300 shapes 1.07 .. 1.22 of the time).
    const bool persistent_ok = la == 16 && a.ldx_bytes * 256 < (1LL << 31) && a.ldw_bytes * 256 < (1LL << 31) &&
                               a.N % 8 == 0 && a.y_vec == 8 && ptq4vm::aligned_to(a.bias, 4) &&
                               a.ldy * 512 < (1LL << 31) && a.L < (1LL << 31) && a.N >= 256 &&
                               ptq4vm::ceil_div(a.N, 256) * 256 * 4 <= a.N * 5 &&
                               a.k_bytes % kSlab == 0 && a.k_bytes >= 2 * kSlab &&
                               ptq4vm::ceil_div(a.M, 256) * ptq4vm::ceil_div(a.N, 256) >= 256;
    if (persistent_ok) return launch_persistent<Path>(a, stream);
    return launch_tiles<Path>(a, stream);
}

}  // namespace

extern "C" int ptq4vm_w8a8_linear_offset(const int8_t *xq, const int8_t *wq, const float *s_tok, const int32_t *z_tok,
                                         const int32_t *rowsum, const float *s_w, const void *bias_f16, void *y_f16,
                                         int32_t *acc_out, int64_t B, int64_t L, int64_t K, int64_t N, int64_t ldxq,
                                         int64_t ldwq, int64_t ldy, void *stream_) {
    if (!xq || !wq || !s_tok || !z_tok || !rowsum || !s_w || !y_f16) return PTQ4VM_ERR_NULL;
    if (B < 0 || N < 0 || L <= 0 || K <= 0 || K > PTQ4VM_MAX_K_OFFSET) return PTQ4VM_ERR_SHAPE;  // |acc| + |z rowsum| < 2^31
    if (B > 0 && L > INT64_MAX / B) return PTQ4VM_ERR_SHAPE;
    if (ldxq < K || ldwq < K || ldy < N) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(xq, 16) || !ptq4vm::aligned_to(wq, 16) || !ptq4vm::aligned_to(y_f16, 2) ||
        !ptq4vm::aligned_to(s_tok, 4) || !ptq4vm::aligned_to(z_tok, 4) || !ptq4vm::aligned_to(rowsum, 4) ||
        !ptq4vm::aligned_to(s_w, 4) || !ptq4vm::aligned_to(bias_f16, 2) || !ptq4vm::aligned_to(acc_out, 4))
        return PTQ4VM_ERR_ALIGN;
    const int64_t M = B * L;
    if (M == 0 || N == 0) return PTQ4VM_OK;
    LinearArgs a{};
    a.x = reinterpret_cast<const char *>(xq);
    a.w = reinterpret_cast<const char *>(wq);
    a.s_tok = s_tok;
    a.s_w = s_w;
    a.z_tok = z_tok;
    a.rowsum = rowsum;
    a.bias = static_cast<const __half *>(bias_f16);
    a.y = static_cast<__half *>(y_f16);
    a.acc_out = acc_out;
    a.M = M;
    a.N = N;
    a.k_bytes = K;
    a.ldx_bytes = ldxq;
    a.ldw_bytes = ldwq;
    a.ldy = ldy;
    a.L = L;
    return dispatch<Int8OffsetPath>(a, static_cast<hipStream_t>(stream_));
}

extern "C" int ptq4vm_w4a4_linear(const uint8_t *xq4, const uint8_t *wq4, const float *s_tok, const float *s_w,
                                  const void *bias_f16, void *y_f16, int32_t *acc_out, int64_t B, int64_t L,
                                  int64_t K, int64_t N, int64_t ldxq, int64_t ldwq, int64_t ldy, void *stream_) {
    if (!xq4 || !wq4 || !s_tok || !s_w || !y_f16) return PTQ4VM_ERR_NULL;
    // operands are codes times 16: the accumulator holds 256 acc, at most 2^14 K with the nibble -8
    if (B < 0 || N < 0 || L <= 0 || K <= 0 || K > PTQ4VM_MAX_K_W4 || K % 2 != 0) return PTQ4VM_ERR_SHAPE;
    if (B > 0 && L > INT64_MAX / B) return PTQ4VM_ERR_SHAPE;
    if (ldxq < K / 2 || ldwq < K / 2 || ldy < N) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(xq4, 16) || !ptq4vm::aligned_to(wq4, 16) || !ptq4vm::aligned_to(y_f16, 2) ||
        !ptq4vm::aligned_to(s_tok, 4) || !ptq4vm::aligned_to(s_w, 4) || !ptq4vm::aligned_to(bias_f16, 2) ||
        !ptq4vm::aligned_to(acc_out, 4))
        return PTQ4VM_ERR_ALIGN;
    const int64_t M = B * L;
    if (M == 0 || N == 0) return PTQ4VM_OK;
    LinearArgs a{};
    a.x = reinterpret_cast<const char *>(xq4);
    a.w = reinterpret_cast<const char *>(wq4);
    a.s_tok = s_tok;
    a.s_w = s_w;
    a.bias = static_cast<const __half *>(bias_f16);
    a.y = static_cast<__half *>(y_f16);
    a.acc_out = acc_out;
    a.M = M;
    a.N = N;
    a.k_bytes = K / 2;  // packed bytes
    a.ldx_bytes = ldxq;
    a.ldw_bytes = ldwq;
    a.ldy = ldy;
    a.L = L;
    return dispatch<Int4Path>(a, static_cast<hipStream_t>(stream_));
}

extern "C" int ptq4vm_w8a8_linear(const int8_t *xq, const int8_t *wq, const float *s_tok, const float *s_w,
                                  const void *bias_f16, void *y_f16, int32_t *acc_out, int64_t B, int64_t L,
                                  int64_t K, int64_t N, int64_t ldxq, int64_t ldwq, int64_t ldy, void *stream_) {
    if (!xq || !wq || !s_tok || !s_w || !y_f16) return PTQ4VM_ERR_NULL;
    if (B < 0 || N < 0 || L <= 0 || K <= 0 || K > PTQ4VM_MAX_K) return PTQ4VM_ERR_SHAPE;
    if (B > 0 && L > INT64_MAX / B) return PTQ4VM_ERR_SHAPE;
    if (ldxq < K || ldwq < K || ldy < N) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(xq, 16) || !ptq4vm::aligned_to(wq, 16) || !ptq4vm::aligned_to(y_f16, 2) ||
        !ptq4vm::aligned_to(s_tok, 4) || !ptq4vm::aligned_to(s_w, 4) || !ptq4vm::aligned_to(bias_f16, 2) ||
        !ptq4vm::aligned_to(acc_out, 4))
        return PTQ4VM_ERR_ALIGN;
    const int64_t M = B * L;
    if (M == 0 || N == 0) return PTQ4VM_OK;
    LinearArgs a{};
    a.x = reinterpret_cast<const char *>(xq);
    a.w = reinterpret_cast<const char *>(wq);
    a.s_tok = s_tok;
    a.s_w = s_w;
    a.bias = static_cast<const __half *>(bias_f16);
    a.y = static_cast<__half *>(y_f16);
    a.acc_out = acc_out;
    a.M = M;
    a.N = N;
    a.k_bytes = K;
    a.ldx_bytes = ldxq;
    a.ldw_bytes = ldwq;
    a.ldy = ldy;
    a.L = L;
    return dispatch<Int8Path>(a, static_cast<hipStream_t>(stream_));
}

extern "C" int ptq4vm_f16_linear(const void *x_f16, const void *w_f16, const void *bias_f16, void *y_f16,
                                 int64_t M, int64_t K, int64_t N, int64_t ldx, int64_t ldw, int64_t ldy,
                                 void *stream_) {
    if (!x_f16 || !w_f16 || !y_f16) return PTQ4VM_ERR_NULL;
    if (M < 0 || N < 0 || K <= 0 || K > (int64_t)1 << 40) return PTQ4VM_ERR_SHAPE;
    if (ldx < K || ldw < K || ldy < N) return PTQ4VM_ERR_STRIDE;
    if (!ptq4vm::aligned_to(x_f16, 16) || !ptq4vm::aligned_to(w_f16, 16) || !ptq4vm::aligned_to(y_f16, 2) ||
        !ptq4vm::aligned_to(bias_f16, 2))
        return PTQ4VM_ERR_ALIGN;
    if (M == 0 || N == 0) return PTQ4VM_OK;
    LinearArgs a{};
    a.x = static_cast<const char *>(x_f16);
    a.w = static_cast<const char *>(w_f16);
    a.bias = static_cast<const __half *>(bias_f16);
    a.y = static_cast<__half *>(y_f16);
    a.M = M;
    a.N = N;
    a.k_bytes = K * 2;
    a.ldx_bytes = ldx * 2;
    a.ldw_bytes = ldw * 2;
    a.ldy = ldy;
    a.L = 1;
    return dispatch<Half16Path>(a, static_cast<hipStream_t>(stream_));
}
