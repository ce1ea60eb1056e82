// Dispatch of the tile kernels (gemm_tile.hpp): every linear that the specialised kernels do not take.
#include "gemm_tile.hpp"

namespace {

using namespace ptq4vm::mfma;

int64_t tiles(const LinearArgs &a, int br, int bo) { return ptq4vm::ceil_div(a.M, br) * ptq4vm::ceil_div(a.N, bo); }

template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES, Copy COPY, bool VIA_LDS = false>
int launch(const LinearArgs &a, hipStream_t stream) {
    TileArgs t;
    dim3 grid;
    if (!tile_args<BR, BO>(a, t, grid)) return PTQ4VM_ERR_SHAPE;
    constexpr int lds_bytes = tile_lds_bytes<BR, BO, SLAB, STAGES>();
    auto kernel = linear_mfma_tile<Path, BR, BO, WR, WO, SLAB, STAGES, false, VIA_LDS, COPY>;
    if constexpr (Path::kElemBytes == 1) {
        if (a.acc_out) kernel = linear_mfma_tile<Path, BR, BO, WR, WO, SLAB, STAGES, true, VIA_LDS, COPY>;
    }
    if constexpr (lds_bytes > 64 * 1024) {
        if (int rc = ptq4vm::set_lds_limit(reinterpret_cast<const void *>(kernel), lds_bytes, "hipFuncSetAttribute(linear_mfma_tile)")) return rc;
    }
    kernel<<<grid, dim3(64 * WR * WO), lds_bytes, stream>>>(t);
    return ptq4vm::check_launch("linear_mfma_tile");
}

// Slabs through registers (any pitch, alignment and K).  A reduction of one slab: as fragments, which every wavefront loads for itself, where rows
// start at multiples of 4 bytes (over 900 shapes the way through LDS takes 1.09 to 1.15 of the time).  The loads of other rows take the
// memory path longer and are better made once for the workgroup (64 x 128 and 128 x 128 tiles 0.66 .. 0.93 of the time, 12748 x 41 -> 2056 25.5 /
// 17.1 us; 64 x 64 0.96 .. 1.01; 32 x 64 0.64 .. 0.95 above 64 bytes), but in 32 x 64 tiles up to 64 bytes latency is all (1.11 .. 1.13).
template <class Path, int BR, int BO, int WR, int WO, int SLAB>
int launch_staged(const LinearArgs &a, hipStream_t stream) {
    if (a.k_bytes > SLAB) return launch<Path, BR, BO, WR, WO, SLAB, 2, Copy::kRegisters>(a, stream);
    const bool fragments = (a.ldx_bytes % 4 == 0 && a.ldw_bytes % 4 == 0) || (BR * BO <= 32 * 64 && a.k_bytes <= 64);
    return fragments ? launch<Path, BR, BO, WR, WO, SLAB, 2, Copy::kOneSlab>(a, stream) : launch<Path, BR, BO, WR, WO, SLAB, 2, Copy::kOneSlab, true>(a, stream);
}

template <class Path, int FR, int FO, int SK, int U, Rows ROWS>
int launch_splitk(LinearArgs a, hipStream_t stream) {
    dim3 grid;
    if (!set_grid<16 * FR, 16 * FO>(a, grid)) return PTQ4VM_ERR_SHAPE;
    linear_mfma_splitk<Path, FR, FO, SK, U, ROWS><<<grid, dim3(64 * SK), 0, stream>>>(a);
    return ptq4vm::check_launch("linear_mfma_splitk");
}

}  // namespace

// The rule: the largest tile that still leaves the 256 CUs a few workgroups each, because a larger tile moves fewer
// operand bytes per product, but a CU needs several resident workgroups to overlap one's copies and stores with
// another's MFMAs; and tiles that take a CU each, where they fill their rounds of 256.  The lines were read off sweeps over 170 random and
// model shapes (M 49 .. 50 240, K 64 .. 2048, N 16 .. 3072, int8 and fp16).  Around the lines (us, int8; tiles in brackets):
//   256 x 256, one round:                    9456 x 384 -> 1536 [222] 11.6 / 13.0 (64 x 128); 18912 x 1536 -> 768 [222] 25.6 / 29.9; 18912 x 192 -> 768 [222] 9.6 / 10.6
//   256 x 192, a round filled to 70 % or two to 75 %: 25216 x 768 -> 384 [198] 12.7 / 14.8 (64 x 128); 6304 x 384 -> 1536 [200] 9.4 / 10.1; 12608 x 1536 -> 768 [200] 19.9 / 22.8;
//                                            50240 x 768 -> 384 [394] 25.3 / 26.2 (128 x 128), but short K 12608 x 192 -> 768 [200] 7.9 / 7.2, half-filled 18912 x 768 -> 384 [148] 12.0 / 11.7;
//                                            over 900 shapes the other tiles take 1.08 of the time at 70 .. 75 % of one round and 1.14 .. 1.18 beyond, of two rounds
//                                            0.96 below 75 % and 1.03 .. 1.12 above, and of three and more 0.88 .. 0.99, most 128 x 256 (offset 49220 x 768 ->
//                                            3072, odd rows of y 242 / 201, 23274 x 832 -> 1024 42.4 / 34.5)
//   128 x 256 against 128 x 128, 800 tiles:  25216 x 384 -> 1536 [1182] 28.1 / 29.8; 13057 x 192 -> 2048 [824] 16.8 / 16.2, but 12608 x 192 -> 768 [297] 7.7 / 7.2
//   128 x 128 against 64 x 128, 384 tiles:   4728 x 384 -> 1536 [444] 7.4 / 7.6;         9456 x 384 -> 192 [148] 5.3 / 5.1, 6304 x 768 -> 384 [150] 6.6 / 6.5
//   64 x 128 against 64 x 64, 384 tiles:     3152 x 384 -> 1536 [600] 6.1 / 7.2;         6304 x 768 -> 384 [297] 6.5 / 6.3
//   64 x 64 against 32 x 64, 200 tiles:      3152 x 768 -> 384 [300] 4.8 / 5.0;          197 x 768 -> 3072 [192] 4.6 / 4.3
//   split reduction, 256 blocks of 16 x 16:  788 x 1536 -> 80 [250] 4.3 / 5.1 (32 x 64); 1576 x 1536 -> 80 [495] 5.6 / 5.1
// 128 x 128 tiles: three 64-byte stages on four wavefronts let three workgroups share a CU and waste no half slab (25216 x 192 -> 1536 21.6 / 25.3);
// over a long reduction twice the barriers cost more (12608 x 1536 -> 768 25.6 / 23.3).  64 x 64 tiles: three stages hold more of a long reduction in flight where few
// tiles are resident (6304 x 1536 -> 80 [198] 6.4 / 8.2 with two), two leave room for a fourth workgroup per CU: from 513 tiles, and from 769 with less
// than 256 bytes of K, which take one or two slabs anyway (over 900 shapes of 513 .. 768 tiles two take 1.02 of the time at 64 bytes, 0.99 up to 383,
// 0.95 up to 1023, 0.93 beyond; 35992 x 1920 -> 64 [563] 16.6 / 15.1).
// A tile that pads the matrix by a third more than the best one is passed over.
template <class Path>
int ptq4vm::mfma::launch_tiles(const LinearArgs &a, hipStream_t stream) {
    const bool aligned = ptq4vm::aligned_to(a.x, 16) && ptq4vm::aligned_to(a.w, 16) && a.ldx_bytes % 16 == 0 && a.ldw_bytes % 16 == 0 &&
                         a.k_bytes % 64 == 0;
    // 32-bit offsets inside a tile and token positions; the split-reduction kernel takes any size
    const bool small = a.ldx_bytes * 256 < (1LL << 31) && a.ldw_bytes * 256 < (1LL << 31) && a.L < (1LL << 31);
    if (aligned && small) {
        if (tiles(a, 16, 16) <= 256) return launch_splitk<Path, 1, 1, 4, 4, Rows::kAligned>(a, stream);
        auto padded = [&](int br, int bo) { return tiles(a, br, bo) * br * bo; };
        const int64_t most = padded(32, 64) * 4 / 3;
        auto fills = [&](int br, int bo, int percent) {  // whole rounds of 256 workgroups, the last one to `percent`
            const int64_t n = tiles(a, br, bo);
            return n * 100 >= ptq4vm::ceil_div(n, 256) * 256 * percent;
        };
        if constexpr (!Path::kPacked4) {  // (packed operands are expanded into more registers than these leave)
            if (tiles(a, 256, 256) <= 256 && fills(256, 256, 80) && padded(256, 256) <= most) return launch<Path, 256, 256, 2, 4, 128, 2, Copy::kDirect>(a, stream);
            const int rounds = tiles(a, 256, 192) <= 256 ? 1 : tiles(a, 256, 192) <= 512 ? 2 : 3;
            if (a.k_bytes >= 384 && rounds < 3 && fills(256, 192, rounds == 1 ? 70 : 75) && padded(256, 192) <= most) return launch<Path, 256, 192, 4, 3, 128, 2, Copy::kDirect>(a, stream);
        }
        if (tiles(a, 128, 256) >= 800 && padded(128, 256) <= most) return launch<Path, 128, 256, 2, 4, 64, 3, Copy::kDirect>(a, stream);
        if (tiles(a, 128, 128) >= 384 && padded(128, 128) <= most)
            return a.k_bytes <= 768 ? launch<Path, 128, 128, 2, 2, 64, 3, Copy::kDirect>(a, stream) : launch<Path, 128, 128, 2, 4, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 128) >= 384 && padded(64, 128) <= most) return launch<Path, 64, 128, 2, 2, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 64) > (a.k_bytes < 256 ? 768 : 512)) return launch<Path, 64, 64, 2, 2, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 64) >= 200) return launch<Path, 64, 64, 2, 2, 128, 3, Copy::kDirect>(a, stream);
        return launch<Path, 32, 64, 2, 2, 128, 3, Copy::kDirect>(a, stream);
    }
    // Any pitch, alignment and K.  Loads go through registers, so the small tiles hide less of their latency and the
    // split reduction, with all of its loads in flight, holds out longer: to 1000 blocks of 32 x 32 where rows start at multiples of 4 bytes
    // (1707 x 1528 -> 424 [756] 9.1 us, staged tiles 9.7; staged tiles take 1.33 of the time at 151 .. 250 blocks, 1.06 to 600, 0.94 beyond, but up to
    // 1.27 of it for single shapes), to 250 where they start at any byte, whose loads take the memory path longer and which the tiles make
    // fewer of (6399 x 993 -> 138 [1000] 17.4 / 10.1, 281 x 581 -> 2543 [720] 10.7 / 6.3, 2436 x 530 -> 127 [308] 7.2 / 5.0; 0.92 of the time at 151 ..
    // 250 blocks, 0.64 to 500, 0.5 beyond).  128 x 128 tiles from 300 of them (to 600 the smaller ones take 1.02 of the time up to 320 bytes of K,
    // 1.12 up to 1023, 1.27 beyond), there with 128-byte slabs from 1024 bytes of K, unless they pad the matrix by a third more than 64 x 64 ones
    // (half-padded ones, 46670 x 1968 -> 61, 1.4 times); with one or two slabs their larger epilogue counts more (11938 x 32 -> 745 [564 tiles]
    // 10.4 / 9.0) and they start at 1600.
    if (is_tiny(a.M, a.ldx_bytes, a.k_bytes)) return launch_splitk<Path, 1, 1, 1, 1, Rows::kTiny>(a, stream);
    if (is_tiny(a.N, a.ldw_bytes, a.k_bytes)) return launch_splitk<Path, 1, 1, 1, 1, Rows::kTinyWeight>(a, stream);
    if (tiles(a, 16, 16) <= 600) return launch_splitk<Path, 1, 1, 4, 4, Rows::kAny>(a, stream);
    const bool words = a.ldx_bytes % 4 == 0 && a.ldw_bytes % 4 == 0;
    if (!small || (a.k_bytes > 256 && tiles(a, 32, 32) <= (words ? 1000 : 250))) return launch_splitk<Path, 2, 2, 4, 3, Rows::kAny>(a, stream);
    if (tiles(a, 128, 128) >= (a.k_bytes > 128 ? 300 : 1600) && 3 * tiles(a, 128, 128) * 128 * 128 <= 4 * tiles(a, 64, 64) * 64 * 64)
        return a.k_bytes < 1024 ? launch_staged<Path, 128, 128, 2, 4, 64>(a, stream) : launch_staged<Path, 128, 128, 2, 4, 128>(a, stream);
    if (tiles(a, 64, 128) >= 800) return launch_staged<Path, 64, 128, 2, 2, 64>(a, stream);
    if (tiles(a, 64, 64) >= 150)
        return a.k_bytes <= 320 ? launch_staged<Path, 64, 64, 2, 2, 64>(a, stream) : launch_staged<Path, 64, 64, 2, 2, 128>(a, stream);
    return launch_staged<Path, 32, 64, 2, 2, 128>(a, stream);
}

template int ptq4vm::mfma::launch_tiles<ptq4vm::mfma::Int8Path>(const LinearArgs &, hipStream_t);
template int ptq4vm::mfma::launch_tiles<ptq4vm::mfma::Int8OffsetPath>(const LinearArgs &, hipStream_t);
template int ptq4vm::mfma::launch_tiles<ptq4vm::mfma::Int4Path>(const LinearArgs &, hipStream_t);
template int ptq4vm::mfma::launch_tiles<ptq4vm::mfma::Half16Path>(const LinearArgs &, hipStream_t);
