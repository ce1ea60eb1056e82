// Dispatch of the tile kernels (gemm_tile.hpp): every linear that the specialised kernels do not take.
#include "gemm_tile.hpp"

namespace {

using namespace ptq4vm::mfma;

int64_t tiles(const LinearArgs &a, int br, int bo) { return ptq4vm::ceil_div(a.M, br) * ptq4vm::ceil_div(a.N, bo); }

template <class Path, int BR, int BO, int WR, int WO, int SLAB, int STAGES, Copy COPY>
int launch(LinearArgs a, hipStream_t stream) {
    dim3 grid;
    if (!set_grid<BR, BO>(a, grid)) return PTQ4VM_ERR_SHAPE;
    constexpr int lds_bytes = tile_lds_bytes<BR, BO, SLAB, STAGES>();
    auto kernel = linear_mfma_tile<Path, BR, BO, WR, WO, SLAB, STAGES, COPY>;
    if constexpr (lds_bytes > 64 * 1024) {
        if (int rc = ptq4vm::set_lds_limit(reinterpret_cast<const void *>(kernel), lds_bytes, "hipFuncSetAttribute(linear_mfma_tile)")) return rc;
    }
    kernel<<<grid, dim3(64 * WR * WO), lds_bytes, stream>>>(a);
    return ptq4vm::check_launch("linear_mfma_tile");
}

// Slabs through registers (any pitch, alignment and K).
template <class Path, int BR, int BO, int WR, int WO, int SLAB>
int launch_staged(const LinearArgs &a, hipStream_t stream) {
    return a.k_bytes <= SLAB ? launch<Path, BR, BO, WR, WO, SLAB, 2, Copy::kOneSlab>(a, stream) : launch<Path, BR, BO, WR, WO, SLAB, 2, Copy::kRegisters>(a, stream);
}

template <class Path, int FR, int FO, int SK, int U, bool ALIGNED>
int launch_splitk(LinearArgs a, hipStream_t stream) {
    dim3 grid;
    if (!set_grid<16 * FR, 16 * FO>(a, grid)) return PTQ4VM_ERR_SHAPE;
    linear_mfma_splitk<Path, FR, FO, SK, U, ALIGNED><<<grid, dim3(64 * SK), 0, stream>>>(a);
    return ptq4vm::check_launch("linear_mfma_splitk");
}

}  // namespace

// The rule: the largest tile that still leaves the 256 CUs a few workgroups each, because a larger tile moves fewer
// operand bytes per product, but a CU needs several resident workgroups to overlap one's copies and stores with
// another's MFMAs.  The thresholds were read off sweeps over 130 random and model shapes (M 50 .. 50 432, K 24 .. 2048,
// N 16 .. 3072, int8 and fp16): the rule costs 2 % on average against the best tile of each shape.  Around the lines
// (us, int8 unless said; tiles in brackets):
//   128 x 256 against 128 x 128, 800 tiles:  12608 x 768 -> 3072 [1188] 46.6 / 52.0;   9485 x 512 -> 1328 [450] 15.0 / 16.0, but 16346 x 384 -> 464 [256] 10.0 / 9.2
//   128 x 128 against 64 x 128, 384 tiles:   50432 x 1536 -> 80 [394] 17.0 / 22.8;     12608 x 384 -> 192 [198] 5.3 / 5.4, 6304 x 768 -> 384 [150] 6.8 / 6.8
//   64 x 128 against 64 x 64, 384 tiles:     3152 x 384 -> 1536 [600] 7.2 / 7.9;       1576 x 384 -> 1536 [300] 5.5 / 5.0
//   64 x 64 against 32 x 64, 190 tiles:      197 x 768 -> 3072 [192] 4.8 / 5.9;        197 x 1536 -> 768 [48] 5.5 / 5.0
//   split reduction, 256 blocks of 16 x 16:  197 x 1536 -> 80 [65] 3.8 / 4.8 (32 x 64); 659 x 256 -> 232 [630] 3.3 / 2.9
// 128 x 128 tiles: three 64-byte stages are 48 KiB, a third workgroup per CU, and waste no half slab; over a long reduction
// twice the barriers cost more (12608 x 192 -> 768 9.0 / 10.8, 6304 x 384 -> 1536 11.2 / 11.8, 50240 x 768 -> 384 32.0 / 33.4,
// but 12608 x 1536 -> 768 25.0 / 24.6).
// A tile that pads the matrix by a third more than the best one is passed over.  Two or three ring stages of 64 x 64
// tiles: three hold more of a long reduction in flight while few tiles are resident anyway (6304 x 1536 -> 80 [198]
// 6.2 / 8.0), two leave room for a fourth workgroup per CU (788 x 768 -> 3072 [624] 7.3 / 7.9).
// Before these kernels everything here ran on 256 x 128 tiles: 12.3 .. 24 us for the 197-row shapes (now 2.9 .. 5.5),
// 17.3 us for 3152 x 768 -> 384 (5.0), 36.0 us for 12608 x 1536 -> 768 (24.4), 72 us for 19231 x 960 -> 1057 (33.4).
template <class Path>
int ptq4vm::mfma::launch_tiles(const LinearArgs &a, hipStream_t stream) {
    const bool aligned = ptq4vm::aligned_to(a.x, 16) && ptq4vm::aligned_to(a.w, 16) && a.ldx_bytes % 16 == 0 && a.ldw_bytes % 16 == 0 &&
                         a.k_bytes % 64 == 0;
    // 32-bit offsets inside a tile and token positions; the split-reduction kernel takes any size
    const bool small = a.ldx_bytes * 256 < (1LL << 31) && a.ldw_bytes * 256 < (1LL << 31) && a.L < (1LL << 31);
    if (aligned && small) {
        if (tiles(a, 16, 16) <= 256) return launch_splitk<Path, 1, 1, 4, 4, true>(a, stream);
        auto padded = [&](int br, int bo) { return tiles(a, br, bo) * br * bo; };
        const int64_t most = padded(32, 64) * 4 / 3;
        if (tiles(a, 128, 256) >= 800 && padded(128, 256) <= most) return launch<Path, 128, 256, 2, 4, 64, 3, Copy::kDirect>(a, stream);
        if (tiles(a, 128, 128) >= 384 && padded(128, 128) <= most)
            return a.k_bytes <= 768 ? launch<Path, 128, 128, 2, 4, 64, 3, Copy::kDirect>(a, stream) : launch<Path, 128, 128, 2, 4, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 128) >= 384 && padded(64, 128) <= most) return launch<Path, 64, 128, 2, 2, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 64) > 512) return launch<Path, 64, 64, 2, 2, 128, 2, Copy::kDirect>(a, stream);
        if (tiles(a, 64, 64) >= 190) return launch<Path, 64, 64, 2, 2, 128, 3, Copy::kDirect>(a, stream);
        return launch<Path, 32, 64, 2, 2, 128, 3, Copy::kDirect>(a, stream);
    }
    // Any pitch, alignment and K.  Loads go through registers, so the small tiles hide less of their latency and the
    // split reduction, with all of its loads in flight, holds out longer (1707 x 1528 -> 424 [756 blocks of 32 x 32] 9.6 us
    // against 12.5); the element-wise loads and stores used before took 86 us there, 396 us for 24104 x 830 -> 760 (now 36)
    // and 79 us for 3184 x 1000 -> 500 (10.3).  128 x 128 tiles from 300 of them unless they pad the matrix by a third more than
    // 64 x 64 ones (against 64 x 128 tiles, over 300 shapes: 0.7 .. 0.85 of the time from 1024 bytes of K, there with 128-byte
    // slabs, 0.85 .. 0.95 below; half-padded ones, 46670 x 1968 -> 61, 1.4 times); with one or two slabs their larger epilogue
    // counts more (11938 x 32 -> 745 [564 tiles] 10.4 / 9.0) and they start at 1600.
    if (tiles(a, 16, 16) <= 600) return launch_splitk<Path, 1, 1, 4, 4, false>(a, stream);
    if (!small || (a.k_bytes > 256 && tiles(a, 32, 32) <= 1000)) return launch_splitk<Path, 2, 2, 4, 3, false>(a, stream);
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
