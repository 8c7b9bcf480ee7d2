// The tile shapes that gemm_kernel is built for, and the choice among them (host side).
#pragma once
#include "pk_gemm.h"

namespace pk {

// A tile shape.  From T32x64 on the waves take k-tiles of their own (WM = WN = 1: not for the all-gather of column chunks).
enum Tile { T256x256, T256x128, T128x256, T128x128, T128x64, T64x64, T32x64, T32x32, N_TILES };

struct TileDim {
    int bm, bn;
};
constexpr TileDim kTileDim[N_TILES] = {{256, 256}, {256, 128}, {128, 256}, {128, 128}, {128, 64}, {64, 64}, {32, 64}, {32, 32}};

// waves (WM x WN x WK), k-tile bytes and ring stages of a tile shape.  bf16: the smaller tiles split the k-steps of a k-tile
// over two groups of waves (WK = 2), which keeps the wave's sub-tile large and with it the LDS reads per flop low: 64 x 64
// sub-tiles of one 128 x 128 tile ran 16.4 us against 18.5 us for four waves without the split (2048 x 1024 x 2048).  fp8 has
// only two k-steps in a 128-byte k-tile and half as many fragment reads per flop: there the split gains nothing.
// A k-contiguous second operand is fetched as one piece per row and k-tile, and 64-byte pieces use half of every 128-byte line
// they touch: 128-byte k-tiles throughout.
// 256x256 in bf16: two stages of 128 bytes.  With the barrier in the middle of a k-step (gemm_kernel, MID) they have time enough to land,
// and there is half the barrier and branch work of 64-byte k-tiles in four stages (2367 cycles per 128 bytes, 2400 so; us a call: 8192 x 8192 x
// 512 reduce-scatter 128 / 131, 8192 x 3584 x 8192 column chunks 365 / 373, 8192 x 8192 x 3584 0.908 / 0.928 of what it was before).
// The two smallest serve calls of a few dozen rows, which stream the second operand past a handful of flops: what bounds them is
// how many compute units load at once, and the time from a load to the MFMA behind it.  A wave that takes every fourth k-tile
// through a ring of its own needs no barrier per k-tile (64 x 3584 x 8192, second operand k-contiguous: 64x32 tiles 19.3 us with
// the ring shared, 19.0 us without; 32x32 tiles 15.4 us, 64x64 tiles 24.0 us).
struct TileWaves {
    int wm, wn, wk, kb, ns;
};
constexpr TileWaves tile_waves(int tile, bool fp8, bool bt, bool sk) {
    switch (tile) {
        case T256x256: return bt || !(fp8 || sk) ? TileWaves{2, 4, 1, 128, 2} : TileWaves{2, 4, 1, 64, 4};
        case T256x128: return fp8 ? TileWaves{4, 2, 1, 128, 3} : TileWaves{2, 2, 2, 128, 3};
        case T128x256: return bt ? TileWaves{2, 4, 1, 128, 3} : TileWaves{2, 4, 1, 64, 4};
        case T128x128: return fp8 ? TileWaves{4, 2, 1, 128, 4} : TileWaves{2, 2, 2, 128, 4};
        case T128x64: return fp8 ? TileWaves{2, 2, 1, 128, 6} : TileWaves{2, 2, 2, 128, 4};
        case T64x64: return fp8 ? TileWaves{2, 1, 1, 128, 6} : TileWaves{2, 1, 2, 128, 6};
        case T32x64: return TileWaves{1, 1, 4, 128, 3};
        default: return TileWaves{1, 1, 4, 128, 4};      // T32x32
    }
}

// bf16 products by 16x16x32 MFMAs.  The large tiles run at the clock that the power limit leaves them, and an MFMA that keeps a quarter
// of the accumulators for twice as long takes less of it: a loop of nothing else on random operands 1990 TFLOP/s at 2.03 GHz, of
// 32x32x16 1730 at 1.76 (with 8-bit operands 16x16x128 4270 and 32x32x64 3890).  us a call, 32x32 / 16x16: 8192 x 3584 x 8192 all-gather 381
// / 354 (k-contiguous 368 / 337), 8192 x 8192 x 3584 reduce-scatter 442 / 411, 4096 x 1792 x 4096 58.0 / 54.5, 1024 x 8192 x 3584 67.4 / 63.4.
// The 128x128 and 128x64 tiles gain up to 2% (296 x 7440 x 1088 16.6 / 16.3; 1512 x 1720 x 5120 37.9 / 38.0, nothing).  The smallest tiles are bound by their loads; the kernels with a
// stream-K tail have no registers left for the second form's addresses.
constexpr bool tile_m16(int tile, bool fp8, bool sk) { return !fp8 && !sk && tile < T64x64; }

// Estimated time, in nanoseconds x grid, of `tiles` tiles over `kt` 128-byte k-tiles on `grid` workgroups: rounds x (fixed part
// + k-tile time), the k-tile time rising with the share of the compute units at work (clock, L2 and memory traffic).  The figures are
// fitted, per layout of the second operand, to 5260 calls of all ops (16 .. 16384 rows, 256 .. 8192 columns, k from 256 to 16384, half of
// them chosen near a tie, on seven cards), each timed with every tile shape.  Of the 2720 that were not, the choice is the fastest tile or
// within 3% of it for 98% (fp8 97%), 0.2% off on average (fp8 0.3%) and more than 6% off for 0.7% (fp8 1.4%); the figures from before the
// 16x16x32 MFMAs, which put the large bf16 tiles too high, were more than 6% off for 2% (fp8 5%).  us a call, by those / by these: 11944 x
// 280 x 6400 k-contiguous 89.5 (128x64) / 58.5 (256x128), 6524 x 2584 x 16256 741 (128x128) / 612 (256x128), 2356 x 7760 x 5376 k-contiguous
// 259 (128x128) / 204 (128x256), fp8 4914 x 3984 x 15360 315 (128x256) / 277 (256x128).  Some are slower: of 130 calls that changed 87 gained
// more than 1% and 11 lost as much (fp8 13131 x 592 x 15872 155 / 178, the worst).  What the estimate does not count are the stores of
// fp32 slots; and many rounds of fp8 tiles are off (see ag_route).
struct TileCost {
    int lo, hi, fixed;        // ns per k-tile with few and with all compute units at work, ns per tile
};
// [fp8][second operand k-contiguous]
constexpr TileCost kTileCost[2][2][N_TILES] = {
    {{{547, 1429, 6055}, {299, 761, 5537}, {399, 887, 3060}, {281, 435, 3247}, {201, 368, 1742}, {170, 217, 2498}, {150, 176, 1767}, {119, 151, 1343}},
     {{469, 1378, 8306}, {319, 719, 6483}, {388, 779, 4348}, {281, 423, 3949}, {210, 295, 2623}, {170, 217, 2498}, {150, 176, 1767}, {119, 151, 1343}}},
    {{{754, 1401, 6071}, {312, 766, 4820}, {399, 885, 2841}, {313, 472, 2616}, {277, 376, 1982}, {245, 295, 1913}, {196, 248, 1638}, {162, 220, 1349}},
     {{754, 1401, 6071}, {297, 802, 4372}, {304, 803, 4313}, {313, 472, 2616}, {277, 376, 1982}, {245, 295, 1913}, {196, 248, 1638}, {162, 220, 1349}}}};
// row_chunks: pk_ag_gemm.  The other calls fill the load ring anew behind the own column chunk or store more of a tile, which costs the 128x64
// tiles of bf16 and a row-major operand more than the smaller 64x64 ones: 600 ns as fitted to 77 calls, in which the choice
// between the two is 0.5% off on average with it and 7% without for pk_ag_gemm_k, 1.4% and 2.3% for the reduce-scatters, but 6% and
// 0.2% for pk_ag_gemm.  us a call, 128x64 / 64x64: ag_gemm_k 180 x 1616 x 768 9.6 / 8.9, 50 x 472 x 512 8.69 / 7.72, gemm_ar 552 x 1400 x
// 704 16.3 / 15.3; ag_gemm 384 x 2688 x 384 15% less.  Of 70 other calls that it moved 59 gained more than 1% and 5
// lost as much (ag_gemm_k 853 x 824 x 512 7.8 -> 8.3; the others are two kernels in 10-15 us, bound by host time), 6% less on average.
inline int64_t tile_cost(int tile, bool fp8, bool bt, bool row_chunks, int tiles, int kt, int grid) {
    TileCost c = kTileCost[fp8 ? 1 : 0][bt ? 1 : 0][tile];
    if (tile == T128x64 && !fp8 && !bt && !row_chunks) c.fixed += 600;
    const int rounds = (int)((((unsigned)tiles + 7) / 8 * 8 + grid - 1) / (unsigned)grid);
    return (int64_t)rounds * grid * (c.fixed + (int64_t)kt * c.lo) + (int64_t)kt * (c.hi - c.lo) * tiles;
}
inline int tiles_across(int64_t size, int tile_size) {       // size / tile_size, rounded up; tile_size is 32, 64, 128 or 256
    const int shift = tile_size == 32 ? 5 : tile_size == 64 ? 6 : tile_size == 128 ? 7 : 8;
    return (int)((size + tile_size - 1) >> shift);
}

// Launches one GEMM on `grid` workgroups with the given tile shape (defined in the gemm_*.hip file of its mode).  a.ktiles
// counts k-tiles of 128 bytes.  `sk`: with the stream-K tail that `a` describes (T256x256, not with bt).
template <int EPI>
pk_status launch_gemm(GemmArgs a, int tile, bool fp8, bool bt, bool sk, int grid, hipStream_t stream);

// ---- definition, included by the gemm_*.hip files only ----
#ifdef PK_DEFINE_LAUNCH
template <int TILE, bool FP8, int EPI, bool BT, bool SK>
static pk_status launch_kernel(GemmArgs a, int grid, hipStream_t stream) {
    constexpr int BM = kTileDim[TILE].bm, BN = kTileDim[TILE].bn;
    constexpr TileWaves W = tile_waves(TILE, FP8, BT, SK);
    static std::atomic<uint64_t> configured{0};              // bit d = dynamic LDS size raised on device d
    auto kern = gemm_kernel<BM, BN, W.wm, W.wn, W.wk, W.kb, W.ns, FP8, EPI, BT, SK, tile_m16(TILE, FP8, SK)>;
    constexpr int lds = gemm_lds_bytes<BM, BN, W.kb, W.ns * (W.wm * W.wn == 1 ? W.wk : 1)>();
    static_assert(lds <= 160 * 1024, "a compute unit has 160 KB of LDS");
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return PK_ERR_HIP;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(configured.load(std::memory_order_acquire) & bit)) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return PK_ERR_HIP;
        configured.fetch_or(bit, std::memory_order_release);
    }
    a.ktiles = a.ktiles * 128 / W.kb;
    a.set_divisors();
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * W.wm * W.wn * W.wk), lds, stream, a);
    return hipGetLastError() == hipSuccess ? PK_OK : PK_ERR_HIP;
}

template <int EPI>
pk_status launch_gemm(GemmArgs a, int tile, bool fp8, bool bt, bool sk, int grid, hipStream_t stream) {
    constexpr bool BASE = EPI == EPI_RS || EPI == EPI_AG;    // the modes with a k-contiguous second operand and a stream-K tail
    if ((bt || sk) && !BASE) return PK_ERR_ARG;
    if constexpr (BASE) {
        if (sk) {
            if (bt || tile != T256x256) return PK_ERR_ARG;
            return fp8 ? launch_kernel<T256x256, true, EPI, false, true>(a, grid, stream)
                       : launch_kernel<T256x256, false, EPI, false, true>(a, grid, stream);
        }
    }
    auto go = [&](auto tile_c) -> pk_status {
        constexpr int T = decltype(tile_c)::value;
        if constexpr (BASE) {
            if (bt)
                return fp8 ? launch_kernel<T, true, EPI, true, false>(a, grid, stream)
                           : launch_kernel<T, false, EPI, true, false>(a, grid, stream);
        }
        return fp8 ? launch_kernel<T, true, EPI, false, false>(a, grid, stream)
                   : launch_kernel<T, false, EPI, false, false>(a, grid, stream);
    };
    switch (tile) {
        case T256x256: return go(std::integral_constant<int, T256x256>{});
        case T256x128: return go(std::integral_constant<int, T256x128>{});
        case T128x256: return go(std::integral_constant<int, T128x256>{});
        case T128x128: return go(std::integral_constant<int, T128x128>{});
        case T128x64: return go(std::integral_constant<int, T128x64>{});
        case T64x64: return go(std::integral_constant<int, T64x64>{});
        default: break;
    }
    if constexpr (EPI != EPI_AGK) {
        if (tile == T32x64) return go(std::integral_constant<int, T32x64>{});
        if (tile == T32x32) return go(std::integral_constant<int, T32x32>{});
    }
    return PK_ERR_ARG;
}
#endif  // PK_DEFINE_LAUNCH

}  // namespace pk
