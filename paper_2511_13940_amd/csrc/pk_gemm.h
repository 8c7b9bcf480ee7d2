// The MFMA GEMM kernel behind pk_gemm_rs and pk_ag_gemm (gfx950 only).
//
// A persistent workgroup of WM x WN waves walks over BM x BN tiles of the local product; each wave owns a
// (BM/WM) x (BN/WN) sub-tile as 32x32 or 16x16 MFMA accumulators.  The reduction runs in k-tiles of KB bytes of
// A-row (KB = 64 or 128: 32 or 64 bf16, 64 or 128 fp8):
//   * the A tile (BM x KB bytes) and B tile (KB*BN bytes) are copied global -> LDS with 16-byte
//     direct-to-LDS loads (no VGPR staging) into a ring of NS LDS stages, NS-1 k-tiles ahead of their use,
//     so that the loads of a k-tile have NS-1 k-tiles of time to land and are issued a few per k-tile;
//   * A fragments are read with ds_read_b128, B fragments with the transposing ds_read_b64_tr_b16 /
//     _tr_b8 (B is row-major K x N, the MFMA wants k-contiguous lanes);
//   * the A tile is XOR-swizzled at 16-byte-chunk granularity; the bf16 B tile is laid out as 64-column
//     panels (the fp8 B tile as swizzled rows); a direct-to-LDS load writes lane l's 16 bytes at
//     base + 16*l, so a layout is applied by choosing which global chunk each lane fetches;
//   * the loop is software-pipelined: the fragments of k-step s+1 are read while the MFMAs of step s issue,
//     and the single barrier of a k-tile sits before its last k-step (16x16 MFMAs: a quarter into it), so the
//     loads of a later k-tile and the first fragments of the next k-tile are issued under that step's MFMAs.
// The operands are passed to the MFMA swapped (B fragment first), which leaves each lane with four
// consecutive columns of one row; the epilogue transposes through a 32 KB LDS staging area so that global
// stores are 16 bytes per lane over whole row segments of the wave's sub-tile.  The epilogue of tile t runs
// after the first loads of tile t+1 have been issued.  Tiles below 256x256, most of them (ROWX), leave behind their own
// main loop instead, all at once through the LDS of the ring.
//
// Roles of the paper's program template (section 3.2.3, appendix D): the direct-to-LDS loads are the
// loader, the MFMA loop the consumer, the epilogue the storer; the epilogue of the reduce-scatter mode
// also does the per-tile `signal` (section 3.1.3, intra-SM overlap: the transfer is issued from the
// compute workgroup itself).  In all-gather mode the workgroup does the `wait` on its chunk's flag
// before its first load (section 3.1.3, inter-SM overlap seen from the compute side).
#pragma once
#include <type_traits>

#include "pk_device.h"

namespace pk {

// reduce-scatter with fp32 slots; all-gather of row chunks; reduce-scatter with bf16 slots; all-gather of column (K) chunks
enum { EPI_RS = 0, EPI_AG = 1, EPI_RS16 = 2, EPI_AGK = 3 };

// Division by a divisor that the host knows: q = floor(n * floor(2^32 / d) / 2^32) is n / d or one less, for every 32-bit n, so
// one correction makes it exact.  Four scalar instructions where a general division takes some forty: the tile mapping stands
// between a launch and its first load.
struct FastDiv {
    uint32_t d, m;
    void set(int64_t div) {                   // host; 1 <= div < 2^31
        d = (uint32_t)div;
        m = div == 1 ? 0xFFFFFFFFu : (uint32_t)(((uint64_t)1 << 32) / (uint64_t)div);
    }
    __device__ __forceinline__ int div(int n) const {
        const uint32_t q = __umulhi((uint32_t)n, m);
        return (int)(q + ((uint32_t)n - q * d >= d ? 1u : 0u));
    }
};

struct GemmArgs {
    const char* A;            // local first operand, row-major
    const char* B;            // local second operand, row-major
    int64_t lda, ldb;         // bytes per row
    int32_t n;                // columns of the local product
    int32_t ktiles;           // local k in k-tiles of KB bytes of A-row
    int32_t rows_per_shard;   // rows of one shard (M/P; all rows for the scatter along the last dimension)
    int32_t tiles_n;          // tile columns
    // Tile rows.  All-gather: tile row t is the (t mod tiles_m_shard)-th tile of span t / tiles_m_shard of rows_per_span rows
    // (one chunk, or all rows at once: a tile then waits for every chunk of rows_per_chunk rows that it touches).
    int32_t rows_per_span, tiles_m_shard, rows_per_chunk;
    // Reduce-scatter: the rows are cut into the row blocks of the ready flags (blks_per_shard blocks of blk_rows rows in every
    // shard = span, the last one shorter); tile row t covers blks_per_tile consecutive blocks, possibly of several shards, at
    // most BM rows together.  Likewise a tile column covers fcols_per_tile of the flag_cols flag columns of a shard.
    int32_t blk_rows, blks_per_shard, blks_per_tile, n_blks;
    int32_t fcols_per_tile, flag_cols;
    int32_t late_signal;      // the flags are published behind this kernel (a tile is finer than a flag)
    // schedule: n_groups groups of grp_tile_rows tile rows, visited group0, group0+1, ... (mod n_groups);
    // inside a group each XCD (workgroup id mod 8) takes a contiguous run of tiles
    int32_t grp_tile_rows;
    int32_t n_groups;
    int32_t group0;
    int32_t wg_per_group;     // 8 * ceil(grp_tile_rows * tiles_n / 8): tile slots of one group
    int32_t band;             // tile rows swept column-major inside a group (1 = plain row-major)
    // scatter along the last dimension (reduce-scatter modes only; 0 = scatter along rows): destination rank from the
    // tile column, tiles_n = P * tiles_n_shard, rows_per_shard = all rows, one row shard
    int32_t cols_per_shard;   // N/P
    int32_t tiles_n_shard;    // tile columns of one column block
    int32_t rank;
    // reduce-scatter epilogue
    void* partials;           // [P][rows_per_shard][n], fp32 (EPI_RS) or bf16 (EPI_RS16)
    void* outgoing;           // [P][rows_per_shard][n]
    uint32_t* flags_in;       // [P][flags_per_slot]
    uint32_t* flags_out;      // [P][flags_per_slot]
    int64_t slot_elems;       // rows_per_shard * n
    int64_t flags_per_slot;   // tiles_m_shard * tiles_n
    // all-gather epilogue
    uint16_t* C;              // (P*rows_per_shard) x n bf16
    const uint32_t* chunk_flags;
    int32_t n_chunks;         // chunks that A arrives in (chunk q from rank q): blocks of rows, EPI_AGK: column blocks of K/n_chunks
    int32_t act;              // pk_activation applied to the accumulator before the bf16 rounding (all-gather mode)
    const float* scale_a;     // fp8 only
    const float* scale_b;
    uint32_t epoch;
    uint32_t* status;
    uint64_t timeout_ticks;
    uint32_t store_gap;       // ticks between the first stores of neighbouring workgroups of an XCD (0: all at once)
    // stream-K tail: the first sk_dp_slots tile slots are computed whole, one per workgroup and round; the k range of the
    // remaining ones is shared out evenly (sk_dp_slots = all slots: no such tail)
    int32_t sk_dp_slots;
    // divisors of the tile mapping (set_divisors)
    FastDiv by_group, by_band, by_band_rows, by_last_rows, by_span, by_blks, by_chunk_rows, by_shard_cols;
    int32_t last_band;        // index of the last band of a group
    void set_divisors() {     // host, once the sizes above are final
        const int b = band > 0 ? band : 1;
        band = b;
        last_band = (grp_tile_rows + b - 1) / b - 1;
        by_group.set(wg_per_group);
        by_band.set((int64_t)b * tiles_n);
        by_band_rows.set(b);
        by_last_rows.set(grp_tile_rows - last_band * b);
        by_span.set(tiles_m_shard > 0 ? tiles_m_shard : 1);
        by_blks.set(blks_per_shard > 0 ? blks_per_shard : 1);
        by_chunk_rows.set(rows_per_chunk > 0 ? rows_per_chunk : 1);
        by_shard_cols.set(tiles_n_shard > 0 ? tiles_n_shard : 1);
    }
    // A launch may cover a range of the problem's tile rows only: its groups span n_groups * grp_tile_rows rows that start
    // at tile row row_rot and wrap around at all_tile_rows (0 = the groups cover every row, no rotation).
    int32_t row_rot, all_tile_rows;
    char* ws_tiles;           // [gridDim.x] raw accumulator tiles of BM * BN fp32 (a workgroup's piece that does not start a tile)
    uint32_t* ws_flags;       // [gridDim.x] ready flags of those pieces (ws_epoch)
    uint32_t ws_epoch;
};

// kinds of work unit: a whole tile; the piece of a tile's k range that starts it (its owner adds the other pieces and
// runs the epilogue); any other piece (accumulators handed to the owner through ws_tiles)
enum { UNIT_FULL = 0, UNIT_HEAD = 1, UNIT_PART = 2 };

// LDS staging of the epilogue, shared out evenly to the waves: 32 KB, or 16 KB where the ring leaves no more of the 160 KB
template <int BM, int BN, int KB, int NS>
constexpr int epi_stage_bytes() { return NS * (BM + BN) * KB + 32 * 1024 <= 160 * 1024 ? 32 * 1024 : 16 * 1024; }

template <int BM, int BN, int KB, int NS>
constexpr int gemm_lds_bytes() { return NS * (BM + BN) * KB + epi_stage_bytes<BM, BN, KB, NS>(); }

// s_waitcnt immediate for vmcnt(N) lgkmcnt(0) (gfx9 encoding, expcnt left alone)
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }
constexpr int kWaitLgkm0 = waitcnt_vm_lgkm0(63);   // vmcnt as high as it goes: not waited for

// The kernel's arguments, every cache line of them fetched at once.  Left to the compiler they come in at their first uses, one trip to
// memory after the other: the main loop of a short kernel starts that much later (128x128 tiles, 2000 x 1168 x 64 reduce-scatter:
// 4100 cycles from the start to the main loop, 3100 so).
// FETCH_BLOCK: as one block, between the loads of which the compiler can put nothing else (256x256 tiles, 5600 x 2064 x 320 all-gather:
// 17.0 us a call, 16.7 so).  FETCH_FIRST: ahead of every other use of an argument too; each is then loaded where it is used, from the
// scalar cache, and none takes a register (or, with a hundred scalar registers in use, a lane of a vector register) through the main
// loops.  us a call, FETCH_BLOCK / FETCH_FIRST: all-gather, 128x256 tiles,
// 2048 x 4096 x 512 13.15 / 12.79, 256x128, 4176 x 1568 x 13248 150.3 / 148.4; column chunks, 256x256, 11347 x 1144 x 1024 34.4 / 33.3.
// For every kernel below 256x256, over 128 calls drawn evenly over the tiles: 0.5% less on average, beside 0.8% by the LDS addresses of
// dma_load16 and 0.2% by the clocks that only workgroup 0 reads; all three together 2% for 256x128 (1024 x 8192 x 3584 reduce-scatter
// 59.4 / 58.2), 2-6% for the small ones.  The arguments of the tile mapping as one block of 192 bytes per tile, so that they come in
// together, was half a percent slower than one by one: the registers it takes.
// Not with stores on their way through the next main loop (256x256 all-gather, 13176 x 872 x 704 28.3 / 29.6).
enum Fetch { FETCH_PLAIN, FETCH_BLOCK, FETCH_FIRST };
template <Fetch HOW>
__device__ __forceinline__ const GemmArgs& fetched(const GemmArgs& g) {
    typedef const __attribute__((address_space(4))) uint32_t* args_t;
    args_t a = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert((sizeof(GemmArgs) + 63) / 64 == 6, "one word of every line below");
    if constexpr (HOW == FETCH_PLAIN) {
        asm volatile("" : : "s"(a[0]), "s"(a[16]), "s"(a[32]), "s"(a[48]), "s"(a[64]), "s"(a[80]));
        return g;
    } else {
        uint32_t x[6];
        asm volatile("s_load_dword %0, %6, 0x0\n\ts_load_dword %1, %6, 0x40\n\ts_load_dword %2, %6, 0x80\n\ts_load_dword %3, %6, 0xc0\n\t"
                     "s_load_dword %4, %6, 0x100\n\ts_load_dword %5, %6, 0x140\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(x[0]), "=&s"(x[1]), "=&s"(x[2]), "=&s"(x[3]), "=&s"(x[4]), "=&s"(x[5]), "+s"(a));
        asm volatile("" : : "s"(x[0]), "s"(x[1]), "s"(x[2]), "s"(x[3]), "s"(x[4]), "s"(x[5]));
        return HOW == FETCH_FIRST ? *(const GemmArgs*)(const __attribute__((address_space(4))) GemmArgs*)a : g;
    }
}

// BT: the second operand is stored k-contiguous (N x K row-major, the transpose of the K x N matrix): its tile then has
// the layout of the A tile and its fragments come in with the same 16-byte reads, no transposing reads.
// SK: built with the stream-K tail (its code paths cost registers, so launches that share out no tile use SK = false).
// M16: bf16 products by 16x16x32 MFMAs instead of 32x32x16 (the same bits: two of those add up as one of these); tile_m16 has when.
template <int BM, int BN, int WM, int WN, int WK, int KB, int NS, bool FP8, int EPI, bool BT = false, bool SK = false, bool M16 = false>
__global__ __launch_bounds__(64 * WM * WN * WK, 1) void gemm_kernel(const GemmArgs args) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    PK_LDS char* lds = (PK_LDS char*)smem_generic;

    constexpr bool IS_RS = EPI == EPI_RS || EPI == EPI_RS16;
    constexpr int NW = WM * WN * WK;                     // waves per workgroup
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;  // 32x32 blocks of accumulators per wave: TM x TN
    constexpr int MF = M16 ? 16 : 32;                    // rows and columns of one MFMA
    constexpr int FM = BM / WM / MF, FN = BN / WN / MF;  // fragments per wave and k-step
    // MID: the barrier of a k-tile comes in the middle of its last step (see kstep and sync).  fp8, cycles per 128 bytes of k: 128x256
    // 1224 -> 1138 of which 1024 MFMAs (4096 x 3584 x 8192 k-contiguous 90.8 -> 87.0 us a call, 1024 x 3584 x 8192 32.8 -> 32.3; with a
    // row-major operand the clock takes back most: reduce-scatter 808 x 4704 x 2048 21.17 -> 21.03, 8768 x 720 x 2048 28.59 -> 28.42).
    // Not in the fp8 256x256 kernels with a row-major operand: they need 233 registers then, of which 224 leave room for the reduce
    // beside them (16384 x 16384 x 2048: 694 us a call, 649 without)
    constexpr bool MID = M16 || (FP8 && FM * FN >= 4 && (BT || BM * BN < 256 * 256));
    static_assert(!MID || FM * FN >= 4, "the barrier comes behind a quarter of a step's MFMAs, and so behind one at least");
    static_assert(!M16 || (!FP8 && BN % 64 == 0), "16x16x32 MFMAs: bf16, panels of 128 bytes");
    constexpr int A_BYTES = BM * KB, B_BYTES = BN * KB, STAGE = A_BYTES + B_BYTES;
    constexpr int ELEM = FP8 ? 1 : 2;
    constexpr int CPA = KB / 16;                         // 16-byte chunks per A tile row (8 or 4)
    constexpr int B_ROWS = KB / ELEM;                    // k-rows in a B tile
    constexpr int B_ROW_BYTES = BN * ELEM;
    constexpr int PB = BN >= 64 ? 128 : 64;              // bytes per k-row of a panel of the bf16 B tile
    constexpr int CPR = B_ROW_BYTES / 16;                // 16-byte chunks per B tile row
    constexpr int RPI = 64 / CPR;                        // B rows covered by one wave-wide load
    // A single wave per group (WM = WN = 1): the groups share no data, so each takes whole k-tiles of its own (every WK-th)
    // through a ring of its own, and the main loop has no barrier
    constexpr bool PRIV = WM * WN == 1 && WK > 1;
    constexpr int RINGS = PRIV ? WK : 1, NWL = PRIV ? 1 : NW;           // rings; waves that share a k-tile's loads
    constexpr int NA = A_BYTES / 1024 / NWL, NB = B_BYTES / 1024 / NWL; // wave-wide loads per wave per k-tile
    static_assert(!PRIV || (EPI != EPI_AGK && !SK), "rings of their own: not built for k ranges in pieces");
    constexpr int NL = NA + NB;
    constexpr int KST = FP8 || M16 ? KB / 64 : KB / 32;  // MFMA k-steps per k-tile
    constexpr int KS = PRIV ? KST : KST / WK;            // ... of which each of the WK wave groups takes its own share
    // SPREAD: the loads of a k-tile are issued a share per k-step over the KS steps that follow the barrier which frees its stage, not
    // all in the first of them: NW * NL KB at once are more than the L1 takes in the time of that step, and a wave whose load does
    // not go out issues no MFMA behind it.  For tiles of two or four k-steps: fp8 256x128 (cycles per 128-byte k-tile, at once / spread,
    // 1295 / 1213 with the barrier before the last step) and 128x256 with the second operand k-contiguous (1409 / 1166).  Of the bf16
    // 256x128 tiles each group of waves has one step per k-tile, with the loads all in it.  The smaller tiles are bound by what the L1
    // takes in all, two stages leave no time to land, and a 64-byte k-tile has half the loads.
    constexpr bool SPREAD = KS % 2 == 0 && KB == 128 && NS >= 3 && BM * BN >= 256 * 128;
    static_assert(!SPREAD || MID, "built for the order of reads and loads that goes with the barrier in the step");
    constexpr int EPI_OFF = RINGS * NS * STAGE;          // LDS offset of the epilogue staging area
    constexpr int EPI_BYTES = epi_stage_bytes<BM, BN, KB, RINGS * NS>();
    // WK > 1 (and not ROWX): the groups' accumulators are summed at the end of a tile and shared out, OTM x OTN blocks to each wave
    constexpr int OB = TM * TN >= WK ? TM * TN / WK : 1;
    constexpr int OTM = OB >= TN ? OB / TN : 1, OTN = OB >= TN ? TN : OB;
    // ROWX: a tile leaves behind its own main loop, row by row (see there), and not under the first loads of the next one through
    // the staging area: in one wave of four for the 32x32 tile, in up to sixteen passes for others, of which a small call saw every latency.
    // All tiles up to 128x128: 2-10% less a call for 32-row tiles (64 x 3584 x 8192 SiLU 25.0 -> 24.0 us, 44 x 3840 x 1152 fp8 5.40 ->
    // 4.81), 1-4% for 64x64, 1-3% for 128x64 and 128x128.  Of 256x128 and 128x256 where it was the faster one over 140 calls: fp32 slots (256x128 1-2%
    // less, fp8 5%), all-gathers (fp8 and 128x256: 1% less, 3-6% with an activation; not bf16 256x128, which has no register left for it);
    // not bf16 slots (0-6% more: one 16-byte chunk of sums a lane, so bf16 rows leave in 8-byte stores; 16 bytes from two chunks have
    // not been tried) and fp8 128x256 with a row-major operand (2% more).  256x256 tiles run many rounds and keep the stores under the
    // next main loop.
    constexpr bool ROWX = BM * BN <= 128 * 128 || (BM * BN == 256 * 128 && EPI != EPI_RS16 &&
                                                   (FP8 ? BM == 256 || BT : EPI == EPI_RS || BM == 128));
    static_assert(ROWX || (OB * WK == TM * TN && OTM * OTN == OB), "the blocks of a wave's sub-tile are shared out evenly");
    static_assert(ROWX || WK == 1 || (!SK && WM * WN * WK * (WK - 1) * OB * 4096 <= gemm_lds_bytes<BM, BN, KB, RINGS * NS>()), "the exchange fits the LDS");
    static_assert(KB == 64 || KB == 128, "k-tile is 64 or 128 bytes of A row");
    static_assert(KS >= 1, "a k-tile holds at least one MFMA k-step");
    static_assert(CPR >= 2 && RPI >= 1, "tile too narrow");
    static_assert((PRIV || KST % WK == 0) && (KS & (KS - 1)) == 0, "the wave groups share the k-steps of a k-tile evenly");
    static_assert(NW % 2 == 0 && NA * NWL * 1024 == A_BYTES && NB * NWL * 1024 == B_BYTES, "wave grid does not fit the tile");
    static_assert((NS - 1) * NL <= 63, "too many loads in flight for the counter");
    typedef typename std::conditional<FP8, i32x8, bf16x8>::type frag_t;

    constexpr int OUT_ELEM = EPI == EPI_RS ? 4 : 2;
    constexpr int EPI_STORES = OTM * OTN * OUT_ELEM;     // 16-byte-per-lane stores of a wave for a whole tile (1 KB each)
    // The stores of a tile may still be on their way while the next tile's main loop starts (shapes that run many rounds)
    constexpr bool DEFER = BM * BN == 256 * 256 && (M16 || NS >= 4) && !SK && EPI != EPI_AGK && EPI_STORES <= 62;

    // TIGHT: kernels that have to leave 80 registers per lane to a communicator's workgroups (pk.h): 216 of their own at most.  They keep
    // nothing in registers through the main loops that can be computed anew (own_lane, report_late, `fetched`): 220-223 otherwise.  Those
    // with a stream-K tail leave none either way (16640 x 1024 x 4096 296 us a call so, 286 without).
    constexpr bool TIGHT = !IS_RS && !FP8 && !SK && BM * BN >= 256 * 128;
    constexpr Fetch FETCH = SK ? FETCH_PLAIN : BM * BN < 256 * 256 || (TIGHT && EPI == EPI_AGK) ? FETCH_FIRST : TIGHT ? FETCH_BLOCK : FETCH_PLAIN;
    const GemmArgs& g = fetched<FETCH>(args);

    const int tid = threadIdx.x;
    const int l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The lane id for what is done once per tile or less.  Opaque (TIGHT): what the compiler computes from `l` there (the address of the
    // lane's chunk flag, its bit in a mask) it computes ahead of the loop over the tiles and keeps.
    auto own_lane = [&]() -> int {
        int x = l;
        if constexpr (TIGHT) asm volatile("" : "+v"(x));
        return x;
    };
    auto first_thread = [&]() -> bool { return TIGHT ? w == 0 && own_lane() == 0 : tid == 0; };
    auto report_late = [&](uint32_t index, uint32_t phase) {
        uint32_t none = 0, code = PK_ERR_TIMEOUT;
        if constexpr (TIGHT) asm volatile("" : "+v"(none), "+v"(code), "+v"(phase));
        report_timeout(g.status, index, phase, none, code);
    };
    const int wk = w / (WM * WN), wm = (w / WN) % WM, wn = w % WN;
    const int kk0 = PRIV ? 0 : wk * KS;                  // first k-step of this wave's group in every k-tile
    const int wl = PRIV ? 0 : w;                         // this wave among those that share a k-tile's loads
    PK_LDS char* ring = lds + (PRIV ? wk * (NS * STAGE) : 0);
    const int h = l >> 5;

    // A-tile swizzle: LDS chunk position = k-chunk ^ fA(row).
    //   128-byte rows: fA(r) = (r & 7) ^ ((r >> 3) & 1);  64-byte rows: fA(r) = ((r >> 1) & 3) ^ ((r >> 3) & 1)
    // Reads of 16 rows by four chunks (M16) want them without the last term.  Measured on every pattern used: 250 B/clk per compute
    // unit, and 128 for the one form's reads with the other form's swizzle.
    auto fA = [](int r) { return (KB == 128 ? r & 7 : (r >> 1) & 3) ^ (M16 ? 0 : (r >> 3) & 1); };

    // fp8 B tile (rows of B_ROW_BYTES): the 32-byte pieces of a row trade places so that eight k-rows, which 32 lanes of a transposing read
    // cover, lie in different banks (256 B/clk per compute unit; 128 where two of the rows shared banks)
    constexpr int ROWS_256 = CPR <= 16 ? 16 / CPR : 1;   // k-rows in 256 bytes
    auto fB = [](int kr) { return (kr & 7) / ROWS_256 % (CPR / 2); };

    // ---- per-lane LDS fragment addresses (relative to a stage) ----
    // Set anew for every tile, from a lane id that the compiler cannot follow from one tile to the next: kept in registers
    // across the epilogue (and its addresses across the main loop) they would not fit beside the accumulators.
    int fa = 0, hf = 0;
    uint32_t a_row_off = 0, b_off[FN];
    auto set_frag_addresses = [&](int l) {
        fa = fA(l & (MF - 1));                               // fA has a period of 16 rows
        hf = l / MF;
        const int h = l >> 5;
        a_row_off = (uint32_t)(wm * (BM / WM) + (l & (MF - 1))) * KB;
        const int s16 = l & 15, nhalf = (l >> 4) & 1;
        const uint32_t bt_row_off = (uint32_t)(A_BYTES + (wn * (BN / WN) + (l & (MF - 1))) * KB);   // BT: B tile = BN rows of KB bytes
        if constexpr (BT) {
#pragma unroll
            for (int tj = 0; tj < FN; ++tj) b_off[tj] = bt_row_off + (uint32_t)(tj * MF * KB);
        } else if constexpr (M16) {
            // the panels of the branch below; each group of 16 lanes takes eight k-rows of the same 16 columns (one 32-byte piece).  The
            // pieces trade places by bit 1 of the k-row, and the 64-byte halves of a row by its bit 3: 32 lanes then cover 256
            // bytes in as many banks (256 B/clk per compute unit; 128 without the latter)
            const int krow_base = 32 * kk0 + 8 * (l >> 4) + (s16 >> 2);
#pragma unroll
            for (int tj = 0; tj < FN; ++tj) {
                const int c16 = wn * FN + tj;                // 16-column block of the tile
                const int piece = (c16 & 3) ^ ((krow_base >> 1) & 1) ^ (2 * ((krow_base >> 3) & 1));
                b_off[tj] = (uint32_t)(A_BYTES + (c16 >> 2) * (B_ROWS * PB) + krow_base * PB + piece * 32 + (s16 & 3) * 8);
            }
        } else if constexpr (!FP8) {
            // bf16 B tile: panels of 64 columns (128 bytes per k-row, k-rows consecutive);
            // inside a row the two 64-byte halves trade places on k-rows with bit 1 set.  A tile of 32 columns is one panel of
            // 64 bytes per k-row.  Either way the 32 lanes of a transposing read cover 256 bytes in as many banks.
            static_assert(BN % 64 == 0 || BN == 32, "the tile is made of whole panels");
            const int krow_base = 16 * kk0 + 8 * h + (s16 >> 2);
#pragma unroll
            for (int tj = 0; tj < TN; ++tj) {
                const int c32 = wn * TN + tj;                // 32-column block of the tile
                const int panel = c32 >> 1;
                const int piece = BN == 32 ? nhalf : (2 * (c32 & 1) + nhalf) ^ (2 * ((s16 >> 3) & 1));
                b_off[tj] = (uint32_t)(A_BYTES + panel * (B_ROWS * PB) + krow_base * PB + piece * 32 + (s16 & 3) * 8);
            }
        } else {
            const int krow_base = 64 * kk0 + 32 * h + (s16 >> 1);
            const int gsw = fB(s16 >> 1);
#pragma unroll
            for (int tj = 0; tj < TN; ++tj) {
                const int c = wn * (BN / WN / 16) + tj * 2 + nhalf;
                b_off[tj] = (uint32_t)(A_BYTES + krow_base * B_ROW_BYTES + (c ^ (2 * gsw)) * 16 + (s16 & 1) * 8);
            }
        }
    };

    // Fragment reads of k-step kk of the k-tile held in LDS stage `st`, as NU = FN + FM units in the order the
    // MFMAs need them: B fragments first, then A fragments.
    constexpr int NU = FN + FM;
    auto read_unit = [&](PK_LDS char* st, int kk, int u, frag_t (&af)[FM], frag_t (&bfr)[FN]) {
        if constexpr (BT) {
            // both operands: rows of KB bytes, 16-byte chunks XOR-swizzled by row; rows of a fragment differ by multiples of MF
            const uint32_t base = u < FN ? b_off[u] : a_row_off + (uint32_t)((u - FN) * MF * KB);
            if constexpr (!FP8) {
                const bf16x8 v = *(PK_LDS bf16x8*)(st + base + (uint32_t)((((64 / MF * (kk0 + kk) + hf) ^ fa) & (CPA - 1)) * 16));
                if (u < FN) bfr[u] = v;
                else af[u - FN] = v;
            } else {
                i32x4 x0 = *(PK_LDS i32x4*)(st + base + (uint32_t)((((4 * (kk0 + kk) + 2 * hf) ^ fa) & (CPA - 1)) * 16));
                i32x4 x1 = *(PK_LDS i32x4*)(st + base + (uint32_t)((((4 * (kk0 + kk) + 2 * hf + 1) ^ fa) & (CPA - 1)) * 16));
                const i32x8 v = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
                if (u < FN) bfr[u] = v;
                else af[u - FN] = v;
            }
        } else if constexpr (!FP8) {
            if (u < FN) {
                const int tj = u;
                s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (PK_LDS s16x4*)(st + b_off[tj] + (512 / MF * kk) * PB));
                s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (PK_LDS s16x4*)(st + b_off[tj] + (512 / MF * kk + 4) * PB));
                s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                bfr[tj] = __builtin_bit_cast(bf16x8, both);
            } else {
                const int ti = u - FN;
                const uint32_t ao = a_row_off + (uint32_t)((((64 / MF * (kk0 + kk) + hf) ^ fa) & (CPA - 1)) * 16);
                af[ti] = *(PK_LDS bf16x8*)(st + ao + ti * MF * KB);
            }
        } else {
            if (u < FN) {
                const int tj = u;
                i32x2 p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    p[r] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                        (PK_LDS i32x2*)(st + b_off[tj] + (64 * kk + 8 * r) * B_ROW_BYTES));
                i32x4 q0 = __builtin_shufflevector(p[0], p[1], 0, 1, 2, 3);
                i32x4 q1 = __builtin_shufflevector(p[2], p[3], 0, 1, 2, 3);
                bfr[tj] = __builtin_shufflevector(q0, q1, 0, 1, 2, 3, 4, 5, 6, 7);
            } else {
                const int ti = u - FN;
                const uint32_t ao0 = a_row_off + (uint32_t)((((4 * (kk0 + kk) + 2 * hf) ^ fa) & (CPA - 1)) * 16);
                const uint32_t ao1 = a_row_off + (uint32_t)((((4 * (kk0 + kk) + 2 * hf + 1) ^ fa) & (CPA - 1)) * 16);
                i32x4 x0 = *(PK_LDS i32x4*)(st + ao0 + ti * 32 * KB);
                i32x4 x1 = *(PK_LDS i32x4*)(st + ao1 + ti * 32 * KB);
                af[ti] = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    };
    auto load_frags = [&](PK_LDS char* st, int kk, frag_t (&af)[FM], frag_t (&bfr)[FN]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) read_unit(st, kk, u, af, bfr);
    };

    // accumulators, one MFMA's each
    typename std::conditional<M16, f32x4, f32x16>::type acc[FM][FN];
    auto mfma_one = [&](int ti, int tj, const frag_t (&af)[FM], const frag_t (&bfr)[FN]) {
        if constexpr (M16)
            acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[tj], af[ti], acc[ti][tj], 0, 0, 0);
        else if constexpr (!FP8)
            acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[tj], af[ti], acc[ti][tj], 0, 0, 0);
        else
            acc[ti][tj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bfr[tj], af[ti], acc[ti][tj], 0, 0, 0, 0, 0, 0);
    };

    // four of the accumulators of 32x32 block (ti, tj), 0 <= b < 4: consecutive columns of one row, row (l & 31), columns 8b + 4(l / 32)
    // and on; M16: row 16(b / 2) + (l & 15), columns 16(b % 2) + 4(l / 16) and on
    auto quad = [&](int ti, int tj, int b) -> f32x4 {
        if constexpr (M16) return acc[2 * ti + (b >> 1)][2 * tj + (b & 1)];
        else return f32x4{acc[ti][tj][4 * b], acc[ti][tj][4 * b + 1], acc[ti][tj][4 * b + 2], acc[ti][tj][4 * b + 3]};
    };
    auto set_quad = [&](int ti, int tj, int b, f32x4 x) {
        if constexpr (M16) {
            acc[2 * ti + (b >> 1)][2 * tj + (b & 1)] = x;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[ti][tj][4 * b + e] = x[e];
        }
    };

    // tile bookkeeping carried from one iteration to the next (the epilogue of a tile runs one iteration late)
    int p_q = -1, p_blk = 0, p_nblk = 0, p_fcol = 0, p_row0 = 0, p_row_end = 0, p_col0 = 0, p_col_end = 0;
    int p_kind = UNIT_FULL, p_part_lo = 0, p_tile_end = 0;
    bool p_full = false;                                 // ... was stored by exactly EPI_STORES stores of every wave
    bool p_dead = false;                                 // the previous tile was given up (a wait timed out): no signal
    const int slots_total = g.wg_per_group * g.n_groups;
    const int G = g.grp_tile_rows * g.tiles_n;
    float scale = 1.f;
    if constexpr (FP8) scale = g.scale_a[0] * g.scale_b[0];
    // the non-linearity between the two GEMMs of the MLP (paper section 4.1), fused into the all-gather epilogue, in fp32 on
    // the accumulators before the rounding.  x/2 (1 + tanh(u)) is x * sigmoid(2u), so both smooth ones are x / (1 + exp(-y)).
    // exp(-y) = 2^n 2^f with the rounding error of y log2 e carried in f.  |y| <= 87 (all values of the wave): the quotient by a
    // reciprocal and one Newton step, which needs no scaling while 1 + exp(-y) < 2^126; for GELU the step also takes back the
    // rounding of 1 + exp(-y).  Otherwise by a full division, for GELU with y > 1 as x - x exp(-y) / (1 + exp(-y)), so that the errors
    // of the exponential and the quotient enter times exp(-y).  Error in units of 2^-24 of the value: SiLU 3.1 at
    // most (0.61 rms) down to x = -88.7, as with the library functions throughout; GELU 1.7 (0.48 rms) for x > 0 (by tanh() 2.5 and
    // 0.66) and for x < 0 what the rounding of y leaves, 3.6 down to x = -1 and 108 down to -8.
    // us a call, with the library functions throughout / so / with the hardware's exponential and reciprocal as they are (SiLU 4.3
    // units, and zero below -87.3; GELU 3.2): SiLU 64 x 3584 x 8192 26.0 / 25.4 / 25.3, 13884 x 1736 x 512 65.7 / 51.4 / 49.6, 8192 x
    // 3584 x 8192 402 / 388 / 386; GELU 1512 x 1720 x 5120 40.2 / 38.7 / 38.1, 13884 x 1736 x 512 65.5 / 54 / 49.6.
    auto activate8 = [&](f32x4 a, f32x4 b) -> bf16x8 {
#pragma clang fp contract(off)
        float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        bf16x8 o;
        if (g.act == PK_ACT_RELU) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)fmaxf(x[e], 0.f);
            return o;
        }
        constexpr float kC1 = 1.5957691216057308f, kC3 = kC1 * 0.044715f;      // 2 sqrt(2/pi)
        constexpr float kLog2e = 1.44269502f, kLog2eLo = 1.92596303e-8f;
        auto exp_minus = [&](float y) -> float {                               // |y| <= 200
#pragma clang fp contract(off)
            const float p = y * -kLog2e, n = __builtin_rintf(p);
            const float f = (p - n) + __builtin_fmaf(y, -kLog2eLo, __builtin_fmaf(y, -kLog2e, -p));
            return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
        };
        auto smooth = [&](auto silu_c) {
#pragma clang fp contract(off)
            constexpr bool SILU = decltype(silu_c)::value;
            auto arg = [&](float x) { return SILU ? x : x * __builtin_fmaf(kC3 * x, x, kC1); };
            float top = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) top = fmaxf(top, fabsf(x[e]));         // (a NaN passes through either way)
            if (__any(top > (SILU ? 87.f : 9.9f))) {                           // GELU: |y| is 85 at 9.9
                float limit = 200.f;
                if constexpr (TIGHT) asm volatile("" : "+v"(limit));           // (see own_lane)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float y = arg(x[e]), ex = exp_minus(__builtin_amdgcn_fmed3f(y, -limit, limit));
                    const bool rest = !SILU && y > 1.f && ex > 0.f;            // (ex = 0: x may be infinite)
                    const float q = (rest ? x[e] * ex : x[e]) / (1.f + ex);
                    o[e] = (__bf16)(rest ? x[e] - q : q);
                }
                return;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float ex = exp_minus(arg(x[e])), d = 1.f + ex, r = __builtin_amdgcn_rcpf(d), q = x[e] * r;
                float rem = __builtin_fmaf(-d, q, x[e]);
                if constexpr (!SILU) rem = __builtin_fmaf(-((1.f - d) + ex), q, rem);
                o[e] = (__bf16)__builtin_fmaf(rem, r, q);
            }
        };
        if (g.act == PK_ACT_SILU) smooth(std::true_type{});
        else smooth(std::false_type{});
        return o;
    };

    // destination of row r, column c of a tile: dst + r * pitch + c * OUT_ELEM, + own_delta for rows own_row0 .. own_row0 + own_rows - 1.
    // Scatter along rows: shard q's slot lies behind those of the shards before it, so row r of the product is row r of
    // `outgoing` (of `partials` if it is own).  Along the last dimension: the tile goes to rank q.
    auto destination = [&](int q, uint64_t& dst, int64_t& pitch, int64_t& own_delta, int& own_row0, int& own_rows) {
        pitch = (int64_t)g.n * OUT_ELEM;
        own_delta = 0;
        own_row0 = own_rows = 0;
        if constexpr (IS_RS) {
            if (g.cols_per_shard > 0) {
                pitch = (int64_t)g.cols_per_shard * OUT_ELEM;
                dst = (uint64_t)(q == g.rank ? g.partials : g.outgoing) + (int64_t)q * (g.slot_elems - g.cols_per_shard) * OUT_ELEM;
            } else {
                dst = (uint64_t)g.outgoing;
                own_delta = (int64_t)((uint64_t)g.partials - (uint64_t)g.outgoing);
                own_row0 = g.rank * g.rows_per_shard;
                own_rows = g.rows_per_shard;
            }
        } else {
            dst = (uint64_t)g.C;
        }
    };

    auto signal_prev = [&]() {   // paper appendix C `signal` for the tile whose stores have completed
        if (SK && p_kind == UNIT_PART) {
            if (first_thread()) flag_publish(g.ws_flags + blockIdx.x, g.ws_epoch);
        } else if constexpr (IS_RS) {
            if (w == 0 && !p_dead && !g.late_signal) {
                const int nf = min(g.fcols_per_tile, g.flag_cols - p_fcol);
                for (int i = l; i < p_nblk * nf; i += 64) {   // one lane per flag of the tile
                    const int bi = i / nf, blk = p_blk + bi;
                    const int q = g.cols_per_shard > 0 ? p_q : g.by_blks.div(blk);
                    const int fr = g.cols_per_shard > 0 ? blk : blk - q * g.blks_per_shard;
                    uint32_t* flags = (q == g.rank ? g.flags_in : g.flags_out) + (int64_t)q * g.flags_per_slot;
                    flag_publish(flags + (int64_t)fr * g.flag_cols + p_fcol + (i - bi * nf), g.epoch);
                }
            }
        }
    };

    // chunks of A known to have landed (the own one, and those this workgroup has waited for): EPI_AG, EPI_AGK
    // workgroup 0 reports how long it ran, in ticks of the 100 MHz wall clock and in core-clock cycles, and how many of
    // those cycles its main loops took: status[4..7] (the ratio of the first two is the clock the chip held).  The others read no
    // clocks: each reading is waited for (a quarter of a percent of the calls of `fetched`'s comment)
    const bool reports = blockIdx.x == 0;
    uint64_t t_wall0 = 0, t_core0 = 0, t_loops = 0;
    if (reports) {
        t_wall0 = wall_clock64();
        t_core0 = clock64();
    }
    uint32_t n_tiles_done = 0;
    uint64_t seen_chunks = 1ull << (g.rank & 63);
    const uint64_t all_chunks = g.n_chunks >= 64 ? ~0ull : (1ull << g.n_chunks) - 1;
    int v = blockIdx.x;
    // EPI_AG: a slot whose chunk has not landed when it is first visited is put aside (bit i = this workgroup's i-th slot)
    // and taken up again, now waiting, once the workgroup has gone through its other slots: tiles of chunks that are
    // already there never queue behind a late one.  Slots beyond the 64th wait on the spot.
    uint64_t deferred = 0;
    int visit = 0;
    // Stream-K tail (the tile slots from sk_dp_slots on): slot sk_dp_slots + 8*i + x belongs to XCD x = workgroup id
    // mod 8, whose W workgroups share the R * KT k-tiles of its R slots evenly, workgroup j of the XCD taking
    // [sk_bnd(j), sk_bnd(j+1)).  A range is cut at tile boundaries into pieces; cuts closer than SK_MINP k-tiles to a
    // tile boundary are moved onto it.  A workgroup has at most one piece that does not start a tile, its first.
    constexpr int SK_Q = (KS % 2) ? 2 : 1, SK_MINP = 2 * NS;
    const int KT = g.ktiles;
    const int sk_x = blockIdx.x & 7, sk_j = blockIdx.x >> 3, sk_W = gridDim.x >> 3;
    const int sk_R = SK ? (slots_total - g.sk_dp_slots) >> 3 : 0;
    auto sk_bnd = [&](int j) -> int {
        int b = (int)((int64_t)sk_R * KT * j / sk_W);
        b -= b % SK_Q;
        const int r = b % KT;
        if (r < SK_MINP) b -= r;
        else if (KT - r < SK_MINP) b += KT - r;
        return b;
    };
    int sk_c = 0, sk_e = 0;
    if (sk_R > 0) {
        sk_c = sk_bnd(sk_j);
        sk_e = sk_bnd(sk_j + 1);
    }
    for (;;) {
        // ---- which tile (paper listing: interpret_task) ----
        int q = 0, tc = 0, row0 = 0, row_end = 0, col0 = 0, col_end = 0, blk = 0, nblk = 0, fcol = 0;
        int kind = UNIT_FULL, kt0 = 0, nkt = KT, part_lo = 0, tile_end = 0;
        bool have = false;
        for (;;) {
            int slot, slot_index = 64;
            bool may_defer = false;
            if (v < g.sk_dp_slots) {
                slot = v;
                slot_index = visit;
                v += gridDim.x;
                ++visit;
                may_defer = (EPI == EPI_AG) && slot_index < 64;
            } else if ((EPI == EPI_AG) && deferred != 0) {
                slot_index = __builtin_ctzll(deferred);
                deferred &= deferred - 1;
                slot = (int)blockIdx.x + slot_index * (int)gridDim.x;
            } else if (SK && sk_c < sk_e) {
                const int i = sk_c / KT;
                tile_end = (i + 1) * KT;
                const int e = min(sk_e, tile_end);
                slot = g.sk_dp_slots + 8 * i + sk_x;
                kt0 = sk_c - i * KT;
                nkt = e - sk_c;
                kind = kt0 != 0 ? UNIT_PART : (nkt == KT ? UNIT_FULL : UNIT_HEAD);
                part_lo = sk_j + 1;          // the workgroups of this XCD that may hold the other pieces of a tile started here
                sk_c = e;
            } else {
                break;
            }
            const int gi = g.by_group.div(slot);
            const int u = slot - gi * g.wg_per_group;
            const int t = (u & 7) * (g.wg_per_group >> 3) + (u >> 3);
            if (t >= G) continue;
            const int band = g.by_band.div(t);
            const int rem = t - band * g.band * g.tiles_n;
            const bool lastb = band == g.last_band;
            const int rows_in_band = lastb ? (int)g.by_last_rows.d : g.band;
            tc = (lastb ? g.by_last_rows : g.by_band_rows).div(rem);
            const int tr = band * g.band + (rem - tc * rows_in_band);
            int grp = g.group0 + gi;
            if (grp >= g.n_groups) grp -= g.n_groups;
            int tile_row = grp * g.grp_tile_rows + tr;
            if (g.all_tile_rows > 0) {
                tile_row += g.row_rot;
                if (tile_row >= g.all_tile_rows) tile_row -= g.all_tile_rows;
            }
            col0 = tc * BN;
            col_end = g.n;
            if constexpr (IS_RS) {
                blk = tile_row * g.blks_per_tile;
                nblk = min(g.blks_per_tile, g.n_blks - blk);
                auto blk_start = [&](int b) {            // first row of a row block; the one past the last of a span starts the next
                    const int sh = g.by_blks.div(b);
                    return sh * g.rows_per_span + (b - sh * g.blks_per_shard) * g.blk_rows;
                };
                row0 = blk_start(blk);
                row_end = blk_start(blk + nblk);
                fcol = tc * g.fcols_per_tile;
                if (g.cols_per_shard > 0) {              // destination rank from the tile column (one row shard)
                    q = g.by_shard_cols.div(tc);
                    const int tci = tc - q * g.tiles_n_shard;
                    col0 = q * g.cols_per_shard + tci * BN;
                    col_end = (q + 1) * g.cols_per_shard;
                    fcol = tci * g.fcols_per_tile;
                }
            } else {
                const int span = g.by_span.div(tile_row);
                row0 = span * g.rows_per_span + (tile_row - span * g.tiles_m_shard) * BM;
                row_end = (span + 1) * g.rows_per_span;
            }
            have = true;

            // all-gather: the chunks this tile reads must have landed (paper appendix C `wait`)
            if constexpr (EPI == EPI_AG) {
                const int c_lo = g.by_chunk_rows.div(row0), c_hi = g.by_chunk_rows.div(min(row0 + BM, row_end) - 1);
                const uint64_t need = ((2ull << (c_hi & 63)) - (1ull << (c_lo & 63))) & ~seen_chunks;
                if (need) {
                    // wave 0 polls, one lane per chunk; the verdict (0 landed, 1 timed out, 2 not yet: put the slot aside) and the
                    // chunks that have landed go through words of the (idle) epilogue staging area, since the kernel leaves no
                    // LDS for a static variable
                    PK_LDS int* verdict = (PK_LDS int*)(lds + EPI_OFF);
                    PK_LDS uint64_t* landed = (PK_LDS uint64_t*)(lds + EPI_OFF + 8);
                    if (w == 0) {
                        const int c = own_lane();
                        uint64_t there = __ballot(c < g.n_chunks && flag_ready(g.chunk_flags + c, g.epoch));
                        int vd = 0;
                        if (need & ~there) {
                            if (may_defer) {
                                vd = 2;
                            } else {
                                const bool late = ((need >> c) & 1) && !flag_wait(g.chunk_flags + c, g.epoch, g.timeout_ticks);
                                if (late) report_late((uint32_t)c, 1u);
                                if (__ballot(late) != 0) vd = 1;
                                there |= need;
                            }
                        }
                        // Also for chunks that are there at the first look: since this kernel started, another one may have read
                        // what their memory held before (an earlier call on the same buffer, on another stream) into this XCD's L2.
                        // An acquire invalidates that whole L2, with the other workgroups' tiles in it: one wave does it, once for
                        // all the chunks that have landed (128x64 tiles, 256 workgroups that need one chunk each, 2048 x 1024 x
                        // 2048: 1.2 us of a call; done by all waves 11 us).
                        if (vd == 0) acquire_agent();
                        if (c == 0) {
                            *verdict = vd;
                            *landed = there;
                        }
                    }
                    __syncthreads();
                    const int vd_all = *verdict;
                    const uint64_t there_all = *landed;
                    __syncthreads();
                    if (vd_all == 2) {
                        deferred |= 1ull << slot_index;
                        have = false;
                        continue;
                    }
                    if (vd_all == 1) {
                        have = false;                       // drain: this tile's and the later tiles' rows stay untouched
                        v = slots_total;
                        deferred = 0;
                        sk_c = sk_e;
                        break;
                    }
                    seen_chunks |= there_all;
                }
            }
            break;
        }
        int lt = l;                                  // the lane id, opaque: what is computed from it stays within this tile
        asm volatile("" : "+v"(lt));
        uint32_t a_voff[NA], b_voff[NB];           // per-lane byte offsets from the k-tile base pointers
        const char* const a_first = g.A;
        const char* const b_first = g.B;
        const char* a_base = a_first;                // wave-uniform, advanced by one k-tile per issue
        const char* b_base = b_first;
        const int64_t b_step = BT ? (int64_t)KB : (int64_t)B_ROWS * g.ldb;   // bytes from one k-tile of B to the next
        // k-tiles handled between two pipeline fills: all of them, or one column chunk of A at a time (EPI_AGK, own
        // chunk); once this workgroup has seen every chunk, its later tiles run the whole k range in one go
        if (EPI == EPI_AGK && have && p_q < 0 && seen_chunks != all_chunks) {
            // every chunk there already: no pipeline refill per chunk
            PK_LDS int* verdict = (PK_LDS int*)(lds + EPI_OFF);
            if (w == 0) {
                const int c = own_lane();
                const uint64_t missing = __ballot(c < g.n_chunks && !((seen_chunks >> c) & 1) && !flag_ready(g.chunk_flags + c, g.epoch));
                if (!missing) acquire_agent();
                if (c == 0) *verdict = missing != 0;
            }
            __syncthreads();
            const int missing_all = *verdict;
            __syncthreads();
            if (!missing_all) seen_chunks = all_chunks;
        }
        const bool by_chunk = (EPI == EPI_AGK) && seen_chunks != all_chunks;
        const int seg_ktiles = by_chunk ? g.ktiles / g.n_chunks : nkt;
        int until_wrap = 0;                          // EPI_AGK: k-tiles from the next one to issue to the end of the k range
        if constexpr (EPI == EPI_AGK) {
            // the k range is taken in ring order from the own chunk, whether or not the chunks are waited for one by one
            const int first = g.rank * (g.ktiles / g.n_chunks);
            a_base += (int64_t)first * KB;
            b_base += (int64_t)first * b_step;
            until_wrap = g.ktiles - first;
        } else {
            if (PRIV) kt0 = wk;
            a_base += (int64_t)kt0 * KB;             // a piece of a stream-K tile starts at k-tile kt0
            b_base += (int64_t)kt0 * b_step;
        }
        if (have) {
            // per-lane global source addresses of the direct-to-LDS loads.  Wave-wide load j of wave w fills
            // the 1 KB LDS block j*NW + w of the A (or B) tile.
            {
                const int r_in = lt / CPA, cp = lt % CPA;
#pragma unroll
                for (int j = 0; j < NA; ++j) {
                    const int r = (64 / CPA) * (j * NWL + wl) + r_in;
                    const int grow = min(row0 + r, row_end - 1);
                    a_voff[j] = (uint32_t)((int64_t)grow * g.lda + (cp ^ fA(r)) * 16);
                }
            }
            if constexpr (BT) {
                // as the A tile: 1 KB block = 64 / CPA rows (columns of the product) of KB bytes
                const int r_in = lt / CPA, cp = lt % CPA;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int r = (64 / CPA) * (j * NWL + wl) + r_in;
                    const int gcol = min(col0 + r, g.n - 1);        // edge tile: valid memory, never stored
                    b_voff[j] = (uint32_t)((int64_t)gcol * g.ldb + (cp ^ fA(r)) * 16);
                }
            } else if constexpr (!FP8) {
                // 1 KB block bi of the B tile = 1024 / PB k-rows of one panel
                constexpr int KR = 1024 / PB;
                const int kr_in = lt / (PB / 16), cp = lt % (PB / 16);
                const int n_bytes = g.n * 2;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int bi = j * NWL + wl;
                    const int panel = bi / (B_ROWS / KR);
                    const int kr = (bi % (B_ROWS / KR)) * KR + kr_in;
                    const int sw = PB == 64 ? 0 : M16 ? 2 * ((kr >> 1) & 1) + 4 * ((kr >> 3) & 1) : 4 * ((kr >> 1) & 1);
                    int colbyte = (col0 + panel * 64) * 2 + (cp ^ sw) * 16;
                    if (colbyte >= n_bytes) colbyte = n_bytes - 16;   // edge tile: valid memory, never stored
                    b_voff[j] = (uint32_t)((int64_t)kr * g.ldb + colbyte);
                }
            } else {
                const int kr_in = lt / CPR, cp = lt % CPR;
                const int n_bytes = g.n;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int kr = (j * NWL + wl) * RPI + kr_in;
                    int colbyte = col0 + (cp ^ (2 * fB(kr))) * 16;
                    if (colbyte >= n_bytes) colbyte = n_bytes - 16;   // edge tile: valid memory, never stored
                    b_voff[j] = (uint32_t)((int64_t)kr * g.ldb + colbyte);
                }
            }
        }
        // load number i (0 .. NL-1) of this wave for the next k-tile to fetch, into LDS stage `stage`
        const uint32_t lds_wave = (uint32_t)(uintptr_t)ring + wl * 1024;
        // k-tiles of this wave: all, or (a ring of its own) every WK-th from the wk-th on
        const int my_ktiles = PRIV ? (seg_ktiles - wk + WK - 1) / WK : seg_ktiles;
        constexpr int STRIDE = PRIV ? WK : 1;
        // Not for column chunks with 256x256 tiles: addresses kept are 5-8% faster there where k is short (11819 x 784 x 512 25.0 / 26.5 us a
        // call, 3887 x 8128 x 512 46.7 / 50.7) and 1-2% slower where it is long (6046 x 4880 x 14208 691 / 678).  Why is not known: the
        // instructions of the loops and of the epilogue are the same.
        constexpr bool ONE_BASE = EPI != EPI_AGK || BM * BN < 256 * 256;
        auto issue_load_at = [&](uint32_t sa, int imm, int i) {
            const int off = imm + (i < NA ? i : i - NA) * NWL * 1024 + (i < NA ? 0 : A_BYTES);
            const uint32_t at = ONE_BASE ? sa : sa + off;
            if (i < NA) dma_load16(a_base, a_voff[i], at, ONE_BASE ? off : 0);
            else dma_load16(b_base, b_voff[i - NA], at, ONE_BASE ? off : 0);
            if (i == NL - 1) {
                a_base += KB * STRIDE;
                b_base += b_step * STRIDE;
                if (EPI == EPI_AGK && --until_wrap == 0) {
                    a_base = a_first;
                    b_base = b_first;
                    until_wrap = KT;
                }
            }
        };
        auto issue_load = [&](int stage, int i) { issue_load_at(lds_wave + stage * STAGE, 0, i); };
        // all of a k-tile's, into stage number `stage` (a constant)
        auto issue_loads = [&](int stage) {
#pragma unroll
            for (int i = 0; i < NL; ++i) issue_load_at(lds_wave, stage * STAGE, i);
        };
        // the LDS stages are free here: every wave passed the last barrier of the previous tile's loop
        // after its final fragment reads were issued and waited for
        if (have) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (s < my_ktiles) issue_loads(s);
        }

        // ---- epilogue of the previous tile (the storer), under the latency of the loads just issued ----
        bool skip_epilogue = false;
        if (SK && p_q >= 0 && p_kind == UNIT_PART) {
            // hand the raw accumulators to the owner of the tile: register image, 16 bytes per lane, written through
            char* wsb = g.ws_tiles + (int64_t)blockIdx.x * (BM * BN * 4) + (w * (TM * TN * 4)) * 1024 + l * 16;
#pragma unroll
            for (int ti = 0; ti < TM; ++ti)
#pragma unroll
                for (int tj = 0; tj < TN; ++tj)
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        store16_writethrough(wsb + ((ti * TN + tj) * 4 + b) * 1024, __builtin_bit_cast(i32x4, quad(ti, tj, b)));
                    }
            skip_epilogue = true;
        }
        if (SK && p_q >= 0 && p_kind == UNIT_HEAD) {
            // add the other pieces of this tile: those of the following workgroups of this XCD whose ranges start inside it
            for (int jp = p_part_lo; jp < sk_W; ++jp) {
                const int s0 = sk_bnd(jp);
                if (s0 >= p_tile_end) break;
                if (sk_bnd(jp + 1) == s0) continue;              // that workgroup has no work
                const int owner = jp * 8 + sk_x;
                PK_LDS int* verdict = (PK_LDS int*)(lds + EPI_OFF);
                if (first_thread()) {
                    const int late = flag_wait(g.ws_flags + owner, g.ws_epoch, g.timeout_ticks) ? 0 : 1;
                    if (late) report_late((uint32_t)owner, 4u);
                    *verdict = late;
                }
                __syncthreads();
                const int late_all = *verdict;
                __syncthreads();
                if (late_all) {
                    skip_epilogue = true;                           // the tile stays unwritten and unsignalled
                    p_dead = true;
                    break;
                }
                // the piece was written through by another compute unit: read it past this XCD's L2
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.ws_tiles + (int64_t)owner * (BM * BN * 4), 0, BM * BN * 4,
                                                                    0x00020000);
                const uint32_t off0 = (uint32_t)((w * (TM * TN * 4)) * 1024 + l * 16);
                // Eight loads of a wave on their way at all times, each register loaded anew as soon as it has been added: the owner adds its
                // pieces one after the other, 15 or 63 of them where few tiles are left over, and the time from a load to its use
                // is all that counts.  In this order, or the compiler makes some wait for one another (us a call, without / with it: 16640 x
                // 1024 x 4096, 4 tiles left over, 286 / 265, 8704 x 2048 x 4096, 16, 211 / 200, fp8 x 8192 211 / 194; cfg4, 192, 400 / 400).
                constexpr int NQ = TM * TN * 4, AHEAD = 8;
                f32x4 pv[AHEAD];
                auto fetch = [&](int i) {
                    pv[i % AHEAD] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off0, i * 1024, 1 | 2 | 16));
                };
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) fetch(i);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const int ti = i / (TN * 4), tj = i / 4 % TN, b = i % 4;
                    set_quad(ti, tj, b, quad(ti, tj, b) + pv[i % AHEAD]);
                    if (i + AHEAD < NQ) fetch(i + AHEAD);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (DEFER && g.store_gap > 0 && n_tiles_done == 1 && have) {
            // Launches of two rounds and more: every workgroup ends its first tile at the same time, and so every later one, and all
            // compute units then wait for the memory (67 MB of a round of 256x256 fp32 tiles in 9-12 us, of which a compute unit alone
            // needs 2.5) that has nothing to write in between.  The workgroups of an XCD start the first stores one eighth of that time
            // after the other, in eight groups: the last of them are through no later than all were before, and from then on the
            // tiles of the groups end at different times.  A guess at the rate is all it takes, so a delay, not a hand-over.
            const uint64_t t0 = wall_clock64(), gap = (uint64_t)g.store_gap * ((blockIdx.x >> 3) & 7);
            while (wall_clock64() - t0 < gap) __builtin_amdgcn_s_sleep(2);
        }
        if (!ROWX && p_q >= 0 && !skip_epilogue) {
            // lane holds, for each 32x32 block, four quads of columns (see `quad`).  Per pass a slab of
            // ROWS_PASS rows of the wave's part of the tile goes through the wave's private staging area, then out as whole
            // row segments, 16 bytes per lane.  The passes are a loop, not unrolled, around one read-back: a workgroup runs
            // most of this code once per launch, out of a cold instruction cache (unrolled, with the activation inlined per
            // element, it took 5-7 us per 256x128 tile instead of 2).
            constexpr int WCOLS = OTN * 32;                  // columns of the wave's part of the tile
            PK_LDS char* stg = lds + EPI_OFF + w * (EPI_BYTES / NW);
            const int row_w0 = p_row0 + wm * (BM / WM) + (wk * OB / TN) * 32;
            const int col_w0 = p_col0 + wn * (BN / WN) + (wk * OB % TN) * 32;
            uint64_t dst;
            int64_t own_delta, dst_pitch;
            int own_row0, own_rows;
            destination(p_q, dst, dst_pitch, own_delta, own_row0, own_rows);
            // FULL: the tile lies inside the matrix and goes to one buffer, so no store is predicated and a wave issues exactly
            // EPI_STORES of them (fp32 slots: and its rows start on 128-byte lines).
            constexpr bool BIG = BM * BN == 256 * 256 && !SK;    // shapes that run many rounds
            auto emit = [&](auto act_c, auto full_c, auto lines_c) {
                constexpr bool ACT = decltype(act_c)::value;     // staged as fp32, activated on the way out
                constexpr bool FULL = decltype(full_c)::value;
                constexpr bool LINES = decltype(lines_c)::value; // the tile's rows start on 128-byte lines
                constexpr int ST_ELEM = (EPI == EPI_RS || ACT) ? 4 : 2;
                constexpr int STG = EPI_BYTES / NW;
                // columns of a pass: 32 where the slab then has 32 rows, so that all lanes write (fp32 slabs of 16 rows x 64
                // columns keep half of them idle).  Not where rows do not start on 128-byte lines: a row piece then writes parts
                // of lines at both of its ends, and the longer the pieces, the fewer of them (256x256 tiles, 5120 x 4840 x 2304: 177
                // us in 128-byte pieces, 161 in 256; 128x256 tiles, 6000 x 1160 x 320: 32.6 and 29.7; on lines, 4096 x 2048 x 320,
                // 22.7 and 23.1).
                constexpr int CP = (ST_ELEM == 4 && !ACT && STG >= 32 * 32 * 4 && LINES) ? 32 : WCOLS;
                constexpr int ROW_BYTES = CP * ST_ELEM;
                constexpr int ROWS_PASS = STG / ROW_BYTES >= 32 ? 32 : STG / ROW_BYTES;
                static_assert(ROWS_PASS == 32 || ROWS_PASS == 16 || ROWS_PASS == 8 || ROWS_PASS == 4, "staging area too small");
                constexpr int CH = ROW_BYTES / 16;               // 16-byte chunks per staged row
                constexpr int LANES_ROW = CP * OUT_ELEM / 16;    // lanes that cover one row on the way out
                constexpr int ROWS_INSTR = 64 / LANES_ROW;       // rows written by one wave-wide store
                static_assert(ROWS_PASS >= ROWS_INSTR, "a wave-wide store takes at most one pass");
                constexpr int HALVES = 32 / ROWS_PASS, CSLABS = WCOLS / CP, NSLABS = OTM * CSLABS, NPASS = NSLABS * HALVES;
                constexpr int NOUT = ROWS_PASS / ROWS_INSTR;
                static_assert(NPASS * NOUT == EPI_STORES, "stores per wave and tile");
                const int cl = lt % LANES_ROW, rl0 = lt / LANES_ROW;
                // write pass ps: lanes whose row falls in it store their quads; chunk position swizzled by row
                auto write = [&](int ps) {
                    int rl = lt & 31;
                    // opaque, so that neither the addresses below nor the scaled results are computed for all passes at once
                    asm volatile("" : "+v"(rl));
                    float sc = scale;
                    if constexpr (FP8) asm volatile("" : "+v"(sc));
                    const int slab = ps / HALVES;
                    const int row = M16 ? rl & 15 : rl, colq = 4 * (M16 ? lt >> 4 : lt >> 5);
                    if (M16 || ROWS_PASS == 32 || (rl / ROWS_PASS) == ps % HALVES) {
                        auto put = [&](auto slab_c) {
                            constexpr int ti = decltype(slab_c)::value / CSLABS, tj0 = decltype(slab_c)::value % CSLABS * (CP / 32);
                            // one quad of block (ti, tj) into row r, column colw of the slab
                            auto put_quad = [&](int tj, int b, int r, int colw) {
                                const int rs = r % ROWS_PASS;
                                const f32x4 x = quad(ti, tj0 + tj, b);
                                f32x4 val = {x[0] * sc, x[1] * sc, x[2] * sc, x[3] * sc};
                                if constexpr (ST_ELEM == 4) {
                                    const int ch = colw >> 2;                  // 16-byte chunk (4 floats)
                                    *(PK_LDS f32x4*)(stg + rs * ROW_BYTES + ((ch ^ (rs & (CH - 1))) * 16)) = val;
                                } else {
                                    const int ch = colw >> 3;                  // 16-byte chunk (8 bf16)
                                    bf16x4 v16 = {(__bf16)val[0], (__bf16)val[1], (__bf16)val[2], (__bf16)val[3]};
                                    *(PK_LDS bf16x4*)(stg + rs * ROW_BYTES + ((ch ^ (rs & (CH - 1))) * 16) + (colw & 4) * 2) = v16;
                                }
                            };
                            if constexpr (M16) {
#pragma unroll
                                for (int i2 = 0; i2 < 2; ++i2)
                                    if (ROWS_PASS == 32 || (16 * i2 + row) / ROWS_PASS == ps % HALVES) {
#pragma unroll
                                        for (int tj = 0; tj < CP / 32; ++tj)
#pragma unroll
                                            for (int j2 = 0; j2 < 2; ++j2) put_quad(tj, 2 * i2 + j2, 16 * i2 + row, tj * 32 + 16 * j2 + colq);
                                        if (ROWS_PASS < 32) asm volatile("; half %0" : : "n"(i2));
                                    }
                            } else {
#pragma unroll
                                for (int tj = 0; tj < CP / 32; ++tj)
#pragma unroll
                                    for (int b = 0; b < 4; ++b) put_quad(tj, b, row, tj * 32 + 8 * b + colq);
                            }
                            // a different last statement in each case: the compiler would otherwise merge the cases into one
                            // that indexes the accumulators at run time, and move them to scratch memory
                            asm volatile("; slab %0" : : "n"(decltype(slab_c)::value));
                        };
                        static_assert(NSLABS <= 8, "up to eight slabs");
                        if (slab == 0) put(std::integral_constant<int, 0>{});
                        if constexpr (NSLABS > 1) if (slab == 1) put(std::integral_constant<int, 1>{});
                        if constexpr (NSLABS > 2) if (slab == 2) put(std::integral_constant<int, 2>{});
                        if constexpr (NSLABS > 3) if (slab == 3) put(std::integral_constant<int, 3>{});
                        if constexpr (NSLABS > 4) if (slab == 4) put(std::integral_constant<int, 4>{});
                        if constexpr (NSLABS > 5) if (slab == 5) put(std::integral_constant<int, 5>{});
                        if constexpr (NSLABS > 6) if (slab == 6) put(std::integral_constant<int, 6>{});
                        if constexpr (NSLABS > 7) if (slab == 7) put(std::integral_constant<int, 7>{});
                    }
                };
                // read back row-wise: lane -> (row = i*ROWS_INSTR + l / LANES_ROW, chunk = l % LANES_ROW)
                auto get = [&](int i) -> i32x4 {
                    const int rr = i * ROWS_INSTR + rl0;
                    if constexpr (ACT) {
                        const f32x4 x0 = *(PK_LDS f32x4*)(stg + rr * ROW_BYTES + (((2 * cl) ^ (rr & (CH - 1))) * 16));
                        const f32x4 x1 = *(PK_LDS f32x4*)(stg + rr * ROW_BYTES + (((2 * cl + 1) ^ (rr & (CH - 1))) * 16));
                        return __builtin_bit_cast(i32x4, activate8(x0, x1));
                    } else {
                        return *(PK_LDS i32x4*)(stg + rr * ROW_BYTES + ((cl ^ (rr & (CH - 1))) * 16));
                    }
                };
                auto store = [&](int ps, int i, i32x4 val) {
                    const int row = row_w0 + (ps / HALVES / CSLABS) * 32 + (ps % HALVES) * ROWS_PASS + i * ROWS_INSTR + rl0;
                    const int col = col_w0 + (ps / HALVES % CSLABS) * CP + cl * (16 / OUT_ELEM);
                    uint64_t d = dst + (int64_t)row * dst_pitch + (int64_t)col * OUT_ELEM;
                    if constexpr (!FULL) {
                        if (row >= p_row_end || col >= p_col_end) return;
                        if (IS_RS && (uint32_t)(row - own_row0) < (uint32_t)own_rows) d += own_delta;
                    }
                    // reduce-scatter tiles are consumed by another kernel through a flag: write through
                    if constexpr (IS_RS) store16_writethrough((void*)d, val);
                    else store16_stream((void*)d, val);
                };
                if constexpr (ACT) {
#pragma clang loop unroll(disable)
                    for (int ps = 0; ps < NPASS; ++ps) {
                        write(ps);
#pragma clang loop unroll(disable)
                        for (int i = 0; i < NOUT; ++i) store(ps, i, get(i));
                    }
                } else {
                    // All the reads of a pass come before its stores (a read behind the bounds check of its store would be waited
                    // for by itself) and before the next pass is written over them: a wave's LDS operations stay in order.
                    auto pass = [&](int ps) {
                        i32x4 v[NOUT];
#pragma unroll
                        for (int i = 0; i < NOUT; ++i) v[i] = get(i);
                        if (ps + 1 < NPASS) write(ps + 1);
#pragma unroll
                        for (int i = 0; i < NOUT; ++i) asm volatile("" : "+v"(v[i]));
#pragma unroll
                        for (int i = 0; i < NOUT; ++i) store(ps, i, v[i]);
                    };
                    write(0);
                    if constexpr (ST_ELEM == 4 && BM * BN < 256 * 256) {
#pragma clang loop unroll(disable)
                        for (int ps = 0; ps < NPASS; ++ps) pass(ps);
                    } else {
                        // unrolled: in a loop the compiler would round all accumulators ahead of it (bf16); a 256x256 tile's
                        // workgroup runs it once per round
#pragma unroll
                        for (int ps = 0; ps < NPASS; ++ps) pass(ps);
                    }
                }
            };
            using T = std::true_type;
            using F = std::false_type;
            const bool lines = ((dst + (uint64_t)p_col0 * OUT_ELEM | (uint64_t)dst_pitch) & 127) == 0;
            bool full = BIG && p_row0 + BM <= p_row_end && p_col0 + BN <= p_col_end;
            if (EPI == EPI_RS) full = full && lines;
            if constexpr (IS_RS) {
                if (full && own_rows > 0) {                  // all rows own, none, or (not full) some of them
                    const bool all = p_row0 >= own_row0 && p_row_end <= own_row0 + own_rows;
                    const bool none = p_row_end <= own_row0 || p_row0 >= own_row0 + own_rows;
                    if (all) dst += own_delta;
                    full = all || none;
                }
                if (BIG && full) emit(F{}, T{}, T{});
                else if (EPI == EPI_RS && !BIG && lines) emit(F{}, F{}, T{});
                else emit(F{}, F{}, F{});
            } else {
                if (g.act != PK_ACT_NONE) {
                    if (BIG && full) emit(T{}, T{}, T{});
                    else emit(T{}, F{}, F{});
                } else {
                    if (BIG && full) emit(F{}, T{}, T{});
                    else emit(F{}, F{}, F{});
                }
            }
            p_full = full;
        }
        if (!have) break;

#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < (M16 ? 4 : 16); ++e) acc[i][j][e] = 0.f;

        bool stores_pending = false;                     // the previous tile's stores may not be complete yet
        if (p_q < 0 && my_ktiles >= NS) {
            // the workgroup's first tile: its first k-tile has landed, the others follow
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 1) * NL));
            __syncthreads();
        } else if (DEFER && p_full && p_q >= 0 && my_ktiles >= 2 * NS) {
            // the first NS k-tiles have landed: they were issued before the previous tile's EPI_STORES stores, and the counter
            // goes down in order
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(EPI_STORES));
            __syncthreads();
            stores_pending = true;
        } else {
            // the first k-tiles have landed; the previous tile's stores (same counter) are complete as well
            __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
            __syncthreads();
            if (p_q >= 0) signal_prev();
        }

        // ---- main loop ----
        set_frag_addresses(lt);
        frag_t af0[FM], bf0[FN], af1[FM], bf1[FN];
        // One k-tile: KS-1 pipelined k-steps, the barrier, then the last k-step, under which the loads of
        // k-tile kt+NS (LOADS) and the first fragments of k-tile kt+1 are issued (behind the last k-tile: stale bytes that
        // nothing uses).  At the barrier every wave has finished reading k-tile kt's stage, so it can be refilled, and
        // k-tile kt+1 has landed: in the steady state only the loads of the NS-2 k-tiles after it may still be in flight.
        // One k-step: the NM MFMAs on fragment set (ca, cb), with, pinned between them in this order, the reads
        // of the next step's fragments into (na, nb) behind the first half of the MFMAs (they then have the
        // second half of the step to arrive) and the direct-to-LDS loads of a later k-tile behind the second half.
        // MID: `sync` (the waits and the barrier of a k-tile, if this is its step) comes behind MFMA number P, and after it, between the
        // rest of them, the reads and the loads (SPREAD: share `part` of these; none if `part` is negative).
        auto kstep = [&](const frag_t (&ca)[FM], const frag_t (&cb)[FN], frag_t (&na)[FM], frag_t (&nb)[FN],
                         PK_LDS char* rd_stage, int rd_kk, int ld_stage, auto part_c, auto sync_c, auto sync) {
            constexpr int PART = decltype(part_c)::value, PARTS = SPREAD ? KS : 1;
            constexpr bool LOADS = PART >= 0;
            constexpr int X0 = LOADS ? NL * PART / PARTS : 0, XN = LOADS ? NL * (PART + 1) / PARTS - X0 : 0;
            constexpr int NM = FM * FN, H = NM >= 2 ? NM / 2 : 1;
            constexpr int P = MID && decltype(sync_c)::value ? NM / 4 : 0;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const int ti = i / FN;
                mfma_one(ti, MID && (ti & 1) ? FN - 1 - i % FN : i % FN, ca, cb);
                if constexpr (MID) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (P > 0 && i == P - 1) sync();
                    // The next step's fragments, evenly spread: unit y is A row 0, the B fragments, then the other A rows, each of these into the
                    // registers of its predecessor, behind the MFMAs that use that one (8-bit operands do likewise, below).
#pragma unroll
                    for (int y = 0; y < NU; ++y) {
                        const int row = y == 0 ? 0 : y - FN, at = P + (NM - P) * y / NU;
                        const int from = row < 0 ? at : at > row * FN + FN - 1 ? at : row * FN + FN - 1;
                        if (i == from) read_unit(rd_stage, rd_kk, row < 0 || (y > 0 && y <= FN) ? y - 1 : FN + row, na, nb);
                    }
                    if constexpr (LOADS) {
#pragma unroll
                        for (int x = 0; x < XN; ++x)
                            if (i == P + (2 * x + 1) * (NM - P) / (2 * XN)) issue_load(ld_stage, X0 + x);
                    }
                } else {
                    if constexpr (FP8) {
                        // 8-bit fragments are 8 registers each: two full sets next to the accumulators do not fit.  The MFMAs run
                        // row by row (ti-major), so the A fragment of row ti is dead after MFMA ti*FN + FN-1, and the next step's
                        // A fragment of that row is read right behind it, into the same registers; only the B fragments are double.
                        if (i == 0) {
#pragma unroll
                            for (int u = 0; u < FN; ++u) read_unit(rd_stage, rd_kk, u, na, nb);
                        }
                        if (i % FN == FN - 1) read_unit(rd_stage, rd_kk, FN + ti, na, nb);
                    } else {
                        if (i < H) {
#pragma unroll
                            for (int u = (NU * i) / H; u < (NU * (i + 1)) / H; ++u) read_unit(rd_stage, rd_kk, u, na, nb);
                        }
                    }
                    if constexpr (LOADS) {
                        if (i >= NM - H) {
#pragma unroll
                            for (int x = NL * (i - (NM - H)) / H; x < NL * (i - (NM - H) + 1) / H; ++x) issue_load(ld_stage, x);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // LANDED, or kt < landed: k-tile kt+1 is known to be there.  CARRY (SPREAD): the steps before the barrier issue what the k-tile before this one
        // left to them of the loads of k-tile kt-1+NS, so at the barrier all loads up to that k-tile are out, as without SPREAD.
        auto ktile = [&](int kt, int nkt, auto loads_c, auto par_c, auto landed_c, auto carry_c, int landed = 0) {
            constexpr bool LOADS = decltype(loads_c)::value, LANDED = decltype(landed_c)::value, CARRY = decltype(carry_c)::value;
            static_assert(SPREAD || !CARRY, "nothing is left over");
            constexpr int P0 = decltype(par_c)::value;   // fragment set that holds this k-tile's first fragments
            const int sidx = (int)((unsigned)kt % NS);
            PK_LDS char* st = ring + sidx * STAGE;
            PK_LDS char* nx = ring + (sidx + 1 == NS ? 0 : sidx + 1) * STAGE;
            // fragment set `par` is consumed, the other one refilled
            auto step = [&](auto par, PK_LDS char* rd_stage, int rd_kk, auto part_c, auto sync_c, auto sync) {
                const int ld_stage = decltype(part_c)::value <= 0 ? sidx : sidx == 0 ? NS - 1 : sidx - 1;
                if constexpr (decltype(par)::value) kstep(af1, bf1, af0, bf0, rd_stage, rd_kk, ld_stage, part_c, sync_c, sync);
                else kstep(af0, bf0, af1, bf1, rd_stage, rd_kk, ld_stage, part_c, sync_c, sync);
            };
            auto none = [] {};
            using NO = std::false_type;
            if constexpr (KS >= 2) step(std::integral_constant<int, P0>{}, st, 1, std::integral_constant<int, CARRY ? 1 : -1>{}, NO{}, none);
            if constexpr (KS >= 3) step(std::integral_constant<int, P0 ^ 1>{}, st, 2, std::integral_constant<int, CARRY ? 2 : -1>{}, NO{}, none);
            if constexpr (KS >= 4) step(std::integral_constant<int, P0>{}, st, 3, std::integral_constant<int, CARRY ? 3 : -1>{}, NO{}, none);
            static_assert(KS <= 4, "at most four k-steps per k-tile");
            static_assert(NS >= 2, "a ring has two stages or more");
            auto sync = [&] {
                if constexpr (LANDED) {
                    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                } else if constexpr (LOADS) {
                    if constexpr (DEFER && M16) {
                        // (the compiler's form of this branch is ten scalar instructions)
                        asm volatile("s_cmp_lt_i32 %0, %1\n\ts_cbranch_scc1 .Llanded%=\n\ts_waitcnt vmcnt(%2)\n.Llanded%=:"
                                     : : "s"(kt), "s"(landed), "n"((NS - 2) * NL) : "scc", "memory");
                        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                    } else {
                        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 2) * NL));
                    }
                } else {
                    // at the end of the range: of the k-tiles left, only those behind the next one may still be in flight
                    const int left = nkt - kt;
                    auto wait = [&](auto self, auto j_c) -> void {
                        constexpr int J = decltype(j_c)::value;
                        if constexpr (J < 3) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
                        else if (left >= J) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((J - 2) * NL));
                        else self(self, std::integral_constant<int, J - 1>{});
                    };
                    wait(wait, std::integral_constant<int, NS>{});
                }
                if constexpr (PRIV) asm volatile("" : : : "memory");   // the loads have written the LDS behind the compiler's back
                else __syncthreads();
            };
            // MID: in the middle of the step.  What a wave does between its k-tiles (branches, addresses, the last fragments' way from the LDS)
            // then runs beside the other waves' MFMAs; next to the barrier it leaves the matrix cores idle (cycles per 128 bytes of k, 2048
            // of them MFMAs: 256x256 tiles 2680, in the middle 2400; k-contiguous 2434 and 2263; 256x128, 1024 of them, 1400 and 1300)
            if constexpr (!MID) sync();
            step(std::integral_constant<int, (P0 + KS - 1) & 1>{}, nx, 0, std::integral_constant<int, LOADS ? 0 : -1>{}, std::true_type{}, sync);
        };
        // the k-tiles of one pipeline fill: the first NS are in flight or landed, stage 0 holds the first
        auto run_ktiles = [&](int nkt) {
            using T = std::true_type;
            using F = std::false_type;
            using E = std::integral_constant<int, 0>;    // k-tile starts on fragment set 0
            using O = std::integral_constant<int, 1>;    // ... on set 1
            // No argument may still be on its way: scalar loads return out of order with the LDS reads, and the compiler would wait for all
            // reads of a k-step at its first MFMA
            if constexpr (FETCH == FETCH_FIRST) __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
            load_frags(ring, 0, af0, bf0);
            int kt = 0;
            if (DEFER && !M16 && stores_pending) {
                // the first NS k-tiles are there; the barrier of k-tile NS-1 waits for k-tile NS, whose loads were issued behind
                // the previous tile's stores: they are complete then
                static_assert(!DEFER || M16 || (KS == 1 && NS % 2 == 0), "the main loop starts on set 0");
#pragma clang loop unroll(disable)
                for (; kt < NS - 2; kt += 2) {
                    ktile(kt, nkt, T{}, E{}, T{}, F{});
                    ktile(kt + 1, nkt, T{}, O{}, T{}, F{});
                }
                ktile(kt, nkt, T{}, E{}, T{}, F{});
                ktile(kt + 1, nkt, T{}, O{}, F{}, F{});
                kt += 2;
                signal_prev();
            }
            if constexpr (SPREAD) {
                if (nkt > NS) {
                    ktile(0, nkt, T{}, E{}, F{}, F{});
#pragma clang loop unroll(disable)
                    for (kt = 1; kt + NS < nkt; ++kt) ktile(kt, nkt, T{}, E{}, F{}, T{});
                    ktile(kt, nkt, F{}, E{}, F{}, T{});
                    ++kt;
                }
#pragma clang loop unroll(disable)
                for (; kt < nkt; ++kt) ktile(kt, nkt, F{}, E{}, F{}, F{});
            } else if constexpr (KS % 2 == 0) {
                static_assert(!DEFER || M16, "part 0");
#pragma clang loop unroll(disable)
                for (int part = DEFER && M16 && stores_pending ? 0 : 1; part < 2; ++part) {
                    // part 0: the first NS k-tiles with the previous tile's stores on their way (above), in the same code: a copy of it
                    // costs 30 registers
                    const int end = part == 0 ? 2 * NS : nkt, landed = part == 0 ? NS - 1 : 0;
#pragma clang loop unroll(disable)
                    for (; kt + NS < end; ++kt) ktile(kt, nkt, T{}, E{}, F{}, F{}, landed);
                    if (DEFER && M16 && part == 0) signal_prev();
                }
#pragma clang loop unroll(disable)
                for (; kt < nkt; ++kt) ktile(kt, nkt, F{}, E{}, F{}, F{});
            } else {
                // one k-step per k-tile: the starting set alternates, so k-tiles go in pairs.  64-byte k-tiles come in even numbers
                // (the host admits only k ranges of whole 128-byte units); of 128-byte ones there may be one more
                static_assert(KS % 2 == 0 || KB == 128 || NS % 2 == 0, "an even ring, or the pairs would not meet its end");
#pragma clang loop unroll(disable)
                for (; kt + NS + (KB == 128 ? 1 : 0) < nkt; kt += 2) {
                    ktile(kt, nkt, T{}, E{}, F{}, F{});
                    ktile(kt + 1, nkt, T{}, O{}, F{}, F{});
                }
                if (KB == 128 && kt + NS < nkt) {
                    ktile(kt, nkt, T{}, E{}, F{}, F{});
                    ++kt;
#pragma unroll
                    for (int i = 0; i < FM; ++i) af0[i] = af1[i];
#pragma unroll
                    for (int j = 0; j < FN; ++j) bf0[j] = bf1[j];
                }
#pragma clang loop unroll(disable)
                for (; kt + (KB == 128 ? 1 : 0) < nkt; kt += 2) {
                    ktile(kt, nkt, F{}, E{}, F{}, F{});
                    ktile(kt + 1, nkt, F{}, O{}, F{}, F{});
                }
                if (KB == 128 && kt < nkt) ktile(kt, nkt, F{}, E{}, F{}, F{});
            }
        };
        if (reports) t_loops -= clock64();
        const int n_seg = by_chunk ? g.n_chunks : 1;
#pragma clang loop unroll(disable)
        for (int sgm = 0; sgm < n_seg; ++sgm) {
            if (EPI == EPI_AGK && sgm > 0) {
                // another column chunk of A, in ring order from the own one; the first tile that touches a chunk waits for
                // its flag (paper appendix C `wait`), later tiles of this workgroup know it has landed
                int c = g.rank + sgm;
                if (c >= g.n_chunks) c -= g.n_chunks;
                if (!((seen_chunks >> c) & 1)) {
                    PK_LDS int* verdict = (PK_LDS int*)(lds + EPI_OFF);
                    if (first_thread()) {
                        const int late = flag_wait(g.chunk_flags + c, g.epoch, g.timeout_ticks) ? 0 : 1;
                        if (late) report_late((uint32_t)c, 1u);
                        *verdict = late;
                        acquire_agent();
                    }
                    __syncthreads();
                    const int late_all = *verdict;
                    __syncthreads();
                    if (late_all) return;                 // drain: this tile and the rest of this workgroup's stay untouched
                    seen_chunks |= 1ull << c;
                }
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (s < seg_ktiles) issue_loads(s);
                __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
                __syncthreads();
            }
            run_ktiles(my_ktiles);
        }
        if (reports) t_loops += clock64();
        if constexpr (ROWX) {
            // Every wave lays its accumulators down row by row (the ring is free; a wave with a ring of its own has it to itself), and of the
            // WK waves that share a sub-tile each adds up a share of its rows, in group order, and stores them: whole row segments straight
            // out of registers, all waves at work.  Where the LDS does not hold all of them at once, in HP turns.
            constexpr int HP = BM * BN * WK * 4 > 160 * 1024 ? 2 : 1;
            constexpr int SR = BM / WM / HP, SC = BN / WN;   // the sub-tile
            constexpr int CH = SC / 4;                       // 16-byte chunks per row
            constexpr int RI = 64 / CH, NI = SR / WK / RI;   // rows of a wave-wide access, accesses to a wave's share
            static_assert((CH == 8 || CH == 16) && NI * RI * WK == SR && TM % HP == 0, "rows of 128 or 256 bytes, shared out evenly");
            constexpr int PART = PRIV ? NS * STAGE : SR * SC * 4;      // bytes from one wave's sums to the next one's
            static_assert(SR * SC * 4 <= PART && WM * WN * WK * PART <= gemm_lds_bytes<BM, BN, KB, RINGS * NS>(), "the sums fit the LDS");
            PK_LDS char* sums = lds + (PRIV ? 0 : (w % (WM * WN)) * WK * PART);
            const int lane = lt;
            // the chunks of a row trade places so that 16 lanes, of a column or of a row, lie in different banks
            auto at = [](int r, int ch) { return r * (SC * 4) + ((ch ^ (CH == 8 ? (r & 7) ^ ((r >> 3) & 1) : r & 15)) * 16); };
            uint64_t dst;
            int64_t own_delta, dst_pitch;
            int own_row0, own_rows;
            destination(q, dst, dst_pitch, own_delta, own_row0, own_rows);
            const int r0 = wk * (SR / WK) + lane / CH, ch = lane % CH;
            auto sum = [&](int i) -> f32x4 {
                f32x4 x = *(PK_LDS f32x4*)(sums + at(r0 + i * RI, ch));
#pragma unroll
                for (int from = 1; from < WK; ++from) x += *(PK_LDS f32x4*)(sums + from * PART + at(r0 + i * RI, ch));
                if constexpr (FP8) x = f32x4{x[0] * scale, x[1] * scale, x[2] * scale, x[3] * scale};
                return x;
            };
            const int col = col0 + wn * SC + ch * 4;
            int row_w0 = row0 + wm * (BM / WM) + r0;
            auto put = [&](int i, auto x) {
                const int row = row_w0 + i * RI;
                if (row >= row_end || col >= col_end) return;
                uint64_t d = dst + (int64_t)row * dst_pitch + (int64_t)col * OUT_ELEM;
                if (IS_RS && (uint32_t)(row - own_row0) < (uint32_t)own_rows) d += own_delta;
                // reduce-scatter tiles are consumed by another kernel through a flag: write through
                if constexpr (EPI == EPI_RS) store16_writethrough((void*)d, __builtin_bit_cast(i32x4, x));
                else if constexpr (EPI == EPI_RS16) store8_writethrough((void*)d, __builtin_bit_cast(i32x2, x));
                else store8_stream((void*)d, __builtin_bit_cast(i32x2, x));
            };
#pragma unroll
            for (int hp = 0; hp < HP; ++hp) {
                if (hp > 0) {
                    __syncthreads();                         // the sums of the turn before have been read
                    row_w0 += SR;
                }
#pragma unroll
                for (int ti = 0; ti < TM / HP; ++ti)
#pragma unroll
                    for (int tj = 0; tj < TN; ++tj)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int r = 32 * ti + (M16 ? 16 * (b >> 1) + (lane & 15) : lane & 31);
                            const int ch = 8 * tj + (M16 ? 4 * (b & 1) + (lane >> 4) : 2 * b + (lane >> 5));
                            *(PK_LDS f32x4*)(sums + wk * PART + at(r, ch)) = quad(hp * (TM / HP) + ti, tj, b);
                        }
                if constexpr (WK > 1) __syncthreads();
                bool stored = false;
                if constexpr (!IS_RS) {
                    if (g.act != PK_ACT_NONE) {
                        stored = true;
#pragma clang loop unroll(disable)
                        for (int i = 0; i < NI; i += 2) {
                            const f32x4 none = {0.f, 0.f, 0.f, 0.f};
                            const bf16x8 o = activate8(sum(i), NI > 1 ? sum(i + 1) : none);
                            put(i, __builtin_shufflevector(o, o, 0, 1, 2, 3));
                            if constexpr (NI > 1) put(i + 1, __builtin_shufflevector(o, o, 4, 5, 6, 7));
                        }
                    }
                }
                if (!stored) {
                    constexpr int NX = NI < 8 ? NI : 8;          // at once
#pragma clang loop unroll(disable)
                    for (int i0 = 0; i0 < NI; i0 += NX) {
                        f32x4 x[NX];
#pragma unroll
                        for (int i = 0; i < NX; ++i) x[i] = sum(i0 + i);
#pragma unroll
                        for (int i = 0; i < NX; ++i) {
                            if constexpr (EPI == EPI_RS) put(i0 + i, x[i]);
                            else put(i0 + i, bf16x4{(__bf16)x[i][0], (__bf16)x[i][1], (__bf16)x[i][2], (__bf16)x[i][3]});
                        }
                    }
                }
            }
            __syncthreads();                                 // the next tile's loads may fill the ring
        } else if constexpr (WK > 1) {
            // The groups' accumulators are added in group order through the LDS (the ring is free: every wave passed the barrier
            // of the last k-tile after its last fragment reads).  Group r ends up with blocks [r*OB, (r+1)*OB) of the sub-tile,
            // in acc[0..OTM)[0..OTN).
            const int sub = w % (WM * WN), lane = own_lane();
            auto piece = [&](int from, int to, int i) {      // LDS address of block i of those that group `from` hands to group `to`
                return lds + ((((sub * WK + to) * (WK - 1) + (from < to ? from : from - 1)) * OB + i) * 4096) + lane * 16;
            };
#pragma unroll
            for (int gr = 0; gr < WK; ++gr)
                if (wk == gr) {
#pragma unroll
                    for (int bl = 0; bl < TM * TN; ++bl)
                        if (bl / OB != gr) {
                            PK_LDS char* dp = piece(gr, bl / OB, bl % OB);
#pragma unroll
                            for (int b = 0; b < 4; ++b) *(PK_LDS f32x4*)(dp + b * 1024) = quad(bl / TN, bl % TN, b);
                        }
                }
            __syncthreads();
#pragma unroll
            for (int gr = 0; gr < WK; ++gr)
                if (wk == gr) {
#pragma unroll
                    for (int i = 0; i < OB; ++i)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            f32x4 sum;
#pragma unroll
                            for (int from = 0; from < WK; ++from) {
                                const f32x4 x = from == gr ? quad((gr * OB + i) / TN, (gr * OB + i) % TN, b) : *(PK_LDS f32x4*)(piece(from, gr, i) + b * 1024);
                                sum = from == 0 ? x : sum + x;
                            }
                            set_quad(i / OTN, i % OTN, b, sum);
                        }
                }
            __syncthreads();                                 // the next tile's loads may fill the ring
        }

        ++n_tiles_done;
        p_dead = false;
        p_kind = kind;
        p_part_lo = part_lo;
        p_tile_end = tile_end;
        p_q = q;
        p_blk = blk;
        p_nblk = nblk;
        p_fcol = fcol;
        p_row0 = row0;
        p_row_end = row_end;
        p_col0 = col0;
        p_col_end = col_end;
    }

    // the last tile's stores: every wave waits for its write-through stores, then the flag is published
    if (p_q >= 0 && (IS_RS || (SK && p_kind == UNIT_PART))) {
        __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
        __syncthreads();
        signal_prev();
    }
    if (reports && first_thread()) {
        g.status[4] = (uint32_t)(wall_clock64() - t_wall0);
        g.status[5] = (uint32_t)(clock64() - t_core0);
        g.status[6] = (uint32_t)t_loops;
        g.status[7] = n_tiles_done;
    }
}

}  // namespace pk
