// libpk: kernels other than the GEMM, and the C-ABI entry points (see include/pk.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include "pk_device.h"
#include "pk_tiles.h"

namespace pk {

// ------------------------------------------------------------------------------------------------
// Fused reduce of the P partial slots of this rank's shard (paper appendix C `reduce`: load the same
// tile from every device, reduce, store to local memory; section 3.1.3: the owner accumulates the
// tiles that the P ranks produced).  Pure streaming: per 8 output elements a thread issues 2 x P
// independent 16-byte loads, adds in slot order 0..P-1 in fp32, rounds to bf16 and stores 16 bytes.
// One workgroup handles `rows_sub` rows of one flag tile after waiting for that tile's P flags.
// ------------------------------------------------------------------------------------------------
struct ReduceArgs {
    const void* partials;     // [P][rows][n] fp32, or bf16 when the kernel is instantiated with S16
    uint16_t* out;            // rows x n bf16
    uint32_t* flags_in;       // [P][flags_per_slot]
    uint32_t* flags_out;      // late_signal only
    int32_t late_signal;      // the GEMM in front of this kernel left its flags unpublished (its tiles are finer than a flag)
    int32_t P, rows, n;
    int32_t tile_m, tile_n, tiles_n, rows_sub;
    FastDiv by_sub, by_tiles_n, by_cpr, by_cpr_last;   // work items of a flag tile; tile columns; 8-element chunks per tile row
    int64_t slot_elems, flags_per_slot;
    uint32_t epoch;
    uint32_t* status;
    uint64_t timeout_ticks;
    // all-reduce mode (bcast_out != nullptr or ar_flags_in != nullptr): the reduced block also goes to every
    // other rank's slot of bcast_out, and each 8-row block is announced per destination
    uint16_t* bcast_out;      // [P][rows][n] bf16
    uint32_t* ar_flags_in;    // [P][ar_flags_per_slot]; only slot `rank` is written
    uint32_t* ar_flags_out;   // [P][ar_flags_per_slot]
    int64_t ar_flags_per_slot;
    int32_t rank;
    int32_t n_items;          // workgroups that reduce; those behind them wait for the peers' rows (PK_PHASE_WAIT in the same launch)
};

// cache policy of the partial-slot loads: system-coherent (sc0 sc1) and streaming (nt).  The slots are written
// by other workgroups / kernels (write-through) and announced through flags; loading them past this XCD's L2
// makes an acquire fence (a whole-L2 invalidate per workgroup) unnecessary.
constexpr int kCoherentStream = 1 | 2 | 16;

// PK_PHASE_WAIT as part of the reduce's launch, by the last few workgroups of it: a launch of its own takes 2 us on the device (64 x
// 8192 x 28672 over 8 ranks: 21.5 us a call, 19.8 so; 1024 x 8192 x 8192 36.5 and 35.1) and 4 us of host time.  They are dispatched when
// every workgroup that reduces on their XCD is on its way, so those never queue behind them.  Flags that are there at the first look
// are all there is to do; the own rows' need no look, as the launch ends with them.  Otherwise the bound of the wait counts, as with a
// launch of its own, from the end of the own reduce: each of these workgroups looks at all the own flags first.
constexpr int kRowFlags = 4;                                 // flags that a thread looks at
__device__ __forceinline__ void wait_for_rows(const ReduceArgs& r) {
    const int64_t fps = r.ar_flags_per_slot, own = r.rank * fps, n = (r.P - 1) * fps;
    const int64_t stride = (int64_t)(gridDim.x - r.n_items) * 256, first = (int64_t)(blockIdx.x - r.n_items) * 256 + threadIdx.x;
    auto index = [&](int k) { return first + k * stride < own ? first + k * stride : first + k * stride + fps; };
    bool late[kRowFlags], any = false;
#pragma unroll
    for (int k = 0; k < kRowFlags; ++k) {
        late[k] = first + k * stride < n && !flag_ready(r.ar_flags_in + index(k), r.epoch);
        any |= late[k];
    }
    if (!__syncthreads_or(any)) return;
    // A workgroup of the reduce either publishes its flag or reports in `status` that it gave up.  The latter is believed after one bound
    // (`status` may hold an older report), and nothing is waited for longer than the reduce can take with 64 workgroups at a time,
    // those of eight compute units.
    const uint64_t t0 = wall_clock64();
    const uint64_t rounds = (uint64_t)(r.n_items / 64 + 1);
    const uint64_t most = r.timeout_ticks > ~0ull / rounds ? ~0ull : rounds * r.timeout_ticks;
    auto given_up = [&] {
        const uint64_t t = wall_clock64() - t0;
        return t > r.timeout_ticks && (t > most || __hip_atomic_load(r.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
    };
    bool wait = true;
    for (int64_t i = threadIdx.x; i < fps && wait; i += 256)
        while (wait && !flag_ready(r.ar_flags_in + own + i, r.epoch)) {
            __builtin_amdgcn_s_sleep(8);
            wait = !given_up();
        }
    __syncthreads();
    // one bound for all the flags of a thread together
    const uint64_t t1 = wall_clock64();
#pragma unroll
    for (int k = 0; k < kRowFlags; ++k)
        while (late[k] && !flag_ready(r.ar_flags_in + index(k), r.epoch)) {
            __builtin_amdgcn_s_sleep(8);
            if (wall_clock64() - t1 > r.timeout_ticks) {
                if (!flag_ready(r.ar_flags_in + index(k), r.epoch)) report_timeout(r.status, (uint32_t)index(k), 3u);
                break;
            }
        }
}

// PT > 0: compile-time P; PT == 0: runtime P.  S16: the slots hold bf16.  AR: all-reduce mode (the reduced rows are also
// pushed to the other ranks and announced).  NARROW: 4 output elements per thread and pass instead of 8 (one 16-byte load
// per slot in flight: under 48 registers), for launches that run beside a GEMM that leaves few registers or little bandwidth.
template <int PT, bool S16, bool AR, bool NARROW = false>
__global__ __launch_bounds__(256) void reduce_kernel(const ReduceArgs r) {
    const int tid = threadIdx.x;
    const int P = PT > 0 ? PT : r.P;
    if constexpr (AR)
        if ((int)blockIdx.x >= r.n_items) {
            wait_for_rows(r);
            return;
        }
    // All arguments are asked for at once, so that their cache lines come in side by side.  Without this the compiler sinks the loads
    // to where each is used, behind the branches below, and a workgroup waits for the second line only after the flags: gemm_rs of
    // 256x256x512 on 2 ranks 6.36 us -> 6.16, of 16x448x512 on 8 ranks 6.37 -> 6.20 (device time of both kernels, 37 calls of 16 to
    // 9776 rows 0.2 to 0.4 us less each).  In all-reduce mode it gave -0.1 and +0.2 us, so there it is left out.
    if constexpr (!AR)
        asm volatile("" ::"s"(r.partials), "s"(r.out), "s"(r.flags_in), "s"(r.flags_out), "s"(r.late_signal), "s"(r.n), "s"(r.tile_n),
                     "s"(r.by_sub.d), "s"(r.by_cpr.d), "s"(r.by_cpr.m), "s"(r.by_cpr_last.d), "s"(r.by_cpr_last.m), "s"(r.slot_elems),
                     "s"(r.flags_per_slot), "s"(r.rank));
    const int tile = r.by_sub.div(blockIdx.x);
    const int sb = blockIdx.x - tile * r.by_sub.d;
    const int tmi = r.by_tiles_n.div(tile), tc = tile - tmi * r.tiles_n;
    const int row_start = tmi * r.tile_m + sb * r.rows_sub;
    const int row_stop = min(min(row_start + r.rows_sub, (tmi + 1) * r.tile_m), r.rows);
    if (row_start >= row_stop) return;               // below the last row of the shard (never the first work item of a tile)

    // wait (paper appendix C): one lane per source rank polls that rank's flag for this tile.  Every wave polls for itself and
    // decides with a ballot: the instantiations without all-reduce mode use no LDS, not even the word a workgroup-wide vote takes,
    // so that their workgroups fit on a compute unit whose LDS a GEMM workgroup holds whole.
    const int p = tid & 63, own = r.late_signal ? r.rank : -1;
    const uint32_t* flag = r.flags_in + (int64_t)p * r.flags_per_slot + tile;
    const bool mine = (!AR || tid < 64) && p < P && p != own;
    bool late = mine && !flag_ready(flag, r.epoch);
    // `signal` for the tiles of the GEMM in front: it has ended, so everything it wrote (through) is in memory.  Behind the first
    // look, whose answer then does not wait for this store (a wave's memory operations complete in order), and before any waiting.
    if (r.late_signal && sb == 0 && tid < P)
        flag_publish((tid == r.rank ? r.flags_in : r.flags_out) + (int64_t)tid * r.flags_per_slot + tile, r.epoch);
    if (late) {
        late = !flag_wait(flag, r.epoch, r.timeout_ticks);
        if (late && tid < 64) report_timeout(r.status, (uint32_t)tile, 2u);
    }
    if constexpr (AR) {
        if (__syncthreads_or(late)) return;      // the whole workgroup leaves together: it meets at a barrier below
    } else {
        if (__ballot(late) != 0) return;
    }

    constexpr int SLOT_ELEM = S16 ? 2 : 4;
    // one buffer descriptor per slot (a slot stays below 4 GiB, all P together need not)
    const uint32_t slot_bytes = (uint32_t)(r.slot_elems * SLOT_ELEM);
    auto slot = [&](int p) {
        return __builtin_amdgcn_make_buffer_rsrc((char*)r.partials + (int64_t)p * r.slot_elems * SLOT_ELEM, 0, (int)slot_bytes,
                                                 0x00020000);
    };
    const int col0 = tc * r.tile_n;
    const FastDiv by_cpr = tc == r.tiles_n - 1 ? r.by_cpr_last : r.by_cpr;
    const int cpr = by_cpr.d;                                // 8-element chunks per row of this tile
    const int total = (row_stop - row_start) * cpr;
    // bf16 -> fp32 of the 8 values of one 16-byte load, added to (s0, s1)
    auto add16 = [](f32x4& s0, f32x4& s1, i32x4 v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t w = (uint32_t)v[e];
            const float lo = __builtin_bit_cast(float, w << 16), hi = __builtin_bit_cast(float, w & 0xFFFF0000u);
            if (e < 2) {
                s0[2 * e] += lo;
                s0[2 * e + 1] += hi;
            } else {
                s1[2 * e - 4] += lo;
                s1[2 * e - 3] += hi;
            }
        }
    };
    if constexpr (NARROW) {
        static_assert(!NARROW || (!S16 && !AR && PT > 0), "the narrow form is built for fp32 slots, compile-time P, no all-reduce");
        const int cpr4 = cpr * 2;
#pragma clang loop unroll(disable)
        for (int idx = tid; idx < total * 2; idx += 256) {
            const int rr = by_cpr.div(idx >> 1), cc = idx - rr * cpr4;
            const int64_t off = (int64_t)(row_start + rr) * r.n + col0 + cc * 4;
            const uint32_t boff = (uint32_t)(off * 4);
            f32x4 v[PT > 0 ? PT : 1];
#pragma unroll
            for (int p = 0; p < PT; ++p)
                v[p] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff, 0, kCoherentStream));
            f32x4 sum = v[0];
#pragma unroll
            for (int p = 1; p < PT; ++p) sum += v[p];
            bf16x4 o = {(__bf16)sum[0], (__bf16)sum[1], (__bf16)sum[2], (__bf16)sum[3]};
            __builtin_nontemporal_store(o, (bf16x4*)(r.out + off));
        }
        return;
    }
    // (not unrolled: 64 registers at most, so that the kernel fits beside a GEMM workgroup; 48 for bf16 slots)
#pragma clang loop unroll(disable)
    for (int idx = tid; idx < total; idx += 256) {
        const int rr = by_cpr.div(idx), cc = idx - rr * cpr;
        const int64_t off = (int64_t)(row_start + rr) * r.n + col0 + cc * 8;
        const uint32_t boff = (uint32_t)(off * SLOT_ELEM);
        f32x4 s0, s1;
        if constexpr (S16) {
            s0 = f32x4{0.f, 0.f, 0.f, 0.f};
            s1 = s0;
            if constexpr (PT > 0) {
                i32x4 v[PT];
#pragma unroll
                for (int p = 0; p < PT; ++p) v[p] = __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff, 0, kCoherentStream);
#pragma unroll
                for (int p = 0; p < PT; ++p) {
                    // one slot after the other: unpacked all at once they took 76 registers, too many beside the fp8 GEMM
                    __builtin_amdgcn_sched_barrier(0);
                    add16(s0, s1, v[p]);
                }
            } else {
                for (int p = 0; p < P; ++p) add16(s0, s1, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff, 0, kCoherentStream));
            }
        } else if constexpr (PT > 0) {
            f32x4 v0[PT], v1[PT];
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                v0[p] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff, 0, kCoherentStream));
                v1[p] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff + 16, 0, kCoherentStream));
            }
            s0 = v0[0];
            s1 = v1[0];
#pragma unroll
            for (int p = 1; p < PT; ++p) {
                s0 += v0[p];
                s1 += v1[p];
            }
        } else {
            s0 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(0), boff, 0, kCoherentStream));
            s1 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(0), boff + 16, 0, kCoherentStream));
            for (int p = 1; p < P; ++p) {
                s0 += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff, 0, kCoherentStream));
                s1 += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot(p), boff + 16, 0, kCoherentStream));
            }
        }
        bf16x8 o = {(__bf16)s0[0], (__bf16)s0[1], (__bf16)s0[2], (__bf16)s0[3],
                    (__bf16)s1[0], (__bf16)s1[1], (__bf16)s1[2], (__bf16)s1[3]};
        if constexpr (AR) {
            // all-reduce: consumers find these rows through flags, so write through
            const i32x4 ov = __builtin_bit_cast(i32x4, o);
            store16_writethrough(r.out + off, ov);
            for (int q = 0; q < P; ++q)
                if (q != r.rank) store16_writethrough(r.bcast_out + (int64_t)q * r.slot_elems + off, ov);
        } else {
            __builtin_nontemporal_store(o, (bf16x8*)(r.out + off));
        }
    }
    if (AR) {
        // `signal` per destination for this 8-row block: every wave waits for its stores, then one lane per rank
        __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
        __syncthreads();
        if (tid < P) {
            const int64_t b = (int64_t)(row_start / PK_AR_ROWS) * r.tiles_n + tc;
            uint32_t* f = (tid == r.rank ? r.ar_flags_in : r.ar_flags_out) + (int64_t)tid * r.ar_flags_per_slot + b;
            flag_publish(f, r.epoch);
        }
    }
}

// `signal` for a GEMM launched without its reduce phase whose tiles are finer than a flag: one thread per flag.
__global__ __launch_bounds__(256) void signal_kernel(uint32_t* flags_in, uint32_t* flags_out, int P, int rank, int64_t flags_per_slot,
                                                     uint32_t epoch) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= P * flags_per_slot) return;
    flag_publish((i / flags_per_slot == rank ? flags_in : flags_out) + i, epoch);
}

// Completion of the all-reduce on this rank: one thread per flag of ar_flags_in waits (bounded) for the epoch.
__global__ __launch_bounds__(256) void ar_wait_kernel(const uint32_t* flags, int64_t n_flags, uint32_t epoch,
                                                      uint32_t* status, uint64_t timeout_ticks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_flags && !flag_wait(flags + i, epoch, timeout_ticks)) report_timeout(status, (uint32_t)i, 3u);
}

// ------------------------------------------------------------------------------------------------
// Peer emulation (not part of the method): what other ranks' communicator workers would push here.
// ------------------------------------------------------------------------------------------------
struct EmuOrder {
    int32_t n;
    int32_t q[PK_EMU_MAX_ORDER];
};

__device__ __forceinline__ void idle_us(uint32_t us) {
    if (us == 0) return;
    const uint64_t t0 = wall_clock64();
    const uint64_t ticks = (uint64_t)us * kWallClockTicksPerUs;
    while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(16);
}

// Both emulators publish like the GEMM epilogue does: write-through stores, every wave waits for its own stores,
// workgroup barrier, then a relaxed device-scope flag store (no L2 write-back fence per workgroup).
__global__ __launch_bounds__(256) void emu_chunks_kernel(const char* staging, char* A_gathered, int64_t chunk_bytes,
                                                         uint32_t* chunk_flags, uint32_t epoch, EmuOrder ord,
                                                         uint32_t gap_us, uint32_t* counters) {
    const int64_t n16 = chunk_bytes >> 4;
    for (int i = 0; i < ord.n; ++i) {
        const int q = ord.q[i];
        const i32x4* src = (const i32x4*)(staging + (int64_t)q * chunk_bytes);
        i32x4* dst = (i32x4*)(A_gathered + (int64_t)q * chunk_bytes);
        // 8 independent 16-byte loads in flight per thread: few workgroups must still move a chunk quickly
        const int64_t stride = (int64_t)gridDim.x * 256;
        int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
        for (; idx + 7 * stride < n16; idx += 8 * stride) {
            i32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(src + idx + u * stride);
#pragma unroll
            for (int u = 0; u < 8; ++u) store16_writethrough(dst + idx + u * stride, v[u]);
        }
        for (; idx < n16; idx += stride) store16_writethrough(dst + idx, __builtin_nontemporal_load(src + idx));
        __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
        __syncthreads();
        if (threadIdx.x == 0) {
            // the last workgroup to finish its part of the chunk publishes the flag
            uint32_t old = __hip_atomic_fetch_add(counters + i, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (old == gridDim.x - 1) flag_publish(chunk_flags + q, epoch);
        }
        idle_us(gap_us);
    }
}

__global__ __launch_bounds__(256) void emu_partials_kernel(const float* staging, float* partials, uint32_t* flags_in,
                                                           uint32_t epoch, EmuOrder ord, uint32_t gap_us,
                                                           int rows, int n, int tile_m, int tile_n,
                                                           int tiles_m, int tiles_n) {
    const int64_t slot_elems = (int64_t)rows * n;
    const int64_t fps = (int64_t)tiles_m * tiles_n;
    for (int i = 0; i < ord.n; ++i) {
        const int q = ord.q[i];
        for (int tile = blockIdx.x; tile < tiles_m * tiles_n; tile += gridDim.x) {
            const int tmi = tile / tiles_n, tc = tile - tmi * tiles_n;
            const int r0 = tmi * tile_m, r1 = min(r0 + tile_m, rows);
            const int c0 = tc * tile_n, w4 = min(tile_n, n - c0) >> 2;
            const int total = (r1 - r0) * w4;
            for (int idx = threadIdx.x; idx < total; idx += 256) {
                const int rr = idx / w4, cc = idx - rr * w4;
                const int64_t off = (int64_t)q * slot_elems + (int64_t)(r0 + rr) * n + c0 + cc * 4;
                store16_writethrough(partials + off, __builtin_nontemporal_load((const i32x4*)(staging + off)));
            }
            __builtin_amdgcn_s_waitcnt(PK_WAIT_VMCNT0);
            __syncthreads();
            if (threadIdx.x == 0) flag_publish(flags_in + (int64_t)q * fps + tile, epoch);
        }
        idle_us(gap_us);
    }
}

// ------------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------------
struct TileCfg {
    int bm, bn;
};

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// 256 x 256 tiles when they still give every CU a tile, else 128 x 128.
static TileCfg pick_tile(int P, int64_t rows_per_shard, int64_t n) {
    const int64_t big = (int64_t)P * ceil_div(rows_per_shard, 256) * ceil_div(n, 256);
    if (rows_per_shard >= 256 && n >= 256 && big >= 256) return {256, 256};
    return {128, 128};
}

// Tile rows that are swept column by column inside a scheduling group, so that the tiles an XCD works on at the same time
// (`run` consecutive ones in the group's linear order, at most one per compute unit of the XCD) share A and B panels in its L2.
// One group for the whole problem: the block of tiles with the smallest half perimeter (1000 x 8192 x 2752, 256x128 tiles: 43.3
// us with 4 x 8 tiles per XCD, 49.9 us with 1 x 32).  One group per chunk of an all-gather (a chunk's tiles are split 8 ways):
// while a run is no longer than a tile row, plain row-major keeps each XCD on one A panel and on the same B columns in every
// chunk.
static int pick_band(int grp_tile_rows, int tiles_n, int run, int n_groups, int bm, int bn) {
    if (n_groups > 1) return run <= tiles_n ? 1 : (grp_tile_rows < 4 ? grp_tile_rows : 4);
    const int block = run < 32 ? run : 32;
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int b = 1; b <= grp_tile_rows && b <= block; ++b) {
        const int64_t cost = (int64_t)b * bm + ceil_div(block, b) * bn;
        if (cost < best_cost) {
            best_cost = cost;
            best = b;
        }
    }
    return best;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// rs: GEMM + reduce-scatter (K sharded) as opposed to all-gather + GEMM (N sharded); rs_cols: the reduce-scatter is along
// the last dimension (then M need not divide by P, N must); ag_k: the all-gather is along the last dimension of A (K)
static pk_status check_dims(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, bool rs,
                            int64_t* lm, int64_t* ln, int64_t* lk, bool rs_cols = false, bool ag_k = false) {
    if (dt != PK_BF16 && dt != PK_FP8_E4M3) return PK_ERR_DTYPE;
    if (P < 1 || P > PK_EMU_MAX_ORDER || M < 1 || N < 1 || K < 1) return PK_ERR_SHAPE;
    if (M % P && !rs_cols && !ag_k) return PK_ERR_SHAPE;
    if (rs ? (K % P) : (N % P)) return PK_ERR_SHAPE;
    if (rs_cols && (N % P || (N / P) % (dt == PK_FP8_E4M3 ? 16 : 8))) return PK_ERR_SHAPE;
    const int64_t m = M, n = rs ? N : N / P, k = rs ? K / P : K;
    const int kt = dt == PK_FP8_E4M3 ? 128 : 64, nv = dt == PK_FP8_E4M3 ? 16 : 8;
    if (k % kt || n % nv) return PK_ERR_SHAPE;
    if (ag_k && (K % P || (K / P) % kt)) return PK_ERR_SHAPE;   // A arrives in column chunks of whole k-tiles
    if (m > (1 << 30) || n > (1 << 30) || k > (1 << 30)) return PK_ERR_SHAPE;
    // the kernels address each operand, and each partial slot (M*N/P elements, at most 4 bytes each), with 32-bit byte
    // offsets from its base
    if (m * k * 2 >= ((int64_t)1 << 32) || k * n * 2 >= ((int64_t)1 << 32)) return PK_ERR_SHAPE;
    if (rs && m * n / P * 4 >= ((int64_t)1 << 32)) return PK_ERR_SHAPE;
    *lm = m;
    *ln = n;
    *lk = k;
    return PK_OK;
}

// compute units of the current device (cached per device ordinal)
static int num_cus() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        int v = 0;
        n = (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

constexpr size_t kWsFlagBytes = 4096;   // the first bytes of a workspace hold one ready flag per workgroup

static pk_status make_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, bool rs, pk_plan* plan) {
    if (!plan) return PK_ERR_NULL;
    int64_t m, n, k;
    pk_status st = check_dims(P, M, N, K, dt, rs, &m, &n, &k);
    if (st != PK_OK) return st;
    const TileCfg tc = pick_tile(P, M / P, n);
    plan->tile_m = tc.bm;
    plan->tile_n = tc.bn;
    plan->tiles_m = (int32_t)ceil_div(M / P, tc.bm);
    plan->tiles_n = (int32_t)ceil_div(n, tc.bn);
    plan->flags_per_slot = (int64_t)plan->tiles_m * plan->tiles_n;
    plan->local_m = m;
    plan->local_n = n;
    plan->local_k = k;
    plan->ar_flags_per_slot = 0;
    plan->workspace_bytes = (int64_t)kWsFlagBytes + (int64_t)num_cus() * tc.bm * tc.bn * 4;
    return PK_OK;
}

// Last-dimension scatter: the shard is M x N/P, flags cover tiles of that shard.
static pk_status make_plan_cols(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    if (!plan) return PK_ERR_NULL;
    int64_t m, n, k;
    pk_status st = check_dims(P, M, N, K, dt, true, &m, &n, &k, true);
    if (st != PK_OK) return st;
    const int64_t ns = N / P;
    const int64_t big = ceil_div(M, 256) * P * ceil_div(ns, 256);
    const TileCfg tc = (M >= 256 && ns >= 256 && big >= 256) ? TileCfg{256, 256} : TileCfg{128, 128};
    plan->tile_m = tc.bm;
    plan->tile_n = tc.bn;
    plan->tiles_m = (int32_t)ceil_div(M, tc.bm);
    plan->tiles_n = (int32_t)ceil_div(ns, tc.bn);
    plan->flags_per_slot = (int64_t)plan->tiles_m * plan->tiles_n;
    plan->local_m = M;
    plan->local_n = N;
    plan->local_k = k;
    plan->ar_flags_per_slot = 0;
    plan->workspace_bytes = 0;
    return PK_OK;
}

// workgroups of a launch that shares out no tile: one per compute unit left to the GEMM (a multiple of 8, so that
// workgroup id mod 8 stays the XCD), or the fewest that finish in the same number of rounds (448 slots on 256 CUs: 2
// rounds of 224)
static int max_grid(int comm_cus) {      // compute units left to a GEMM, a multiple of 8 (see schedule_grid)
    const int grid = (num_cus() - comm_cus) / 8 * 8;
    return grid < 8 ? 8 : grid;
}
static int schedule_grid(int slots, int comm_cus) {
    const int grid = max_grid(comm_cus);
    const int rounds = (slots + grid - 1) / grid;
    const int even = ((slots + rounds - 1) / rounds + 7) / 8 * 8;
    return even < grid ? even : grid;
}

// Whether a workspace takes a launch of `slots` tile slots to the stream-K tail (where the plan's tile is 256 x 256), and whether
// the given one is too small for it.  Plans with 128 x 128 tiles take no tail: there the choice among all tile shapes fills the
// compute units better than a tail of 128 x 128 tiles did (4096 x 14336 x 4096 over 8 ranks: 60 us against 91 us), and a workspace
// is only checked for its size.
static bool sk_applies(int64_t slots, int grid, int64_t ktiles) {
    return slots > grid && slots % grid != 0 && ktiles >= 16 && grid <= (int)(kWsFlagBytes / 4);
}
static bool sk_too_small(int64_t slots, int grid, int64_t ktiles, int tile, size_t ws_bytes) {
    return sk_applies(slots, grid, ktiles) && ws_bytes < kWsFlagBytes + (size_t)grid * tile * tile * 4;
}

// The time by which the first stores of neighbouring workgroups are set apart (gemm_kernel: `store_gap`), in ticks: an eighth of what
// the stores of a round take at 5.6 TB/s.  Only for the shape that is used for many rounds, 256 x 256, and not where the two rounds
// of a launch are all there is and their stores are short against the rest.  us a call, without / with it: fp32 slots, 4 rounds, 8192 x
// 8192 x 512 148 / 133, x 256 128 / 122, 16 rounds, 16384 x 16384 x 256 446 / 425, 2 rounds, 2048 x 16384 x 512 85 / 79, 16384 x 2048 x
// 4096 243 / 242; bf16 slots, 8192 x 8192 x 512 104 / 98 (fp8 79 / 71); all-gather, 16384 x 4096 x 256 49 / 46, 2 rounds, 4096 x 8192 x
// 256 31 / 28.  Left out: bf16 results in two rounds with a longer k (16384 x 2048 x 4096 212 / 214) or on three quarters of the
// compute units (6144 x 4096 x 512 43.8 / 44.8), and tiles of shards that fill little of them (1600 x 16384 x 512 72.5 / 74.7).
static uint32_t store_gap(int tile, int slots, int grid, int cus, bool full, int out_elem, int ktiles) {
    const int rounds = (slots + grid - 1) / grid;
    if (tile != T256x256 || rounds < 2) return 0;
    if (rounds == 2 && (!full || (out_elem == 2 && (ktiles > 8 || grid * 8 < cus * 7)))) return 0;
    return (uint32_t)((int64_t)grid * 256 * 256 * out_elem * kWallClockTicksPerUs / 8 / 5600000);
}

// Launches a GEMM whose tile space is set up in `a` (m: rows of the whole product): with a workspace (256 x 256 tiles only; the caller
// has checked its size) and a last round that is not full, with the stream-K tail, otherwise whole tiles.
template <int EPI>
static pk_status run_gemm(GemmArgs& a, int64_t m, int tile, int comm_cus, bool fp8, bool bt, void* ws, hipStream_t stream) {
    const int bm = kTileDim[tile].bm, bn = kTileDim[tile].bn;
    const int64_t G = (int64_t)a.grp_tile_rows * a.tiles_n;
    a.wg_per_group = (int32_t)(8 * ceil_div(G, 8));
    a.band = pick_band(a.grp_tile_rows, a.tiles_n, a.wg_per_group / 8, a.n_groups, bm, bn);
    const int slots = a.wg_per_group * a.n_groups;
    const int grid = max_grid(comm_cus);
    const int rem = slots % grid;
    a.sk_dp_slots = slots;
    const int64_t tile_rows = a.all_tile_rows > 0 ? a.all_tile_rows : (int64_t)a.n_groups * a.grp_tile_rows;
    const bool full = m * a.n * 8 >= tile_rows * a.tiles_n * bm * bn * 7;       // the tiles, seven eighths of them
    a.store_gap = EPI == EPI_AGK ? 0 : store_gap(tile, slots, schedule_grid(slots, comm_cus), grid, full, EPI == EPI_RS ? 4 : 2, a.ktiles);
    if (ws && sk_applies(slots, grid, a.ktiles)) {
        // With a workspace every compute unit works to the end: whole rounds of tiles, then the k range of the left-over
        // tiles shared out evenly (448 slots on 256 CUs: 256 whole tiles, then 192 tiles as 256 pieces of 3/4 tile).
        a.sk_dp_slots = slots - rem;
        a.ws_flags = (uint32_t*)ws;
        a.ws_tiles = (char*)ws + kWsFlagBytes;
        if (a.ws_epoch == 0) a.ws_epoch = a.epoch;     // a caller's workspace follows the caller's epochs
        return launch_gemm<EPI>(a, tile, fp8, bt, true, grid, stream);
    }
    return launch_gemm<EPI>(a, tile, fp8, bt, false, schedule_grid(slots, comm_cus), stream);
}

// ------------------------------------------------------------------------------------------------
// Scratch memory of the library itself, for pk_ag_gemm_static (callers that cannot allocate): the workspace of the
// stream-K tail.  Each device that loads the library holds its own copy of the array at its own address.
// ------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PK_STATIC_WS_BYTES];

// address of this device's copy of `scratch` (looked up once per device; the array's name itself is no device address)
static pk_status scratch_of_device(void** out) {
    static std::atomic<void*> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return PK_ERR_HIP;
    void* p = cache[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PK_ERR_HIP;
        cache[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return PK_OK;
}

__global__ __launch_bounds__(1024) void fill_zero_kernel(uint32_t* p, int n) {
    for (int i = threadIdx.x; i < n; i += 1024) p[i] = 0u;
}

static uint64_t timeout_ticks(uint64_t timeout_us) {
    if (timeout_us == 0) timeout_us = 2000000;
    return timeout_us * kWallClockTicksPerUs;
}

// ------------------------------------------------------------------------------------------------
// Measurement aid (not part of the method): register-only MFMA loop.  Each wave runs `iters` rounds of 16
// independent 32x32x16 bf16 MFMAs on operands held in registers, either all 1.0 or random sign + mantissa.
// The chip lowers its clock under data-dependent power: the sustained rate with random operands is the ceiling of a
// GEMM on random data with this MFMA (16x16x32, which the large bf16 tiles use, sustains about 15% more).  One lane also reports wall-clock ticks and core-clock cycles.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void probe_mfma_kernel(int iters, int random_operands, uint64_t* report) {
    const uint64_t w0 = wall_clock64(), c0 = clock64();
    f32x16 acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    bf16x8 a[4], b[4];
    uint32_t x = 1u + threadIdx.x * 2654435761u + blockIdx.x * 40503u;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        s16x8 ra, rb;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x = x * 1664525u + 1013904223u;
            const uint32_t m1 = x >> 16;
            x = x * 1664525u + 1013904223u;
            const uint32_t m2 = x >> 16;
            ra[j] = random_operands ? (short)((m1 & 0x807F) | 0x3C00) : (short)0x3F80;
            rb[j] = random_operands ? (short)((m2 & 0x807F) | 0x3C00) : (short)0x3F80;
        }
        a[f] = __builtin_bit_cast(bf16x8, ra);
        b[f] = __builtin_bit_cast(bf16x8, rb);
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i & 3], b[i >> 2], acc[i], 0, 0, 0);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += acc[i][0];
    if (threadIdx.x == 0 && blockIdx.x == 7) {
        report[0] = wall_clock64() - w0;
        report[1] = clock64() - c0;
    }
    if (sum == 12345.678f) report[2] = 1;   // keeps the loop alive
}

}  // namespace pk


using namespace pk;

// A second stream per device, with the two events that fork it from and join it to the caller's stream: the reduce
// phase of pk_gemm_rs runs on it beside the rest of the GEMM (PK_PHASE_OVERLAP).  Created at the first such call on a
// device and kept until the process ends; default priority.  `lock` serialises the callers' fork/join sequences.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    bool ready = false;
};
static std::mutex side_lock;
static SideStream side_streams[64];

static pk_status side_stream_of_device(SideStream** out) {   // call with side_lock held
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return PK_ERR_HIP;
    SideStream& h = side_streams[dev];
    if (!h.ready) {
        if (hipStreamCreateWithFlags(&h.stream, hipStreamNonBlocking) != hipSuccess) return PK_ERR_HIP;
        if (hipEventCreateWithFlags(&h.fork, hipEventDisableTiming) != hipSuccess) return PK_ERR_HIP;
        if (hipEventCreateWithFlags(&h.join, hipEventDisableTiming) != hipSuccess) return PK_ERR_HIP;
        h.ready = true;
    }
    *out = &h;
    return PK_OK;
}

// How gemm_rs_impl cuts the local product into tiles.
struct RsTiling {
    int tile;             // shape
    bool late;            // finer than a ready flag: the flags are published behind the GEMM
    int blks_per_tile;    // row blocks of the ready flags in a tile row (late: the tile's own rows are one block)
    int fcols_per_tile;   // flag columns in a tile column
};
// false: the shape cannot take this problem that way
static bool rs_tiling(const pk_plan& pl, int tile, bool late, int64_t rows, RsTiling* t) {
    const int bm = kTileDim[tile].bm, bn = kTileDim[tile].bn;
    *t = {tile, late, 1, 1};
    if (late) return true;
    if (bn < pl.tile_n) return false;
    t->fcols_per_tile = bn / pl.tile_n;
    // a shard of one block may be lower than a flag tile: several of them then share a tile
    const int blk = pl.tiles_m == 1 ? (int)rows : pl.tile_m;
    t->blks_per_tile = bm / blk;
    return t->blks_per_tile >= 1;
}
static void rs_tile_space(const pk_plan& pl, const RsTiling& t, int P, int64_t m_all, int64_t slot_cols, int n_blks, bool cols,
                          int* tile_rows, int* tile_cols) {
    const int c = t.late ? tiles_across(slot_cols, kTileDim[t.tile].bn) : (pl.tiles_n + t.fcols_per_tile - 1) / t.fcols_per_tile;
    *tile_rows = t.late ? tiles_across(m_all, kTileDim[t.tile].bm) : (n_blks + t.blks_per_tile - 1) / t.blks_per_tile;
    *tile_cols = cols ? P * c : c;
}

struct AllReduceOut {
    uint16_t* bcast_out;
    uint32_t* ar_flags_in;
    uint32_t* ar_flags_out;
    int64_t ar_flags_per_slot;
    bool wait;                           // the peers' rows are still to be waited for; cleared by a launch that does
};

// Tile rows in the first part of an overlapped GEMM + reduce-scatter: the own block's rows rounded up to whole bands of 4, then as
// many more bands (up to 7) as waste the least of its last round.  0: no second part left, one launch, reduce afterwards.
static int first_part(int own_rows, int all_rows, int tiles_n, int grid) {
    const int band = 4;
    int best = 0;
    double best_waste = 2.0;
    for (int k = 0; k < 8; ++k) {
        const int r1 = (int)ceil_div(own_rows, band) * band + k * band;
        if (r1 >= all_rows) break;
        const int64_t t1 = (int64_t)r1 * tiles_n;
        const double waste = (double)(ceil_div(t1, grid) * grid - t1) / grid + 0.02 * k;
        if (waste < best_waste) {
            best_waste = waste;
            best = r1;
        }
    }
    return best;
}

// Which way a GEMM + reduce-scatter goes: the tiles, and whether the GEMM is cut into two launches with the reduce beside the second.
struct RsRoute {
    RsTiling t;
    int all_rows, tiles_n;    // the tile space of the whole local product
    int own_row, own_rows;    // the tile rows that hold this rank's own blocks
    int first_rows;           // tile rows of the first launch (0: one launch for everything)
    bool overlap;             // two launches
    bool narrow_reduce;       // then the reduce runs in its narrow form
};
static RsRoute rs_route(const pk_plan& pl, int P, int rank, int64_t rows, int64_t slot_cols, bool fp8, bool bt, bool bf16_slots, bool cols,
                        bool do_gemm, bool do_reduce, bool overlap, int grid) {
    const int64_t m_all = cols ? rows : P * rows;
    const int n_blks = cols ? pl.tiles_m : P * pl.tiles_m;       // row blocks of the ready flags
    RsRoute r = {};
    // The tile shape.  A tile covers whole ready flags (several, where it is larger) and signals them itself, or it is finer than
    // a flag and the flags are published behind the GEMM: that only where all tiles run at once (they end together anyway) and
    // costs a kernel of its own if the reduce phase is not part of the call.
    r.t = {pl.tile_m == 256 ? T256x256 : T128x128, false, 1, 1};
    if (do_gemm && pl.tile_m != 256) {
        int64_t best = INT64_MAX;
        for (int id = 0; id < N_TILES; ++id)
            for (int late = 0; late < 2; ++late) {
                RsTiling c;
                if (!rs_tiling(pl, id, late != 0, rows, &c)) continue;
                int tile_rows, tile_cols;
                rs_tile_space(pl, c, P, m_all, slot_cols, n_blks, cols, &tile_rows, &tile_cols);
                const int tiles = tile_rows * tile_cols;
                if (late && (tiles + 7) / 8 * 8 > grid) continue;
                const int64_t cost = tile_cost(id, fp8, bt, false, tiles, (int)(pl.local_k >> (fp8 ? 7 : 6)), grid) + (late && !do_reduce ? 4000 * grid : 0);
                if (cost < best) {
                    best = cost;
                    r.t = c;
                }
            }
    }
    rs_tile_space(pl, r.t, P, m_all, slot_cols, n_blks, cols, &r.all_rows, &r.tiles_n);

    if (r.t.late || ceil_div((int64_t)r.all_rows * r.tiles_n, 8) * 8 <= grid) overlap = false;   // all tiles at once: nothing to run beside
    r.own_row = rank * pl.tiles_m / r.t.blks_per_tile;
    r.own_rows = ((rank + 1) * pl.tiles_m - 1) / r.t.blks_per_tile - r.own_row + 1;
    // Registers per lane that the 256x256 GEMM kernels of this mode leave beside their two waves per SIMD (512 less twice their own, in
    // steps of 8): 64.  A wave of the reduce kernel takes 64 at most, 48 in the forms that run beside fp8: the narrow one for fp32
    // slots and P = 2, 4, 8, else the one for bf16 slots or a run-time P.
    // The narrow form is the faster one beside every GEMM: with twice the loads in flight the reduce takes more bandwidth and clock
    // from it (us a call, narrow / wide: fp8 16384 x 16384 x 2048 676 / 706; bf16, 256x256 tiles, P = 8: 8192 x 8192 x 3584 402 / 407,
    // 16384 x 8192 x 1024 325 / 335, 1600 x 12304 x 128 57.5 / 65.2; P = 4, 8192 x 8192 x 3584 404 / 410; P = 2, x 4096 465 / 466;
    // k-contiguous 3624 x 12472 x 576 152 / 165; 128x256 tiles, 1600 x 10152 x 768 83.2 / 93.1; 256x128, 1896 x 11800 x 1984 144.4 /
    // 148.5; 128x128, P = 2, 15178 x 640 x 4480 108.3 / 109.4).
    r.narrow_reduce = !bf16_slots && (P == 2 || P == 4 || P == 8);
    // Beside fp8 the other forms pay from about 200 MB of slots on (bf16 slots, P = 8: 16384 x 8192 x 2048 288 -> 272 us; 8192 x 8192 x
    // 1024, half the bytes, 102 -> 107 us; 15728 x 1376 x 1152 45 -> 57 us): splitting the GEMM costs about 12 us.  The same line for a
    // k-contiguous second operand (6064 x 2640 x 3328, fp32 slots: 88 -> 95 us; at 128 MB 105 -> 103).
    if (fp8 && (bt || !r.narrow_reduce) && m_all * slot_cols * (bf16_slots ? 2 : 4) < (192 << 20)) overlap = false;
    if (overlap) r.first_rows = first_part(r.own_rows, r.all_rows, r.tiles_n, grid);
    r.overlap = r.first_rows > 0;
    return r;
}

// Whether a workspace may take the call to the stream-K tail.  The tail is for one launch: two launches of a call would share the
// workspace's flags under one epoch, and a tile's owner in the second would take the pieces of the first for its own.  Beside the
// reduce a tail does not pay either (bf16, P = 8, us a call: 8192 x 7168 x 28672 389 without against 457 with it, 8192 x 5120 x 28672
// 285 / 331, 8192 x 7168 x 8192 171 / 219).
static bool rs_takes_tail(const pk_plan& pl, const RsRoute& r, bool bt, bool bf16_slots) {
    return pl.tile_m == 256 && !r.overlap && !bt && !bf16_slots;
}

// GEMM + reduce-scatter; with `ar` the reduce phase also hands the reduced rows to every rank (all-reduce)
static pk_status gemm_rs_impl(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                              const void* A_local, const void* B_local, const float* scale_a, const float* scale_b,
                              void* partials, void* outgoing, uint32_t* flags_in, uint32_t* flags_out,
                              uint32_t epoch, void* out_shard, AllReduceOut* ar, uint32_t phases, int comm_cus,
                              int partial_dt, bool cols, void* ws, size_t ws_bytes, uint32_t* status, uint64_t timeout_us,
                              void* stream, int b_layout = PK_B_ROW_MAJOR) {
    pk_plan pl;
    pk_status st = cols ? make_plan_cols(P, M, N, K, dt, &pl) : make_plan(P, M, N, K, dt, true, &pl);
    if (st != PK_OK) return st;
    if (rank < 0 || rank >= P) return PK_ERR_RANK;
    if (comm_cus < 0 || comm_cus > 4096) return PK_ERR_ARG;
    if (partial_dt != PK_PARTIAL_F32 && partial_dt != PK_PARTIAL_BF16) return PK_ERR_DTYPE;
    if (b_layout != PK_B_ROW_MAJOR && b_layout != PK_B_K_CONTIGUOUS) return PK_ERR_ARG;
    const bool bf16_slots = partial_dt == PK_PARTIAL_BF16;
    const bool bt = b_layout == PK_B_K_CONTIGUOUS;
    if (bt && bf16_slots) return PK_ERR_ARG;
    const bool fp8 = dt == PK_FP8_E4M3;
    const bool do_gemm = phases & PK_PHASE_GEMM, do_reduce = phases & PK_PHASE_REDUCE;
    if (!partials || !flags_in || !status) return PK_ERR_NULL;
    if (do_gemm && (!A_local || !B_local)) return PK_ERR_NULL;
    if (do_gemm && P > 1 && (!outgoing || !flags_out)) return PK_ERR_NULL;
    if (do_reduce && !out_shard) return PK_ERR_NULL;
    if (do_gemm && fp8 && (!scale_a || !scale_b)) return PK_ERR_DTYPE;
    if (!aligned16(A_local) || !aligned16(B_local) || !aligned16(partials) || !aligned16(outgoing) ||
        !aligned16(out_shard))
        return PK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    // one shard (slot): rows x cols.  Scatter along rows: M/P x N; along the last dimension: M x N/P
    const int64_t rows = cols ? M : M / P;
    const int64_t slot_cols = cols ? N / P : N;
    const int64_t m_all = cols ? M : P * rows;
    const int n_blks = cols ? pl.tiles_m : P * pl.tiles_m;      // row blocks of the ready flags
    const int grid = max_grid(comm_cus);

    // Overlapped reduce: the GEMM is launched in two parts, the tile rows of this rank's own block (plus as many of the
    // next ranks' as fill whole rounds) and the rest; the reduce runs on the library's second stream beside the second
    // part: its workgroups use no LDS and few enough registers to sit next to a GEMM workgroup.  It waits for nothing
    // the second part produces, so whichever of the two the hardware places first, both finish.
    bool overlap = (phases & PK_PHASE_OVERLAP) && do_gemm && do_reduce && !ar && !cols && P > 1;
    if (overlap) {
        // a stream that is being captured into a graph takes the second stream along only if that one exists already
        // (it is created by the first eager call with the flag): no stream is created in the middle of a capture
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) return PK_ERR_HIP;
        if (cap != hipStreamCaptureStatusNone) {
            std::lock_guard<std::mutex> guard(side_lock);
            int dev = 0;
            if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return PK_ERR_HIP;
            if (!side_streams[dev].ready) overlap = false;
        }
    }
    const RsRoute rt = rs_route(pl, P, rank, rows, slot_cols, fp8, bt, bf16_slots, cols, do_gemm, do_reduce, overlap, grid);
    const RsTiling& t = rt.t;
    const int all_rows = rt.all_rows, tiles_n_all = rt.tiles_n, own_row = rt.own_row, first_rows = rt.first_rows;
    if (do_gemm && ws && !bt && !bf16_slots) {
        // the size of a workspace, checked over the launches of the plan's tiles, whether or not these take the tail
        const bool parts = pl.tile_m == 256 ? rt.overlap : overlap;
        const int plan_rows = P * pl.tiles_m, kt = (int)(pl.local_k / (fp8 ? 128 : 64));
        const int first = parts ? first_part(pl.tiles_m, plan_rows, pl.tiles_n, grid) : 0;
        for (int n_rows : {first, plan_rows - first})
            if (sk_too_small(ceil_div((int64_t)n_rows * pl.tiles_n, 8) * 8, grid, kt, pl.tile_m, ws_bytes)) return PK_ERR_ARG;
    }
    overlap = rt.overlap;
    if (!rs_takes_tail(pl, rt, bt, bf16_slots)) ws = nullptr;

    GemmArgs a = {};
    // one launch over `n_rows` tile rows that start at tile row `row0` (wrapping around at all_rows)
    auto gemm = [&](int row0, int n_rows) {
        a.grp_tile_rows = n_rows;
        a.row_rot = row0;
        a.all_tile_rows = (row0 == 0 && n_rows == all_rows) ? 0 : all_rows;
        return bf16_slots ? run_gemm<EPI_RS16>(a, m_all, t.tile, comm_cus, fp8, false, nullptr, s)
                          : run_gemm<EPI_RS>(a, m_all, t.tile, comm_cus, fp8, bt, ws, s);
    };
    if (do_gemm) {
        const int elem = fp8 ? 1 : 2;
        a.A = (const char*)A_local;
        a.B = (const char*)B_local;
        a.lda = pl.local_k * elem;
        a.ldb = (bt ? pl.local_k : pl.local_n) * elem;
        a.n = (int32_t)pl.local_n;
        a.ktiles = (int32_t)(pl.local_k / (fp8 ? 128 : 64));
        a.rows_per_shard = (int32_t)rows;
        a.tiles_n = tiles_n_all;
        a.cols_per_shard = cols ? (int32_t)slot_cols : 0;
        a.tiles_n_shard = cols ? tiles_n_all / P : 0;
        a.late_signal = t.late;
        a.blks_per_tile = t.blks_per_tile;
        if (t.late) {                        // the tiles ignore the flags' blocks: blocks of their own height over all rows
            a.blk_rows = kTileDim[t.tile].bm;
            a.n_blks = a.blks_per_shard = all_rows;
            a.rows_per_span = (int32_t)m_all;
        } else {
            a.blk_rows = pl.tile_m;
            a.blks_per_shard = pl.tiles_m;
            a.n_blks = n_blks;
            a.rows_per_span = (int32_t)rows;
            a.fcols_per_tile = t.fcols_per_tile;
            a.flag_cols = pl.tiles_n;
        }
        a.n_groups = 1;
        a.group0 = 0;
        a.rank = rank;
        a.partials = partials;
        a.outgoing = outgoing;
        a.flags_in = flags_in;
        a.flags_out = flags_out;
        a.slot_elems = rows * slot_cols;
        a.flags_per_slot = pl.flags_per_slot;
        a.scale_a = scale_a;
        a.scale_b = scale_b;
        a.epoch = epoch;
        a.status = status;
        a.timeout_ticks = timeout_ticks(timeout_us);
        st = overlap ? gemm(own_row, first_rows) : gemm(0, all_rows);
        if (st != PK_OK) return st;
        if (t.late && !do_reduce) {
            hipLaunchKernelGGL(signal_kernel, dim3((unsigned)ceil_div(P * pl.flags_per_slot, 256)), dim3(256), 0, s, flags_in, flags_out,
                               P, rank, pl.flags_per_slot, epoch);
            if (hipGetLastError() != hipSuccess) return PK_ERR_HIP;
        }
    }
    std::unique_lock<std::mutex> side_guard(side_lock, std::defer_lock);
    SideStream* side = nullptr;
    hipStream_t reduce_stream = s;
    if (overlap) {
        side_guard.lock();
        st = side_stream_of_device(&side);
        if (st != PK_OK) return st;
        if (hipEventRecord(side->fork, s) != hipSuccess || hipStreamWaitEvent(side->stream, side->fork, 0) != hipSuccess)
            return PK_ERR_HIP;
        reduce_stream = side->stream;
        // the rest of the GEMM is enqueued before the reduce, so that it is first in line for the compute units
        st = gemm((own_row + first_rows) % all_rows, all_rows - first_rows);
        if (st != PK_OK) return st;
    }
    if (do_reduce) {
        ReduceArgs r = {};
        r.partials = partials;
        r.out = (uint16_t*)out_shard;
        r.flags_in = flags_in;
        r.flags_out = flags_out;
        r.late_signal = do_gemm && t.late;
        r.P = P;
        r.rows = (int32_t)rows;
        r.n = (int32_t)slot_cols;
        r.tile_m = pl.tile_m;
        r.tile_n = pl.tile_n;
        r.tiles_n = pl.tiles_n;
        r.rows_sub = 8;                       // 8 rows x tile_n columns x P slots per work item
        // work items of a flag tile; a shard lower than a flag tile has fewer (a decode step's 8 rows: one instead of 16)
        const int sub = (int)ceil_div(pl.tiles_m == 1 ? rows : pl.tile_m, r.rows_sub);
        r.by_sub.set(sub);
        r.by_tiles_n.set(pl.tiles_n);
        r.by_cpr.set(pl.tile_n / 8);
        r.by_cpr_last.set((slot_cols - (int64_t)(pl.tiles_n - 1) * pl.tile_n) / 8);
        r.slot_elems = rows * slot_cols;
        r.flags_per_slot = pl.flags_per_slot;
        r.epoch = epoch;
        r.status = status;
        r.timeout_ticks = timeout_ticks(timeout_us);
        r.rank = rank;
        if (ar) {
            r.bcast_out = ar->bcast_out;
            r.ar_flags_in = ar->ar_flags_in;
            r.ar_flags_out = ar->ar_flags_out;
            r.ar_flags_per_slot = ar->ar_flags_per_slot;
        }
        int grid = (int)(pl.flags_per_slot * sub);         // one workgroup per work item
        r.n_items = grid;
        if (ar && ar->wait) {
            // up to eight more that wait for the peers' rows (wait_for_rows); a call with more flags than these look at takes several
            // times as long and a launch of its own for the wait
            const int64_t n = (P - 1) * ar->ar_flags_per_slot;
            if (n <= 8 * 256 * kRowFlags) {
                grid += (int)std::min<int64_t>(8, ceil_div(n, 256));
                ar->wait = false;
            }
        }
        hipStream_t s = reduce_stream;
        auto launch = [&](auto s16, auto armode) {
            constexpr bool S16 = decltype(s16)::value, AR = decltype(armode)::value;
            switch (P) {
                case 1: hipLaunchKernelGGL((reduce_kernel<1, S16, AR>), dim3(grid), dim3(256), 0, s, r); break;
                case 2: hipLaunchKernelGGL((reduce_kernel<2, S16, AR>), dim3(grid), dim3(256), 0, s, r); break;
                case 4: hipLaunchKernelGGL((reduce_kernel<4, S16, AR>), dim3(grid), dim3(256), 0, s, r); break;
                case 8: hipLaunchKernelGGL((reduce_kernel<8, S16, AR>), dim3(grid), dim3(256), 0, s, r); break;
                default: hipLaunchKernelGGL((reduce_kernel<0, S16, AR>), dim3(grid), dim3(256), 0, s, r); break;
            }
        };
        const bool ar_mode = r.ar_flags_in != nullptr;
        if (overlap && rt.narrow_reduce) {
            switch (P) {
                case 2: hipLaunchKernelGGL((reduce_kernel<2, false, false, true>), dim3(grid), dim3(256), 0, s, r); break;
                case 4: hipLaunchKernelGGL((reduce_kernel<4, false, false, true>), dim3(grid), dim3(256), 0, s, r); break;
                default: hipLaunchKernelGGL((reduce_kernel<8, false, false, true>), dim3(grid), dim3(256), 0, s, r); break;
            }
        } else if (bf16_slots) ar_mode ? launch(std::true_type{}, std::true_type{}) : launch(std::true_type{}, std::false_type{});
        else ar_mode ? launch(std::false_type{}, std::true_type{}) : launch(std::false_type{}, std::false_type{});
        if (hipGetLastError() != hipSuccess) return PK_ERR_HIP;
    }
    if (overlap) {
        if (hipEventRecord(side->join, side->stream) != hipSuccess || hipStreamWaitEvent(s, side->join, 0) != hipSuccess)
            return PK_ERR_HIP;
    }
    return PK_OK;
}

static pk_status make_plan_ag_k(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    if (!plan) return PK_ERR_NULL;
    int64_t m, n, k;
    pk_status st = check_dims(P, M, N, K, dt, false, &m, &n, &k, false, true);
    if (st != PK_OK) return st;
    const TileCfg tc = pick_tile(1, M, n);
    plan->tile_m = tc.bm;
    plan->tile_n = tc.bn;
    plan->tiles_m = (int32_t)ceil_div(M, tc.bm);
    plan->tiles_n = (int32_t)ceil_div(n, tc.bn);
    plan->flags_per_slot = (int64_t)plan->tiles_m * plan->tiles_n;
    plan->local_m = m;
    plan->local_n = n;
    plan->local_k = k;
    plan->ar_flags_per_slot = 0;
    plan->workspace_bytes = 0;
    return PK_OK;
}

// Which way an all-gather + GEMM goes.
struct AgRoute {
    int tile;
    bool one_span;            // tile rows over all rows instead of chunk by chunk
    bool sk;                  // with the stream-K tail
};
static int64_t ag_plan_slots(const pk_plan& pl, int P) { return ((int64_t)pl.tiles_m * pl.tiles_n + 7) / 8 * 8 * P; }
static AgRoute ag_route(const pk_plan& pl, int P, int64_t M, bool fp8, bool bt, bool k_chunks, bool ws, int grid) {
    const int ktiles = (int)(pl.local_k / (fp8 ? 128 : 64));
    AgRoute r = {T256x256, k_chunks, ws && !k_chunks && pl.tile_m == 256 && sk_applies(ag_plan_slots(pl, P), grid, ktiles)};
    if (r.sk) return r;
    // The tile shape, and how tile rows and row chunks go together.  Where all tiles run at once, or a chunk is lower than a
    // tile: tile rows over all rows, from the one that holds the own chunk on; a tile waits for every chunk it touches.
    // Otherwise one scheduling group per chunk, visited from the own one.  Column chunks: every tile needs every chunk.
    const int64_t chunk_rows = M / P;
    auto tiles_of = [&](int id, bool* one_span) -> int {
        const int bm = kTileDim[id].bm;
        const int all = tiles_across(M, bm), tn = tiles_across(pl.local_n, kTileDim[id].bn);
        *one_span = k_chunks || P == 1 || chunk_rows < bm || (all * tn + 7) / 8 * 8 <= grid;
        return (*one_span ? all : P * tiles_across(chunk_rows, bm)) * tn;
    };
    int64_t best = INT64_MAX;
    for (int id = 0; id < (k_chunks ? T32x64 : N_TILES); ++id) {
        bool span;
        int64_t cost = tile_cost(id, fp8, bt, !k_chunks, tiles_of(id, &span), ktiles, grid);
        // Many rounds of fp8 tiles run at a lower clock than those the estimate was fitted to, and the largest tile loses least by
        // it: another one has to be a sixteenth better (6960 x 7728 x 4096: 128x256, estimated at 3% less than 256x256, takes 284
        // us for 210; 5000 x 5200 x 4096 129 for 109)
        if (fp8 && pl.tile_m == 256 && id != T256x256) cost += cost / 16;
        if (cost < best) {
            best = cost;
            r.tile = id;
            r.one_span = span;
        }
    }
    return r;
}

static pk_status ag_gemm_impl(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                              const void* A_gathered, const void* B_local, const float* scale_a, const float* scale_b,
                              const uint32_t* chunk_flags, uint32_t epoch, void* C_local, int comm_cus, int activation,
                              bool k_chunks, void* ws, size_t ws_bytes, bool ws_is_static, uint32_t* status, uint64_t timeout_us,
                              void* stream, int b_layout = PK_B_ROW_MAJOR) {
    pk_plan pl;
    pk_status st = k_chunks ? make_plan_ag_k(P, M, N, K, dt, &pl) : make_plan(P, M, N, K, dt, false, &pl);
    if (st != PK_OK) return st;
    if (rank < 0 || rank >= P) return PK_ERR_RANK;
    if (comm_cus < 0 || comm_cus > 4096) return PK_ERR_ARG;
    if (activation < PK_ACT_NONE || activation > PK_ACT_SILU) return PK_ERR_ARG;
    if (b_layout != PK_B_ROW_MAJOR && b_layout != PK_B_K_CONTIGUOUS) return PK_ERR_ARG;
    const bool bt = b_layout == PK_B_K_CONTIGUOUS;
    if (bt && k_chunks) return PK_ERR_ARG;
    const bool fp8 = dt == PK_FP8_E4M3;
    if (!A_gathered || !B_local || !C_local || !status) return PK_ERR_NULL;
    if (P > 1 && !chunk_flags) return PK_ERR_NULL;
    if (fp8 && (!scale_a || !scale_b)) return PK_ERR_DTYPE;
    if (!aligned16(A_gathered) || !aligned16(B_local) || !aligned16(C_local)) return PK_ERR_ALIGN;
    const int elem = fp8 ? 1 : 2;
    GemmArgs a = {};
    a.A = (const char*)A_gathered;
    a.B = (const char*)B_local;
    a.lda = pl.local_k * elem;
    a.ldb = (bt ? pl.local_k : pl.local_n) * elem;
    a.n = (int32_t)pl.local_n;
    a.ktiles = (int32_t)(pl.local_k / (fp8 ? 128 : 64));
    a.n_chunks = P;
    a.act = activation;
    const int64_t chunk_rows = M / P;
    const int grid = max_grid(comm_cus);
    if (ws && !bt && !k_chunks && sk_too_small(ag_plan_slots(pl, P), grid, a.ktiles, pl.tile_m, ws_bytes)) return PK_ERR_ARG;
    const AgRoute rt = ag_route(pl, P, M, fp8, bt, k_chunks, ws && !bt, grid);
    const int tile = rt.tile;
    const bool one_span = rt.one_span, sk = rt.sk;
    const int bm = kTileDim[tile].bm;
    a.rows_per_shard = (int32_t)(k_chunks ? M : chunk_rows);
    a.rows_per_chunk = a.rows_per_shard;
    a.rows_per_span = (int32_t)(one_span ? M : chunk_rows);
    a.tiles_m_shard = (int32_t)ceil_div(a.rows_per_span, bm);
    a.tiles_n = (int32_t)ceil_div(pl.local_n, kTileDim[tile].bn);
    a.grp_tile_rows = a.tiles_m_shard;
    a.n_groups = one_span ? 1 : P;
    a.group0 = one_span ? 0 : rank;
    if (one_span && !k_chunks) {
        a.row_rot = (int32_t)(rank * chunk_rows / bm);
        a.all_tile_rows = a.tiles_m_shard;
    }
    a.rank = rank;
    a.C = (uint16_t*)C_local;
    a.chunk_flags = chunk_flags;
    a.scale_a = scale_a;
    a.scale_b = scale_b;
    a.epoch = epoch;
    a.status = status;
    a.timeout_ticks = timeout_ticks(timeout_us);
    if (ws_is_static && sk) {
        // the library's own scratch keeps the last call's flags, whatever its epoch was: clear them (with a kernel, so
        // that the call can be captured into a graph) and use an epoch of its own
        hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, (uint32_t*)ws, (int)(kWsFlagBytes / 4));
        if (hipGetLastError() != hipSuccess) return PK_ERR_HIP;
        a.ws_epoch = 1;
    }
    return k_chunks ? run_gemm<EPI_AGK>(a, M, tile, comm_cus, fp8, false, nullptr, (hipStream_t)stream)
                    : run_gemm<EPI_AG>(a, M, tile, comm_cus, fp8, bt, sk ? ws : nullptr, (hipStream_t)stream);
}

static pk_status make_order(const int* order, int n_order, int P, EmuOrder* o) {
    if (n_order < 0 || n_order > PK_EMU_MAX_ORDER) return PK_ERR_ARG;
    if (n_order > 0 && !order) return PK_ERR_NULL;
    o->n = n_order;
    for (int i = 0; i < n_order; ++i) {
        if (order[i] < 0 || order[i] >= P) return PK_ERR_ARG;
        for (int j = 0; j < i; ++j)
            if (order[j] == order[i]) return PK_ERR_ARG;
        o->q[i] = order[i];
    }
    return PK_OK;
}

extern "C" {

int pk_version(void) { return 1; }

const char* pk_status_str(int s) {
    switch (s) {
        case PK_OK: return "ok";
        case PK_ERR_NULL: return "null pointer";
        case PK_ERR_SHAPE: return "unsupported shape";
        case PK_ERR_DTYPE: return "bad dtype or missing scales";
        case PK_ERR_ALIGN: return "pointer not 16-byte aligned";
        case PK_ERR_RANK: return "rank out of range";
        case PK_ERR_ARG: return "invalid argument";
        case PK_ERR_HIP: return "HIP launch failed";
        case PK_ERR_TIMEOUT: return "timed out waiting for a ready flag";
        default: return "unknown status";
    }
}

pk_status pk_gemm_rs_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    return make_plan(P, M, N, K, dt, true, plan);
}

pk_status pk_ag_gemm_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    return make_plan(P, M, N, K, dt, false, plan);
}

pk_status pk_gemm_rs(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                     const void* A_local, const void* B_local, const float* scale_a, const float* scale_b,
                     void* partials, void* outgoing, uint32_t* flags_in, uint32_t* flags_out, uint32_t epoch,
                     void* out_shard, uint32_t phases, int comm_cus, int partial_dt, int b_layout, void* workspace,
                     size_t workspace_bytes, uint32_t* status, uint64_t timeout_us, void* stream) {
    if ((phases & PK_PHASE_ALL) == 0 || (phases & ~(PK_PHASE_ALL | PK_PHASE_OVERLAP))) return PK_ERR_ARG;
    if ((phases & PK_PHASE_OVERLAP) && (phases & PK_PHASE_ALL) != PK_PHASE_ALL) return PK_ERR_ARG;
    if (!aligned16(workspace)) return PK_ERR_ALIGN;
    return gemm_rs_impl(P, rank, M, N, K, dt, A_local, B_local, scale_a, scale_b, partials, outgoing, flags_in,
                        flags_out, epoch, out_shard, nullptr, phases, comm_cus, partial_dt, false, workspace, workspace_bytes,
                        status, timeout_us, stream, b_layout);
}

pk_status pk_gemm_rs_cols_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    return make_plan_cols(P, M, N, K, dt, plan);
}

pk_status pk_gemm_rs_cols(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                          const void* A_local, const void* B_local, const float* scale_a, const float* scale_b,
                          void* partials, void* outgoing, uint32_t* flags_in, uint32_t* flags_out, uint32_t epoch,
                          void* out_shard, uint32_t phases, int comm_cus, int partial_dt, uint32_t* status,
                          uint64_t timeout_us, void* stream) {
    if (phases == 0 || (phases & ~PK_PHASE_ALL)) return PK_ERR_ARG;
    return gemm_rs_impl(P, rank, M, N, K, dt, A_local, B_local, scale_a, scale_b, partials, outgoing, flags_in,
                        flags_out, epoch, out_shard, nullptr, phases, comm_cus, partial_dt, true, nullptr, 0, status, timeout_us,
                        stream);
}

pk_status pk_gemm_ar_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    pk_status st = make_plan(P, M, N, K, dt, true, plan);
    if (st != PK_OK) return st;
    plan->ar_flags_per_slot = ceil_div(M / P, PK_AR_ROWS) * plan->tiles_n;
    return PK_OK;
}

pk_status pk_gemm_ar(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                     const void* A_local, const void* B_local, const float* scale_a, const float* scale_b,
                     void* partials, void* outgoing, uint32_t* flags_in, uint32_t* flags_out,
                     void* out_full, void* bcast_out, uint32_t* ar_flags_in, uint32_t* ar_flags_out,
                     uint32_t epoch, uint32_t phases, int comm_cus, int partial_dt, uint32_t* status,
                     uint64_t timeout_us, void* stream) {
    if (phases == 0 || (phases & ~(PK_PHASE_ALL | PK_PHASE_WAIT))) return PK_ERR_ARG;
    if (!out_full || !ar_flags_in || !status) return PK_ERR_NULL;
    if (P > 1 && (!bcast_out || !ar_flags_out)) return PK_ERR_NULL;
    if (!aligned16(out_full) || !aligned16(bcast_out)) return PK_ERR_ALIGN;
    pk_plan pl;
    pk_status st = pk_gemm_ar_plan(P, M, N, K, dt, &pl);
    if (st != PK_OK) return st;
    if (rank < 0 || rank >= P) return PK_ERR_RANK;
    AllReduceOut ar = {(uint16_t*)bcast_out, ar_flags_in, ar_flags_out, pl.ar_flags_per_slot, (phases & PK_PHASE_WAIT) != 0};
    if (phases & PK_PHASE_ALL) {
        // the reduce phase writes rows R_rank of out_full
        uint16_t* own_rows = (uint16_t*)out_full + (int64_t)rank * (M / P) * N;
        st = gemm_rs_impl(P, rank, M, N, K, dt, A_local, B_local, scale_a, scale_b, partials, outgoing, flags_in,
                          flags_out, epoch, own_rows, &ar, phases & PK_PHASE_ALL, comm_cus, partial_dt, false, nullptr, 0, status,
                          timeout_us, stream);
        if (st != PK_OK) return st;
    }
    if (ar.wait) {
        const int64_t n_flags = (int64_t)P * pl.ar_flags_per_slot;
        hipLaunchKernelGGL(ar_wait_kernel, dim3((unsigned)ceil_div(n_flags, 256)), dim3(256), 0, (hipStream_t)stream,
                           (const uint32_t*)ar_flags_in, n_flags, epoch, status, timeout_ticks(timeout_us));
        if (hipGetLastError() != hipSuccess) return PK_ERR_HIP;
    }
    return PK_OK;
}

pk_status pk_ag_gemm(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                     const void* A_gathered, const void* B_local, const float* scale_a, const float* scale_b,
                     const uint32_t* chunk_flags, uint32_t epoch, void* C_local, int comm_cus, int activation,
                     int b_layout, void* workspace, size_t workspace_bytes, uint32_t* status, uint64_t timeout_us,
                     void* stream) {
    if (!aligned16(workspace)) return PK_ERR_ALIGN;
    return ag_gemm_impl(P, rank, M, N, K, dt, A_gathered, B_local, scale_a, scale_b, chunk_flags, epoch, C_local, comm_cus,
                        activation, false, workspace, workspace_bytes, false, status, timeout_us, stream, b_layout);
}

pk_status pk_ag_gemm_static(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                            const void* A_gathered, const void* B_local, const float* scale_a, const float* scale_b,
                            const uint32_t* chunk_flags, uint32_t epoch, void* C_local, int comm_cus, int activation,
                            uint32_t* status, uint64_t timeout_us, void* stream) {
    // the tiles of one launch must fit the scratch array: one fp32 tile per workgroup, one workgroup per compute unit
    pk_plan pl;
    pk_status st = make_plan(P, M, N, K, dt, false, &pl);
    if (st != PK_OK) return st;
    if ((size_t)pl.workspace_bytes > (size_t)PK_STATIC_WS_BYTES) return PK_ERR_ARG;
    void* ws = nullptr;
    st = scratch_of_device(&ws);
    if (st != PK_OK) return st;
    return ag_gemm_impl(P, rank, M, N, K, dt, A_gathered, B_local, scale_a, scale_b, chunk_flags, epoch, C_local, comm_cus,
                        activation, false, ws, (size_t)PK_STATIC_WS_BYTES, true, status, timeout_us, stream);
}

pk_status pk_ag_gemm_k_plan(int P, int64_t M, int64_t N, int64_t K, pk_dtype dt, pk_plan* plan) {
    return make_plan_ag_k(P, M, N, K, dt, plan);
}

pk_status pk_ag_gemm_k(int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt,
                       const void* A_gathered, const void* B_local, const float* scale_a, const float* scale_b,
                       const uint32_t* chunk_flags, uint32_t epoch, void* C_local, int comm_cus, int activation,
                       uint32_t* status, uint64_t timeout_us, void* stream) {
    return ag_gemm_impl(P, rank, M, N, K, dt, A_gathered, B_local, scale_a, scale_b, chunk_flags, epoch, C_local, comm_cus,
                        activation, true, nullptr, 0, false, status, timeout_us, stream);
}

pk_status pk_emu_deliver_kchunks_dma(int P, int64_t M, int64_t K, int elem_bytes, const void* staging, void* A_gathered,
                                     uint32_t* chunk_flags, uint32_t epoch, const int* order, int n_order, void* stream) {
    if (P < 1 || P > PK_EMU_MAX_ORDER || M < 1 || K < 1 || K % P) return PK_ERR_SHAPE;
    if (elem_bytes != 1 && elem_bytes != 2) return PK_ERR_DTYPE;
    if (!staging || !A_gathered || !chunk_flags) return PK_ERR_NULL;
    const size_t pitch = (size_t)K * elem_bytes, width = (size_t)(K / P) * elem_bytes;
    EmuOrder o;
    pk_status st = make_order(order, n_order, P, &o);
    if (st != PK_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    for (int i = 0; i < o.n; ++i) {
        const size_t off = (size_t)o.q[i] * width;
        // M pieces of K/P elements, one per row: the strided layout of a gather along the last dimension
        if (hipMemcpy2DAsync((char*)A_gathered + off, pitch, (const char*)staging + off, pitch, width, (size_t)M,
                             hipMemcpyDeviceToDevice, s) != hipSuccess)
            return PK_ERR_HIP;
        if (hipStreamWriteValue32(s, chunk_flags + o.q[i], epoch, 0) != hipSuccess) return PK_ERR_HIP;
    }
    return PK_OK;
}

pk_status pk_emu_deliver_chunks(int P, int64_t M, int64_t K, int elem_bytes, const void* staging, void* A_gathered,
                                uint32_t* chunk_flags, uint32_t epoch, const int* order, int n_order,
                                uint32_t gap_us, int n_wg, uint32_t* counters, void* stream) {
    if (P < 1 || P > PK_EMU_MAX_ORDER || M < 1 || K < 1 || M % P) return PK_ERR_SHAPE;
    if (elem_bytes != 1 && elem_bytes != 2) return PK_ERR_DTYPE;
    if (n_wg < 0 || n_wg > 4096) return PK_ERR_ARG;
    if (!staging || !A_gathered || !chunk_flags || !counters) return PK_ERR_NULL;
    const int64_t chunk_bytes = (M / P) * K * elem_bytes;
    if (chunk_bytes % 16) return PK_ERR_SHAPE;
    if (!aligned16(staging) || !aligned16(A_gathered)) return PK_ERR_ALIGN;
    EmuOrder o;
    pk_status st = make_order(order, n_order, P, &o);
    if (st != PK_OK) return st;
    if (n_order == 0) return PK_OK;
    hipLaunchKernelGGL(emu_chunks_kernel, dim3(n_wg ? n_wg : 32), dim3(256), 0, (hipStream_t)stream, (const char*)staging,
                       (char*)A_gathered, chunk_bytes, chunk_flags, epoch, o, gap_us, counters);
    return hipGetLastError() == hipSuccess ? PK_OK : PK_ERR_HIP;
}

pk_status pk_emu_deliver_chunks_dma(int P, int64_t M, int64_t K, int elem_bytes, const void* staging, void* A_gathered,
                                    uint32_t* chunk_flags, uint32_t epoch, const int* order, int n_order, void* stream) {
    if (P < 1 || P > PK_EMU_MAX_ORDER || M < 1 || K < 1 || M % P) return PK_ERR_SHAPE;
    if (elem_bytes != 1 && elem_bytes != 2) return PK_ERR_DTYPE;
    if (!staging || !A_gathered || !chunk_flags) return PK_ERR_NULL;
    const int64_t chunk_bytes = (M / P) * K * elem_bytes;
    EmuOrder o;
    pk_status st = make_order(order, n_order, P, &o);
    if (st != PK_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    for (int i = 0; i < o.n; ++i) {
        const int64_t off = (int64_t)o.q[i] * chunk_bytes;
        // stream order puts the flag write behind the completed copy
        if (hipMemcpyAsync((char*)A_gathered + off, (const char*)staging + off, (size_t)chunk_bytes, hipMemcpyDeviceToDevice,
                           s) != hipSuccess)
            return PK_ERR_HIP;
        if (hipStreamWriteValue32(s, chunk_flags + o.q[i], epoch, 0) != hipSuccess) return PK_ERR_HIP;
    }
    return PK_OK;
}

pk_status pk_emu_deliver_partials(int P, int64_t M, int64_t N, int tile_m, int tile_n, const float* staging,
                                  float* partials, uint32_t* flags_in, uint32_t epoch, const int* order, int n_order,
                                  uint32_t gap_us, int n_wg, void* stream) {
    if (P < 1 || P > PK_EMU_MAX_ORDER || M < 1 || N < 1 || M % P || N % 4) return PK_ERR_SHAPE;
    if (tile_m < 1 || tile_n < 4 || tile_n % 4 || n_wg < 0 || n_wg > 4096) return PK_ERR_ARG;
    if (!staging || !partials || !flags_in) return PK_ERR_NULL;
    if (!aligned16(staging) || !aligned16(partials)) return PK_ERR_ALIGN;
    EmuOrder o;
    pk_status st = make_order(order, n_order, P, &o);
    if (st != PK_OK) return st;
    if (n_order == 0) return PK_OK;
    const int rows = (int)(M / P);
    const int tiles_m = (int)ceil_div(rows, tile_m), tiles_n = (int)ceil_div(N, tile_n);
    hipLaunchKernelGGL(emu_partials_kernel, dim3(n_wg ? n_wg : 32), dim3(256), 0, (hipStream_t)stream, staging, partials, flags_in,
                       epoch, o, gap_us, rows, (int)N, tile_m, tile_n, tiles_m, tiles_n);
    return hipGetLastError() == hipSuccess ? PK_OK : PK_ERR_HIP;
}

pk_status pk_probe_mfma(int iters, int random_operands, uint64_t* report, double* flops_out, void* stream) {
    if (!report) return PK_ERR_NULL;
    if (iters < 1 || iters > (1 << 22)) return PK_ERR_ARG;
    const int n_wg = 2 * num_cus();
    hipLaunchKernelGGL(probe_mfma_kernel, dim3(n_wg), dim3(256), 0, (hipStream_t)stream, iters, random_operands ? 1 : 0, report);
    if (hipGetLastError() != hipSuccess) return PK_ERR_HIP;
    if (flops_out) *flops_out = (double)n_wg * 4.0 * (double)iters * 16.0 * 32768.0;
    return PK_OK;
}

pk_status pk_partition_create(int comm_cus, void** compute_stream, void** comm_stream) {
    if (!compute_stream || !comm_stream) return PK_ERR_NULL;
    const int ncu = num_cus();
    if (comm_cus < 8 || comm_cus % 8 || comm_cus > ncu - 8 || ncu > 1024) return PK_ERR_ARG;
    // Bit i of the mask is compute unit i/8 of XCD i%8 (checked on the device: a mask of the first 8*k bits
    // enables k compute units on each of the 8 XCDs), so both partitions span all XCDs and their L2s.
    uint32_t comm[32] = {0}, comp[32] = {0};
    const int words = (ncu + 31) / 32;
    for (int i = 0; i < ncu; ++i) (i < comm_cus ? comm : comp)[i >> 5] |= 1u << (i & 31);
    hipStream_t sc = nullptr, sm = nullptr;
    if (hipExtStreamCreateWithCUMask(&sc, words, comp) != hipSuccess) return PK_ERR_HIP;
    if (hipExtStreamCreateWithCUMask(&sm, words, comm) != hipSuccess) {
        (void)hipStreamDestroy(sc);
        return PK_ERR_HIP;
    }
    *compute_stream = sc;
    *comm_stream = sm;
    return PK_OK;
}

pk_status pk_partition_destroy(void* compute_stream, void* comm_stream) {
    pk_status st = PK_OK;
    if (compute_stream && hipStreamDestroy((hipStream_t)compute_stream) != hipSuccess) st = PK_ERR_HIP;
    if (comm_stream && hipStreamDestroy((hipStream_t)comm_stream) != hipSuccess) st = PK_ERR_HIP;
    return st;
}

// Digest of the interface that this library was compiled with, by which pk.py tells whether the extension module belongs to it: not
// part of the interface.
#ifndef PK_HEADER_DIGEST
#define PK_HEADER_DIGEST ""
#endif
const char* pk_header_digest(void) { return PK_HEADER_DIGEST; }

// Which way a call goes, for the tests: host only, launches nothing, not part of the interface.  op: 0 pk_gemm_rs, 1 pk_gemm_rs_cols,
// 2 pk_gemm_ar, 3 pk_ag_gemm, 4 pk_ag_gemm_k.  route: rows and columns of the tiles; 1 if their ready flags are published behind the
// GEMM; tiles of the first and of the second launch (0: one launch); 1 with a stream-K tail; all-gather: 1 if tile rows run over all
// chunks, reduce-scatter: 1 with two launches and the narrow reduce beside the second.
pk_status pk_test_route(int op, int P, int rank, int64_t M, int64_t N, int64_t K, pk_dtype dt, int partial_dt, int b_layout, uint32_t phases,
                        int comm_cus, int has_workspace, int32_t* route) {
    const bool fp8 = dt == PK_FP8_E4M3, bt = b_layout == PK_B_K_CONTIGUOUS, s16 = partial_dt == PK_PARTIAL_BF16;
    const bool cols = op == 1, k_chunks = op == 4;
    const int grid = max_grid(comm_cus);
    pk_plan pl;
    if (!route) return PK_ERR_NULL;
    if (op < 0 || op > 4) return PK_ERR_ARG;
    if (op >= 3) {
        const pk_status st = k_chunks ? make_plan_ag_k(P, M, N, K, dt, &pl) : make_plan(P, M, N, K, dt, false, &pl);
        if (st != PK_OK) return st;
        const AgRoute r = ag_route(pl, P, M, fp8, bt, k_chunks, has_workspace && !bt, grid);
        const TileDim d = kTileDim[r.tile];
        const int64_t rows = r.one_span ? tiles_across(M, d.bm) : P * (int64_t)tiles_across(M / P, d.bm);
        const int32_t v[7] = {d.bm, d.bn, 0, (int32_t)(rows * tiles_across(pl.local_n, d.bn)), 0, r.sk, r.one_span};
        for (int i = 0; i < 7; ++i) route[i] = v[i];
        return PK_OK;
    }
    const pk_status st = cols ? make_plan_cols(P, M, N, K, dt, &pl) : make_plan(P, M, N, K, dt, true, &pl);
    if (st != PK_OK) return st;
    const bool overlap = (phases & PK_PHASE_OVERLAP) && op == 0 && P > 1;
    const RsRoute r = rs_route(pl, P, rank, cols ? M : M / P, cols ? N / P : N, fp8, bt, s16, cols, phases & PK_PHASE_GEMM, phases & PK_PHASE_REDUCE,
                               overlap, grid);
    const int tiles = r.all_rows * r.tiles_n, first = r.first_rows * r.tiles_n;
    const int kt = (int)(pl.local_k / (fp8 ? 128 : 64));
    const bool sk = has_workspace && op == 0 && rs_takes_tail(pl, r, bt, s16) && sk_applies(ceil_div(tiles, 8) * 8, grid, kt);
    const int32_t v[7] = {kTileDim[r.t.tile].bm, kTileDim[r.t.tile].bn, r.t.late, r.overlap ? first : tiles, r.overlap ? tiles - first : 0, sk,
                          r.overlap && r.narrow_reduce};
    for (int i = 0; i < 7; ++i) route[i] = v[i];
    return PK_OK;
}

}  // extern "C"
