// Shared device/host definitions of the gfx950 fused-MoE library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/uniep_moe.h"

namespace uniep {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

constexpr int kMaxTopK = 16;
constexpr int kMaxExperts = 1024;
constexpr int kWave = 64;
constexpr int kMaxDevices = 64;                           // per-device host caches are indexed by the HIP device id
constexpr size_t kRouteStaticScratchBytes = 4u << 20;     // file-scope scratch of moe_route_static

// The tail kernels (combine, dX) have a wave for each piece of work.  A launch has to have fewer than 2^32
// work-items (hipErrorInvalidConfiguration otherwise): beyond 2^22 workgroups of 256 threads another launch
// goes on where the last one stopped.  (A loop in the kernel instead made it slower at every size: training
// step of 60001 tokens 3186 -> 3296 us.)
constexpr int kTailWaves = 4;   // of a workgroup
constexpr size_t kTailGroups = 1u << 22;
template <class F>
inline void launch_tail_waves(size_t waves, F launch) {
    const size_t groups = (waves + kTailWaves - 1) / kTailWaves;
    for (size_t g = 0; g < groups; g += kTailGroups)
        launch(dim3((unsigned)(groups - g < kTailGroups ? groups - g : kTailGroups)), (uint32_t)(g * kTailWaves));
}

// ---- bf16 <-> fp32 (round-to-nearest-even; gfx950 has a native packed convert)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2_t v = {lo, hi};
    bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return __builtin_bit_cast(uint32_t, b);
}
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// ---- scoreboard primitives (agent scope: visible across all 8 XCDs' L2s)
__device__ __forceinline__ int ld_acquire(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void add_release(int* p, int v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Write-through stores (agent scope): the data goes past this XCD's L2 to the
// memory side, so a consumer on any XCD sees it once the store has completed
// (s_waitcnt vmcnt(0)) and the consumer has acquired.  Producers that publish a
// tile written only with these stores can signal with a relaxed atomic instead
// of a release, which would write back the whole L2 of the XCD.
__device__ __forceinline__ void store_wt8(void* p, u32x2_t v) {
    __hip_atomic_store((uint64_t*)p, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
// (two 8-byte stores: the compiler has no 16-byte atomic store, and a store hidden in inline
// assembly would escape its hazard handling for the data registers)
__device__ __forceinline__ void store_wt16(void* p, u32x4_t v) {
    store_wt8(p, u32x2_t{v[0], v[1]});
    store_wt8((char*)p + 8, u32x2_t{v[2], v[3]});
}
// Streaming store for outputs that are written once and not read again soon
// (o, the G|U stash, dXp, dW, y, dX): they should not displace operands in L2.
__device__ __forceinline__ void store_stream16(void* p, u32x4_t v) {
    __builtin_nontemporal_store(v, (u32x4_t*)p);
}
// All write-through stores of this wave have completed.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }
__device__ __forceinline__ void add_relaxed(int* p, int v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ---- work queues -----------------------------------------------------------
// The GEMM tasks are cut into kQueues lists, one per XCD (each XCD has its own
// L2): every expert belongs to one list (see QueuePlan), so the tiles that share
// an expert's weights and rows run on one XCD and meet in its L2.  Inside a list
// the experts are pipelined with a lag: the producer block of the list's
// (i+L)-th expert comes before the consumer block of its i-th, so consumers
// rarely wait.  A workgroup drains its own XCD's list first and then steals from the
// others; the token-parallel tail tasks (combine / dX) come last.  Dependencies
// point to earlier entries of the same list, and an entry is fetched only by a
// running workgroup, so the lowest unfinished entry of every list can always run.
constexpr int kQueues = 8;
// Cursor sets: 1+p = staged launch of phase p; the last set = persistent launch.  The
// persistent launches' cursors take one atomic per task from every worker and must not share
// a 128-byte line with the table (list lengths and bases) that every task fetch reads: with
// set 0, which does, the whole step was 3 % slower.
constexpr int kPasses = 7;
constexpr int kPersistentPass = kPasses - 1;

// Control words at the head of a forward/backward workspace.
enum CtrlWord {
    CTRL_STATUS = 0,   // 0 ok, else MOE_ERR_DEVICE
    CTRL_NRT = 1,      // scoreboard slots of the row tiles
    CTRL_NTAIL = 2,    // number of tail tasks
    CTRL_NWAIT = 3,    // completions the tail tasks wait for
    CTRL_DONE = 4,     // completion counter of the last GEMM phase
    CTRL_WAIT_TICKS = 5,   // sum over workers of 10 ns ticks spent in scoreboard waits (diagnostic)
    CTRL_TAIL_WAIT_TICKS = 6,   // the same for the waits of the tail tasks
    CTRL_QLEN = 8,     // [8]  entries per list
    CTRL_QBASE = 16,   // [8]  first entry of each list in the task array
    CTRL_CURSOR = 24,  // [kPasses][kQueues + 1]  list cursors and tail cursor per pass
    CTRL_XCD_WORKERS = 24 + kPasses * (kQueues + 1) + 2,   // [8] workers that started on each XCD
    CTRL_XCD_ARRIVED = CTRL_XCD_WORKERS + kQueues,         // [8] workers of each XCD that ran out of GEMM work
    CTRL_STARTED = CTRL_XCD_ARRIVED + kQueues,             // workers that started
    CTRL_WORDS = CTRL_STARTED + 1
};

constexpr int kFetchDone = INT32_MIN;

__device__ __forceinline__ int xcc_id() {
    unsigned v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return (int)(v & (kQueues - 1));
}

// Called by one thread.  Returns an index into the task array (>= 0), or
// -1 - t for tail task t, or kFetchDone.  `exhausted` is the caller's bitmask of
// lists already seen empty.  use_lists / use_tail restrict a staged launch.
__device__ __forceinline__ int fetch_task(int* ctrl, int pass, int home, unsigned& exhausted,
                                          bool use_lists, bool use_tail) {
    int* cur = ctrl + CTRL_CURSOR + pass * (kQueues + 1);
    if (use_lists) {
        // (not unrolled: `home` is fixed for the kernel, and eight precomputed cursor addresses
        // would occupy registers, or scratch, across the worker's whole loop)
#pragma unroll 1
        for (int i = 0; i < kQueues; ++i) {
            const int q = (home + i) & (kQueues - 1);
            if (exhausted & (1u << q)) continue;
            const int len = ctrl[CTRL_QLEN + q];
            const int id = (len > 0) ? atomicAdd(cur + q, 1) : len;
            if (id < len) return ctrl[CTRL_QBASE + q] + id;
            exhausted |= 1u << q;
        }
    }
    if (use_tail) {
        const int t = atomicAdd(cur + kQueues, 1);
        if (t < ctrl[CTRL_NTAIL]) return -1 - t;
    }
    return kFetchDone;
}

// Split fetch, so that the round trip of the cursor atomic overlaps with the
// current task: fetch_issue() is called (by one thread) before the task runs and
// only issues the atomic on the first list not yet seen empty; fetch_finish()
// after the task turns the result into the next task, falling back to the
// blocking walk over the remaining lists and the tail.
struct PendingFetch {
    int q;     // list the atomic was issued on, -1 if none
    int id;    // value the atomic returned
};
__device__ __forceinline__ PendingFetch fetch_issue(int* ctrl, int pass, int home, unsigned exhausted,
                                                    bool use_lists) {
    PendingFetch f;
    f.q = -1;
    f.id = 0;
    // first list from `home` on (cyclically) that has not been seen empty: one computed address, so
    // that the compiler does not keep eight cursor addresses alive across the worker's whole loop
    const unsigned live = ~exhausted & ((1u << kQueues) - 1u);
    if (use_lists && live != 0) {
        const unsigned rot = ((live >> home) | (live << (kQueues - home))) & ((1u << kQueues) - 1u);
        const int q = (home + __builtin_ctz(rot)) & (kQueues - 1);
        f.q = q;
        f.id = atomicAdd(ctrl + CTRL_CURSOR + pass * (kQueues + 1) + q, 1);
    }
    return f;
}
__device__ __forceinline__ int fetch_finish(const PendingFetch f, int* ctrl, int pass, int home,
                                            unsigned& exhausted, bool use_lists, bool use_tail) {
    if (f.q >= 0) {
        if (f.id < ctrl[CTRL_QLEN + f.q]) return ctrl[CTRL_QBASE + f.q] + f.id;
        exhausted |= 1u << f.q;
    }
    return fetch_task(ctrl, pass, home, exhausted, use_lists, use_tail);
}

// Order of the nt x nct tiles (row tile j, column tile ct) of one expert inside its block of
// a list.  The CUs of an XCD take consecutive entries, and every tile they run at the same
// time streams its own A rows and its own B columns through the XCD's L2.  Entry i walks
// groups of kColGroup column tiles, inside a column group row groups of kRowGroup row tiles:
// 32 consecutive entries cover 4 row tiles x 8 column tiles (12 operand streams) where a
// row-major order covers 1 x 32 (33 streams: the weights of a 1024-row expert were fetched
// four times).  Inside a 4 x 8 group the row-tile GEMMs (forward, dH, dXp) put the row tiles
// innermost, so that the tiles that share a weight tile are fetched back to back (measured
// 1 % on the forward pass and 0.7 % on the backward pass of 512-row experts); the
// weight-gradient blocks, whose two operands are both row slabs of the expert, keep the column
// tiles innermost (the other order cost 0.5 %).
// block_pos() gives the entry of tile (j, ct); for_each_tile() hands every tile of the grid to
// the lanes of one wave, 8 row tiles x 8 column tiles per round, without a division.
constexpr int kColGroup = 8;   // 4 x 8 and 6 x 6 (rows x columns) measured within 1 % of 8 x 4
constexpr int kRowGroup = 4;
template <bool ROWS_INNERMOST>
__device__ __forceinline__ int block_pos(int j, int ct, int nt, int nct) {
    const int g = ct / kColGroup;
    const int width = min(kColGroup, nct - g * kColGroup);   // the last group may be narrower
    const int base = g * nt * kColGroup;
    if (ROWS_INNERMOST) {
        const int rg = j / kRowGroup;
        const int rows = min(kRowGroup, nt - rg * kRowGroup);   // and the last row group shorter
        return base + rg * kRowGroup * width + (ct - g * kColGroup) * rows + (j - rg * kRowGroup);
    }
    return base + j * width + (ct - g * kColGroup);
}
template <class F>
__device__ __forceinline__ void for_each_tile(int lane, int nt, int nct, F f) {
    for (int j0 = 0; j0 < nt; j0 += 8)
        for (int c0 = 0; c0 < nct; c0 += 8) {
            const int j = j0 + (lane >> 3), ct = c0 + (lane & 7);
            if (j < nt && ct < nct) f(j, ct);
        }
}

// Which expert goes to which list, and where its blocks stand in it.  The lists should end at the
// same time: work that one XCD steals from another list has lost the L2 sharing between the
// tiles of a row tile and of an expert, and runs about half as fast.  So the experts are sorted
// by rows (descending, in 63 classes of equal width and one of those without rows; ties by id) and dealt to the lists in
// boustrophedon order (ranks 0..7 to lists 0..7, ranks 8..15 to lists 7..0, ...).  Big experts
// come first in every list, small ones fill the end.  The producer block of a list's (i + lag)-th
// expert comes before the consumer block of its i-th: A0, A1, B0, A2, B1, ..., A(n-1), B(n-2),
// B(n-1) for a lag of 1.  The plan depends only on the counts, so it is the same on every run.
// Experts without rows never share a class with those of few rows: dealt together by id, one list could get
// all of the latter (600 tokens under Zipf(1.2) routing, 80 of 512 experts of width 2048 and inner width 512 with
// rows: backward 971 -> 847 us, 907 us where the experts were sorted exactly).
//
// Latency is all that counts here (one launch in front of every pass, nothing else can run), so
// every one of kPlanBlocks workgroups makes the whole plan for itself, without a word to
// the others (ranks from ballots, positions from scans: five barriers), and writes the tasks
// of its share of the experts.  One workgroup of 1024 threads with a loop over the experts per
// thread took 11 us for 128 experts of which 8 have rows, 15 us for 128 with 512 rows each and
// 45 us for 512 experts.
constexpr int kPlanThreads = 256;
constexpr int kPlanBlocks = 32;   // 128 waves: up to 128 experts, one wave writes one expert's tasks
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kListSlots = kMaxExperts / kQueues;
struct QueuePlan {
    int32_t a[kQueues][kListSlots + 1];   // producer tasks in front of slot i of a list, without the other blocks
    int32_t b[kQueues][kListSlots + 1];   // consumer tasks likewise
    int32_t rows[kMaxExperts];
    int32_t rt0[kMaxExperts];             // first scoreboard slot of the expert
    int32_t sums[kPlanWaves];             // slots of each wave's experts
    int32_t most[kPlanWaves], total[kPlanWaves];   // rows: of the expert that has most, together
    int32_t counts[kPlanWaves][2];        // experts with few (and, shifted left by 16, medium) and with more rows
    int32_t hist[kPlanWaves][64];
    int32_t first[kPlanWaves][64];
    uint16_t slot[kMaxExperts];           // list * kListSlots + slot
    int32_t base[kQueues + 1];            // first entry of each list
    int32_t lag, n_row_tiles;
};
// Lag (in experts) between an expert's producer and consumer blocks: enough
// producer tasks in between (about four rounds of one XCD's workgroups) that a
// consumer's inputs are complete when it is fetched, also near the end of the
// lists, where stealing workgroups drain the consumer blocks quickly.
__device__ __forceinline__ int queue_lag(int total_producer_tasks, int ec) {
    const int per = max(1, total_producer_tasks / max(1, ec));
    return min(16, max(1, (128 + per - 1) / per));
}


// How a pass cuts an expert's rows into tiles of bm = 256 or 128 rows.  A tile costs its stream of weights whatever its rows (one of
// some 20 rows 0.43 of a full one), and batches are powers of two more often than not, so that many experts have just over a
// multiple of 256 rows: up to most_higher of the others take 32 rows each of a last tile that has no more.  A higher tile
// costs 0.11 of a tile beyond its share of the work: with eight of them in place of one (4096 rows) the layer took 3 %
// longer, with three (1875 rows) 1 % less, with one (512 rows and some) the forward pass 6 % less and (256 and some) 17 %.
// Past 16 tiles there is nothing to gain.
struct TileRule {
    int bm;
    int most_higher;   // kMostHigher or 0
    // scoreboard slots of an expert: one for every 256 rows; tiles of 128 rows have two flags a slot
    static __device__ __forceinline__ int slots(int rows) { return (rows + 255) >> 8; }
    __device__ __forceinline__ int flags(int slot) const { return bm == 256 ? slot : 2 * slot; }
    // how many of the tiles are 32 rows higher
    __device__ __forceinline__ int higher(int rows) const {
        const int n = slots(rows), m = (rows - (n - 1) * 256 + 31) >> 5;
        return n <= kMostTiles && m <= min(most_higher, n - 1) ? m : 0;
    }
    __device__ __forceinline__ int tiles(int rows) const {
        return bm == 256 ? slots(rows) - (higher(rows) > 0 ? 1 : 0) : (rows + 127) >> 7;
    }
    // first row of tile j, the first `h` tiles being higher, and the rows of it
    __device__ __forceinline__ int first(int j, int h) const { return j * bm + 32 * min(j, h); }
    __device__ __forceinline__ int rows_of(int j, int h, int rows) const { return min(bm + (j < h ? 32 : 0), rows - first(j, h)); }
    static constexpr int kMostHigher = 3, kMostTiles = 16;
};
// Chooses the rule from the rows that the queue has, which only the device knows (a share of the experts may hold several times
// the rows that even routing would give it, or a fraction), the same in every planning workgroup.
// halves / 2: tasks of 256 rows a CU (on average) below which tiles have 128 rows.  Where CUs are idle, two tiles side by side
// take less than one, and low tiles keep two stages on their way (mma_low; not worth it for GEMMs of a few stages); where
// the CUs are full they cost more, as each streams the weights for itself.  Measured, us with tiles of 256 / of 128 rows (tasks a CU):
// training steps of 1000 tokens on 8 experts of 512 x 1024 (0.3) 176 / 133, 1500 on 2 of 8 of 4096 x 14336 (0.8) 1660 / 1407,
// 4096 on 16 of 128 of 4096 x 1536 (1.4) 806 / 762, 8000 on 8 of 512 x 1024 (1.5) 320 / 318, 20000 on 32 of 128 of 1024 x 384
// (2.8) 413 / 441; forward passes of 4099 tokens on 16 of 64 of 2048 x 1408 (1.8) 180 / 173, 10000 on 8 of 512 x 1024 (3.0)
// 111 / 125, 46158 rows on 32 of 1024 x 384 163 / 194.  Of 400 batches of eleven layers (shares, even and skewed routing) the bound is on
// average 0.8 % forward and 0.2 % backward from the better height; an estimate of both times from the tiles, the rows and
// the largest expert was 0.7 % and 0.4 %, but up to 21 % from it.
// Higher tiles from 3 tasks a CU on: training steps without / with, 3000 tokens on 16 of 64 experts of 1280 x 896 (0.8)
// 265 / 276, 8192 on 32 of 256 of 7168 x 2048 (5.5) 3169 / 2960.
struct TileChoice {
    static int rows_of(const moe_shape_t& s, int caller) { return caller == 0 && s.d + s.I < 8 * 64 ? 256 : caller; }
    int tile_rows;   // 128, 256, or 0 = by the rows
    int col_tiles;   // column tiles an expert of the pass's row-tile GEMMs
    int workers, halves;
    __device__ __forceinline__ TileRule rule(int rows) const {
        const long long tasks = (long long)rows * col_tiles / 256;
        if (tile_rows == 128 || (tile_rows == 0 && 2 * tasks < (long long)halves * workers)) return TileRule{128, 0};
        return TileRule{256, tasks >= 3ll * workers ? TileRule::kMostHigher : 0};
    }
};
// The plan of this workgroup (kPlanThreads threads, all of them call; ends with a barrier).
// Returns how rows are cut.  a_of(rule, rows) / b_of(rule, rows): tasks of an expert's producer and consumer block; `per_row_tile`
// producer tasks for each scoreboard slot.  skips: experts with up to skip_of(few, medium, more) rows have no tasks, the numbers
// of experts with rows whose class_of(rows) is 0, 1 and 2.
template <class FC, class FS, class FA, class FB>
__device__ __forceinline__ TileRule make_plan(QueuePlan& P, const int32_t* offsets, int ec, bool skips, FC class_of, FS skip_of, const TileChoice& choice,
                                              int per_row_tile, FA a_of, FB b_of) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    constexpr int kRounds = kMaxExperts / kPlanThreads;
    int rows[kRounds], run = 0, most = 0, sum = 0, counts = 0, more = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {   // wave w looks at experts 256 w + 64 r + lane
        const int e = 256 * w + 64 * r + lane;
        rows[r] = offsets[min(e + 1, ec)] - offsets[min(e, ec)];
        counts += __popcll(__ballot(rows[r] > 0 && class_of(rows[r]) == 0)) + (__popcll(__ballot(class_of(rows[r]) == 1)) << 16);
        more += __popcll(__ballot(class_of(rows[r]) == 2));
    }
    if (skips) {
        if (lane == 0) {
            P.counts[w][0] = counts;
            P.counts[w][1] = more;
        }
        __syncthreads();
        counts = more = 0;
#pragma unroll
        for (int i = 0; i < kPlanWaves; ++i) {
            counts += P.counts[i][0];
            more += P.counts[i][1];
        }
        const int skip = skip_of(rfl(counts & 0xffff), rfl((uint32_t)counts >> 16), rfl(more));
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            if (rows[r] <= skip) rows[r] = 0;
    }
    for (int i = tid; i < kQueues * (kListSlots + 1); i += kPlanThreads) (&P.a[0][0])[i] = (&P.b[0][0])[i] = 0;
    P.hist[w][lane] = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int e = 256 * w + 64 * r + lane, nt = TileRule::slots(rows[r]);
        int incl = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        P.rows[e] = rows[r];
        P.rt0[e] = run + incl - nt;   // inside the wave; the waves before are added by the reader (plan_rt0)
        run += __shfl(incl, 63);
        most = max(most, rows[r]);
        sum += rows[r];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        most = max(most, __shfl_xor(most, o));
        sum += __shfl_xor(sum, o);
    }
    if (lane == 0) {
        P.sums[w] = run;
        P.most[w] = most;
        P.total[w] = sum;
    }
    __syncthreads();
    int total = 0, n_slots = 0;
#pragma unroll
    for (int i = 0; i < kPlanWaves; ++i) {
        total += P.total[i];
        most = max(most, P.most[i]);
        n_slots += P.sums[i];
    }
    const TileRule tile = choice.rule(total);
    // rank inside the class: the wave's experts of the class so far + the lanes below
    const float scale = most > 0 ? 62.f / (float)most : 0.f;
    int cls[kRounds], rank[kRounds];
    volatile int32_t* hist = P.hist[w];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool in = 256 * w + 64 * r + lane < ec;
        cls[r] = rows[r] > 0 ? 1 + min(62, (int)((float)rows[r] * scale)) : 0;
        uint64_t m = __ballot(in);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const uint64_t bb = __ballot((cls[r] >> b) & 1);
            m &= ((cls[r] >> b) & 1) ? bb : ~bb;
        }
        if (in) rank[r] = hist[cls[r]] + __popcll(m & below);
        __builtin_amdgcn_wave_barrier();
        if (in && (m >> lane) <= 1ull) hist[cls[r]] = rank[r] + 1;   // the class's last lane moves its count
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {   // lane l: class 63 - l.  Experts in higher classes, then those of the class in the waves before
        const int c = 63 - lane;
        int mine = 0, tot = 0;
#pragma unroll
        for (int i = 0; i < kPlanWaves; ++i) {
            if (i < w) mine += P.hist[i][c];
            tot += P.hist[i][c];
        }
        int incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        P.first[w][c] = incl - tot + mine;
    }
    __builtin_amdgcn_wave_barrier();
    volatile int32_t* first = P.first[w];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int e = 256 * w + 64 * r + lane;
        if (e < ec) {
            const int k = first[cls[r]] + rank[r], i = k / kQueues, c = k % kQueues;
            const int q = (i & 1) ? kQueues - 1 - c : c;
            P.slot[e] = (uint16_t)(q * kListSlots + i);
            P.a[q][i] = a_of(tile, rows[r]);
            P.b[q][i] = b_of(tile, rows[r]);
        }
    }
    __syncthreads();
    {   // exclusive sums along each list: 32 threads a list, 4 slots a thread
        const int q = tid >> 5, i0 = (tid & 31) * 4;
        int va[4], vb[4], sa = 0, sb = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            va[j] = P.a[q][i0 + j];
            vb[j] = P.b[q][i0 + j];
            sa += va[j];
            sb += vb[j];
        }
        int ia = sa, ib = sb;
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) {
            const int x = __shfl_up(ia, o, 32), y = __shfl_up(ib, o, 32);
            if ((tid & 31) >= o) {
                ia += x;
                ib += y;
            }
        }
        int xa = ia - sa, xb = ib - sb;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            P.a[q][i0 + j] = xa;
            P.b[q][i0 + j] = xb;
            xa += va[j];
            xb += vb[j];
        }
        if (i0 + 4 == kListSlots) {
            P.a[q][kListSlots] = xa;
            P.b[q][kListSlots] = xb;
        }
    }
    __syncthreads();
    if (tid == 0) {
        int base = 0;
        for (int q = 0; q < kQueues; ++q) {
            P.base[q] = base;
            base += P.a[q][kListSlots] + P.b[q][kListSlots];
        }
        P.base[kQueues] = base;
        P.n_row_tiles = n_slots;
        P.lag = queue_lag(tile.flags(n_slots) * per_row_tile, ec);
    }
    __syncthreads();
    return tile;
}
// First entries of expert e's two blocks in the task array, and its first scoreboard slot.
__device__ __forceinline__ int plan_a(const QueuePlan& P, int e) {
    const int q = P.slot[e] / kListSlots, i = P.slot[e] % kListSlots;
    return P.base[q] + P.a[q][i] + P.b[q][max(0, i - P.lag)];
}
__device__ __forceinline__ int plan_b(const QueuePlan& P, int e) {
    const int q = P.slot[e] / kListSlots, i = P.slot[e] % kListSlots;
    return P.base[q] + P.a[q][min(i + P.lag + 1, kListSlots)] + P.b[q][i];
}
__device__ __forceinline__ int plan_rt0(const QueuePlan& P, int e) {
    int r = P.rt0[e];
    for (int i = 0; i < e / 256; ++i) r += P.sums[i];
    return r;
}
// The control words of a pass, by one workgroup.
__device__ __forceinline__ void write_ctrl(const QueuePlan& P, int* ctrl, int n_tail, int n_wait) {
    for (int i = threadIdx.x; i < CTRL_WORDS; i += kPlanThreads) {
        int v = 0;
        if (i == CTRL_NRT) v = P.n_row_tiles;
        if (i == CTRL_NTAIL) v = n_tail;
        if (i == CTRL_NWAIT) v = n_wait;
        if (i >= CTRL_QLEN && i < CTRL_QLEN + kQueues) v = P.base[i - CTRL_QLEN + 1] - P.base[i - CTRL_QLEN];
        if (i >= CTRL_QBASE && i < CTRL_QBASE + kQueues) v = P.base[i - CTRL_QBASE];
        ctrl[i] = v;
    }
}

// Bounded wait for *p >= need.  Returns false (and raises the status word) if
// the bound is exceeded or another worker already raised it, so that every
// wave leaves the kernel in finite time whatever happens.
__device__ __forceinline__ void fence_acquire() {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}
// The polls are relaxed loads; the one acquire fence follows the successful
// poll.  An acquire per poll would invalidate this XCD's L2 at the polling
// rate and slow down every tile still running on it.
__device__ __forceinline__ bool wait_ge(const int* p, int need, int* ctrl, long long limit_ticks,
                                        int stat_word = CTRL_WAIT_TICKS) {
    if (ld_relaxed(p) >= need) {
        fence_acquire();
        return true;
    }
    const long long t0 = wall_clock64();
    // Back off to one poll per ~3 us: a few hundred waiting workgroups polling one address at full
    // rate saturate its memory channel and slow down the tiles that are still running.
    for (int round = 0;; ++round) {
        if (round < 4) __builtin_amdgcn_s_sleep(16);
        else if (round < 8) __builtin_amdgcn_s_sleep(48);
        else __builtin_amdgcn_s_sleep(127);
        if (ld_relaxed(p) >= need) {
            fence_acquire();
            atomicAdd(ctrl + stat_word, (int)(wall_clock64() - t0));
            return true;
        }
        if (ld_relaxed(ctrl + CTRL_STATUS) != 0) return false;
        if (wall_clock64() - t0 > limit_ticks) {
            __hip_atomic_store(ctrl + CTRL_STATUS, (int)MOE_ERR_DEVICE, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
    }
}

// Publication of the rows a persistent worker wrote with ordinary (write-back)
// stores, for consumers that wait for ALL workers (the tail tasks).  A release
// writes back the whole L2 of the XCD, which stalls the tiles still running on
// it, so only the last worker of each XCD to run out of GEMM work releases, on
// behalf of the XCD: the others only count themselves in after their own stores
// have completed, which orders those stores before the releasing worker's
// write-back.  worker_started() is called once at kernel start, worker_arrived()
// once when the worker has no GEMM work left (both by one thread, the second
// after s_waitcnt vmcnt(0) and a workgroup barrier).
__device__ __forceinline__ void worker_started(int* ctrl, int xcd) {
    add_relaxed(ctrl + CTRL_XCD_WORKERS + xcd, 1);
    add_relaxed(ctrl + CTRL_STARTED, 1);
}
__device__ __forceinline__ void worker_arrived(int* ctrl, int xcd, int workers, long long limit_ticks) {
    if (!wait_ge(ctrl + CTRL_STARTED, workers, ctrl, limit_ticks)) return;   // every worker is registered
    const int on_xcd = ld_relaxed(ctrl + CTRL_XCD_WORKERS + xcd);
    const int before = __hip_atomic_fetch_add(ctrl + CTRL_XCD_ARRIVED + xcd, 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1 == on_xcd) add_release(ctrl + CTRL_DONE, on_xcd);
}

struct RowTile {   // one row tile of one local expert
    int32_t expert;  // local expert id
    int32_t row0;    // first row (position in the expert-sorted order)
    int32_t rows;    // valid rows in this tile (1..288)
};

// One GEMM task, self-contained so that a worker needs a single 16-byte load
// before it can start: no second trip to a row-tile table or to the offsets.
struct Task {
    int32_t idx;      // row-tile tasks: row tile index (its scoreboard flag); weight-gradient tasks: row-tile of the output (m index)
    int32_t code;     // (type << 28) | (local expert << 16) | column tile
    int32_t row0;     // row-tile tasks: first row of the tile; weight-gradient tasks: first row of the expert
    int32_t rows;     // row-tile tasks: rows in the tile; weight-gradient tasks: rows of the expert (the reduction length)
};
__host__ __device__ __forceinline__ int32_t task_code(int type, int expert, int ct) {
    return (int32_t)(((uint32_t)type << 28) | ((uint32_t)expert << 16) | (uint32_t)ct);
}
__device__ __forceinline__ int task_type(const Task& t) { return (int)((uint32_t)t.code >> 28); }
__device__ __forceinline__ int task_expert(const Task& t) { return (t.code >> 16) & 0xfff; }
__device__ __forceinline__ int task_ct(const Task& t) { return t.code & 0xffff; }
__device__ __forceinline__ RowTile task_row_tile(const Task& t) { return RowTile{task_expert(t), t.row0, t.rows}; }

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace uniep
