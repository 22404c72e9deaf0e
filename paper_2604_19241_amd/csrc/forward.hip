// Forward MegaKernel: dispatch(gather) + grouped GEMM gate/up + SwiGLU +
// grouped GEMM down + combine, as one persistent work-queue kernel.
//
// Paper: Section 3.1 (persistent workers, scoreboard, dynamic scheduling),
// Section 3.2 (GroupGEMM+Combine, top-k accumulation constraint), Section 4.3
// (producers and consumers walk the experts in the same ascending order),
// Listing 1 (the fetch loop).  On one GPU the "dispatch" of a token to its
// expert is a gather: the GEMM1 tile reads the rows of x through the
// permutation while it stages them into LDS, so the dispatched copy is never
// written to HBM; the scoreboard that remains orders GEMM1 -> GEMM2 per row
// tile and GEMM2 -> combine.  SwiGLU runs in the GEMM1 epilogue on the fp32
// accumulators.
#include "thin.hpp"

#include <algorithm>
#include <mutex>

namespace uniep {

enum TaskType { TASK_GEMM1 = 0, TASK_GEMM2 = 1, TASK_COMBINE = 2 };

constexpr int kCombineTokens = 16;   // tokens per combine task (2 per wave)

struct FwdParams {
    moe_shape_t s;
    const char* x;
    const char* w_gate;
    const char* w_up;
    const char* w_down;
    const float* topk_w;
    const int32_t* offsets;
    const int32_t* perm;
    const int32_t* inv_perm;
    char* y;
    char* gu;   // saved G|U [A,2I] or null
    char* h;    // [A,I]
    char* o;    // [A,d]
    int* ctrl;
    int* flag1;   // per row tile: GEMM1 column tiles finished
    Task* tasks;
    int nct1, nct2;   // column tiles of GEMM1 (128 h-columns each) and GEMM2 (256 each)
    int workers;   // workgroups of the worker launch (the tail waits for all of them)
    TileChoice tile;   // rows of the row tiles
    ThinRule rule;     // which experts are run outside the work queue; max_rows = 0: none
    long long spin_ticks;
};

// ------------------------------------------------------------- first launch
// The work queue of the experts that thin_run leaves to it, made by the first kPlanBlocks workgroups:
// row-tile table from the expert offsets, the per-XCD task lists (GEMM1 block of expert i+1 ahead of the
// GEMM2 block of expert i) and a cleared scoreboard.
template <bool TWO>
__device__ __forceinline__ void fwd_setup(const FwdParams& p, int block, QueuePlan& P) {
    const int ec = p.s.e_count, rows_here = p.offsets[ec];
    const TileRule tile = make_plan(P, p.offsets, ec, p.rule.max_rows > 0, [&](int rows) { return p.rule.size_class<TWO>(rows); },
                                    [&](int few, int medium, int more) { return p.rule.limit(few, medium, more, rfl(rows_here)); }, p.tile, p.nct1,
                                    [&](const TileRule& t, int rows) { return t.tiles(rows) * p.nct1; },
                                    [&](const TileRule& t, int rows) { return t.tiles(rows) * p.nct2; });
    const int lane = threadIdx.x & 63;
    for (int x = block * kPlanWaves + (threadIdx.x >> 6); x < ec; x += kPlanBlocks * kPlanWaves) {
        const int rows_x = P.rows[x], nt_x = tile.tiles(rows_x);
        if (nt_x == 0) continue;
        const int rt0 = tile.flags(plan_rt0(P, x)), r0 = p.offsets[x], higher = tile.higher(rows_x);
        for (int i = lane; i < nt_x; i += 64) p.flag1[rt0 + i] = 0;
        Task* t1 = p.tasks + plan_a(P, x);
        Task* t2 = p.tasks + plan_b(P, x);
        for_each_tile(lane, nt_x, p.nct1, [&](int j, int ct) {
            t1[block_pos<true>(j, ct, nt_x, p.nct1)] =
                Task{rt0 + j, task_code(TASK_GEMM1, x, ct), r0 + tile.first(j, higher), tile.rows_of(j, higher, rows_x)};
        });
        for_each_tile(lane, nt_x, p.nct2, [&](int j, int ct) {
            t2[block_pos<true>(j, ct, nt_x, p.nct2)] =
                Task{rt0 + j, task_code(TASK_GEMM2, x, ct), r0 + tile.first(j, higher), tile.rows_of(j, higher, rows_x)};
        });
    }
    if (block == 0) write_ctrl(P, p.ctrl, (p.s.T + kCombineTokens - 1) / kCombineTokens, p.workers);
}

__device__ __forceinline__ ThinParams thin_params(const FwdParams& p) {
    return ThinParams{p.s, p.x, p.w_gate, p.w_up, p.w_down, p.offsets, p.perm, p.gu, p.h, p.o, p.rule, p.workers};
}
// The queue (unless every expert is thin) and the thin experts' GEMM1, side by side: neither reads
// what the other writes.
// TWO: thin_may_be_two.
template <bool TWO>
__global__ void __launch_bounds__(kThinThreads) __attribute__((amdgpu_waves_per_eu(2)))
fwd_first_kernel(FwdParams p) {
    __shared__ __attribute__((aligned(16))) char smem[sizeof(ThinShared) > sizeof(QueuePlan) ? sizeof(ThinShared) : sizeof(QueuePlan)];
    const int block = (int)blockIdx.x - kPlanBlocks;
    if (block < 0) fwd_setup<TWO>(p, (int)blockIdx.x, *(QueuePlan*)smem);
    else thin_run<1, TWO ? kThinTwo : kThinFew>(thin_params(p), block, (int)gridDim.x - kPlanBlocks, *(ThinShared*)smem);
}
template <bool TWO>
__global__ void __launch_bounds__(kThinThreads) __attribute__((amdgpu_waves_per_eu(2)))
fwd_second_kernel(FwdParams p) {
    __shared__ __attribute__((aligned(16))) char smem[sizeof(ThinShared)];
    thin_run<2, TWO ? kThinTwo : kThinFew>(thin_params(p), (int)blockIdx.x, (int)gridDim.x, *(ThinShared*)smem);
}
// The same where there is no queue.
__global__ void __launch_bounds__(kThinThreads) __attribute__((amdgpu_waves_per_eu(2)))
thin_first_kernel(FwdParams p) {
    __shared__ __attribute__((aligned(16))) char smem[sizeof(ThinShared)];
    if (blockIdx.x == 0 && threadIdx.x < CTRL_WORDS) p.ctrl[threadIdx.x] = 0;
    thin_run<1, kThinAll>(thin_params(p), (int)blockIdx.x, (int)gridDim.x, *(ThinShared*)smem);
}
__global__ void __launch_bounds__(kThinThreads) __attribute__((amdgpu_waves_per_eu(2)))
thin_second_kernel(FwdParams p) {
    __shared__ __attribute__((aligned(16))) char smem[sizeof(ThinShared)];
    thin_run<2, kThinAll>(thin_params(p), (int)blockIdx.x, (int)gridDim.x, *(ThinShared*)smem);
}

// ------------------------------------------------------------- GEMM1 task
// h[row0.., ct*128 .. +128) = silu(x_e W_gate) * (x_e W_up) for one row tile.
// Tile rows = the tile's tokens (their rows of x fetched through the permutation: the dispatch);
// tile columns = 128 gate columns and the same 128 up columns, a column fragment being 16 gate columns and the same
// 16 up columns: G and U of one h element sit in the same lane and accumulator, elements v and 8 + v.
template <class Hook>
__device__ __forceinline__ void gemm1_task(const FwdParams& p, const RowTile rt, int ct,
                                           char* smem, Hook after_mainloop) {
    const int d = p.s.d, I = p.s.I, k = p.s.k;
    const int n0h = ct * (BN / 2);
    const Lane ln;
    FragAddr fa;
    frag_addresses<kKsPair, false>(fa, lds_addr(smem), ln);
    KsPairLoader la;
    const size_t first = (size_t)rt.expert * d * I * 2;
    la.init(ln, p.w_gate + first, p.w_up + first, n0h, I, I * 2);
    Acc acc;
    row_tile_gemm<kKsPair>(ln, la, d / BK, rt.rows, smem, fa, acc,
                           [&](int m) { return p.x + (size_t)(p.perm[rt.row0 + m] / k) * d * 2; });
    after_mainloop();

    // epilogue.  The wave's sub-tile is 128 rows x (32 gate columns | the same 32 up columns).
    // First the G|U stash, through the wave's LDS region so that 4 neighbouring lanes store 64
    // contiguous bytes; then h = silu(G) * U on the accumulators, out the same way in 8-byte
    // write-through pieces (8 lanes per 64-byte row segment): GEMM2 tiles on any XCD read it.
    const Lane le;
    const int l31 = le.l31, hf = le.hf;
    const int wm = le.wm, wn = le.wn;
    const int hc0 = n0h + 32 * wn;        // first h column of this wave
    const int rows_w = rt.rows - 128 * wm; // rows of the tile inside this wave's 128
    const int rows_m = rt.rows - BMAX;     // rows past 256: 16 of the wave's h columns, from 16 wm on
    auto h8 = [](const f32x16_t& a) {
        float hv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float g = a[e], u = a[8 + e];
            hv[e] = g * sigmoid_f(g) * u;
        }
        return u32x4_t{pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3]), pack_bf16x2(hv[4], hv[5]),
                       pack_bf16x2(hv[6], hv[7])};
    };
    if (p.gu) {
        WaveRepack<8> rp(smem, le);
#pragma unroll
        for (int tf = 0; tf < 4; ++tf)
#pragma unroll
            for (int af = 0; af < 2; ++af)
#pragma unroll
                for (int vg = 0; vg < 2; ++vg) rp.put(32 * tf + l31, 4 * vg + 2 * af + hf, pack8(acc.a[tf][af], vg));
        const int pc = rp.get_piece();                       // 0..3: G pieces, 4..7: U pieces
        const int col = hc0 + 8 * (pc & 3);
        char* gbase = p.gu + ((size_t)(rt.row0 + 128 * wm) * 2 * I + ((pc & 4) ? I : 0) + col) * 2;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int row = rp.get_row(j);
            const u32x4_t v = rp.get(j);
            if (row < rows_w && col < I) store_stream16(gbase + (size_t)row * 2 * I * 2, v);
        }
        if (rows_m > 0) {
            WaveRepack<4> rm(smem, le);
#pragma unroll
            for (int vg = 0; vg < 2; ++vg) rm.put(l31, 2 * vg + hf, pack8(acc.more, vg));
            const int pm = rm.get_piece(), mcol = hc0 + 16 * wm + 8 * (pm & 1);   // 0, 1: G pieces, 2, 3: U pieces
            char* mbase = p.gu + ((size_t)(rt.row0 + BMAX) * 2 * I + ((pm & 2) ? I : 0) + mcol) * 2;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int row = rm.get_row(j);
                const u32x4_t v = rm.get(j);
                if (row < rows_m && mcol < I) store_stream16(mbase + (size_t)row * 2 * I * 2, v);
            }
        }
    }
    {
        WaveRepack<4> rp(smem, le);
#pragma unroll
        for (int tf = 0; tf < 4; ++tf)
#pragma unroll
            for (int af = 0; af < 2; ++af) rp.put(32 * tf + l31, 2 * af + hf, h8(acc.a[tf][af]));
        const int col = hc0 + 4 * rp.get8_piece();   // 8-byte pieces: 4 columns each
        char* hbase = p.h + ((size_t)(rt.row0 + 128 * wm) * I + col) * 2;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int row = rp.get8_row(j);
            const u32x2_t v = rp.get8(j);
            if (row < rows_w && col < I) store_wt8(hbase + (size_t)row * I * 2, v);
        }
        if (rows_m > 0) {   // the lane's 8 columns of row 256 + l31 as they are: a few rows
            const int mcol = hc0 + 16 * wm + 8 * hf;
            if (l31 < rows_m && mcol < I) store_wt16(p.h + ((size_t)(rt.row0 + BMAX + l31) * I + mcol) * 2, h8(acc.more));
        }
    }
}

// ------------------------------------------------------------- GEMM2 task
// o[row0.., ct*256 .. +256) = h_e W_down[e] for one row tile.
template <class Hook>
__device__ __forceinline__ void gemm2_task(const FwdParams& p, const RowTile rt, int ct,
                                           char* smem, Hook after_mainloop) {
    const int d = p.s.d, I = p.s.I;
    const int n0 = ct * BN;
    const Lane ln;
    FragAddr fa;
    frag_addresses<kKs, false>(fa, lds_addr(smem), ln);
    KsLoader la;
    la.init(ln, p.w_down + (size_t)rt.expert * I * d * 2, n0, d, d * 2);
    Acc acc;
    row_tile_gemm<kKs>(ln, la, I / BK, rt.rows, smem, fa, acc,
                       [&](int m) { return p.h + (size_t)(rt.row0 + m) * I * 2; });
    after_mainloop();
    char* obase = p.o + ((size_t)rt.row0 * d + n0) * 2;
    store_subtile_bf16<true>(acc, smem, rt.rows, d - n0, [&](int row, int col, u32x4_t v) {
        store_stream16(obase + ((size_t)row * d + col) * 2, v);
    });
}

// ------------------------------------------------------------- combine task
// y[t] = sum_j w[t,j] * o[row(t,j)], slot order, fp32; one wave per token, 16
// bytes per lane, no LDS (Section 5.2 "Relay & Reduce Workers").
// KM = compile-time bound on k (8 or kMaxTopK): the row loads of all KM slots are in flight
// at once, so the smaller bound halves the registers and doubles the waves per SIMD.

// Slots of one token: the o row of each local one (-1: not here) and its gate.
template <int KM>
struct CombineSlots {
    int rows[KM];
    float w[KM];
    __device__ __forceinline__ void load(const FwdParams& p, int t) {
        const int k = p.s.k;
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            rows[j] = (j < k) ? p.inv_perm[(size_t)t * k + j] : -1;
            w[j] = (j < k) ? p.topk_w[(size_t)t * k + j] : 0.f;
        }
    }
};

// Two 16-byte column pieces of a lane, c0 (below d) and c0 + 512: all 2k row loads are issued before
// the first is used, so a wave keeps up to 2k KB in flight.
constexpr int kCombineCols = 2 * 64 * 8;   // columns of a wave's round
template <int KM>
__device__ __forceinline__ void combine_piece(const FwdParams& p, int t, int c0, const CombineSlots<KM>& slots) {
    const int d = p.s.d, k = p.s.k;
    const int (&rows)[KM] = slots.rows;
    const float (&w)[KM] = slots.w;
    const int c1 = c0 + 64 * 8;
    const bool two = c1 < d;
    u32x4_t v0[KM], v1[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        v0[j] = zero4();
        v1[j] = zero4();
        if (j < k && rows[j] >= 0) {
            const char* src = p.o + (size_t)rows[j] * d * 2;
            v0[j] = *(const u32x4_t*)(src + (size_t)c0 * 2);
            if (two) v1[j] = *(const u32x4_t*)(src + (size_t)c1 * 2);
        }
    }
    float a0[8], a1[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) a0[q] = a1[q] = 0.f;
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (j < k && rows[j] >= 0) {   // slot order, local slots only
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a0[2 * q] += w[j] * bf16_lo(v0[j][q]);
                a0[2 * q + 1] += w[j] * bf16_hi(v0[j][q]);
                a1[2 * q] += w[j] * bf16_lo(v1[j][q]);
                a1[2 * q + 1] += w[j] * bf16_hi(v1[j][q]);
            }
        }
    }
    u32x4_t y0, y1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        y0[q] = pack_bf16x2(a0[2 * q], a0[2 * q + 1]);
        y1[q] = pack_bf16x2(a1[2 * q], a1[2 * q + 1]);
    }
    store_stream16(p.y + ((size_t)t * d + c0) * 2, y0);
    if (two) store_stream16(p.y + ((size_t)t * d + c1) * 2, y1);
}

template <int NW, int KM = kMaxTopK>
__device__ __forceinline__ void combine_task(const FwdParams& p, int block) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int tt = wave; tt < kCombineTokens; tt += NW) {
        const int t = block * kCombineTokens + tt;
        if (t >= p.s.T) break;
        CombineSlots<KM> slots;
        slots.load(p, t);
        for (int c0 = lane * 8; c0 < p.s.d; c0 += kCombineCols) combine_piece<KM>(p, t, c0, slots);
    }
}

// ------------------------------------------------------------- the worker loop
// phase = -1: all tasks with scoreboard waits (persistent MegaKernel).
// phase = -2: every GEMM task with scoreboard waits, no tail tasks: the workers leave
// when the lists are empty and the combine runs as a launch of its own (fwd_tail_kernel).
// phase >= 0: only that phase's tasks (staged schedule; the waits are already
// satisfied by stream order).
__global__ void __launch_bounds__(kMmaThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
fwd_worker_kernel(FwdParams p, int phase) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int s_task;
    __shared__ int s_ok;
    int* ctrl = p.ctrl;
    const int pass = phase < 0 ? kPersistentPass : 1 + phase;
    const int home = xcc_id();
    const bool use_lists = phase != TASK_COMBINE;
    const bool use_tail = phase == -1 || phase == TASK_COMBINE;
    // this launch runs GEMM2 tiles: its workers publish their o rows once, when they run out of
    // GEMM work, instead of once per tile
    const bool publishes = phase == -1 || phase == TASK_GEMM2;
    bool arrived = false;
    unsigned exhausted = 0;
    if (phase == -2 && ctrl[CTRL_NRT] == 0) return;   // no expert with rows is left
    if (threadIdx.x == 0) {
        if (phase == -1) worker_started(ctrl, home);
        s_task = fetch_task(ctrl, pass, home, exhausted, use_lists, use_tail);
    }
    __syncthreads();
    for (;;) {
        const int id = s_task;
        if (id == kFetchDone) break;
        // The cursor atomic of the next task is issued behind the main loop of this one: vector
        // memory results return in order, so an atomic issued ahead of a tile would hold back
        // the first loads of its wave by the atomic's round trip.
        PendingFetch pf;
        pf.q = -1;
        pf.id = 0;
        bool issued = false;
        auto issue = [&]() {
            if (!issued && threadIdx.x == 0) pf = fetch_issue(ctrl, pass, home, exhausted, use_lists);
            issued = true;
        };
        if (id >= 0) {
            // the task is the same for every lane: keep its fields in scalar registers
            Task task = p.tasks[id];
            task.idx = rfl(task.idx);
            task.code = rfl(task.code);
            task.row0 = rfl(task.row0);
            task.rows = rfl(task.rows);
            const int type = task_type(task), ct = task_ct(task);
            if (phase >= 0 && type != phase) {
                // staged launch: another phase's task, nothing to do
            } else if (type == TASK_GEMM1) {
                const RowTile rt = task_row_tile(task);
                gemm1_task(p, rt, ct, smem, issue);
                wait_stores();
                __syncthreads();   // the write-through h stores of every wave have completed
                if (threadIdx.x == 0) add_relaxed(p.flag1 + task.idx, 1);
            } else {
                if (threadIdx.x == 0) s_ok = wait_ge(p.flag1 + task.idx, p.nct1, ctrl, p.spin_ticks);
                __syncthreads();
                if (s_ok) {
                    const RowTile rt = task_row_tile(task);
                    gemm2_task(p, rt, ct, smem, issue);
                }
            }
        } else {
            if (publishes && !arrived) {   // first tail task: all of this worker's o rows are written
                arrived = true;
                wait_stores();
                __syncthreads();
                if (threadIdx.x == 0) {
                    if (phase < 0) worker_arrived(ctrl, home, ctrl[CTRL_NWAIT], p.spin_ticks);
                    else add_release(ctrl + CTRL_DONE, 1);
                }
            }
            if (threadIdx.x == 0)
                s_ok = wait_ge(ctrl + CTRL_DONE, ctrl[CTRL_NWAIT], ctrl, p.spin_ticks, CTRL_TAIL_WAIT_TICKS);
            __syncthreads();
            if (s_ok) combine_task<8>(p, -1 - id);
        }
        issue();           // tasks without a main loop (tail, skipped, given up)
        __syncthreads();   // every thread has read s_task / s_ok of this round
        if (threadIdx.x == 0) s_task = fetch_finish(pf, ctrl, pass, home, exhausted, use_lists, use_tail);
        __syncthreads();
    }
    if (phase == -2) return;   // the kernel boundary publishes the rows
    if (publishes && !arrived) {   // ran out of work without seeing a tail task
        wait_stores();
        __syncthreads();
        if (threadIdx.x == 0) {
            if (phase < 0) worker_arrived(ctrl, home, ctrl[CTRL_NWAIT], p.spin_ticks);
            else add_release(ctrl + CTRL_DONE, 1);
        }
    }
}

// The combine as a plain grid launch for the default schedule: it follows the GEMM MegaKernel in
// stream order, so it needs no scoreboard wait, no task cursor and no LDS, and as many workgroups
// as fit share a CU.  A wave is one token by one round of columns: a generation step has too few
// tokens to fill the chip otherwise (32 tokens of width 2048 kept 2 CUs busy, four dependent
// rounds a wave: 198 -> 191 us for the layer; one token 35.8 -> 34.8 us; 256 tokens of width 7168
// 529 -> 518 us), and 8192 tokens gain a little as well (training step 2428 -> 2421 us).
template <int KM>
__global__ void __launch_bounds__(64 * kTailWaves) fwd_tail_kernel(FwdParams p, uint32_t first) {
    const uint32_t rounds = (p.s.d + kCombineCols - 1) / kCombineCols;
    const uint32_t id = first + rfl((int)blockIdx.x * kTailWaves + (int)(threadIdx.x >> 6));
    const int t = id / rounds, c0 = (id - t * rounds) * kCombineCols + (int)(threadIdx.x & 63) * 8;
    if (t >= p.s.T || c0 >= p.s.d) return;
    CombineSlots<KM> slots;
    slots.load(p, t);
    combine_piece<KM>(p, t, c0, slots);
}

// ------------------------------------------------------------------ host side

struct FwdLayout {
    size_t ctrl, flag1, tasks, h, o, total;
    int max_rt, nct1, nct2;   // (tiles of 128 rows)
    size_t max_tasks;
};

FwdLayout fwd_layout(const moe_shape_t& s, bool with_ho) {
    FwdLayout L;
    const size_t A_cap = (size_t)s.T * s.k;
    L.max_rt = (int)((A_cap + 127) / 128) + s.e_count;
    L.nct1 = (s.I + BN / 2 - 1) / (BN / 2);
    L.nct2 = (s.d + BN - 1) / BN;
    L.max_tasks = (size_t)L.max_rt * (L.nct1 + L.nct2) + (s.T + kCombineTokens - 1) / kCombineTokens;
    size_t off = 0;
    L.ctrl = off;  off = align_up(off + CTRL_WORDS * sizeof(int), 256);
    L.flag1 = off; off = align_up(off + ((size_t)L.max_rt + s.e_count) * sizeof(int), 256);   // (two an expert more than whole slots)
    L.tasks = off; off = align_up(off + L.max_tasks * sizeof(Task), 256);
    L.h = off;     if (with_ho) off = align_up(off + A_cap * s.I * 2, 256);
    L.o = off;     if (with_ho) off = align_up(off + A_cap * s.d * 2, 256);
    L.total = off;
    return L;
}

size_t fwd_workspace_bytes(const moe_shape_t& s) { return fwd_layout(s, true).total; }
size_t fwd_ctrl_bytes(const moe_shape_t& s) { return fwd_layout(s, false).total; }

// Resident worker slots per device: the one piece of process-wide state, filled on first use
// under a lock and constant afterwards.
static std::mutex g_workers_mu;
static int g_workers[kMaxDevices];

static int resident_workers(int* out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_workers_mu);
    if (g_workers[dev] == 0) {
        if (hipFuncSetAttribute((const void*)fwd_worker_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kMmaSmem) != hipSuccess)
            return MOE_ERR_HIP;
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fwd_worker_kernel, kMmaThreads,
                                                         kMmaSmem) != hipSuccess)
            return MOE_ERR_HIP;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return MOE_ERR_HIP;
        if (per_cu < 1 || cus < 1) return MOE_ERR_HIP;
        g_workers[dev] = per_cu * cus;
    }
    *out = g_workers[dev];
    return MOE_OK;
}

static void launch_tail(const FwdParams& p, hipStream_t st) {
    const size_t waves = (size_t)p.s.T * ((p.s.d + kCombineCols - 1) / kCombineCols);
    launch_tail_waves(waves, [&](dim3 grid, uint32_t first) {
        if (p.s.k <= 8)
            hipLaunchKernelGGL((fwd_tail_kernel<8>), grid, dim3(64 * kTailWaves), 0, st, p, first);
        else
            hipLaunchKernelGGL((fwd_tail_kernel<kMaxTopK>), grid, dim3(64 * kTailWaves), 0, st, p, first);
    });
}

static int fwd_launch_tiles(FwdParams& p, const moe_opts_t& opts, hipStream_t st) {
    int resident = 0;
    int rc = resident_workers(&resident);
    if (rc != MOE_OK) return rc;
    int workers = opts.workers > 0 ? min(opts.workers, resident) : resident;
    p.workers = workers;
    p.tile = TileChoice{TileChoice::rows_of(p.s, opts.tile_rows), p.nct1 + p.nct2, workers, 4};
    // A token selects an expert at most once, so up to kThinRows tokens no expert has more rows than
    // that: every expert is thin and no work queue is set up.
    const bool all_thin = p.s.T <= kThinRows;
    // Otherwise the counts decide, which only the device has.  But few or small experts never spare the queue enough
    // beside one with more rows, and there is one where the rows are more than kThinRows an expert and all experts are
    // here, or hardly ever none in a part of them with four times as many (the queue takes any counts).  Their launch
    // without work took 2 us (256 tokens on 8 experts of 512 x 1024 48.3 us, without it 46.3 us).  (Where the rule might send experts with medium
    // rows ahead, in layers of more than 128 experts, thin_may_pay is false only with one width at 64: such a layer keeps the queue for them.)
    const long long enough = (long long)kThinRows * p.s.E * (p.s.e_count == p.s.E ? 1 : 4);
    const bool none_thin = !all_thin && (long long)p.s.T * p.s.k > enough && !thin_may_pay(thin_rule(p.s, kThinRows), p.s);
    p.rule = thin_rule(p.s, all_thin ? INT_MAX : none_thin ? 0 : kThinRows);
    const size_t most = std::min<size_t>(p.s.e_count, (size_t)p.s.T * p.s.k);   // experts with rows
    // A caller's bound on the workers leaves the rest of the chip to somebody else: as many workgroups here.
    const size_t slots = workers < resident ? (size_t)workers : (size_t)kThinGroupsPerCu * resident;
    const size_t n1 = none_thin ? 0 : std::min(slots, most * (p.s.I / 32));
    const size_t n2 = std::min(slots, most * (p.s.d / 64));
    if (all_thin) {
        hipLaunchKernelGGL(thin_first_kernel, dim3((unsigned)n1), dim3(kThinThreads), 0, st, p);
        hipLaunchKernelGGL(thin_second_kernel, dim3((unsigned)n2), dim3(kThinThreads), 0, st, p);
        if (!opts.skip_tail || opts.schedule == 1 || opts.schedule == 2) launch_tail(p, st);
        return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
    }
    const bool two = thin_may_be_two(p.s);
    hipLaunchKernelGGL(two ? fwd_first_kernel<true> : fwd_first_kernel<false>, dim3((unsigned)(n1 + kPlanBlocks)), dim3(kThinThreads), 0, st, p);
    if (!none_thin)
        hipLaunchKernelGGL(two ? fwd_second_kernel<true> : fwd_second_kernel<false>, dim3((unsigned)n2), dim3(kThinThreads), 0, st, p);
    if (opts.schedule == 2) {
        for (int phase = 0; phase < 3; ++phase)
            hipLaunchKernelGGL(fwd_worker_kernel, dim3(workers), dim3(kMmaThreads), kMmaSmem, st, p, phase);
    } else if (opts.schedule != 1) {   // 0 (default) and 3: GEMM MegaKernel, then the tail tasks
        hipLaunchKernelGGL(fwd_worker_kernel, dim3(workers), dim3(kMmaThreads), kMmaSmem, st, p, -2);
        if (!opts.skip_tail) launch_tail(p, st);
    } else {
        hipLaunchKernelGGL(fwd_worker_kernel, dim3(workers), dim3(kMmaThreads), kMmaSmem, st, p, -1);
    }
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

int fwd_launch(const moe_shape_t& s, const void* x, const void* w_gate, const void* w_up,
               const void* w_down, const moe_routing_t& r, void* y, char* gu, char* h, char* o,
               char* ws, const moe_opts_t& opts, hipStream_t st) {
    const FwdLayout L = fwd_layout(s, false);
    FwdParams p;
    p.s = s;
    p.x = (const char*)x;
    p.w_gate = (const char*)w_gate;
    p.w_up = (const char*)w_up;
    p.w_down = (const char*)w_down;
    p.topk_w = r.topk_w;
    p.offsets = r.offsets;
    p.perm = r.perm;
    p.inv_perm = r.inv_perm;
    p.y = (char*)y;
    p.gu = gu;
    p.h = h;
    p.o = o;
    p.ctrl = (int*)(ws + L.ctrl);
    p.flag1 = (int*)(ws + L.flag1);
    p.tasks = (Task*)(ws + L.tasks);
    p.nct1 = L.nct1;
    p.nct2 = L.nct2;
    const int ms = opts.spin_limit_ms > 0 ? opts.spin_limit_ms : 2000;
    p.spin_ticks = (long long)ms * 100000ll;   // wall_clock64 ticks at 100 MHz
    return fwd_launch_tiles(p, opts, st);
}



}  // namespace uniep
