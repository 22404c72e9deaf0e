// The forward GEMMs of experts with few rows (a generation step, a short prompt, the cold experts
// of a skewed batch): the weights are read once and hardly reused, so the time is their stream
// from HBM and what a task costs before its first and after its last load.
//
// A workgroup is 4 waves and owns 128 weight columns (GEMM1: 64 gate columns and the same 64 up
// columns) of one expert, with all of its rows; the k axis is dealt to the waves in steps of 32
// and the four partial sums meet in LDS, added in wave order.  A lane loads 16 bytes (8 columns)
// of 8 consecutive k rows straight into registers, and 32 byte permutes turn them into the 8
// operands of v_mfma_f32_16x16x32_bf16 (one per column of the piece): no LDS staging, no barrier
// in the loop, and two steps (16 KB a wave) on their way at any time.
#pragma once
#include "mma.hpp"

namespace uniep {

constexpr int kThinRows = 32;       // rows up to which an expert takes this path
constexpr int kThinThreads = 256;
constexpr int kThinGroupsPerCu = 3;
constexpr int kThinCols = 128;      // weight columns of a task
constexpr int kThinPad = kThinCols + 4;   // floats between two rows of a partial sum: all 64 banks in both directions

struct ThinParams {
    moe_shape_t s;
    const char* x;
    const char* w_gate;
    const char* w_up;
    const char* w_down;
    const int32_t* offsets;
    const int32_t* perm;
    char* gu;
    char* h;
    char* o;
    int max_rows;    // experts with 1..max_rows rows are run here
};

// Where a lane's next step comes from.  The pointers are advanced in place and kept opaque:
// the compiler would otherwise carry one induction address per load and spill.
typedef const __attribute__((address_space(1))) char* glb_ptr_t;   // an opaque generic pointer would be read with flat loads
typedef const __attribute__((address_space(1))) u32x4_t* glb_vec_t;
template <int NR>
struct ThinSource {
    glb_ptr_t w;       // k row 8 (l / 16) of the step, this lane's 8 columns
    size_t ldw;          // bytes from one k row to the next (uniform)
    glb_ptr_t x[NR];     // row 16 f + l % 16, the same 8 k
    __device__ __forceinline__ void advance() {   // to this wave's next step, 4 steps on
        w += 128 * ldw;
        asm volatile("" : "+v"(w));
#pragma unroll
        for (int f = 0; f < NR; ++f) {
            x[f] += 256;
            asm volatile("" : "+v"(x[f]));
        }
    }
};

template <int NR>
struct ThinStep {
    u32x4_t w[8];
    u32x4_t x[NR];
    __device__ __forceinline__ void load(ThinSource<NR>& s) {
        const glb_ptr_t p = s.w;
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = __builtin_nontemporal_load((glb_vec_t)(p + j * s.ldw));
#pragma unroll
        for (int f = 0; f < NR; ++f) x[f] = *(glb_vec_t)s.x[f];
        s.advance();
    }
    // acc[f][c][v]: row 16 f + l % 16, column 32 (l / 16) + 8 v + c
    __device__ __forceinline__ void mma(f32x4_t (&acc)[NR][8]) const {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
            u32x4_t a;
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = __builtin_amdgcn_perm(w[2 * q + 1][c >> 1], w[2 * q][c >> 1], sel);
#pragma unroll
            for (int f = 0; f < NR; ++f)
                acc[f][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                                    __builtin_bit_cast(bf16x8_t, x[f]), acc[f][c], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);   // not all 32 permutes ahead of the first product: no registers for that
        }
    }
};

// n steps (4 apart) of this wave; the loads of one step ahead of the matrix work of another
template <int NR>
__device__ __forceinline__ void thin_loop(ThinSource<NR>& src, int n, f32x4_t (&acc)[NR][8]) {
#pragma unroll
    for (int f = 0; f < NR; ++f)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            acc[f][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+v"(acc[f][c]));   // one copy, whatever the number of steps
        }
    if (n <= 0) return;
    ThinStep<NR> a, b;
    a.load(src);
    int i = 0;
    for (; i + 2 < n; i += 2) {
        b.load(src);
        __builtin_amdgcn_sched_barrier(0);
        a.mma(acc);
        __builtin_amdgcn_sched_barrier(0);
        a.load(src);
        __builtin_amdgcn_sched_barrier(0);
        b.mma(acc);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (i + 1 < n) {
        b.load(src);
        __builtin_amdgcn_sched_barrier(0);
        a.mma(acc);
        a = b;
    }
    a.mma(acc);
}

// One block of up to 16 NR rows (row0 .., `rows` valid) by the task's columns.
// GEMM 1: h = silu(x W_gate) * (x W_up), columns [64 ct, +64); GEMM 2: o = h W_down, columns [128 ct, +128).
template <int GEMM, int NR>
__device__ __forceinline__ void thin_block(const ThinParams& p, int e, int ct, int row0, int rows, float* red) {
    const int d = p.s.d, I = p.s.I;
    const Lane in;
    const int n = in.l & 15, q = in.l >> 4, w = in.wave_uniform();
    const int K = GEMM == 1 ? d : I;
    ThinSource<NR> src;
    src.ldw = (size_t)(GEMM == 1 ? I : d) * 2;
    const char* wp;
    if (GEMM == 1) {
        wp = (n & 8 ? p.w_up : p.w_gate) + (size_t)e * d * src.ldw + (size_t)(64 * ct + 8 * (n & 7)) * 2;
    } else {   // pieces past d alias the last one
        wp = p.w_down + (size_t)e * I * src.ldw + (size_t)min(kThinCols * ct + 8 * n, d - 8) * 2;
    }
    src.w = (glb_ptr_t)(wp + (size_t)(32 * w + 8 * q) * src.ldw);
#pragma unroll
    for (int f = 0; f < NR; ++f) {
        const int r = row0 + min(16 * f + n, rows - 1);   // rows past the last alias it
        const char* row = GEMM == 1 ? p.x + (size_t)(p.perm[r] / p.s.k) * d * 2 : p.h + (size_t)r * I * 2;
        src.x[f] = (glb_ptr_t)(row + 64 * w + 16 * q);
    }
    f32x4_t acc[NR][8];
    thin_loop<NR>(src, (K / 32 - w + 3) / 4, acc);

    const Lane out;
    const int tr = out.tid >> 4, tc = out.tid & 15;   // on the way out: row of the fragment, piece of its columns
#pragma unroll
    for (int f = 0; f < NR; ++f) {
        __syncthreads();   // the partial sums of the fragment before (or of the task before) have been read
        float* mine = red + (out.w * 16 + (out.l & 15)) * kThinPad + 32 * (out.l >> 4);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            *(f32x4_t*)(mine + 8 * v) = f32x4_t{acc[f][0][v], acc[f][1][v], acc[f][2][v], acc[f][3][v]};
            *(f32x4_t*)(mine + 8 * v + 4) = f32x4_t{acc[f][4][v], acc[f][5][v], acc[f][6][v], acc[f][7][v]};
        }
        __syncthreads();
        const int c0 = GEMM == 1 ? 4 * tc : 8 * tc, c1 = GEMM == 1 ? 64 + 4 * tc : 8 * tc + 4;
        f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            const float* src = red + (ww * 16 + tr) * kThinPad;
            s0 += *(const f32x4_t*)(src + c0);
            s1 += *(const f32x4_t*)(src + c1);
        }
        const int r = 16 * f + tr;
        if (r < rows) {
            const size_t row = (size_t)(row0 + r);
            if (GEMM == 1) {
                const int col = 64 * ct + 4 * tc;
                if (p.gu) {
                    char* g = p.gu + (row * 2 * I + col) * 2;
                    __builtin_nontemporal_store(u32x2_t{pack_bf16x2(s0[0], s0[1]), pack_bf16x2(s0[2], s0[3])}, (u32x2_t*)g);
                    __builtin_nontemporal_store(u32x2_t{pack_bf16x2(s1[0], s1[1]), pack_bf16x2(s1[2], s1[3])},
                                                (u32x2_t*)(g + (size_t)I * 2));
                }
                float hv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) hv[j] = s0[j] * sigmoid_f(s0[j]) * s1[j];
                *(u32x2_t*)(p.h + (row * I + col) * 2) = u32x2_t{pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3])};
            } else {
                const int col = kThinCols * ct + 8 * tc;
                if (col < d)
                    *(u32x4_t*)(p.o + (row * d + col) * 2) =
                        u32x4_t{pack_bf16x2(s0[0], s0[1]), pack_bf16x2(s0[2], s0[3]), pack_bf16x2(s1[0], s1[1]),
                                pack_bf16x2(s1[2], s1[3])};
            }
        }
    }
}

struct ThinShared {
    float red[4 * 16 * kThinPad];
    int32_t row0[kMaxExperts];
    int32_t rows[kMaxExperts];
    uint16_t expert[kMaxExperts];
    int32_t wave[4];
};

// Workgroup `block` of `blocks` (a multiple of 8, unless there are fewer tasks): it finds the
// experts of this path by itself (their row counts come from the offsets) and takes every
// `blocks`-th task.  Workgroups go to the XCDs in turn, so for as many experts as fill all eight
// the tasks of one expert share an XCD (its rows are then fetched by one L2); what is left over
// is spread task by task.
template <int GEMM>
__device__ __forceinline__ void thin_run(const ThinParams& p, int block, int blocks, ThinShared& S) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ec = p.s.e_count;
    int off[5], mine = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) off[j] = p.offsets[min(4 * tid + j, ec)];
#pragma unroll
    for (int j = 0; j < 4; ++j) mine += (off[j + 1] > off[j] && off[j + 1] - off[j] <= p.max_rows) ? 1 : 0;
    int pre = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(pre, o);
        if (lane >= o) pre += v;
    }
    if (lane == 63) S.wave[wave] = pre;
    __syncthreads();
    int at = pre - mine, count = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) at += S.wave[w];
        count += S.wave[w];
    }
    if (count == 0) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (off[j + 1] > off[j] && off[j + 1] - off[j] <= p.max_rows) {
            S.expert[at] = (uint16_t)(4 * tid + j);
            S.row0[at] = off[j];
            S.rows[at] = off[j + 1] - off[j];
            ++at;
        }
    __syncthreads();
    const int nct = GEMM == 1 ? p.s.I / 64 : (p.s.d + kThinCols - 1) / kThinCols;
    const int even = (count & ~7) * nct;
    for (int id = block; id < count * nct; id += blocks) {
        int x, ct;
        if (id < even) {
            const int slot = id >> 3;
            x = (slot / nct) * 8 + (id & 7);
            ct = slot % nct;
        } else {
            x = (count & ~7) + (id - even) / nct;
            ct = (id - even) % nct;
        }
        const int e = rfl(S.expert[x]), row0 = rfl(S.row0[x]), rows = rfl(S.rows[x]);
        for (int r = 0; r < rows; r += kThinRows) {   // more than one round only where max_rows is larger
            const int left = min(rows - r, kThinRows);
            if (left <= 16) thin_block<GEMM, 1>(p, e, ct, row0 + r, left, S.red);
            else thin_block<GEMM, 2>(p, e, ct, row0 + r, left, S.red);
        }
    }
}

}  // namespace uniep
