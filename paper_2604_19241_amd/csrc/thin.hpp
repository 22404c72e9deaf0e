// The forward GEMMs of experts with few rows (a generation step, a short prompt, the cold experts
// of a skewed batch): the weights are read once and hardly reused, so the time is their stream
// from HBM and what a task costs before its first and after its last load.
//
// A workgroup is 4 waves and owns 256, 128 or 64 weight columns (GEMM1: half of them gate columns, the other half the same up
// columns) of one expert, with all of its rows.  K advances in stages of 64.  A stage is loaded into
// registers (a wave: 16 k rows of the weights and 8 rows of activations, 16 bytes a lane and load), two or four stages
// ahead, and passes through one of two LDS images; one barrier a stage.  Loads to registers and not the DMA of the big
// tiles: the loads of several stages are on their way at any time.
//
// HBM delivers 256-byte runs of a k row faster than 128-byte ones wherever the rows lie a multiple of 1024 bytes apart (a
// plain read of 512 experts of 2048 x 512, gate and up, 6.2 and 5.2 TB/s; 32 of 7168 x 2048 6.2 and 5.4), and a longer task has fewer
// beginnings: 256 columns where they fill the chip (thin_cols).
//
// Every output is ONE chain of v_mfma_f32_32x32x16_bf16 in ascending k, weights as the A operand,
// with the same k in the same lane and element as in the 256-row tiles (mma.hpp): a row's results
// are bit for bit those of the work queue, so they do not depend on how many rows its expert has, i.e.
// on what else is in the batch.  That rules out a split of the k axis over waves: a wave multiplies
// one fragment of 32 columns (two of 256) of the task over the whole k axis.  Measured against a form that dealt the k axis to the
// four waves and added four partial sums (no LDS image, no barrier): 32 tokens of width 2048 on 128 experts of
// inner width 768 185 -> 183 us for the layer, 1021 tokens on 512 experts of 512 728 -> 718 us, one token
// 33.8 -> 33.6 us; and against 256-row tiles for these experts 258 -> 190, 755 -> 705 and 82 -> 34 us.
#pragma once
#include "mma.hpp"

namespace uniep {

// Rows up to which an expert has few: one fragment of the matrix instruction.  Experts with up to kThinMostRows, two fragments that share
// the weights, may take this path too (ThinRule::limit).  More would be blocks of 32, each
// with the weights again.  128 experts of 2048 x 768 with 16 / 32 rows each 206 / 213 us, on the queue 239 / 244 us, with
// 40 on the queue 245 us (in two blocks 419 us, with tasks of 128 columns); 16 of 2048 x 1408 55 / 56 us, on the queue
// 81 / 81 us, with 40 82 us (106 us).
constexpr int kThinRows = 32;
constexpr int kThinThreads = 256;
constexpr int kThinGroupsPerCu = 2;   // as many as the LDS holds (80 KB each)
constexpr int kThinXBytes = kThinRows * BK * 2;                       // rows of a stage: image [32 rows][128 B]
constexpr int kThinMostImage = BK * 256 * 2 + kThinXBytes;
constexpr int kThinMostRows = 2 * kThinRows;
// Weight columns of a task where `experts` of them have `columns` each, on `cus` CUs.  A CU draws some 57 GB/s from HBM
// at most, whatever it has on its way (its L1 holds 32 KB of lines in flight), so that the time is the tasks of the CU that
// has most of them; a task of 128 columns takes 0.58 of one of 256, one of 64 (runs of 64 bytes) 0.42.  Measured, us of the
// layer with 128 columns everywhere / with this rule (tokens, experts of width and inner width): 1021, 512 of 2048 x 512 690 / 624;
// 256, 32 of 7168 x 2048 506 / 459; 300, 256 of 2304 x 1024 677 / 608; 32, 128 of 2048 x 768 192 / 180; 20, 32 of
// 7168 x 2048 251 / 225; 1, 128 of 2048 x 768 34.2 / 32.0; 1, 8 of 4096 x 14336 184 / 150.  With 256 columns everywhere: 1 token
// 46.9 and 229, 3 tokens on 128 experts of 4096 x 1536 189 us for 177; with 64 32 tokens 258 us.
__device__ __forceinline__ int thin_cols(int experts, int columns, int cus) {
    auto cost = [&](int width, int weight) { return (experts * ((columns + width - 1) / width) + cus - 1) / cus * weight; };
    const int wide = cost(256, 100), mid = cost(128, 58), narrow = cost(64, 42);
    return wide <= min(mid, narrow) ? 256 : mid <= narrow ? 128 : 64;
}
// NR: blocks of 32 rows
template <int NC, int NR>
struct ThinShape {
    static constexpr int kRow = NC * 2;              // bytes of a k row in the weights' image [64 k][kRow]
    static constexpr int kW = BK * kRow;
    static constexpr int kImage = kW + NR * kThinXBytes;
    static_assert(kImage <= kThinMostImage, "");
    static constexpr int kLoads = NC / 32;           // of a wave and stage, 1 KB each
    static constexpr int kFrags = NC == 256 ? 2 : 1; // column fragments of a wave; of 64 columns waves 2 and 3 have none
    static constexpr int kAhead = NC == 256 ? 2 : 4; // stages in flight (even: stage t is in registers t % kAhead and in image t % 2)
};

// Whether the experts with few rows leave the queue.  Both paths give the same bits, so this is a matter of time
// alone: the two launches of this path stand in front of the queue's, one after the other, and add their latency
// where the queue would have had CUs to spare for the same experts.  In whole numbers and from the counts alone,
// so that every workgroup of a pass comes to the same answer by itself.  It pays
//  - where no expert has more rows: nothing is left for the queue (8 experts of 2048 x 1408 with 10 rows each 36 us,
//    on the queue 70 us; 128 of 2048 x 768 with 4 rows each 191 and 223 us; 512 of 2048 x 512 with 2 521 and 560 us);
//  - where nearly all have few or the others are bound by matrix work, and the queue is spared more time than this path
//    takes.  The queue takes no less than a chain of GEMM1 and GEMM2 stages of 1 us each, else 30 us and the weights
//    at 5.2 TB/s; this path 20 us and 6.4 TB/s (117 experts of 2048 x 768 with few rows beside 8 with 1900 each 350 us,
//    on the queue 364 us; 112 beside 16 with 2000 each 510 and 525 us).
// It did not pay for 13 experts of 2048 x 1408 beside 3 with more rows (124 and 93 us, now 81 us on the queue), 14 beside 2 of
// 2048 x 768 (83 and 65 us), 43 beside 19 of 5120 x 1536 (749 and 687 us, now 527), 3 beside 5 of 4096 x 14336 (835 and 746 us, now 565).
// The second line is from before the queue's low tiles kept two stages on their way (mma_low), and the queue would now be
// the faster of the two in most of what lies on this side of it: 58 beside 4 with 2000 rows of 5120 x 1536 960 us, on the queue 790 us,
// 28 beside 4 with 800 of 7168 x 2048 822 and 678 us, 95 beside one with 33 of 2048 x 768 192 and 179 us, 63 beside 38 with
// 800 each 435 and 428 us.  Of 402 combinations of eight layers that the rule sends ahead of it the queue takes more
// than 1 % less in 335 (half of all 4 % less or better, at best 22 %) and more than 1 % more in 20 (at most 4 %).
struct ThinRule {
    static constexpr int kOftenMedium = 128;
    int max_rows;              // an expert has few rows up to here
    // Up to so many experts with more rows have so many that matrix work bounds them: 512 rows each, of those that even routing
    // gives the experts here, but no more than there are.  (A share with few of the tokens' rows was taken for one with many: 19
    // experts of 5120 x 1536 with 60 rows beside 43 with 10, 40000 tokens elsewhere, 579 us, now on the queue 517 us; 8 of 7168 x
    // 2048 with 50 beside 24 with 20, 64000 elsewhere, 547 -> 490 us.)
    int many_most;
    long long chain_ns;
    int queue_ns, thin_ns;     // an expert's weights
    int full_ns, medium_ns;    // the same where no expert has more than medium rows
    __host__ __device__ __forceinline__ long long queue(int experts) const {
        const long long stream = 30000 + (long long)experts * queue_ns;
        return stream > chain_ns ? stream : chain_ns;
    }
    __device__ __forceinline__ bool pays(int few, int many, int rows) const {
        if (many == 0) return true;
        if (few < 8 * many && many > min(many_most, rows / 512)) return false;
        return queue(few + many) - queue(many) > 20000 + (long long)few * thin_ns;
    }
    // 0: up to max_rows rows, 1 (TWO): medium, up to kThinMostRows, 2: more
    template <bool TWO>
    __device__ __forceinline__ int size_class(int rows) const { return rows <= max_rows ? 0 : TWO && max_rows > 0 && rows <= kThinMostRows ? 1 : 2; }
    // Rows up to which an expert of this batch takes this path (0 = none does); experts with few, medium and more rows,
    // and the rows of all of them.
    // Where no expert has more than medium rows and there are more than kOftenMedium experts, all of them take this path if that is
    // the faster way for them together: tasks of two blocks of rows (128 columns) stream the weights at 4.5 TB/s, the queue takes 30 us and
    // 5.4 TB/s and 50 ns an expert.  Measured, us of the layer, with medium experts on the queue / here (experts of width and inner width, with few + medium
    // rows): 512 of 2048 x 512, 477 + 35 624 / 590, 280 + 232 633 / 599, 93 + 419 637 / 662; 256 of 2304 x 1024, 250 + 6 665 / 648, 192 + 64 675 / 645,
    // 76 + 128 557 / 596, 0 + 256 707 / 770; 160 of 5120 x 1536, 144 + 16 1348 / 1300, 46 + 80 1067 / 1150; 256 of 7168 x 2048, 192 + 64 3834 / 3665, 18 + 230
    // 3876 / 4308.  Of 462 batches of 18 layers the estimate sends 322 here, half of them 4 % faster or more, 6 more than 1 % slower (at most 4 %); of the others 17
    // would be more than 1 % faster (at most 7 %).  (At 5.0 and 5.5 TB/s and no time an expert it sent 18 here that were slower, by up to 7 %.)
    // Beside an expert with more than medium rows the queue keeps them all: of 90 batches of five layers with 1 to 32 such experts 59 were more than 1 % slower
    // with the medium ones here, 5 faster, the middle one 2 % slower (512 of 2048 x 512, one with 300 rows, 154 medium 636 / 660; 256 of 2304 x 1024, 8 with 200, 77 medium 675 / 731; 160 of 1024 x 384,
    // 2 with 100, 48 medium 111 / 118; the best one 139 on the queue, 132 here).
    // Fewer experts would often gain as well (512 tokens on 128 of 1024 x 384, 24 rows each, 96 / 71; 500 on 128 of 2048 x 768, 31 rows,
    // 247 / 232; 250 on 64 of 2048 x 1408, 23 rows, 229 / 202): they keep the choice that is tested for them.
    __device__ __forceinline__ int limit(int few, int medium, int more, int rows) const {
        if (more == 0 && medium > 0 && few + medium > kOftenMedium) {
            const long long stream = 30000 + (long long)(few + medium) * full_ns;
            const long long here = 20000 + (long long)few * thin_ns + (long long)medium * medium_ns;
            if (here < (stream > chain_ns ? stream : chain_ns)) return kThinMostRows;
        }
        return pays(few, medium + more, rows) ? max_rows : 0;
    }
};
inline ThinRule thin_rule(const moe_shape_t& s, int max_rows) {
    const long long bytes = 6ll * s.d * s.I;
    return ThinRule{max_rows, (int)((long long)s.T * s.k * s.e_count / s.E / 512), 1000ll * ((s.d + s.I) / BK),
                    (int)(bytes / 5200), (int)(bytes / 6400), (int)(bytes / 5400) + 50, (int)(bytes / 4500)};
}
// Whether the rule may send experts with medium rows here, whatever the counts.
inline bool thin_may_be_two(const moe_shape_t& s) { return s.e_count > ThinRule::kOftenMedium; }
// Whether it can pay beside an expert with many rows, whatever the counts.
inline bool thin_may_pay(const ThinRule& r, const moe_shape_t& s) { return r.queue(s.e_count) - r.chain_ns > 20000; }

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
    ThinRule rule;
    int workers;   // CUs that the launch may fill
};

typedef const __attribute__((address_space(1))) u32x4_t* glb_vec_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((address_space(3))) char* lds_ptr_t;
typedef __attribute__((address_space(3))) u32x4_t* lds_vec_t;
typedef __attribute__((address_space(3))) bf16x4_t* lds_tr_t;

// Where a wave's next stage comes from.  GEMM1: the first half of the weight loads are gate columns, the second the same up
// columns; a load is kRows k rows of kLanes lanes.
template <int GEMM, int NC, int NR>
struct ThinSource {
    static constexpr int kLoads = ThinShape<NC, NR>::kLoads;
    static constexpr int kLanes = GEMM == 1 ? NC / 16 : NC / 8, kRows = 64 / kLanes;
    static constexpr int kOf = GEMM == 1 ? kLoads / 2 : kLoads;   // loads of a matrix
    glb_ptr_t w[2];      // first k row of this wave in the stage to come (uniform); GEMM2: w[0] only
    uint32_t off;        // this lane's k row and columns behind it
    uint32_t ldw;        // bytes from one k row to the next (uniform)
    glb_ptr_t x[NR];     // this lane's rows and chunk
    // advance: 0 = stay on this stage (the last one).  The loads are never left out: behind a branch
    // around them the compiler could not tell how many are in flight and would wait for all.
    __device__ __forceinline__ void load(u32x4_t (&r)[kLoads + NR], int advance) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            glb_ptr_t base = w[i / kOf] + (size_t)(kRows * (i % kOf)) * ldw;
            asm volatile("" : "+s"(base));   // scalar base + 32-bit lane offset, not one 64-bit lane address per load
            r[i] = __builtin_nontemporal_load((glb_vec_t)(base + off));
        }
#pragma unroll
        for (int n = 0; n < NR; ++n) r[kLoads + n] = *(glb_vec_t)x[n];
        const size_t step = (size_t)(BK * advance) * ldw;
        w[0] += step;
        if (GEMM == 1) w[1] += step;
#pragma unroll
        for (int n = 0; n < NR; ++n) x[n] += BK * 2 * advance;
    }
};

// The LDS images: weights, 16-byte chunk c of k row k at c ^ swz(k) (the bank bits that the chunks and, of 64 columns, the k rows
// of a fragment read leave free); rows, chunk c of row r at c ^ ((r >> 1) & 7).  Chunks 4 f .. 4 f + 3 of a k row are fragment f's
// 32 columns (GEMM1: 16 gate columns, then the same 16 up columns).
template <int GEMM, int NC, int NR>
struct ThinLds {
    using S = ThinShape<NC, NR>;
    using Src = ThinSource<GEMM, NC, NR>;
    lds_ptr_t wput[2], xput, wget[S::kFrags], xget[4];
    static __device__ __forceinline__ int swz(int k) { return NC == 64 ? (k & 2) << 1 : (k & 3) << 2; }
    __device__ __forceinline__ ThinLds(lds_ptr_t base, const Lane& ln) {
        const int l = ln.l, w = ln.w, kh = ln.hf, g = (l >> 4) & 1, e = (l & 15) >> 2, q = l & 3;
        const int kr = l / Src::kLanes, p = l % Src::kLanes, c = GEMM == 1 ? 4 * (p >> 1) + (p & 1) : p;
#pragma unroll
        for (int i = 0; i < 2; ++i)   // loads with i even and odd: only two k rows a load make a difference
            wput[i] = base + (16 * w + kr) * S::kRow + ((c ^ swz(kr + (Src::kRows == 2 ? 2 * i : 0))) << 4);
        const int row = 8 * w + (l >> 3);
        xput = base + S::kW + row * 128 + (((l & 7) ^ ((row >> 1) & 7)) << 4);
        const int sq = ((q & 1) << 1) | (q >> 1);   // piece -> position of its 4 columns inside the 16
#pragma unroll
        for (int f = 0; f < S::kFrags; ++f)
            wget[f] = base + (8 * kh + e) * S::kRow + (((4 * (S::kFrags * (NC == 64 ? w & 1 : w) + f) + 2 * g + (sq >> 1)) ^ swz(e)) << 4) +
                      (sq & 1) * 8;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            xget[kk] = base + S::kW + ln.l31 * 128 + (((2 * kk + kh) ^ ((ln.l31 >> 1) & 7)) << 4);
    }
    __device__ __forceinline__ void put(int image, const u32x4_t (&r)[S::kLoads + NR]) const {
#pragma unroll
        for (int i = 0; i < S::kLoads; ++i)
            *(lds_vec_t)(wput[i & 1] + image * S::kImage + (i % Src::kOf) * Src::kRows * S::kRow + (i / Src::kOf) * 32) = r[i];
#pragma unroll
        for (int n = 0; n < NR; ++n) *(lds_vec_t)(xput + image * S::kImage + n * kThinXBytes) = r[S::kLoads + n];
    }
    // acc[f][v]: row l % 32, column position 16 (v / 8) + 8 (l / 32) + v % 8 of the wave's f-th 32
    __device__ __forceinline__ void multiply(int image, f32x16_t (&acc)[NR][S::kFrags]) const {
        bf16x4_t lo[S::kFrags][4], hi[S::kFrags][4];
        u32x4_t b[NR][4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int n = 0; n < NR; ++n) b[n][kk] = *(lds_vec_t)(xget[kk] + image * S::kImage + n * kThinXBytes);
#pragma unroll
            for (int f = 0; f < S::kFrags; ++f) {
                const lds_ptr_t a = wget[f] + image * S::kImage + kk * 16 * S::kRow;
                lo[f][kk] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)a);
                hi[f][kk] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)(a + 4 * S::kRow));
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // all reads on their way before the first product: one latency a stage, not four
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int f = 0; f < S::kFrags; ++f)
#pragma unroll
                for (int n = 0; n < NR; ++n)
                    acc[n][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(lo[f][kk], hi[f][kk], 0, 1, 2, 3, 4, 5, 6, 7),
                                                                        __builtin_bit_cast(bf16x8_t, b[n][kk]), acc[n][f], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// LDS writes of this wave done, then all waves: what __syncthreads() does without its wait for the
// loads in flight.
__device__ __forceinline__ void thin_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One stage: registers -> image, the loads of the stage kAhead further on into the same registers,
// barrier, matrix work.  An image is written again two stages later, behind the barrier that every wave
// reaches with its reads of it done.
template <int GEMM, int NC, int NR, bool LOAD>
__device__ __forceinline__ void thin_stage(ThinSource<GEMM, NC, NR>& src, const ThinLds<GEMM, NC, NR>& lds, int image,
                                           u32x4_t (&r)[ThinShape<NC, NR>::kLoads + NR], f32x16_t (&acc)[NR][ThinShape<NC, NR>::kFrags], int advance) {
    lds.put(image, r);
    __builtin_amdgcn_sched_barrier(0);
    if (LOAD) src.load(r, advance);
    thin_barrier();
    lds.multiply(image, acc);
}

// n >= 1 stages: t is in registers t % kAhead and in image t % 2.
template <int GEMM, int NC, int NR>
__device__ __forceinline__ void thin_loop(ThinSource<GEMM, NC, NR>& src, const ThinLds<GEMM, NC, NR>& lds, int n, f32x16_t (&acc)[NR][ThinShape<NC, NR>::kFrags]) {
    constexpr int kAhead = ThinShape<NC, NR>::kAhead;
#pragma unroll
    for (int n = 0; n < NR; ++n)
#pragma unroll
        for (int f = 0; f < ThinShape<NC, NR>::kFrags; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][f][v] = 0.f;
    u32x4_t r[kAhead][ThinShape<NC, NR>::kLoads + NR];
    thin_barrier();   // the task before has read its last image
#pragma unroll
    for (int j = 0; j < kAhead; ++j) src.load(r[j], j + 1 < n ? 1 : 0);
    int t = 0;
    for (; t + kAhead < n; t += kAhead)
#pragma unroll
        for (int j = 0; j < kAhead; ++j)
            thin_stage<GEMM, NC, NR, true>(src, lds, j & 1, r[j], acc, t + j + 1 + kAhead < n ? 1 : 0);
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
        if (t + j < n) thin_stage<GEMM, NC, NR, false>(src, lds, j & 1, r[j], acc, 0);
}

// Up to 32 NR rows (row0 .., `rows` valid) by the task's columns.
// GEMM 1: h = silu(x W_gate) * (x W_up), columns [NC/2 ct, +NC/2); GEMM 2: o = h W_down, columns [NC ct, +NC).
template <int GEMM, int NC, int NR>
__device__ __forceinline__ void thin_block(const ThinParams& p, int e, int ct, int row0, int rows, lds_ptr_t images) {
    constexpr int kFrags = ThinShape<NC, NR>::kFrags;
    const int d = p.s.d, I = p.s.I;
    f32x16_t acc[NR][kFrags];
    {
        const Lane in;
        const int K = GEMM == 1 ? d : I, n = GEMM == 1 ? I : d;
        ThinSource<GEMM, NC, NR> src;
        src.ldw = (uint32_t)n * 2;
        const size_t first = ((size_t)e * K + 16 * in.wave_uniform()) * src.ldw;
        src.w[0] = (glb_ptr_t)((GEMM == 1 ? p.w_gate : p.w_down) + first);
        src.w[1] = (glb_ptr_t)((GEMM == 1 ? p.w_up : p.w_down) + first);
        // pieces past the last column alias it
        src.off = (in.l / src.kLanes) * src.ldw + (uint32_t)min((GEMM == 1 ? NC / 2 : NC) * ct + 8 * (in.l % src.kLanes), n - 8) * 2;
#pragma unroll
        for (int b = 0; b < NR; ++b) {
            const int r = row0 + min(32 * b + 8 * in.w + (in.l >> 3), rows - 1);   // rows past the last alias it
            const char* row = GEMM == 1 ? p.x + (size_t)(p.perm[r] / p.s.k) * d * 2 : p.h + (size_t)r * I * 2;
            src.x[b] = (glb_ptr_t)(row + (in.l & 7) * 16);
        }
        thin_loop<GEMM, NC, NR>(src, ThinLds<GEMM, NC, NR>(images, in), K / BK, acc);
    }
    const Lane out;
    if (NC == 64 && out.w >= 2) return;
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        if (32 * n + out.l31 >= rows) return;
        const size_t row = (size_t)(row0 + 32 * n + out.l31);
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            if (GEMM == 1) {
                const int col = NC / 2 * ct + 16 * (kFrags * out.w + f) + 8 * out.hf;
                if (NC == 256 && col >= I) continue;
                if (p.gu) {
                    *(u32x4_t*)(p.gu + (row * 2 * I + col) * 2) = pack8(acc[n][f], 0);
                    *(u32x4_t*)(p.gu + (row * 2 * I + I + col) * 2) = pack8(acc[n][f], 1);
                }
                float hv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float g = acc[n][f][j], u = acc[n][f][8 + j];
                    hv[j] = g * sigmoid_f(g) * u;
                }
                *(u32x4_t*)(p.h + (row * I + col) * 2) = u32x4_t{pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3]),
                                                                 pack_bf16x2(hv[4], hv[5]), pack_bf16x2(hv[6], hv[7])};
            } else {
                const int col = NC * ct + 32 * (kFrags * out.w + f) + 8 * out.hf;
#pragma unroll
                for (int vg = 0; vg < 2; ++vg)
                    if (col + 16 * vg < d) *(u32x4_t*)(p.o + (row * d + col + 16 * vg) * 2) = pack8(acc[n][f], vg);
            }
        }
    }
}

struct ThinShared {
    union {
        __attribute__((aligned(512))) char images[2 * kThinMostImage];
        int32_t wave[2][4];        // of the search, before the first image
    };
    int32_t row0[kMaxExperts];
    uint16_t rows[kMaxExperts];    // (up to 32 tokens of 16 slots each, were they all of one expert)
    uint16_t expert[kMaxExperts];
};
static_assert(kThinGroupsPerCu * sizeof(ThinShared) <= 160 * 1024, "");

// The tasks of `count` listed experts from the `first`-th on, every `blocks`-th from `block` on.
template <int GEMM, int NC, int NR>
__device__ __forceinline__ void thin_tasks(const ThinParams& p, int first, int count, int block, int blocks, ThinShared& S) {
    const int nct = GEMM == 1 ? (2 * p.s.I + NC - 1) / NC : (p.s.d + NC - 1) / NC;
    const int even = (count & ~7) * nct;
    for (int id = block; id < count * nct; id += blocks) {
        int x, ct;
        if (id < even) {
            const int slot = id >> 3;
            x = (slot / nct) * 8 + (id & 7);
            ct = slot % nct;
        } else {
            int t = id - even;
            // Two tasks that share 128-byte lines (64 columns, half of them gate columns) go to one XCD, eight ids apart: apart, each L2
            // fetched the lines for itself (one row on 4 experts of 7168 x 2048 111 -> 86 us, with 128 columns 88 us).
            if (GEMM == 1 && NC == 64 && (t | 15) < (count & 7) * nct) t = (t & ~15) + 2 * (t & 7) + ((t >> 3) & 1);
            x = (count & ~7) + t / nct;
            ct = t % nct;
        }
        x += first;
        const int e = rfl(S.expert[x]), row0 = rfl(S.row0[x]), rows = rfl(S.rows[x]);
        for (int r = 0; r < rows; r += NR * kThinRows)   // more than one round only where max_rows is larger
            thin_block<GEMM, NC, NR>(p, e, ct, row0 + r, min(rows - r, NR * kThinRows), (lds_ptr_t)S.images);
    }
}

// Workgroup `block` of `blocks` (a multiple of 8, unless there are fewer tasks or the caller bounds the
// workers): it finds the experts of this path by itself (their row counts come from the offsets) and takes
// every `blocks`-th task.  Workgroups go to the XCDs in turn, so for as many experts as fill all eight
// the tasks of one expert share an XCD (its rows are then fetched by one L2); what is left over
// is spread task by task.
// kThinAll: every expert is of this path, whatever its rows, and the choices above are left out (one token on 128 experts of 2048 x 768, 8 selected,
// 31.5 -> 31.0 us).  kThinTwo: experts may have two blocks of rows here.  The code for these costs 0.2 to 0.7 us a launch, 2 % of a
// small share's layer, where the rule never sends them here (300 tokens on 16 of 128 of 1024 x 384 20.3 us, with it 21.1; 128 on 16 of 128 of 2048 x 768
// 36.8 and 37.9; 300 on 8 of 64 of 1280 x 896 52.9 and 53.6).
enum ThinForm { kThinAll, kThinFew, kThinTwo };
template <int GEMM, ThinForm FORM>
__device__ __forceinline__ void thin_run(const ThinParams& p, int block, int blocks, ThinShared& S) {
    constexpr bool ALL = FORM == kThinAll, TWO = FORM == kThinTwo;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ec = p.s.e_count;
    const int rows_here = ALL ? 0 : p.offsets[ec];
    int off[5], mine = 0, more = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) off[j] = p.offsets[min(4 * tid + j, ec)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // few and, shifted left by 16, medium (without those: more) rows
        const int rows = off[j + 1] - off[j], c = ALL ? 0 : p.rule.size_class<TWO>(rows);
        mine += rows <= 0 ? 0 : c == 0 ? 1 : c == 1 || !TWO ? 1 << 16 : 0;
        if (TWO) more += __popcll(__ballot(c == 2));
    }
    int pre = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(pre, o);
        if (lane >= o) pre += v;
    }
    if (lane == 63) {
        S.wave[0][wave] = pre;
        if (TWO) S.wave[1][wave] = more;
    }
    __syncthreads();
    int at = pre - mine, count = 0;
    more = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) at += S.wave[0][w];
        count += S.wave[0][w];
        if (TWO) more += S.wave[1][w];
    }
    const int few = rfl(count & 0xffff), rest = rfl((uint32_t)count >> 16);
    const int limit = ALL ? INT_MAX : TWO ? p.rule.limit(few, rest, rfl(more), rfl(rows_here)) : p.rule.limit(few, 0, rest, rfl(rows_here));
    const int two = TWO && limit == kThinMostRows ? rest : 0;   // experts with two blocks of rows here
    if (limit == 0 || few + two == 0) return;
    int at_few = at & 0xffff, at_two = few + (int)((uint32_t)at >> 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int rows = off[j + 1] - off[j];
        if (rows > 0 && rows <= limit) {
            const int i = !TWO || p.rule.size_class<TWO>(rows) == 0 ? at_few++ : at_two++;
            S.expert[i] = (uint16_t)(4 * tid + j);
            S.row0[i] = off[j];
            S.rows[i] = (uint16_t)rows;
        }
    }
    __syncthreads();
    const int columns = GEMM == 1 ? 2 * p.s.I : p.s.d;
    if constexpr (TWO) {
        if (two > 0) {   // the longer tasks first; who has had one more of them gets one less of the others
            thin_tasks<GEMM, 128, 2>(p, few, two, block, blocks, S);
            block -= (two * ((columns + 127) / 128) & ~7) % blocks;
            if (block < 0) block += blocks;
        }
    }
    const int cols = thin_cols(few, columns, p.workers);
    if (cols == 256) thin_tasks<GEMM, 256, 1>(p, 0, few, block, blocks, S);
    else if (cols == 128) thin_tasks<GEMM, 128, 1>(p, 0, few, block, blocks, S);
    else thin_tasks<GEMM, 64, 1>(p, 0, few, block, blocks, S);
}

}  // namespace uniep
