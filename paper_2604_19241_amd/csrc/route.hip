// Routing and deterministic token mapping on one GPU.
//
// Paper: Section 2.1 (gating, top-k), Section 3.1 "Deterministic Token Mapping",
// Algorithm 1 lines 1-2 (BinCount, CumSum) and the local stable order M_loc; with
// one rank the global offset base is zero, so the destination row of a
// (token, slot) pair is  offsets[e] + rank of the pair among the pairs of e.
//
// No position is ever handed out by an atomic: the tokens are cut into fixed chunks, a slot's
// rank inside its chunk comes from wave ballots in flat-slot order, and a scan over the chunks
// gives every chunk its starting row per expert.  The result is therefore the same on every run.
#include "common.hpp"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace uniep {

constexpr int kChunk = 256;        // flat slots per chunk, rounded up to whole tokens
constexpr int kRouteThreads = 256; // 4 waves per workgroup
constexpr int kChunkThreads = 1024;
constexpr int kPieces = (kChunk + kMaxTopK - 1 + 63) / 64;   // 64-slot pieces of a chunk
// Up to this many chunks every workgroup of the last kernel adds the chunks in front of its own
// by itself (one launch less): 40 chunks of 512 experts are 80 KB from L2 for each of 40 workgroups.
// 44 chunks of 256 experts 13.6 us (with the scan's launch 15.7), 128 chunks 16.8 us (15.9).
constexpr int kFewChunks = 64;

// From kManyChunks chunks on a chunk has up to 1024 slots, a thread each: a quarter of the workgroups or half of them, whose 16 waves
// rank a piece each instead of 4 of them, and as much less of the table to scan.  With fewer, CUs would stay idle.
// The chunks are as many as make whole rounds of kChunkCus, of equal length: 1100 short ones made 275 of 1024 slots, and the
// last 19 took as long as the 256 before.
// Measured, us of the whole routing, chunks of 256 slots / of 1024 / as they are (tokens x experts x k): 32768 x 256 x 8 38.2 / 36.8,
// 65536 x 64 x 8 49.1 / 35.2, 35200 x 256 x 8 48.6 / 47.3 / 33.2, 35200 x 513 x 8 89.4 / 133 / 68.9, 281600 x 8 x 1 51.3 / 64.0 / 38.7,
// 64000 x 256 x 8 70.9 / 50.2 / 49.2; but 16384 x 256 x 8 22.4 / 34.7, 24000 x 128 x 6 27.5 / 29.2.
constexpr int kLongPieces = kChunkThreads / 64;
constexpr int kManyChunks = 1024;
constexpr int kChunkCus = 256;   // CUs of the chip
struct Chunks {
    int tokens, n;   // of a chunk; chunks
    bool lng;
};
static Chunks chunks_of(const moe_shape_t& s) {
    const int tokens = (kChunk + s.k - 1) / s.k, n = (s.T + tokens - 1) / tokens;
    // Up to a slot a thread make one chunk, whose workgroup writes the rows as well: without the launch behind it 256 tokens of 8 experts, 2 selected,
    // take 5.6 us for 6.9, 512 slots of 64 tokens of 128 6.5 for 7.8, 1000 of 100 tokens of 512 9.1 for 10.9, 1024 of 64 of 1024 14.4 for 15.8.
    if ((long long)s.T * s.k <= kChunkThreads) return Chunks{s.T, 1, s.T * s.k > kPieces * 64};
    if (n < kManyChunks) return Chunks{tokens, n, false};
    const int round = kChunkCus * (kChunkThreads / s.k), rounds = (s.T + round - 1) / round;
    const int more = (s.T + kChunkCus * rounds - 1) / (kChunkCus * rounds);
    return Chunks{more, (s.T + more - 1) / more, true};
}
// Whether the top-k is a launch of its own, over the whole chip, ahead of the ranking
// (one launch more), instead of part of the chunk's workgroup (on as many CUs as there are chunks).
// RowSelect: a workgroup's 16 waves have 64 tokens at a time, so that a chunk of no more, or as many chunks as CUs, need no launch
// ahead.  Measured, us of the whole routing, in one launch with the ranking / apart (tokens x experts x k): 64 x 128 x 8 6.5 / 7.8, 512 x 256 x 8
// 8.5 / 9.3, 1000 x 256 x 8 9.3 / 10.0, 4099 x 64 x 6 11.7 / 12.6, 16384 x 64 x 2 12.2 / 12.6, 32768 x 256 x 2 18.0 / 19.0; but 128 x 128 x 8 9.9 / 6.8,
// 1024 x 64 x 1 18.8 / 6.1, 1024 x 256 x 2 11.6 / 8.4, 2048 x 256 x 4 10.2 / 9.7, 8192 x 64 x 1 10.0 / 8.5.  With 16 keys a lane a launch of its own
// pays from 33 tokens a chunk on, up to 96 chunks: 256 x 129 x 5 9.95 / 9.55, 512 x 129 x 5 9.97 / 9.12, 4096 x 144 x 5 13.9 / 13.2, 256 x 160 x 7 10.4 / 9.8, but 32 tokens a
// chunk 256 x 129 x 8 8.0 / 8.7, and 5000 x 129 x 6 13.6 / 14.3, 8192 x 144 x 7 14.1 / 14.8.
// WaveSelect: up to 16 tokens a wave, one after the other.  Up to 16 tokens a chunk have a wave each: 16 x 256 x 1 4.0 / 5.1, 16 x 512 x 4 5.7 / 6.4 (but from
// eight selected of 512 on it is the other way round: 16 x 512 x 16 10.9 / 9.5, 16 x 1024 x 8 11.0 / 9.3);
// one chunk: 24 x 256 x 1 4.2 / 5.0, 32 x 129 x 2 5.0 / 5.4, 24 x 512 x 1 4.9 / 5.6, but 32 x 512 x 4 8.0 / 6.3, 64 x 129 x 1 6.0 / 5.4, 100 x 129 x 1 7.6 / 5.6,
// 200 x 1024 x 1 26.6 / 6.5; fewer chunks than CUs: 2000 x 256 x 2 13.8 / 8.5, 1000 x 512 x 8 14.9 / 11.2, 8192 x 512 x 4 20.3 / 16.8; as many: 4096 x 129 x 16
// 15.6 / 17.1, 8192 x 512 x 8 19.9 / 19.9, 65536 x 1024 x 1 51.8 / 50.5; more, where the chip is full either way: 16384 x 257 x 8 26.4 / 28.1, 65536 x 257 x 2 32.6 / 36.0,
// but 8192 x 256 x 9 19.7 / 17.9, 8192 x 512 x 10 26.2 / 22.7 (283 and 316 chunks, which stay in one launch).
constexpr int kTopkGroups = 1 << 16;
// RowSelect or WaveSelect.  Of 129 to 256 experts RowSelect sorts 16 keys a lane, whatever k; WaveSelect's time is its k rounds.  One or two selected, in batches that
// are bound by latency, are the faster by WaveSelect, as are the first few tokens with up to 7.  Us of the whole routing, RowSelect / WaveSelect: 1 x 256 x 1
// 4.08 / 3.56, 24 x 256 x 1 4.77 / 4.20, 256 x 256 x 1 5.90 / 5.47, 128 x 129 x 2 5.85 / 5.60, 700 x 160 x 2 9.08 / 8.89, 5000 x 256 x 2 10.5 / 10.0,
// 1 x 256 x 4 4.30 / 4.08, 2 x 129 x 3 4.24 / 3.93; but 32 x 256 x 2 4.89 / 5.38, 24 x 256 x 3 5.1 / 5.5, 6 x 256 x 8 4.7 / 5.0, 8192 x 129 x 2 11.4 / 11.7,
// 60001 x 256 x 1 23.2 / 24.6, x 2 25.2 / 28.0.
static bool rows_select(const moe_shape_t& s) {
    if (s.E <= 128) return true;
    return s.E <= 256 && s.k <= 8 && !(s.T < 8192 && s.T * (s.k - 2) < 6);
}
static bool topk_alone(const moe_shape_t& s, const Chunks& c) {
    if (c.lng && c.n > 1) return false;
    const int n = c.n, tokens = std::min(s.T, c.tokens);
    const long long work = (long long)tokens * s.E;
    if (rows_select(s)) {
        if (s.E > 128 && tokens > kChunkThreads / 32 && n < 96) return true;
        return n < (s.E <= 64 ? 128 : 256) && (tokens > kChunkThreads / 16 || work > 8192);
    }
    if (c.lng) return true;   // (more than 320 slots of more than 128 experts: past both lines below)
    if (tokens <= kChunkThreads / 64 && (n == 1 || s.E <= 256)) return false;
    if (n == 1) return work * s.k > 13000 || (s.E <= 256 && tokens > 48);
    return n < 128 || (n < 256 && work >= 4096) || (n < 512 && work >= 16384);
}

// Largest value over the wave, on the data-parallel-primitive path of the vector ALU: six
// instructions; six shuffles through LDS took ten times as long.
template <int NT>
__device__ __forceinline__ void wave_max(uint32_t (&v)[NT]) {
#define UNIEP_DPP_MAX(ctrl, rows)                                                                                     \
    _Pragma("unroll") for (int n = 0; n < NT; ++n) v[n] =                                                             \
        max(v[n], (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[n], ctrl, rows, 0xf, false))
    UNIEP_DPP_MAX(0x111, 0xf);   // row_shr:1
    UNIEP_DPP_MAX(0x112, 0xf);   // row_shr:2
    UNIEP_DPP_MAX(0x114, 0xf);   // row_shr:4
    UNIEP_DPP_MAX(0x118, 0xf);   // row_shr:8  -> lane 15 of every row of 16 has the row's
    UNIEP_DPP_MAX(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    UNIEP_DPP_MAX(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef UNIEP_DPP_MAX
#pragma unroll
    for (int n = 0; n < NT; ++n) v[n] = (uint32_t)__builtin_amdgcn_readlane((int)v[n], 63);
}
// Unsigned integers in the order of the floats.  0 stands for a NaN (which is never selected),
// an expert already taken and the padding; both zeros get one key, as they compare equal.
__device__ __forceinline__ uint32_t logit_key(float x) {
    const uint32_t u = __float_as_uint(x + 0.f);
    return x == x ? ((u & 0x80000000u) ? ~u : u | 0x80000000u) : 0u;
}
__device__ __forceinline__ float key_logit(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k);
}

// Exclusive sum over the workgroup's threads (W waves); `total` = sum over all of them.
// s_wave: W words of LDS that nobody uses across the call's two barriers.
template <int W>
__device__ __forceinline__ int block_exclusive_sum(int v, int32_t* s_wave, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
    }
    __syncthreads();
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int x = s_wave[w];
        if (w < wave) before += x;
        all += x;
    }
    *total = all;
    return before + incl - v;
}

// One token's logits: lane l has experts l, l + 64, ...  The loads are unconditional (lanes past the last expert load it once
// more): behind a branch each waited for its data before the next went out, a round trip to memory for every 64 experts
// (8192 tokens of 512 experts 30.4 -> 28.5 us for the whole routing, 65536 of 256, one selected, 32.3 -> 27.8 us).
// `row` the same for the whole wave, and EPL the least power of two that holds E, so that the first half of the loads
// needs no bound: a scalar base and a few offsets.  An address a lane and load took 77 registers for 16 loads, with which one
// ranking workgroup fits a CU instead of two (28800 tokens of 513 experts, 8 selected, 85 -> 68 us).
template <int EPL>
__device__ __forceinline__ void load_logits(const float* __restrict__ row, int E, int lane, float (&x)[EPL]) {
#pragma unroll
    for (int i = 0; i < EPL; ++i) x[i] = row[i < EPL / 2 ? lane + 64 * i : min(lane + 64 * i, E - 1)];
}
// Top-k where RowSelect is not taken, NT tokens by one wave: lane j < k gets a token's j-th expert and its gate.  A round is one
// chain of dependent instructions: the tokens' chains run side by side, without a branch between them.
template <int EPL, int NT>
__device__ __forceinline__ void select_experts(const float (&x)[NT][EPL], int E, int k, int lane, int (&my_idx)[NT], float (&gate)[NT]) {
    uint32_t key[NT][EPL], my_key[NT], best[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
        for (int i = 0; i < EPL; ++i) key[n][i] = lane + 64 * i < E ? logit_key(x[n][i]) : 0u;
        my_idx[n] = 0;
        my_key[n] = 0;
    }
    for (int j = 0; j < k; ++j) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            best[n] = key[n][0];
#pragma unroll
            for (int i = 1; i < EPL; ++i) best[n] = max(best[n], key[n][i]);
        }
        wave_max<NT>(best);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            int be = 0;
#pragma unroll
            for (int i = EPL - 1; i >= 0; --i) {
                const uint64_t m = __ballot(key[n][i] == best[n]);
                be = m ? 64 * i + (int)__builtin_ctzll(m) : be;
            }
#pragma unroll
            for (int i = 0; i < EPL; ++i) key[n][i] = (lane + 64 * i == be) ? 0u : key[n][i];
            // (nothing but NaN left: no expert, and a key that was 0 already)
            my_key[n] = lane == j ? best[n] : my_key[n];
            my_idx[n] = lane == j ? (best[n] ? be : 0x7fffffff) : my_idx[n];
        }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const float my_val = my_key[n] ? key_logit(my_key[n]) : -INFINITY;
        const float top1 = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(my_val)));
        const float p = (lane < k) ? __expf(my_val - top1) : 0.f;
        float s = p;
#pragma unroll
        for (int off = kMaxTopK / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        gate[n] = p / s;
    }
}

template <int EPL>
struct WaveSelect {
    // tokens t, t + BY, ... of the wave, two at a time where the registers allow it (16 keys a lane, twice, take too many)
    template <int BY, class Put>
    static __device__ __forceinline__ void run(const float* __restrict__ logits, int wave, int n, int E, int k, Put put) {
        const int lane = threadIdx.x & 63;
        auto tokens = [&](int t, auto count) {
            constexpr int NT = decltype(count)::value;
            float x[NT][EPL], gate[NT];
            int idx[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) load_logits<EPL>(logits + (size_t)(t + i * BY) * E, E, lane, x[i]);
            select_experts<EPL, NT>(x, E, k, lane, idx, gate);
#pragma unroll
            for (int i = 0; i < NT; ++i)
                if (lane < k) put(t + i * BY, lane, idx[i], gate[i]);
        };
        int t = wave;
        if constexpr (EPL <= 8)
            for (; t + BY < n; t += 2 * BY) tokens(t, std::integral_constant<int, 2>{});
        for (; t < n; t += BY) tokens(t, std::integral_constant<int, 1>{});
    }
    static constexpr int kTokens = 1;
    template <class Put>
    static __device__ __forceinline__ void one(const float* __restrict__ logits, int t, int, int E, int k, Put put) {
        run<1>(logits + (size_t)t * E, 0, 1, E, k, [&](int, int slot, int expert, float gate) { put(t, slot, expert, gate); });
    }
};

// ------------------------------------------- top-k of up to 256 experts
// Four tokens a wave, one in each row of 16 lanes: lane q of a row has the experts q, q + 16, ... of its token, as doubles that are
// ordered as (value, then lower expert id): the logit's key in the high bits, 1023 - id below.  No two experts
// have the same one, so a lane's list needs no ids beside it, and a compare-and-exchange is two instructions.  Every lane sorts its
// EPL keys; a round takes the largest head of the row (four rotations, for the four tokens at once) and the
// lane that had it moves its list up by one.  Bound by instruction issue: some 150 instructions a token with 256 experts and 8
// selected, where a token on all 64 lanes (six steps a maximum, a ballot for every key) took 480.  The whole routing, us, so / now (tokens x
// experts x k): 32768 x 256 x 8 33.3 / 23.2, 60001 x 256 x 8 47.0 / 33.9, 65536 x 128 x 8 38.4 / 27.1, 24000 x 128 x 6 25.5 / 21.6, 8192 x 128 x 8
// 13.8 / 12.3, 65536 x 8 x 2 18.3 / 13.7, 32 x 128 x 8 6.0 / 6.0.  With one workgroup of the ranking a CU instead of two, the registers
// of which hold the next tokens' logits, 60001 x 256 x 8 took 39.6.  More than 8 of 129 to 256 experts stay with WaveSelect: 16 sorted keys a
// lane and 16 rounds that move them were slower.
// The keys are positive, normal and finite: those of -inf and +inf have the exponents 0x003 and 0x7fc.
// 0.0 stands for a NaN (never selected) and for the padding.
__device__ __forceinline__ double expert_key(float x, int id) {
    const uint32_t key = logit_key(x);
    const uint32_t lo = (key << 31) | (uint32_t)(kMaxExperts - 1 - id);
    return __builtin_bit_cast(double, (uint64_t)(key >> 1) << 32 | (key ? lo : 0u));
}
__device__ __forceinline__ uint32_t double_key(double v) { return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 31); }
__device__ __forceinline__ int double_expert(double v) {
    return kMaxExperts - 1 - (int)((uint32_t)__builtin_bit_cast(uint64_t, v) & (kMaxExperts - 1));
}
// The value of the lane BY further on in the row of 16 (in a circle).
template <int BY>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + BY, 0xf, 0xf, true);
}
template <int BY>
__device__ __forceinline__ double row_ror(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)row_ror<BY>((uint32_t)(u >> 32)) << 32 | row_ror<BY>((uint32_t)u));
}
template <int BY>
__device__ __forceinline__ float row_ror(float v) {
    return __uint_as_float(row_ror<BY>(__float_as_uint(v)));
}
// Larger one to a, smaller one to b.
__device__ __forceinline__ void exchange(double& a, double& b) {
    const double m = fmin(a, b);
    a = fmax(a, b);
    b = m;
}
// Descending (Batcher's odd-even merge sort).  The scheduler would otherwise run the passes into one another and need twice the registers.
template <int N>
__device__ __forceinline__ void sort_descending(double* v) {
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int q = p; q >= 1; q /= 2) {
#pragma unroll
            for (int j = q % p; j + q < N; j += 2 * q)
#pragma unroll
                for (int i = 0; i < q; ++i)
                    if (i + j + q < N && (i + j) / (2 * p) == (i + j + q) / (2 * p)) exchange(v[i + j], v[i + j + q]);
            __builtin_amdgcn_sched_barrier(0);
        }
}

// How a wave selects the experts of its tokens.  KM: compile-time bound on k.
template <int EPL_, int KM>
struct RowSelect {
    static constexpr int kTokens = 4;   // of a wave, at a time
    static constexpr int EPL = EPL_, D = EPL < KM ? EPL : KM;
    // (a scalar base and 32-bit byte offsets; rows past the n-th alias it)
    static __device__ __forceinline__ void load(const float* __restrict__ logits, int t, int n, int E, float (&x)[EPL]) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // nothing is kept over the loop: every lane offset would take a register
        const int q = tid & 15;
        const char* base = (const char*)(logits + (size_t)t * E);
        const uint32_t row = (uint32_t)(min((tid >> 4) & 3, n - 1 - t) * E);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const uint32_t e = (uint32_t)(EPL > 2 && i < EPL / 2 ? q + 16 * i : min(q + 16 * i, E - 1));
            x[i] = *(const float*)(base + (row + e) * 4u);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // tokens t .. t + 3, the wave's t = 4 wave, 4 (wave + BY), ...: put(token, slot, expert, gate) for every slot below k
    template <int BY, class Put>
    static __device__ __forceinline__ void run(const float* __restrict__ logits, int wave, int n, int E, int k, Put put) {
        for (int t = 4 * wave; t < n; t += 4 * BY) one(logits, t, n, E, k, put);
    }
    template <class Put>
    static __device__ __forceinline__ void one(const float* __restrict__ logits, int t, int n, int E, int k, Put put) {
        float x[EPL];
        load(logits, t, n, E, x);
        select(x, t, n, E, k, put);
    }
    template <class Put>
    static __device__ __forceinline__ void select(const float (&x)[EPL], int t, int n, int E, int k, Put put) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int q = tid & 15, mine = t + ((tid >> 4) & 3);
        double v[EPL];
        // the D largest of the lane's, descending
#pragma unroll
        for (int h = 0; h < EPL; h += D) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = h; i < h + D; ++i) {
                const bool any = (EPL > 2 && i < EPL / 2) || q + 16 * i < E;
                v[i] = expert_key(any ? x[i] : __builtin_nanf(""), q + 16 * i);
            }
            sort_descending<D>(v + h);
        }
        if constexpr (EPL > D) {   // of two such lists the larger ones in turn are the D largest, and rise and fall at most once
            static_assert(EPL == 2 * D, "");
#pragma unroll
            for (int i = 0; i < D; ++i) v[i] = fmax(v[i], v[EPL - 1 - i]);
#pragma unroll
            for (int o = D / 2; o >= 1; o /= 2) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < D; ++i)
                    if ((i & o) == 0) exchange(v[i], v[i + o]);
            }
        }
        double taken = 0.0, top = 0.0;
        auto round = [&](int j, int depth) {   // depth: entries of the lists that a later round may still take
            double best = fmax(v[0], row_ror<8>(v[0]));
            best = fmax(best, row_ror<4>(best));
            best = fmax(best, row_ror<2>(best));
            best = fmax(best, row_ror<1>(best));
            if (j == 0) top = best;
            taken = q == j ? best : taken;
            const bool won = __builtin_bit_cast(uint64_t, v[0]) == __builtin_bit_cast(uint64_t, best);
#pragma unroll
            for (int i = 0; i < D && i < depth; ++i) v[i] = won ? (i + 1 < D ? v[i + 1] : 0.0) : v[i];
        };
        if constexpr (KM <= 8) {
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                if (j >= k) break;
                round(j, KM - 1 - j);
            }
        } else {
            for (int j = 0; j < k; ++j) round(j, D);
        }
        // nothing but NaN left: no expert
        const uint32_t key = double_key(taken), top_key = double_key(top);
        const float val = key ? key_logit(key) : -INFINITY, top1 = top_key ? key_logit(top_key) : -INFINITY;
        const float p = q < k ? __expf(val - top1) : 0.f;
        float s = p + row_ror<8>(p);
        s += row_ror<4>(s);
        s += row_ror<2>(s);
        s += row_ror<1>(s);
        if (q < k && mine < n) put(mine, q, key ? double_expert(taken) : 0x7fffffff, p / s);
    }
};

struct NoSelect {
    static constexpr int kTokens = 0;
};

// ------------------------------------------- top-k, gates and ranks inside a chunk
// One workgroup per chunk, whose waves select the experts of four tokens (RowSelect) or one or two (WaveSelect: lane l holds experts l,
// l+64, ... as sortable keys; a round of arg-max under the order (value desc, expert id asc) is one wave
// maximum and one ballot per key, whose first set bit is the lowest expert id) at a time.  Gates come from
// the k selected logits (the softmax denominator over all E cancels in the renormalisation).
// Then wave i ranks the chunk's slots [64 i, 64 i + 64): lanes that share an expert are the
// intersection of the ballots of the expert id's bits.  chunk_cnt[c][e] = slots of chunk c
// routed to local expert e; inv_perm[f] = rank of slot f among its chunk's slots of that expert.
// SEL: RowSelect, WaveSelect, or NoSelect where topk_kernel has selected the experts already.
// Bound by instruction issue.  With the maximum by shuffles and counts, scan and positions in three
// launches of their own the whole routing took 101 us for 32768 tokens of 256 experts, 8 selected
// (now 23 us), and 11-15 us in four launches for up to 16 tokens of 128 experts (now one launch of 3.6-5 us).
//
// ONE: the batch is a single chunk (a generation step): the ranks are complete, and the same
// workgroup scans the counts and writes the rows.
// PIECES: 64-slot pieces of a chunk (a wave's counts of an expert in a piece are at most 64).
// Two workgroups of 16 waves share a CU: 8 waves a SIMD, up to 64 registers a lane, for which RowSelect<16, 8> puts two away in
// memory in two of its four forms (with one workgroup a CU 60001 tokens of 256 experts, 8 selected, took 39.6 us for 33.9).
template <class SEL, bool ONE, int PIECES>
__global__ void __launch_bounds__(kChunkThreads) __attribute__((amdgpu_waves_per_eu(8)))
topk_rank_kernel(const float* __restrict__ logits, int T, int E, int k, int per_chunk, int e_start, int e_count,
                 int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int32_t* __restrict__ chunk_cnt,
                 int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
                 int32_t* __restrict__ inv_perm) {
    __shared__ int32_t s_idx[PIECES * 64];
    __shared__ std::conditional_t<(PIECES > kPieces), uint16_t, int32_t> s_cnt[PIECES][kMaxExperts];
    __shared__ int32_t s_off[ONE ? kMaxExperts : 1];
    __shared__ int32_t s_wave[kChunkThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * per_chunk, nt = min(per_chunk, T - t0), n = nt * k;
    const size_t f0 = (size_t)t0 * k;
    if (tid < e_count)
#pragma unroll
        for (int i = 0; i < PIECES; ++i) s_cnt[i][tid] = 0;
    if constexpr (SEL::kTokens > 0) {
        SEL::template run<kChunkThreads / 64>(
            logits + (size_t)t0 * E, __builtin_amdgcn_readfirstlane(wave), nt, E, k, [&](int token, int slot, int expert, float gate) {
                const int f = token * k + slot;
                s_idx[f] = expert;
                topk_idx[f0 + f] = expert;
                topk_w[f0 + f] = gate;
            });
    } else if (tid < n) {
        s_idx[tid] = topk_idx[f0 + tid];
    }
    __syncthreads();
    int el = -1, rank = -1;
    if (wave < PIECES) {
        if (tid < n) {
            el = s_idx[tid] - e_start;
            if (el < 0 || el >= e_count) el = -1;
        }
        uint64_t m = __ballot(el >= 0);
        for (int b = 0; (1 << b) < e_count; ++b) {
            const uint64_t bb = __ballot((el >> b) & 1);
            m &= ((el >> b) & 1) ? bb : ~bb;
        }
        if (el >= 0) {
            rank = __popcll(m & ((1ull << lane) - 1ull));
            if ((m >> lane) <= 1ull) s_cnt[wave][el] = rank + 1;   // the group's last lane knows its size
        }
    }
    __syncthreads();
    if (el >= 0)
        for (int w = 0; w < wave; ++w) rank += s_cnt[w][el];
    int total = 0;
    if (tid < e_count)
#pragma unroll
        for (int i = 0; i < PIECES; ++i) total += s_cnt[i][tid];
    if (!ONE) {
        if (tid < n) inv_perm[f0 + tid] = rank;
        if (tid < e_count) chunk_cnt[(size_t)blockIdx.x * e_count + tid] = total;
        return;
    }
    int rows;
    const int off = block_exclusive_sum<kChunkThreads / 64>(total, s_wave, &rows);
    if (tid < e_count) {
        counts[tid] = total;
        offsets[tid] = s_off[tid] = off;
    }
    if (tid == 0) offsets[e_count] = rows;
    __syncthreads();
    if (tid < n) {
        const int row = el >= 0 ? s_off[el] + rank : -1;
        inv_perm[tid] = row;
        if (row >= 0) perm[row] = tid;
        if (tid >= rows) perm[tid] = -1;   // rows at and beyond the routed ones
    }
}

// ------------------------------------------- top-k alone
// Over the whole chip, four tokens or one a wave; topk_rank_kernel<NoSelect, ..> then ranks what this wrote.
template <class SEL>
__global__ void __launch_bounds__(kRouteThreads)
topk_kernel(const float* __restrict__ logits, int T, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    constexpr int kPer = kRouteThreads / 64 * SEL::kTokens;
    for (int t = blockIdx.x * kPer + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * SEL::kTokens; t < T; t += gridDim.x * kPer)
        SEL::one(logits, t, T, E, k, [&](int token, int slot, int expert, float gate) {
            topk_idx[(size_t)token * k + slot] = expert;
            topk_w[(size_t)token * k + slot] = gate;
        });
}

// ------------------------------------------------------------- scan over chunks
// In place: chunk_cnt[c][e] becomes the number of e-slots in chunks before c; counts[e] = total.
// A workgroup has 16 experts (64-byte row pieces) by 64 chunk lanes of 8 chunks: the table is read
// once, 8 loads in flight a thread.
constexpr int kScanExperts = 16, kScanLanes = kChunkThreads / kScanExperts, kScanPer = 8;
__global__ void __launch_bounds__(kChunkThreads)
chunk_scan_kernel(int32_t* __restrict__ chunk_cnt, int n_chunks, int e_count, int32_t* __restrict__ counts) {
    __shared__ int32_t s_sum[kScanLanes][kScanExperts + 1];
    const int col = threadIdx.x & (kScanExperts - 1), g = threadIdx.x / kScanExperts;
    const int e = blockIdx.x * kScanExperts + col;
    int32_t carry = 0;
    for (int base = 0; base < n_chunks; base += kScanLanes * kScanPer) {
        const int c0 = base + g * kScanPer;
        int32_t v[kScanPer], sum = 0;
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) {
            v[u] = (e < e_count && c0 + u < n_chunks) ? chunk_cnt[(size_t)(c0 + u) * e_count + e] : 0;
            sum += v[u];
        }
        s_sum[g][col] = sum;
        __syncthreads();
        int32_t run = carry;
#pragma unroll 8
        for (int i = 0; i < kScanLanes; ++i) {
            const int32_t x = s_sum[i][col];
            if (i < g) run += x;
            carry += x;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) {
            if (e < e_count && c0 + u < n_chunks) chunk_cnt[(size_t)(c0 + u) * e_count + e] = run;
            run += v[u];
        }
    }
    if (g == 0 && e < e_count) counts[e] = carry;
}

// ------------------------------------------------------------ rows
// One workgroup per chunk: row of a slot = first row of its expert (scan of the counts over the
// experts, by every workgroup for itself) + the expert's slots in the chunks before + its rank
// in the chunk.  SCANNED: chunk_cnt already holds the sums over the chunks before.
template <bool SCANNED>
__global__ void __launch_bounds__(kChunkThreads)
rows_kernel(const int32_t* __restrict__ topk_idx, int T, int k, int per_chunk, int n_chunks, int e_start, int e_count,
            const int32_t* __restrict__ chunk_cnt, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
            int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm) {
    __shared__ int32_t s_base[kMaxExperts];
    __shared__ int32_t s_wave[kChunkThreads / 64];
    const int tid = threadIdx.x, c = blockIdx.x;
    const int t0 = c * per_chunk, n = min(per_chunk, T - t0) * k;
    const int f = t0 * k + tid;
    int el = -1, rank = 0;
    if (tid < n) {
        el = topk_idx[f] - e_start;
        rank = inv_perm[f];
    }
    int before = 0, total = 0;
    if (tid < e_count) {
        if (SCANNED) {
            before = chunk_cnt[(size_t)c * e_count + tid];
            total = counts[tid];
        } else {
#pragma unroll 8
            for (int i = 0; i < n_chunks; ++i) {
                const int x = chunk_cnt[(size_t)i * e_count + tid];
                if (i < c) before += x;
                total += x;
            }
        }
    }
    int rows;
    const int off = block_exclusive_sum<kChunkThreads / 64>(total, s_wave, &rows);
    if (tid < e_count) {
        s_base[tid] = off + before;
        if (c == 0) {
            if (!SCANNED) counts[tid] = total;
            offsets[tid] = off;
        }
    }
    if (c == 0 && tid == 0) offsets[e_count] = rows;
    __syncthreads();
    if (tid < n) {
        const int row = rank >= 0 ? s_base[el] + rank : -1;
        inv_perm[f] = row;
        if (row >= 0) perm[row] = f;
        if (f >= rows) perm[f] = -1;   // rows at and beyond the routed ones
    }
}

// No tokens: no expert has rows.
__global__ void __launch_bounds__(kChunkThreads) no_rows_kernel(int e_count, int32_t* counts, int32_t* offsets) {
    if ((int)threadIdx.x < e_count) counts[threadIdx.x] = 0;
    if ((int)threadIdx.x < e_count) offsets[threadIdx.x + 1] = 0;
    if (threadIdx.x == 0) offsets[0] = 0;
}

// ------------------------------------------------------------ router gradient
// One wave per token.  Lanes j < k hold slot j; s = sum_j w_j g_j by a wave reduction; then the
// k experts and their values go to scalar registers and every lane writes its experts of the
// row: the value of the slot that selected the expert, or zero.  Bound by the stores of the
// [T,E] array: 60001 tokens of 256 experts, 8 selected, 18 us (3.4 TB/s); with two shuffles through LDS per slot
// and 64 experts 48 us.
// KM = compile-time bound on k (2, 4, 8 or kMaxTopK): every element is compared with KM experts, which shows where
// few are selected (32768 tokens of 1024 experts, KM = 8 / 4 / 2: 24.2 / 19.5 / 18.9 us).
template <int KM>
__global__ void __launch_bounds__(kRouteThreads)
route_backward_kernel(const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w,
                      const float* __restrict__ dtopk_w, int T, int E, int k,
                      float* __restrict__ dlogits) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (kRouteThreads / 64) + (threadIdx.x >> 6);
    if (t >= T) return;
    int idx = -1;
    float w = 0.f, g = 0.f;
    if (lane < k) {
        idx = topk_idx[(size_t)t * k + lane];
        w = topk_w[(size_t)t * k + lane];
        g = dtopk_w[(size_t)t * k + lane];
    }
    float s = w * g;
#pragma unroll
    for (int off = kMaxTopK / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    const float mine = w * (g - s);
    int ej[KM];
    float vj[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {   // (lanes from k on hold expert -1)
        ej[j] = __builtin_amdgcn_readlane(idx, j);
        vj[j] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(mine), j));
    }
    for (int e = lane; e < E; e += 64) {
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (ej[j] == e) v = vj[j];
        dlogits[(size_t)t * E + e] = v;
    }
}

// ------------------------------------------------------------------ global mapping, W > 1
// Algorithm 1 for one rank of W (Section 3.1).  The AllGather of the per-rank
// histograms is the caller's; c_all [W, E] is its result.

// By a workgroup of kMapThreads, thread e per expert: Eq. 1 along the rank axis,
// the total rows every expert receives, and the start of every expert's segment
// in its destination rank's buffer (exclusive scan inside each group of n_epr
// experts).  off_base = O_all[rank, e] - O_exp[e] and row_base = segment start + off_base, so that the mapping only
// adds M_loc; `recv` writes this rank's own segment table recv_offsets [n_epr + 1].  Ends with a barrier.
constexpr int kMapThreads = 1024;
struct MapScan {
    int32_t first[kMapThreads];
    int32_t wave[kMapThreads / 64];
};
__device__ __forceinline__ void global_bases(MapScan& S, const int32_t* __restrict__ c_all, const int32_t* __restrict__ o_exp, int E, int W, int rank,
                                             int n_epr, int32_t* off_base, int32_t* row_base, bool recv, int32_t* __restrict__ recv_offsets) {
    const int e = threadIdx.x;
    int total = 0, before = 0;
    if (e < E) {
#pragma unroll 8
        for (int r = 0; r < W; ++r) {
            const int c = c_all[(size_t)r * E + e];
            if (r < rank) before += c;
            total += c;
        }
    }
    int all;
    const int first = block_exclusive_sum<kMapThreads / 64>(total, S.wave, &all);
    S.first[e] = first;
    __syncthreads();
    if (e < E) {
        const int g0 = (e / n_epr) * n_epr;              // first expert of e's rank
        const int start = first - S.first[g0];
        const int ob = before - o_exp[e];
        off_base[e] = ob;
        row_base[e] = start + ob;
        if (recv && e / n_epr == rank) {
            recv_offsets[e - g0] = start;
            if (e - g0 == n_epr - 1) recv_offsets[n_epr] = start + total;
        }
    }
    __syncthreads();
}
__global__ void __launch_bounds__(kMapThreads)
global_offsets_kernel(const int32_t* __restrict__ c_all, const int32_t* __restrict__ o_exp, int E,
                      int W, int rank, int n_epr, int32_t* __restrict__ off_base,
                      int32_t* __restrict__ row_base, int32_t* __restrict__ recv_offsets) {
    __shared__ MapScan S;
    global_bases(S, c_all, o_exp, E, W, rank, n_epr, off_base, row_base, true, recv_offsets);
}

// One thread per slot: destination (rank, local expert, offset inside the expert's
// segment, row of the destination buffer); `send` marks the first
// slot, in slot order, that targets a rank (the copy that crosses the link; the relay
// worker of Section 3.2 replicates it for the token's other experts on that rank).
// A workgroup has per_group whole tokens and their slots' ranks in LDS, where a slot finds the
// earlier slots of its token.  Bound by its seven arrays, which a
// thread per token read and wrote with a stride: 8.3 us for 32768 tokens with 8 slots, then 4.7 us.
// BASES: every workgroup makes the experts' bases for itself, one launch less, and reads the W histograms for that (see global_map_launch); such a
// workgroup has kMapThreads threads, one without kRouteThreads.
template <bool BASES>
__global__ void __launch_bounds__(BASES ? kMapThreads : kRouteThreads)
global_map_kernel(const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ m_loc, int T,
                  int k, int per_group, int E, int n_epr, const int32_t* __restrict__ c_all, const int32_t* __restrict__ o_exp, int W, int rank,
                  const int32_t* __restrict__ off_base, const int32_t* __restrict__ row_base, int32_t* __restrict__ dst_rank,
                  int32_t* __restrict__ dst_expert, int32_t* __restrict__ dst_off,
                  int32_t* __restrict__ dst_row, int32_t* __restrict__ send,
                  int32_t* __restrict__ n_dst_ranks, int32_t* __restrict__ recv_offsets) {
    __shared__ int32_t s_rank[BASES ? kMapThreads : kRouteThreads];
    const int tid = threadIdx.x;
    const int t0 = blockIdx.x * per_group, nt = min(per_group, T - t0);
    const size_t f = (size_t)t0 * k + tid;
    const bool live = tid < nt * k;
    int e = 0, loc = 0;
    if (live) {
        e = topk_idx[f];
        loc = m_loc[f];
    }
    const int32_t *off = off_base, *row = row_base;
    if constexpr (BASES) {
        __shared__ MapScan S;
        __shared__ int32_t s_off[kMapThreads], s_row[kMapThreads];
        global_bases(S, c_all, o_exp, E, W, rank, n_epr, s_off, s_row, blockIdx.x == 0, recv_offsets);
        off = s_off;
        row = s_row;
    }
    if (live) {
        const bool any = (uint32_t)e < (uint32_t)E;   // a token with fewer than k logits that are numbers has slots without an expert
        const int r_tgt = any ? e / n_epr : -1;
        s_rank[tid] = r_tgt;
        dst_rank[f] = r_tgt;
        dst_expert[f] = any ? e - r_tgt * n_epr : -1;
        dst_off[f] = any ? loc + off[e] : -1;
        dst_row[f] = any ? loc + row[e] : -1;
    }
    __syncthreads();
    if (live) {
        bool first = s_rank[tid] >= 0;
        for (int i = tid - tid % k; i < tid; ++i) first = first && s_rank[i] != s_rank[tid];
        send[f] = first ? 1 : 0;
    }
    if (tid < nt) {
        unsigned long long seen = 0ull;
        for (int j = 0; j < k; ++j) {
            const int r = s_rank[tid * k + j];
            if (r >= 0) seen |= 1ull << r;
        }
        n_dst_ranks[t0 + tid] = __popcll(seen);
    }
}

// ------------------------------------------------------------------ host side

// Up to so many counts, and no more workgroups than run at a time (two a CU), every workgroup of the mapping makes the bases for itself.  Us, by a launch
// of their own / so (tokens x experts x k, ranks): 100 x 256 x 8, 8 6.0 / 4.9, 32768 7.4 / 6.0, 65536 (512 workgroups) 9.1 / 8.2, but 80000 (625)
// 10.1 / 10.7, 131072 (1024) 12.0 / 12.9, 300001 19.2 / 24.8; 52000 x 512 x 10, 8 (510) 10.3 / 8.8, 65536 (643) 11.2 / 11.5; 32768 x 128 x 16, 32 (512)
// 11.1 / 10.1, 45000 (704) 13.3 / 14.2.  By the counts: 16384 x 1024 x 8 with 4 ranks 7.1 / 5.9, with 8 7.0 / 5.8, with 64 8.7 / 7.7, but 45000 with 16 8.7 / 8.6, with
// 64 10.2 / 12.2.  Where the bases have their launch, 1024 threads a workgroup are the slower: 300001 x 256 x 8 21.9 for 19.2, 1000 x 1024 x 8 7.0 for 6.5.
constexpr int kMapTable = 4096;
constexpr int kMapGroups = 2 * kChunkCus;

int global_map_launch(const moe_shape_t& s, int W, int rank, const moe_routing_t& r,
                      const int32_t* c_all, const moe_global_map_t& out, void* ws, hipStream_t st) {
    int32_t* off_base = (int32_t*)ws;
    int32_t* row_base = off_base + s.E;
    const int n_epr = s.E / W;
    auto launch = [&](auto kernel, int threads) {
        const int per_group = threads / s.k;   // whole tokens whose slots fill a workgroup
        hipLaunchKernelGGL(kernel, dim3((s.T + per_group - 1) / per_group), dim3(threads), 0, st, r.topk_idx, r.inv_perm, s.T, s.k, per_group, s.E, n_epr,
                           c_all, r.offsets, W, rank, off_base, row_base, out.dst_rank, out.dst_expert, out.dst_off, out.dst_row, out.send,
                           out.n_dst_ranks, out.recv_offsets);
    };
    if (s.T > 0 && W * s.E <= kMapTable && s.T <= kMapGroups * (kMapThreads / s.k)) {
        launch(global_map_kernel<true>, kMapThreads);
    } else {
        hipLaunchKernelGGL(global_offsets_kernel, dim3(1), dim3(kMapThreads), 0, st, c_all, r.offsets, s.E, W, rank, n_epr, off_base, row_base,
                           out.recv_offsets);
        if (s.T > 0) launch(global_map_kernel<false>, kRouteThreads);
    }
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}


int route_backward_launch(const moe_shape_t& s, const int32_t* topk_idx, const float* topk_w,
                          const float* dtopk_w, float* dlogits, hipStream_t st) {
    if (s.T == 0) return MOE_OK;
    const int per = kRouteThreads / 64;
    const dim3 grid((s.T + per - 1) / per);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kRouteThreads), 0, st, topk_idx, topk_w, dtopk_w, s.T, s.E, s.k, dlogits);
    };
    if (s.k <= 2) launch(route_backward_kernel<2>);
    else if (s.k <= 4) launch(route_backward_kernel<4>);
    else if (s.k <= 8) launch(route_backward_kernel<8>);
    else launch(route_backward_kernel<kMaxTopK>);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// (a chunk has at least kChunk slots, so there are at most this many)
size_t route_workspace_bytes(const moe_shape_t& s) {
    const size_t F = (size_t)s.T * s.k;
    const size_t n_chunks = (F + kChunk - 1) / kChunk;
    return align_up(n_chunks * (size_t)s.e_count * sizeof(int32_t) + 256, 256);
}

template <class SEL>
static void launch_rank(const moe_shape_t& s, const Chunks& c, const float* logits, const moe_routing_t& out, int32_t* chunk_cnt,
                        hipStream_t st) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(c.n), dim3(kChunkThreads), 0, st, logits, s.T, s.E, s.k, c.tokens, s.e_start, s.e_count,
                           (int32_t*)out.topk_idx, (float*)out.topk_w, chunk_cnt, (int32_t*)out.counts, (int32_t*)out.offsets,
                           (int32_t*)out.perm, (int32_t*)out.inv_perm);
    };
    if constexpr (SEL::kTokens > 0)
        if (c.lng && c.n > 1) return launch(topk_rank_kernel<SEL, false, kLongPieces>);
    if constexpr (SEL::kTokens != 1)   // (by WaveSelect the top-k of one long chunk is apart)
        if (c.lng) return launch(topk_rank_kernel<SEL, true, kLongPieces>);
    if (c.n == 1) launch(topk_rank_kernel<SEL, true, kPieces>);
    else launch(topk_rank_kernel<SEL, false, kPieces>);
}

template <class SEL>
static void launch_topk(const moe_shape_t& s, const Chunks& c, const float* logits, const moe_routing_t& out, int32_t* chunk_cnt,
                        hipStream_t st) {
    if (!topk_alone(s, c)) return launch_rank<SEL>(s, c, logits, out, chunk_cnt, st);
    const int per = kRouteThreads / 64 * SEL::kTokens, grid = std::min((s.T + per - 1) / per, kTopkGroups);
    hipLaunchKernelGGL(topk_kernel<SEL>, dim3(grid), dim3(kRouteThreads), 0, st, logits, s.T, s.E, s.k,
                       (int32_t*)out.topk_idx, (float*)out.topk_w);
    launch_rank<NoSelect>(s, c, logits, out, chunk_cnt, st);
}

int route_launch(const moe_shape_t& s, const float* logits, const moe_routing_t& out, void* ws,
                 hipStream_t st) {
    int32_t* chunk_cnt = (int32_t*)ws;
    if (s.T == 0) {
        hipLaunchKernelGGL(no_rows_kernel, dim3(1), dim3(kChunkThreads), 0, st, s.e_count, (int32_t*)out.counts,
                           (int32_t*)out.offsets);
        return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
    }
    const Chunks c = chunks_of(s);
    const int n = c.n;
    auto rows_of = [&](auto most) {   // up to 256 experts: keys a lane of 16
        constexpr int KM = decltype(most)::value;
        if (s.E <= 32) launch_topk<RowSelect<2, KM>>(s, c, logits, out, chunk_cnt, st);
        else if (s.E <= 64) launch_topk<RowSelect<4, KM>>(s, c, logits, out, chunk_cnt, st);
        else if (s.E <= 128) launch_topk<RowSelect<8, KM>>(s, c, logits, out, chunk_cnt, st);
        else if constexpr (KM == 8) launch_topk<RowSelect<16, KM>>(s, c, logits, out, chunk_cnt, st);
    };
    if (rows_select(s) && s.k <= 8) rows_of(std::integral_constant<int, 8>{});
    else if (s.E <= 128) rows_of(std::integral_constant<int, kMaxTopK>{});
    else if (s.E <= 256) launch_topk<WaveSelect<4>>(s, c, logits, out, chunk_cnt, st);
    else if (s.E <= 512) launch_topk<WaveSelect<8>>(s, c, logits, out, chunk_cnt, st);
    else launch_topk<WaveSelect<16>>(s, c, logits, out, chunk_cnt, st);
    if (n > 1 && n <= kFewChunks) {
        hipLaunchKernelGGL((rows_kernel<false>), dim3(n), dim3(kChunkThreads), 0, st, out.topk_idx, s.T, s.k, c.tokens,
                           n, s.e_start, s.e_count, chunk_cnt, (int32_t*)out.counts, (int32_t*)out.offsets,
                           (int32_t*)out.perm, (int32_t*)out.inv_perm);
    } else if (n > 1) {
        hipLaunchKernelGGL(chunk_scan_kernel, dim3((s.e_count + kScanExperts - 1) / kScanExperts), dim3(kChunkThreads), 0, st,
                           chunk_cnt, n, s.e_count, (int32_t*)out.counts);
        hipLaunchKernelGGL((rows_kernel<true>), dim3(n), dim3(kChunkThreads), 0, st, out.topk_idx, s.T, s.k, c.tokens,
                           n, s.e_start, s.e_count, chunk_cnt, (int32_t*)out.counts, (int32_t*)out.offsets,
                           (int32_t*)out.perm, (int32_t*)out.inv_perm);
    }
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// ------------------------------------------------ routing without a caller workspace
// For callers that may not allocate (code under graph capture, tight serving loops): the
// per-chunk histogram lives in a file-scope device array instead of a workspace argument.
// Each device holds its own copy of the array at its own address, looked up once per
// device (with that device current) and kept; host code never uses the array's name as an
// address.  Every entry the kernels read is written earlier in the same call, so nothing
// has to be cleared; calls that overlap on one device share the array and race.
static __device__ __align__(256) unsigned char scratch[kRouteStaticScratchBytes];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];

int route_static_launch(const moe_shape_t& s, const float* logits, const moe_routing_t& out,
                        hipStream_t st) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_ERR_HIP;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        ptr = g_scratch_ptr[dev];
        if (!ptr) {
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MOE_ERR_HIP;
            g_scratch_ptr[dev] = ptr;
        }
    }
    return route_launch(s, logits, out, ptr, st);
}

}  // namespace uniep
