// bf16 MFMA tile machinery for gfx950 (CDNA4): operands by global->LDS DMA, fragments by
// LDS reads that run one k-sub-step ahead of the matrix instructions.
//
// A workgroup is 8 waves (two per SIMD) and owns an output tile of 256 x 256: 256 "row"
// indices (the B role of the MFMA: one index per lane) by 256 "column" indices (the A role:
// 16 values per lane and accumulator, arranged so that a lane ends with runs of 8 consecutive
// columns and stores 16 bytes).  Wave w = 4 wm + wn owns rows [128 wm, +128) as 4 fragments
// of 32 and columns [64 wn, +64) as 2 fragments of 32: 8 accumulators of
// v_mfma_f32_32x32x16_bf16, 6 fragment reads per 8 matrix instructions.  A tile of a row-tile GEMM may have
// 32 rows more (see TileRule): the two waves of a wave column then each multiply them by one of its two
// column fragments, a ninth accumulator.
//
// K advances in stages of 64.  A stage of an operand is a 32 KB LDS image in one of two forms (36 KB for 288 rows):
//   KC  the operand's k runs along its memory rows (activations [rows, k]; weights read
//       "transposed"): image [288 rows][128 B], the 16-byte chunk c of row r at chunk position
//       c ^ ((r >> 1) & 7), fragments by ds_read_b128;
//   KS  the operand's k is its memory row index (weights [k, n]; both operands of the
//       weight-gradient GEMMs): image [64 k][512 B], the 16-byte chunk c of k row k at chunk
//       position c ^ ((k & 3) << 2), fragments by ds_read_b64_tr_b16, which hands lane l of a
//       group of 16 the element l % 4 of the 8-byte pieces that lanes 4e + l / 4 addressed
//       (e = 0..3): four k rows of one column.
// Both swizzles make the fragment reads bank-conflict free, and both are applied by the DMA
// side through the choice of the global address each lane fetches: a DMA instruction writes
// lane p's 16 bytes to (LDS base) + 16 p, so nothing is staged in registers and no LDS
// write instruction or register transpose exists.
//
// Two stage buffers (136 KB of LDS; three, 144 KB, for tiles of up to 128 rows, see mma_low).  The first two stages are requested together, stage t+2 right behind the barrier that
// ends the fragment reads of stage t, so it has a whole stage of matrix work to land; one
// workgroup barrier per stage.  The fragment reads are inline assembly: the compiler would put
// a full vmcnt(0) in front of every LDS read it knows about while a DMA load is in flight.
// The waits that make their results usable are therefore written by hand (lgkmcnt counts,
// LDS operations complete in order) and tie the fragment registers, so that no matrix
// instruction can be scheduled ahead of them.
#pragma once
#include "common.hpp"

namespace uniep {

constexpr int BK = 64;
constexpr int BN = 256;                 // tile columns (A role)
constexpr int BMAX = 256;               // tile rows (B role) of the waves' own fragments
constexpr int kMoreRows = 32;           // and those that a wave column shares
enum OperandForm { kKc = 0, kKs = 1, kKsPair = 2 };   // of an LDS image; the last see KsPairLoader
constexpr int kOperandBytes = 32768;    // 256 rows or columns, one stage
constexpr int kRowBytes = kOperandBytes + kMoreRows * 128;
constexpr int kStageBytes = kRowBytes + kOperandBytes;   // rows (B role) first, columns (A role) second
constexpr int kLowRows = 128;           // tiles with no more rows
constexpr int kLowRowBytes = kLowRows * 128;
constexpr int kLowStageBytes = kLowRowBytes + kOperandBytes;
constexpr int kMmaSmem = 3 * kLowStageBytes;
static_assert(kMmaSmem >= 2 * kStageBytes, "");
constexpr int kMmaThreads = 512;

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void glb_void_t;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
__device__ __forceinline__ u32x4_t zero4() { return u32x4_t{0u, 0u, 0u, 0u}; }

// This thread's coordinates, derived from an opaque copy of threadIdx.x.  Address arithmetic
// that depends only on threadIdx.x is loop-invariant for the persistent task loop, so the
// compiler computes all of it once at kernel start, runs out of registers and reloads it from
// scratch next to the stores (each reload waits for the previous store to complete).  A task
// makes its own Lane before its main loop and another one for its epilogue.
struct Lane {
    int tid, l, l31, hf, w, wm, wn;
    __device__ __forceinline__ Lane() {
        unsigned t = threadIdx.x;
        asm volatile("" : "+v"(t));
        tid = (int)t;
        l = tid & 63;
        l31 = tid & 31;
        hf = (tid >> 5) & 1;
        w = tid >> 6;
        wm = tid >> 8;
        wn = (tid >> 6) & 3;
    }
    __device__ __forceinline__ int wave_uniform() const { return __builtin_amdgcn_readfirstlane(w); }
};

// MFMA row index i (0..31) -> position of that column inside the 32 columns of an A-role
// fragment: accumulator element v of lane half hf holds MFMA row 8 (v / 4) + 4 hf + v % 4, and
// this bit swap turns v = 0..7 into 8 consecutive columns (16 hf' ... see acc_col()).
__device__ __forceinline__ int swap23(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }

// Tile row / column of accumulator (tf, af) element v of this lane.
__device__ __forceinline__ int acc_row(const Lane& ln, int tf) { return 128 * ln.wm + 32 * tf + ln.l31; }
// first of the 8 consecutive columns that elements v = 8 vg .. 8 vg + 7 hold
__device__ __forceinline__ int acc_col8(const Lane& ln, int af, int vg) {
    return 64 * ln.wn + 32 * af + 16 * vg + 8 * ln.hf;
}

// ------------------------------------------------------------------ fragment addresses
struct FragAddr {
    uint32_t b[4];   // B role: KC -> per k-sub-step (+ tf * 4096); KS -> b[0] + ((tf << 6) ^ b[1]) per row fragment (+ kk * 8192 + hr * 2048)
    uint32_t a[4];   // A role: KC -> per k-sub-step (+ af * 4096); KS -> a[0..1] per column fragment (+ kk * 8192 + hr * 2048)
    uint32_t more;   // B role, KC: from this wave's first row to row 256
};

// kKsPair: a column fragment is 16 columns of one matrix and the same 16 of another (GEMM1: gate, up), so that it yields
// h by itself (the images of KsPairLoader).
template <int A_FORM, bool B_KS>
__device__ __forceinline__ void frag_addresses(FragAddr& fa, uint32_t lds0, const Lane& ln) {
    const int l = ln.l;
    const int wm = ln.wm, wn = ln.wn;
    const int kh = ln.hf, l31 = ln.l31;
    const int g = (l >> 4) & 1, jj = l & 15, e = jj >> 2, q = jj & 3;
    if (B_KS) {
        // chunk of row fragment tf = (16 wm + 2 g + q / 2) | ((tf ^ e) << 2): the swizzle only touches the
        // fragment bits, so one base and the lane's e << 6 describe all four addresses
        fa.b[0] = lds0 + (8 * kh + e) * 512 + ((16 * wm + 2 * g + (q >> 1)) << 4) + (q & 1) * 8;
        fa.b[1] = e << 6;
        fa.b[2] = fa.b[3] = 0;
    } else {
        const int x0 = (l >> 1) & 7;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            fa.b[kk] = lds0 + (128 * wm + l31) * 128 + (((2 * kk + kh) ^ x0) << 4);
    }
    const uint32_t a0 = lds0 + kRowBytes;
    fa.more = (BMAX - 128 * wm) * 128;
    if (A_FORM != kKc) {
        const int sq = ((q & 1) << 1) | (q >> 1);   // piece -> position of its 4 columns inside the 16
#pragma unroll
        for (int af = 0; af < 2; ++af) {
            if (A_FORM == kKsPair) {
                const int c = (4 * wn + 2 * af + (sq >> 1)) ^ (e << 2) ^ (2 * g);
                fa.a[af] = a0 + g * (kOperandBytes / 2) + (8 * kh + e) * 256 + (c << 4) + (sq & 1) * 8;
            } else {
                const int c = 8 * wn + 4 * af + 2 * g + (sq >> 1);
                fa.a[af] = a0 + (8 * kh + e) * 512 + ((c ^ (e << 2)) << 4) + (sq & 1) * 8;
            }
        }
        fa.a[2] = fa.a[3] = 0;
    } else {
        const int n = swap23(l31);
        const int x1 = (n >> 1) & 7;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            fa.a[kk] = a0 + (64 * wn + n) * 128 + (((2 * kk + kh) ^ x1) << 4);
    }
}

// ------------------------------------------------------------------ fragments
struct Frags {
    u32x4_t b[4];   // B role, one per row fragment
    u32x4_t a[2];   // A role, one per column fragment
    u32x4_t more;   // B role, rows 256..287
};

// The two halves of a transposing read land in the low and high register pair of one
// 128-bit fragment: the pair is addressed through a 64-bit view of the same registers.
#define UNIEP_TR2(dst, addr, off, next)                                                            \
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:" #off "\n ds_read_b64_tr_b16 %1, %2 offset:" #off "+" #next \
                 : "=&v"(lo_), "=&v"(hi_) : "v"(addr) : "memory");                                   \
    dst = u32x4_t{lo_[0], lo_[1], hi_[0], hi_[1]}

// FORM: kKs = k rows of 512 bytes, kKsPair = of 256 bytes
template <int FORM, int KK>
__device__ __forceinline__ void read_ks(u32x4_t& dst, uint32_t addr) {
    u32x2_t lo_, hi_;
    if (FORM == kKs) {
        if (KK == 0) { UNIEP_TR2(dst, addr, 0, 2048); }
        else if (KK == 1) { UNIEP_TR2(dst, addr, 8192, 2048); }
        else if (KK == 2) { UNIEP_TR2(dst, addr, 16384, 2048); }
        else { UNIEP_TR2(dst, addr, 24576, 2048); }
    } else {
        if (KK == 0) { UNIEP_TR2(dst, addr, 0, 1024); }
        else if (KK == 1) { UNIEP_TR2(dst, addr, 4096, 1024); }
        else if (KK == 2) { UNIEP_TR2(dst, addr, 8192, 1024); }
        else { UNIEP_TR2(dst, addr, 12288, 1024); }
    }
}
#undef UNIEP_TR2

template <int F>
__device__ __forceinline__ void read_kc(u32x4_t& dst, uint32_t addr) {
    if (F == 0) asm volatile("ds_read_b128 %0, %1" : "=&v"(dst) : "v"(addr) : "memory");
    else if (F == 1) asm volatile("ds_read_b128 %0, %1 offset:4096" : "=&v"(dst) : "v"(addr) : "memory");
    else if (F == 2) asm volatile("ds_read_b128 %0, %1 offset:8192" : "=&v"(dst) : "v"(addr) : "memory");
    else asm volatile("ds_read_b128 %0, %1 offset:12288" : "=&v"(dst) : "v"(addr) : "memory");
}

// Fragments of k-sub-step KK of the stage whose images lie `boff` (rows) and `aoff` (columns) bytes behind the first one's.
template <int NTF, int MORE, int A_FORM, bool B_KS, int KK>
__device__ __forceinline__ void read_frags(Frags& f, const FragAddr& fa, uint32_t boff, uint32_t aoff) {
    if (A_FORM != kKc) {
        read_ks<A_FORM, KK>(f.a[0], fa.a[0] + aoff);
        read_ks<A_FORM, KK>(f.a[1], fa.a[1] + aoff);
    } else {
        const uint32_t ad = fa.a[KK] + aoff;
        read_kc<0>(f.a[0], ad);
        read_kc<1>(f.a[1], ad);
    }
    if (B_KS) {
        const uint32_t bd = fa.b[0] + boff;
        if (NTF > 0) read_ks<kKs, KK>(f.b[0], bd + fa.b[1]);
        if (NTF > 1) read_ks<kKs, KK>(f.b[1], bd + (fa.b[1] ^ 64u));
        if (NTF > 2) read_ks<kKs, KK>(f.b[2], bd + (fa.b[1] ^ 128u));
        if (NTF > 3) read_ks<kKs, KK>(f.b[3], bd + (fa.b[1] ^ 192u));
    } else {
        const uint32_t bd = fa.b[KK] + boff;
        if (NTF > 0) read_kc<0>(f.b[0], bd);
        if (NTF > 1) read_kc<1>(f.b[1], bd);
        if (NTF > 2) read_kc<2>(f.b[2], bd);
        if (NTF > 3) read_kc<3>(f.b[3], bd);
        if (MORE) read_kc<0>(f.more, bd + fa.more);
    }
}

// Wait until at most N LDS operations are outstanding; ties the fragment registers.
template <int N, int MORE>
__device__ __forceinline__ void wait_frags(Frags& f) {
    if (MORE)
        asm volatile("s_waitcnt lgkmcnt(%7)"
                     : "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]), "+v"(f.b[3]), "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.more)
                     : "n"(N) : "memory");
    else
        asm volatile("s_waitcnt lgkmcnt(%6)"
                     : "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]), "+v"(f.b[3]), "+v"(f.a[0]), "+v"(f.a[1])
                     : "n"(N) : "memory");
}

// Accumulators of a wave: a[row fragment][column fragment], and rows 256..287 by one of the column fragments.
struct Acc {
    f32x16_t a[4][2];
    f32x16_t more;
};

// The matrix instructions of one k-sub-step (fragments `cur`) with the fragment reads of sub-step KK
// (into `nxt`) between the first three of them: a wave issues in order, and a matrix instruction
// keeps its pipe busy for 32 clocks during which the same wave may issue other instructions, so
// the reads cost no matrix issue slot, and the LDS sees them spread out instead of in bursts of
// six to twelve from every wave at once.
// MORE = 1 + the column fragment that this wave multiplies rows 256..287 by; 0 = the tile has none.
template <int NTF, int MORE, int A_FORM, bool B_KS, int KK>
__device__ __forceinline__ void mfma_step_reading(const Frags& cur, Frags& nxt, const FragAddr& fa, uint32_t boff,
                                                  uint32_t aoff, Acc& acc) {
    auto mm = [&](int tf, int af) {
        acc.a[tf][af] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, cur.a[af]),
                                                                __builtin_bit_cast(bf16x8_t, cur.b[tf]), acc.a[tf][af], 0, 0, 0);
    };
    const uint32_t ad = (A_FORM != kKc ? 0u : fa.a[KK]) + aoff, bd = (B_KS ? fa.b[0] : fa.b[KK]) + boff;
    auto rb = [&](int tf) {
        if (B_KS) {
            if (tf == 0) read_ks<kKs, KK>(nxt.b[0], bd + fa.b[1]);
            if (tf == 1) read_ks<kKs, KK>(nxt.b[1], bd + (fa.b[1] ^ 64u));
            if (tf == 2) read_ks<kKs, KK>(nxt.b[2], bd + (fa.b[1] ^ 128u));
            if (tf == 3) read_ks<kKs, KK>(nxt.b[3], bd + (fa.b[1] ^ 192u));
        } else {
            if (tf == 0) read_kc<0>(nxt.b[0], bd);
            if (tf == 1) read_kc<1>(nxt.b[1], bd);
            if (tf == 2) read_kc<2>(nxt.b[2], bd);
            if (tf == 3) read_kc<3>(nxt.b[3], bd);
        }
    };
    auto ra = [&](int af) {
        if (A_FORM != kKc) {
            if (af == 0) read_ks<A_FORM, KK>(nxt.a[0], fa.a[0] + aoff);
            else read_ks<A_FORM, KK>(nxt.a[1], fa.a[1] + aoff);
        } else {
            if (af == 0) read_kc<0>(nxt.a[0], ad);
            else read_kc<1>(nxt.a[1], ad);
        }
    };
    if (NTF > 0) mm(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    ra(0);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 0) mm(0, 1);
    __builtin_amdgcn_sched_barrier(0);
    ra(1);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 1) mm(1, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 0) rb(0);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 1) mm(1, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 1) rb(1);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 2) mm(2, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 2) rb(2);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 2) mm(2, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 3) rb(3);
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 3) mm(3, 0);
    if (MORE) {
        __builtin_amdgcn_sched_barrier(0);
        read_kc<0>(nxt.more, bd + fa.more);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (NTF > 3) mm(3, 1);
    if (MORE)
        acc.more = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, cur.a[MORE == 2]),
                                                           __builtin_bit_cast(bf16x8_t, cur.more), acc.more, 0, 0, 0);
}

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ------------------------------------------------------------------ DMA sources
// Every loader moves one operand: issue(dst) requests the next stage into the image at
// `dst` (4 DMA instructions per wave, 1 KB each) and advances; DMA instruction i of wave w
// fills the 1 KB block u = 4 w + i of the image, and a fifth one of waves 0..3 block 32 + w (rows 256..287).
__device__ __forceinline__ void dma16(const char* src, char* dst) {
    __builtin_amdgcn_global_load_lds((glb_void_t*)src, (lds_void_t*)dst, 16, 0, 0);
}
// this wave's first 1 KB block of an operand image, as a wave-uniform byte offset
__device__ __forceinline__ int wave_block_off() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 4096;
}
__device__ __forceinline__ int wave_block_off(const Lane& ln) { return ln.wave_uniform() * 4096; }

// KC image: block u holds rows 8u .. 8u+7; lane p moves the chunk of row 8u + p/8 that belongs
// at chunk position p%8.  row_of(i) / chunk_of(i) tell a task which (row, chunk) this lane
// fetches with instruction i; p[i] = address of that chunk in stage 0.
struct KcGeom {
    static __device__ __forceinline__ int row(const Lane& ln, int i) { return 8 * (4 * ln.w + i) + (ln.l >> 3); }
    static __device__ __forceinline__ int chunk(const Lane& ln, int i) { return (ln.l & 7) ^ ((row(ln, i) >> 1) & 7); }
    // of the fifth instruction (waves 0..3)
    static __device__ __forceinline__ int more_row(const Lane& ln) { return BMAX + 8 * ln.w + (ln.l >> 3); }
    static __device__ __forceinline__ int more_chunk(const Lane& ln) { return (ln.l & 7) ^ ((more_row(ln) >> 1) & 7); }
};
// The column operands of the row-tile GEMMs (weights) are addressed by scalar bases and two 32-bit offsets a lane, for the
// instructions with i even and odd: a 64-bit address a lane and instruction takes 8 registers and 8 vector additions a stage.
typedef const __attribute__((address_space(1))) char* glb_ptr_t;
__device__ __forceinline__ void dma16s(glb_ptr_t base, uint32_t off, char* dst) {
    asm volatile("" : "+s"(base), "+v"(off));   // scalar base + lane offset, not one 64-bit lane address
    __builtin_amdgcn_global_load_lds((glb_void_t*)(base + off), (lds_void_t*)dst, 16, 0, 0);
}
// What mma_loop asks of a loader beside issue(), for one that knows its addresses without memory (see KsGatherLoader).
template <class L>
struct PlainLoader {
    __device__ __forceinline__ void prepare() {}
    __device__ __forceinline__ void prepare_two() {}
    __device__ __forceinline__ void fetch() {}
    __device__ __forceinline__ void issue_first(char* dst) { static_cast<L*>(this)->issue(dst); }
    __device__ __forceinline__ void issue_second(char* dst) { static_cast<L*>(this)->issue(dst); }
};
// Rows whose k runs on (weights read transposed): every stage is 128 bytes further along each row, and after `left` more stages
// in a second matrix of the same layout (W_gate then W_up along k), `delta` bytes on.
struct KcLoader : PlainLoader<KcLoader> {
    glb_ptr_t p[4];     // first k of the instruction's eight rows in the stage to come (uniform)
    uint32_t off[2];
    long long delta;
    int left;
    // n rows from first_row on, ld_bytes apart (n a multiple of 8; those past the last alias the last eight)
    __device__ __forceinline__ void init(const Lane& ln, const char* first_row, int n, uint32_t ld_bytes) {
        const int w = ln.wave_uniform();
        left = INT_MAX;
        delta = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = (glb_ptr_t)(first_row + (size_t)min(8 * (4 * w + i), n - 8) * ld_bytes);
#pragma unroll
        for (int i = 0; i < 2; ++i) off[i] = (ln.l >> 3) * ld_bytes + KcGeom::chunk(ln, i) * 16;
    }
    __device__ __forceinline__ void issue(char* dst) {
        char* d = dst + wave_block_off();
        const long long jump = left == 0 ? delta : 0;
        --left;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] += jump;
            dma16s(p[i], off[i & 1], d + i * 1024);
            p[i] += BK * 2;
        }
    }
};
// The row operand: up to 288 rows, row_of(r) = address of row r's first k (r below `rows`; rows past the last alias it).
struct RowLoader : PlainLoader<RowLoader> {
    const char* p[4];
    const char* pm;   // the fifth instruction's
    int n;            // blocks of this wave that hold rows of the tile (wave-uniform); bit 3: the fifth one does too
    __device__ __forceinline__ bool full() const { return (n & 7) == 4; }   // at least 4 requests a stage
    template <class F>
    __device__ __forceinline__ void init(const Lane& ln, int rows, F row_of) {
        const int w = ln.wave_uniform();
        n = min(4, max(0, (rows - 32 * w + 7) >> 3)) | (w < 4 && rows > BMAX + 8 * w ? 8 : 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = row_of(min(KcGeom::row(ln, i), rows - 1)) + KcGeom::chunk(ln, i) * 16;
        pm = p[0];
        if (n & 8) pm = row_of(min(KcGeom::more_row(ln), rows - 1)) + KcGeom::more_chunk(ln) * 16;
    }
    __device__ __forceinline__ void issue(char* dst) {
        const int off = wave_block_off();
        char* d = dst + off;
        // one branch for a wave whose blocks all hold rows: a branch around every request delays the last of them
        if ((n & 7) == 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) dma16(p[i], d + i * 1024);
        } else if (n & 7) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < (n & 7)) dma16(p[i], d + i * 1024);
        }
        if (n & 8) dma16(pm, dst + kOperandBytes + (off >> 2));
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] += BK * 2;
        pm += BK * 2;
    }
};
// The same for tiles of up to 128 rows: instruction i of wave w fills block 2 w + i.  Both are always issued (rows past the last
// alias it), so that every wave has as many requests on their way.
struct LowRowLoader {
    const char* p[2];
    template <class F>
    __device__ __forceinline__ void init(const Lane& ln, int rows, F row_of) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * (2 * ln.w + i) + (ln.l >> 3);
            p[i] = row_of(min(r, rows - 1)) + ((ln.l & 7) ^ ((r >> 1) & 7)) * 16;
        }
    }
    __device__ __forceinline__ void issue(char* dst) {
        char* d = dst + (wave_block_off() >> 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dma16(p[i], d + i * 1024);
            p[i] += BK * 2;
        }
    }
};

// KS image: block u holds k rows 2u, 2u+1 (512 B = 32 chunks each); lane p moves the chunk of
// k row 2u + p/32 that belongs at chunk position p%32.
struct KsGeom {
    static __device__ __forceinline__ int krow(const Lane& ln, int i) { return 2 * (4 * ln.w + i) + ln.hf; }
    static __device__ __forceinline__ int chunk(const Lane& ln, int i) { return ln.l31 ^ ((krow(ln, i) & 3) << 2); }
};
// Dense matrix [K, n], K a multiple of 64.
struct KsLoader : PlainLoader<KsLoader> {
    glb_ptr_t p[4];     // first k row of the instruction in the stage to come (uniform)
    uint32_t off[2];
    uint32_t step;      // 64 memory rows
    // columns from `first` (first_row's address, of n) on, ld_bytes a k row; chunks past n alias the last one
    __device__ __forceinline__ void init(const Lane& ln, const char* first_row, int first, int n, uint32_t ld_bytes) {
        const int w = ln.wave_uniform();
        step = BK * ld_bytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = (glb_ptr_t)(first_row + (size_t)(2 * (4 * w + i)) * ld_bytes);
#pragma unroll
        for (int i = 0; i < 2; ++i) off[i] = ln.hf * ld_bytes + min(first + KsGeom::chunk(ln, i) * 8, n - 8) * 2;
    }
    __device__ __forceinline__ void issue(char* dst) {
        char* d = dst + wave_block_off();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dma16s(p[i], off[i & 1], d + i * 1024);
            p[i] += step;
        }
    }
};
// Two such matrices, 128 columns of each (GEMM1: gate, up): two images [64 k][256 B], one behind the other, the chunk c of k row
// k at c ^ ((k & 3) << 2), in the second with bit 1 turned over as well.  Instructions 0, 1 of a wave move 4 k rows
// each of the first, 2, 3 of the second.
struct KsPairLoader : PlainLoader<KsPairLoader> {
    glb_ptr_t p[2];     // this wave's first k row in the stage to come (uniform)
    uint32_t off[2];
    uint32_t ld;
    __device__ __forceinline__ void init(const Lane& ln, const char* row0, const char* row1, int first, int n, uint32_t ld_bytes) {
        ld = ld_bytes;
        p[0] = (glb_ptr_t)(row0 + (size_t)(8 * ln.wave_uniform()) * ld);
        p[1] = (glb_ptr_t)(row1 + (size_t)(8 * ln.wave_uniform()) * ld);
        const int e = ln.l >> 4, c = (ln.l & 15) ^ (e << 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) off[i] = e * ld + min(first + (c ^ (2 * i)) * 8, n - 8) * 2;
    }
    __device__ __forceinline__ void issue(char* dst) {
        char* d = dst + (wave_block_off() >> 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) dma16s(p[i >> 1] + (i & 1) * 4 * ld, off[i >> 1], d + (i >> 1) * (kOperandBytes / 2) + (i & 1) * 1024);
        p[0] += BK * ld;
        p[1] += BK * ld;
    }
};
// Reduction over K memory rows with K not a multiple of 64 (the rows of one expert): k rows at
// and beyond K are written as zeros instead of fetched.  The four k rows a lane moves are
// krow(0) + 2i, and its chunk depends on i only through i % 2, so two addresses describe them:
// p[j] = address of (k row krow(j), chunk(j)) of stage 0, j = 0, 1; instructions 2, 3 are 4
// memory rows further.
__device__ __forceinline__ void lds_zero16(char* dst) {
    const uint32_t ad = lds_addr(dst) + (threadIdx.x & 63) * 16;   // (cheap; recomputed where it is used)
    asm volatile("ds_write_b128 %0, %1" : : "v"(ad), "v"(zero4()) : "memory");
}

struct KsTailLoader : PlainLoader<KsTailLoader> {
    __device__ __forceinline__ bool full() const { return true; }   // 4 requests a stage, but the last
    const char* p[2];
    long long ld_bytes;   // one memory row (wave-uniform)
    int k0;               // reduction index of instruction 0's k row in the stage to come
    int K;
    __device__ __forceinline__ void issue(char* dst) {
        char* d = dst + wave_block_off();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (k0 + 2 * i < K) dma16(p[i & 1] + (i >> 1) * 4 * ld_bytes, d + i * 1024);
            else lds_zero16(d + i * 1024);
        }
        p[0] += BK * ld_bytes;
        p[1] += BK * ld_bytes;
        k0 += BK;
    }
};
// The same with a gather: reduction index k is memory row rows[k] of a [T, ld] matrix.  The
// row indices of the first two stages are fetched at once, those of every later one by a plain load right behind the DMA of the stage before
// it, complete by the barrier in between.  init() is called once per tile, after
// coloff[] is filled.
// A wave moves 8 rows a stage, and each half of it 4 of them: lane l loads the index for instruction l % 4, and prepare()
// hands it to the four lanes of its quad (a load for each instruction was four times as many, and 0.2 to 0.4 % slower).
// prepare() turns the fetched indices into the four source addresses, and the main loop calls
// it for both loaders before either requests anything: while a DMA is pending the compiler puts
// a full vmcnt(0) in front of every use of a register that an ordinary load filled (it cannot
// order the two kinds of operation), so address arithmetic between the DMA instructions would
// make every request wait for the one before it to land.
struct KsGatherLoader {
    const char* src;          // matrix base
    uint32_t coloff[2];       // byte offset, inside a memory row, of the chunk instructions i, i % 2 = j move
    long long ld_bytes;       // wave-uniform
    const int32_t* rows;      // row_tok + first row of the expert (wave-uniform)
    int32_t tok;              // memory row of instruction l % 4 in the stage whose DMA goes out next
    int32_t tok1;             // the same of stage 1, until that is requested
    const char* a[4];         // the instructions' addresses (prepare)
    int k0;                   // reduction index of instruction 0's k row in that stage
    int mine;                 // from there to the one that this lane fetches the index of
    int K;
    __device__ __forceinline__ bool full() const { return true; }
    __device__ __forceinline__ void fetch() { tok = rows[min(k0 + mine, K - 1)]; }
    __device__ __forceinline__ void init(const Lane& ln, const char* src_, long long ld_bytes_, const int32_t* rows_, int K_) {
        src = src_;
        ld_bytes = ld_bytes_;
        rows = rows_;
        K = K_;
        k0 = KsGeom::krow(ln, 0);
        mine = 2 * (ln.l & 3);
        tok = tok1 = 0;
        if (K <= 0) return;   // an expert without rows has no index to read: its first one may lie past the last row
        fetch();
        tok1 = rows[min(k0 + BK + mine, K - 1)];
    }
    template <int I>
    __device__ __forceinline__ const char* address(int32_t from) const {   // quad_perm [I, I, I, I]
        const int32_t t = __builtin_amdgcn_update_dpp(0, from, I * 0x55, 0xf, 0xf, true);
        const char* p = src + (long long)t * ld_bytes + coloff[I & 1];
        asm volatile("" : "+v"(p));   // the address exists before the first request
        return p;
    }
    __device__ __forceinline__ void prepare() {
        a[0] = address<0>(tok);
        a[1] = address<1>(tok);
        a[2] = address<2>(tok);
        a[3] = address<3>(tok);
    }
    __device__ __forceinline__ void prepare_two() {
        prepare();
        asm volatile("" : "+v"(tok1));   // here before the first request, so that issue_second() does not wait for it behind that
    }
    __device__ __forceinline__ void issue_first(char* dst) {
        char* d = dst + wave_block_off();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (k0 + 2 * i < K) dma16(a[i], d + i * 1024);
            else lds_zero16(d + i * 1024);
        }
        k0 += BK;
    }
    __device__ __forceinline__ void issue_second(char* dst) {
        tok = tok1;
        prepare();
        issue_first(dst);
    }
    __device__ __forceinline__ void issue(char* dst) {
        issue_first(dst);
        fetch();
    }
};

// ------------------------------------------------------------------ main loop
// acc[tf][af] += (column fragment af) x (row fragment tf) over nk stages (nk >= 1).
// NTF = row fragments of this wave that hold rows of the tile (0..4): the others are neither
// read nor multiplied.  Every wave takes part in the DMA and in the barriers whatever its NTF.
// Pipeline per stage t (buffer t % 2), k-sub-steps 0..3 of 16:
//   sub-step s < 3: wait for the fragments of s, 8 matrix instructions with the fragment reads
//                   of s+1 between the first three of them (mfma_step_reading);
//   sub-step 3:     wait for its fragments (the last reads of the buffer), wait for this wave's
//                   DMA of stage t+1, barrier, request the row operand of stage t+2 into the
//                   buffer just freed, request the fragments of (t+1, 0), 8 matrix instructions,
//                   request the column operand of stage t+2 (a CU takes about 64 DMA requests
//                   before issue blocks, which is what one stage has: the second half goes out
//                   behind a burst of matrix work instead of in front of it; 1 % on the step).
// Stages 0 and 1 are requested together: stage 1 used to wait for stage 0 to land, and had then only that stage's matrix work to arrive
// in, once a tile.  A reduction over an expert's rows has `last` sub-steps in its last stage: those that hold only zeros were an eighth of the matrix
// work at 256 rows an expert.  Backward pass, us, before / with both stages together / without the empty sub-steps too: 8192 tokens on 128 experts of 2048 x 768
// 1570 / 1552 / 1531, 1000 585 / 570 / 557, 4099 on 64 of 2048 x 1408 1165 / 1152 / 1120.  Whole training steps, before / both: 8192 on 128 of 2048 x 768 2288 / 2251,
// 8001 with Zipf(1.2) routing 2401 / 2376, 8192 on 32 of 256 of 7168 x 2048 2910 / 2825, 60001 on 32 of 256 of 2304 x 1024, added to fp32 gradients, 3181 / 3144.
template <int NTF, int MORE, int A_FORM, bool B_KS, class LB, class LA>
__device__ __forceinline__ void mma_loop(LB& lb, LA& la, int nk, char* smem, const FragAddr& fa, Acc& acc, int last = 4) {
    int full = rfl(nk > (B_KS ? 2 : 1) && lb.full());
    asm volatile("" : "+s"(full));   // (otherwise the branches of issue() and of the wait are threaded, with scalar addresses in vector registers)
    lb.prepare_two();
    la.prepare_two();
    __builtin_amdgcn_sched_barrier(0);
    lb.issue_first(smem);
    la.issue_first(smem + kRowBytes);
    // stage 1 right behind stage 0: its requests wait for nothing but their turn
    if (nk > 1) {
        lb.issue_second(smem + kStageBytes);
        la.issue_second(smem + kStageBytes + kRowBytes);
    }
    // (a wave's requests of stage 1 are 8 or 9, or fewer where it has few rows or the reduction ends in it)
    if (full) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    lb.fetch();
    la.fetch();
    Frags f0, f1;
    if (NTF > 0) read_frags<NTF, MORE, A_FORM, B_KS, 0>(f0, fa, 0, 0);
    const int whole = B_KS ? nk - 1 : nk;   // the last stage of a reduction over rows may have fewer than 64
    for (int t = 0; t < whole; ++t) {
        const uint32_t boff = (t & 1) * kStageBytes, noff = kStageBytes - boff;
        __builtin_amdgcn_sched_barrier(0);
        if (NTF > 0) {
            wait_frags<0, MORE>(f0);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, MORE, A_FORM, B_KS, 1>(f0, f1, fa, boff, boff, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, MORE>(f1);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, MORE, A_FORM, B_KS, 2>(f1, f0, fa, boff, boff, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, MORE>(f0);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, MORE, A_FORM, B_KS, 3>(f0, f1, fa, boff, boff, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, MORE>(f1);
        }
        if (t + 1 < nk) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (t + 2 < nk) {
                lb.prepare();
                la.prepare();
                __builtin_amdgcn_sched_barrier(0);
                lb.issue(smem + boff);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // the matrix instructions of sub-step 3, with the first fragment reads of stage t+1 between them (behind the last
        // stage they read what is there: a branch around each of them costs every stage)
        if (NTF > 0) mfma_step_reading<NTF, MORE, A_FORM, B_KS, 0>(f1, f0, fa, noff, noff, acc);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 2 < nk) la.issue(smem + boff + kRowBytes);   // the second operand's requests behind a burst of matrix work
    }
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 0) wait_frags<0, MORE>(f0);
    if constexpr (B_KS && NTF > 0) {
        // sub-steps without a row are left out: they would add zeros
        const uint32_t boff = ((nk - 1) & 1) * kStageBytes;
        mfma_step_reading<NTF, MORE, A_FORM, B_KS, 1>(f0, f1, fa, boff, boff, acc);
        __builtin_amdgcn_sched_barrier(0);
        wait_frags<0, MORE>(f1);
        __builtin_amdgcn_sched_barrier(0);
        if (last > 1) {
            mfma_step_reading<NTF, MORE, A_FORM, B_KS, 2>(f1, f0, fa, boff, boff, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, MORE>(f0);
            __builtin_amdgcn_sched_barrier(0);
            if (last > 2) {
                mfma_step_reading<NTF, MORE, A_FORM, B_KS, 3>(f0, f1, fa, boff, boff, acc);
                __builtin_amdgcn_sched_barrier(0);
                wait_frags<0, MORE>(f1);
                __builtin_amdgcn_sched_barrier(0);
                if (last > 3) mfma_step_reading<NTF, MORE, A_FORM, B_KS, 3>(f1, f0, fa, boff, boff, acc);
                __builtin_amdgcn_sched_barrier(0);
                wait_frags<0, MORE>(f0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_barrier();   // every wave has read its last fragments: the buffers may be refilled
}

// The loop for reductions of one stage that is run whole, by a wave whose four fragments hold rows (see kShortSum).  The workgroup's other waves run mma_loop:
// as many barriers for one stage, two.
template <class LB, class LA>
__device__ __forceinline__ void mma_short(LB& lb, LA& la, char* smem, const FragAddr& fa, Acc& acc) {
    lb.prepare();
    la.prepare();
    __builtin_amdgcn_sched_barrier(0);
    lb.issue_first(smem);
    la.issue_first(smem + kRowBytes);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    Frags f0, f1;
    read_frags<4, 0, kKs, true, 0>(f0, fa, 0, 0);
    wait_frags<0, 0>(f0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step_reading<4, 0, kKs, true, 1>(f0, f1, fa, 0, 0, acc);
    __builtin_amdgcn_sched_barrier(0);
    wait_frags<0, 0>(f1);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step_reading<4, 0, kKs, true, 2>(f1, f0, fa, 0, 0, acc);
    __builtin_amdgcn_sched_barrier(0);
    wait_frags<0, 0>(f0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step_reading<4, 0, kKs, true, 3>(f0, f1, fa, 0, 0, acc);
    __builtin_amdgcn_sched_barrier(0);
    wait_frags<0, 0>(f1);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step_reading<4, 0, kKs, true, 3>(f1, f0, fa, 0, 0, acc);
    __builtin_amdgcn_sched_barrier(0);
    wait_frags<0, 0>(f0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();   // every wave has read its last fragments: the buffers may be refilled
}

// Row fragments of this wave that hold rows when the tile has `rows` of them.
__device__ __forceinline__ int active_row_frags(int rows) {
    const int mine = rows - 128 * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8));
    return __builtin_amdgcn_readfirstlane(mine <= 0 ? 0 : (mine >= 128 ? 4 : (mine + 31) >> 5));
}

// The loop for tiles of up to 128 rows (waves 4..7 only move operands): their stages are 48 KB, so that three buffers fit and
// stages t+1 and t+2 are on their way while stage t is multiplied.  The matrix work of a stage takes a quarter to a
// half of the time that its requests take to arrive: with two buffers such a tile took a round trip to memory a stage
// (training step of 256 tokens on 8 experts of 512 x 1024, 64 rows each, 135 -> 123 us; 4099 tokens on 64 experts of
// 2048 x 1408, tiles of 256 and 128 rows, forward 510 -> 502 us; Zipf(1.2) routing of 8001 tokens 2444 -> 2419 us).
template <int NTF, int A_FORM, class LA>
__device__ __forceinline__ void mma_low(LowRowLoader& lb, LA& la, int nk, char* smem, const FragAddr& fa, Acc& acc) {
    constexpr int kRequests = 6;   // of a wave, a stage
    constexpr uint32_t kA = kLowRowBytes - kRowBytes;   // fa.a is made for the larger row image
#pragma unroll
    for (int t = 0; t < 3; ++t)
        if (t < nk) {
            lb.issue(smem + t * kLowStageBytes);
            la.issue(smem + t * kLowStageBytes + kLowRowBytes);
        }
    if (nk > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kRequests) : "memory");
    else if (nk > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kRequests) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    Frags f0, f1;
    if (NTF > 0) read_frags<NTF, 0, A_FORM, false, 0>(f0, fa, 0, kA);
    uint32_t boff = 0;
    for (int t = 0; t < nk; ++t) {
        const uint32_t noff = boff == 2 * kLowStageBytes ? 0 : boff + kLowStageBytes;
        __builtin_amdgcn_sched_barrier(0);
        if (NTF > 0) {
            wait_frags<0, 0>(f0);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, 0, A_FORM, false, 1>(f0, f1, fa, boff, boff + kA, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, 0>(f1);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, 0, A_FORM, false, 2>(f1, f0, fa, boff, boff + kA, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, 0>(f0);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step_reading<NTF, 0, A_FORM, false, 3>(f0, f1, fa, boff, boff + kA, acc);
            __builtin_amdgcn_sched_barrier(0);
            wait_frags<0, 0>(f1);
        }
        if (t + 1 < nk) {
            // stage t+1 is here; stage t+2, if there is one, may still be on its way
            if (t + 2 < nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kRequests) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (t + 3 < nk) {
                lb.issue(smem + boff);
                la.issue(smem + boff + kLowRowBytes);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (NTF > 0) mfma_step_reading<NTF, 0, A_FORM, false, 0>(f1, f0, fa, noff, noff + kA, acc);
        boff = noff;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (NTF > 0) wait_frags<0, 0>(f0);
    __builtin_amdgcn_s_barrier();
}

__device__ __forceinline__ void zero_acc(Acc& acc, bool more) {
#pragma unroll
    for (int tf = 0; tf < 4; ++tf)
#pragma unroll
        for (int af = 0; af < 2; ++af)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc.a[tf][af][v] = 0.f;
    if (more)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc.more[v] = 0.f;
}

// A tile of a row-tile GEMM (nk >= 1; row_of as in RowLoader), by the loop for its rows and the wave's NTF (scalar branches: every
// wave runs exactly one instance, and all instances of a loop execute the same barriers).
// Instances for odd numbers of row fragments are 16 % of the library's code.  Without them (one and three fragments by the loops
// for two and four), us with / without: 128 experts of 2048 x 768 with 144, 208, 340 and 460 rows each, forward 340 / 344, 393 / 402,
// 562 / 577 and 727 / 736, backward 802 / 812, 933 / 942, 1252 / 1263 and 1548 / 1570; 24 of 4096 x 1536 with 460 467 / 479 and 1065 / 1074.  Fewer
// instances are faster only on small layers (8 experts of 512 x 1024 with 112 and 176 rows each 49.8 / 49.0 and 57.9 / 56.0,
// with 80 and 208 47.4 / 48.2 and 60.1 / 60.9).
template <int A_FORM, class LA, class F>
__device__ __forceinline__ void row_tile_gemm(const Lane& ln, LA& la, int nk, int rows, char* smem, const FragAddr& fa, Acc& acc,
                                              F row_of) {
    const int ntf = active_row_frags(rows);
    if (rows <= kLowRows) {
        LowRowLoader lb;
        lb.init(ln, rows, row_of);
        zero_acc(acc, false);
        if (ntf == 4) mma_low<4, A_FORM>(lb, la, nk, smem, fa, acc);
        else if (ntf == 3) mma_low<3, A_FORM>(lb, la, nk, smem, fa, acc);
        else if (ntf == 2) mma_low<2, A_FORM>(lb, la, nk, smem, fa, acc);
        else if (ntf == 1) mma_low<1, A_FORM>(lb, la, nk, smem, fa, acc);
        else mma_low<0, A_FORM>(lb, la, nk, smem, fa, acc);
        return;
    }
    RowLoader lb;
    lb.init(ln, rows, row_of);
    zero_acc(acc, true);
    if (rows > BMAX) {
        if (ln.wave_uniform() < 4) mma_loop<4, 1, A_FORM, false>(lb, la, nk, smem, fa, acc);
        else mma_loop<4, 2, A_FORM, false>(lb, la, nk, smem, fa, acc);
    } else if (ntf == 4) mma_loop<4, 0, A_FORM, false>(lb, la, nk, smem, fa, acc);
    else if (ntf == 3) mma_loop<3, 0, A_FORM, false>(lb, la, nk, smem, fa, acc);
    else if (ntf == 2) mma_loop<2, 0, A_FORM, false>(lb, la, nk, smem, fa, acc);
    else mma_loop<1, 0, A_FORM, false>(lb, la, nk, smem, fa, acc);
}

// Reductions of up to so many rows run their one stage whole (mma_short) where the gradients are written, not added to.  Such a pass is bound by memory, by
// the weights that the row tiles read and the gradients that these tiles write, and quicker tiles crowd the reads out: the tiles alone (a launch a
// phase) take 2 to 7 % less without their empty sub-steps, the pass takes more.  Backward pass, us, without / whole (tokens, experts of width and inner width; rows an
// expert): 33, 128 of 2048 x 768 (2) 535 / 525; 64, 256 of 2304 x 1024 (2) 1385 / 1358; 102, 512 of 2048 x 512 (2) 1269 / 1245; 33, 64 of 2048 x 1408 (3) 519 / 509;
// 107, 64 of 1280 x 896 (10) 235 / 231; but 128, 128 of 1024 x 384 (6) 157 / 159.  Over 18 shares of 10 layers the pass takes 1.5 % less with it from 2 to 10 rows
// an expert (from 1.5 % more to 2 % less), 1 % less at 24 and the same from 32 on.  With gradients added to fp32 buffers it takes 0.5 % more with it.
// For other waves, or by the loop above with all of its sub-steps, it costs long reductions 0.3 %: the more code, the slower they are.
constexpr int kShortSum = 32;
// A tile of a weight-gradient GEMM: both operands have k as their memory rows.  SHORT: see kShortSum.
template <bool SHORT, class LB, class LA>
__device__ __forceinline__ void weight_tile_gemm(LB& lb, LA& la, int nk, int rows, char* smem, const FragAddr& fa, Acc& acc) {
    zero_acc(acc, false);
    if (nk <= 0) return;   // empty reduction (an expert without rows): the tile is all zeros
    const int ntf = active_row_frags(rows);
    if (SHORT && lb.K <= kShortSum && ntf == 4) {
        mma_short(lb, la, smem, fa, acc);
        return;
    }
    const int last = rfl(((lb.K - 1) % BK) / 16 + 1);   // sub-steps of the last stage: the rest are zeros
    if (ntf == 4) mma_loop<4, 0, kKs, true>(lb, la, nk, smem, fa, acc, last);
    else if (ntf == 3) mma_loop<3, 0, kKs, true>(lb, la, nk, smem, fa, acc, last);
    else if (ntf == 2) mma_loop<2, 0, kKs, true>(lb, la, nk, smem, fa, acc, last);
    else if (ntf == 1) mma_loop<1, 0, kKs, true>(lb, la, nk, smem, fa, acc, last);
    else mma_loop<0, 0, kKs, true>(lb, la, nk, smem, fa, acc, last);
}

// ------------------------------------------------------------------ epilogue helpers
// The 8 consecutive columns of accumulator elements 8 vg .. 8 vg + 7, packed to bf16.
__device__ __forceinline__ u32x4_t pack8(const f32x16_t& a, int vg) {
    u32x4_t r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = pack_bf16x2(a[8 * vg + 2 * q], a[8 * vg + 2 * q + 1]);
    return r;
}

// Stores that cover whole 128-byte lines.  After the main loop a lane holds, per row fragment,
// 16-byte pieces of 32 different rows, so a store instruction straight from the accumulators
// touches 32 rows with 32 contiguous bytes each: four times the write requests of a row-major
// store, as partial lines, and the next tile's first loads queue behind them.  Instead every
// wave passes its 128 x 64 sub-tile through its own 16 KB of the (now idle) stage buffers:
// put() writes a lane's 16-byte pieces, get() hands lane l the piece l % NP of row
// (64 / NP) j + l / NP, so NP neighbouring lanes store one contiguous run of NP * 16 bytes.
// Rows are NP * 16 bytes apart and the piece position is XORed with row bits so that both
// directions are bank-conflict free.  Wave-private: LDS operations of a wave execute in
// order, no barrier is involved.  NP = 8: 64 bf16 columns per row (or 32 fp32); NP = 4: 32 bf16 columns.
template <int NP>
struct WaveRepack {
    char* base;   // this wave's 16 KB
    int l;        // lane
    __device__ __forceinline__ WaveRepack(char* smem, const Lane& ln) : base(smem + ln.w * 16384), l(ln.l) {}
    // eight neighbouring lanes of a put() hold eight consecutive rows: their 16-byte slots must differ
    static __device__ __forceinline__ int swz(int row) { return NP == 8 ? (row & 7) : ((row >> 1) & 3); }
    // piece pi (0..NP-1) of sub-tile row `row` (0..127)
    __device__ __forceinline__ void put(int row, int pi, u32x4_t v) {
        *(u32x4_t*)(base + row * (NP * 16) + ((pi ^ swz(row)) << 4)) = v;
    }
    __device__ __forceinline__ int get_row(int j) const { return (64 / NP) * j + l / NP; }
    __device__ __forceinline__ int get_piece() const { return l % NP; }
    __device__ __forceinline__ u32x4_t get(int j) const {
        const int row = get_row(j);
        return *(const u32x4_t*)(base + row * (NP * 16) + ((get_piece() ^ swz(row)) << 4));
    }
    // The same in 8-byte pieces (2 NP per row), for outputs that leave through 8-byte write-through
    // stores: lane l gets piece l % (2 NP) of row (32 / NP) j + l / (2 NP).
    __device__ __forceinline__ int get8_row(int j) const { return (32 / NP) * j + l / (2 * NP); }
    __device__ __forceinline__ int get8_piece() const { return l % (2 * NP); }
    __device__ __forceinline__ u32x2_t get8(int j) const {
        const int row = get8_row(j), p8 = get8_piece();
        return *(const u32x2_t*)(base + row * (NP * 16) + (((p8 >> 1) ^ swz(row)) << 4) + (p8 & 1) * 8);
    }
};

// The wave's 128 x 64 bf16 sub-tile of the accumulators, handed to store(tile row, tile column,
// 8 columns as 16 bytes) with 8 neighbouring lanes on one row (128 contiguous bytes); rows at
// and beyond `rows` and 8-column pieces at and beyond `cols` (tile coordinates) are left out.  MORE: the tile may have rows 256..287.
template <bool MORE, class StoreFn>
__device__ __forceinline__ void store_subtile_bf16(const Acc& acc, char* smem, int rows, int cols, StoreFn store) {
    const Lane ln;
    WaveRepack<8> rp(smem, ln);
    const int l31 = ln.l31, hf = ln.hf;
    const int wm = ln.wm, wn = ln.wn;
#pragma unroll
    for (int tf = 0; tf < 4; ++tf)
#pragma unroll
        for (int af = 0; af < 2; ++af)
#pragma unroll
            for (int vg = 0; vg < 2; ++vg) rp.put(32 * tf + l31, 4 * af + 2 * vg + hf, pack8(acc.a[tf][af], vg));
    const int col = 64 * wn + 8 * rp.get_piece();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int row = 128 * wm + rp.get_row(j);
        const u32x4_t v = rp.get(j);
        if (row < rows && col < cols) store(row, col, v);
    }
    if (MORE && rows > BMAX) {   // rows 256..287 by column fragment wm
        WaveRepack<4> rm(smem, ln);
#pragma unroll
        for (int vg = 0; vg < 2; ++vg) rm.put(l31, 2 * vg + hf, pack8(acc.more, vg));
        const int mcol = 64 * wn + 32 * wm + 8 * rm.get_piece();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = BMAX + rm.get_row(j);
            const u32x4_t v = rm.get(j);
            if (row < rows && mcol < cols) store(row, mcol, v);
        }
    }
}

// v_exp_f32 and v_rcp_f32 (1 ulp each): far inside the bf16 rounding of the results
__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

}  // namespace uniep
