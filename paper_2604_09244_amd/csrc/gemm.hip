// bf16 GEMM on the gfx950 matrix cores:  C[M,N] = A[M,K] * W[N,K]^T, fp32
// accumulation.  Both operands are contiguous along K, so HBM reads, LDS tiles
// and MFMA fragments all move 16-byte chunks of 8 K-elements.
//
// Data path.  K-slabs of the A and W tiles go from global memory straight into
// LDS (global_load_lds, 16 bytes per lane, no register staging) into a ring of
// NS stages, so the next slab(s) are in flight while the matrix cores work on
// the current one.  The LDS image is XOR-swizzled; because a direct load
// always lands its 64 lanes on 1 KiB of consecutive LDS, the swizzle is applied
// on the global side: lane l fetches the chunk that belongs at its slot.
// MFMA fragments are double-buffered in registers: the ds_reads of k-step s+1
// (and, across the stage barrier, of the next slab) are dealt out between the
// MFMAs of step s, and so are the next slabs' direct loads.
//
// Work split.  A workgroup owns a BM x BN tile; its waves own (BM/WM) x (BN/WN)
// sub-tiles in 16x16x32 products (the wave rows of the recordable 288x192 shape overlap by 32 rows).
// Tiles that fill whole rounds of the chip are computed start to finish by one workgroup.  The tiles of the last,
// partial round are cut along K into equal ranges of k-iterations handed out
// contiguously to the otherwise idle CUs; the pieces of a tile meet in an fp32
// partial buffer and whichever piece arrives last (integer arrival counter)
// adds them up in fixed piece order and runs the epilogue, so results do not
// depend on timing.
// The four-wave 256x256 shape runs as a persistent kernel of its own (persistent_body), its cut last
// round in quarters on another shape where that is predicted faster.  Row counts in between take whole tiles of
// a height and width that fit them (fitted_tile_kernel).
//
// Epilogues: the q/k/v projection (q and k columns rotated by the row's position
// on the fp32 accumulators and stored as bf16, v columns stored transposed for
// the attention kernel); residual add (bf16 residual in, fp32 out -- or
// fp32 residual in, bf16 out: the residual stream between the two halves of a
// layer stays in fp32, so it is rounded to bf16 once per layer); SiLU(gate)*up,
// where gate and up columns alternate in blocks of 32 (one 64-column group holds a
// gate block and its up block).  Every epilogue lays the accumulator tile down in
// LDS as fp32 rows first, so residual reads and result stores are 16 bytes per
// lane on whole cache lines; K-split tiles take the same route after the pieces
// are summed.
#include "common.h"
#include "mfma.h"

namespace mvla {

// Direct global -> LDS copy of 16 bytes per lane, from a wave-uniform base and a 32-bit per-lane byte
// offset: the wave's 64 lanes land on 1 KiB starting at the wave-uniform LDS byte address lds_base + OFF.
// Not tracked by the compiler's wait-count insertion; every consumer is ordered behind wait_vm<>() and a
// workgroup barrier.
template <int OFF>
__device__ __forceinline__ void dma16_at(const void* base, uint32_t off, uint32_t lds_base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base),
                 "v"(off), "s"(base), "i"(OFF)
                 : "memory", "m0", "scc");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Partial sums cross between CUs (and XCDs, each with its own L2) through agent-coherent
// accesses, which go to the shared level of the memory system one access at a time; nothing
// here needs a whole-cache write-back or invalidate.
typedef float f32q_t __attribute__((ext_vector_type(4)));
// The wait states after the store keep the next VALU write away from the data registers
// (a store of more than 64 bits reads them late; the compiler cannot see that inside asm).
// (wave-uniform base and a 32-bit per-lane byte offset: with whole addresses per access the compiler keeps
// a table of 64-bit constants in scalar registers, more than there are)
__device__ __forceinline__ void st16_coherent(float* base, uint32_t off, f32q_t v) {
    asm volatile("global_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 2" ::"v"(off), "v"(v), "s"(base) : "memory");
}
// Issues the load; the value may be used only after settle() has been applied to it.
__device__ __forceinline__ f32q_t ld16_coherent(const float* base, uint32_t off) {
    f32q_t v;
    asm volatile("global_load_dwordx4 %0, %1, %2 sc1" : "=v"(v) : "v"(off), "s"(base) : "memory");
    return v;
}
// Output (and residual) of the epilogues as a bounds-checked buffer: a lane whose byte offset lies
// at or beyond the record count is dropped (stores) or reads zeros (loads) by the hardware.  A
// lane that has nothing to write gets the offset OOB_OFFSET instead of a branch around its store:
// the stream of memory instructions is then the same for every lane, and the compiler's count of
// outstanding ones -- which places the waits for the residual reads -- is exact (a store that may
// or may not have been issued makes it wait for the stores before as well: loads and stores
// return in issue order).
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
constexpr int OOB_OFFSET = 0x7FFF0000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes > 0 ? bytes : 0, 0x00020000);
}
__device__ __forceinline__ void settle(f32q_t& a, f32q_t& b, f32q_t& c, f32q_t& d) {
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d)::"memory");
}

constexpr int GROUP_M = 8;
constexpr int SK_MIN_ITERS = 8;    // smallest K-range worth its own workgroup (in slabs)
constexpr int SK_MAX_PIECES = 64;  // most pieces one tile is ever cut into

// An LDS row holds one K-slab of a tile row: CPR = BK/8 chunks of 16 bytes.  Chunk c of row r
// lives at slot r*CPR + (c ^ swz(r)) with swz(r) = (r >> 1) & 7 for 128-byte rows and
// (r >> 2) & 3 for 64-byte rows: both conflict-free for the 32-row x 16-byte fragment reads
// (measured: SQ_LDS_BANK_CONFLICT = 0).
template <int CPR>
__device__ __forceinline__ int swz(int row) {
    return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3;
}

struct GemmPlan {
    int tiles_m, tiles_n, k_tiles;
    int dp_tiles;     // tiles computed whole by one workgroup
    int dp_grid;      // dp_tiles rounded up to a multiple of 8 (workgroup ids 0 .. dp_grid-1)
    int sk_tiles;     // tiles of the last partial round, split along K
    int sk_blocks;    // workgroups sharing the sk_tiles * k_tiles iterations
    int quarter_of;   // >= 0: the dp_tiles are quarters (128x128) of the 256x256 tiles from this one on
    float norm_eps;   // of rows that are normalised on their way in (see norms_rows)
};

// A second q/k/v-type projection in the same launch, with the same N, K and row pitches: the workgroups from
// first_block on are its (0: there is none).  Two projections that would each leave compute units idle
// run side by side.
struct PairedGemm {
    const bf16_t *A, *W;
    void* C;
    const int32_t* pos;
    int M, tiles_m, first_block;
};

// Workgroup ids are dealt round-robin to the 8 XCDs (each has its own L2).  Give every XCD a
// contiguous range of the sequence, and run the sequence through groups of GROUP_M row-tiles
// column by column, so the tiles an XCD has in flight share activation rows and weight panels.
__device__ __forceinline__ int xcd_chunked(int id, int total) {
    return (id & 7) * ((total + 7) >> 3) + (id >> 3);  // may be >= total for padded ids
}
__device__ __forceinline__ void tile_of(int lin, int tiles_m, int tiles_n, int* tm, int* tn) {
    if (tiles_m <= GROUP_M) {   // (one group: a division less before a short projection's first load)
        *tn = lin / tiles_m;
        *tm = lin - *tn * tiles_m;
        return;
    }
    const int group_tiles = GROUP_M * tiles_n;
    const int g = lin / group_tiles, r = lin % group_tiles;
    const int gm = min(GROUP_M, tiles_m - g * GROUP_M);
    *tm = g * GROUP_M + r % gm;
    *tn = r / gm;
}

// Gate/up projections of short rows on 64x64 tiles take the fp32 residual stream and normalise it themselves: a
// workgroup's rows fit the A places of its LDS stages whole, and the launch of the norm, its output's way through
// memory and the wait in between are gone.  Told by a negative row pitch; A is the residual, Rv the gain.
// Bound by the chain of one row read, its sum and one slab after the other.  us, norm and projection / this, back to
// back in a graph: D = 256, F = 1024, 80 rows 6.1 / 5.2, 237 6.2 / 5.3, 512 6.4 / 5.6 (where the choice by size leaves the tile);
// D = 64, F = 256, 2048 rows 6.2 / 4.1; D = 384, F = 1024, 80 rows 6.3 / 6.1, F = 1536, 300 rows 6.6 / 6.7.  The small model's
// pruned prefill 44.7 -> 42.4.  Longer rows do not fit beside the weights, and larger tiles have their rows from a norm
// of their own.
constexpr int NORM_MAX_K = 384;   // six stages of 64
constexpr bool norms_rows(int BM, int BN, int NS, int EPI) {
    return EPI == EPI_SILU_MUL && BM == 64 && BN == 64 && NS * 64 >= NORM_MAX_K;
}

// The three families of tile kernels: shapes with the K-split path (recordable choices), small whole tiles, and
// whole tiles whose height is fitted to the row count.
enum KernelKind { SPLITTING, SMALL, FITTED };
constexpr int rows_unit(KernelKind kind) { return kind == FITTED ? 16 : 32; }

// Epilogue staging: the output tile goes through LDS as fp32 rows of BN + 4 floats (the 4 keep
// 16-byte accesses of 32 consecutive rows on different banks), RP rows per pass.  The whole tile
// in one pass if the LDS a workgroup may use holds it, else one wave row per pass.
template <int BM, int BN, int WM, int NS, int RU = 32 /* rows a wave's blocks come in */>
struct EpiGeom {
    static constexpr int LDT = BN + 4;
    static constexpr int CAP = (NS == 2 && BM == 128 && BN == 128) ? 76 * 1024 : 156 * 1024;
    static constexpr int TM = (BM / RU + WM - 1) / WM * RU;   // rows of a wave row
    static constexpr int PASSES = BM * LDT * 4 <= CAP ? 1 : WM;
    static constexpr int RP = PASSES == 1 ? BM : TM;
    // (where the accumulators are in the second register file, a spare strip of 16 rows: see the lay-down)
    static constexpr int BYTES = (RP + (TM / 16 * (BN / 32) >= 54 ? 16 : 0)) * LDT * 4;
    static_assert(BYTES <= CAP, "epilogue tile does not fit the LDS");
    static_assert(TM * WM == BM || PASSES == WM, "overlapping wave rows go one per pass");
};

// ---------------------------------------------------------------------------------------------
// The four-wave 256x256 shape (128x128 per wave, its 256 accumulator registers in the second register
// file) as a persistent kernel: one workgroup per CU walks through its tiles, and the stream of slab
// loads runs on across tile borders -- the last two slabs of a tile are followed by the first two of
// the next one, into the same two stages, so the epilogue starts with the next tile's operands in
// flight and no tile but the first waits for its first slab.  The epilogue needs no workgroup
// barrier and none of the stages: every wave turns its accumulator blocks through 4.5 KiB of LDS of
// its own (LDS accesses of a wave are in order) into whole 128-byte lines of the output.
//
// Bound by the matrix core, and that by the part's power: the main loop takes about 2280 clocks a slab of
// which 2048 are products, at 1.6 GHz instead of 2.4; the epilogue (9 k clocks of a gate/up tile's 155 k,
// 11 k q/k/v, 20 k with a residual) is what nothing overlaps.  Hence the 16x16x32 products (see mfma16).
// Against one workgroup per tile with 32x32x16 products, M = 21504: gate/up 2832 -> 2546 us
// (1.50 PFLOP/s), q/k/v 1701 -> 1543, down 1375 -> 1292, output 555 -> 525; of that the persistent form
// alone, with 32x32x16 products, gave 3 %, 6 %, 1 % and 4 %.
//
// Main loop, per 64-deep slab: the fragments of k-steps 2 and 3 are read during k-step 0, those of the
// next slab's k-steps 0 and 1 during k-step 3, one LDS read after each MFMA, so the stage is free after
// k-step 0; the direct loads of the slab after next go out a third each over k-steps 1 to 3 (the load
// unit takes one 64-lane load per 16 clocks: 64 loads are two k-steps of it).
// ---------------------------------------------------------------------------------------------
constexpr int PT_BK = 64, PT_STAGE = 512 * 8, PT_LD = 8, PT_P = 2 * PT_LD;   // 16-byte slots of a stage; loads per thread
constexpr int PT_TLD = 36;                                   // floats per row of a wave's turning area
constexpr int PT_TURN = 32 * PT_TLD;                         // floats of it
constexpr int PT_LDS_BYTES = 2 * PT_STAGE * 16 + 4 * PT_TURN * 4;

// Workgroup barrier for LDS traffic: this wave's LDS reads have returned; its global stores (of the
// epilogue before) may be on their way, which __syncthreads() would wait for.
__device__ __forceinline__ void lds_only_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int EPI>
__device__ __forceinline__ void persistent_body(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W,
                                                int M, int N, int K, void* __restrict__ Cv, int ldc,
                                                const void* __restrict__ Rv, int ldr, const GemmPlan& plan,
                                                const RopeEpilogue& rope) {
    extern __shared__ uint4 lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    const int k_tiles = plan.k_tiles;
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
    float* turn = reinterpret_cast<float*>(lds + 2 * PT_STAGE) + wave * PT_TURN;

    // tile r of this workgroup: launch id blockIdx.x + r * gridDim.x, as if every tile were a workgroup
    // (the ids of a launch of whole tiles; see xcd_chunked); -1 when there is none
    auto next_tile = [&](int& id) __attribute__((always_inline)) {
        while (id < plan.dp_grid) {
            const int lin = xcd_chunked(id, plan.dp_tiles);
            id += (int)gridDim.x;
            if (lin < plan.dp_tiles) return lin;
        }
        return -1;
    };

    // ---- stream of slab loads: where the next slab comes from ------------------------------------
    // (v tiles of the q/k/v projection are computed transposed -- weight rows take the place of the
    // activation rows and the other way round -- so that a lane's registers run along the tokens)
    const char *dma_a, *dma_b;           // wave-uniform: first row of the tile, current slab
    uint32_t off_a[PT_LD], off_b[PT_LD]; // per lane, from there
    int dma_left;                        // slabs of the stream's tile not issued yet
    auto aim = [&](int lin) __attribute__((always_inline)) {
        int tm, tn;
        tile_of(lin, plan.tiles_m, plan.tiles_n, &tm, &tn);
        const bool turned = EPI == EPI_QKV_ROPE && tn * 256 >= 2 * rope.D;
        const bf16_t* act = A + (size_t)tm * 256 * lda;
        const bf16_t* wgt = W + (size_t)tn * 256 * K;
        dma_a = reinterpret_cast<const char*>(turned ? wgt : act);
        dma_b = reinterpret_cast<const char*>(turned ? act : wgt);
        const int lim_m = M - 1 - tm * 256, lim_n = N - 1 - tn * 256;
        const int lim_a = turned ? lim_n : lim_m, lim_b = turned ? lim_m : lim_n;
        const int ld_a = turned ? K : lda, ld_b = turned ? lda : K;
#pragma unroll
        for (int i = 0; i < PT_LD; ++i) {
            const int sl = i * 256 + tid, row = sl >> 3, ch = (sl & 7) ^ swz<8>(row);
            off_a[i] = ((uint32_t)min(row, lim_a) * (uint32_t)ld_a + (uint32_t)ch * 8u) * 2u;
            off_b[i] = ((uint32_t)min(row, lim_b) * (uint32_t)ld_b + (uint32_t)ch * 8u) * 2u;
        }
        dma_left = k_tiles;
    };
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)wave * 1024u);
    // load l of the stream's current slab into stage STG
    // (the index is a constant once the loops are unrolled; "n"-type operands need it before that)
    auto load_one = [&](int l, uint32_t to) __attribute__((always_inline)) {
        switch (l) {
#define PT_CASE(L) \
    case L: dma16_at<L * 4096>(L < PT_LD ? dma_a : dma_b, L < PT_LD ? off_a[L % PT_LD] : off_b[L % PT_LD], to); break;
            PT_CASE(0) PT_CASE(1) PT_CASE(2) PT_CASE(3) PT_CASE(4) PT_CASE(5) PT_CASE(6) PT_CASE(7)
            PT_CASE(8) PT_CASE(9) PT_CASE(10) PT_CASE(11) PT_CASE(12) PT_CASE(13) PT_CASE(14) PT_CASE(15)
#undef PT_CASE
        }
    };
#define PT_LOAD(L, STG) load_one(L, lds_wave + (uint32_t)(STG) * (PT_STAGE * 16u));
    int ahead_id = blockIdx.x;           // launch id the stream looks at next
    int tile = next_tile(ahead_id);      // tile being computed
    if (tile < 0) return;
    int ahead = tile;                    // tile the stream loads (-1: none left, the last one is loaded again)
    aim(tile);
    // after a slab: on to the next one, or to the next tile's first
    auto advance = [&]() __attribute__((always_inline)) {
        dma_a += PT_BK * 2;
        dma_b += PT_BK * 2;
        if (--dma_left == 0) {
            if (ahead >= 0) ahead = next_tile(ahead_id);
            if (ahead >= 0) {
                aim(ahead);
            } else {                     // (keeps the count of loads in flight; never read)
                dma_a -= (size_t)PT_BK * 2;
                dma_b -= (size_t)PT_BK * 2;
                dma_left = 1;
            }
        }
    };

    // fragments: lane -> row lane % 16 of a 16-row block, chunk lane / 16 of the k-step's four
    const int fr16 = lane & 15, fq = lane >> 4;
    const int a_row = (wm * 128 + fr16) * 8, b_row = 2048 + (wn * 128 + fr16) * 8;
    const int sw = swz<8>(fr16);         // (rows of a lane differ by multiples of 16: one pattern)
    // fragment read R of the sixteen of k-step KS, in the order the products need them
#define PT_READ(DST_A, DST_B, STG, KS, R)                                                        \
    {                                                                                            \
        const uint4* st_ = lds + (STG) * PT_STAGE + (((KS) * 4 + fq) ^ sw);                      \
        if ((R) == 0 || (R) > 8) DST_A[(R) > 8 ? (R) - 8 : 0] = st_[a_row + ((R) > 8 ? (R) - 8 : 0) * 128]; \
        else DST_B[((R) - 1) & 7] = st_[b_row + (((R) - 1) & 7) * 128];                          \
    }
    // 32 of the 64 MFMAs of a k-step: block rows I0 .. I0+3.  After every other MFMA a fragment read of
    // k-step RKS of stage RSTG (when READS), and the loads [L0, L1) of the stream's slab into stage
    // LSTG spread out
#define PT_HALF(AF, BF, I0, READS, DA, DB, RSTG, RKS, LSTG, L0, L1)                              \
    {                                                                                            \
        constexpr int EVERY_ = (L1) > (L0) ? 32 / ((L1) - (L0)) : 99;                            \
        int l_ = (L0);                                                                           \
        _Pragma("unroll") for (int n_ = 0; n_ < 32; ++n_) {                                      \
            const int i_ = (I0) + (n_ >> 3), j_ = n_ & 7;                                        \
            acc[i_][j_] = mfma16(BF[j_], AF[i_], acc[i_][j_]);                                   \
            if ((READS) && (n_ & 1) == 0) PT_READ(DA, DB, RSTG, RKS, (n_ >> 1))                  \
            if (n_ % EVERY_ == EVERY_ - 1 && l_ < (L1)) {                                        \
                PT_LOAD(l_, LSTG)                                                                \
                ++l_;                                                                            \
            }                                                                                    \
            __builtin_amdgcn_sched_barrier(0);                                                   \
        }                                                                                        \
    }

    uint4 af0[8], bf0[8], af1[8], bf1[8];
    f32x4_t acc[8][8];                   // block (i, j): 16 rows x 16 columns
#pragma unroll
    for (int l = 0; l < PT_P; ++l) PT_LOAD(l, 0)
    advance();
#pragma unroll
    for (int l = 0; l < PT_P; ++l) PT_LOAD(l, 1)
    advance();
    wait_vm<PT_P>();
    lds_only_barrier();
    int stage = 0;
    int tile_id = blockIdx.x;            // launch ids of the tiles computed
    (void)next_tile(tile_id);
    constexpr int L1_ = PT_P / 3, L2_ = 2 * PT_P / 3;

    while (tile >= 0) {
        // (the first fragments are read again here rather than carried across the epilogue before,
        // which needs their registers)
#pragma unroll
        for (int r = 0; r < 16; ++r) PT_READ(af0, bf0, stage, 0, r)
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int kt = 0; kt < k_tiles; ++kt) {
            // first k-step, reading the fragments of the second: after it this slab is in registers
            PT_HALF(af0, bf0, 0, true, af1, bf1, stage, 1, 0, 0, 0)
            lds_only_barrier();   // ... for every wave: the stage is free for the slab after next
            PT_HALF(af0, bf0, 4, false, af1, bf1, 0, 0, stage, 0, L1_)
            PT_HALF(af1, bf1, 0, false, af1, bf1, 0, 0, stage, L1_, L2_)
            // the next slab has landed for every wave (two thirds of the one after may be in flight)
            wait_vm<L2_>();
            lds_only_barrier();
            PT_HALF(af1, bf1, 4, true, af0, bf0, stage ^ 1, 0, stage, L2_, PT_P)
            advance();
            stage ^= 1;
        }

        // ---- epilogue, wave by wave: rows r0w .. r0w+127, columns c0w .. c0w+127 of the tile ----
        int tile_m, tile_n;
        tile_of(tile, plan.tiles_m, plan.tiles_n, &tile_m, &tile_n);
        const int m0 = tile_m * 256, n0 = tile_n * 256;
        tile = next_tile(tile_id);
        int el = lane, ew = wave;        // (the epilogue's indices are computed here, not held across the loop)
        asm volatile("" : "+v"(el), "+s"(ew));
        const int efr = el & 15, efq = (el >> 4) * 4;    // a lane's row and first column in a 16x16 block
        const int trow = el >> 3, tcol = (el & 7) * 4;   // turned: row (of 8 a read) and first of 4 floats
        const int r0w = (ew >> 1) * 128, c0w = (ew & 1) * 128;
        // 32x32 accumulators (blocks 2i, 2i+1 by 2j, 2j+1) into the turning area as fp32 rows
        auto lay = [&](int i, int j) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 4; ++h)
                *reinterpret_cast<f32x4_t*>(turn + ((h >> 1) * 16 + efr) * PT_TLD + (h & 1) * 16 + efq) =
                    acc[2 * i + (h >> 1)][2 * j + (h & 1)];
            asm volatile("" ::: "memory");   // (the reads stay behind the writes; the LDS keeps a wave's order)
        };
        auto turned4 = [&](int t) __attribute__((always_inline)) {
            return *reinterpret_cast<const f32x4_t*>(turn + (t * 8 + trow) * PT_TLD + tcol);
        };
        // a quad of packed bf16 pairs into the area as rows of 64 bf16 (same row pitch)
        auto lay_bf16 = [&](int row, int col, uint32_t x, uint32_t y) __attribute__((always_inline)) {
            *reinterpret_cast<u32x2_t*>(reinterpret_cast<bf16_t*>(turn) + row * (PT_TLD * 2) + col) = u32x2_t{x, y};
            asm volatile("" ::: "memory");
        };
        auto turned8 = [&](int t) __attribute__((always_inline)) {
            return *reinterpret_cast<const u32x4_t*>(turn + (t * 8 + trow) * PT_TLD + tcol);
        };
        // (the compiler fetched all 256 accumulators from the second register file at once otherwise)
        auto pin_rows = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(acc[2 * i][j]), "+a"(acc[2 * i + 1][j]));
        };
        const int rows_here = min(256, M - m0);
        if constexpr (EPI == EPI_SILU_MUL) {
            const int out_n0 = n0 / 2, cols_here = min(128, N / 2 - out_n0);
            const __amdgpu_buffer_rsrc_t c_buf = buffer_of(static_cast<bf16_t*>(Cv) + (size_t)m0 * ldc + out_n0,
                                                           ((rows_here - 1) * ldc + cols_here) * 2);
            const int col = c0w / 2 + tcol * 2;          // 8 output columns of a lane
            int off[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                off[t] = col < cols_here ? ((r0w + t * 8 + trow) * ldc + col) * 2 : OOB_OFFSET;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pin_rows(i);
                // gate and up columns alternate in blocks of 32: block columns 4p, 4p+1 and 4p+2, 4p+3
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        const f32x4_t g = acc[2 * i + (h >> 1)][4 * p + (h & 1)];
                        const f32x4_t u = acc[2 * i + (h >> 1)][4 * p + 2 + (h & 1)];
                        float x[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            x[e] = g[e] * u[e] * __builtin_amdgcn_rcpf(1.f + __expf(-g[e]));
                        lay_bf16((h >> 1) * 16 + efr, p * 32 + (h & 1) * 16 + efq, pack_bf16x2(x[0], x[1]),
                                 pack_bf16x2(x[2], x[3]));
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    __builtin_amdgcn_raw_buffer_store_b128(turned8(t), c_buf,
                                                           off[t] == OOB_OFFSET ? OOB_OFFSET : off[t] + i * 64 * ldc, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if constexpr (EPI == EPI_RES_BF16_TO_F32 || EPI == EPI_RES_F32_TO_BF16) {
            constexpr int ES = EPI == EPI_RES_BF16_TO_F32 ? 4 : 2, RS = 6 - ES;   // bytes per output / residual value
            const int cols_here = min(256, N - n0);
            const __amdgpu_buffer_rsrc_t c_buf = buffer_of(static_cast<char*>(Cv) + ((size_t)m0 * ldc + n0) * ES,
                                                           ((rows_here - 1) * ldc + cols_here) * ES);
            const __amdgpu_buffer_rsrc_t r_buf = buffer_of(static_cast<const char*>(Rv) + ((size_t)m0 * ldr + n0) * RS,
                                                           ((rows_here - 1) * ldr + cols_here) * RS);
            const int row = r0w + trow, col = c0w + tcol;
            // residual of the 32 rows i: 16 loads, one set of 32 rows ahead of its use
            constexpr int RW = RS == 2 ? 2 : 4;
            uint32_t res[2][16][RW];
            auto request = [&](int i) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int o = ((row + i * 32 + t * 8) * ldr + col + j * 32) * RS;
                        if constexpr (RW == 2) {
                            const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r_buf, o, 0, 0);
                            res[i & 1][j * 4 + t][0] = v.x;
                            res[i & 1][j * 4 + t][1] = v.y;
                        } else {
                            const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r_buf, o, 0, 0);
                            res[i & 1][j * 4 + t][0] = v.x;
                            res[i & 1][j * 4 + t][1] = v.y;
                            res[i & 1][j * 4 + t][RW - 2] = v.z;
                            res[i & 1][j * 4 + t][RW - 1] = v.w;
                        }
                    }
            };
            request(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i < 3) request(i + 1);
                __builtin_amdgcn_sched_barrier(0);
                pin_rows(i);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lay(i, j);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const f32x4_t a = turned4(t);
                        const uint32_t* r = res[i & 1][j * 4 + t];
                        const int o = col + j * 32 < cols_here
                                          ? ((row + i * 32 + t * 8) * ldc + col + j * 32) * ES : OOB_OFFSET;
                        if constexpr (RW == 2) {
                            const u32x4_t v = {__float_as_uint(a.x + __uint_as_float(r[0] << 16)),
                                               __float_as_uint(a.y + __uint_as_float(r[0] & 0xFFFF0000u)),
                                               __float_as_uint(a.z + __uint_as_float(r[1] << 16)),
                                               __float_as_uint(a.w + __uint_as_float(r[1] & 0xFFFF0000u))};
                            __builtin_amdgcn_raw_buffer_store_b128(v, c_buf, o, 0, 0);
                        } else {
                            const u32x2_t v = {pack_bf16x2(a.x + __uint_as_float(r[0]), a.y + __uint_as_float(r[1])),
                                               pack_bf16x2(a.z + __uint_as_float(r[RW - 2]), a.w + __uint_as_float(r[RW - 1]))};
                            __builtin_amdgcn_raw_buffer_store_b64(v, c_buf, o, 0, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else if (n0 < 2 * rope.D) {
            // q and k columns: a head's first half sits in one block (dh = 64) or two (dh = 128), its
            // second half in the block(s) after; both are turned together, rotated in fp32 and packed
            const int cols_here = min(256, N - n0), half = rope.dh >> 1;
            const __amdgpu_buffer_rsrc_t c_buf = buffer_of(static_cast<bf16_t*>(Cv) + (size_t)m0 * ldc + n0,
                                                           ((rows_here - 1) * ldc + cols_here) * 2);
            const int row = r0w + trow;
            auto rotate = [&](int j1, int j2, const float4 (&c)[4], const float4 (&s)[4], int i,
                              int colb) __attribute__((always_inline)) {
                f32x4_t a[4];
                lay(i, j1);
#pragma unroll
                for (int t = 0; t < 4; ++t) a[t] = turned4(t);
                lay(i, j2);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const f32x4_t b = turned4(t);
                    const int col = colb + tcol;
                    const int o = col < cols_here ? ((row + i * 32 + t * 8) * ldc + col) * 2 : OOB_OFFSET;
                    const u32x2_t x = {pack_bf16x2(a[t].x * c[t].x - b.x * s[t].x, a[t].y * c[t].y - b.y * s[t].y),
                                       pack_bf16x2(a[t].z * c[t].z - b.z * s[t].z, a[t].w * c[t].w - b.w * s[t].w)};
                    const u32x2_t y = {pack_bf16x2(b.x * c[t].x + a[t].x * s[t].x, b.y * c[t].y + a[t].y * s[t].y),
                                       pack_bf16x2(b.z * c[t].z + a[t].z * s[t].z, b.w * c[t].w + a[t].w * s[t].w)};
                    __builtin_amdgcn_raw_buffer_store_b64(x, c_buf, o, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(y, c_buf, o + half * 2, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // (the position ids of 32 rows are asked for one step, their table rows another step ahead)
            auto place = [&](int i, int (&pos)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < 4; ++t) pos[t] = rope.pos[min(m0 + row + i * 32 + t * 8, M - 1)];
            };
            auto table = [&](const int (&pos)[4], int c0, float4 (&c)[4], float4 (&s)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const size_t at = (size_t)min(max(pos[t], 0), rope.rope_len - 1) * half + c0 + tcol;
                    c[t] = *reinterpret_cast<const float4*>(rope.rc + at);
                    s[t] = *reinterpret_cast<const float4*>(rope.rs + at);
                }
            };
            int pos[2][4];
            float4 c[2][4], s[2][4];
            place(0, pos[0]);
            place(1, pos[1]);
            table(pos[0], 0, c[0], s[0]);
            if (rope.dh == 128) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {            // (rows k/2, half a half head k%2)
                    const int i = k >> 1, n = (k + 1) & 1;
                    if (k < 7) table(pos[((k + 1) >> 1) & 1], n * 32, c[n], s[n]);
                    if (n == 0 && i < 2) place(i + 2, pos[i & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    pin_rows(i);
                    rotate(k & 1, (k & 1) + 2, c[k & 1], s[k & 1], i, c0w + (k & 1) * 32);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i < 3) table(pos[(i + 1) & 1], 0, c[(i + 1) & 1], s[(i + 1) & 1]);
                    if (i < 2) place(i + 2, pos[i & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    pin_rows(i);
                    rotate(0, 1, c[i & 1], s[i & 1], i, c0w);
                    rotate(2, 3, c[i & 1], s[i & 1], i, c0w + 64);
                }
            }
        } else {
            // v columns: rows of the turned tile are columns of V (n0 ..), columns are tokens (m0 ..);
            // vt [B, H, dh, S_pad] is [B*D, S_pad] by (sample, V column), addressed from the row of the
            // tile's first sample and V column (offsets below 2^31: see launch_gemm)
            const int S = rope.S, S_pad = rope.S_pad, D = rope.D, v0 = n0 - 2 * D, b0 = m0 / S;
            const int v_here = min(256, N - n0);
            const __amdgpu_buffer_rsrc_t v_buf = buffer_of(rope.vt + ((size_t)b0 * D + v0) * S_pad, OOB_OFFSET - 65536);
            auto lay_tokens = [&](int i, int jp) __attribute__((always_inline)) {   // 32 V columns x 64 tokens
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4_t a = acc[2 * i + h][jp * 4 + q];
                        lay_bf16(h * 16 + efr, q * 16 + efq, pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
                    }
            };
            // byte offset of a token's entry in the first V column, or out of range
            auto token_at = [&](int tok) __attribute__((always_inline)) {
                const int bs = tok / S;
                return tok < M ? ((bs - b0) * D * S_pad + tok - bs * S) * 2 : OOB_OFFSET;
            };
            if ((S & 7) == 0) {          // every 8 tokens from a tile's start are of one sample
                const int off[2] = {token_at(m0 + c0w + (el & 7) * 8), token_at(m0 + c0w + 64 + (el & 7) * 8)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pin_rows(i);
#pragma unroll
                    for (int jp = 0; jp < 2; ++jp) {
                        lay_tokens(i, jp);
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int r = r0w + i * 32 + t * 8 + trow;
                            __builtin_amdgcn_raw_buffer_store_b128(
                                turned8(t), v_buf, off[jp] != OOB_OFFSET && r < v_here ? off[jp] + r * S_pad * 2 : OOB_OFFSET,
                                0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {                     // one token a lane: 64 consecutive ones of a V column per store
                const int off[2] = {token_at(m0 + c0w + el), token_at(m0 + c0w + 64 + el)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pin_rows(i);
#pragma unroll
                    for (int jp = 0; jp < 2; ++jp) {
                        lay_tokens(i, jp);
#pragma unroll 8
                        for (int r = 0; r < 32; ++r) {
                            const bf16_t v = reinterpret_cast<const bf16_t*>(turn)[r * (PT_TLD * 2) + el];
                            const int vr = r0w + i * 32 + r;
                            __builtin_amdgcn_raw_buffer_store_b16(
                                v, v_buf, off[jp] != OOB_OFFSET && vr < v_here ? off[jp] + vr * S_pad * 2 : OOB_OFFSET, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            // padding behind every sample whose last token is in this tile
            const int z = S + el;
            for (int b = b0; (b + 1) * S - 1 < m0 + rows_here; ++b)
                for (int r = ew; r < v_here; r += 4)
                    if (z < S_pad) rope.vt[((size_t)b * D + v0 + r) * S_pad + z] = 0;
        }
    }
    wait_vm<0>();   // (the last loads into the stages have landed before the workgroup's LDS is given back)
#undef PT_LOAD
#undef PT_READ
#undef PT_HALF
}

template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI, KernelKind KIND>
__device__ __forceinline__ void tile_body(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int M, int N, int K,
    void* __restrict__ Cv, int ldc, const void* __restrict__ Rv, int ldr, GemmPlan plan,
    float* __restrict__ partial, uint32_t* __restrict__ counters, RopeEpilogue rope, const PairedGemm& pair) {
    int bid = blockIdx.x;
    if (EPI == EPI_QKV_ROPE && pair.first_block > 0 && bid >= pair.first_block) {
        bid -= pair.first_block;
        A = pair.A;
        W = pair.W;
        Cv = pair.C;
        M = pair.M;
        rope.pos = pair.pos;
        plan.tiles_m = pair.tiles_m;
        plan.dp_tiles = pair.tiles_m * plan.tiles_n;
        plan.dp_grid = (plan.dp_tiles + 7) / 8 * 8;
    }
    constexpr int RU = rows_unit(KIND);
    constexpr int NT = WM * WN * 64;
    constexpr int CPR = BK / 8;             // 16-byte chunks per LDS row
    // A wave owns GM x GN blocks of 16x16.  Where its rows come in blocks of 32 and the tile's do not divide among the WM
    // wave rows (288 rows on two wave rows), every wave row still takes the larger share
    // and the last one starts early: the rows both cover are computed twice
    // (identical values) so that the main loop stays free of branches.
    constexpr int TM = (BM / RU + WM - 1) / WM * RU, TN = BN / WN, GM = TM / 16, GN = TN / 16;
    static_assert(BM % RU == 0 && BN % (16 * WN) == 0 && TM <= BM, "");
    constexpr int STAGE = (BM + BN) * CPR;  // 16-byte slots per stage
    constexpr int A_SLOTS = BM * CPR, B_SLOTS = BN * CPR;   // 16-byte slots of the A and W tiles
    constexpr int A_LD = A_SLOTS / NT, B_LD = B_SLOTS / NT;
    constexpr int P = A_LD + B_LD;          // direct loads per thread per slab
    static_assert(A_SLOTS % NT == 0 && B_SLOTS % NT == 0, "tile/thread mismatch");
    static_assert(BK == 64 && CPR == 8 && NS >= 2, "two k-steps of 32 a slab");

    extern __shared__ uint4 lds[];
    __shared__ int sh_last;
    __shared__ int sh_slot[SK_MAX_PIECES];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int wrow0 = min(wm * TM, BM - TM);   // first tile row of this wave's blocks
    const int k_tiles = plan.k_tiles;

    // ---- which part of which tile is ours --------------------------------------------------
    int n_seg_work;   // 1 for a whole tile, up to 2 for a K-range that straddles two tiles
    int it_begin = 0, it_end = 0, sk_id = 0;
    const bool is_dp = KIND != SPLITTING || bid < plan.dp_grid;
    if (is_dp) {
        n_seg_work = xcd_chunked(bid, plan.dp_tiles) < plan.dp_tiles ? 1 : 0;
    } else {
        // K-split workgroups in XCD-contiguous order too: the pieces of a tile, and the tiles that
        // share a weight panel, then run on one XCD at the same time and share its L2
        const int id = bid - plan.dp_grid, x = id & 7;   // dp_grid is a multiple of 8
        sk_id = x * (plan.sk_blocks >> 3) + min(x, plan.sk_blocks & 7) + (id >> 3);
        const long total = (long)plan.sk_tiles * k_tiles;
        it_begin = (int)(total * sk_id / plan.sk_blocks);
        it_end = (int)(total * (sk_id + 1) / plan.sk_blocks);
        n_seg_work = (it_begin / k_tiles == (it_end - 1) / k_tiles) ? 1 : 2;
    }

    for (int seg = 0; seg < n_seg_work; ++seg) {
        int stid = tid;   // (per-lane indices of the main loop are made per segment, not held across epilogues)
        asm volatile("" : "+v"(stid));
        const int fr = stid & 15, fq = (stid & 63) >> 4;   // row in a 16-row block; 16-byte chunk of a k-step's four
        int lin, k0, k1, sk_tile = -1, first_blk = 0, last_blk = 0;
        if (is_dp) {
            lin = xcd_chunked(bid, plan.dp_tiles);
            k0 = 0;
            k1 = k_tiles;
        } else {
            const int it0 = seg == 0 ? it_begin : (it_begin / k_tiles + 1) * k_tiles;
            sk_tile = it0 / k_tiles;
            const int it1 = min(it_end, (sk_tile + 1) * k_tiles);
            k0 = it0 - sk_tile * k_tiles;
            k1 = it1 - sk_tile * k_tiles;
            lin = plan.dp_tiles + sk_tile;
            // workgroups whose ranges touch this tile: the one holding its first and its last slab
            const long total = (long)plan.sk_tiles * k_tiles;
            first_blk = (int)((((long)sk_tile * k_tiles + 1) * plan.sk_blocks - 1) / total);
            last_blk = (int)((((long)(sk_tile + 1) * k_tiles) * plan.sk_blocks - 1) / total);
        }
        int tile_m, tile_n;
        int m0, n0;
        if (BM == 128 && BN == 128 && WM * WN == 8 && plan.quarter_of >= 0) {
            tile_of(plan.quarter_of + (lin >> 2), plan.tiles_m, plan.tiles_n, &tile_m, &tile_n);
            m0 = tile_m * 256 + ((lin >> 1) & 1) * 128;
            n0 = tile_n * 256 + (lin & 1) * 128;
            if (m0 >= M || n0 >= N) continue;
        } else {
            tile_of(lin, plan.tiles_m, plan.tiles_n, &tile_m, &tile_n);
            m0 = tile_m * BM;
            n0 = tile_n * BN;
        }

        // ---- direct-load mapping: op i covers slot i*NT + tid of the A (or W) tile ----------
        // (wave-uniform base of the tile's rows, per-lane 32-bit byte offsets from there)
        const char* a_base = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
        const char* b_base = reinterpret_cast<const char*>(W + (size_t)n0 * K);
        uint32_t a_off[A_LD], b_off[B_LD];
        const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds + (uint32_t)wave * 1024u);
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            const int sl = i * NT + stid, row = sl / CPR, ch = (sl % CPR) ^ swz<CPR>(row);
            a_off[i] = ((uint32_t)min(row, M - 1 - m0) * (uint32_t)lda + (uint32_t)ch * 8u) * 2u;
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            const int sl = i * NT + stid, row = sl / CPR, ch = (sl % CPR) ^ swz<CPR>(row);
            b_off[i] = ((uint32_t)min(row, N - 1 - n0) * (uint32_t)K + (uint32_t)ch * 8u) * 2u;
        }
        // load l (of P) of the slab at byte offset koff into the stage at lds_wave + soff
        auto load_one = [&](int l, size_t koff, uint32_t soff) __attribute__((always_inline)) {
            switch (l) {
#define MVLA_CASE(L) \
    case L: \
        dma16_at<L * NT * 16>(L < A_LD ? a_base + koff : b_base + koff, \
                              L < A_LD ? a_off[L < A_LD ? L : 0] : b_off[L >= A_LD && L < P ? L - A_LD : 0], \
                              lds_wave + soff); \
        break;
                MVLA_CASE(0) MVLA_CASE(1) MVLA_CASE(2) MVLA_CASE(3) MVLA_CASE(4) MVLA_CASE(5) MVLA_CASE(6) MVLA_CASE(7)
                MVLA_CASE(8) MVLA_CASE(9) MVLA_CASE(10) MVLA_CASE(11) MVLA_CASE(12) MVLA_CASE(13) MVLA_CASE(14)
                MVLA_CASE(15)
#undef MVLA_CASE
            }
        };
        static_assert(P <= 16, "load_one has sixteen cases");
        const int a_row = (wrow0 + fr) * CPR, b_row = (BM + wn * TN + fr) * CPR;
        const int sw = swz<CPR>(fr);   // (rows of a lane differ by multiples of 16: one pattern)

        f32x4_t acc[GM][GN];
#pragma unroll
        for (int i = 0; i < GM; ++i)
#pragma unroll
            for (int j = 0; j < GN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        // ---- epilogue: its geometry, and what of its operands is asked for ahead of the slabs -------
        using EG = EpiGeom<BM, BN, WM, NS, RU>;
        constexpr int LDT = EG::LDT, PASSES = EG::PASSES, RP = EG::RP;
        constexpr int OUT_COLS = EPI == EPI_SILU_MUL ? BN / 2 : BN;   // output columns per tile
        const int out_n0 = EPI == EPI_SILU_MUL ? n0 / 2 : n0;
        const int out_N = EPI == EPI_SILU_MUL ? N / 2 : N;
        // (whole tiles that leave the LDS in one pass: position ids and the first residual rows arrive with the first slab)
        constexpr bool EARLY = KIND != SPLITTING && PASSES == 1;
        // q/k rotation: an item is 8 columns of a half head and their partners, BN/16 per row; QB items' table rows
        // fly together
        constexpr int PER_ROW = BN / 16, PER_THREAD = (RP * PER_ROW + NT - 1) / NT;
        constexpr int QB_MAX = (GM * GN >= 32 && WM * WN >= 8) ? 2 : 4;
        constexpr int QB = PER_THREAD < QB_MAX ? PER_THREAD : QB_MAX;
        constexpr int NB = (RP * PER_ROW + QB * NT - 1) / (QB * NT);
        constexpr bool PREFETCH = EPI == EPI_QKV_ROPE && QB_MAX == 4;   // (registers to spare)
        int pos_pre[PREFETCH ? NB * QB : 1];
        auto pos_request = [&](int t, int prow0) __attribute__((always_inline)) {
            if (PREFETCH && (EARLY || n0 < 2 * rope.D)) {   // (early: no branch to wait behind; v tiles load them for nothing)
#pragma unroll
                for (int q = 0; q < NB * QB; ++q) {
                    const int row = m0 + prow0 + min((t + q * NT) / PER_ROW, RP - 1);
                    pos_pre[q] = rope.pos[min(row, M - 1)];
                }
            }
        };
        // Residual epilogues: an item is 4 columns of a row (16 bytes of fp32: a wave's load
        // or store covers consecutive whole cache lines; with 8-column items a lane's two
        // 16-byte fp32 accesses lay 32 bytes apart and a store burst of that form takes 1.4-1.8
        // times as long).  Items go in batches of RB whose residual reads are in flight
        // together, the first batch requested before the tile is laid down; reads and stores
        // are unconditional buffer accesses (behind a per-item branch the compiler made each
        // read wait for the one before it -- a memory round trip per item -- and behind
        // conditional stores for the stores before it).
        constexpr bool RES = EPI == EPI_RES_BF16_TO_F32 || EPI == EPI_RES_F32_TO_BF16;
        // (register room: shapes with none to spare request after the lay-down, and fewer at a time)
        constexpr bool TIGHT = !EARLY && ((WM * WN == 8 && BM == 256 && BN == 256) || BM == 288 ||
                                          (WM * WN == 4 && BM == 128));
        constexpr int IPR = OUT_COLS / 4;                                 // items per tile row
        constexpr int RPT = (RP * IPR + NT - 1) / NT;                     // items per thread and pass
        constexpr int RREG = EPI == EPI_RES_BF16_TO_F32 ? 2 : 4;          // registers per item
        constexpr int RES_ES = EPI == EPI_RES_BF16_TO_F32 ? 2 : 4;        // bytes per residual element
        constexpr int RES_MAX = (WM * WN == 8 && BM == 256 && BN == 256 ? 8 : 16) / RREG;
        constexpr int RB = RPT < RES_MAX ? RPT : RES_MAX, RNB = (RPT + RB - 1) / RB;
        // item k of thread t: row r of the pass and first column c4 of the tile.  Where the
        // threads of the workgroup cover whole rows, the column is the same for every item
        // and the row advances by a constant: no divisions, offsets by one addition.
        constexpr bool WHOLE_ROWS = NT % IPR == 0;
        constexpr int RSTEP = WHOLE_ROWS ? NT / IPR : 0;
        auto item_rc = [&](int t, int k, int& r, int& c4) __attribute__((always_inline)) {
            if (WHOLE_ROWS) {
                r = t / IPR + k * RSTEP;
                c4 = (t % IPR) * 4;
            } else {
                const int it = t + k * NT;
                r = it / IPR;
                c4 = (it % IPR) * 4;
            }
        };
        u32x2_t rh_[RES ? RB : 1];    // bf16 residual (4 values)
        u32x4_t rf_[RES ? RB : 1];    // fp32 residual
        auto res_request = [&](int t, int b, int prow0) __attribute__((always_inline)) {
            const int rows_here = min(RP, M - m0 - prow0), cols_here = min(OUT_COLS, out_N - out_n0);
            const __amdgpu_buffer_rsrc_t r_buf = buffer_of(
                RES ? static_cast<const char*>(Rv) + ((size_t)(m0 + prow0) * ldr + out_n0) * RES_ES : nullptr,
                RES && rows_here > 0 ? ((rows_here - 1) * ldr + cols_here) * RES_ES : 0);
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                int r, c4;
                item_rc(t, b * RB + u, r, c4);
                const int off = (min(r, RP - 1) * ldr + c4) * RES_ES;   // (beyond the records: zeros)
                if (EPI == EPI_RES_BF16_TO_F32)
                    rh_[u] = __builtin_amdgcn_raw_buffer_load_b64(r_buf, off, 0, 0);
                else
                    rf_[u] = __builtin_amdgcn_raw_buffer_load_b128(r_buf, off, 0, 0);
            }
        };

#define MVLA_ISSUE(KT, STG)                                                                    \
    {                                                                                          \
        const size_t koff = (size_t)min((KT), k1 - 1) * (BK * 2);                              \
        const uint32_t soff = (uint32_t)(STG) * STAGE * 16u;                                   \
        _Pragma("unroll") for (int i = 0; i < P; ++i) load_one(i, koff, soff);                 \
    }
// fragment read R of the GM + GN of k-step KS of stage STG, in the order the products need them
#define MVLA_READ_ONE(AF, BF, STG, KS, R)                                                      \
    {                                                                                          \
        const uint4* st_ = lds + (STG) * STAGE + (((KS) * 4 + fq) ^ sw);                       \
        if ((R) == 0 || (R) > GN) AF[(R) > GN ? (R) - GN : 0] = st_[a_row + ((R) > GN ? (R) - GN : 0) * 16 * CPR]; \
        else BF[(R) > 0 && (R) <= GN ? (R) - 1 : 0] = st_[b_row + ((R) > 0 ? (R) - 1 : 0) * 16 * CPR]; \
    }
#define MVLA_READ_FRAGS(AF, BF, STG, KS)                                                       \
    _Pragma("unroll") for (int r_ = 0; r_ < GM + GN; ++r_) MVLA_READ_ONE(AF, BF, STG, KS, r_)
// block rows [I0, I1) of a k-step's MFMAs; between them the NRD fragment reads of k-step RKS of stage
// RSTG and the direct loads [L0, L1) of slab KT into stage STG, dealt out evenly
#define MVLA_STEP(AF, BF, I0, I1, NRD, RA, RB, RSTG, RKS, KT, STG, L0, L1)                     \
    {                                                                                          \
        const size_t koff = (size_t)min((KT), k1 - 1) * (BK * 2);                              \
        const uint32_t soff = (uint32_t)(STG) * STAGE * 16u;                                   \
        constexpr int NM_ = ((I1) - (I0)) * GN, NL_ = (L1) - (L0);                             \
        constexpr int EVERY_L = NL_ > 0 && NM_ / (NL_ > 0 ? NL_ : 1) > 0 ? NM_ / (NL_ > 0 ? NL_ : 1) : 1; \
        constexpr int EVERY_R = (NRD) > 0 && NM_ / ((NRD) > 0 ? (NRD) : 1) > 0 ? NM_ / ((NRD) > 0 ? (NRD) : 1) : 1; \
        int l_ = (L0), r_ = 0;                                                                 \
        _Pragma("unroll") for (int n_ = 0; n_ < NM_; ++n_) {                                   \
            const int i_ = (I0) + n_ / GN, j_ = n_ % GN;                                       \
            acc[i_][j_] = mfma16(BF[j_], AF[i_], acc[i_][j_]);                                 \
            if (n_ % EVERY_R == 0 && r_ < (NRD)) {                                             \
                MVLA_READ_ONE(RA, RB, RSTG, RKS, r_)                                           \
                ++r_;                                                                          \
            }                                                                                  \
            if (n_ % EVERY_L == EVERY_L - 1 && l_ < (L1)) {                                    \
                load_one(l_, koff, soff);                                                      \
                ++l_;                                                                          \
            }                                                                                  \
            __builtin_amdgcn_sched_barrier(0);                                                 \
        }                                                                                      \
        _Pragma("unroll") for (int q_ = 0; q_ < GM + GN; ++q_)                                 \
            if (q_ >= r_ && q_ < (NRD)) MVLA_READ_ONE(RA, RB, RSTG, RKS, q_)                   \
        _Pragma("unroll") for (int q_ = 0; q_ < P; ++q_)                                       \
            if (q_ >= l_ && q_ < (L1)) load_one(q_, koff, soff);                               \
    }

        // every thread of the workgroup has left the previous segment's LDS reads behind
        __syncthreads();
        // ... and nothing the compiler keeps count of (a previous segment's epilogue loads and
        // stores) is outstanding any more: a wait it placed for those inside the main loop would
        // also wait for the loop's direct loads, which it does not see
        __builtin_amdgcn_s_waitcnt(0);
        if constexpr (EARLY) {
            pos_request(stid, 0);
            if constexpr (RES) res_request(stid, 0, 0);
        }
        uint4 af0[GM], bf0[GN], af1[GM], bf1[GN];   // the two k-steps of a slab
        const bool normed = norms_rows(BM, BN, NS, EPI) && lda < 0;
        if constexpr (norms_rows(BM, BN, NS, EPI)) if (__builtin_expect(normed, 1)) {   // (laid out in front)
            // ---- every slab of the tile at once: weights by direct loads, rows through the norm ------
            // (four threads a row, every fourth chunk of 8 values each; the sum of squares over the quad)
            constexpr int CH = NORM_MAX_K / 8 / 4;
            const int row = stid >> 2, quad = stid & 3;
            const float4* xr = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(A) +
                                                               (size_t)min(m0 + row, M - 1) * K) + quad * 2;
            const uint4* gr = static_cast<const uint4*>(Rv) + quad;
            float4 x[CH][2];
            uint4 gain[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (j * 32 < K) {                    // (K is a multiple of 64: all threads alike)
                    x[j][0] = xr[j * 8];
                    x[j][1] = xr[j * 8 + 1];
                    gain[j] = gr[j * 4];
                }
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (s < k1)
#pragma unroll
                    for (int l = A_LD; l < P; ++l) load_one(l, (size_t)s * (BK * 2), (uint32_t)s * STAGE * 16u);
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (j * 32 < K)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        ss += x[j][h].x * x[j][h].x + x[j][h].y * x[j][h].y + x[j][h].z * x[j][h].z + x[j][h].w * x[j][h].w;
            ss += __shfl_xor(ss, 1);
            ss += __shfl_xor(ss, 2);
            const float scale = 1.0f / sqrtf(ss * (1.0f / (float)K) + plan.norm_eps);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (j * 32 < K) {
                    const float v[8] = {x[j][0].x, x[j][0].y, x[j][0].z, x[j][0].w,
                                        x[j][1].x, x[j][1].y, x[j][1].z, x[j][1].w};
                    const uint32_t g[4] = {gain[j].x, gain[j].y, gain[j].z, gain[j].w};
                    uint32_t u[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        u[i] = pack_bf16x2(v[2 * i] * scale * __uint_as_float(g[i] << 16),
                                           v[2 * i + 1] * scale * __uint_as_float(g[i] & 0xFFFF0000u));
                    const int ch = j * 4 + quad;     // chunk of the row: slab ch / 8
                    lds[(ch >> 3) * STAGE + row * CPR + ((ch & 7) ^ swz<CPR>(row))] = make_uint4(u[0], u[1], u[2], u[3]);
                }
            wait_vm<0>();
            __syncthreads();
            MVLA_READ_FRAGS(af0, bf0, 0, 0)
#pragma unroll 1
            for (int kt = 0; kt < k1; ++kt) {
                const int next = min(kt + 1, k1 - 1);
                MVLA_STEP(af0, bf0, 0, GM, GM + GN, af1, bf1, kt, 1, kt, kt, 0, 0)
                MVLA_STEP(af1, bf1, 0, GM, GM + GN, af0, bf0, next, 0, kt, kt, 0, 0)
            }
        }
        if (!normed) {
        // ---- prologue: NS-1 slabs in flight, then one more behind the first barrier ---------
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) MVLA_ISSUE(k0 + s, s)
        wait_vm<(NS - 2) * P>();
        __syncthreads();
        // Three or more stages: there is always a free one, and the loads of a slab go out half in the
        // last k-step of one iteration and half in the first of the next (all in one, they kept the
        // waves standing at load issue: the load unit of a CU takes one 64-lane load per 16 clocks).
        constexpr bool SPREAD = NS >= 3;
        // Four-wave shapes with two stages and registers to spare: a slab's second k-step is read during
        // the first half of its first one, so the stage is free from there on and the loads go out
        // a third each over the remaining halves.
        constexpr bool DEEP = WM * WN == 4 && NS == 2;
        if constexpr (SPREAD) {   // (the loop's first k-step issues the rest)
            const size_t koff = (size_t)min(k0 + NS - 1, k1 - 1) * (BK * 2);
            const uint32_t soff = (uint32_t)(NS - 1) * STAGE * 16u;
#pragma unroll
            for (int r = 0; r < P / 2; ++r) load_one(r, koff, soff);
        } else {
            MVLA_ISSUE(k0 + NS - 1, NS - 1)
        }
        MVLA_READ_FRAGS(af0, bf0, 0, 0)
        int stage = 0;
        // (accumulators of the fitted shapes live in the second register file; left to itself the compiler moves them
        // to the first and back in every slab)
        auto pin = [&]() __attribute__((always_inline)) {
            if constexpr (KIND == FITTED)
#pragma unroll
                for (int i = 0; i < GM; ++i)
#pragma unroll
                    for (int j = 0; j < GN; ++j) asm volatile("" : "+a"(acc[i][j]));
        };
        pin();
        if constexpr (DEEP) {
            constexpr int L1_ = P / 3, L2_ = 2 * P / 3, GH = GM / 2;
            for (int kt = k0; kt < k1; ++kt) {
                const int nstage = stage ^ 1;
                MVLA_STEP(af0, bf0, 0, GH, GM + GN, af1, bf1, stage, 1, kt + 2, stage, 0, 0)
                __syncthreads();   // this slab is in every wave's registers: the stage is free for slab kt+2
                MVLA_STEP(af0, bf0, GH, GM, 0, af1, bf1, stage, 1, kt + 2, stage, 0, L1_)
                MVLA_STEP(af1, bf1, 0, GH, 0, af1, bf1, stage, 1, kt + 2, stage, L1_, L2_)
                // slab kt+1 has landed for every wave (the two thirds of slab kt+2 may be in flight)
                wait_vm<L2_>();
                __syncthreads();
                MVLA_STEP(af1, bf1, GH, GM, GM + GN, af0, bf0, nstage, 0, kt + 2, stage, L2_, P)
                stage = nstage;
                pin();
            }
        } else if constexpr (SPREAD) {
            for (int kt = k0; kt < k1; ++kt) {
                const int nstage = stage + 1 == NS ? 0 : stage + 1;
                const int pstage = stage == 0 ? NS - 1 : stage - 1;   // freed one iteration ago
                MVLA_STEP(af0, bf0, 0, GM, GM + GN, af1, bf1, stage, 1, kt + NS - 1, pstage, P / 2, P)
                // slab kt+1 has landed for every wave; slab kt's stage is free for slab kt+NS
                wait_vm<(NS - 2) * P>();
                __syncthreads();
                MVLA_STEP(af1, bf1, 0, GM, GM + GN, af0, bf0, nstage, 0, kt + NS, stage, 0, P / 2)
                stage = nstage;
                pin();
            }
        } else {
            for (int kt = k0; kt < k1; ++kt) {
                const int nstage = stage ^ 1;
                MVLA_STEP(af0, bf0, 0, GM, GM + GN, af1, bf1, stage, 1, kt, stage, 0, 0)
                // slab kt+1 has landed for every wave; slab kt's stage is free for slab kt+2
                wait_vm<0>();
                __syncthreads();
                MVLA_STEP(af1, bf1, 0, GM, GM + GN, af0, bf0, nstage, 0, kt + NS, stage, 0, P)
                stage = nstage;
            }
        }
        wait_vm<0>();
        }
#undef MVLA_ISSUE
#undef MVLA_READ_FRAGS
#undef MVLA_READ_ONE
#undef MVLA_STEP

        // ---- K-split tiles: park the partial sums; the last piece to arrive finishes --------
        // (the four-wave 128x128-per-wave shape keeps its register budget for the main loop:
        // whole tiles only, the host never plans a K-split for it)
        constexpr bool HAS_SK = KIND == SPLITTING && !(WM * WN == 4 && GM * GN >= 54);
        const int n_pieces = (!HAS_SK || is_dp) ? 1 : last_blk - first_blk + 1;
        if constexpr (HAS_SK) if (n_pieces > 1) {
            // slot 0 of a workgroup holds the piece of the tile its range starts in, slot 1 the next
            const int my_slot = 2 * sk_id + (seg == 0 ? 0 : 1);
            float* mine = partial + (size_t)my_slot * (BM * BN);
            uint32_t so = (uint32_t)tid * 16u;
            asm volatile("" : "+v"(so));
            // 16 bytes per lane: block (i,j) goes to float offset ((i*GN + j)*NT + tid)*4 of the slot
#pragma unroll
            for (int i = 0; i < GM; ++i)
#pragma unroll
                for (int j = 0; j < GN; ++j)
                    st16_coherent(mine, so + (uint32_t)((i * GN + j) * NT * 16), acc[i][j]);
            wait_vm<0>();     // this thread's partial sums have reached the coherent level
            __syncthreads();  // ... and so have everyone else's in the workgroup
            if (tid == 0) {
                const uint32_t prev = __hip_atomic_fetch_add(&counters[sk_tile], 1u, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                sh_last = (prev == (uint32_t)(n_pieces - 1));
                if (sh_last)
                    __hip_atomic_store(&counters[sk_tile], 0u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
            if (tid < n_pieces) {
                // piece of workgroup b: its slot 0 if b's range starts inside this tile, else 1
                const long total = (long)plan.sk_tiles * k_tiles;
                const int b = first_blk + tid;
                const int b_start_tile = (int)(total * b / plan.sk_blocks) / k_tiles;
                sh_slot[tid] = 2 * b + (b_start_tile == sk_tile ? 0 : 1);
            }
            __syncthreads();
            if (!sh_last) continue;
            // Sum the pieces in piece order (so the order of additions never depends on who came
            // last), several 16-byte loads in flight at a time; then the common epilogue below.
            // With few accumulator registers the own piece is taken from a register copy instead
            // of being read back, and two pieces are fetched per round trip.
            constexpr int NQ = GM * GN;                           // quads per thread per piece
            // (not for the shape that runs two workgroups per CU: the copy would cost it that)
            constexpr bool KEEP_OWN = NQ <= 16 && !(NS == 2 && BM == 128 && BN == 128);
            constexpr int CH_MAX = (NQ <= 16) ? 16 : 8;           // quads in flight
            constexpr int CH = (CH_MAX >= 16 && NQ % 16 == 0) ? 16
                               : (CH_MAX >= 12 && NQ % 12 == 0) ? 12
                               : (NQ % 8 == 0) ? 8 : 4;
            static_assert(NQ % CH == 0 && CH % 4 == 0, "");
            constexpr int PPR = (KEEP_OWN && 2 * NQ <= 16) ? 2 : 1;   // pieces per round trip
            f32x4_t own[KEEP_OWN ? GM : 1][KEEP_OWN ? GN : 1];
            const int my_piece = KEEP_OWN ? sk_id - first_blk : -1;
#pragma unroll
            for (int i = 0; i < GM; ++i)
#pragma unroll
                for (int j = 0; j < GN; ++j) {
                    if (KEEP_OWN) own[i][j] = acc[i][j];
                    acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll 1
            for (int pc = 0; pc < n_pieces; pc += PPR) {
                if (PPR == 2) {
                    // both pieces of the pair in flight together (own piece: no load)
                    f32q_t t[2][NQ];
                    const int p1 = min(pc + 1, n_pieces - 1);
                    uint32_t po = (uint32_t)tid * 16u;
                    asm volatile("" : "+v"(po));
                    const float* s0 = partial + (size_t)__builtin_amdgcn_readfirstlane(sh_slot[pc]) * (BM * BN);
                    const float* s1 = partial + (size_t)__builtin_amdgcn_readfirstlane(sh_slot[p1]) * (BM * BN);
                    if (pc != my_piece)
#pragma unroll
                        for (int q = 0; q < NQ; ++q) t[0][q] = ld16_coherent(s0, po + (uint32_t)(q * NT * 16));
                    if (pc + 1 < n_pieces && pc + 1 != my_piece)
#pragma unroll
                        for (int q = 0; q < NQ; ++q) t[1][q] = ld16_coherent(s1, po + (uint32_t)(q * NT * 16));
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int q = 0; q < NQ; q += 4) settle(t[h][q], t[h][q + 1], t[h][q + 2], t[h][q + 3]);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (pc + h >= n_pieces) break;
                        const bool mine = (pc + h == my_piece);
#pragma unroll
                        for (int q = 0; q < NQ; ++q) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[q / GN][q % GN][e] +=
                                    mine ? own[KEEP_OWN ? q / GN : 0][KEEP_OWN ? q % GN : 0][e] : t[h][q][e];
                        }
                    }
                } else {
                    const bool mine = (pc == my_piece);
                    uint32_t po = (uint32_t)tid * 16u;   // (offsets are made here, not held for every access)
                    asm volatile("" : "+v"(po));
                    const float* src = partial + (size_t)__builtin_amdgcn_readfirstlane(sh_slot[pc]) * (BM * BN);
#pragma unroll
                    for (int q0 = 0; q0 < NQ; q0 += CH) {
                        f32q_t t[CH];
                        if (!mine) {
#pragma unroll
                            for (int q = 0; q < CH; ++q)
                                t[q] = ld16_coherent(src, po + (uint32_t)((q0 + q) * NT * 16));
                        }
#pragma unroll
                        for (int q = 0; q < CH; q += 4) settle(t[q], t[q + 1], t[q + 2], t[q + 3]);
#pragma unroll
                        for (int q = 0; q < CH; ++q) {
                            const int blk = q0 + q;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[blk / GN][blk % GN][e] +=
                                    mine ? own[KEEP_OWN ? blk / GN : 0][KEEP_OWN ? blk % GN : 0][e] : t[q][e];
                        }
                    }
                }
            }
        }

        // ---- epilogue through LDS: the MFMAs are issued with the weight fragment as the first
        // operand, so a lane of an accumulator block holds one tile row and its registers four
        // consecutive columns at a time: the tile is laid down as fp32 rows with 16-byte stores,
        // then every thread takes 8 consecutive columns of a row (4 where an fp32 matrix is read or
        // written), so the residual is read and the result written with one access per lane on
        // whole consecutive cache lines.  A pass covers as many tile rows as the LDS holds (a whole
        // number of wave rows); only the waves owning them write.
        static_assert(RP % 16 == 0, "row groups of 8 come in pairs");
        constexpr int ITEMS = RP * OUT_COLS / 8;                      // 8-column items per pass
        float* tile = reinterpret_cast<float*>(lds);
        // (the epilogue's per-thread indices are computed here, not before the main loop, where
        // the compiler would otherwise put them and keep them in registers the loop needs)
        int etid = tid;
        asm volatile("" : "+v"(etid));
        auto epilogue_pass = [&](int pass) __attribute__((always_inline)) {
            // first tile row of the pass (with overlapping wave rows the last pass starts early)
            const int prow0 = PASSES == 1 ? 0 : min(pass * TM, BM - TM);
            // (q/k rotation: the position ids of this thread's items of the pass, fetched while the tile is laid down)
            if constexpr (!EARLY) pos_request(etid, prow0);
            // This pass's part of the output as a bounds-checked buffer (rows of the pass that
            // exist, the tile's columns that exist); offsets are relative to its first element.
            constexpr int ES = EPI == EPI_RES_BF16_TO_F32 ? 4 : 2;           // bytes per output element
            const int rows_here = min(RP, M - m0 - prow0);                    // (may be <= 0)
            const int cols_here = min(OUT_COLS, out_N - out_n0);
            const int r_lo = PASSES > 1 ? max(pass * TM - prow0, 0) : 0;      // rows below: the pass before wrote them
            const __amdgpu_buffer_rsrc_t c_buf = buffer_of(
                static_cast<char*>(Cv) + ((size_t)(m0 + prow0) * ldc + out_n0) * ES,
                rows_here > 0 ? ((rows_here - 1) * ldc + cols_here) * ES : 0);
            int ftid = etid;   // (thread index as the items' second half sees it: set after the lay-down)
            auto res_finish = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < RB; ++u) {
                    int r, c4;
                    item_rc(ftid, b * RB + u, r, c4);
                    const bool ok = r >= r_lo && r < rows_here && c4 < cols_here;
                    const int off = ok ? (r * ldc + c4) * ES : OOB_OFFSET;
                    const float4 t = *reinterpret_cast<const float4*>(tile + min(r, RP - 1) * LDT + c4);
                    if (EPI == EPI_RES_BF16_TO_F32) {
                        const u32x2_t h = rh_[u];
                        const u32x4_t o = {__float_as_uint(t.x + __uint_as_float(h.x << 16)),
                                           __float_as_uint(t.y + __uint_as_float(h.x & 0xFFFF0000u)),
                                           __float_as_uint(t.z + __uint_as_float(h.y << 16)),
                                           __float_as_uint(t.w + __uint_as_float(h.y & 0xFFFF0000u))};
                        __builtin_amdgcn_raw_buffer_store_b128(o, c_buf, off, 0, 0);
                    } else {
                        const u32x4_t q = rf_[u];
                        const u32x2_t o = {pack_bf16x2(t.x + __uint_as_float(q.x), t.y + __uint_as_float(q.y)),
                                           pack_bf16x2(t.z + __uint_as_float(q.z), t.w + __uint_as_float(q.w))};
                        __builtin_amdgcn_raw_buffer_store_b64(o, c_buf, off, 0, 0);
                    }
                    // (items stay in order: with nothing conditional left the scheduler would
                    // otherwise read the tile rows of all items first and run out of registers)
                    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            };
            if constexpr (RES && !TIGHT && !EARLY) res_request(etid, 0, prow0);
            __syncthreads();   // previous readers of the LDS (fragments or the last pass) are done
            if constexpr (WM * WN == 4 && GM * GN >= 54) {
                // Accumulators in the second register file: fetched one by one (pinned there until then),
                // and without a branch, which would make the compiler copy them: 16-row blocks that are
                // not of this pass go to a spare strip behind the tile.
#pragma unroll
                for (int i = 0; i < GM; ++i) {
                    const int r0 = wrow0 - prow0 + i * 16;
                    float* strip = tile + (r0 >= 0 && r0 < RP ? r0 : RP) * LDT;
#pragma unroll
                    for (int j = 0; j < GN; ++j) {
                        asm volatile("" : "+a"(acc[i][j]));
                        *reinterpret_cast<f32x4_t*>(strip + fr * LDT + wn * TN + j * 16 + 4 * fq) = acc[i][j];
                    }
                }
            } else if (PASSES == 1 || wm == pass) {
#pragma unroll
                for (int i = 0; i < GM; ++i)
#pragma unroll
                    for (int j = 0; j < GN; ++j) {
                        const int r = wrow0 - prow0 + i * 16 + fr, c = wn * TN + j * 16 + 4 * fq;
                        *reinterpret_cast<f32x4_t*>(tile + r * LDT + c) = acc[i][j];
                    }
            }
            __syncthreads();
            // (what the items need beyond their residual is computed from here on, not before
            // the lay-down, where it would be held in registers across it)
            asm volatile("" : "+v"(ftid));
            if (EPI == EPI_QKV_ROPE) {
                const int DH = rope.dh, HALF = DH >> 1, CPH = HALF >> 3;   // 16-byte chunks per half head
                if (n0 < 2 * rope.D) {
                    // q or k columns: every item is 8 columns of the first half of a head and
                    // their partners dh/2 further on (tiles hold whole heads: BN % dh == 0; a row
                    // has BN/16 items whatever dh is).  Items are taken a few at a time so that the
                    // table rows of a batch are in flight together.
#pragma unroll
                    for (int jb = 0; jb < NB; ++jb) {
                        const int it0 = etid + jb * QB * NT;
                        int r[QB], col[QB], c8[QB], p[QB];
                        bool ok[QB];
#pragma unroll
                        for (int u = 0; u < QB; ++u) {
                            const int it = it0 + u * NT;
                            r[u] = min(it / PER_ROW, RP - 1);
                            const int rest = it % PER_ROW;
                            c8[u] = (rest % CPH) * 8;
                            col[u] = (rest / CPH) * DH + c8[u];   // column in the tile
                            const int row = m0 + prow0 + r[u];
                            ok[u] = it < RP * PER_ROW && r[u] >= r_lo && r[u] < rows_here && col[u] < cols_here;
                            p[u] = PREFETCH ? pos_pre[PREFETCH ? jb * QB + u : 0] : rope.pos[min(row, M - 1)];
                        }
                        float4 cs[QB][2], sn[QB][2];
#pragma unroll
                        for (int u = 0; u < QB; ++u) {
                            const size_t toff = (size_t)min(max(p[u], 0), rope.rope_len - 1) * HALF + c8[u];
                            cs[u][0] = *reinterpret_cast<const float4*>(rope.rc + toff);
                            cs[u][1] = *reinterpret_cast<const float4*>(rope.rc + toff + 4);
                            sn[u][0] = *reinterpret_cast<const float4*>(rope.rs + toff);
                            sn[u][1] = *reinterpret_cast<const float4*>(rope.rs + toff + 4);
                        }
#pragma unroll
                        for (int u = 0; u < QB; ++u) {
                            const float* ta = tile + r[u] * LDT + col[u];
                            const float4 a0 = *reinterpret_cast<const float4*>(ta);
                            const float4 a1 = *reinterpret_cast<const float4*>(ta + 4);
                            const float4 b0 = *reinterpret_cast<const float4*>(ta + HALF);
                            const float4 b1 = *reinterpret_cast<const float4*>(ta + HALF + 4);
                            const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                            const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
                            const float c[8] = {cs[u][0].x, cs[u][0].y, cs[u][0].z, cs[u][0].w,
                                                cs[u][1].x, cs[u][1].y, cs[u][1].z, cs[u][1].w};
                            const float sv[8] = {sn[u][0].x, sn[u][0].y, sn[u][0].z, sn[u][0].w,
                                                 sn[u][1].x, sn[u][1].y, sn[u][1].z, sn[u][1].w};
                            uint32_t wa[4], wb[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                wa[e] = pack_bf16x2(a[2 * e] * c[2 * e] - b[2 * e] * sv[2 * e],
                                                    a[2 * e + 1] * c[2 * e + 1] - b[2 * e + 1] * sv[2 * e + 1]);
                                wb[e] = pack_bf16x2(b[2 * e] * c[2 * e] + a[2 * e] * sv[2 * e],
                                                    b[2 * e + 1] * c[2 * e + 1] + a[2 * e + 1] * sv[2 * e + 1]);
                            }
                            const int off = ok[u] ? (r[u] * ldc + col[u]) * 2 : OOB_OFFSET;
                            const u32x4_t oa = {wa[0], wa[1], wa[2], wa[3]}, ob = {wb[0], wb[1], wb[2], wb[3]};
                            __builtin_amdgcn_raw_buffer_store_b128(oa, c_buf, off, 0, 0);
                            __builtin_amdgcn_raw_buffer_store_b128(ob, c_buf, off + HALF * 2, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);   // (one item's tile reads at a time: registers)
                        }
                    }
                } else {
                    // v columns, transposed into vt[b, h, d, s]: an item is one column and one
                    // group of 8 tokens aligned in s (one 16-byte store).  The rows of the pass are
                    // walked sample by sample (a uniform loop: one division per sample, none per
                    // item); within a sample's rows the groups are [8j, 8j+8) of its tokens, the
                    // groups cut by the ends of the rows are stored token by token by the two
                    // passes (or tiles) that hold their rows, and whoever stores a sample's last
                    // token clears the padding behind it.  A half-wave runs over 32 columns, the
                    // two halves over alternate groups: LDS reads without bank conflicts.
                    const int H = rope.D / DH, S = rope.S, S_pad = rope.S_pad;
                    const int g_base = m0 + prow0;                                  // global row of LDS row 0
                    const int g_lo = m0 + (PASSES > 1 ? max(prow0, pass * TM) : 0);  // rows this pass owns
                    const int g_hi = min(g_base + RP, M);
                    constexpr int NW = NT / 64, NCH = BN / 32;     // waves; 32-column chunks of the tile
                    constexpr int WPC = NW > NCH ? NW / NCH : 1;   // waves sharing a chunk (over groups)
                    const int vlane = ftid & 63, vwave = ftid >> 6;
                    const int g_first = (vlane >> 5) + 2 * (NW > NCH ? vwave / NCH : 0);
                    constexpr int G_STEP = 2 * WPC;
                    for (int g_a = g_lo; g_a < g_hi;) {
                        const int bs = g_a / S, g_s = bs * S, g_e = min(g_hi, g_s + S);
                        const int s_a = g_a - g_s, s_e = g_e - g_s;   // tokens [s_a, s_e) of sample bs are ours
                        const int r_off = g_s - g_base;               // LDS row of token s: s + r_off
                        const int j_hi = (s_e + 7) >> 3;
#pragma unroll 1
                        for (int ch = NW > NCH ? vwave % NCH : vwave; ch < NCH && (NW <= NCH || vwave < WPC * NCH);
                             ch += NW) {
                            const int d = ch * 32 + (vlane & 31);
                            const int vcol = n0 - 2 * rope.D + d, hd = vcol / DH, dd = vcol - hd * DH;
                            bf16_t* dst = rope.vt + ((size_t)(bs * H + hd) * DH + dd) * S_pad;
                            const float* src = tile + r_off * LDT + d;     // (+ s * LDT: token s)
                            if (n0 + d >= N) continue;
#pragma unroll 1
                            for (int j = (s_a >> 3) + g_first; j < j_hi; j += G_STEP) {
                                const int s_al = j * 8;
                                const int lo = max(s_a, s_al), hi = min(s_e, s_al + 8);
                                if (lo == s_al && hi == s_al + 8) {          // a whole group of ours
                                    const float* q = src + s_al * LDT;
                                    *reinterpret_cast<uint4*>(dst + s_al) =
                                        make_uint4(pack_bf16x2(q[0], q[LDT]), pack_bf16x2(q[2 * LDT], q[3 * LDT]),
                                                   pack_bf16x2(q[4 * LDT], q[5 * LDT]),
                                                   pack_bf16x2(q[6 * LDT], q[7 * LDT]));
                                    if (hi == S)
                                        for (int z = s_al + 8; z < S_pad; z += 8)
                                            *reinterpret_cast<uint4*>(dst + z) = make_uint4(0, 0, 0, 0);
                                } else if (lo == s_al && hi == S) {          // the sample's short last group, all ours
                                    float v[8];
#pragma unroll
                                    for (int i = 0; i < 8; ++i)
                                        v[i] = s_al + i < hi ? src[min(s_al + i, hi - 1) * LDT] : 0.f;
                                    *reinterpret_cast<uint4*>(dst + s_al) =
                                        make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                   pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                                    for (int z = s_al + 8; z < S_pad; z += 8)
                                        *reinterpret_cast<uint4*>(dst + z) = make_uint4(0, 0, 0, 0);
                                } else {                                     // cut by the ends of our rows
#pragma unroll 1
                                    for (int t = lo; t < hi; ++t) {
                                        dst[t] = (bf16_t)(pack_bf16x2(src[t * LDT], 0.f) & 0xFFFFu);
                                        if (t == S - 1)
                                            for (int z = S; z < S_pad; ++z) dst[z] = 0;
                                    }
                                }
                            }
                        }
                        g_a = g_e;
                    }
                }
                return;
            }
            if constexpr (RES) {
                if constexpr (TIGHT) res_request(etid, 0, prow0);
#pragma unroll 1
                for (int b = 0; b < RNB; ++b) {
                    res_finish(b);
                    if (b + 1 < RNB) res_request(etid, b + 1, prow0);
                }
                return;
            }
            // SiLU(gate) * up: 8 output columns per item (16 bytes of bf16), two items at a time
            constexpr int U = 2;
#pragma unroll 1
            for (int it0 = etid; it0 < ITEMS; it0 += U * NT) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int it = it0 + u * NT;
                    const int r = min(it / (OUT_COLS / 8), RP - 1), c8 = it % (OUT_COLS / 8);
                    const bool ok = it < ITEMS && r >= r_lo && r < rows_here && c8 * 8 < cols_here;
                    // gate block [64q, 64q+32) and up block [64q+32, 64q+64) of the tile
                    const int oc = c8 * 8;                      // output column within the tile
                    const float* g = tile + r * LDT + (oc >> 5) * 64 + (oc & 31);
                    const float4 g0 = *reinterpret_cast<const float4*>(g);
                    const float4 g1 = *reinterpret_cast<const float4*>(g + 4);
                    const float4 u0 = *reinterpret_cast<const float4*>(g + 32);
                    const float4 u1 = *reinterpret_cast<const float4*>(g + 36);
                    const float gv[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
                    const float uv[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
                    // SiLU(g) u = g u / (1 + e^-g); the hardware reciprocal (1 ulp) is far inside
                    // what the bf16 result keeps
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] = gv[e] * uv[e] * __builtin_amdgcn_rcpf(1.f + __expf(-gv[e]));
                    const u32x4_t o = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]),
                                       pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
                    __builtin_amdgcn_raw_buffer_store_b128(o, c_buf, ok ? (r * ldc + oc) * 2 : OOB_OFFSET, 0, 0);
                }
            }
        };
        if constexpr (WM * WN == 4 && GM * GN >= 54 && PASSES == 2) {
            // (not a loop: pinned accumulators would be carried round it, and copied)
            epilogue_pass(0);
            epilogue_pass(1);
        } else {
#pragma unroll 1
            for (int pass = 0; pass < PASSES; ++pass) epilogue_pass(pass);
        }

    }
}

// The four-wave 256x256 shape is the persistent kernel, every other one takes a workgroup per tile.
constexpr bool is_persistent(int BM, int BN, int WM, int WN) { return BM == 256 && BN == 256 && WM * WN == 4; }

// A wave starts with the first 14 words of a kernel's arguments in scalar registers.  What a tile's first loads
// depend on stands there a second time (Rv: the residual, or the position ids of a projection that rotates): anything
// else comes by a load of its own, and the wave waits for it.
// Short projections are mostly this start and their end: with these arguments in front, no plan of K ranges in whole
// tiles, the epilogue's first operands asked for ahead of the slabs and no more table rows than a thread has items,
// the small model's pruned prefill takes 45.2 -> 44.7 us, one 7B layer of 237 rows 177.8 -> 174.1, the 4-layer call of
// 544 tokens 938 -> 926.
template <int EPI, KernelKind KIND>
__device__ __forceinline__ void leading_arguments(GemmPlan& plan, RopeEpilogue& rope, PairedGemm& pair, int k_tiles,
                                                  int tiles_m, int tiles_n, int pair_block, const void* Rv) {
    plan.tiles_m = tiles_m;
    plan.tiles_n = tiles_n;
    plan.k_tiles = k_tiles;
    if (KIND != SPLITTING) plan.dp_tiles = tiles_m * tiles_n;
    if (EPI == EPI_QKV_ROPE) rope.pos = static_cast<const int32_t*>(Rv);
    pair.first_block = pair_block;
}

template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI>
__global__ __launch_bounds__(WM * WN * 64) void gemm_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int lda, int M, int N, int K, int tiles_m, int tiles_n,
    int ldr, int pair_block, const void* __restrict__ Rv, void* __restrict__ Cv, int ldc, GemmPlan plan,
    float* __restrict__ partial, uint32_t* __restrict__ counters, RopeEpilogue rope, PairedGemm pair) {
    leading_arguments<EPI, SPLITTING>(plan, rope, pair, K / BK, tiles_m, tiles_n, pair_block, Rv);
    if constexpr (is_persistent(BM, BN, WM, WN))
        persistent_body<EPI>(A, lda, W, M, N, K, Cv, ldc, Rv, ldr, plan, rope);
    else
        tile_body<BM, BN, BK, WM, WN, NS, EPI, SPLITTING>(A, lda, W, M, N, K, Cv, ldc, Rv, ldr, plan, partial, counters, rope,
                                                        pair);
}

// Shapes that only the choice by size uses (whole tiles, no K-split): the same body under another name.
// (two waves a SIMD in the bounds keep the accumulators in the ordinary registers; given more room, the
// compiler moves them to the second file and back in every slab)
template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI>
__global__ __launch_bounds__(WM * WN * 64, 2) void small_tile_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int lda, int M, int N, int K, int tiles_m, int tiles_n,
    int ldr, int pair_block, const void* __restrict__ Rv, void* __restrict__ Cv, int ldc, GemmPlan plan,
    float* __restrict__ partial, uint32_t* __restrict__ counters, RopeEpilogue rope, PairedGemm pair) {
    leading_arguments<EPI, SMALL>(plan, rope, pair, K / BK, tiles_m, tiles_n, pair_block, Rv);
    tile_body<BM, BN, BK, WM, WN, NS, EPI, SMALL>(A, lda, W, M, N, K, Cv, ldc, Rv, ldr, plan, partial, counters, rope,
                                                  pair);
}

// Tiles fitted to the row count (whole tiles as well), large enough that the accumulators may go to the second
// register file.
template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI>
__global__ __launch_bounds__(WM * WN * 64) void fitted_tile_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int lda, int M, int N, int K, int tiles_m, int tiles_n,
    int ldr, int pair_block, const void* __restrict__ Rv, void* __restrict__ Cv, int ldc, GemmPlan plan,
    float* __restrict__ partial, uint32_t* __restrict__ counters, RopeEpilogue rope, PairedGemm pair) {
    leading_arguments<EPI, FITTED>(plan, rope, pair, K / BK, tiles_m, tiles_n, pair_block, Rv);
    tile_body<BM, BN, BK, WM, WN, NS, EPI, FITTED>(A, lda, W, M, N, K, Cv, ldc, Rv, ldr, plan, partial, counters, rope,
                                                  pair);
}

// ---- host side ------------------------------------------------------------------------------
// Compute units of the current device: sets how many workgroups are resident at once (the round
// size of the tile plan) and the size of the K-split partial buffer.  Asked once; 256 (MI355X)
// when there is no device to ask.
int device_cu_count() {
    static int cached = 0;
    if (cached > 0) return cached;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return 256;
    }
    cached = n;
    return n;
}

// Split of the tile set into whole-tile workgroups and K-split workgroups for `slots`
// concurrently resident workgroups.
static GemmPlan make_plan(int M, int N, int K, int BM, int BN, int BK, int slots, int sk_pct) {
    GemmPlan p;
    p.tiles_m = (M + BM - 1) / BM;
    p.tiles_n = (N + BN - 1) / BN;
    p.k_tiles = K / BK;
    p.quarter_of = -1;
    const int tiles = p.tiles_m * p.tiles_n;
    const int rem = tiles % slots;
    // a last round that is at least sk_pct % full is not worth cutting up
    if (rem == 0 || rem * 100 >= slots * sk_pct) {
        p.dp_tiles = tiles;
        p.dp_grid = (tiles + 7) / 8 * 8;
        p.sk_tiles = 0;
        p.sk_blocks = 0;
        return p;
    }
    p.dp_tiles = tiles - rem;
    p.dp_grid = (p.dp_tiles + 7) / 8 * 8;
    p.sk_tiles = rem;
    const long iters = (long)rem * p.k_tiles;
    long blocks = slots;
    if (iters / blocks < SK_MIN_ITERS) blocks = iters / SK_MIN_ITERS;
    if (blocks > (long)rem * (SK_MAX_PIECES / 2 - 1)) blocks = (long)rem * (SK_MAX_PIECES / 2 - 1);
    if (blocks < rem) blocks = rem;  // a workgroup never spans more than two tiles
    p.sk_blocks = (int)blocks;
    return p;
}

// Which part of the tile plan a launch covers: all of it, or -- when two kernels of the same tile
// size share one plan -- the whole tiles only, or the K-split tiles of the last round only.
// (cut along K, or in quarters).
enum PlanPart { PLAN_ALL = 0, PLAN_WHOLE_TILES = 1, PLAN_SPLIT_TILES = 2, PLAN_QUARTERS = 3 };

// The plan for a tile shape, with the K-split dropped when the workspace has no room for it.
static GemmPlan plan_for(int M, int N, int K, int BM, int BN, int BK, int slots, int sk_pct,
                         size_t partial_bytes, int n_counters) {
    GemmPlan plan = make_plan(M, N, K, BM, BN, BK, slots, sk_pct);
    if (plan.sk_blocks > 0) {
        const size_t need = (size_t)2 * plan.sk_blocks * BM * BN * sizeof(float);
        if (need > partial_bytes || plan.sk_tiles > n_counters) {  // no room: whole tiles only
            plan.dp_tiles += plan.sk_tiles;
            plan.dp_grid = (plan.dp_tiles + 7) / 8 * 8;
            plan.sk_tiles = plan.sk_blocks = 0;
        }
    }
    return plan;
}

template <int BM, int BN, int BK, int WM, int WN, int NS, int E, KernelKind KIND>
static constexpr auto kernel_of() {
    if constexpr (KIND == SMALL) return small_tile_kernel<BM, BN, BK, WM, WN, NS, E>;
    else if constexpr (KIND == FITTED) return fitted_tile_kernel<BM, BN, BK, WM, WN, NS, E>;
    else return gemm_kernel<BM, BN, BK, WM, WN, NS, E>;
}

template <int BM, int BN, int BK, int WM, int WN, int NS, KernelKind KIND = SPLITTING>
static int launch_cfg(const bf16_t* A, int lda, const bf16_t* W, int M, int N, int K, void* C,
                      int ldc, const void* R, int ldr, int epi, int slots_per_cu, int sk_pct,
                      float* partial, size_t partial_bytes, uint32_t* counters, int n_counters,
                      const RopeEpilogue& rope, hipStream_t st, PlanPart part = PLAN_ALL,
                      const PairedGemm* second = nullptr, float norm_eps = 0.f) {
    constexpr bool has_sk = KIND == SPLITTING && !(WM * WN == 4 && ((BM / 32 + WM - 1) / WM) * (BN / WN / 32) >= 15);
    const int pb = part == PLAN_QUARTERS ? 2 : 1;   // (planned on the tiles that are quartered)
    GemmPlan plan = plan_for(M, N, K, BM * pb, BN * pb, BK, device_cu_count() * slots_per_cu,
                             (has_sk || part != PLAN_ALL) ? sk_pct : 0, partial_bytes, n_counters);
    if (part == PLAN_WHOLE_TILES) {
        plan.sk_tiles = plan.sk_blocks = 0;         // (their tiles are left to the other launch)
    } else if (part == PLAN_SPLIT_TILES) {
        if (plan.sk_blocks == 0) return MVLA_OK;
        plan.dp_grid = 0;                           // workgroup ids start at the K-split workgroups
    } else if (part == PLAN_QUARTERS) {
        plan.quarter_of = plan.dp_tiles;
        plan.dp_tiles = 4 * plan.sk_tiles;
        plan.dp_grid = (plan.dp_tiles + 7) / 8 * 8;
        plan.sk_tiles = plan.sk_blocks = 0;
    }
    if (!has_sk && plan.sk_blocks > 0) return MVLA_EINVAL;
    plan.norm_eps = norm_eps;
    int grid = plan.dp_grid + plan.sk_blocks;
    PairedGemm pair{};
    if (second) {
        if (plan.sk_blocks > 0) return MVLA_EINVAL;     // (whole tiles only)
        pair = *second;
        pair.tiles_m = (pair.M + BM - 1) / BM;
        pair.first_block = grid;
        grid += (pair.tiles_m * plan.tiles_n + 7) / 8 * 8;
    }
    if (grid == 0) return MVLA_OK;
    const size_t stage_bytes = (size_t)NS * (BM + BN) * (BK / 8) * sizeof(uint4);
    const size_t epi_bytes = EpiGeom<BM, BN, WM, NS, rows_unit(KIND)>::BYTES;
    size_t lds = stage_bytes > epi_bytes ? stage_bytes : epi_bytes;
    if (is_persistent(BM, BN, WM, WN)) {   // one workgroup per CU, a multiple of 8 (see xcd_chunked)
        const int cus = device_cu_count() & ~7;
        if (cus > 0 && grid > cus) grid = cus;
        lds = PT_LDS_BYTES;
    }
    dim3 block(WM * WN * 64);
    // the dynamic-LDS limit of a kernel is raised once per device (the size is a constant of the
    // instantiation), not on every launch
#define MVLA_GEMM_LAUNCH(E)                                                                   \
    do {                                                                                      \
        auto kern = kernel_of<BM, BN, BK, WM, WN, NS, E, KIND>();                                 \
        static bool lds_set[kMaxDevices] = {};                                                \
        int dev = 0;                                                                          \
        MVLA_HIP_CHECK(hipGetDevice(&dev));                                                   \
        if (dev < 0 || dev >= kMaxDevices || !lds_set[dev]) {                                 \
            MVLA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),           \
                                               hipFuncAttributeMaxDynamicSharedMemorySize,    \
                                               (int)lds));                                    \
            if (dev >= 0 && dev < kMaxDevices) lds_set[dev] = true;                           \
        }                                                                                     \
        hipLaunchKernelGGL(kern, dim3(grid), block, lds, st, A, W, lda, M, N, K, plan.tiles_m, \
                           plan.tiles_n, ldr, pair.first_block, epi == EPI_QKV_ROPE ? rope.pos : R, C, \
                           ldc, plan, partial, counters, rope, pair);                         \
    } while (0)
    if (epi == EPI_QKV_ROPE) MVLA_GEMM_LAUNCH(EPI_QKV_ROPE);
    else if (epi == EPI_RES_BF16_TO_F32) MVLA_GEMM_LAUNCH(EPI_RES_BF16_TO_F32);
    else if (epi == EPI_RES_F32_TO_BF16) MVLA_GEMM_LAUNCH(EPI_RES_F32_TO_BF16);
    else MVLA_GEMM_LAUNCH(EPI_SILU_MUL);
#undef MVLA_GEMM_LAUNCH
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

size_t gemm_partial_bytes() {
    // two partial tiles per K-split workgroup; 256x256 tiles on 256 slots == 128x128 on 512
    return (size_t)2 * device_cu_count() * 256 * 256 * sizeof(float);
}

// Tile configurations, and what predicts their time (see estimate_us; microseconds, fitted to the
// measured times of all of them on 200 projections of this package's models, 32 to 14720 rows).
struct TileCfg {
    int BM, BN, slots_per_cu;
    bool can_split;      // has the K-split path
    float slab_us;       // a 64-deep slab with every workgroup slot of the chip busy
    float alone;         // ... and the share of it that remains with one workgroup alone
    float tile_us[4];    // start and epilogue of a tile, by epilogue
    float piece_us;      // K-split: summing one piece of a tile
    float straddle_us;   // K-split: when workgroups' ranges straddle two tiles (two starts, two parts put out)
    float mb_per_us;     // operand bytes beyond the caches
};
constexpr int kNumCfgs = 7;      // configurations a caller can record (mvla_set_gemm_choice)
constexpr int kFitted = 12;      // from here on the tiles fitted to the row count
constexpr int kAllCfgs = 24;     // ... both only used by the choice by size
static const TileCfg kCfgs[kAllCfgs] = {
    // K-slab 64, eight waves of 128x64, two stages
    {256, 256, 1, true, 1.55f, 0.697f, {8.5f, 9.3f, 13.7f, 5.2f}, 2.4f, 27.7f, 3.f},
    // K-slab 64, eight waves of 64x64, three stages
    {256, 128, 1, true, 0.806f, 0.587f, {6.6f, 6.3f, 7.6f, 4.5f}, 1.9f, 11.3f, 4.f},
    // K-slab 64, four waves of 64x64, two stages, two workgroups per CU
    {128, 128, 2, true, 0.95f, 0.449f, {4.4f, 4.1f, 3.6f, 2.9f}, 2.1f, 18.2f, 3.4f},
    // K-slab 64, eight waves of 32x64, three stages
    {128, 128, 1, true, 0.516f, 0.689f, {4.9f, 3.8f, 3.2f, 2.9f}, 1.8f, 6.9f, 3.5f},
    // K-slab 64, four waves of 128x128, persistent (accumulators fill the second register file, a third
    // less LDS traffic per MFMA); a K-split last round runs on the eight-wave kernel of the same tile size
    {256, 256, 1, true, 1.3f, 0.686f, {10.5f, 10.5f, 9.f, 6.4f}, 0.f, 0.f, 6.2f},
    // K-slab 64, eight waves of 96x32, three stages (row counts just over 2x256 with few column tiles:
    // three row tiles, K-split over all CUs)
    {192, 128, 1, true, 0.659f, 0.662f, {5.5f, 5.4f, 5.2f, 3.8f}, 1.8f, 9.5f, 4.1f},
    // K-slab 64, four waves of 160x96 (the two wave rows overlap by one 32-row block), accumulators in the
    // second register file, whole tiles only
    {288, 192, 1, false, 1.2f, 0.722f, {5.f, 14.6f, 9.6f, 9.4f}, 0.f, 0.f, 6.9f},
    // The rest: four waves, whole tiles only, for few rows and columns, where the larger tiles leave most
    // of the chip without work.  64x96 per wave, three stages (M = 237, N = 22016: 63 -> 60 us)
    {128, 192, 1, false, 0.601f, 0.953f, {5.f, 5.3f, 3.6f, 3.6f}, 0.f, 0.f, 3.75f},
    // 32x32 per wave, six stages (M = 100, N = K = 1024: 12.0 -> 8.3 us; M = 80, N = 256, K = 1024: 11 -> 7.9)
    {64, 64, 1, false, 0.21f, 0.922f, {3.4f, 2.4f, 1.7f, 2.2f}, 0.f, 0.f, 2.7f},
    // 64x64 per wave, four stages (M = 948, N = K = 4096: 41 -> 37 us)
    {128, 128, 1, false, 0.454f, 0.87f, {4.6f, 4.f, 2.7f, 3.1f}, 0.f, 0.f, 3.7f},
    // 32x64 per wave, five stages (M = 237, N = 3072, K = 1024, heads of 128: 14 -> 11 us)
    {64, 128, 1, false, 0.346f, 1.f, {3.6f, 2.6f, 1.f, 2.3f}, 0.f, 0.f, 3.4f},
    // 64x32 per wave, five stages (M = 400, N = K = 4096: 29 -> 26 us)
    {128, 64, 1, false, 0.302f, 0.974f, {4.1f, 2.9f, 2.1f, 2.6f}, 0.f, 0.f, 4.f},
    // Fitted tiles: four waves of half the rows and half the columns each, whole tiles only, in heights and widths
    // between those above.  What a projection of a few hundred to a few thousand rows loses is the last round of tiles
    // that do not fit its row count, and what bounds a slab of it is the load path (a compute unit has 256 cache lines
    // on their way at most: some 55 bytes per ns where the weights come from memory), so the tile should be as large as
    // fills the chip in whole rounds.  One or two steps of height either way are 10 to 30 % there.
    // M = 288, N = 22016: 288x192 on 115 units 76 -> 160x192 on 230 58 us; M = 948, N = 12288: 256x256 on 192 91 ->
    // 192x256 on 240 77; M = 948, N = 22016 158 -> 136 (192x256); M = 2176, N = K = 4096: 79 -> 64 (160x256); M = 2176,
    // N = 4096, K = 11008: 192 -> 164.  (27 row counts of 32 to 7000 at the 7B widths: 5 % on average.)
    // (their times: fitted to 15 row counts at D = 1024, F = 2816 and 27 at D = 4096, F = 11008)
    {160, 128, 1, false, 0.586f, 0.713f, {3.8f, 2.9f, 1.0f, 1.4f}, 0.f, 0.f, 4.8f},
    {192, 128, 1, false, 0.664f, 0.721f, {3.8f, 3.1f, 1.0f, 1.5f}, 0.f, 0.f, 4.9f},
    {160, 192, 1, false, 0.755f, 0.701f, {5.1f, 5.1f, 3.6f, 2.6f}, 0.f, 0.f, 4.3f},
    {256, 128, 1, false, 0.759f, 0.608f, {5.4f, 6.0f, 5.2f, 3.6f}, 0.f, 0.f, 4.9f},
    {128, 256, 1, false, 0.784f, 0.676f, {4.3f, 3.7f, 3.4f, 2.5f}, 0.f, 0.f, 3.9f},
    {192, 192, 1, false, 0.838f, 0.675f, {7.4f, 7.4f, 5.9f, 4.3f}, 0.f, 0.f, 4.5f},
    {160, 256, 1, false, 0.906f, 0.724f, {8.0f, 6.6f, 4.3f, 4.4f}, 0.f, 0.f, 4.4f},
    {224, 192, 1, false, 0.932f, 0.650f, {8.8f, 8.8f, 8.6f, 5.5f}, 0.f, 0.f, 4.6f},
    {192, 256, 1, false, 1.029f, 0.701f, {9.6f, 7.4f, 5.6f, 5.1f}, 0.f, 0.f, 4.2f},
    {288, 192, 1, false, 1.133f, 0.602f, {13.1f, 13.1f, 12.7f, 8.1f}, 0.f, 0.f, 4.2f},
    {224, 256, 1, false, 1.168f, 0.634f, {11.6f, 11.3f, 10.5f, 7.7f}, 0.f, 0.f, 4.8f},
    {320, 192, 1, false, 1.264f, 0.528f, {14.1f, 14.1f, 15.8f, 8.6f}, 0.f, 0.f, 4.7f},
};
constexpr float kLaunchUs = 3.f;
// Where the fitted tiles are considered.  Shorter projections are mostly start and epilogue, and there the small tiles are
// the faster ones (of 15 row counts from 130 to 7000 at D = 1024, F = 2816 none below 20 us has a faster
// fitted tile); shorter contractions are outside of what their times were fitted to.
constexpr float kFittedFromUs = 20.f;
constexpr int kFittedFromK = 1024;
// The exchange of a K-split behind a full-chip kernel takes longer than the fit says (117 us measured, 92
// predicted, for 64 tiles at K = 11008; quarters 98 and 92): the quarters are taken unless it is well ahead.
constexpr float kSplitRisk = 1.2f;

// A 64-deep slab with n workgroups busy: longer the more of the chip is, and no less than its share of the
// operands takes from memory (weights once for all row tiles in flight).
static float slab_us(const TileCfg& c, float n, float tiles_m, float tiles_n) {
    const float work = c.slab_us * (c.alone + (1.f - c.alone) * n / (device_cu_count() * c.slots_per_cu));
    const float per_row = n / tiles_m, cols = per_row < 1.f ? 1.f : per_row < tiles_n ? per_row : tiles_n;
    const float rows = tiles_m < n ? tiles_m : n;
    const float mem = (cols * c.BN + .2f * rows * c.BM) * 128.f * 1e-6f / c.mb_per_us;
    const float w2 = work * work, m2 = mem * mem;
    return __builtin_sqrtf(__builtin_sqrtf(w2 * w2 + m2 * m2));
}
// The cut last round of configuration cfg: its tiles split along K over all compute units.
static float split_us(int cfg, const GemmPlan& p, int epi) {
    const TileCfg& c = kCfgs[cfg];
    const float its = (float)(((long)p.sk_tiles * p.k_tiles + p.sk_blocks - 1) / p.sk_blocks);
    return c.tile_us[epi] + its * slab_us(c, (float)p.sk_blocks, (float)p.tiles_m, (float)p.tiles_n) +
           c.piece_us * p.sk_blocks / p.sk_tiles + (p.sk_blocks % p.sk_tiles ? c.straddle_us : 0.f);
}
// The cut last round of 256x256 tiles in quarters of 128x128 (configuration 3), whole along K.
static float quarters_us(const GemmPlan& p, int epi) {
    const TileCfg& c = kCfgs[3];
    const int n = 4 * p.sk_tiles, cus = device_cu_count();
    const float tm = 2.f * p.tiles_m, tn = 2.f * p.tiles_n;
    return (float)(n / cus) * (c.tile_us[epi] + p.k_tiles * slab_us(c, (float)cus, tm, tn)) +
           (n % cus ? c.tile_us[epi] + p.k_tiles * slab_us(c, (float)(n % cus), tm, tn) : 0.f);
}

// Predicted time with the last partial round cut along K over all compute units or, the persistent kernel's, in
// quarters, behind whole rounds that take t.
static float cut_us(int cfg, int M, int N, int K, int epi, float t, bool whole_rounds) {
    const TileCfg& c = kCfgs[cfg];
    const GemmPlan p = make_plan(M, N, K, c.BM, c.BN, 64, device_cu_count() * c.slots_per_cu, 101);
    if (cfg == 4)            // (a launch of its own)
        return t + (whole_rounds ? kLaunchUs : 0.f) + fminf(kSplitRisk * split_us(0, p, epi), quarters_us(p, epi));
    return t + split_us(cfg, p, epi);
}

// Whole tiles of two row counts in one launch.
static float estimate_pair_us(int cfg, int M1, int M2, int N, int K, int epi) {
    const TileCfg& c = kCfgs[cfg];
    const int tm = (M1 + c.BM - 1) / c.BM + (M2 + c.BM - 1) / c.BM, tn = (N + c.BN - 1) / c.BN;
    const int slots = device_cu_count() * c.slots_per_cu;
    const long full = (long)tm * tn / slots, rem = (long)tm * tn % slots;
    return kLaunchUs + full * (c.tile_us[epi] + K / 64 * slab_us(c, (float)slots, (float)tm, (float)tn)) +
           (rem ? c.tile_us[epi] + K / 64 * slab_us(c, (float)rem, (float)tm, (float)tn) : 0.f);
}

int gemm_num_configs() { return kNumCfgs; }

// The rotating q/k/v epilogue works on tiles that hold whole heads and lie inside one of the
// q, k, v column sections.
static bool cfg_runs(const TileCfg& c, int epilogue, const RopeEpilogue* rope) {
    return epilogue != EPI_QKV_ROPE || (c.BN % rope->dh == 0 && rope->D % c.BN == 0);
}

bool gemm_config_runs(int cfg, int epilogue, const RopeEpilogue* rope) {
    return cfg >= 0 && cfg < kNumCfgs && (epilogue != EPI_QKV_ROPE || rope) &&
           cfg_runs(kCfgs[cfg], epilogue, rope);
}

// Fastest configuration for a shape by the prediction: whole rounds of its tiles, then the last partial round
// either as it is or cut (-1: none runs it; of equal ones the first, whole before cut).  Over those 200
// projections the configuration this picks is 1.2 % slower than the best one (a round-count model with one
// constant per configuration and a fixed threshold for the cut: 7.4 %).
// Runs on the host before every launch without a recorded choice: what cannot be faster than the best so far is
// left as soon as that shows, smallest tiles first (0.17 us for a small model's projections, 0.4 with every
// prediction worked out, on the same processor).
static int predict(int M, int N, int K, int epilogue, const RopeEpilogue* rope, int* split_pct, float* us) {
    int best = -1;
    *us = INFINITY;
    auto consider = [&](int i) {
        const TileCfg& c = kCfgs[i];
        if (!cfg_runs(c, epilogue, rope)) return;
        const int tiles_m = (M + c.BM - 1) / c.BM, tiles_n = (N + c.BN - 1) / c.BN, k_tiles = K / 64;
        const int slots = device_cu_count() * c.slots_per_cu;
        const long tiles = (long)tiles_m * tiles_n, full = tiles < slots ? 0 : tiles / slots;
        const int rem = (int)(tiles - full * slots);
        const float tm = (float)tiles_m, tn = (float)tiles_n, last = c.tile_us[epilogue];
        float t = kLaunchUs;
        if (full) t += (float)full * (last + k_tiles * slab_us(c, (float)slots, tm, tn));
        auto take = [&](float total, int pct) {
            if (total <= *us) {
                *us = total;
                best = i;
                *split_pct = pct;
            }
        };
        if (rem == 0) {
            take(t, 0);
            return;
        }
        const float slab = c.slab_us * c.alone;      // (no slab takes less)
        const float least = i == 4 ? t : t + last + (float)((long)rem * k_tiles / slots) * slab;   // (4: cut on others)
        if (c.can_split && least <= *us) take(cut_us(i, M, N, K, epilogue, t, full > 0), 101);
        if (t + last + k_tiles * slab <= *us) take(t + last + k_tiles * slab_us(c, (float)rem, tm, tn), 0);
    };
    for (int i = kFitted - 1; i >= 0; --i) consider(i);
    if (*us >= kFittedFromUs && K >= kFittedFromK)
        for (int i = kFitted; i < kAllCfgs; ++i) consider(i);
    return best;
}

int gemm_choice_by_size(int M, int N, int K, int epilogue, const RopeEpilogue* rope) {
    int split_pct = 0;
    float us = 0.f;
    return predict(M, N, K, epilogue, rope, &split_pct, &us);
}

// Whether the choice by size normalises the rows of a gate/up projection itself (rows shorter than the limit, and the
// tile that can is the one it takes).
bool gemm_norms_rows(int M, int N, int K, int epilogue) {
    return epilogue == EPI_SILU_MUL && K <= NORM_MAX_K && gemm_choice_by_size(M, N, K, epilogue, nullptr) == 8;
}

// force_cfg >= 0 picks that tile configuration and force_split_pct the K-split threshold
// (0 = never, 101 = whenever the last round is not full); force_cfg < 0, or a configuration
// that cannot run this epilogue, leaves the choice to the cost model.
int launch_gemm(const bf16_t* A, int lda, const bf16_t* W, int M, int N, int K, void* C, int ldc,
                const void* R, int ldr, int epilogue, float* partial, size_t partial_bytes,
                uint32_t* counters, int n_counters, int force_cfg, int force_split_pct,
                const RopeEpilogue* rope, hipStream_t st, const NormedRows* norm) {
    if (M <= 0 || N <= 0) return MVLA_OK;
    if (K < 64 || K % 64 != 0 || lda % 8 != 0 || (norm && !gemm_norms_rows(M, N, K, epilogue))) return MVLA_EUNSUPPORTED;
    if (epilogue == EPI_SILU_MUL && N % 64 != 0) return MVLA_EUNSUPPORTED;
    if (N % 8 != 0 || ldc % 8 != 0 || (R && ldr % 8 != 0)) return MVLA_EUNSUPPORTED;
    if (ldc > (1 << 20) || ldr > (1 << 20)) return MVLA_EUNSUPPORTED;   // (32-bit byte offsets inside a tile)
    if (epilogue == EPI_QKV_ROPE) {
        if (!rope || !rope->pos || !rope->rc || !rope->rs || rope->S <= 0 || rope->rope_len <= 0)
            return MVLA_EINVAL;
        if ((rope->dh != 64 && rope->dh != 128) || rope->D % rope->dh != 0) return MVLA_EUNSUPPORTED;
        // N = 3D: q, k, v; N = 2D: q and k; N = D: one of q, k alone (W points at its rows)
        if (N != 3 * rope->D && N != 2 * rope->D && N != rope->D) return MVLA_EINVAL;
        if ((N == 3 * rope->D) != (rope->vt != nullptr)) return MVLA_EINVAL;
        if (M % rope->S != 0 || rope->S_pad < rope->S || rope->S_pad % 8 != 0) return MVLA_EINVAL;
    }
    if (norm)    // (chosen by size: see gemm_norms_rows)
        return launch_cfg<64, 64, 64, 2, 2, 6, SMALL>(reinterpret_cast<const bf16_t*>(norm->x), -1, W, M, N, K, C, ldc,
                                                      norm->gain, 0, epilogue, 1, 0, partial, partial_bytes, counters,
                                                      n_counters, RopeEpilogue{}, st, PLAN_ALL, nullptr, norm->eps);
    int best = -1, split_pct = 0;
    if (force_cfg >= 0 && force_cfg < kNumCfgs && cfg_runs(kCfgs[force_cfg], epilogue, rope)) {
        best = force_cfg;
        split_pct = force_split_pct;
    } else {
        float us = 0.f;
        best = predict(M, N, K, epilogue, rope, &split_pct, &us);
        if (best < 0) return MVLA_EUNSUPPORTED;
    }
    const RopeEpilogue rope_args = rope ? *rope : RopeEpilogue{};
#define MVLA_ARGS A, lda, W, M, N, K, C, ldc, R, ldr, epilogue, kCfgs[best].slots_per_cu, split_pct, \
                  partial, partial_bytes, counters, n_counters, rope_args, st
    switch (best) {
        case 0: return launch_cfg<256, 256, 64, 2, 4, 2>(MVLA_ARGS);
        case 1: return launch_cfg<256, 128, 64, 4, 2, 3>(MVLA_ARGS);
        case 2: return launch_cfg<128, 128, 64, 2, 2, 2>(MVLA_ARGS);
        case 3: return launch_cfg<128, 128, 64, 4, 2, 3>(MVLA_ARGS);
        case 4: {
            // (the persistent kernel addresses V^T with 32-bit offsets from a tile's first sample: at most
            // 256 / S + 2 samples of D * S_pad values; beyond that the eight-wave kernel takes the call)
            if (epilogue == EPI_QKV_ROPE && N == 3 * rope->D &&
                (size_t)(256 / rope->S + 2) * rope->D * rope->S_pad * 2 >= (size_t)OOB_OFFSET - 65536)
                return launch_cfg<256, 256, 64, 2, 4, 2>(MVLA_ARGS);
            // four waves of 128x128 have no registers for the K-split exchange: when the last round is to be
            // cut, its tiles go to the eight-wave kernel of the same tile size in a second launch (same
            // plan, same tile numbering), or in quarters to the 128x128 kernel where that is predicted
            // to be faster: nothing is exchanged then (K = 4096: 64 tiles 66 -> 45 us, 48 tiles 71 -> 35 us)
            const GemmPlan pl = plan_for(M, N, K, 256, 256, 64, device_cu_count(), split_pct,
                                         partial_bytes, n_counters);
            if (pl.sk_blocks == 0) return launch_cfg<256, 256, 64, 2, 2, 2>(MVLA_ARGS);
            const int rc = launch_cfg<256, 256, 64, 2, 2, 2>(MVLA_ARGS, PLAN_WHOLE_TILES);
            if (rc) return rc;
            // (the quarter tiles hold whole heads only of 128 and, as every tile, lie in one q, k, v section)
            if (cfg_runs(kCfgs[3], epilogue, rope) && quarters_us(pl, epilogue) < kSplitRisk * split_us(0, pl, epilogue))
                return launch_cfg<128, 128, 64, 4, 2, 3>(MVLA_ARGS, PLAN_QUARTERS);
            return launch_cfg<256, 256, 64, 2, 4, 2>(MVLA_ARGS, PLAN_SPLIT_TILES);
        }
        case 5: return launch_cfg<192, 128, 64, 2, 4, 3>(MVLA_ARGS);
        case 6: return launch_cfg<288, 192, 64, 2, 2, 2>(MVLA_ARGS);
        case 7: return launch_cfg<128, 192, 64, 2, 2, 3, SMALL>(MVLA_ARGS);
        case 8: return launch_cfg<64, 64, 64, 2, 2, 6, SMALL>(MVLA_ARGS);
        case 9: return launch_cfg<128, 128, 64, 2, 2, 4, SMALL>(MVLA_ARGS);
        case 10: return launch_cfg<64, 128, 64, 2, 2, 5, SMALL>(MVLA_ARGS);
        case 11: return launch_cfg<128, 64, 64, 2, 2, 5, SMALL>(MVLA_ARGS);
        case 12: return launch_cfg<160, 128, 64, 2, 2, 4, FITTED>(MVLA_ARGS);
        case 13: return launch_cfg<192, 128, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 14: return launch_cfg<160, 192, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 15: return launch_cfg<256, 128, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 16: return launch_cfg<128, 256, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 17: return launch_cfg<192, 192, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 18: return launch_cfg<160, 256, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 19: return launch_cfg<224, 192, 64, 2, 2, 3, FITTED>(MVLA_ARGS);
        case 20: return launch_cfg<192, 256, 64, 2, 2, 2, FITTED>(MVLA_ARGS);
        case 21: return launch_cfg<288, 192, 64, 2, 2, 2, FITTED>(MVLA_ARGS);
        case 22: return launch_cfg<224, 256, 64, 2, 2, 2, FITTED>(MVLA_ARGS);
        case 23: return launch_cfg<320, 192, 64, 2, 2, 2, FITTED>(MVLA_ARGS);
        default: return MVLA_EINVAL;
    }
#undef MVLA_ARGS
}

int rope_pair_config(int M1, const RopeEpilogue& rope1, int M2, const RopeEpilogue& rope2, int D) {
    // what launch_gemm would refuse is left to it
    if (M1 <= 0 || M2 <= 0 || D < 64 || D % 64 != 0 || D > (1 << 20)) return -1;
    for (const RopeEpilogue* r : {&rope1, &rope2})
        if (!r->pos || !r->rc || !r->rs || r->vt || r->rope_len <= 0 || r->D != D || (r->dh != 64 && r->dh != 128))
            return -1;
    if (rope1.dh != rope2.dh || D % rope1.dh != 0 || rope1.rope_len != rope2.rope_len) return -1;
    int split = 0, best = -1;
    float t1 = 0.f, t2 = 0.f, best_us = 0.f;
    if (predict(M1, D, D, EPI_QKV_ROPE, &rope1, &split, &t1) < 0 ||
        predict(M2, D, D, EPI_QKV_ROPE, &rope2, &split, &t2) < 0)
        return -1;
    // (the larger ones are for shapes that fill the chip by themselves; 128x128 on eight waves is never the fastest)
    for (int i : {1, 5, 8, 9, 10, 11}) {
        if (!cfg_runs(kCfgs[i], EPI_QKV_ROPE, &rope1)) continue;
        const float t = estimate_pair_us(i, M1, M2, D, D, EPI_QKV_ROPE);
        if (best < 0 || t < best_us) {
            best_us = t;
            best = i;
        }
    }
    return best_us < t1 + t2 ? best : -1;
}

int launch_rope_pair(int cfg, const bf16_t* A1, const bf16_t* W1, int M1, void* C1, const RopeEpilogue& rope1,
                     const bf16_t* A2, const bf16_t* W2, int M2, void* C2, const RopeEpilogue& rope2, int D,
                     hipStream_t st) {
    const PairedGemm second = {A2, W2, C2, rope2.pos, M2, 0, 0};
#define MVLA_PAIR(BM, BN, WM, WN, NS, KIND)                                                        \
    launch_cfg<BM, BN, 64, WM, WN, NS, KIND>(A1, D, W1, M1, D, D, C1, D, nullptr, 0, EPI_QKV_ROPE, 1, 0, nullptr, 0, \
                                              nullptr, 0, rope1, st, PLAN_ALL, &second)
    switch (cfg) {
        case 1: return MVLA_PAIR(256, 128, 4, 2, 3, SPLITTING);
        case 5: return MVLA_PAIR(192, 128, 2, 4, 3, SPLITTING);
        case 8: return MVLA_PAIR(64, 64, 2, 2, 6, SMALL);
        case 9: return MVLA_PAIR(128, 128, 2, 2, 4, SMALL);
        case 10: return MVLA_PAIR(64, 128, 2, 2, 5, SMALL);
        case 11: return MVLA_PAIR(128, 64, 2, 2, 5, SMALL);
        default: return MVLA_EINVAL;
    }
#undef MVLA_PAIR
}

}  // namespace mvla
