// Causal flash attention on the gfx950 matrix cores.
//
// Both products are computed transposed so that a lane owns one query:
//   S^T = K * Q^T   (MFMA rows = keys, columns = queries)
//   O^T = V^T * P^T (MFMA rows = head-dim, columns = queries)
// The S^T accumulator layout (lane = query column, registers = key rows) is
// exactly the B-operand layout P^T needs when the K rows are laid down in LDS
// with the two middle runs of four keys of every 16 swapped (att_key): a lane's
// eight probabilities of a step are then eight consecutive keys, one 16-byte
// V^T fragment, and go from one product to the next without leaving registers.
// Softmax statistics are
// per-lane scalars; the two lanes that share a query exchange one value per
// tile.  K tiles [64 keys x dh] and V^T tiles [dh x 64 keys] travel from global
// memory straight into a ring of LDS stages (global_load_lds, 16 bytes per
// lane; the XOR swizzle is applied on the global side because a direct load
// always lands a wave on 1 KiB of consecutive LDS), so the next tiles are in
// flight while the current one is consumed.  V^T is produced by the rotary
// kernel, which makes both tiles contiguous along the contraction axis of
// their product.
#include "common.h"
#include "mfma.h"

namespace mvla {

constexpr int ATT_THREADS = 256;
constexpr int ATT_QT = 128;  // queries per workgroup (32 per wave)
constexpr int ATT_KT = 64;   // keys per tile

// untracked direct global -> LDS copy (see gemm.hip): order consumers behind att_wait_vm + barrier
// (address = wave-uniform base + per-lane unsigned 32-bit byte offset)
__device__ __forceinline__ void att_dma16(const void* base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr),
                 "v"(off), "s"(base)
                 : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void att_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// K rows are dh/8 chunks long (16 or 8), V^T rows 8 chunks; conflict-free XOR patterns
template <int CPR>
__device__ __forceinline__ int att_swz(int row) {
    return CPR == 16 ? (row & 15) : ((row >> 1) & 7);
}

// Key of a tile that LDS row r holds: bits 2 and 3 swapped.  (In key order a lane needs two 8-byte pieces of two
// V^T chunks, 32 reads a tile with two lanes on every bank; 16 whole chunks instead take the LDS's busy cycles from
// 46 to 31 million at B = 16, S = 1344, 383 -> 366 us, and 1161 -> 1109 us at S = 2624.)
__device__ __forceinline__ int att_key(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

template <int DH, int NS>
__global__ __launch_bounds__(ATT_THREADS, 2) void attention_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, int ld, const bf16_t* __restrict__ vt,
    int S_pad, int S, int H, float scale_log2e, bf16_t* __restrict__ out, int ldo) {
    constexpr int CPR = DH / 8;           // 16-byte chunks per K row
    constexpr int STEPS = DH / 16;        // MFMA k-steps over the head dim
    constexpr int DB = DH / 32;           // 32-row blocks of O^T
    constexpr int K_SLOTS = ATT_KT * CPR, V_SLOTS = DH * 8, STAGE = K_SLOTS + V_SLOTS;
    constexpr int K_LD = K_SLOTS / ATT_THREADS, V_LD = V_SLOTS / ATT_THREADS;
    constexpr int P = K_LD + V_LD;        // direct loads per thread per tile

    extern __shared__ uint4 lds[];

    // Workgroups are dispatched in blockIdx order, x fastest.  Heads run along x and query tiles
    // along y, heavier (later) tiles first: a sample's tiles then start in order of decreasing
    // work across all its heads (the light ones fill the end instead of a heavy tile of the last
    // head starting late), and because the head count is a multiple of the 8 XCDs that workgroup
    // ids are dealt to, every tile of a head runs on the same XCD and finds its K/V in that L2.
    const int qtile = gridDim.y - 1 - blockIdx.y, h = blockIdx.x, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 31, fg = lane >> 5;
    const int q0 = qtile * ATT_QT;
    const int qw0 = q0 + wave * 32;           // first query of this wave
    const int my_q = qw0 + fr;                // this lane's query (sequence row)

    // B operand of S^T: this lane's query row
    uint4 qf[STEPS];
    {
        const bf16_t* src = q + ((size_t)b * S + min(my_q, S - 1)) * ld + h * DH + fg * 8;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = *reinterpret_cast<const uint4*>(src + st * 16);
        // The fragments are pinned here, before any direct load is in flight: otherwise the
        // compiler's waits for these loads sit inside the key loop, where they would also wait
        // for the (untracked) direct loads of the next tile.
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
            asm volatile("" : "+v"(qf[st].x), "+v"(qf[st].y), "+v"(qf[st].z), "+v"(qf[st].w));
    }

    const int last_row = min(q0 + ATT_QT, S) - 1;
    const int n_kt = last_row / ATT_KT + 1;   // key tiles this workgroup needs (causal)

    // direct-load mapping: op i of this thread covers slot i*256 + tid of the K (or V^T) tile
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
    // (bases are wave-uniform, the per-lane parts 32-bit byte offsets within one sample's keys
    // or one head's V^T: fewer address registers than one pointer per op)
    const bf16_t* k_base = k + (size_t)b * S * ld + h * DH;
    const bf16_t* v_base = vt + (size_t)(b * H + h) * DH * S_pad;
    uint32_t k_off[K_LD], k_lds[K_LD];
    const uint32_t k_pitch = (uint32_t)ld * 2u;
#pragma unroll
    for (int i = 0; i < K_LD; ++i) {
        const int sl = i * ATT_THREADS + tid, row = sl / CPR, ch = (sl % CPR) ^ att_swz<CPR>(row);
        k_off[i] = (uint32_t)att_key(row) * k_pitch + (uint32_t)ch * 16u;
        k_lds[i] = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)(i * ATT_THREADS + wave * 64) * 16u);
    }
    uint32_t v_off[V_LD], v_lds[V_LD];
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
        const int sl = i * ATT_THREADS + tid, row = sl >> 3, ch = (sl & 7) ^ att_swz<8>(row);
        v_off[i] = ((uint32_t)row * (uint32_t)S_pad + (uint32_t)ch * 8u) * 2u;
        v_lds[i] = __builtin_amdgcn_readfirstlane(
            lds_base + (uint32_t)(K_SLOTS + i * ATT_THREADS + wave * 64) * 16u);
    }
    // (a key beyond the sequence: the last 16 bytes of its last row instead, which the mask leaves out)
#define ATT_ISSUE(KT, STG)                                                                  \
    {                                                                                       \
        const int kt_ = min((KT), n_kt - 1);                                                \
        const uint32_t soff = (uint32_t)(STG) * STAGE * 16u;                                \
        const size_t k_tile = (size_t)(kt_ * ATT_KT) * k_pitch;                             \
        const uint32_t k_last = (uint32_t)(S - 1 - kt_ * ATT_KT) * k_pitch + (uint32_t)(DH - 8) * 2u; \
        _Pragma("unroll") for (int i = 0; i < K_LD; ++i)                                    \
            att_dma16(reinterpret_cast<const char*>(k_base) + k_tile, min(k_off[i], k_last), k_lds[i] + soff); \
        _Pragma("unroll") for (int i = 0; i < V_LD; ++i)                                    \
            att_dma16(v_base + kt_ * ATT_KT, v_off[i], v_lds[i] + soff);                    \
    }

    f32x16_t o_acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) o_acc[d][v] = 0.f;
    float run_m = -INFINITY, run_l = 0.f;   // run_l: this lane's share of the row sum

#pragma unroll
    for (int s = 0; s < NS - 1; ++s) ATT_ISSUE(s, s)

    int stage = 0;
    for (int kt = 0; kt < n_kt; ++kt) {
        // tile kt has landed for every wave; the stage of tile kt-1 is free for tile kt+NS-1
        att_wait_vm<(NS - 2) * P>();
        __syncthreads();
        {
            int nstage = stage + NS - 1;
            if (nstage >= NS) nstage -= NS;
            ATT_ISSUE(kt + NS - 1, nstage)
        }
        const int key0 = kt * ATT_KT;
        // a wave whose queries all precede this tile has nothing to add
        if (key0 <= qw0 + 31 && qw0 < S) {
            const uint4* Kc = lds + stage * STAGE;
            const uint4* Vc = Kc + K_SLOTS;
            // ---- S^T for the two 32-key halves of the tile
            // (the two independent accumulator chains alternate, so the matrix core does not
            // wait on its own results)
            f32x16_t s_acc[2];
            uint4 kf[2][STEPS];
#pragma unroll
            for (int st = 0; st < STEPS; ++st)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int row = t * 32 + fr;
                    kf[t][st] = Kc[row * CPR + ((st * 2 + fg) ^ att_swz<CPR>(row))];
                }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) s_acc[t][v] = 0.f;
#pragma unroll
            for (int st = 0; st < STEPS; ++st)
#pragma unroll
                for (int t = 0; t < 2; ++t) s_acc[t] = mfma32(kf[t][st], qf[st], s_acc[t]);
            // V^T fragments of the first two head-dim blocks: in flight during the softmax arithmetic
            uint4 vfrag[2][4];
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int row = min(d, DB - 1) * 32 + fr;
                const int sw = att_swz<8>(row);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) vfrag[d][ks] = Vc[row * 8 + ((ks * 2 + fg) ^ sw)];
            }
            // ---- (mask,) row max on the raw logits; only tiles that reach the diagonal or the end
            // of the sequence need the mask (wave-uniform test).  The softmax scale is positive, so
            // the max commutes with it, and scale and subtraction fuse into one FMA per logit (the
            // kernel is bound by vector-ALU issue, not by the matrix core).
            float tile_m = -INFINITY;
            if (key0 + ATT_KT - 1 <= qw0 && key0 + ATT_KT <= S) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) tile_m = fmaxf(tile_m, s_acc[t][v]);
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int key = key0 + t * 32 + 16 * (v >> 3) + 8 * fg + (v & 7);   // att_key of the row
                        const float x = (key <= my_q && key < S) ? s_acc[t][v] : -INFINITY;
                        s_acc[t][v] = x;
                        tile_m = fmaxf(tile_m, x);
                    }
            }
            tile_m = fmaxf(tile_m, __shfl_xor(tile_m, 32));
            const float new_m = fmaxf(run_m, tile_m);   // (raw logits) finite from the first tile on (key 0)
            const float neg_m = -new_m * scale_log2e;
            float psum = 0.f;
            uint4 pf[4];  // P^T B-operand fragments: one per 16-key step
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    float e[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        e[i] = __builtin_amdgcn_exp2f(fmaf(s_acc[t][hh * 8 + i], scale_log2e, neg_m));
                        psum += e[i];
                    }
                    pf[t * 2 + hh] = make_uint4(pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]),
                                                pack_bf16x2(e[4], e[5]), pack_bf16x2(e[6], e[7]));
                }
            // rescale only when the running max moved for some query of the wave (a factor of exactly 1 otherwise)
            if (__any(new_m != run_m)) {
                const float corr = __builtin_amdgcn_exp2f((run_m - new_m) * scale_log2e);
                run_l *= corr;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o_acc[d][v] *= corr;
                run_m = new_m;
            }
            run_l += psum;
            // ---- O^T += V^T * P^T ; the A fragment takes keys 8g..8g+7 of each 16-key step,
            // matching the key order of the P^T registers (see att_key).  The fragments of a pair
            // of head-dim blocks are read ahead of their MFMAs (the first pair before the softmax
            // arithmetic above, see vfrag), so the matrix core does not wait on LDS latency.
#pragma unroll
            for (int dp = 0; dp < DB; dp += 2) {
                uint4 vnext[2][4];
                if (dp + 2 < DB) {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const int row = (dp + 2 + d) * 32 + fr;
                        const int sw = att_swz<8>(row);
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) vnext[d][ks] = Vc[row * 8 + ((ks * 2 + fg) ^ sw)];
                    }
                }
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int d = 0; d < 2; ++d)
                        if (dp + d < DB) o_acc[dp + d] = mfma32(vfrag[d][ks], pf[ks], o_acc[dp + d]);
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) vfrag[d][ks] = vnext[d][ks];
            }
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    att_wait_vm<0>();
#undef ATT_ISSUE

    // ---- normalise and store: lane holds query my_q, rows = head-dim
    const float tot = run_l + __shfl_xor(run_l, 32);
    if (my_q < S) {
        const float inv = 1.0f / tot;
        bf16_t* orow = out + ((size_t)b * S + my_q) * ldo + h * DH;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const int col = d * 32 + 8 * v4 + 4 * fg;
                uint2 w;
                w.x = pack_bf16x2(o_acc[d][v4 * 4 + 0] * inv, o_acc[d][v4 * 4 + 1] * inv);
                w.y = pack_bf16x2(o_acc[d][v4 * 4 + 2] * inv, o_acc[d][v4 * 4 + 3] * inv);
                *reinterpret_cast<uint2*>(orow + col) = w;
            }
    }
}

// The same product for grids that leave the chip idle: one workgroup per 32 queries, whose waves deal the key
// tiles (32 keys each) out among themselves and add up their parts at the end.
//
// Such a launch is bound by its longest chain of dependent tiles, not by any rate: in the kernel above a wave
// walks every 64-key tile up to its queries (0.9 us each).  Here a wave takes one of NW 32-key tiles.  Every
// wave stages its own tiles in its own part of LDS, so nothing in the loop waits for another wave; one stage is
// enough, because the next K tile is asked for as soon as the fragments of this one are in registers (behind
// the softmax and O^T), and the next V^T tile the same (behind the next S^T).  A wave's O^T takes the
// place of its tiles in LDS (16 KiB each at dh = 128), the waves add up the parts of all, in wave order, a share of
// the head dimension each.
// 32 heads of 128: S = 237 9.3 -> 6.6 us, S = 448 12.8 -> 9.8; 4 heads of 64: S = 144 5.1 -> 4.3,
// S = 1344 19.3 -> 9.6.  Once the chip is full it is the slower one (every 32 queries fetch their keys for
// themselves: B = 4, S = 544 28 against 38 us), see short_limit.  Eight waves: slower wherever a second round of
// workgroups is needed (128 KiB of LDS leave one per CU), 5-15 % faster only with few heads and S > 1000.
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 2) void short_attention_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, int ld, const bf16_t* __restrict__ vt,
    int S_pad, int S, int H, float scale_log2e, bf16_t* __restrict__ out, int ldo) {
    constexpr int CPR = DH / 8;            // 16-byte chunks per K row
    constexpr int STEPS = DH / 16;         // MFMA k-steps over the head dim
    constexpr int DB = DH / 32;            // 32-row blocks of O^T
    constexpr int KT = 32;                 // keys per tile
    constexpr int K_SLOTS = KT * CPR, V_SLOTS = DH * (KT / 8), STAGE = K_SLOTS + V_SLOTS;
    constexpr int K_LD = K_SLOTS / 64, V_LD = V_SLOTS / 64;   // direct loads per lane per tile
    constexpr int GROUPS = DB * 4;         // a lane's accumulators in fours
    static_assert(GROUPS % NW == 0 && GROUPS * 64 == STAGE, "");

    extern __shared__ uint4 lds[];
    __shared__ float sh_m[NW][32], sh_l[NW][32];

    // (heads along x, heavier query blocks first: as above)
    const int qblock = gridDim.y - 1 - blockIdx.y, h = blockIdx.x, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int fr = lane & 31, fg = lane >> 5;
    const int q0 = qblock * 32, my_q = q0 + fr;
    const int n_kt = qblock + 1;           // key tiles up to these queries; only the last needs the mask

    const bf16_t* k_base = k + (size_t)b * S * ld + h * DH;
    const bf16_t* v_base = vt + (size_t)(b * H + h) * DH * S_pad;
    const uint32_t lds_wave = (uint32_t)(uintptr_t)lds + (uint32_t)(wave * STAGE) * 16u;
    const uint32_t k_pitch = (uint32_t)ld * 2u;
    uint32_t k_off[K_LD], v_off[V_LD];
#pragma unroll
    for (int i = 0; i < K_LD; ++i) {
        const int sl = i * 64 + lane, row = sl / CPR, ch = (sl % CPR) ^ att_swz<CPR>(row);
        k_off[i] = (uint32_t)att_key(row) * k_pitch + (uint32_t)ch * 16u;
    }
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
        const int sl = i * 64 + lane, row = sl >> 2, ch = (sl & 3) ^ ((row >> 2) & 3);
        v_off[i] = ((uint32_t)row * (uint32_t)S_pad + (uint32_t)ch * 8u) * 2u;
    }
    // (a key beyond the sequence: the last 16 bytes of its last row instead, which the mask leaves out)
    auto issue_k = [&](int kt) __attribute__((always_inline)) {
        const char* base = reinterpret_cast<const char*>(k_base) + (size_t)(kt * KT) * k_pitch;
        const uint32_t k_last = (uint32_t)(S - 1 - kt * KT) * k_pitch + (uint32_t)(DH - 8) * 2u;
#pragma unroll
        for (int i = 0; i < K_LD; ++i) att_dma16(base, min(k_off[i], k_last), lds_wave + (uint32_t)(i * 64) * 16u);
    };
    auto issue_v = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < V_LD; ++i)
            att_dma16(v_base + kt * KT, v_off[i], lds_wave + (uint32_t)(K_SLOTS + i * 64) * 16u);
    };

    if (wave < n_kt) {
        issue_k(wave);
        issue_v(wave);
    }
    // B operand of S^T: this lane's query row, one memory round trip with the first tiles (pinned: the compiler's
    // wait for it stands here and not in the loop)
    uint4 qf[STEPS];
    {
        const bf16_t* src = q + ((size_t)b * S + min(my_q, S - 1)) * ld + h * DH + fg * 8;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = *reinterpret_cast<const uint4*>(src + st * 16);
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
            asm volatile("" : "+v"(qf[st].x), "+v"(qf[st].y), "+v"(qf[st].z), "+v"(qf[st].w));
    }

    f32x16_t o_acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) o_acc[d][v] = 0.f;
    float run_m = -INFINITY, run_l = 0.f;   // run_l: this lane's share of the row sum

    const uint4* Kc = lds + wave * STAGE;
    const uint4* Vc = Kc + K_SLOTS;
    for (int kt = wave; kt < n_kt; kt += NW) {
        const bool more = kt + NW < n_kt;
        att_wait_vm<V_LD>();               // K landed (V^T of the tile behind it)
        uint4 kf[STEPS];
#pragma unroll
        for (int st = 0; st < STEPS; ++st) kf[st] = Kc[fr * CPR + ((st * 2 + fg) ^ att_swz<CPR>(fr))];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read: its place is free
        if (more) issue_k(kt + NW);
        f32x16_t s_acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) s_acc[v] = 0.f;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) s_acc = mfma32(kf[st], qf[st], s_acc);
        if (more) att_wait_vm<K_LD>();     // V^T landed (the next K behind it)
        else att_wait_vm<0>();
        uint4 vf[DB][2];
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            const int row = d * 32 + fr;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) vf[d][ks] = Vc[row * 4 + ((ks * 2 + fg) ^ ((row >> 2) & 3))];
        }
        // ---- softmax of the tile against the wave's own running maximum
        float tile_m = -INFINITY;
        if (kt == n_kt - 1) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = kt * KT + 16 * (v >> 3) + 8 * fg + (v & 7);   // att_key of the row
                s_acc[v] = (key <= my_q && key < S) ? s_acc[v] : -INFINITY;
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) tile_m = fmaxf(tile_m, s_acc[v]);
        tile_m = fmaxf(tile_m, __shfl_xor(tile_m, 32));
        const float new_m = fmaxf(run_m, tile_m);
        // (a wave's tiles may hold nothing but logits of -inf, where another wave's do not: they weigh 0)
        const float neg_m = new_m == -INFINITY ? 0.f : -new_m * scale_log2e;
        float psum = 0.f;
        uint4 pf[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            float e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                e[i] = __builtin_amdgcn_exp2f(fmaf(s_acc[hh * 8 + i], scale_log2e, neg_m));
                psum += e[i];
            }
            pf[hh] = make_uint4(pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]), pack_bf16x2(e[4], e[5]),
                                pack_bf16x2(e[6], e[7]));
        }
        if (__any(new_m != run_m)) {
            const float corr = new_m == run_m ? 1.f : __builtin_amdgcn_exp2f((run_m - new_m) * scale_log2e);
            run_l *= corr;
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) o_acc[d][v] *= corr;
            run_m = new_m;
        }
        run_l += psum;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // V^T read: its place is free
        if (more) issue_v(kt + NW);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int d = 0; d < DB; ++d) o_acc[d] = mfma32(vf[d][ks], pf[ks], o_acc[d]);
    }

    // ---- parts of all waves: O^T in fours per lane, one after the other, maximum and sum per query
    // (a wave's tiles have all been read, and no load is in flight)
    run_l += __shfl_xor(run_l, 32);
    float4* part = reinterpret_cast<float4*>(lds);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        part[wave * STAGE + g * 64 + lane] =
            make_float4(o_acc[g >> 2][(g & 3) * 4], o_acc[g >> 2][(g & 3) * 4 + 1], o_acc[g >> 2][(g & 3) * 4 + 2],
                        o_acc[g >> 2][(g & 3) * 4 + 3]);
    if (fg == 0) {
        sh_m[wave][fr] = run_m;
        sh_l[wave][fr] = run_l;
    }
    __syncthreads();
    float top = sh_m[0][fr];
#pragma unroll
    for (int w = 1; w < NW; ++w) top = fmaxf(top, sh_m[w][fr]);
    float f[NW], tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float m = sh_m[w][fr];
        f[w] = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - top) * scale_log2e);
        tot += sh_l[w][fr] * f[w];
    }
    if (my_q < S) {
        const float inv = 1.0f / tot;
        bf16_t* orow = out + ((size_t)b * S + my_q) * ldo + h * DH;
#pragma unroll
        for (int j = 0; j < GROUPS / NW; ++j) {
            const int g = wave * (GROUPS / NW) + j;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float4 t = part[w * STAGE + g * 64 + lane];
                a.x = fmaf(t.x, f[w], a.x);
                a.y = fmaf(t.y, f[w], a.y);
                a.z = fmaf(t.z, f[w], a.z);
                a.w = fmaf(t.w, f[w], a.w);
            }
            uint2 o;
            o.x = pack_bf16x2(a.x * inv, a.y * inv);
            o.y = pack_bf16x2(a.z * inv, a.w * inv);
            *reinterpret_cast<uint2*>(orow + (g >> 2) * 32 + 8 * (g & 3) + 4 * fg) = o;
        }
    }
}

template <typename Kernel>
static int start_attention(Kernel kern, bool* lds_set, dim3 grid, int threads, size_t lds, const bf16_t* q,
                           const bf16_t* k, int ldqkv, const bf16_t* vt, int S_pad, int S, int H, int dh, bf16_t* out,
                           int ldo, hipStream_t st) {
    int dev = 0;   // (the dynamic-LDS limit is raised once per device)
    MVLA_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices || !lds_set[dev]) {
        MVLA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        if (dev >= 0 && dev < kMaxDevices) lds_set[dev] = true;
    }
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)dh);
    hipLaunchKernelGGL(kern, grid, dim3(threads), lds, st, q, k, ldqkv, vt, S_pad, S, H, scale_log2e, out, ldo);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

template <int DH, int NS>
static int launch_att(const bf16_t* q, const bf16_t* k, int ldqkv, const bf16_t* vt, int S_pad,
                      int B, int S, int H, bf16_t* out, int ldo, hipStream_t st) {
    static bool lds_set[kMaxDevices] = {};
    const size_t lds = (size_t)NS * (ATT_KT * (DH / 8) + DH * 8) * sizeof(uint4);
    return start_attention(attention_kernel<DH, NS>, lds_set, dim3(H, (S + ATT_QT - 1) / ATT_QT, B), ATT_THREADS, lds,
                           q, k, ldqkv, vt, S_pad, S, H, DH, out, ldo, st);
}

template <int DH, int NW>
static int launch_short(const bf16_t* q, const bf16_t* k, int ldqkv, const bf16_t* vt, int S_pad,
                        int B, int S, int H, bf16_t* out, int ldo, hipStream_t st) {
    static bool lds_set[kMaxDevices] = {};
    const size_t lds = (size_t)NW * (32 * (DH / 8) + DH * 4) * sizeof(uint4);
    return start_attention(short_attention_kernel<DH, NW>, lds_set, dim3(H, (S + 31) / 32, B), NW * 64, lds, q, k,
                           ldqkv, vt, S_pad, S, H, DH, out, ldo, st);
}

// Workgroups of 32 queries up to which short_attention_kernel is the faster one (us, long chain / short chains): one per
// compute unit for a few tiles (S = 80: 240 6.3 / 5.5, 288 6.4 / 6.9; up to 64 keys there is no chain to cut, 5.0 / 5.2),
// from four long tiles on what is resident at once, two per compute unit at dh = 128 (S = 237: 512 9.7 / 9.1, 640
// 10.1 / 11.6) and, once the chain is long, four at dh = 64, whose workgroups take half the LDS (S = 900: 928 15.3 / 12.9;
// S = 448: 512 8.6 / 7.0, 896 9.0 / 9.4).
// Longer chains pay for a partial third round of short ones too, while it is made of the ends of a sample: a
// sample's tiles go out longest first, the samples one after the other, so few samples end in short tiles and many
// in the long tiles of the last ones.  dh = 128, within 32 workgroups a tile of keys (32 heads of one sample, at any length):
//   up to 3 samples up to 1024: 32 heads S = 545 576 14.9 / 13.7, S = 600 608 16.6 / 14.1, S = 705 736 18.8 / 17.4, S = 1000 1024
//     24.9 / 23.2, S = 1200 1216 29.5 / 31.3 (16 heads of 3 samples, 48 a tile: S = 700 1056 20.0 / 21.2)
//   up to 7 up to 700: 6 samples S = 880 672 22.1 / 20.0; 7 samples S = 760 672 19.9 / 19.8, S = 900 812 22.5 / 24.0; 4 samples
//     S = 760 768 19.8 / 20.4
//   up to 16 up to 544: 16 samples S = 528 544 15.3 / 14.7, S = 620 640 17.5 / 18.1; 8 samples S = 704 704 18.2 / 19.0
//   more up to what is resident: 32 samples S = 512 512 15.0 / 15.0, S = 560 576 15.7 / 18.2
// and from S = 1400 on 912 of up to 8 samples (S = 1800, 4 samples 39.3 / 39.2; 5 samples S = 1600 1000 36.6 / 36.8), 704 of
// more (S = 1400, 16 samples 704 32.0 / 29.3, 20 samples 880 32.7 / 34.5).  dh = 64 from S = 640 on: 1280 (8 samples S = 640
// 14.4 / 13.4, S = 704 1408 14.9 / 15.2; 16 samples S = 640 16.5 / 15.2) unless the samples are many (28 of them S = 672 1176
// 14.8 / 16.1, 56 S = 640 1120 15.3 / 16.5).
// (The sums' order is no reason: attention outputs behind short chains are 0.96 to 0.99 times as far from their
// 64-bit values over 24 inputs of 544 to 1400 tokens.)
static int short_limit(int B, int S, int dh) {
    if (S <= ATT_KT) return 0;
    if (S <= 3 * ATT_KT) return 256;
    if (S < 512) return 512;
    if (dh == 64) return S < 640 || B > 24 ? 1024 : 1280;
    if (S >= 1400) return B <= 3 ? 1024 : B <= 8 ? 912 : 704;
    const int most = B <= 3 ? 1024 : B <= 7 ? 700 : B <= 16 ? 544 : 512, per_tile = 32 * ((S + 31) / 32);
    return per_tile < most ? per_tile : most;
}

int launch_attention(const bf16_t* q, const bf16_t* k, int ldqkv, const bf16_t* vt, int S_pad,
                     int B, int S, int H, int dh, bf16_t* out, int ldo, hipStream_t st) {
    if (B <= 0 || S <= 0) return MVLA_OK;
    if (S_pad % ATT_KT != 0 || S_pad < S) return MVLA_EINVAL;
    // per-lane byte offsets inside one sample's keys / one head's V^T are 32-bit (kept below 2^31)
    if ((size_t)S * ldqkv * 2 >= ((size_t)1 << 31) || (size_t)dh * S_pad * 2 >= ((size_t)1 << 31))
        return MVLA_EUNSUPPORTED;
    if ((size_t)B * H * ((S + 31) / 32) <= (size_t)short_limit(B, S, dh)) {
        if (dh == 128) return launch_short<128, 4>(q, k, ldqkv, vt, S_pad, B, S, H, out, ldo, st);
        if (dh == 64) return launch_short<64, 4>(q, k, ldqkv, vt, S_pad, B, S, H, out, ldo, st);
    }
    // two stages of 32 KiB each: two workgroups per CU, whose waves overlap softmax and MFMA
    if (dh == 128) return launch_att<128, 2>(q, k, ldqkv, vt, S_pad, B, S, H, out, ldo, st);
    if (dh == 64) return launch_att<64, 2>(q, k, ldqkv, vt, S_pad, B, S, H, out, ldo, st);
    return MVLA_EUNSUPPORTED;
}

}  // namespace mvla
