// Pruning-step kernels for gfx950: attention-column salience, modality budget,
// per-modality top-k selection, gather-compaction.  All are bandwidth- or
// latency-bound; none uses floating-point atomics, so every result is
// reproducible bit for bit.
#include "common.h"
#include "wave.h"
#include <type_traits>

namespace mvla {

// ---------------------------------------------------------------------------
// Salience (paper Sec. 3.2, Eq. 3): column sums of the language-query
// attention rows over the visual columns, divided by the number of rows.
//
// A wave is laid out as 4 row-groups x 16 lanes; a lane owns VEC consecutive
// columns, so one row-group reads 16*VEC consecutive floats of one row
// (coalesced 16-byte loads when VEC == 4).  Row-groups are folded with two
// wavefront shuffles, the block's four waves through LDS, and the blocks that
// share a column chunk through a partial buffer summed in fixed order by
// whichever of them arrives last (integer arrival counter, no float atomics).
// ---------------------------------------------------------------------------
// forward declarations of the per-sample steps that the fused kernel runs after the salience
struct FusedPrune {
    int n2, n3, n_text, k_total, min2, min3;
    int32_t* k2k3;
    int32_t* kept_idx;
    uint32_t* sample_counters;  // one arrival counter per sample (kept at zero between calls)
};
template <typename Load>
__device__ __forceinline__ void finish_sample(Load load, const FusedPrune& f, int b, uint32_t* keys);

constexpr int SAL_THREADS = 256;
constexpr int SEL_MAX_N = 16384;    // largest segment the selection takes
constexpr int SEL_FOUR_WAVES = 2048;  // longest segment that four waves select; beyond it sixteen
constexpr int SAL_LPR = 16;                        // lanes per row-group
// Attention tensors above this are read past the caches.  344 MB (B = 16, 32 heads x 64 queries x 2624
// columns): 57 us against 87 us with plain loads, which also push the layer output out that the gather
// reads next.  Below the Infinity Cache's 256 MB the next reader (the per-patch indicators) finds the
// tensor there: 8.9 MB read non-temporally made that pair 1.6 us slower.
constexpr size_t SAL_STREAM_BYTES = size_t(256) << 20;
constexpr int FIN_U = 8;            // columns a thread takes at a time when a sample is finished
constexpr long SAL_FEW = 96 * 1024;                // values up to which more splits pay (see salience_shape)
constexpr int SAL_GROUPS = SAL_THREADS / SAL_LPR;  // 16 row-groups per block

typedef float f32v4_t __attribute__((ext_vector_type(4)));

// read_once: non-temporal loads, for a tensor that is larger than the caches (SAL_STREAM_BYTES).
// FUSED: the workgroup that completes the last column chunk of a sample goes on to split the
// budget and select that sample's tokens (same arithmetic as budget_kernel / select_kernel).
template <int VEC, bool FUSED>
__global__ __launch_bounds__(SAL_THREADS) void salience_kernel(
    const float* __restrict__ attn, int R, int S, int n_vis, int rows_per_split, int n_split,
    float inv_rows, float* __restrict__ sal, float* __restrict__ partial,
    uint32_t* __restrict__ counters, int read_once, FusedPrune fused) {
    extern __shared__ uint32_t dyn_lds[];  // selection keys (fused variant only)
    constexpr int CW = SAL_LPR * VEC;  // columns per chunk
    const int chunk = blockIdx.x, split = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int lane16 = tid % SAL_LPR;
    const int group = tid / SAL_LPR;
    const int col0 = chunk * CW + lane16 * VEC;
    const int r_begin = split * rows_per_split;
    const int r_end = min(R, r_begin + rows_per_split);
    const float* base = attn + (size_t)b * R * S;

    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;

    if (VEC == 4) {
        if (col0 + 3 < n_vis) {
            // eight loads in flight per lane, the rows left over in batches of four, two and one (one by one,
            // every one of up to seven was a memory round trip)
            auto add_rows = [&](auto load) __attribute__((always_inline)) {
                int r = r_begin + group;
                auto batch = [&](auto rows) __attribute__((always_inline)) {
                    constexpr int U = decltype(rows)::value;
                    f32v4_t t[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) t[u] = load(base + (size_t)(r + u * SAL_GROUPS) * S + col0);
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[v] += t[u][v];
                    r += U * SAL_GROUPS;
                };
                while (r + 7 * SAL_GROUPS < r_end) batch(std::integral_constant<int, 8>{});
                if (r + 3 * SAL_GROUPS < r_end) batch(std::integral_constant<int, 4>{});
                if (r + SAL_GROUPS < r_end) batch(std::integral_constant<int, 2>{});
                if (r < r_end) batch(std::integral_constant<int, 1>{});
            };
            if (read_once)
                add_rows([](const float* p) { return __builtin_nontemporal_load(reinterpret_cast<const f32v4_t*>(p)); });
            else
                add_rows([](const float* p) { return *reinterpret_cast<const f32v4_t*>(p); });
        } else {
            for (int r = r_begin + group; r < r_end; r += SAL_GROUPS)
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (col0 + v < n_vis) acc[v] += base[(size_t)r * S + col0 + v];
        }
    } else {
        for (int r = r_begin + group; r < r_end; r += SAL_GROUPS)
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                if (col0 + v < n_vis) acc[v] += base[(size_t)r * S + col0 + v];
    }

    // fold the wave's 4 row-groups (lanes l, l^16, l^32, l^48 own the same columns)
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        acc[v] += __shfl_xor(acc[v], 16);
        acc[v] += __shfl_xor(acc[v], 32);
    }
    __shared__ float red[SAL_THREADS / 64][CW];
    __shared__ int is_last;
    const int wave = tid / 64, lane = tid % 64;
    if (lane < SAL_LPR) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) red[wave][lane * VEC + v] = acc[v];
    }
    __syncthreads();
    float tot = 0.f;
    const int c = chunk * CW + tid;
    if (tid < CW) {
#pragma unroll
        for (int w = 0; w < SAL_THREADS / 64; ++w) tot += red[w][tid];
    }
    // store of a finished salience value: plain, or agent-coherent when another workgroup
    // (maybe on another XCD) will read it in this same launch
    auto put = [&](float v) {
        if (FUSED)
            __hip_atomic_store(&sal[(size_t)b * n_vis + c], v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        else
            sal[(size_t)b * n_vis + c] = v;
    };
    if (n_split == 1) {
        if (tid < CW && c < n_vis) put(tot * inv_rows);
        if (!FUSED) return;
    } else {
        // several blocks share this column chunk: publish, last arrival finishes
        float* pslot = partial + ((size_t)(b * gridDim.x + chunk) * n_split) * CW;
        // partial sums cross CUs/XCDs through agent-coherent accesses (no cache-wide flushes)
        if (tid < CW)
            __hip_atomic_store(&pslot[(size_t)split * CW + tid], tot, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            uint32_t* ctr = counters + (b * gridDim.x + chunk);
            const uint32_t prev =
                __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = (prev == (uint32_t)(n_split - 1));
            if (is_last) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!is_last) return;
        if (tid < CW && c < n_vis) {
            // (eight in flight together; a last batch of fewer loads the last one again and leaves it out)
            float s = 0.f;
            int i = 0;
            auto part = [&](int j) __attribute__((always_inline)) {
                return __hip_atomic_load(&pslot[(size_t)j * CW + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            for (; i + 8 <= n_split; i += 8) {
                float t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t[u] = part(i + u);
#pragma unroll
                for (int u = 0; u < 8; ++u) s += t[u];
            }
            if (i < n_split) {
                float t[7];
#pragma unroll
                for (int u = 0; u < 7; ++u) t[u] = part(min(i + u, n_split - 1));
#pragma unroll
                for (int u = 0; u < 7; ++u)
                    if (i + u < n_split) s += t[u];
            }
            put(s * inv_rows);
        }
        if (!FUSED) return;
    }
    // ---- fused tail: this chunk of sample b is complete; the last chunk's workgroup finishes b
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(&fused.sample_counters[b], 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        is_last = (prev == gridDim.x - 1);
        if (is_last)
            __hip_atomic_store(&fused.sample_counters[b], 0u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!is_last) return;
    // (all loads of a batch in flight together: one by one, each waited a round trip to the level
    // of memory that all XCDs share)
    const float* sal_b = sal + (size_t)b * n_vis;
    finish_sample([&](const int (&col)[FIN_U], float (&v)[FIN_U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < FIN_U; ++u)
            v[u] = __hip_atomic_load(&sal_b[col[u]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }, fused, b, dyn_lds);
}

static void salience_shape(int B, int R, int n_vis, int vec, int* chunks, int* n_split,
                           int* rows_per_split) {
    const int cw = SAL_LPR * vec;
    *chunks = (n_vis + cw - 1) / cw;
    // Aim for ~2048 blocks, at least 8 passes of the 16 row-groups each (a thread's eight loads then fly
    // together, and the last block to arrive has fewer partial sums to fetch: 1024 rows x 512 columns
    // (B = 4) 14.4 -> 5.3 us against 2 passes); few rows are not split at all.
    long blocks = (long)B * *chunks;
    int split = (int)((2048 + blocks - 1) / blocks);
    int max_split = (R + 8 * SAL_GROUPS - 1) / (8 * SAL_GROUPS);
    // Where all of it is little, a compute unit's reads of its rows take longer than the exchange: down to two
    // passes in up to eight splits, whose partial sums are still one batch of loads (512 rows x 160 columns
    // 4.1 -> 3.7 us; 256 rows x 512 columns 3.7 with two splits, 3.8 with eight).
    if (max_split > 1 && (long)B * R * n_vis < SAL_FEW) max_split = max(max_split, min(8, R / (2 * SAL_GROUPS)));
    if (split > max_split) split = max_split;
    if (split < 1) split = 1;
    *rows_per_split = (R + split - 1) / split;
    *n_split = (R + *rows_per_split - 1) / *rows_per_split;
}

size_t salience_scratch_bytes(int B, int H, int Nq, int n_vis) {
    // worst case over VEC in {1,4}: chunks*CW <= n_vis + 63, n_split <= R/32 + 1
    const size_t R = (size_t)H * Nq;
    return align_up((size_t)B * (size_t)(n_vis + 64) * (R / (2 * SAL_GROUPS) + 2) * 4, 256);
}

// mean_rows: the row count the sums are divided by; 0 means the R = H*Nq rows read.  (When the
// rows are already sums over a tile of queries, the caller passes the original row count.)
static int launch_salience_any(const float* attn, int B, int H, int Nq, int S, int n_vis,
                               float* sal, float* partial, uint32_t* counters,
                               const FusedPrune* fused, int mean_rows, hipStream_t st) {
    const int R = H * Nq;
    const bool vec4 = (S % 4 == 0) && ((reinterpret_cast<uintptr_t>(attn) & 15) == 0);
    int chunks, n_split, rps;
    salience_shape(B, R, n_vis, vec4 ? 4 : 1, &chunks, &n_split, &rps);
    // counters: [0, B*chunks) chunk arrivals, then B sample arrivals (first half of the area)
    if ((long)B * chunks + B > kCounterWords / 2) return MVLA_EUNSUPPORTED;
    dim3 grid(chunks, n_split, B);
    const float inv_rows = 1.0f / (float)(mean_rows > 0 ? mean_rows : R);
    const int read_once = (size_t)B * R * S * 4 > SAL_STREAM_BYTES;
    FusedPrune f{};
    size_t lds = 0;
    if (fused) {
        f = *fused;
        f.sample_counters = counters + (size_t)B * chunks;
        lds = (size_t)max(f.n2 + f.n3, 1) * 4;   // selection keys of both segments
    }
    // (the fused variants keep the keys of both segments in LDS: up to 128 KiB, above the default
    // limit of a kernel, which is raised once per device)
#define MVLA_SAL(V, F)                                                                          \
    do {                                                                                        \
        auto kern = salience_kernel<V, F>;                                                      \
        if (F) {                                                                                \
            static bool lds_set[kMaxDevices] = {};                                              \
            int dev = 0;                                                                        \
            MVLA_HIP_CHECK(hipGetDevice(&dev));                                                 \
            if (dev < 0 || dev >= kMaxDevices || !lds_set[dev]) {                               \
                MVLA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),         \
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,  \
                                                   2 * SEL_MAX_N * 4));                         \
                if (dev >= 0 && dev < kMaxDevices) lds_set[dev] = true;                         \
            }                                                                                   \
        }                                                                                       \
        hipLaunchKernelGGL(kern, grid, dim3(SAL_THREADS), lds, st, attn, R, S, n_vis, rps,      \
                           n_split, inv_rows, sal, partial, counters, read_once, f);                       \
    } while (0)
    if (vec4) {
        if (fused) MVLA_SAL(4, true); else MVLA_SAL(4, false);
    } else {
        if (fused) MVLA_SAL(1, true); else MVLA_SAL(1, false);
    }
#undef MVLA_SAL
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

int launch_salience(const float* attn, int B, int H, int Nq, int S, int n_vis, float* sal,
                    float* partial, uint32_t* counters, int mean_rows, hipStream_t st) {
    return launch_salience_any(attn, B, H, Nq, S, n_vis, sal, partial, counters, nullptr, mean_rows,
                               st);
}

int launch_prune_fused(const float* attn, int B, int H, int Nq, int S, int n2, int n3, int n_text,
                       int k_total, int min2, int min3, float* sal, int32_t* k2k3,
                       int32_t* kept_idx, float* partial, uint32_t* counters, int mean_rows,
                       hipStream_t st) {
    FusedPrune f{n2, n3, n_text, k_total, min2, min3, k2k3, kept_idx, nullptr};
    return launch_salience_any(attn, B, H, Nq, S, n2 + n3, sal, partial, counters, &f, mean_rows,
                               st);
}

// ---------------------------------------------------------------------------
// Salience without a context or workspace, for callers that cannot allocate
// device memory (code under graph capture, serving loops): the row-split
// partial sums and the arrival counters live in a fixed array of this module.
// Every GPU holds its own copy of the array until the process ends.
// ---------------------------------------------------------------------------
constexpr size_t kStaticCounterBytes = size_t(kCounterWords / 2) * 4;   // 32 KiB of arrival counters
constexpr size_t kStaticPartialBytes = size_t(16) << 20;                // 16 MiB of partial sums
static __device__ __align__(256) unsigned char scratch[kStaticCounterBytes + kStaticPartialBytes];
// device address of `scratch` on each GPU (the array's name is only a host-side handle)
static void* g_scratch_addr[kMaxDevices] = {};

__global__ void clear_words_kernel(uint32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

}  // namespace mvla

extern "C" int mvla_salience_noalloc(void* hip_stream, const float* attn, int B, int H, int Nq, int S,
                                     int n_vis, float* sal) {
    using namespace mvla;
    if (!attn || !sal) return MVLA_EINVAL;
    if (B <= 0 || H <= 0 || Nq <= 0 || S <= 0 || n_vis <= 0 || n_vis > S) return MVLA_EINVAL;
    if ((reinterpret_cast<uintptr_t>(attn) & 3) || (reinterpret_cast<uintptr_t>(sal) & 3))
        return MVLA_EINVAL;
    // the fixed scratch bounds the shape: partial sums and one counter per (sample, column chunk)
    const bool vec4 = (S % 4 == 0) && ((reinterpret_cast<uintptr_t>(attn) & 15) == 0);
    int chunks, n_split, rps;
    salience_shape(B, H * Nq, n_vis, vec4 ? 4 : 1, &chunks, &n_split, &rps);
    const long n_counters = (long)B * chunks + B;
    if (salience_scratch_bytes(B, H, Nq, n_vis) > kStaticPartialBytes ||
        n_counters > (long)(kStaticCounterBytes / 4))
        return MVLA_ELIMIT;
    int dev = 0;
    MVLA_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return MVLA_EUNSUPPORTED;
    if (!g_scratch_addr[dev]) {   // once per device, with that device current
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MVLA_EHIP;
        g_scratch_addr[dev] = p;
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint32_t* counters = static_cast<uint32_t*>(g_scratch_addr[dev]);
    float* partial = reinterpret_cast<float*>(static_cast<char*>(g_scratch_addr[dev]) + kStaticCounterBytes);
    // the array keeps whatever the last call left: the counters this call uses start at zero
    // (a kernel, not a memset, so that the call can be recorded into a graph)
    hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)((n_counters + 255) / 256)), dim3(256), 0, st,
                       counters, (int)n_counters);
    MVLA_HIP_CHECK(hipGetLastError());
    return launch_salience(attn, B, H, Nq, S, n_vis, sal, partial, counters, 0, st);
}

namespace mvla {

// ---------------------------------------------------------------------------
// Modality budget (paper Eq. 5): fp64 masses per sample, integer split.
// ---------------------------------------------------------------------------
constexpr int BUD_THREADS = 256;

// Workgroup barrier for data that is exchanged through LDS only: it waits for this wave's LDS
// operations, not for its outstanding global stores.  (__syncthreads() waits for those too --
// a full write round trip whenever budget or index stores are in flight, several times per
// sample in the tail of the fused kernel.)
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// two sums over the workgroup, each a fixed-shape tree: over the wave, then the waves' partials in LDS
__device__ inline void block_sum2_f64(double& a, double& b, double* sh /*LDS [2 * waves]*/) {
    a = wave_sum_f64(a);
    b = wave_sum_f64(b);
    constexpr int NW = BUD_THREADS / 64;
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = a;
        sh[NW + (threadIdx.x >> 6)] = b;
    }
    lds_barrier();
    a = b = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        a += sh[w];
        b += sh[NW + w];
    }
}

__device__ inline void budget_split(double a2, double a3, int n2, int n3, int k_total, int min2,
                                    int min3, int* k2_out, double* m2_out) {
    const double tot = a2 + a3;
    const double m2 = tot > 0.0 ? a2 / tot : (double)n2 / (double)(n2 + n3);
    int k2 = (int)floor((double)k_total * m2 + 0.5);
    const int lo = max(min2, k_total - n3);
    const int hi = min(n2, k_total - min3);
    k2 = min(max(k2, lo), hi);
    *k2_out = k2;
    *m2_out = m2;
}

__global__ __launch_bounds__(BUD_THREADS) void budget_kernel(const float* __restrict__ sal, int n2,
                                                             int n3, int k_total, int min2,
                                                             int min3, int32_t* __restrict__ k2k3,
                                                             float* __restrict__ mass) {
    __shared__ double sh[2 * (BUD_THREADS / 64)];
    const int b = blockIdx.x;
    const float* s = sal + (size_t)b * (n2 + n3);
    double a2 = 0.0, a3 = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < n2; i += BUD_THREADS) a2 += (double)s[i];
#pragma unroll 8
    for (int i = threadIdx.x; i < n3; i += BUD_THREADS) a3 += (double)s[n2 + i];
    block_sum2_f64(a2, a3, sh);
    if (threadIdx.x == 0) {
        int k2;
        double m2;
        budget_split(a2, a3, n2, n3, k_total, min2, min3, &k2, &m2);
        k2k3[2 * b] = k2;
        k2k3[2 * b + 1] = k_total - k2;
        if (mass) {
            mass[2 * b] = (float)m2;
            mass[2 * b + 1] = (float)(1.0 - m2);
        }
    }
}

int launch_budget(const float* sal, int B, int n2, int n3, int k_total, int min2, int min3,
                  int32_t* k2k3, float* mass, hipStream_t st) {
    hipLaunchKernelGGL(budget_kernel, dim3(B), dim3(BUD_THREADS), 0, st, sal, n2, n3, k_total,
                       min2, min3, k2k3, mass);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Per-modality top-k.  The scores are held as order-preserving 32-bit keys; a
// group of waves works on one segment (one workgroup per segment in
// select_kernel, half a workgroup each in the tail of the fused kernel, both
// segments in step).  Exact search for the K-th largest key T: a 1024-bin
// histogram over [smallest, largest key] -- the keys of a segment share their
// top bits, so bins over the whole 32-bit range put nearly all of them on a few
// counters -- narrows the range to the bin that holds T; as soon as at most 64
// keys are left in it, one wave ranks those directly (at once for short
// segments), else the bin is split again (four times at most).  Tokens with
// key > T are kept, and of those with key == T the lowest-indexed ones.  Each
// wave owns a contiguous run of the indices and places its tokens 64 at a time
// by ballots behind the counts of the waves before it, so the output is in
// ascending index order without a sort.
//
// Bound by the chain of dependent LDS accesses and barriers, not by bytes.
// Against four 8-bit radix passes over the whole key range and one segment
// after the other: 16384 + 16384 tokens
// (B = 1) 52 -> 17 us, 768 + 1024 (B = 8) 7.8 -> 6.4; the fused step and its gather, 64 rows of two segments of
// 64 tokens, 13.1 -> 8.0.
// The kernel of its own keeps each thread's keys in registers (they were read from LDS five times, and laid
// down there first): calls of 1024 + 1024 (B = 8) 6.2 -> 4.9 us, 2048 + 2048 8.1 -> 6.6, 16384 + 16384 (B = 1)
// 16.7 -> 14.5.  In the fused tail half a workgroup takes a segment of up to 16384, and the keys stay in LDS.
// ---------------------------------------------------------------------------

__device__ inline uint32_t sal_key(float x) {
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;  // -0 ranks with +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// one step of a wave-wide combination: the value CTRL fetches for this lane, or `none`
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_get(uint32_t v, uint32_t none) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xf, false);
}
// inclusive prefix sum over the 64 lanes: row shifts by 1, 2, 4, 8, then row totals handed on
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v) {
    v += dpp_get<0x111, 0xf>(v, 0u);
    v += dpp_get<0x112, 0xf>(v, 0u);
    v += dpp_get<0x114, 0xf>(v, 0u);
    v += dpp_get<0x118, 0xf>(v, 0u);
    v += dpp_get<0x142, 0xa>(v, 0u);
    v += dpp_get<0x143, 0xc>(v, 0u);
    return v;
}
// maximum over the 64 lanes, in every lane
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = max(v, dpp_get<0x111, 0xf>(v, 0u));
    v = max(v, dpp_get<0x112, 0xf>(v, 0u));
    v = max(v, dpp_get<0x114, 0xf>(v, 0u));
    v = max(v, dpp_get<0x118, 0xf>(v, 0u));
    v = max(v, dpp_get<0x142, 0xa>(v, 0u));
    v = max(v, dpp_get<0x143, 0xc>(v, 0u));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

constexpr int SEL_BINS = 1024;
constexpr int SEL_CAND = 64;    // keys that one wave ranks directly

// LDS of NG groups of GW waves that select side by side
template <int GW, int NG>
struct SelShared {
    uint32_t hist[NG][SEL_BINS];
    uint32_t cand[NG][SEL_CAND];
    uint32_t wave[NG][GW][2];
    uint32_t found[NG][3];      // bin, rank within it, keys in it
    uint32_t n_cand[NG];
    uint32_t result[NG][2];     // T, how many keys equal to T are kept
    uint32_t open;              // groups whose threshold is not found yet
};

// Every thread of the workgroup calls this with its group's segment (group-uniform arguments;
// k <= 0 or n <= 0: nothing to do, but the barriers are taken part in; all_short: every group's n is
// at most 64, the same for the whole workgroup).  KPT == 0: the keys were written to LDS by this workgroup; the
// first barrier orders those writes before the reads.  KPT > 0: key(i) fetches one, and a thread keeps its up to KPT
// in registers throughout (those that it places, 64 apart).
template <int GW, int NG, int KPT = 0, typename Key = const uint32_t*>
__device__ __forceinline__ void select_groups(Key keys /*LDS [n], or a function of the index*/, int n, int k,
                                              int idx_offset, int32_t* __restrict__ out, bool all_short,
                                              SelShared<GW, NG>& sh) {
    constexpr int GT = GW * 64, BPT = SEL_BINS / GT;
    static_assert(SEL_BINS % GT == 0, "");
    const int wave_id = (int)threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = wave_id / GW, gw = wave_id % GW, gt = (int)threadIdx.x - g * GT;
    if (k > n) k = n;
    const bool work = k > 0;
    uint32_t lo = 0u, hi = ~0u, remaining = (uint32_t)max(k, 0);   // T has this rank (from the top) in [lo, hi]
    bool done = !work;                          // threshold known
    bool rank_now = work && n <= SEL_CAND;      // few enough keys in [lo, hi] to rank directly

    const int per = (n + GT - 1) / GT * 64, i0 = min(n, gw * per), i1 = min(n, i0 + per);   // (this wave's to place)
    uint32_t own[KPT > 0 ? KPT : 1];
    if constexpr (KPT > 0)
#pragma unroll
        for (int j = 0; j < KPT; ++j) own[j] = keys(min(i0 + j * 64 + lane, n - 1));
    // all keys of the group, each by one thread
    auto each = [&](auto take) __attribute__((always_inline)) {
        if constexpr (KPT > 0) {
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if (i0 + j * 64 + lane < i1) take(own[j]);
        } else {
#pragma unroll 4
            for (int i = gt; i < n; i += GT) take(keys[i]);
        }
    };
    // the 64 keys at i0 + 64 j of this wave, for every j that it has
    auto each_run = [&](auto take) __attribute__((always_inline)) {
        if constexpr (KPT > 0) {
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if (i0 + j * 64 < i1) take(i0 + j * 64, i0 + j * 64 + lane < i1, own[j]);
        } else {
            for (int i = i0; i < i1; i += 64) {
                const bool in = i + lane < i1;
                take(i, in, in ? keys[i + lane] : 0u);
            }
        }
    };
    if (gt == 0) sh.n_cand[g] = 0u;
    if (threadIdx.x == 0) sh.open = 0u;
    lds_barrier();   // (the keys are in LDS)
    if (all_short) {
        // (no segment of the workgroup is longer than a wave: one wave each ranks and places its
        // keys, nothing crosses waves)
        if (work && gw == 0) {
            const bool in = lane < n;
            uint32_t key;
            if constexpr (KPT > 0) key = in ? own[0] : 0u;
            else key = in ? keys[lane] : 0u;
            uint32_t above = 0u, equal = 0u;
            for (int j = 0; j < n; j += 8)       // (lanes beyond n hold 0, below every valid key)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)key, j + e);
                    above += v > key;
                    equal += v == key;
                }
            // keys above T all have a rank below k, T itself straddles it
            const bool is_t = in && above < remaining && remaining <= above + equal;
            const unsigned long long bt = __ballot(is_t);
            const unsigned long long below = (1ull << lane) - 1ull;
            const uint32_t eq_rank = (uint32_t)__popcll(bt & below), need = remaining - min(above, remaining);
            const bool keep = in && (is_t ? eq_rank < need : above + equal < remaining);
            const unsigned long long bk = __ballot(keep);
            if (keep) out[__popcll(bk & below)] = idx_offset + lane;
        }
        return;
    }
    if (work && !rank_now) {
        uint32_t mx = 0u, mn_inv = 0u;          // (the minimum as the maximum of the complements)
        each([&](uint32_t key) __attribute__((always_inline)) {
            mx = max(mx, key);
            mn_inv = max(mn_inv, ~key);
        });
        mx = wave_max(mx);
        mn_inv = wave_max(mn_inv);
        if (lane == 0) {
            sh.wave[g][gw][0] = mx;
            sh.wave[g][gw][1] = mn_inv;
        }
    }
    if (gt == 0 && work) atomicAdd(&sh.open, 1u);
    lds_barrier();
    if (work && !rank_now) {
        uint32_t mx = 0u, mn_inv = 0u;
#pragma unroll
        for (int w = 0; w < GW; ++w) {
            mx = max(mx, sh.wave[g][w][0]);
            mn_inv = max(mn_inv, sh.wave[g][w][1]);
        }
        hi = mx;
        lo = ~mn_inv;
    }
    // 32 key bits in steps of 10: a fifth round never has anything left to narrow
    for (int pass = 0; pass < 5 && sh.open != 0u; ++pass) {
        const bool narrow = !done && !rank_now;
        const uint32_t range = hi - lo;
        const int shift = range < SEL_BINS ? 0 : 22 - __clz((int)range);
        if (narrow) {
#pragma unroll
            for (int j = 0; j < BPT; ++j) sh.hist[g][j * GT + gt] = 0u;
        }
        lds_barrier();
        if (narrow) {
            each([&](uint32_t key) __attribute__((always_inline)) {
                const uint32_t d = key - lo;
                if (d <= range) atomicAdd(&sh.hist[g][d >> shift], 1u);
            });
        }
        lds_barrier();
        // counts from the top bin down: thread t looks at bins SEL_BINS-1 - t*BPT ...
        uint32_t c[BPT], mine = 0u, incl = 0u;
        if (narrow) {
#pragma unroll
            for (int j = 0; j < BPT; ++j) {
                c[j] = sh.hist[g][SEL_BINS - 1 - (gt * BPT + j)];
                mine += c[j];
            }
            incl = wave_scan_incl(mine);
            if (lane == 63) sh.wave[g][gw][0] = incl;
        }
        lds_barrier();
        if (narrow) {
            uint32_t before = incl - mine;
#pragma unroll
            for (int w = 0; w < GW - 1; ++w) before += w < gw ? sh.wave[g][w][0] : 0u;
            if (before < remaining && remaining <= before + mine) {
#pragma unroll
                for (int j = 0; j < BPT; ++j) {
                    if (before < remaining && remaining <= before + c[j]) {
                        sh.found[g][0] = (uint32_t)(SEL_BINS - 1 - (gt * BPT + j));
                        sh.found[g][1] = remaining - before;
                        sh.found[g][2] = c[j];
                    }
                    before += c[j];
                }
            }
        }
        lds_barrier();
        if (narrow) {
            lo += sh.found[g][0] << shift;
            remaining = sh.found[g][1];
            if (shift == 0) {                    // the bin is one key value
                hi = lo;
                done = true;
                if (gt == 0) {
                    sh.result[g][0] = lo;
                    sh.result[g][1] = remaining;
                    atomicSub(&sh.open, 1u);
                }
            } else {
                hi = lo + min(hi - lo, (1u << shift) - 1u);
                rank_now = sh.found[g][2] <= SEL_CAND;
            }
        }
        const bool rank_pass = !done && rank_now;
        if (rank_pass) {
            each([&](uint32_t key) __attribute__((always_inline)) {
                if (key >= lo && key <= hi) sh.cand[g][atomicAdd(&sh.n_cand[g], 1u)] = key;
            });
        }
        lds_barrier();
        if (rank_pass) {
            done = true;
            if (gw == 0) {
                // rank of this lane's key by value among the candidates; every lane whose key is T
                // writes the same result
                const int m = (int)sh.n_cand[g];
                const uint32_t my = lane < m ? sh.cand[g][lane] : 0u;
                uint32_t above = 0u, equal = 0u;
                for (int j = 0; j < m; ++j) {
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)my, j);
                    above += v > my;
                    equal += v == my;
                }
                if (lane < m && above < remaining && remaining <= above + equal) {
                    sh.result[g][0] = my;
                    sh.result[g][1] = remaining - above;
                }
                if (lane == 0) atomicSub(&sh.open, 1u);
            }
        }
        lds_barrier();
    }
    // placement: wave gw owns `per` consecutive indices
    const uint32_t T = sh.result[g][0], need_eq = sh.result[g][1];
    uint32_t n_gt = 0u, n_eq = 0u;
    if (work) {
        each_run([&](int, bool in, uint32_t key) __attribute__((always_inline)) {
            n_gt += (uint32_t)__popcll(__ballot(in && key > T));
            n_eq += (uint32_t)__popcll(__ballot(in && key == T));
        });
        if (lane == 0) {
            sh.wave[g][gw][0] = n_gt;
            sh.wave[g][gw][1] = n_eq;
        }
    }
    lds_barrier();
    if (work) {
        uint32_t gt_before = 0u, eq_before = 0u;
#pragma unroll
        for (int w = 0; w < GW - 1; ++w) {
            gt_before += w < gw ? sh.wave[g][w][0] : 0u;
            eq_before += w < gw ? sh.wave[g][w][1] : 0u;
        }
        const unsigned long long below = (1ull << lane) - 1ull;
        each_run([&](int i, bool in, uint32_t key) __attribute__((always_inline)) {
            const unsigned long long bg = __ballot(in && key > T), be = __ballot(in && key == T);
            const uint32_t eq_rank = eq_before + (uint32_t)__popcll(be & below);
            const bool keep = in && (key > T || (key == T && eq_rank < need_eq));
            const uint32_t slot = gt_before + (uint32_t)__popcll(bg & below) + min(eq_rank, need_eq);
            if (keep && slot < (uint32_t)k) out[slot] = idx_offset + i + lane;
            gt_before += (uint32_t)__popcll(bg);
            eq_before += (uint32_t)__popcll(be);
        });
    }
}

// One workgroup of GW waves per (sample, segment), up to KPT keys a thread.
template <int GW, int KPT>
__global__ __launch_bounds__(GW * 64) void select_kernel(const float* __restrict__ sal,
                                                         const int32_t* __restrict__ k2k3, int n2,
                                                         int n3, int n_text, int k_total,
                                                         int32_t* __restrict__ kept_idx) {
    __shared__ SelShared<GW, 1> sh;
    const int b = blockIdx.y, which = blockIdx.x;
    int32_t* row = kept_idx + (size_t)b * (k_total + n_text);
    // clamp a malformed budget row into the feasible range
    int k2 = k2k3[2 * b];
    k2 = min(max(k2, max(0, k_total - n3)), min(n2, k_total));
    if (which == 2) {
        for (int i = threadIdx.x; i < n_text; i += GW * 64) row[k_total + i] = n2 + n3 + i;
        return;
    }
    const float* seg = sal + (size_t)b * (n2 + n3) + (which ? n2 : 0);
    const int n = which ? n3 : n2;
    if (n <= 0) return;
    select_groups<GW, 1, KPT>([&](int i) __attribute__((always_inline)) { return sal_key(seg[i]); }, n, which ? k_total - k2 : k2, which ? n2 : 0, which ? row + k2 : row,
                         n <= SEL_CAND, sh);
}

// Budget and selection of one sample by one workgroup (end of the fused kernels).  Same
// summation order as budget_kernel, same selection as select_kernel; the two segments are
// selected side by side, half the workgroup's waves each.  load: the salience of FIN_U columns.
template <typename Load>
__device__ __forceinline__ void finish_sample(Load load, const FusedPrune& f, int b, uint32_t* keys) {
    __shared__ double sh_d[2 * (BUD_THREADS / 64)];
    __shared__ SelShared<SAL_THREADS / 128, 2> sh;
    __shared__ int sh_k2;
    // one pass over the sample's scores feeds both the masses and the selection keys of both
    // segments (keys [0, n2) and [n2, n2 + n3) of the LDS array)
    auto feed = [&](int off, int n) __attribute__((always_inline)) {
        double a = 0.0;
        for (int i = threadIdx.x; i < n; i += FIN_U * BUD_THREADS) {
            int col[FIN_U];
            float v[FIN_U];
#pragma unroll
            for (int u = 0; u < FIN_U; ++u) col[u] = off + min(i + u * BUD_THREADS, n - 1);
            load(col, v);
#pragma unroll
            for (int u = 0; u < FIN_U; ++u)
                if (i + u * BUD_THREADS < n) {
                    a += (double)v[u];
                    keys[col[u]] = sal_key(v[u]);
                }
        }
        return a;
    };
    double a2 = feed(0, f.n2), a3 = feed(f.n2, f.n3);
    block_sum2_f64(a2, a3, sh_d);
    if (threadIdx.x == 0) {
        int k2;
        double m2;
        budget_split(a2, a3, f.n2, f.n3, f.k_total, f.min2, f.min3, &k2, &m2);
        f.k2k3[2 * b] = k2;
        f.k2k3[2 * b + 1] = f.k_total - k2;
        sh_k2 = k2;
    }
    int32_t* row = f.kept_idx + (size_t)b * (f.k_total + f.n_text);
    for (int i = threadIdx.x; i < f.n_text; i += SAL_THREADS)
        row[f.k_total + i] = f.n2 + f.n3 + i;
    lds_barrier();
    const int k2 = sh_k2;
    const bool second = threadIdx.x >= SAL_THREADS / 2;   // (wave-uniform)
    select_groups<SAL_THREADS / 128, 2>(second ? keys + f.n2 : keys, second ? f.n3 : f.n2,
                                        second ? f.k_total - k2 : k2, second ? f.n2 : 0,
                                        second ? row + k2 : row, max(f.n2, f.n3) <= SEL_CAND, sh);
}

int launch_select(const float* sal, const int32_t* k2k3, int B, int n2, int n3, int n_text,
                  int k_total, int32_t* kept_idx, hipStream_t st) {
    if (n2 > SEL_MAX_N || n3 > SEL_MAX_N) return MVLA_EUNSUPPORTED;
    // (four waves up to SEL_FOUR_WAVES, else sixteen, with as many keys a thread as the longer segment needs)
    const int longest = max(n2, n3);
#define MVLA_SELECT(GW, KPT)                                                                               \
    hipLaunchKernelGGL((select_kernel<GW, KPT>), dim3(3, B), dim3(GW * 64), 0, st, sal, k2k3, n2, n3, n_text, k_total, \
                       kept_idx)
    if (longest <= 4 * 64 * 4) MVLA_SELECT(4, 4);
    else if (longest <= SEL_FOUR_WAVES) MVLA_SELECT(4, 8);
    else if (longest <= 16 * 64 * 8) MVLA_SELECT(16, 8);
    else MVLA_SELECT(16, 16);
#undef MVLA_SELECT
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Gather-compaction (paper Sec. 4.4 / Eq. 10): copy kept rows and their
// position ids.  One workgroup per output row, 16 bytes per lane per access.
// ---------------------------------------------------------------------------
constexpr int CMP_THREADS = 256;

__global__ __launch_bounds__(CMP_THREADS) void compact_kernel(
    const uint4* __restrict__ h, const int32_t* __restrict__ pos,
    const int32_t* __restrict__ kept_idx, int S, int S_out, int row_vec /* D*2/16 */,
    uint4* __restrict__ h_out, int32_t* __restrict__ pos_out) {
    const int i = blockIdx.x, b = blockIdx.y;
    int src = kept_idx[(size_t)b * S_out + i];
    src = min(max(src, 0), S - 1);
    const uint4* from = h + ((size_t)b * S + src) * row_vec;
    uint4* to = h_out + ((size_t)b * S_out + i) * row_vec;
    int c = threadIdx.x;
    for (; c + CMP_THREADS < row_vec; c += 2 * CMP_THREADS) {
        const uint4 a = from[c];
        const uint4 d = from[c + CMP_THREADS];
        to[c] = a;
        to[c + CMP_THREADS] = d;
    }
    for (; c < row_vec; c += CMP_THREADS) to[c] = from[c];
    if (threadIdx.x == 0) pos_out[(size_t)b * S_out + i] = pos[(size_t)b * S + src];
}

int launch_compact(const bf16_t* h, const int32_t* pos, const int32_t* kept_idx, int B, int S,
                   int S_out, int D, bf16_t* h_out, int32_t* pos_out, hipStream_t st) {
    if (S_out == 0 || B == 0) return MVLA_OK;
    hipLaunchKernelGGL(compact_kernel, dim3(S_out, B), dim3(CMP_THREADS), 0, st,
                       reinterpret_cast<const uint4*>(h), pos, kept_idx, S, S_out, D / 8,
                       reinterpret_cast<uint4*>(h_out), pos_out);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Per-patch modality indicators of the semantic stage (paper Sec. 3.2,
// Eqs. 4-6): the 3D attention vector of a patch (over the head x query rows)
// is split into its projection on the 2D vector and the orthogonal rest; the
// outputs are the L1 shares |a2| / (|a2|+|a3|) and |a3_ortho| / (|a2|+|a3|).
// One workgroup handles 16 patches of one sample; a thread owns VEC patches and every RG-th row.  Up to RPT
// rows a thread (1024 rows at sixteen waves) stay in registers between the two
// sums -- <a2,a2>, <a2,a3>, |a2|, |a3|, then the L1 norm of the residual --, so the rows are read once,
// all requests in flight together; longer ones are read a second time (served by the caches).
// Bound by latency: 1024 rows x 2 x 256 patches (B = 4) 11.0 -> 5.5 us against 8 patches a
// workgroup of four waves, read twice in 32-byte pieces.  Few rows take four or eight waves: a wave's
// reductions cost the same however few rows it has, and the waves of a SIMD take turns at them.
// ---------------------------------------------------------------------------
constexpr int DEC_PP = 16;                      // patches per workgroup

// Sum over the lanes of a wave that hold the same patches (every LP-th lane), in all of them: rotations
// within 16 lanes, then the 16-lane rows, then the halves.
template <int LP>
__device__ __forceinline__ float same_patch_sum(float x) {
    if (LP <= 4) x += __uint_as_float(dpp_get<0x124, 0xf>(__float_as_uint(x), 0u));   // row_ror:4
    if (LP <= 8) x += __uint_as_float(dpp_get<0x128, 0xf>(__float_as_uint(x), 0u));   // row_ror:8
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

template <int THREADS, int VEC, int RPT /* rows a thread keeps; 0: read twice */>
__global__ __launch_bounds__(THREADS) void decompose_kernel(const float* __restrict__ attn,
                                                                int R, int S, int n_patch,
                                                                float* __restrict__ m2d,
                                                                float* __restrict__ m3d) {
    constexpr int LP = DEC_PP / VEC, RG = THREADS / LP;   // lanes across the patches; row groups
    __shared__ float red[4][THREADS / 64][DEC_PP], tot[4][DEC_PP];
    const int tid = threadIdx.x, l = tid % LP, g = tid / LP, wave = tid >> 6;
    const int b = blockIdx.y, p0 = blockIdx.x * DEC_PP + l * VEC;
    const float* base = attn + (size_t)b * R * S + p0;
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    // (VEC == 4: n_patch % 4 == 0, so a lane's patches exist all or none)
    const bool live = p0 < n_patch;
    auto load = [&](int r, int col) __attribute__((always_inline)) {
        return *reinterpret_cast<const vec_t*>(base + (size_t)r * S + col);
    };
    vec_t s22 = 0.f, s23 = 0.f, l2 = 0.f, l3 = 0.f;
    auto add = [&](vec_t a2, vec_t a3) __attribute__((always_inline)) {
        s22 += a2 * a2;
        s23 += a2 * a3;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            l2[v] += fabsf(a2[v]);
            l3[v] += fabsf(a3[v]);
        }
    };
    vec_t k2[RPT > 0 ? RPT : 1], k3[RPT > 0 ? RPT : 1];
    if (RPT > 0) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = g + i * RG;
            k2[i] = k3[i] = 0.f;
            if (live && r < R) {
                k2[i] = load(r, 0);
                k3[i] = load(r, n_patch);
            }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) add(k2[i], k3[i]);     // (rows that are not there add zeros)
    } else if (live) {
#pragma unroll 4
        for (int r = g; r < R; r += RG) add(load(r, 0), load(r, n_patch));
    }
    const vec_t sums[4] = {s22, s23, l2, l3};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const float t = same_patch_sum<LP>(sums[q][v]);
            if ((tid & 63) < LP) red[q][wave][l * VEC + v] = t;
        }
    __syncthreads();
    if (tid < 4 * DEC_PP) {              // one wave folds the waves' sums: 4 quantities x 16 patches
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) t += red[tid / DEC_PP][w][tid % DEC_PP];
        tot[tid / DEC_PP][tid % DEC_PP] = t;
    }
    __syncthreads();
    vec_t c;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        const float a = tot[0][l * VEC + v];
        c[v] = a > 0.f ? tot[1][l * VEC + v] / a : 0.f;
    }
    vec_t lo = 0.f;
    auto rest = [&](vec_t a2, vec_t a3) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) lo[v] += fabsf(a3[v] - c[v] * a2[v]);
    };
    if (RPT > 0) {
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (g + i * RG < R) rest(k2[i], k3[i]);   // (0 - c * 0 is no zero where c has overflowed)
    } else if (live) {
#pragma unroll 4
        for (int r = g; r < R; r += RG) rest(load(r, 0), load(r, n_patch));
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        const float t = same_patch_sum<LP>(lo[v]);
        if ((tid & 63) < LP) red[0][wave][l * VEC + v] = t;   // (read by the first wave before the last barrier)
    }
    __syncthreads();
    const int p = blockIdx.x * DEC_PP + tid;
    if (tid < DEC_PP && p < n_patch) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) t += red[0][w][tid];
        const float den = tot[2][tid] + tot[3][tid];
        m2d[(size_t)b * n_patch + p] = den > 0.f ? tot[2][tid] / den : 0.f;
        m3d[(size_t)b * n_patch + p] = den > 0.f ? t / den : 0.f;
    }
}

int launch_decompose(const float* attn, int B, int H, int Nq, int S, int n_patch, float* m2d,
                     float* m3d, hipStream_t st) {
    const int R = H * Nq;
    const dim3 grid((n_patch + DEC_PP - 1) / DEC_PP, B);
#define MVLA_DEC(T, V, N)                                                                              \
    hipLaunchKernelGGL((decompose_kernel<T, V, N>), grid, dim3(T), 0, st, attn, R, S, n_patch, m2d, m3d)
    // As few threads as hold all rows in registers.  16 bytes a lane where every row of both halves is
    // aligned for it, T / 4 row groups of four rows each; else, and for up to 256 rows, 4 bytes, T / 16 row groups of
    // sixteen (a quarter of the reductions).  64 rows x 2 x 256 patches (B = 4) 3.0 us, with 256 threads and
    // 16 bytes 3.6, with 1024 threads 4.7; 256 rows 3.4, 4.0 and 4.8; 512 rows with 512 threads 4.2, with 1024 5.0.
    // Beyond 1024 rows they are read twice (1024 rows 5.5 us, 1056 10.2).
    if (R <= 256) {
        MVLA_DEC(256, 1, 16);
    } else if (S % 4 == 0 && n_patch % 4 == 0 && (reinterpret_cast<uintptr_t>(attn) & 15) == 0) {
        if (R <= 512) MVLA_DEC(512, 4, 4);
        else if (R <= 1024) MVLA_DEC(1024, 4, 4);
        else MVLA_DEC(1024, 4, 0);
    } else {
        if (R <= 512) MVLA_DEC(512, 1, 16);
        else if (R <= 1024) MVLA_DEC(1024, 1, 16);
        else MVLA_DEC(1024, 1, 0);
    }
#undef MVLA_DEC
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Action-iteration smoothing of an indicator (paper Sec. 4.3 Eq. 7, Sec. 4.4
// Eqs. 8-9): observation at the cold start, running mean while the window
// fills, exponential moving average afterwards.  w_prev and w_new are the two
// weights of the step, computed on the host in fp64 and rounded to fp32.
// ---------------------------------------------------------------------------
__global__ void smooth_kernel(const float* __restrict__ x_t, float* __restrict__ x_hat, size_t n,
                              float w_prev, float w_new, int cold) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = x_t[i];
    x_hat[i] = cold ? x : w_prev * x_hat[i] + w_new * x;
}

int launch_smooth(const float* x_t, float* x_hat, size_t n, int t, int k, double beta,
                  hipStream_t st) {
    if (n == 0) return MVLA_OK;
    double wp, wn;
    if (t < k) {
        wp = (double)(t - 1) / (double)t;
        wn = 1.0 / (double)t;
    } else {
        wp = beta;
        wn = 1.0 - beta;
    }
    hipLaunchKernelGGL(smooth_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x_t,
                       x_hat, n, (float)wp, (float)wn, t == 1 ? 1 : 0);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

}  // namespace mvla
