// Element-wise and small kernels of the decoder layer on gfx950: RMSNorm,
// rotary table (the rotation itself and the V transpose happen in the q/k/v
// projection's epilogue, gemm.hip), and the language-query scoring
// probabilities (paper Sec. 3.2: the attention rows that salience is read from).
#include "common.h"
#include "mfma.h"
#include "wave.h"

namespace mvla {

// ---------------------------------------------------------------------------
// RMSNorm: out = x * gain / sqrt(mean(x^2) + eps), fp32 maths, bf16 out.  One
// workgroup per row; a thread keeps its 16-byte chunks in registers between the
// sum of squares and the scaling, so the row is read once.
// Bound by memory at large batches, by latency at small ones: the gain is asked for with the row, the sum goes
// over the vector unit, and a row of up to 512 or 1024 values takes one or two waves (NT threads) instead of four that
// meet at a barrier.
// ---------------------------------------------------------------------------
constexpr int NORM_MAX_CHUNKS = 4;  // per thread of 256: D <= 256 * 4 * 8 = 8192

template <int NT>
__device__ __forceinline__ float block_sum(float v, float* sh) {
    v = wave_sum_f32(v);
    if (NT == 64) return v;
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += sh[w];
    return t;
}

// The rows a norm kernel works on.
enum NormRows {
    NORM_BF16,      // all rows of x (bf16)
    NORM_F32,       // ... of the mid-layer residual stream (fp32)
    NORM_GATHER     // rows of x that `index` names, copied to x_out as well, their position ids to pos_out
};
struct NormSide {   // what else a norm kernel reads and writes
    int S, tail;                 // tail > 0: the last `tail` rows of every sample of S rows are written a second time,
    uint4* out2;                 // packed into out2 [B*tail, D] (the scoring pass projects queries for those rows only);
    const int32_t* pos;          // NORM_GATHER: the copied rows
    int32_t* pos_out;
    const int32_t* index;        // NORM_GATHER: [B, S_out] rows of each sample
    int S_out;
};

template <NormRows ROWS, int NT, int CHUNKS>
__global__ __launch_bounds__(NT) void rmsnorm_kernel(const void* __restrict__ xv, const uint4* __restrict__ gain,
                                                     int row_vec /* D/8 */, float inv_d, float eps,
                                                     uint4* __restrict__ out, NormSide side) {
    __shared__ float sh[NT / 64];
    const int row = blockIdx.x, tid = threadIdx.x;
    int from = row;                      // row of x
    int row2 = -1;                       // row of out2, if this row has one
    if (ROWS == NORM_GATHER) {
        const int b = row / side.S_out;
        from = b * side.S + min(max(side.index[row], 0), side.S - 1);
        row2 = row;
    } else if (ROWS == NORM_BF16 && side.tail > 0) {
        const int b = row / side.S, s_ = row - b * side.S;
        if (s_ >= side.S - side.tail) row2 = b * side.tail + s_ - (side.S - side.tail);
    }
    uint4 in[CHUNKS], in_hi[ROWS == NORM_F32 ? CHUNKS : 1], g[CHUNKS];
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        const int c = min(tid + k * NT, row_vec - 1);   // (chunks beyond the row: its last one, left out of the sum)
        if (ROWS == NORM_F32) {
            const uint4* xr = static_cast<const uint4*>(xv) + (size_t)from * row_vec * 2;
            in[k] = xr[2 * c];
            in_hi[ROWS == NORM_F32 ? k : 0] = xr[2 * c + 1];
        } else {
            in[k] = (static_cast<const uint4*>(xv) + (size_t)from * row_vec)[c];
        }
        g[k] = gain[c];
    }
    if (row2 >= 0 && tid == 0) side.pos_out[row2] = side.pos[from];
    auto value = [&](int k, int i) __attribute__((always_inline)) {
        if (ROWS == NORM_F32) {
            const uint4& v = i < 4 ? in[k] : in_hi[ROWS == NORM_F32 ? k : 0];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            return __uint_as_float(w[i & 3]);
        }
        const uint32_t w[4] = {in[k].x, in[k].y, in[k].z, in[k].w};
        return __uint_as_float((i & 1) ? w[i >> 1] & 0xFFFF0000u : w[i >> 1] << 16);
    };
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k)
        if (tid + k * NT < row_vec)
#pragma unroll
            for (int i = 0; i < 8; ++i) ss += value(k, i) * value(k, i);
    ss = block_sum<NT>(ss, sh);
    const float scale = 1.0f / sqrtf(ss * inv_d + eps);
    uint4* optr = out + (size_t)row * row_vec;
    uint4* ptr2 = side.out2 + (size_t)(row2 >= 0 ? row2 : 0) * row_vec;
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        const int c = tid + k * NT;
        if (c < row_vec) {
            const uint32_t gw[4] = {g[k].x, g[k].y, g[k].z, g[k].w};
            uint32_t r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                r[i] = pack_bf16x2(value(k, 2 * i) * scale * __uint_as_float(gw[i] << 16),
                                   value(k, 2 * i + 1) * scale * __uint_as_float(gw[i] & 0xFFFF0000u));
            optr[c] = make_uint4(r[0], r[1], r[2], r[3]);
            if (row2 >= 0) ptr2[c] = ROWS == NORM_GATHER ? in[k] : make_uint4(r[0], r[1], r[2], r[3]);
        }
    }
}

template <NormRows ROWS>
static int launch_rmsnorm_any(const void* x, const bf16_t* gain, int M, int D, float eps, bf16_t* out,
                              const NormSide& side, hipStream_t st) {
    if (M <= 0) return MVLA_OK;
    if (D % 8 != 0 || D / 8 > 256 * NORM_MAX_CHUNKS) return MVLA_EUNSUPPORTED;
#define MVLA_NORM(NT, CHUNKS)                                                                          \
    hipLaunchKernelGGL((rmsnorm_kernel<ROWS, NT, CHUNKS>), dim3(M), dim3(NT), 0, st, x,                \
                       reinterpret_cast<const uint4*>(gain), D / 8, 1.0f / (float)D, eps,              \
                       reinterpret_cast<uint4*>(out), side)
    if (D <= 512) MVLA_NORM(64, 1);
    else if (D <= 1024) MVLA_NORM(128, 1);
    else if (D <= 2048) MVLA_NORM(256, 1);
    else if (D <= 4096) MVLA_NORM(256, 2);
    else MVLA_NORM(256, NORM_MAX_CHUNKS);
#undef MVLA_NORM
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

int launch_rmsnorm(const bf16_t* x, const bf16_t* gain, int M, int D, float eps, bf16_t* out,
                   hipStream_t st) {
    return launch_rmsnorm_any<NORM_BF16>(x, gain, M, D, eps, out, NormSide{}, st);
}
int launch_rmsnorm_f32(const float* x, const bf16_t* gain, int M, int D, float eps, bf16_t* out,
                       hipStream_t st) {
    return launch_rmsnorm_any<NORM_F32>(x, gain, M, D, eps, out, NormSide{}, st);
}

int launch_rmsnorm_tail(const bf16_t* x, const int32_t* pos, const bf16_t* gain, int B, int S,
                        int tail, int D, float eps, bf16_t* out, bf16_t* out_tail, int32_t* pos_out,
                        hipStream_t st) {
    if (B <= 0 || S <= 0) return MVLA_OK;
    if (tail <= 0 || tail > S || !pos || !pos_out || !out_tail) return MVLA_EINVAL;
    return launch_rmsnorm_any<NORM_BF16>(x, gain, B * S, D, eps, out,
                                         {S, tail, reinterpret_cast<uint4*>(out_tail), pos, pos_out, nullptr, 0}, st);
}

int launch_compact_norm(const bf16_t* h, const int32_t* pos, const int32_t* kept_idx, int B, int S, int S_out, int D,
                        bf16_t* h_out, int32_t* pos_out, const bf16_t* gain, float eps, bf16_t* u, hipStream_t st) {
    return launch_rmsnorm_any<NORM_GATHER>(h, gain, B * S_out, D, eps, u,
                                           {S, 0, reinterpret_cast<uint4*>(h_out), pos, pos_out, kept_idx, S_out}, st);
}

// ---------------------------------------------------------------------------
// Rotary table in fp64: angle = pos * base^(-2i/dh).
// ---------------------------------------------------------------------------
__global__ void rope_table_kernel(double base, int rope_len, int half, float* __restrict__ c,
                                  float* __restrict__ s) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rope_len * half) return;
    const int pos = idx / half, i = idx % half;
    const double inv_freq = pow(base, -(double)i / (double)half);
    const double ang = (double)pos * inv_freq;
    c[idx] = (float)cos(ang);
    s[idx] = (float)sin(ang);
}

int launch_rope_table(double base, int rope_len, int dh, float* c, float* s, hipStream_t st) {
    const int n = rope_len * (dh / 2);
    if (n <= 0) return MVLA_OK;
    hipLaunchKernelGGL(rope_table_kernel, dim3((n + 255) / 256), dim3(256), 0, st, base, rope_len,
                       dh / 2, c, s);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Scoring probabilities of the last nq rows (the language-token queries):
//   P[b,h,i,:] = softmax_j( q_i . k_j / sqrt(dh) + key_bias[b,j] ),  j <= row(i).
// One workgroup per (32-query tile, head, sample).  Logits are MFMA tiles with
// queries on the rows and keys on the columns, so a register holds 32
// consecutive keys of one query across lanes and stores are coalesced.  Pass 1
// keeps a running max / sum per query; pass 2 recomputes the logits and writes
// normalised probabilities (nothing is staged in memory in between).
// ---------------------------------------------------------------------------
constexpr int SC_THREADS = 256;

// COLSUM: instead of the probabilities, write for every key column j < n_out the sum of the
// probabilities over the tile's (up to 32) queries: out[b, h, tile, j].  The salience
// reduction then runs over H * tiles short rows and the [B,H,nq,S] tensor never exists.
template <int DH, bool COLSUM>
__global__ __launch_bounds__(SC_THREADS) void score_probs_kernel(
    const bf16_t* __restrict__ q, int ldq, int q_rows /* per sample */, const bf16_t* __restrict__ k,
    int ldk, const float* __restrict__ key_bias, int S, int H, int nq, float scale,
    float* __restrict__ probs, int n_out) {
    constexpr int STEPS = DH / 16;
    const int qt = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 31, fg = lane >> 5;
    const int row0 = S - nq;            // sequence row of scoring query 0
    const int qi0 = qt * 32;            // first query of this tile

    // A operand: this lane's query row, all of dh
    uint4 qf[STEPS];
    {
        const int qi = min(qi0 + fr, nq - 1);
        // q holds either all S rows of a sample or only its nq scoring rows
        const bf16_t* src = q + ((size_t)b * q_rows + (q_rows - nq) + qi) * ldq + h * DH + fg * 8;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = *reinterpret_cast<const uint4*>(src + st * 16);
    }
    const int n_kb = (S + 31) / 32;
    const bf16_t* kbase = k + (size_t)b * S * ldk + h * DH + fg * 8;
    const float* bias = key_bias ? key_bias + (size_t)b * S : nullptr;

    float run_m[16], run_l[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) { run_m[v] = -INFINITY; run_l[v] = 0.f; }

    __shared__ float sh_m[SC_THREADS / 64][32], sh_l[SC_THREADS / 64][32];

    for (int pass = 0; pass < 2; ++pass) {
        // the key fragments of the wave's next block are requested before this block's products
        // (rows past the end are clamped: loaded, never used)
        uint4 kf[STEPS], kn[STEPS];
        {
            const bf16_t* ksrc = kbase + (size_t)min(wave * 32 + fr, S - 1) * ldk;
#pragma unroll
            for (int st = 0; st < STEPS; ++st) kn[st] = *reinterpret_cast<const uint4*>(ksrc + st * 16);
        }
        for (int kb = wave; kb < n_kb; kb += SC_THREADS / 64) {
            const int key = kb * 32 + fr;  // this lane's key column
#pragma unroll
            for (int st = 0; st < STEPS; ++st) kf[st] = kn[st];
            {
                const bf16_t* nsrc = kbase + (size_t)min(key + (SC_THREADS / 64) * 32, S - 1) * ldk;
#pragma unroll
                for (int st = 0; st < STEPS; ++st)
                    kn[st] = *reinterpret_cast<const uint4*>(nsrc + st * 16);
            }
            f32x16_t acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int st = 0; st < STEPS; ++st) acc = mfma32(qf[st], kf[st], acc);
            const float kbias = (bias && key < S) ? bias[key] : 0.f;
            float csum = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int qi = qi0 + mfma32_row(v, lane);
                const bool valid = key < S && key <= row0 + qi;
                const float logit = valid ? acc[v] * scale + kbias : -INFINITY;
                if (pass == 0) {
                    // per-lane running (max, sum) over this lane's key column
                    const float nm = fmaxf(run_m[v], logit);
                    if (nm != -INFINITY) {
                        run_l[v] = run_l[v] * __expf(run_m[v] - nm) + __expf(logit - nm);
                        run_m[v] = nm;
                    }
                } else if (qi < nq && key < S) {
                    const float p = valid ? __expf(logit - run_m[v]) * run_l[v] : 0.f;
                    if (COLSUM) csum += p;
                    else probs[(((size_t)b * H + h) * nq + qi) * S + key] = p;
                }
            }
            if (COLSUM && pass == 1) {
                csum += __shfl_xor(csum, 32);      // the other 16 query rows of the tile
                if (fg == 0 && key < n_out)
                    probs[(((size_t)b * H + h) * gridDim.x + qt) * n_out + key] = csum;
            }
        }
        if (pass == 0) {
            // combine (max, sum) over the 32 lanes that share a query row, then over the
            // four waves; afterwards run_m = global max, run_l = 1 / global sum
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                for (int o = 16; o > 0; o >>= 1) {
                    const float om = __shfl_xor(run_m[v], o), ol = __shfl_xor(run_l[v], o);
                    const float nm = fmaxf(run_m[v], om);
                    if (nm != -INFINITY)
                        run_l[v] = run_l[v] * __expf(run_m[v] - nm) + ol * __expf(om - nm);
                    run_m[v] = nm;
                }
            }
            if (fr == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sh_m[wave][mfma32_row(v, lane)] = run_m[v];
                    sh_l[wave][mfma32_row(v, lane)] = run_l[v];
                }
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = mfma32_row(v, lane);
                float gm = -INFINITY;
                for (int w = 0; w < SC_THREADS / 64; ++w) gm = fmaxf(gm, sh_m[w][r]);
                float gl = 0.f;
                for (int w = 0; w < SC_THREADS / 64; ++w)
                    gl += (sh_m[w][r] == -INFINITY) ? 0.f : sh_l[w][r] * __expf(sh_m[w][r] - gm);
                run_m[v] = gm;
                run_l[v] = 1.0f / gl;
            }
        }
    }
}

// Combination over the 16 lanes of a row, result in all of them: rotations within the row (vector-ALU only; the
// general shuffle goes through the LDS unit)
template <typename Op>
__device__ __forceinline__ float row_all(float x, Op op) {
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)));   // row_ror:8
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false)));
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, false)));
    return op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, false)));
}
// ... over the 32 lanes of a half-wave: its two rows exchange what they have
template <typename Op>
__device__ __forceinline__ float half_wave_all(float x, Op op) {
    x = row_all(x, op);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

constexpr int SC32_MAX = 8 * 8 * 32;       // keys that score_probs_reg_kernel holds
// Single-pass variant for S <= NW waves * KBW key blocks * 32 keys: every wave keeps the logits
// of its KBW key blocks in registers, so Q*K^T is computed once and the keys are read once.  AHEAD key
// blocks are in flight (all of them for short rows: one memory round trip).
// Bound by latency at batch 1 (one workgroup per head), by the key reads at large batches.  With two key
// blocks in flight and row reductions through the LDS unit: S = 144 10.5 us, S = 544 17.1 us; now
// 6.4 and 13.1 us.  (Eleven blocks a wave, for S up to 2816, spill: 868 us at B = 16, S = 2624
// against 279 us of the two-pass kernel; such rows take 16 queries a workgroup.)
template <int DH, int NW, int KBW, int AHEAD, bool COLSUM>
__global__ __launch_bounds__(NW * 64) void score_probs_reg_kernel(
    const bf16_t* __restrict__ q, int ldq, int q_rows /* per sample */, const bf16_t* __restrict__ k,
    int ldk, const float* __restrict__ key_bias, int S, int H, int nq, float scale,
    float* __restrict__ probs, int n_out) {
    constexpr int STEPS = DH / 16;
    const int qt = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 31, fg = lane >> 5;
    const int row0 = S - nq, qi0 = qt * 32;
    const int n_kb = (S + 31) / 32;
    const bf16_t* kbase = k + (size_t)b * S * ldk + h * DH + fg * 8;
    const float* bias = key_bias ? key_bias + (size_t)b * S : nullptr;
    // (rows past the end are clamped: loaded, never used)
    uint4 kf[AHEAD][STEPS];
    auto fetch = [&](int i) __attribute__((always_inline)) {
        const bf16_t* src = kbase + (size_t)min((wave + NW * i) * 32 + fr, S - 1) * ldk;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) kf[i % AHEAD][st] = *reinterpret_cast<const uint4*>(src + st * 16);
    };
    uint4 qf[STEPS];
    {
        const int qi = min(qi0 + fr, nq - 1);
        // q holds either all S rows of a sample or only its nq scoring rows
        const bf16_t* src = q + ((size_t)b * q_rows + (q_rows - nq) + qi) * ldq + h * DH + fg * 8;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = *reinterpret_cast<const uint4*>(src + st * 16);
    }
#pragma unroll
    for (int i = 0; i < AHEAD && i < KBW; ++i) fetch(i);
    // (asked for here where the rows are short, else where it is used: registers)
    constexpr bool EARLY_BIAS = KBW <= 3;
    auto key_bias_of = [&](int i) __attribute__((always_inline)) {
        return bias ? bias[min((wave + NW * i) * 32 + fr, S - 1)] : 0.f;
    };
    float kbias[EARLY_BIAS ? KBW : 1];
    if (EARLY_BIAS)
#pragma unroll
        for (int i = 0; i < KBW; ++i) kbias[i] = key_bias_of(i);

    f32x16_t lg[KBW];
#pragma unroll
    for (int i = 0; i < KBW; ++i) {
        const int kb = wave + NW * i;
#pragma unroll
        for (int v = 0; v < 16; ++v) lg[i][v] = 0.f;
        if (kb < n_kb) {   // wave-uniform
#pragma unroll
            for (int st = 0; st < STEPS; ++st) lg[i] = mfma32(qf[st], kf[i % AHEAD][st], lg[i]);
        }
        if (i + AHEAD < KBW) fetch(i + AHEAD);
    }
    float run_m[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) run_m[v] = -INFINITY;
#pragma unroll
    for (int i = 0; i < KBW; ++i) {
        const int kb = wave + NW * i, key = kb * 32 + fr;
        const float kbv = EARLY_BIAS ? kbias[EARLY_BIAS ? i : 0] : key_bias_of(i);
        // a key up to the first scoring row is seen by every query (wave-uniform test)
        if (kb * 32 + 31 <= row0 + qi0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                lg[i][v] = lg[i][v] * scale + kbv;
                run_m[v] = fmaxf(run_m[v], lg[i][v]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int qi = qi0 + mfma32_row(v, lane);
                const bool valid = key < S && key <= row0 + qi;
                lg[i][v] = valid ? lg[i][v] * scale + kbv : -INFINITY;
                run_m[v] = fmaxf(run_m[v], lg[i][v]);
            }
        }
    }
    __shared__ float sh_m[NW][32], sh_l[NW][32];
    // row maxima: over the 32 lanes of a half-wave, then over the waves
#pragma unroll
    for (int v = 0; v < 16; ++v) run_m[v] = half_wave_all(run_m[v], [](float a, float c) { return fmaxf(a, c); });
    if (fr == 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sh_m[wave][mfma32_row(v, lane)] = run_m[v];
    }
    __syncthreads();
    float run_l[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = mfma32_row(v, lane);
        float gm = sh_m[0][r];
#pragma unroll
        for (int w = 1; w < NW; ++w) gm = fmaxf(gm, sh_m[w][r]);
        run_m[v] = gm;     // finite: key 0 is visible to every query
        run_l[v] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < KBW; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            lg[i][v] = __expf(lg[i][v] - run_m[v]);   // exp(-inf) = 0 for masked entries
            run_l[v] += lg[i][v];
        }
#pragma unroll
    for (int v = 0; v < 16; ++v) run_l[v] = half_wave_all(run_l[v], [](float a, float c) { return a + c; });
    if (fr == 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sh_l[wave][mfma32_row(v, lane)] = run_l[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = mfma32_row(v, lane);
        float gl = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) gl += sh_l[w][r];
        run_l[v] = 1.0f / gl;
    }
#pragma unroll
    for (int i = 0; i < KBW; ++i) {
        const int kb = wave + NW * i;
        const int key = kb * 32 + fr;
        if (COLSUM) {
            float csum = 0.f;   // masked entries hold exp(-inf) = 0
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (qi0 + mfma32_row(v, lane) < nq) csum += lg[i][v] * run_l[v];
            csum += __shfl_xor(csum, 32);
            if (fg == 0 && kb < n_kb && key < n_out)
                probs[(((size_t)b * H + h) * gridDim.x + qt) * n_out + key] = csum;
        } else if (kb < n_kb && key < S) {
            float* out = probs + (((size_t)b * H + h) * nq + qi0) * S + key;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = mfma32_row(v, lane);
                if (qi0 + r < nq) out[(size_t)r * S] = lg[i][v] * run_l[v];
            }
        }
    }
}

// Direct global -> LDS copy of 16 bytes a lane: the wave's 64 lanes land on 1 KiB from the wave-uniform LDS address.
// (The compiler does not count it among its loads: wait_loads.  A wait of its own, for loads asked for before these,
// takes them for none and so waits for them too.)
__device__ __forceinline__ void load_to_lds16(const void* base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(off), "s"(base)
                 : "memory", "m0");
}
// All but the last n of this wave's loads have returned (n: a constant once the loop around it is unrolled).
__device__ __forceinline__ void wait_loads(int n) {
    switch (n) {
#define MVLA_WAIT(N) case N: asm volatile("s_waitcnt vmcnt(" #N ")" ::: "memory"); break;
        MVLA_WAIT(12) MVLA_WAIT(8) MVLA_WAIT(6) MVLA_WAIT(4) MVLA_WAIT(2)
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef MVLA_WAIT
    }
}

// As score_probs_reg_kernel with 16 queries a workgroup: twice the workgroups, and a lane holds 4 instead of 16 queries of
// a key, so the scaling, the exponentials and above all the reductions over the keys of a row (which every lane does for each of its
// queries) are a quarter of the instructions between the products, and rows of up to 2688 keys fit the registers.
// Bound by the key reads and the two reductions.  A key fragment that a wave takes from memory itself is 64 pieces of
// 16 bytes on 64 different cache lines as the load path counts them; keys come to LDS as whole rows instead, every
// wave's into a ring of its own of AHEAD blocks of 16 (the first AHEAD land together: the wait for the queries, asked for in
// front of them, counts them).  us, a tile of 32 queries with the keys in two passes or
// in registers / 16 with fragments from memory / now (32 heads of 128): S = 544, 32 rows 13.0 / 8.9 / 6.6; S = 1400 23.7 / -
// / 16.5; S = 2500, 64 rows 103 / - / 18.6; B = 16, S = 2624, 64 rows 278 / 221 / 163.
// A ring leaves room for a second workgroup per compute unit: with four blocks (128 KiB at DH = 128) one scoring tile of 16
// rows took, us, fragments / four blocks / two, S = 300, 512 workgroups 12.0 / 15.3 / 11.8, S = 544, 1024 of them
// 25.0 / 35.3 / 26.9, and fewer workgroups lose nothing (S = 1000, 64 of them 11.9 / 8.0 / 7.6).  (At 64-wide heads the
// keys of 256 tokens fit whole.)  A block of clamped rows costs as much as one of keys: rows of up to 128 take one a wave
// (us, fragments / two blocks / one, S = 80, 64 rows of 4 heads of 64, 1024 workgroups 8.0 / 8.7 / 7.5; 32 heads of 128, 32
// workgroups 5.0 / 5.0 / 4.1, 2048 of them 18.8 / 18.0 / 15.5).
template <int DH, int NW, int KBW, int AHEAD, bool COLSUM>
__global__ __launch_bounds__(NW * 64) void score_probs_rows16_kernel(
    const bf16_t* __restrict__ q, int ldq, int q_rows /* per sample */, const bf16_t* __restrict__ k,
    int ldk, const float* __restrict__ key_bias, int S, int H, int nq, float scale,
    float* __restrict__ probs, int n_out) {
    constexpr int STEPS = DH / 32;
    extern __shared__ uint4 key_rows[];          // ring of AHEAD blocks of 16 key rows per wave
    // (heads and samples are the grid's axes, or there is one axis: the tiles of a head are eight apart, on one XCD side by
    // side, and read its keys once)
    const int tiles = (nq + 15) / 16;
    int qt = 0, b = blockIdx.y, h = blockIdx.x;
    if ((int)gridDim.x != H) {
        const int pack = gridDim.x % (8 * tiles) == 0 ? 8 : 1;
        qt = (int)blockIdx.x / pack % tiles;
        const int hb = (int)blockIdx.x % pack * ((int)gridDim.x / (pack * tiles)) + (int)blockIdx.x / (pack * tiles);
        b = hb / H;
        h = hb - b * H;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;      // key column (operand row), query rows 4g ..
    const int row0 = S - nq, qi0 = qt * 16;
    const bf16_t* kbase = k + (size_t)b * S * ldk + h * DH;
    const float* bias = key_bias ? key_bias + (size_t)b * S : nullptr;
    uint4 qf[STEPS];
    {
        const int qi = min(qi0 + c, nq - 1);
        // q holds either all S rows of a sample or only its nq scoring rows
        const bf16_t* src = q + ((size_t)b * q_rows + (q_rows - nq) + qi) * ldq + h * DH + g * 8;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = *reinterpret_cast<const uint4*>(src + st * 32);
    }
    float kbias[KBW];
#pragma unroll
    for (int i = 0; i < KBW; ++i) kbias[i] = bias ? bias[min((wave + NW * i) * 16 + c, S - 1)] : 0.f;
    // Direct loads of whole key rows: chunk ch of row r of a block lies at place ch ^ (r & 15) of the row, or, of the
    // eight of a short row, ch ^ (r >> 1): fragment reads without bank conflicts.  (Rows past the end are clamped:
    // loaded, never used.)
    constexpr int CPR = DH / 8, LOADS = 16 * CPR / 64;
    const auto place = [](int row) { return DH == 128 ? row & 15 : (row >> 1) & 7; };
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)key_rows) + (uint32_t)wave * (AHEAD * 16 * CPR * 16);
    auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            const int row = (l * 64 + lane) / CPR, ch = lane % CPR ^ place(row);
            const int key = min((wave + NW * i) * 16 + row, S - 1);
            load_to_lds16(kbase, ((uint32_t)key * (uint32_t)ldk + (uint32_t)ch * 8u) * 2u,
                          lds_wave + (uint32_t)((i % AHEAD) * 16 * CPR + l * 64) * 16u);
        }
    };
#pragma unroll
    for (int i = 0; i < AHEAD && i < KBW; ++i) fetch(i);
    float run[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) run[v] = -INFINITY;
    f32x4_t lg[KBW];
#pragma unroll
    for (int i = 0; i < KBW; ++i) {
        lg[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        wait_loads(min(AHEAD - 1, KBW - 1 - i) * LOADS);     // block i has landed (a wave's loads return in order)
        uint4 kf[STEPS];
        const uint4* rows = key_rows + ((size_t)wave * AHEAD + i % AHEAD) * 16 * CPR + c * CPR;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) kf[st] = rows[(st * 4 + g) ^ place(c)];
#pragma unroll
        for (int st = 0; st < STEPS; ++st) lg[i] = mfma16(qf[st], kf[st], lg[i]);
        if (i + AHEAD < KBW) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and has been read: its place is free
            fetch(i + AHEAD);
        }
        const int kb = wave + NW * i, key = kb * 16 + c;
        // a key up to the first scoring row is seen by every query (wave-uniform test)
        const bool all = kb * 16 + 15 <= row0 + qi0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool valid = all || (key < S && key <= row0 + qi0 + 4 * g + v);
            lg[i][v] = valid ? lg[i][v] * scale + kbias[i] : -INFINITY;
            run[v] = fmaxf(run[v], lg[i][v]);
        }
    }
    __shared__ alignas(16) float sh_m[NW][16], sh_l[NW][16];   // (written four values at a time)
#pragma unroll
    for (int v = 0; v < 4; ++v) run[v] = row_all(run[v], [](float a, float o) { return fmaxf(a, o); });
    if (c == 0) *reinterpret_cast<float4*>(&sh_m[wave][4 * g]) = make_float4(run[0], run[1], run[2], run[3]);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float gm = sh_m[0][4 * g + v];
#pragma unroll
        for (int w = 1; w < NW; ++w) gm = fmaxf(gm, sh_m[w][4 * g + v]);
        float l = 0.f;       // (the maximum is finite: key 0 is visible to every query)
#pragma unroll
        for (int i = 0; i < KBW; ++i) {
            lg[i][v] = __expf(lg[i][v] - gm);   // exp(-inf) = 0 for masked entries
            l += lg[i][v];
        }
        run[v] = row_all(l, [](float a, float o) { return a + o; });
    }
    if (c == 0) *reinterpret_cast<float4*>(&sh_l[wave][4 * g]) = make_float4(run[0], run[1], run[2], run[3]);
    __syncthreads();
    float* out = probs + (((size_t)b * H + h) * nq + qi0) * S;
    float csum[KBW];
#pragma unroll
    for (int i = 0; i < KBW; ++i) csum[i] = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * g + v;
        float gl = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) gl += sh_l[w][r];
        const float inv = 1.0f / gl;
        if (qi0 + r < nq)
#pragma unroll
            for (int i = 0; i < KBW; ++i) {
                const int key = (wave + NW * i) * 16 + c;
                if (COLSUM) csum[i] += lg[i][v] * inv;
                else if (key < S) out[(size_t)r * S + key] = lg[i][v] * inv;
            }
    }
    if (COLSUM) {
        float* sums = probs + (((size_t)b * H + h) * tiles + qt) * n_out;
#pragma unroll
        for (int i = 0; i < KBW; ++i) {
            const int key = (wave + NW * i) * 16 + c;
            float t = csum[i];       // (over the four rows of lanes: the tile's other queries)
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (g == 0 && key < n_out) sums[key] = t;
        }
    }
}

// Where 16 queries a workgroup are the faster ones (us, 32 / 16 queries, 32 heads of 128, probabilities; every workgroup
// reads all keys): while these workgroups fit one per compute unit (S = 544, B = 4, 32 rows, 256 of them 14.0 / 7.8, S = 1000
// 21.6 / 11.8, S = 1840, 96 of them 28.7 / 16.0; S = 1500, 512 of them 31.2 / 39.8); where 32 queries would be no fewer
// workgroups (16 rows, B = 16: S = 544 27.1 / 17.0, S = 1025 43.6 / 42.8); for two key blocks a wave
// (S = 256) at any number where probabilities are written (B = 16, 64 rows 41.4 / 20.0), up to 512 where their sums are
// (9.2 / 7.1), whose number doubles; and wherever 32 queries take two passes over the keys (S > 2048: S = 2600, 512 of
// them 101 / 46).  (The lines at 256 and 512 date from rings of four blocks; with two there is room beyond them: S = 544, 512
// workgroups 15.9 / 13.9, sums of S = 256, 1024 of them 13.1 / 10.8.)
constexpr int SC16_MAX = 8 * 16 * 21;      // keys that eight waves hold
constexpr size_t SC16_GROUPS = ((size_t)1 << 32) / 512 - 1;   // workgroups of 512 threads that one grid axis holds
// One tile of queries has no keys to share: heads and samples are the grid's axes, and the workgroups run in the order of the
// key rows (us, one axis with its divisions / two: 32 heads of 128, S = 144, 256 workgroups 5.2 / 4.8, S = 544, 1024 of them
// 26.9 / 25.8; 16 heads of 64, S = 544, 1024 of them 18.1 / 15.9).
static bool score_axes(int B, int nq) { return nq <= 16 && B <= 65535; }
int score_tile_queries(int B, int H, int S, int nq, bool sums) {
    const size_t groups = (size_t)((nq + 15) / 16) * H * B;
    if (!score_axes(B, nq) && groups > SC16_GROUPS) return 32;
    if (S <= 8 * 16 * 2) return !sums || groups <= 512 || nq <= 16 ? 16 : 32;
    return S <= SC16_MAX && (groups <= 256 || nq <= 16 || S > SC32_MAX) ? 16 : 32;
}

template <int DH, bool COLSUM>
static int launch_score_rows16(const bf16_t* q, int ldq, int q_rows, const bf16_t* k, int ldk, const float* key_bias,
                                int B, int S, int H, int nq, float scale, float* out, int n_out, hipStream_t st) {
    const dim3 grid = score_axes(B, nq) ? dim3(H, B) : dim3((nq + 15) / 16 * H * B);
    // (the limit of a kernel's LDS is raised once per device)
#define MVLA_SCR(NW, KBW, AHEAD)                                                                              \
    do {                                                                                                      \
        constexpr int lds = NW * AHEAD * 16 * DH * 2;                                                         \
        auto kern = score_probs_rows16_kernel<DH, NW, KBW, AHEAD, COLSUM>;                                    \
        static bool lds_set[kMaxDevices] = {};                                                                \
        int dev = 0;                                                                                          \
        MVLA_HIP_CHECK(hipGetDevice(&dev));                                                                   \
        if (dev < 0 || dev >= kMaxDevices || !lds_set[dev]) {                                                 \
            MVLA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                           \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds));             \
            if (dev >= 0 && dev < kMaxDevices) lds_set[dev] = true;                                           \
        }                                                                                                     \
        hipLaunchKernelGGL(kern, grid, dim3(NW * 64), lds, st, q, ldq, q_rows, k, ldk, key_bias, S, H, nq, scale, \
                           out, n_out);                                                                       \
    } while (0)
    // (rings of up to 64 KiB, two workgroups per compute unit; the longest rows hold the registers of one)
    if (S <= 8 * 16) MVLA_SCR(8, 1, 1);
    else if (S <= 8 * 16 * 2) MVLA_SCR(8, 2, (DH == 128 ? 1 : 2));
    else if (S <= 8 * 16 * 5) MVLA_SCR(8, 5, 2);
    else if (S <= 8 * 16 * 8) MVLA_SCR(8, 8, 2);
    else MVLA_SCR(8, 21, 4);
#undef MVLA_SCR
    return MVLA_OK;
}

template <int DH, bool COLSUM>
static bool launch_score_reg(const bf16_t* q, int ldq, int q_rows, const bf16_t* k, int ldk,
                             const float* key_bias, int B, int S, int H, int nq, float scale,
                             float* out, int n_out, hipStream_t st) {
    dim3 grid((nq + 31) / 32, H, B);
    const int blocks = (S + 31) / 32;
#define MVLA_SCR(NW, KBW, AHEAD)                                                            \
    hipLaunchKernelGGL((score_probs_reg_kernel<DH, NW, KBW, AHEAD, COLSUM>), grid, dim3(NW * 64), 0, st, \
                       q, ldq, q_rows, k, ldk, key_bias, S, H, nq, scale, out, n_out)
    if (COLSUM && blocks <= 8 * 1) {   // (probabilities of so few keys: score_probs_rows16_kernel)
        if constexpr (COLSUM) MVLA_SCR(8, 1, 1);
    } else if (blocks <= 8 * 3) MVLA_SCR(8, 3, 3);
    else if (blocks <= 8 * 6) MVLA_SCR(8, 6, 2);
    else if (blocks <= 8 * 8) MVLA_SCR(8, 8, 2);
    else return false;
#undef MVLA_SCR
    return true;
}

template <int DH, bool COLSUM>
static int launch_score_dh(const bf16_t* q, int ldq, int q_rows, const bf16_t* k, int ldk,
                            const float* key_bias, int B, int S, int H, int nq, float scale,
                            float* out, int n_out, int tile, hipStream_t st) {
    if (tile == 16)
        return launch_score_rows16<DH, COLSUM>(q, ldq, q_rows, k, ldk, key_bias, B, S, H, nq, scale, out, n_out, st);
    // register-resident single pass when the row fits, else two passes
    if (launch_score_reg<DH, COLSUM>(q, ldq, q_rows, k, ldk, key_bias, B, S, H, nq, scale, out, n_out,
                                     st))
        return MVLA_OK;
    dim3 grid((nq + 31) / 32, H, B);
    hipLaunchKernelGGL((score_probs_kernel<DH, COLSUM>), grid, dim3(SC_THREADS), 0, st, q, ldq, q_rows,
                       k, ldk, key_bias, S, H, nq, scale, out, n_out);
    return MVLA_OK;
}

// colsum_n == 0: out = probabilities [B,H,nq,S]; colsum_n > 0: out = per-tile column sums
// [B, H, ceil(nq/tile), colsum_n] over the first colsum_n key columns.  tile: 32, or 16 where
// score_tile_queries says so.
int launch_score_probs(const bf16_t* q, int q_row_stride, bool q_tail_only, const bf16_t* k,
                       int k_row_stride, const float* key_bias, int B, int S, int H, int dh, int nq,
                       float* out, int colsum_n, int tile, hipStream_t st) {
    if (B <= 0 || nq <= 0) return MVLA_OK;
    const float scale = 1.0f / sqrtf((float)dh);
    const int q_rows = q_tail_only ? nq : S;
#define MVLA_SC(DH_, CS_)                                                                       \
    launch_score_dh<DH_, CS_>(q, q_row_stride, q_rows, k, k_row_stride, key_bias, B, S, H, nq, scale, \
                              out, colsum_n, tile, st)
    int rc;
    if (dh == 128) {
        rc = colsum_n > 0 ? MVLA_SC(128, true) : MVLA_SC(128, false);
    } else if (dh == 64) {
        rc = colsum_n > 0 ? MVLA_SC(64, true) : MVLA_SC(64, false);
    } else {
        return MVLA_EUNSUPPORTED;
    }
#undef MVLA_SC
    if (rc) return rc;
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

}  // namespace mvla
