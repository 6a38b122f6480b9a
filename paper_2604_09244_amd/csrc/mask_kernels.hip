// Mask generation of the tri-stage framework for gfx950 (paper Sec. 4.1-4.4,
// Algorithm 1): per-patch L1 feature share (Eq. 1), and one workgroup per
// sample that clusters the patches' attention scores (1-D k-means, K = 3),
// applies the semantic rules with their two baselines, fuses with the
// dual-threshold candidates and writes the two retention masks (Eq. 10);
// then a scan that turns the masks into ascending token indices.
// Every reduction has a fixed shape, so results are reproducible bit for bit.
#include "common.h"
#include "wave.h"

namespace mvla {

// ---------------------------------------------------------------------------
// Eq. 1: for patch p, l2 = |f_2D|_1 (row p), l3 = |f_3D|_1 (row n_patch + p);
// outputs l2/(l2+l3) and l3/(l2+l3), 0 when the denominator is 0.
// One workgroup per (patch, sample): waves 0-1 read the 2D row, waves 2-3 the
// 3D row, 16 bytes (8 bf16) per lane per access.
// ---------------------------------------------------------------------------
constexpr int FS_THREADS = 256;

__device__ inline float abs_sum8(uint4 v) {
    // bf16 -> fp32 is a 16-bit shift; |x| clears the sign bit
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s += __uint_as_float((w[i] << 16) & 0x7fffffffu);
        s += __uint_as_float(w[i] & 0x7fff0000u);
    }
    return s;
}

__global__ __launch_bounds__(FS_THREADS) void feature_share_kernel(
    const uint4* __restrict__ feat, int S, int row_vec /* D*2/16 */, int n_patch,
    float* __restrict__ m2d, float* __restrict__ m3d) {
    __shared__ float part[FS_THREADS / 64];
    const int p = blockIdx.x, b = blockIdx.y;
    const int half = threadIdx.x >> 7, t = threadIdx.x & 127;
    const uint4* row = feat + ((size_t)b * S + (half ? n_patch + p : p)) * row_vec;
    float s = 0.f;
    // (four chunks in flight together: one by one, each was a memory round trip; 2 x 256 rows of 4096 values, B = 4,
    // 4.7 -> 4.1 us; what is left, and rows of fewer than 4096 values, one by one)
    int c = t;
    for (; c + 3 * (FS_THREADS / 2) < row_vec; c += 4 * (FS_THREADS / 2)) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = row[c + u * (FS_THREADS / 2)];
#pragma unroll
        for (int u = 0; u < 4; ++u) s += abs_sum8(v[u]);
    }
    for (; c < row_vec; c += FS_THREADS / 2) s += abs_sum8(row[c]);
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float l2 = part[0] + part[1], l3 = part[2] + part[3];
        const float den = l2 + l3;
        m2d[(size_t)b * n_patch + p] = den > 0.f ? l2 / den : 0.f;
        m3d[(size_t)b * n_patch + p] = den > 0.f ? l3 / den : 0.f;
    }
}

int launch_feature_share(const bf16_t* feat, int B, int S, int D, int n_patch, float* m2d,
                         float* m3d, hipStream_t st) {
    hipLaunchKernelGGL(feature_share_kernel, dim3(n_patch, B), dim3(FS_THREADS), 0, st,
                       reinterpret_cast<const uint4*>(feat), S, D / 8, n_patch, m2d, m3d);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Candidate sets and masks, one workgroup per sample.
// ---------------------------------------------------------------------------
constexpr int CM_THREADS = 256;
constexpr int CM_WAVES = CM_THREADS / 64;

struct CmShared {
    double d[2][3][CM_WAVES];
    uint32_t n[2][CM_WAVES];
    int any[2][CM_WAVES];
    float f[2][CM_WAVES];
};

// Sums three doubles and a count (or two, 16 bits each) over the workgroup, same order every time; returns
// whether any thread's flag was set.  The LDS areas alternate from call to call, so one barrier is enough.
__device__ inline bool block_sum3(double s[3], uint32_t& n, bool flag, CmShared& sh, int parity) {
#pragma unroll
    for (int j = 0; j < 3; ++j) s[j] = wave_sum_f64(s[j]);
    n = wave_sum_u32(n);
    const bool any = __ballot(flag) != 0ull;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) sh.d[parity][j][threadIdx.x >> 6] = s[j];
        sh.n[parity][threadIdx.x >> 6] = n;
        sh.any[parity][threadIdx.x >> 6] = any;
    }
    __syncthreads();
    int f = 0;
    n = 0u;
#pragma unroll
    for (int w = 0; w < CM_WAVES; ++w) {
        f |= sh.any[parity][w];
        n += sh.n[parity][w];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        s[j] = 0.0;
#pragma unroll
        for (int w = 0; w < CM_WAVES; ++w) s[j] += sh.d[parity][j][w];
    }
    return f != 0;
}

enum : uint32_t { C_2D = 1u, C_3D = 2u };

__global__ __launch_bounds__(CM_THREADS) void candidate_kernel(
    const float* __restrict__ x_hat /* [4,B,P] */, const float* __restrict__ sal /* [B,2P] */,
    const float* __restrict__ u /* [B,P] */, int B, int P, int n_text, mvla_mask_rules rules,
    uint8_t* __restrict__ mask2d, uint8_t* __restrict__ mask3d, uint8_t* __restrict__ sem,
    int32_t* __restrict__ kept_len) {
    extern __shared__ float dyn[];
    float* score = dyn;                                         // [P]
    uint8_t* label = reinterpret_cast<uint8_t*>(dyn + P);       // [P]
    __shared__ CmShared sh;
    const int b = blockIdx.x, tid = threadIdx.x;
    const float* sal_b = sal + (size_t)b * 2 * P;

    // patch score: the 2D token's salience plus the 3D token's (summand of Eq. 3), in fp32
    float lo = INFINITY, hi = -INFINITY;
    for (int p = tid; p < P; p += CM_THREADS) {
        const float v = sal_b[p] + sal_b[P + p];
        score[p] = v;
        label[p] = 255;
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if ((tid & 63) == 0) {
        sh.f[0][tid >> 6] = lo;
        sh.f[1][tid >> 6] = hi;
    }
    __syncthreads();
    for (int w = 0; w < CM_WAVES; ++w) {
        lo = fminf(lo, sh.f[0][w]);
        hi = fmaxf(hi, sh.f[1][w]);
    }

    // Lloyd iterations (Sec. 4.2): centres start at min, mid-range, max; nearest centre, the
    // lower-numbered one on equal distance; a centre without points stays; stop when an
    // assignment repeats the previous one or after kmeans_max_iter assignments.
    // (One barrier an iteration.  A patch costs one LDS round trip: its score and label are asked for
    // together, nothing in the loop is conditional, and the counts stay with the thread.  16384 patches
    // 253 us; with ballots for the counts and a branch around the label in here 490; with shuffles and four
    // barriers an iteration 270.  Up to 8192 patches sorted_candidate_kernel takes the call.)
    double c0 = (double)lo, c2 = (double)hi, c1 = 0.5 * (c0 + c2);
    for (int it = 0; it < rules.kmeans_max_iter; ++it) {
        double s[3] = {0.0, 0.0, 0.0};
        uint32_t n01 = 0u;      // patches of labels 0 and 1, 16 bits each (P <= 16384)
        bool changed = false;
        for (int p = tid; p < P; p += CM_THREADS) {
            const int was = label[p];
            const double x = (double)score[p];
            const double d0 = fabs(x - c0), d1 = fabs(x - c1), d2 = fabs(x - c2);
            int l = 0;
            double best = d0;
            if (d1 < best) {
                best = d1;
                l = 1;
            }
            if (d2 < best) l = 2;
            changed |= l != was;
            label[p] = (uint8_t)l;
#pragma unroll
            for (int j = 0; j < 3; ++j) s[j] += l == j ? x : 0.0;
            n01 += l == 0 ? 1u : (l == 1 ? 0x10000u : 0u);
        }
        if (!block_sum3(s, n01, changed, sh, it & 1)) break;
        const int n0 = (int)(n01 & 0xFFFFu), n1 = (int)(n01 >> 16), n2 = P - n0 - n1;
        if (n0 > 0) c0 = s[0] / (double)n0;
        if (n1 > 0) c1 = s[1] / (double)n1;
        if (n2 > 0) c2 = s[2] / (double)n2;
    }
    __syncthreads();

    // baselines: means of the two semantic indicators over the sample's patches (Eqs. 5, 6)
    const float* m3_s1 = x_hat + ((size_t)1 * B + b) * P;
    const float* m2_s2 = x_hat + ((size_t)2 * B + b) * P;
    const float* m3_s2 = x_hat + ((size_t)3 * B + b) * P;
    double mu[3] = {0.0, 0.0, 0.0};
    uint32_t unused = 0u;
    for (int p = tid; p < P; p += CM_THREADS) {
        mu[0] += (double)m2_s2[p];
        mu[1] += (double)m3_s2[p];
    }
    block_sum3(mu, unused, false, sh, 0);
    const double mu2 = mu[0] / (double)P, mu3 = mu[1] / (double)P;

    uint32_t kept = 0u;
    for (int p = tid; p < P; p += CM_THREADS) {
        // data-preprocessing stage (Sec. 4.1): dual threshold on the 3D feature share
        const float share3 = m3_s1[p];
        const uint32_t cand1 = share3 < rules.tau_2d ? C_2D : (share3 > rules.tau_3d ? C_3D : C_2D | C_3D);
        // semantic stage (Sec. 4.2): lowest centre = background, middle = robot, highest = object
        const int l = label[p];
        const float a2 = m2_s2[p], a3 = m3_s2[p];
        uint32_t cand2;
        if (l == 0)
            cand2 = u[(size_t)b * P + p] < rules.bg_drop ? 0u : (C_2D | C_3D);
        else if (l == 1)
            cand2 = (double)a3 > mu3 ? (C_2D | C_3D) : ((double)a2 > mu2 ? C_2D : 0u);
        else
            cand2 = (a2 > rules.obj_2d_min && a3 < rules.obj_3d_max) ? C_2D : (C_2D | C_3D);
        // fusion (Sec. 4.4): intersection, falling back to the semantic proposal when empty;
        // patches without a semantic proposal are dropped
        uint32_t fin = cand2 & cand1;
        if (fin == 0u) fin = cand2;
        mask2d[(size_t)b * P + p] = (uint8_t)(fin & C_2D ? 1 : 0);
        mask3d[(size_t)b * P + p] = (uint8_t)(fin & C_3D ? 1 : 0);
        if (sem) sem[(size_t)b * P + p] = (uint8_t)l;
        kept += (fin & 1u) + (fin >> 1);
    }
    double z[3] = {0.0, 0.0, 0.0};
    block_sum3(z, kept, false, sh, 1);
    if (tid == 0) kept_len[b] = (int)kept + n_text;
}

// ---------------------------------------------------------------------------
// The same on sorted scores, for up to 8192 patches.  Labels of sorted scores are three runs, so an assignment is two
// boundaries, found 64 ways at a time by one wave, and the sums of a run are differences of prefix sums: an
// iteration costs the same few LDS round trips and one division whatever the patch count, and its barriers are gone.
// (The scores are fp32 and the sums fp64: exact, and so the same in any order, unless scores of one sample differ
// by more than 2^15; then their last bits may differ.  Final labels are taken score by score with the
// centres of the last assignment.)
// Bound by latency: the sort (bitonic, E keys a thread, on the vector unit within a wave and through LDS across
// waves), then 0.3 to 0.7 us an iteration.  64 patches 6.1 -> 3.5 us, 256 (B = 4) 15.2 -> 9.6, 1024 28.4 -> 12.9, 4096
// (B = 8) 88 -> 33.  (Beyond 8192 the prefix sums and the keys no longer fit: candidate_kernel.)
// ---------------------------------------------------------------------------
// value of lane xor D, or (16, 32) any value that leaves the pair {own, other} the same
template <int D>
__device__ __forceinline__ void lane_pair(uint32_t x, uint32_t& a, uint32_t& b) {
    a = x;
    if (D == 1) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);        // quad_perm 1,0,3,2
    else if (D == 2) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false);   // quad_perm 2,3,0,1
    else if (D == 4) b = (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x101F);                     // xor 4
    else if (D == 8) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false);  // row_ror:8
    else if (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    }
}
// one step of the bitonic network between lanes D apart, all E keys of a thread
template <int E, int D>
__device__ __forceinline__ void sort_lanes(uint32_t (&key)[E], bool keep_min) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        uint32_t a, b;
        lane_pair<D>(key[e], a, b);
        const uint32_t mn = min(a, b), mx = max(a, b);
        key[e] = keep_min ? mn : mx;
    }
}
// ascending over NT * E keys, thread t holds positions t*E .. t*E+E-1; buf: LDS of NT * E words
template <int NT, int E>
__device__ __forceinline__ void sort_keys(uint32_t (&key)[E], uint32_t* buf) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 2; k <= NT * E; k <<= 1) {
        // a run of k ascends where bit k of the position is clear
#pragma unroll
        for (int j = k >> 1; j >= E; j >>= 1) {
            const int d = j / E;
            const bool keep_min = ((tid & d) == 0) == (((tid * E) & k) == 0);
            switch (d) {
                case 1: sort_lanes<E, 1>(key, keep_min); break;
                case 2: sort_lanes<E, 2>(key, keep_min); break;
                case 4: sort_lanes<E, 4>(key, keep_min); break;
                case 8: sort_lanes<E, 8>(key, keep_min); break;
                case 16: sort_lanes<E, 16>(key, keep_min); break;
                case 32: sort_lanes<E, 32>(key, keep_min); break;
                default: {           // other waves
                    __syncthreads();
#pragma unroll
                    for (int e = 0; e < E; ++e) buf[e * NT + tid] = key[e];
                    __syncthreads();
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const uint32_t o = buf[e * NT + (tid ^ d)];
                        key[e] = keep_min ? min(key[e], o) : max(key[e], o);
                    }
                }
            }
        }
#pragma unroll
        for (int j = E >> 1; j >= 1; j >>= 1) {
            if (j >= k) continue;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e & j) continue;
                const bool up = ((tid * E + e) & k) == 0;
                const uint32_t mn = min(key[e], key[e | j]), mx = max(key[e], key[e | j]);
                key[e] = up ? mn : mx;
                key[e | j] = up ? mx : mn;
            }
        }
    }
}
__device__ __forceinline__ uint32_t score_key(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
// what a lane gets from another one of its row (CTRL), zero where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double x) {
    const long long v = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_scan_f64(double x) {      // inclusive
    x += dpp_or_zero<0x111, 0xf>(x);
    x += dpp_or_zero<0x112, 0xf>(x);
    x += dpp_or_zero<0x114, 0xf>(x);
    x += dpp_or_zero<0x118, 0xf>(x);
    x += dpp_or_zero<0x142, 0xa>(x);
    x += dpp_or_zero<0x143, 0xc>(x);
    return x;
}
__device__ __forceinline__ double lane_f64(double x, int lane) {
    const long long v = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// nearest centre, the lower-numbered one on equal distance
__device__ __forceinline__ int nearest_centre(double x, double c0, double c1, double c2) {
    const double d0 = fabs(x - c0), d1 = fabs(x - c1), d2 = fabs(x - c2);
    const bool one = d1 < d0;
    return d2 < (one ? d1 : d0) ? 2 : (one ? 1 : 0);
}

// The clustering score by score, as in candidate_kernel, on scores that are not all finite: those of a run are no
// difference of prefix sums (one score of -inf would make all centres NaN; here the finite ones stay objects).
// Nothing is kept in registers for it: scores are read again, a patch's previous label is worked out again from the
// previous centres.  The centres of the last assignment are left in c.
template <int NT>
__device__ __forceinline__ void cluster_scores(const float* sal_b, int P, int max_iter, double (&c)[3],
                                               double (&sums)[3][NT / 64], uint32_t (&counts)[NT / 64]) {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float lo = INFINITY, hi = -INFINITY;         // (NaN is left out)
#pragma unroll 1
    for (int p = tid; p < P; p += NT) {
        const float x = sal_b[p] + sal_b[P + p];
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if (lane == 0) {
        sums[0][wave] = (double)lo;
        sums[1][wave] = (double)hi;
    }
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < NW; ++w) {
        lo = fminf(lo, (float)sums[0][w]);
        hi = fmaxf(hi, (float)sums[1][w]);
    }
    __syncthreads();
    double next[3] = {(double)lo, 0.5 * ((double)lo + (double)hi), (double)hi};
#pragma unroll 1
    for (int it = 0; it < max_iter; ++it) {
        double s[3] = {0.0, 0.0, 0.0};
        uint32_t n01 = 0u;                       // patches of labels 0 and 1, 15 bits each
        bool changed = it == 0;
#pragma unroll 1
        for (int p = tid; p < P; p += NT) {
            const double x = (double)(sal_b[p] + sal_b[P + p]);
            const int l = nearest_centre(x, next[0], next[1], next[2]);
            if (it > 0) changed |= l != nearest_centre(x, c[0], c[1], c[2]);
#pragma unroll
            for (int j = 0; j < 3; ++j) s[j] += l == j ? x : 0.0;
            n01 += l == 0 ? 1u : (l == 1 ? 0x8000u : 0u);
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            c[j] = next[j];
            s[j] = wave_sum_f64(s[j]);
        }
        n01 = wave_sum_u32(n01);
        const bool any = __ballot(changed) != 0ull;
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 3; ++j) sums[j][wave] = s[j];
            counts[wave] = n01 | (any ? 0x80000000u : 0u);
        }
        __syncthreads();
        uint32_t n[3] = {0u, 0u, 0u}, moved = 0u;
#pragma unroll
        for (int j = 0; j < 3; ++j) s[j] = 0.0;
#pragma unroll 1
        for (int w = 0; w < NW; ++w) {
            const uint32_t v = counts[w];
            n[0] += v & 0x7FFFu;
            n[1] += (v >> 15) & 0x7FFFu;
            moved |= v >> 31;
#pragma unroll
            for (int j = 0; j < 3; ++j) s[j] += sums[j][w];
        }
        __syncthreads();                         // (read before the next assignment writes)
        if (!moved) break;
        n[2] = (uint32_t)P - n[0] - n[1];
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (n[j] > 0u) next[j] = s[j] / (double)n[j];
    }
}

template <int NT, int E>
__global__ __launch_bounds__(NT) void sorted_candidate_kernel(
    const float* __restrict__ x_hat /* [4,B,P] */, const float* __restrict__ sal /* [B,2P] */,
    const float* __restrict__ u /* [B,P] */, int B, int P, int n_text, mvla_mask_rules rules,
    uint8_t* __restrict__ mask2d, uint8_t* __restrict__ mask3d, uint8_t* __restrict__ sem,
    int32_t* __restrict__ kept_len) {
    constexpr int NW = NT / 64;
    __shared__ uint32_t sorted[NT * E];          // (keys while they are sorted, then the scores' bits)
    // sum of the scores in front of every RUN-th (each one's own where the LDS holds that)
    constexpr int RUN = NT * E <= 4096 ? 1 : E;
    __shared__ double before[NT * E / RUN + 1];
    __shared__ double wave_sums[3][NW];
    __shared__ double centres[3];
    __shared__ uint32_t counts[NW];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* sal_b = sal + (size_t)b * 2 * P;
    const float* m3_s1 = x_hat + ((size_t)1 * B + b) * P;
    const float* m2_s2 = x_hat + ((size_t)2 * B + b) * P;
    const float* m3_s2 = x_hat + ((size_t)3 * B + b) * P;
    const float* u_b = u + (size_t)b * P;

    // patch score (summand of Eq. 3) and, where registers allow it, all that the rules read, in one round trip
    constexpr bool EARLY = E <= 4;
    constexpr int KEEP = EARLY ? E : 1;
    uint32_t key[E];
    double mu2 = 0.0, mu3 = 0.0;
    float score[E], a2[KEEP], a3[KEEP], share3[KEEP], draw[KEEP];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = min(tid + e * NT, P - 1);
        score[e] = sal_b[p] + sal_b[P + p];
        if (EARLY) {
            a2[e % KEEP] = m2_s2[p];
            a3[e % KEEP] = m3_s2[p];
            share3[e % KEEP] = m3_s1[p];
            draw[e % KEEP] = u_b[p];
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = min(tid + e * NT, P - 1);
        const bool in = tid + e * NT < P;
        key[e] = in ? score_key(score[e]) : 0xFFFFFFFFu;
        mu2 += in ? (double)(EARLY ? a2[e % KEEP] : m2_s2[p]) : 0.0;
        mu3 += in ? (double)(EARLY ? a3[e % KEEP] : m3_s2[p]) : 0.0;
    }
    sort_keys<NT, E>(key, sorted);
    double mine = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) mine += tid * E + e < P ? (double)key_score(key[e]) : 0.0;
    const double incl = wave_scan_f64(mine);
    mu2 = wave_sum_f64(mu2);
    mu3 = wave_sum_f64(mu3);
    __syncthreads();                             // (the sort's last exchange has been read)
#pragma unroll
    for (int e = 0; e < E; ++e) sorted[tid * E + e] = __float_as_uint(key_score(key[e]));
    if (lane == 63) wave_sums[0][wave] = incl;
    if (lane == 0) {
        wave_sums[1][wave] = mu2;
        wave_sums[2][wave] = mu3;
    }
    __syncthreads();
    double front = 0.0, total = 0.0;
    mu2 = mu3 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        front += w < wave ? wave_sums[0][w] : 0.0;
        total += wave_sums[0][w];
        mu2 += wave_sums[1][w];
        mu3 += wave_sums[2][w];
    }
    mu2 /= (double)P;                            // baselines: means over the sample's patches (Eqs. 5, 6)
    mu3 /= (double)P;
    front += incl - mine;
    if (RUN == 1) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            before[(tid * E + e) / RUN] = front;
            front += tid * E + e < P ? (double)key_score(key[e]) : 0.0;
        }
    } else {
        before[tid] = front;
    }
    if (tid == NT - 1) before[NT * E / RUN] = total;
    __syncthreads();

    // Lloyd iterations (Sec. 4.2), as in candidate_kernel: centres start at min, mid-range, max; stop when an
    // assignment repeats the previous one or after kmeans_max_iter assignments
    if (!__builtin_isfinite(__uint_as_float(sorted[0])) || !__builtin_isfinite(__uint_as_float(sorted[P - 1]))) {
        double c[3];
        cluster_scores<NT>(sal_b, P, rules.kmeans_max_iter, c, wave_sums, counts);
        if (tid == 0)
#pragma unroll
            for (int j = 0; j < 3; ++j) centres[j] = c[j];
    } else if (wave == 0) {
        auto x = [&](int i) __attribute__((always_inline)) { return __uint_as_float(sorted[i]); };
        double c0 = (double)x(0), c2 = (double)x(P - 1), c1 = 0.5 * (c0 + c2);
        double l0 = c0, l1 = c1, l2 = c2;        // centres of the last assignment
        int was0 = -1, was01 = -1;               // its runs: labels 0, and 0 or 1
        for (int it = 0; it < rules.kmeans_max_iter; ++it) {
            l0 = c0;
            l1 = c1;
            l2 = c2;
            int n0, n01;
            if (NT == 64) {                      // every lane has its scores at hand: count labels
                n0 = n01 = 0;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int l = nearest_centre((double)key_score(key[e]), c0, c1, c2);
                    const bool in = tid * E + e < P;
                    n0 += __popcll(__ballot(in && l == 0));
                    n01 += __popcll(__ballot(in && l != 2));
                }
            } else {
                // first position of a label above 0 in [r0, r0 + len), of label 2 in [r1, r1 + len) (P for none):
                // all lanes look for both while the ranges are one, half of them for each afterwards
                int len = (P + 63) >> 6, r0, r1;
                {
                    const int at = min((lane + 1) * len, P) - 1;
                    const int l = nearest_centre((double)x(at), c0, c1, c2);
                    const unsigned long long m0 = __ballot(l >= 1), m1 = __ballot(l == 2);
                    r0 = m0 ? (__ffsll((long long)m0) - 1) * len : P;
                    r1 = m1 ? (__ffsll((long long)m1) - 1) * len : P;
                }
                while (len > 1) {
                    const int step = (len + 31) >> 5, from = lane < 32 ? r0 : r1;
                    const int at = min(min(from + ((lane & 31) + 1) * step, from + len), P) - 1;
                    const int l = nearest_centre((double)x(at), c0, c1, c2);
                    const unsigned long long m = __ballot(lane < 32 ? l >= 1 : l == 2);
                    const uint32_t m0 = (uint32_t)m, m1 = (uint32_t)(m >> 32);
                    if (r0 < P) r0 += m0 ? (__ffs((int)m0) - 1) * step : 0;
                    if (r1 < P) r1 += m1 ? (__ffs((int)m1) - 1) * step : 0;
                    len = step;
                }
                n0 = r0;
                n01 = max(r0, r1);
            }
            if (n0 == was0 && n01 == was01) break;
            was0 = n0;
            was01 = n01;
            // lanes 0, 1 and 2 (and on): the mean of run 0, 1 and 2, from the sums up to its end and its start
            auto up_to = [&](int end) __attribute__((always_inline)) {
                const int t = end / RUN;
                double sum = before[t];
                if (RUN > 1) {
                    float v[RUN];
#pragma unroll
                    for (int e = 0; e < RUN; ++e) v[e] = x(min(t * RUN + e, NT * E - 1));
#pragma unroll
                    for (int e = 0; e < RUN; ++e) sum += t * RUN + e < end ? (double)v[e] : 0.0;
                }
                return sum;
            };
            const int end = lane == 0 ? n0 : lane == 1 ? n01 : P, start = lane == 0 ? 0 : lane == 1 ? n0 : n01;
            const double run = up_to(end) - up_to(start), mean = run / (double)max(end - start, 1);
            if (n0 > 0) c0 = lane_f64(mean, 0);
            if (n01 > n0) c1 = lane_f64(mean, 1);
            if (P > n01) c2 = lane_f64(mean, 2);
        }
        if (lane == 0) {
            centres[0] = l0;
            centres[1] = l1;
            centres[2] = l2;
        }
    }
    __syncthreads();
    const double c0 = centres[0], c1 = centres[1], c2 = centres[2];

    uint32_t kept = 0u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = tid + e * NT;
        if (p < P) {
            // data-preprocessing stage (Sec. 4.1), semantic stage (Sec. 4.2) and fusion (Sec. 4.4): see candidate_kernel
            const float s3 = EARLY ? share3[e % KEEP] : m3_s1[p];
            const float v2 = EARLY ? a2[e % KEEP] : m2_s2[p], v3 = EARLY ? a3[e % KEEP] : m3_s2[p];
            const uint32_t cand1 = s3 < rules.tau_2d ? C_2D : (s3 > rules.tau_3d ? C_3D : C_2D | C_3D);
            const int l = nearest_centre((double)score[e], c0, c1, c2);
            uint32_t cand2;
            if (l == 0)
                cand2 = (EARLY ? draw[e % KEEP] : u_b[p]) < rules.bg_drop ? 0u : (C_2D | C_3D);
            else if (l == 1)
                cand2 = (double)v3 > mu3 ? (C_2D | C_3D) : ((double)v2 > mu2 ? C_2D : 0u);
            else
                cand2 = (v2 > rules.obj_2d_min && v3 < rules.obj_3d_max) ? C_2D : (C_2D | C_3D);
            uint32_t fin = cand2 & cand1;
            if (fin == 0u) fin = cand2;
            mask2d[(size_t)b * P + p] = (uint8_t)(fin & C_2D ? 1 : 0);
            mask3d[(size_t)b * P + p] = (uint8_t)(fin & C_3D ? 1 : 0);
            if (sem) sem[(size_t)b * P + p] = (uint8_t)l;
            kept += (fin & 1u) + (fin >> 1);
        }
    }
    kept = wave_sum_u32(kept);
    if (lane == 0) counts[wave] = kept;
    __syncthreads();
    if (tid == 0) {
        uint32_t n = 0u;
#pragma unroll
        for (int w = 0; w < NW; ++w) n += counts[w];
        kept_len[b] = (int)n + n_text;
    }
}

int launch_candidate_masks(const float* x_hat, const float* sal, const float* u, int B, int P,
                           int n_text, const mvla_mask_rules& rules, uint8_t* mask2d,
                           uint8_t* mask3d, uint8_t* sem, int32_t* kept_len, hipStream_t st) {
#define MVLA_SORTED(NT, E)                                                                              \
    hipLaunchKernelGGL((sorted_candidate_kernel<NT, E>), dim3(B), dim3(NT), 0, st, x_hat, sal, u, B, P, n_text, rules, \
                       mask2d, mask3d, sem, kept_len);                                                  \
    MVLA_HIP_CHECK(hipGetLastError());                                                                  \
    return MVLA_OK
    if (P <= 64) { MVLA_SORTED(64, 1); }
    if (P <= 128) { MVLA_SORTED(64, 2); }
    if (P <= 256) { MVLA_SORTED(64, 4); }
    if (P <= 512) { MVLA_SORTED(128, 4); }
    if (P <= 1024) { MVLA_SORTED(256, 4); }
    if (P <= 2048) { MVLA_SORTED(512, 4); }
    if (P <= 4096) { MVLA_SORTED(512, 8); }
    if (P <= 8192) { MVLA_SORTED(1024, 8); }
#undef MVLA_SORTED
    const size_t lds = (size_t)P * 4 + (((size_t)P + 3) & ~(size_t)3);
    hipLaunchKernelGGL(candidate_kernel, dim3(B), dim3(CM_THREADS), lds, st, x_hat, sal, u, B, P,
                       n_text, rules, mask2d, mask3d, sem, kept_len);
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

// ---------------------------------------------------------------------------
// Masks -> ascending token indices (Eq. 10): kept 2D tokens, kept 3D tokens
// (offset by the patch count), all language tokens; the rest of the row up to
// S_pad repeats the last language token's index.  One workgroup per sample;
// a wave owns a contiguous run of the 2P flags, reads them 64 side by side, eight such
// reads in flight, and places its tokens by ballots behind the counts of the waves before it.
// (256 patches 2.8 us, as a thread for each run of flags, a byte after the other; 1024 4.4 -> 3.0,
// 4096 13.0 -> 4.4, B = 4 and 8.)
// ---------------------------------------------------------------------------
template <int NT, int U /* reads in flight */>
__global__ __launch_bounds__(NT) void mask_index_kernel(
    const uint8_t* __restrict__ mask2d, const uint8_t* __restrict__ mask3d, int P, int n_text,
    int S_pad, int32_t* __restrict__ kept_idx) {
    constexpr int NW = NT / 64;
    __shared__ uint32_t counts[NW];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = 2 * P, per = (n + NT - 1) / NT * 64;
    const int i0 = min(wave * per, n), i1 = min(i0 + per, n);
    const uint8_t* m2 = mask2d + (size_t)b * P;
    const uint8_t* m3 = mask3d + (size_t)b * P;
    // ballots of U times 64 flags from i on (none beyond this wave's run)
    auto flags = [&](int i, unsigned long long (&kept)[U]) __attribute__((always_inline)) {
        uint8_t f[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int at = min(i + k * 64 + lane, n - 1);
            f[k] = at < P ? m2[at] : m3[at - P];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) kept[k] = __ballot(f[k] != 0 && i + k * 64 + lane < i1);
    };
    uint32_t mine = 0u;
    unsigned long long kept[U];
    const bool once = per <= U * 64;     // the run is one batch: its ballots are kept
    for (int i = i0; i < i1; i += U * 64) {
        flags(i, kept);
#pragma unroll
        for (int k = 0; k < U; ++k) mine += (uint32_t)__popcll(kept[k]);
    }
    if (lane == 0) counts[wave] = mine;
    __syncthreads();
    uint32_t before = 0u, total = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        before += w < wave ? counts[w] : 0u;
        total += counts[w];
    }
    int32_t* out = kept_idx + (size_t)b * S_pad;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int i = i0; i < i1; i += U * 64) {
        if (!once) flags(i, kept);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t slot = before + (uint32_t)__popcll(kept[k] & below);
            if (((kept[k] >> lane) & 1ull) && slot < (uint32_t)S_pad) out[slot] = i + k * 64 + lane;
            before += (uint32_t)__popcll(kept[k]);
        }
    }
    const int len = (int)total + n_text;
    for (int j = (int)total + tid; j < S_pad; j += NT)
        out[j] = j < len ? n + (j - (int)total) : n + n_text - 1;
}

int launch_mask_indices(const uint8_t* mask2d, const uint8_t* mask3d, int B, int P, int n_text,
                        int S_pad, int32_t* kept_idx, hipStream_t st) {
    // as few threads and reads as take the flags in one batch a wave; sixteen waves of eight beyond
#define MVLA_MASK_INDEX(NT, U)                                                                         \
    hipLaunchKernelGGL((mask_index_kernel<NT, U>), dim3(B), dim3(NT), 0, st, mask2d, mask3d, P, n_text, S_pad, kept_idx)
    if (2 * P <= 256) MVLA_MASK_INDEX(256, 1);
    else if (2 * P <= 512) MVLA_MASK_INDEX(256, 2);
    else if (2 * P <= 2048) MVLA_MASK_INDEX(512, 4);
    else MVLA_MASK_INDEX(1024, 8);
#undef MVLA_MASK_INDEX
    MVLA_HIP_CHECK(hipGetLastError());
    return MVLA_OK;
}

}  // namespace mvla
