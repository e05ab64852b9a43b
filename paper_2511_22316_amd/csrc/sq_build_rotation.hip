// sq_build_rotation: the closed-form construction of the rotation from calibration activations
// (Sec. 4.2: ART with the angle of Lemma 1, URT, the Hadamard factor, the composition of "The
// Overall SingleQuant Method"), and sq_kron_factor (Alg. 1).
//
// One pass over the calibration activations finds the calibration row (HBM-bound, the only part
// that touches more than a few hundred KB); everything after it is small and runs in a handful
// of tiny launches:
//   row_absmax_kernel     max |x| of every token row
//   art_urt_kernel        one workgroup: calibration row, P ART steps, the vectors of the two URTs,
//                         their uniform targets, and the four chains of plane rotations
//   urt_columns_kernel    R^U = R_map R'_map^T, eight columns per workgroup, the maps to e_1 entry by entry in
//                         closed form: side 1 is R1, side 2 goes through the Hadamard factor, R2 = H R^U_2
//
// Wherever floating point decides an index -- the ART channels and the rank order of the URT --
// the deciding values (the calibration vector as the ART steps rewrite it, the means, the Hadamard
// image) are kept and compared in fp64: the paper defines these choices over the reals, and at
// fp64 only values that agree to about fifteen digits could be ordered differently from that.
// The matrices that follow the decisions are fp32.
#include "sq_common.h"

#include <math.h>

namespace sq {

namespace {

constexpr int kBuildThreads = 1024;
constexpr int kBuildWaves = kBuildThreads / kWave;
constexpr int kMaxSide = 256;                 // n1 <= 128, n2 <= 256
static_assert(kBuildThreads == 4 * kMaxSide, "one thread per step of each of the four chains");
static_assert(SQ_MAX_N1 <= kMaxSide && SQ_MAX_N2 <= kMaxSide && SQ_MAX_GIVENS <= kBuildThreads, "limits");
// reduction slots (two sets of three words per wave), five small fp64 vectors, the ART pairs
constexpr int kBuildSmallBytes = 6 * kBuildWaves * 4 + 5 * kMaxSide * 8 + 2 * SQ_MAX_GIVENS * 8;
// ART candidates: the 2 P largest and the 2 P smallest channels of the calibration row
constexpr int kMaxCandidates = 4 * SQ_MAX_GIVENS;
static_assert(kMaxCandidates == 4 * kWave, "one wave holds them, four per lane");
// two histograms of 256 bins, the candidates' channels, one count per wave, results of the two searches, a counter
constexpr int kSelectWords = 2 * 256 + kMaxCandidates + kBuildWaves + 4 + 2;
static_assert(kBuildSmallBytes % 8 == 0, "the fp64 vectors behind the slots are 8-byte aligned");

// workspace, in floats
struct BuildWorkspace {
    float *rowmax;      // [T]
    float *chain;       // [side 0..1][vector V, U][cos, sin][kMaxSide]
};

// (the size is part of the interface; what follows the chain is not used)
__host__ int64_t build_workspace_floats(int64_t T, int n1, int n2)
{
    const int64_t t_pad = (T + 63) / 64 * 64;
    return t_pad + 8 * kMaxSide + 2 * (int64_t)n1 * n1 + 3 * (int64_t)n2 * n2;
}

__host__ BuildWorkspace carve_workspace(void *workspace, int64_t T)
{
    BuildWorkspace w;
    float *p = static_cast<float *>(workspace);
    w.rowmax = p;
    p += (T + 63) / 64 * 64;
    w.chain = p;
    return w;
}

typedef unsigned short v2us __attribute__((ext_vector_type(2)));

// max |x| per token row.  One wave per row; a lane reads 16 bytes at a time, four loads in
// flight.  |fp16| bit patterns order like unsigned integers, so the maximum is taken on the
// masked 16-bit patterns, two per instruction, and converted once at the end.
__global__ __launch_bounds__(256) void row_absmax_kernel(const __half *__restrict__ X, int64_t ldx, int T, int K,
                                                         float *__restrict__ rowmax)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int chunks = K / 8;
    for (int t = blockIdx.x * 4 + wave; t < T; t += gridDim.x * 4) {
        const uint4 *row = reinterpret_cast<const uint4 *>(X + (int64_t)t * ldx);
        v2us m = {0, 0};
        for (int c0 = 0; c0 < chunks; c0 += 4 * kWave) {
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * kWave + lane;
                v[u] = (c < chunks) ? row[c] : uint4{0, 0, 0, 0};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    m = __builtin_elementwise_max(m, __builtin_bit_cast(v2us, w[e] & 0x7FFF7FFFu));
            }
        }
        const unsigned short top = m[0] > m[1] ? m[0] : m[1];
        const float f = wave_max(__half2float(__ushort_as_half(top)));
        if (lane == 0) rowmax[t] = f;
    }
}

// Largest (or smallest) 32-bit unsigned value of the wave, in every lane.  DPP steps as in
// wave_max; lanes a step does not write keep the identity of the operation.
template <bool LARGEST>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v)
{
    constexpr int kIdentity = LARGEST ? 0 : -1;
#define SQ_DPP_STEP(ctrl, row_mask)                                                                  \
    do {                                                                                             \
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(kIdentity, (int)v, ctrl, row_mask, 0xF, false); \
        v = LARGEST ? (o > v ? o : v) : (o < v ? o : v);                                             \
    } while (0)
    SQ_DPP_STEP(0xB1, 0xF);     // quad_perm [1,0,3,2]
    SQ_DPP_STEP(0x4E, 0xF);     // quad_perm [2,3,0,1]
    SQ_DPP_STEP(0x141, 0xF);    // row_half_mirror
    SQ_DPP_STEP(0x140, 0xF);    // row_mirror: every lane holds the result of its row of 16
    SQ_DPP_STEP(0x142, 0xA);    // row_bcast:15 into rows 1 and 3
    SQ_DPP_STEP(0x143, 0xC);    // row_bcast:31 into rows 2 and 3: lane 63 holds the wave's result
#undef SQ_DPP_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Index of the largest (or smallest) 64-bit key (hi, lo) in the workgroup, the lowest index among
// equal keys; every thread passes the best (key, index) of its own elements and gets the result.
// Magnitudes of finite fp64 (and fp32) values order like their bit patterns read as unsigned
// integers.  `slots` ([3][kBuildWaves] words) must not be rewritten before every thread has passed
// a later barrier.
template <bool LARGEST>
__device__ __forceinline__ uint32_t wave_arg(uint32_t hi, uint32_t lo, uint32_t idx, uint32_t &best_hi,
                                             uint32_t &best_lo)
{
    constexpr uint32_t kNone = LARGEST ? 0u : 0xFFFFFFFFu;
    best_hi = wave_extreme<LARGEST>(hi);
    best_lo = wave_extreme<LARGEST>(hi == best_hi ? lo : kNone);
    return wave_extreme<false>((hi == best_hi && lo == best_lo) ? idx : 0xFFFFFFFFu);
}

template <bool LARGEST>
__device__ __forceinline__ uint32_t block_arg(uint32_t hi, uint32_t lo, uint32_t idx, uint32_t *slots)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    constexpr uint32_t kNone = LARGEST ? 0u : 0xFFFFFFFFu;
    uint32_t bh, bl;
    const uint32_t who = wave_arg<LARGEST>(hi, lo, idx, bh, bl);
    if (lane == 0) {
        slots[wave] = bh;
        slots[kBuildWaves + wave] = bl;
        slots[2 * kBuildWaves + wave] = who;
    }
    __syncthreads();
    // every wave combines the per-wave results on its own; a wave whose threads had no element
    // passes index 0xFFFFFFFF and never wins against one that had
    const bool in = lane < kBuildWaves;
    const uint32_t i2 = in ? slots[2 * kBuildWaves + lane] : 0xFFFFFFFFu;
    const bool has = i2 != 0xFFFFFFFFu;
    return wave_arg<LARGEST>(has ? slots[lane] : kNone, has ? slots[kBuildWaves + lane] : kNone, i2, bh, bl);
}

// The same over one wave: every lane passes its best key as two halves and its channel, and gets the key too.  Nearly always
// a few lanes at most hold the extreme upper half, and those are looked at one by one.
template <bool LARGEST>
__device__ __forceinline__ uint32_t wave_arg_short(uint32_t hi, uint32_t lo, uint32_t idx, uint32_t &best_hi,
                                                   uint32_t &best_lo)
{
    best_hi = wave_extreme<LARGEST>(hi);
    uint64_t holders = __ballot(hi == best_hi);
    if (__popcll(holders) > 4) return wave_arg<LARGEST>(hi, lo, idx, best_hi, best_lo);
    uint32_t who = 0xFFFFFFFFu;
    best_lo = LARGEST ? 0u : 0xFFFFFFFFu;
    do {
        const int l = __ffsll((unsigned long long)holders) - 1;
        const uint32_t lo_l = (uint32_t)__builtin_amdgcn_readlane((int)lo, l), idx_l = (uint32_t)__builtin_amdgcn_readlane((int)idx, l);
        if ((LARGEST ? lo_l > best_lo : lo_l < best_lo) || (lo_l == best_lo && idx_l < who)) best_lo = lo_l, who = idx_l;
        holders &= holders - 1;
    } while (holders != 0);
    return who;
}

// One wave: the bin of a histogram of 4 * 64 bins in which the running count, from the last bin down (DOWN) or from the
// first up, reaches `target` (1 .. sum of all bins); `before`: the count in front of that bin.
template <bool DOWN>
__device__ __forceinline__ int bin_reaching(const uint32_t *hist, uint32_t target, uint32_t &before)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t n[4], sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) sum += n[u] = hist[DOWN ? 255 - (4 * lane + u) : 4 * lane + u];
    uint32_t upto = sum;
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) {
        const uint32_t o = __shfl_up(upto, d);
        if (lane >= d) upto += o;
    }
    uint32_t run = upto - sum;
    const int owner = __ffsll((unsigned long long)__ballot(run < target && target <= upto)) - 1;
    int bin = 4 * lane;
#pragma unroll
    for (int u = 0; u < 3; ++u)
        if (bin == 4 * lane + u && run + n[u] < target) run += n[u], ++bin;
    before = __shfl(run, owner);
    bin = __shfl(bin, owner);
    return DOWN ? 255 - bin : bin;
}

__device__ __forceinline__ void magnitude_key(double v, uint32_t &hi, uint32_t &lo)
{
    const uint64_t bits = (uint64_t)__double_as_longlong(fabs(v));
    hi = (uint32_t)(bits >> 32);
    lo = (uint32_t)bits;
}

// Step k of the Givens chain that takes `vec` (n entries) to ||vec|| e_1: entry k is zeroed by a
// rotation in the plane (k - 1, k), k = n - 1 down to 1.  When step k acts, entry k holds the norm
// of the original entries k .. n-1, so with S_k the sum of their squares
//   cos_k = v_{k-1} / sqrt(S_{k-1}),   sin_k = sqrt(S_k / S_{k-1})     (cos = 1, sin = 0 if S_{k-1} = 0;
//   sin_{n-1} = v_{n-1} / sqrt(S_{n-2}), because the last entry enters with its sign)
// and the steps can be computed independently of one another.  Stored at cs[k], cs[kMaxSide + k].
__device__ __forceinline__ void chain_step(const double *vec, int n, int k, float *cs)
{
    double tail = 0.0;
    // (every thread reads every entry, eight at a time, rather than each its own number of them one after another)
#pragma unroll 8
    for (int m = n - 1; m >= 1; --m) {
        const double o = vec[m];
        tail += m >= k ? o * o : 0.0;
    }
    const double x = vec[k - 1], all = tail + x * x;
    cs[k] = (all == 0.0) ? 1.f : (float)(x / sqrt(all));
    // the first step (k = n-1) meets the last entry itself, sign included; later ones meet a norm
    cs[kMaxSide + k] = (all == 0.0) ? 0.f : (float)(k == n - 1 ? vec[k] / sqrt(all) : sqrt(tail / all));
}

// One workgroup.  All of its LDS is dynamic (kBuildSmallBytes + 8 (K + n1) + 4 kSelectWords bytes): the reduction slots,
// the small vectors, the calibration vector in fp64 (its rows of n2 entries one apart, so that the threads that
// sum a row each read different banks), and what the choice of the ART candidates needs.
//
// What bounds it is the chain of P dependent ART steps.  Step p (from 0) has at most 2 p channels rewritten by the steps
// before it, so what it picks is one of those or among the first 2 p + 1 in order of the calibration row as it was:
// the 2 P largest and the 2 P smallest channels are all that can ever be chosen.  A radix selection on the
// 15-bit magnitudes (two histograms of 256 bins, ties by channel) finds them, and one wave then holds them in registers
// and takes the steps without a barrier, 0.73 us each.  T = 2048, K = 4096, P = 32: 91.5 -> 41.5 us against a
// reduction over all channels by the whole workgroup in every step.
// BY_ALL: that reduction instead, which is faster for few steps over few channels (steps_by_all).
template <bool BY_ALL>
__global__ __launch_bounds__(kBuildThreads) void art_urt_kernel(
    const __half *__restrict__ X, int64_t ldx, int T, int K, int n1, int n2, int P, double inv_sqrt_n2,
    const float *__restrict__ rowmax, int32_t *__restrict__ giv_i, int32_t *__restrict__ giv_j,
    float *__restrict__ giv_theta, float *__restrict__ chain)
{
    extern __shared__ uint32_t build_lds[];
    uint32_t *slots_a = build_lds, *slots_b = build_lds + 3 * kBuildWaves;
    double(*vec)[kMaxSide] = reinterpret_cast<double(*)[kMaxSide]>(build_lds + 6 * kBuildWaves);   // V1 | V2 H
    double *v2 = vec[2];
    double(*target)[kMaxSide] = reinterpret_cast<double(*)[kMaxSide]>(vec[3]);                     // U1 | U2
    double *pair_a = vec[5], *pair_b = pair_a + SQ_MAX_GIVENS;     // (c_i, c_j) each ART angle is made for
    double *cvec = pair_b + SQ_MAX_GIVENS;
    uint32_t *hist = reinterpret_cast<uint32_t *>(cvec + K + n1);  // [2][256]
    uint32_t *cand = hist + 2 * 256;                               // [kMaxCandidates]
    uint32_t *wave_ties = cand + kMaxCandidates;                   // [kBuildWaves]
    uint32_t *found = wave_ties + kBuildWaves;                     // bin and count before it, from above and from below
    uint32_t *n_cand = found + 4;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int n2_log = 31 - __clz(n2);                             // n2 is a power of two
    auto at = [n2_log](int k) { return k + (k >> n2_log); };

    // calibration row: the largest row maximum, lowest row among equals
    uint32_t top = 0, top_at = 0xFFFFFFFFu;
    for (int t = tid; t < T; t += kBuildThreads) {
        const uint32_t m = __float_as_uint(rowmax[t]);
        if (m > top || top_at == 0xFFFFFFFFu) top = m, top_at = (uint32_t)t;      // t ascends: ties keep the lower row
    }
    if (tid < 2 * 256) hist[tid] = 0;
    if (tid == 0) *n_cand = 0;
    const int t_star = (int)block_arg<true>(top, 0u, top_at, slots_a);

    // Thread tid takes the channels [tid per, (tid + 1) per).
    constexpr int kMost = SQ_MAX_K / kBuildThreads;
    static_assert(kMost * kBuildThreads == SQ_MAX_K, "every channel has a thread");
    const int per = (K + kBuildThreads - 1) / kBuildThreads, k0 = tid * per;
    uint32_t key[kMost];                                           // 15-bit magnitudes; 0xFFFF: no channel
#pragma unroll
    for (int e = 0; e < kMost; ++e) {
        const bool in = e < per && k0 + e < K;
        const __half h = in ? X[(int64_t)t_star * ldx + k0 + e] : __float2half(0.f);
        key[e] = in ? (__half_as_ushort(h) & 0x7FFFu) : 0xFFFFu;
        if (in) cvec[at(k0 + e)] = (double)__half2float(h);
    }
    if (P > 0 && !BY_ALL && K <= kMaxCandidates) {
        if (tid < K) cand[tid] = (uint32_t)tid;
        if (tid == 0) *n_cand = (uint32_t)K;
    } else if (P > 0 && !BY_ALL) {
        const uint32_t wanted = 2 * (uint32_t)P;
#pragma unroll
        for (int e = 0; e < kMost; ++e)
            if (key[e] != 0xFFFFu) atomicAdd(&hist[key[e] >> 7], 1u);
        __syncthreads();
        uint32_t before;
        if (wave == 0) {
            const int b = bin_reaching<true>(hist, wanted, before);
            if (lane == 0) found[0] = (uint32_t)b, found[1] = before;
        } else if (wave == 1) {
            const int b = bin_reaching<false>(hist, wanted, before);
            if (lane == 0) found[2] = (uint32_t)b, found[3] = before;
        }
        __syncthreads();
        const uint32_t bin_hi = found[0], bin_lo = found[2], want_hi = wanted - found[1], want_lo = wanted - found[3];
        if (tid < 2 * 256) hist[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kMost; ++e) {
            if (key[e] == 0xFFFFu) continue;
            if ((key[e] >> 7) == bin_hi) atomicAdd(&hist[key[e] & 127], 1u);
            if ((key[e] >> 7) == bin_lo) atomicAdd(&hist[256 + (key[e] & 127)], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            const int b = bin_reaching<true>(hist, want_hi, before);
            if (lane == 0) found[0] = (uint32_t)b, found[1] = before;
        } else if (wave == 1) {
            const int b = bin_reaching<false>(hist + 256, want_lo, before);
            if (lane == 0) found[2] = (uint32_t)b, found[3] = before;
        }
        __syncthreads();
        // everything beyond the two magnitudes found, and of the channels that hold one of them the lowest
        const uint32_t key_hi = (bin_hi << 7) | found[0], key_lo = (bin_lo << 7) | found[2];
        const uint32_t ties_hi = want_hi - found[1], ties_lo = want_lo - found[3];
        uint32_t mine = 0;                                         // this thread's channels at them: 16 bits each
#pragma unroll
        for (int e = 0; e < kMost; ++e) mine += (key[e] == key_hi ? 1u : 0u) + (key[e] == key_lo ? 1u << 16 : 0u);
        uint32_t upto = mine;
#pragma unroll
        for (int d = 1; d < kWave; d *= 2) {
            const uint32_t o = __shfl_up(upto, d);
            if (lane >= d) upto += o;
        }
        if (lane == kWave - 1) wave_ties[wave] = upto;
        __syncthreads();
        uint32_t rank = upto - mine;
        for (int w = 0; w < wave; ++w) rank += wave_ties[w];
        uint32_t rank_hi = rank & 0xFFFFu, rank_lo = rank >> 16;
#pragma unroll
        for (int e = 0; e < kMost; ++e) {
            if (key[e] == 0xFFFFu) continue;
            bool take = key[e] > key_hi || key[e] < key_lo;
            if (key[e] == key_hi) take |= rank_hi++ < ties_hi;
            if (key[e] == key_lo) take |= rank_lo++ < ties_lo;
            if (take) cand[atomicAdd(n_cand, 1u)] = (uint32_t)(k0 + e);
        }
    }
    __syncthreads();

    // ART (Sec. 4.2; several steps as in the "ART steps" study): largest against smallest
    // magnitude, angle of Lemma 1, after which both channels hold r / sqrt(2)
    if constexpr (BY_ALL) {
        for (int p = 0; p < P; ++p) {
            // k ascends within a thread, so strict comparisons keep the lower channel among equals
            uint32_t hi_h = 0, hi_l = 0, hi_at = 0xFFFFFFFFu, lo_h = 0xFFFFFFFFu, lo_l = 0xFFFFFFFFu, lo_at = 0xFFFFFFFFu;
            for (int k = tid; k < K; k += kBuildThreads) {
                uint32_t h, l;
                magnitude_key(cvec[at(k)], h, l);
                if (hi_at == 0xFFFFFFFFu || h > hi_h || (h == hi_h && l > hi_l)) hi_h = h, hi_l = l, hi_at = (uint32_t)k;
            }
            const int i = (int)block_arg<true>(hi_h, hi_l, hi_at, slots_a);
            for (int k = tid; k < K; k += kBuildThreads) {
                uint32_t h, l;
                magnitude_key(cvec[at(k)], h, l);
                if (k != i && (lo_at == 0xFFFFFFFFu || h < lo_h || (h == lo_h && l < lo_l)))
                    lo_h = h, lo_l = l, lo_at = (uint32_t)k;
            }
            const int j = (int)block_arg<false>(lo_h, lo_l, lo_at, slots_b);
            if (tid == 0) {
                const double a = cvec[at(i)], b = cvec[at(j)];
                const double e = sqrt(a * a + b * b) * 0.70710678118654752440;
                giv_i[p] = i;
                giv_j[p] = j;
                pair_a[p] = a;
                pair_b[p] = b;
                cvec[at(i)] = cvec[at(j)] = e;
            }
            __syncthreads();
        }
    } else if (wave == 0 && P > 0) {
        // This lane's candidates by channel, their magnitudes as integers; no channel: zero among the largest, all
        // ones among the smallest.
        uint32_t idx[4];
        uint64_t large[4], small[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) idx[u] = (uint32_t)(lane + 64 * u) < *n_cand ? cand[lane + 64 * u] : 0xFFFFFFFFu;
        auto order = [&](int x, int y) {
            const uint32_t lower = min(idx[x], idx[y]), upper = max(idx[x], idx[y]);
            idx[x] = lower, idx[y] = upper;
        };
        order(0, 1), order(2, 3), order(0, 2), order(1, 3), order(1, 2);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = idx[u] != 0xFFFFFFFFu;
            const uint64_t mag = (uint64_t)__double_as_longlong(fabs(in ? cvec[at((int)idx[u])] : 0.0));
            large[u] = mag;
            small[u] = in ? mag : ~(uint64_t)0;
        }
        auto smallest_but = [&](uint32_t skip, uint32_t &hi, uint32_t &lo) {
            uint64_t best = ~(uint64_t)0;
            uint32_t who = 0xFFFFFFFFu;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (small[u] < best && idx[u] != skip) best = small[u], who = idx[u];
            return wave_arg_short<false>((uint32_t)(best >> 32), (uint32_t)best, who, hi, lo);
        };
        auto value = [](uint32_t hi, uint32_t lo) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); };
        for (int p = 0; p < P; ++p) {
            uint64_t best = large[0];
            uint32_t who = idx[0], ah, al, bh, bl;
#pragma unroll
            for (int u = 1; u < 4; ++u)
                if (large[u] > best) best = large[u], who = idx[u];
            const uint32_t i = wave_arg_short<true>((uint32_t)(best >> 32), (uint32_t)best, who, ah, al);
            uint32_t j = smallest_but(0xFFFFFFFFu, bh, bl);
            if (j == i) j = smallest_but(i, bh, bl);   // every magnitude the same
            const double a = value(ah, al), b = value(bh, bl);
            const double e = sqrt(a * a + b * b) * 0.70710678118654752440;
            if (lane == 0) {                           // beside the chain: the LDS traffic of a wave is in order
                giv_i[p] = (int)i;
                giv_j[p] = (int)j;
                pair_a[p] = cvec[at((int)i)];
                pair_b[p] = cvec[at((int)j)];
                cvec[at((int)i)] = e;
                cvec[at((int)j)] = e;
            }
            const uint64_t mag = (uint64_t)__double_as_longlong(e);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (idx[u] == i || idx[u] == j) large[u] = mag, small[u] = mag;
        }
    }
    __syncthreads();

    // vectors of the two URTs: means of the n1 x n2 view over the other dimension; the second one
    // goes through the Hadamard matrix first, because H acts first in R2
    if (tid < n1) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < n2; ++q) s += cvec[at(tid * n2) + q];
        vec[0][tid] = s / (double)n2;
    }
    if (tid >= 512 && tid - 512 < n2) {
        const int q = tid - 512;
        double s = 0.0;
#pragma unroll 8
        for (int pp = 0; pp < n1; ++pp) s += cvec[pp * (n2 + 1) + q];
        v2[q] = s / (double)n1;
    }
    __syncthreads();
    if (tid < n2) {
        double s = 0.0;
#pragma unroll 8
        for (int a = 0; a < n2; ++a) s += (__popc(a & tid) & 1) ? -v2[a] : v2[a];
        vec[1][tid] = s * inv_sqrt_n2;
    }
    __syncthreads();

    // uniform targets (Sec. 4.2 URT): template q_k = (2k - n - 1)/n by rank (ties: lower index
    // first), scaled to the norm of the vector; ||q||^2 = (n^2 - 1)/(3n)
    {
        const int side = tid >= 512, k = tid - 512 * side, n = side ? n2 : n1;
        if (k < n) {
            const double *v = vec[side];
            const double mine = v[k];
            int rank = 0;
            double norm2 = 0.0;
#pragma unroll 8
            for (int m = 0; m < n; ++m) {
                const double o = v[m];
                rank += (o < mine) || (o == mine && m < k);
                norm2 += o * o;
            }
            const double qnorm2 = ((double)n * n - 1.0) / (3.0 * n);
            target[side][k] = sqrt(norm2 / qnorm2) * (2.0 * (rank + 1) - n - 1.0) / n;
        }
    }
    __syncthreads();

    // the four chains: thread (which, k) computes step k of chain `which`
    {
        const int which = tid / kMaxSide, k = tid % kMaxSide, side = which >> 1, is_target = which & 1;
        const int n = side ? n2 : n1;
        if (k >= 1 && k < n) chain_step(is_target ? target[side] : vec[side], n, k, chain + which * 2 * kMaxSide);
    }

    // the angles of Lemma 1, one thread per ART step
    if (tid < P) giv_theta[tid] = (float)(atan2(pair_b[tid], pair_a[tid]) - 0.78539816339744830962);
}

// R^U = R_map R'_map^T (Sec. 4.2 URT) for eight columns per workgroup; blockIdx.y = side.  Entry (r, k) of the
// product of a chain (step n-1 first): row r starts as e_r; step r+1 leaves (cos, -sin) in columns r and r+1, and
// every later step k <= r multiplies what is carried in column k by sin_k on its way to column k-1 and leaves
// carry * cos_k behind.  Nothing ever reaches a column right of r+1.  A thread walks row r of R_map with the carry in a
// register and multiplies every entry, as it appears, with eight entries of R'_map out of LDS: neither map is ever
// stored.  Side 1 leaves as fp16 R1.  Side 2 goes through the normalised Sylvester Hadamard matrix first,
// H[a][m] = (-1)^popcount(a & m) / sqrt n, as a fast transform over the rows (R2 = H R^U_2).
// A few KB and a chain of n dependent steps: one launch and 11 us where the three launches (maps, product, Hadamard
// factor) took 6.3 + 4.7 + 6.0 us at 64 x 64.
constexpr int kUrtCols = 8;

__global__ __launch_bounds__(kMaxSide) void urt_columns_kernel(const float *__restrict__ chain, int n1, int n2,
                                                               float inv_sqrt_n2, __half *__restrict__ R1,
                                                               __half *__restrict__ R2)
{
    constexpr int kPadded = kMaxSide + 8;
    __shared__ float co[2][kPadded], si[2][kPadded];             // [V, U]
    __shared__ __align__(16) float bt[kPadded][kUrtCols];        // R'_map transposed: [k][column]
    __shared__ float ru[kMaxSide][kUrtCols + 1];
    const int side = blockIdx.y, n = side ? n2 : n1, c0 = blockIdx.x * kUrtCols, r = threadIdx.x;
    if (c0 >= n) return;                                         // whole workgroup: the grid is sized for the larger side
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const float *src = chain + (2 * side + v) * 2 * kMaxSide;
        co[v][r] = (r >= 1 && r < n) ? src[r] : 1.f;             // (step 0 does not exist: column 0 keeps the carry)
        si[v][r] = (r >= 1 && r < n) ? src[kMaxSide + r] : 0.f;
        if (r < 8) co[v][kMaxSide + r] = 1.f, si[v][kMaxSide + r] = 0.f;
    }
    for (int k = r; k < kPadded * kUrtCols; k += kMaxSide) (&bt[0][0])[k] = 0.f;
    __syncthreads();
    // Row `row` of the map of chain v, from the last column to the first, eight columns at a time: nothing is carried
    // until column row + 1.  (Column n, which does not exist, has cos 1 and sin 0: the last row leaves it with a carry of 1.)
    auto walk = [&](int v, int row, auto entry) {
        float carry = 0.f;
        for (int kb = n / 8 * 8; kb >= 0; kb -= 8) {
#pragma unroll
            for (int u = 7; u >= 0; --u) {
                const int k = kb + u;
                const float cos_k = co[v][k], sin_k = si[v][k];
                const bool first = k == row + 1;
                entry(k, first ? -sin_k : carry * cos_k);
                carry = first ? cos_k : carry * sin_k;
            }
        }
    };
    if (r < kUrtCols && c0 + r < n) walk(1, c0 + r, [&](int k, float x) { bt[k][r] = x; });
    __syncthreads();
    float s[kUrtCols];
#pragma unroll
    for (int c = 0; c < kUrtCols; ++c) s[c] = 0.f;
    if (r < n)
        walk(0, r, [&](int k, float x) {
            const float4 lo = *reinterpret_cast<const float4 *>(&bt[k][0]), hi = *reinterpret_cast<const float4 *>(&bt[k][4]);
            s[0] = fmaf(x, lo.x, s[0]), s[1] = fmaf(x, lo.y, s[1]), s[2] = fmaf(x, lo.z, s[2]), s[3] = fmaf(x, lo.w, s[3]);
            s[4] = fmaf(x, hi.x, s[4]), s[5] = fmaf(x, hi.y, s[5]), s[6] = fmaf(x, hi.z, s[6]), s[7] = fmaf(x, hi.w, s[7]);
        });
    if (side == 0) {
#pragma unroll
        for (int c = 0; c < kUrtCols; ++c)
            if (r < n && c0 + c < n) R1[r * n + c0 + c] = __float2half_rn(s[c]);
        return;
    }
    for (int h = 1; h < n; h *= 2) {                             // n is a power of two
#pragma unroll
        for (int c = 0; c < kUrtCols; ++c) ru[r][c] = s[c];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kUrtCols; ++c) s[c] = (r & h) ? ru[r ^ h][c] - s[c] : s[c] + ru[r ^ h][c];
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < kUrtCols; ++c)
        if (r < n && c0 + c < n) R2[r * n + c0 + c] = __float2half_rn(s[c] * inv_sqrt_n2);
}

// A step over all channels by the whole workgroup takes 1.5 us at K = 512 and 2 us at 1024, the choice of the candidates 5 us
// whatever P (whole call in us, candidates / all channels: K = 512, P = 1 24.1 / 20.3, P = 4 26.7 / 25.2, P = 6 28.6 / 28.5;
// K = 1024, P = 1 25.4 / 21.6, P = 3 26.7 / 25.1, P = 4 27.7 / 28.0; K = 1536, P = 1 25.6 / 21.9, P = 2 26.5 / 26.4).
bool steps_by_all(int32_t K, int32_t P) { return K > kMaxCandidates && 256 * P + K <= 1792; }

bool build_shape_ok(int64_t T, int32_t K, int32_t n1, int32_t n2, int32_t P)
{
    if (T < 1 || T > SQ_MAX_ROWS || K <= 0 || P < 0 || P > SQ_MAX_GIVENS) return false;
    if (n1 < 2 || n1 > SQ_MAX_N1 || n2 < 8 || n2 > SQ_MAX_N2 || (n2 & (n2 - 1)) != 0) return false;
    return (int64_t)n1 * n2 == K && K <= SQ_MAX_K;
}

}  // namespace

}  // namespace sq

extern "C" sq_status sq_kron_factor(int32_t n, int32_t *n1, int32_t *n2)
{
    if (!n1 || !n2) return SQ_ERR_NULL;
    if (n < 1) return SQ_ERR_SHAPE;
    // Alg. 1 asks for the power of two dividing n nearest to sqrt(n).  Distances to sqrt(n) shrink
    // while a^2 <= n and grow afterwards, so only two candidates matter: the largest divisor `below`
    // with below^2 <= n, and its double if that divides n as well.  2 below - sqrt(n) < sqrt(n) - below
    // is 3 below < 2 sqrt(n), i.e. 9 below^2 < 4 n, in integers; equality keeps the smaller one.
    const int64_t m = n;
    int64_t below = 1;
    while (m % (2 * below) == 0 && 4 * below * below <= m) below *= 2;
    const bool above_divides = m % (2 * below) == 0;
    const int64_t best = (above_divides && 9 * below * below < 4 * m) ? 2 * below : below;
    *n2 = (int32_t)best;
    *n1 = (int32_t)(n / best);
    return SQ_OK;
}

extern "C" int64_t sq_build_rotation_workspace_bytes(int64_t T, int32_t n1, int32_t n2)
{
    if (T < 1 || n1 < 1 || n2 < 1 || n1 > SQ_MAX_N1 || n2 > SQ_MAX_N2) return 0;
    return 4 * sq::build_workspace_floats(T, n1, n2);
}

extern "C" sq_status sq_build_rotation(const void *X, int64_t T, int32_t K, int64_t ldx, int32_t n1, int32_t n2,
                                       int32_t P, int32_t *giv_i, int32_t *giv_j, float *giv_theta, void *R1,
                                       void *R2, void *workspace, void *stream)
{
    if (!X || !R1 || !R2 || !workspace) return SQ_ERR_NULL;
    if (P > 0 && (!giv_i || !giv_j || !giv_theta)) return SQ_ERR_NULL;
    if (!sq::build_shape_ok(T, K, n1, n2, P) || ldx < K) return SQ_ERR_SHAPE;
    if ((ldx % 8) != 0 || ((uintptr_t)X & 15) || ((uintptr_t)R1 & 1) || ((uintptr_t)R2 & 1) ||
        ((uintptr_t)workspace & 15) || ((uintptr_t)giv_i & 3) || ((uintptr_t)giv_j & 3) || ((uintptr_t)giv_theta & 3))
        return SQ_ERR_ALIGN;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const sq::BuildWorkspace w = sq::carve_workspace(workspace, T);
    const double inv_sqrt_n2 = 1.0 / sqrt((double)n2);
    const __half *Xh = static_cast<const __half *>(X);

    const int64_t row_groups = (T + 3) / 4;
    hipLaunchKernelGGL(sq::row_absmax_kernel, dim3((unsigned)(row_groups < 4096 ? row_groups : 4096)), dim3(256), 0,
                       st, Xh, ldx, (int)T, K, w.rowmax);
    auto art = sq::steps_by_all(K, P) ? sq::art_urt_kernel<true> : sq::art_urt_kernel<false>;
    // 143.5 KiB at the largest K
    const size_t lds = sq::kBuildSmallBytes + (size_t)(K + n1) * sizeof(double) + sq::kSelectWords * sizeof(uint32_t);
    if (!sq::allow_large_lds(reinterpret_cast<const void *>(art))) return SQ_ERR_LAUNCH;
    hipLaunchKernelGGL(art, dim3(1), dim3(sq::kBuildThreads), lds, st, Xh, ldx, (int)T, K, n1, n2, P, inv_sqrt_n2,
                       w.rowmax, giv_i, giv_j, giv_theta, w.chain);
    const int big = n1 > n2 ? n1 : n2;
    hipLaunchKernelGGL(sq::urt_columns_kernel, dim3((unsigned)((big + sq::kUrtCols - 1) / sq::kUrtCols), 2), dim3(sq::kMaxSide), 0,
                       st, w.chain, n1, n2, (float)inv_sqrt_n2, static_cast<__half *>(R1), static_cast<__half *>(R2));
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}
