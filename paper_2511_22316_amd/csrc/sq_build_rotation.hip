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
// the histograms, the candidates, one count per wave, results of the two searches, a counter, the channels of
// the P largest and the P smallest in order
// (one histogram of 2048 bins, four words of padding behind every 32, or two of 256)
constexpr int kFineBins = 2048, kFineWords = kFineBins / 32 * 36;
constexpr int kSelectWords = kFineWords + kMaxCandidates + kBuildWaves + 4 + 2 + 2 * SQ_MAX_GIVENS;
constexpr uint32_t kChannelMask = 0x3FFF;      // a candidate: its 15-bit magnitude above its channel
static_assert(SQ_MAX_K <= kChannelMask + 1 && SQ_MAX_GIVENS <= kWave, "limits");
static_assert(kBuildSmallBytes % 16 == 0, "the fp64 vectors behind the slots are 8-byte aligned, the histograms 16");

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

// r / sqrt(2) of Lemma 1
__device__ __forceinline__ double equalised(double a, double b)
{
    return sqrt(fma(a, a, b * b)) * 0.70710678118654752440;
}

// The same for finite a that a step can pick (0 <= b <= a; the largest fp16 channel is at least 2^-24, and 64 steps leave more than
// 2^-32 of it), whose squares are far from both ends of fp64, so that the root needs neither scaling nor special cases.
// Goldschmidt's iteration from the hardware's estimate r of 1 / sqrt(x): root and half = 1 / (2 sqrt(x)) improved together, then two
// corrections of the root by its remainder x - root^2, which is exact in an fma.  The result is the correctly rounded root,
// which is what sqrt returns: no difference on 4.3e9 random pairs, half of them with the mantissas of fp16.  (The function
// above serves where a may be infinite.)
__device__ __forceinline__ double equalised_in_range(double a, double b)
{
    const double x = fma(a, a, b * b), r = __builtin_amdgcn_rsq(x);
    double root = x * r, half = 0.5 * r;
    const double d = fma(-half, root, 0.5);
    root = fma(root, d, root), half = fma(half, d, half);
    root = fma(fma(-root, root, x), half, root);
    root = fma(fma(-root, root, x), half, root);
    return root * 0.70710678118654752440;
}

// lane l takes the value of lane l - 1 (lane 0: zero)
__device__ __forceinline__ uint32_t wave_up(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);      // wave_shr:1
}

__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }

// The wave's list of the largest channels, in order: value (as the two halves of a double, magnitudes) descending, among
// equals the channel ascending (above its sign bit).  What is pushed past lane 63 is never asked for again: a step takes one,
// and there are 64 steps.
struct Largest {
    static constexpr uint32_t kNone = 0xFFFFFFFFu;
    uint32_t hi = 0, lo = 0, channel = kNone;

    __device__ __forceinline__ double value() const { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); }
    __device__ __forceinline__ void drop_first(int r, int lane)
    {
        hi = __shfl(hi, lane + r), lo = __shfl(lo, lane + r), channel = __shfl(channel, lane + r);
        if (lane + r >= kWave) hi = 0, lo = 0, channel = kNone;
    }
    // the value e for channels c1 < c2
    __device__ __forceinline__ void insert(uint32_t eh, uint32_t el, uint32_t c1, uint32_t c2, int lane)
    {
        const double e = __longlong_as_double((long long)(((uint64_t)eh << 32) | el)), mine = value();
        const uint64_t above = __ballot(mine > e), same = __ballot(mine == e);
        const int at1 = __popcll(above | (same & __ballot(channel < c1))), at2 = __popcll(above | (same & __ballot(channel < c2))) + 1;
        const uint32_t hi1 = wave_up(hi), lo1 = wave_up(lo), ch1 = wave_up(channel);
        const uint32_t hi2 = wave_up(hi1), lo2 = wave_up(lo1), ch2 = wave_up(ch1);
        const bool first = lane == at1, second = lane == at2, one = lane > at1, two = lane > at2;
        hi = first || second ? eh : two ? hi2 : one ? hi1 : hi;
        lo = first || second ? el : two ? lo2 : one ? lo1 : lo;
        channel = first ? c1 : second ? c2 : two ? ch2 : one ? ch1 : channel;
    }
};

// One wave: the same over kFineBins bins, a lane 32 of them (at 36 l); `upto`: the count up to and with that bin.
template <bool DOWN>
__device__ __forceinline__ int fine_bin_reaching(const uint32_t *hist, uint32_t target, uint32_t &upto)
{
    const int lane = threadIdx.x & (kWave - 1), place = DOWN ? kWave - 1 - lane : lane;
    static_assert(kFineBins == 32 * kWave, "32 bins a lane");
    uint32_t n[32], sum = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const uint4 v = *reinterpret_cast<const uint4 *>(hist + 36 * place + 4 * u);
        n[4 * u] = v.x, n[4 * u + 1] = v.y, n[4 * u + 2] = v.z, n[4 * u + 3] = v.w;
        sum += v.x + v.y + v.z + v.w;
    }
    uint32_t run = sum;
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) {
        const uint32_t o = __shfl_up(run, d);
        if (lane >= d) run += o;
    }
    const int owner = __ffsll((unsigned long long)__ballot(run - sum < target && target <= run)) - 1;
    run -= sum;
    int steps = 0;                                                 // bins in front of the one that reaches it
#pragma unroll
    for (int u = 0; u < 32; ++u) {
        const uint32_t c = n[DOWN ? 31 - u : u];
        if (run < target) run += c, steps = u;
    }
    upto = __shfl(run, owner);
    return 32 * __shfl(place, owner) + (DOWN ? 31 - __shfl(steps, owner) : __shfl(steps, owner));
}

__device__ __forceinline__ void magnitude_key(double v, uint32_t &hi, uint32_t &lo)
{
    const uint64_t bits = (uint64_t)__double_as_longlong(fabs(v));
    hi = (uint32_t)(bits >> 32);
    lo = (uint32_t)bits;
}

// Step k of the Givens chain that takes `vec` (n entries) to ||vec|| e_1: entry k is zeroed by a
// rotation in the plane (k - 1, k), k = n - 1 down to 1.  When step k acts, entry k holds the norm
// of the original entries k .. n-1, so with S_k the sum of their squares (tail[k])
//   cos_k = v_{k-1} / sqrt(S_{k-1}),   sin_k = sqrt(S_k / S_{k-1})     (cos = 1, sin = 0 if S_{k-1} = 0;
//   sin_{n-1} = v_{n-1} / sqrt(S_{n-2}), because the last entry enters with its sign)
// and the steps can be computed independently of one another.  Stored at cs[k], cs[kMaxSide + k].
__device__ __forceinline__ void chain_step(const double *vec, const double *tails, int n, int k, float *cs)
{
    const double x = vec[k - 1], tail = tails[k], all = tail + x * x;
    cs[k] = (all == 0.0) ? 1.f : (float)(x / sqrt(all));
    // the first step (k = n-1) meets the last entry itself, sign included; later ones meet a norm
    cs[kMaxSide + k] = (all == 0.0) ? 0.f : (float)(k == n - 1 ? vec[k] / sqrt(all) : sqrt(tail / all));
}

// tails[k] = sum of the squares of the entries k .. n-1, k = n-1 .. 1, by one wave (four entries a lane); returns the sum of all
__device__ __forceinline__ double sum_tails(const double *vec, int n, double *tails)
{
    const int lane = threadIdx.x & (kWave - 1);
    static_assert(kMaxSide == 4 * kWave, "four entries a lane");
    double own[4], sum = 0.0;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
        const double o = 4 * lane + u < n ? vec[4 * lane + u] : 0.0;
        own[u] = sum += o * o;
    }
    double from = sum;                                             // of this lane's entries and all behind them
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) {
        const double o = __shfl_down(from, d);
        if (lane + d < kWave) from += o;
    }
    double next = __shfl_down(from, 1);
    if (lane == kWave - 1) next = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (4 * lane + u >= 1 && 4 * lane + u < n) tails[4 * lane + u] = own[u] + next;
    return __shfl(from, 0);
}

// One workgroup.  All of its LDS is dynamic (kBuildSmallBytes + 8 (K + n1) + 4 kSelectWords bytes): the reduction slots,
// the small vectors, the calibration vector in fp64 (its rows of n2 entries one apart, so that the threads that
// sum a row each read different banks), and what the choice of the ART candidates needs.
//
// What bounds it is the chain of P dependent ART steps.  Step p (from 0) has at most 2 p channels rewritten by the steps
// before it, so what it picks is one of those or among the first 2 p + 1 in order of the calibration row as it was:
// the 2 P largest and the 2 P smallest channels are all that can ever be chosen.  A histogram of the 15-bit magnitudes in
// 2048 bins finds the outer bins that hold them, 3 us; where the channels of those number more than 256 (P > 48, runs of equals), a
// radix selection over two histograms of 256 bins, ties by channel, cuts them out exactly, 5.6 us.  Where the two sets are
// disjoint, counting puts the P outermost of either in order (1.5 us), and one wave takes the steps from those two ends, several at
// once (T = 2048, K = 4096, P = 32: 0.18 us a step).  What that does not cover (generated values among the smallest, a row nearly all
// of one magnitude, at most 256 channels) one wave does with the candidates in registers and two reductions a step, 0.73 us each.
// The whole kernel at that size: 91.5 us with a reduction over all channels by the whole workgroup in every step, 41.5 with
// the reductions of one wave, 22.1 with the steps from the ends, 19.6 with the finer histogram.
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
    uint32_t *hist = reinterpret_cast<uint32_t *>(cvec + (K + n1 + 1) / 2 * 2);      // 16-byte aligned
    uint32_t *cand = hist + kFineWords;                            // [kMaxCandidates]
    uint32_t *wave_ties = cand + kMaxCandidates;                   // [kBuildWaves]
    uint32_t *found = wave_ties + kBuildWaves;                     // bin and count before it, from above and from below
    uint32_t *n_cand = found + 4;
    uint32_t *in_order = n_cand + 2;                               // [2][SQ_MAX_GIVENS]
    double *pair_norm = reinterpret_cast<double *>(slots_a);       // [2]: the slots are free by then
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int n2_log = 31 - __clz(n2);                             // n2 is a power of two
    auto at = [n2_log](int k) { return k + (k >> n2_log); };

    // calibration row: the largest row maximum, lowest row among equals
    uint32_t top = 0, top_at = 0xFFFFFFFFu;
    for (int t = tid; t < T; t += kBuildThreads) {
        const uint32_t m = __float_as_uint(rowmax[t]);
        if (m > top || top_at == 0xFFFFFFFFu) top = m, top_at = (uint32_t)t;      // t ascends: ties keep the lower row
    }
    for (int w = tid; w < kFineWords; w += kBuildThreads) hist[w] = 0;
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
    bool ordered = false;                                          // in_order holds the ends of two disjoint sets
    bool chosen = false;
    if (P > 0 && !BY_ALL && K > kMaxCandidates && P <= 48) {
        // Bins of sixteen magnitudes: where all channels of the outer bins that hold the 2 P largest and the 2 P smallest
        // number no more than a wave takes, they are the candidates.
#pragma unroll
        for (int e = 0; e < kMost; ++e)
            if (key[e] != 0xFFFFu) atomicAdd(&hist[(key[e] >> 4) + (key[e] >> 9) * 4], 1u);
        __syncthreads();
        uint32_t upto;
        if (wave == 0) {
            const int b = fine_bin_reaching<true>(hist, 2 * (uint32_t)P, upto);
            if (lane == 0) found[0] = (uint32_t)b, found[1] = upto;
        } else if (wave == 1) {
            const int b = fine_bin_reaching<false>(hist, 2 * (uint32_t)P, upto);
            if (lane == 0) found[2] = (uint32_t)b, found[3] = upto;
        }
        __syncthreads();
        const uint32_t bin_hi = found[0], bin_lo = found[2];
        chosen = ordered = bin_hi > bin_lo && found[1] + found[3] <= (uint32_t)kMaxCandidates;
        if (chosen) {
#pragma unroll
            for (int e = 0; e < kMost; ++e)
                if (key[e] != 0xFFFFu && ((key[e] >> 4) >= bin_hi || (key[e] >> 4) <= bin_lo))
                    cand[atomicAdd(n_cand, 1u)] = (key[e] << 14) | (uint32_t)(k0 + e);
        } else if (tid < 2 * 256) {
            hist[tid] = 0;
        }
        __syncthreads();
    }
    if (P > 0 && !BY_ALL && K <= kMaxCandidates) {
        if (tid < K) cand[tid] = (uint32_t)tid;
        if (tid == 0) *n_cand = (uint32_t)K;
    } else if (P > 0 && !BY_ALL && !chosen) {
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
            if (take) cand[atomicAdd(n_cand, 1u)] = (key[e] << 14) | (uint32_t)(k0 + e);
        }
        ordered = key_hi > key_lo;
        __syncthreads();
    }
    // Four threads count how many candidates come before theirs, from above and from below (lower channels first).
    if (ordered) {
        const int n = (int)*n_cand;
        const uint32_t self = (tid >> 2) < n ? cand[tid >> 2] : 0u;
        uint32_t larger = 0, smaller = 0;
#pragma unroll 8
        for (int m = tid & 3; m < n; m += 4) {
            const uint32_t o = cand[m];
            larger += (o ^ kChannelMask) > (self ^ kChannelMask);
            smaller += o < self;
        }
        larger += __shfl_xor(larger, 1), smaller += __shfl_xor(smaller, 1);
        larger += __shfl_xor(larger, 2), smaller += __shfl_xor(smaller, 2);
        if ((tid & 3) == 0 && (tid >> 2) < n) {
            if (larger < (uint32_t)P) in_order[larger] = self & kChannelMask;
            if (smaller < (uint32_t)P) in_order[SQ_MAX_GIVENS + smaller] = self & kChannelMask;
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
                const double e = equalised(a, b);
                giv_i[p] = i;
                giv_j[p] = j;
                pair_a[p] = a;
                pair_b[p] = b;
                cvec[at(i)] = cvec[at(j)] = e;
            }
            __syncthreads();
        }
    } else if (wave == 0 && P > 0) {
        auto value = [](uint32_t hi, uint32_t lo) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); };
        // While the smallest untouched channels are below everything generated, a step takes the next one of those, which lie in
        // lane order, and the first of the list of the largest, where what it makes is put in its place by counting: no
        // reduction on the chain.  What a step makes of a >= 4 b is below 0.73 a, so all channels of the list above 0.73 of the
        // first one are taken, in order, before anything the steps between make: those steps are done at once, a lane each.
        // (Magnitudes of fp16 values have no lower half.)
        int p0 = 0;
        if (ordered) {
            Largest largest;
            uint32_t low_hi = 0, low_ch = 0;                       // channel above its sign bit
            if (lane < P) {
                const uint32_t t = in_order[lane], l = in_order[SQ_MAX_GIVENS + lane];
                const uint32_t th = (uint32_t)__double2hiint(cvec[at((int)t)]), lh = (uint32_t)__double2hiint(cvec[at((int)l)]);
                largest.hi = th & 0x7FFFFFFFu, largest.channel = t << 1 | th >> 31;
                low_hi = lh & 0x7FFFFFFFu, low_ch = l << 1 | lh >> 31;
            }
            uint32_t least = 0x7FFFFFFFu;                          // upper half of the smallest value made
            while (p0 < P) {
                const uint32_t bh = __shfl(low_hi, lane + p0), cj = __shfl(low_ch, lane + p0), ci = largest.channel;
                const double a = largest.value(), b = value(bh, 0), first = value(lane_of(largest.hi, 0), lane_of(largest.lo, 0));
                // no value left, or one that is not finite (the square root below is for finite ones): the other steps' turn
                if (first == 0.0 || lane_of(largest.hi, 0) >= 0x7FF00000u) break;
                int r = __popcll(__ballot(lane < P - p0 && a > 0.73 * first && 4.0 * b <= first && bh < least));
                if (r == 0) {
                    if (lane_of(bh, 0) >= least) break;
                    r = 1;
                }
                const double e = equalised_in_range(a, b);
                const uint32_t eh = (uint32_t)__double2hiint(e), el = (uint32_t)__double2loint(e), i = ci >> 1, j = cj >> 1;
                if (lane < r) {
                    giv_i[p0 + lane] = (int)i;
                    giv_j[p0 + lane] = (int)j;
                    pair_a[p0 + lane] = (ci & 1) ? -a : a;
                    pair_b[p0 + lane] = (cj & 1) ? -b : b;
                    cvec[at((int)i)] = cvec[at((int)j)] = e;
                }
                largest.drop_first(r, lane);
                for (int q = 0; q < r; ++q) {
                    const uint32_t qh = lane_of(eh, q), qi = lane_of(i, q) << 1, qj = lane_of(j, q) << 1;
                    largest.insert(qh, lane_of(el, q), min(qi, qj), max(qi, qj), lane);
                    least = min(least, qh);
                }
                p0 += r;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        // The other steps, if any (generated values among the smallest, few channels, nearly all of one magnitude).
        // This lane's candidates by channel, their magnitudes as integers; no channel: zero among the largest, all
        // ones among the smallest.
        uint32_t idx[4];
        uint64_t large[4], small[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) idx[u] = (uint32_t)(lane + 64 * u) < *n_cand ? cand[lane + 64 * u] & kChannelMask : 0xFFFFFFFFu;
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
        for (int p = p0; p < P; ++p) {
            uint64_t best = large[0];
            uint32_t who = idx[0], ah, al, bh, bl;
#pragma unroll
            for (int u = 1; u < 4; ++u)
                if (large[u] > best) best = large[u], who = idx[u];
            const uint32_t i = wave_arg_short<true>((uint32_t)(best >> 32), (uint32_t)best, who, ah, al);
            uint32_t j = smallest_but(0xFFFFFFFFu, bh, bl);
            if (j == i) j = smallest_but(i, bh, bl);   // every magnitude the same
            const double a = value(ah, al), b = value(bh, bl);
            const double e = equalised(a, b);
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

    // Uniform targets (Sec. 4.2 URT): template q_k = (2k - n - 1)/n by rank (ties: lower index
    // first), scaled to the norm of the vector; ||q||^2 = (n^2 - 1)/(3n).  Half of the workgroup per side, two threads an
    // entry; the sums of squares by a wave that has few or no entries to rank.  The tails lie where the calibration vector was.
    const int half = tid / 512, in_half = tid % 512, n_half = half ? n2 : n1;
    double *tail_v = cvec + (half ? 2 * n1 - 2 : 0) - 1, *tail_u = tail_v + n_half - 1;      // entries 1 .. n - 1
    const double *v_half = vec[half];
    int rank = 0;
    if (in_half / 2 < n_half) {
        const int k = in_half / 2;
        const double mine = v_half[k];
#pragma unroll 8
        for (int m = in_half & 1; m < n_half; m += 2) {
            const double o = v_half[m];
            rank += (o < mine) || (o == mine && m < k);
        }
    }
    rank += __shfl_xor(rank, 1);
    if (in_half >= 448) {
        const double norm2 = sum_tails(v_half, n_half, tail_v);
        if (lane == 0) pair_norm[half] = sqrt(norm2 / (((double)n_half * n_half - 1.0) / (3.0 * n_half)));
    }
    __syncthreads();
    if (in_half / 2 < n_half && (in_half & 1) == 0)
        target[half][in_half / 2] = pair_norm[half] * (2.0 * (rank + 1) - n_half - 1.0) / n_half;
    __syncthreads();
    if (in_half < kWave) sum_tails(target[half], n_half, tail_u);
    __syncthreads();

    // the four chains: a thread computes step k of the chain of V or of U
    {
        const int is_target = in_half / kMaxSide, k = in_half % kMaxSide;
        if (k >= 1 && k < n_half)
            chain_step(is_target ? target[half] : v_half, is_target ? tail_u : tail_v, n_half, k, chain + (2 * half + is_target) * 2 * kMaxSide);
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
// A few KB and a chain of n dependent steps: one launch and 8.4 us (11.2 with a barrier for every stage of the transform) where
// the three launches (maps, product, Hadamard factor) took 6.3 + 4.7 + 6.0 us at 64 x 64.
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
    // n is a power of two: six stages between the lanes of a wave, what is left through LDS
    for (int h = 1; h < n && h < kWave; h *= 2) {
#pragma unroll
        for (int c = 0; c < kUrtCols; ++c) {
            const float o = __shfl_xor(s[c], h);
            s[c] = (r & h) ? o - s[c] : s[c] + o;
        }
    }
    for (int h = kWave; h < n; h *= 2) {
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

// A step over all channels by the whole workgroup takes 1.2 us at K = 512 and 6 us at 16384; the choice of the candidates and
// their order take 5 us whatever P, and hardly more with every step (whole call in us, in order / all channels: K = 288, P = 2
// 18.7 / 17.7, P = 3 19.1 / 19.4; K = 2048, P = 2 22.6 / 22.6, P = 3 23.0 / 24.8; K = 4096, P = 1 23.3 / 22.3, P = 2 23.6 / 24.6;
// K = 8192, P = 1 32.8 / 32.8; K = 16384, P = 1 41.2 / 43.0).
bool steps_by_all(int32_t K, int32_t P)
{
    return K > kMaxCandidates && (P == 0 || (P == 1 && K <= 8192) || (P == 2 && K <= 2048));
}

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
    // 151 KiB at the largest K
    const size_t lds = sq::kBuildSmallBytes + (size_t)((K + n1 + 1) / 2 * 2) * sizeof(double) + sq::kSelectWords * sizeof(uint32_t);
    if (!sq::allow_large_lds(reinterpret_cast<const void *>(art))) return SQ_ERR_LAUNCH;
    hipLaunchKernelGGL(art, dim3(1), dim3(sq::kBuildThreads), lds, st, Xh, ldx, (int)T, K, n1, n2, P, inv_sqrt_n2,
                       w.rowmax, giv_i, giv_j, giv_theta, w.chain);
    const int big = n1 > n2 ? n1 : n2;
    hipLaunchKernelGGL(sq::urt_columns_kernel, dim3((unsigned)((big + sq::kUrtCols - 1) / sq::kUrtCols), 2), dim3(sq::kMaxSide), 0,
                       st, w.chain, n1, n2, (float)inv_sqrt_n2, static_cast<__half *>(R1), static_cast<__half *>(R2));
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}
