// W4A4 GEMM on the 6-bit float matrix instruction of gfx950: the tile kernel for many tokens.
//
//   acc[t, n] = sum_k Qx[t, k] Qw[n, k]   (exact)      Y[t, n] = fp16(acc * sx[t] * sw[n])
//
// v_mfma_f32_32x32x64_f8f6f4 multiplies E2M3 values at twice the rate of the int8 instruction.  With its sign and upper
// exponent bit clear, an E2M3 field is a linear four-bit number: field u is the value u / 8, u = 0 .. 15.  A code goes
// in as u = code + 8, so that per pair of codes the product is (a + 8)(b + 8) / 64, and
//
//   acc = 64 P - 8 sum_k a - 8 sum_k b - 64 K
//
// with P the fp32 accumulator (a multiple of 1/64 below 2^24 / 64: every sum is exact) and the row sums of the codes
// taken beside it.  What the encoding buys over the codes times 16 as int8 is power: with the codes of Gaussian rows a
// register-only loop on all CUs sustains 7.6 POP/s against 4.3 POP/s, both at the power limit of the chip.
//
// What bounds the kernel is its instruction stream, at the power limit.  Widening a nibble operand takes 14 instructions per
// fragment and step of 64 codes, and a wave issues one instruction in four cycles (4.5 for the eight-byte forms used here),
// so a wave's tile is as large as the registers allow: 128 x 128 (7 instructions of conversion per matrix instruction), one
// wave per SIMD.  Built up in registers, per matrix instruction and SIMD: alone 17.3 ns (7.7 POP/s), with the conversion
// 23.1, with the reads from LDS 26.5, with the barriers 27.1; this loop takes 32, the rest being the row sums (1) and the
// global -> LDS requests (4; half of them left out: 3 - 5 % of the kernel).
//   256 x 256 tile: four waves, a persistent walk over the output tiles.
//   128 x 256 tile, for fewer tokens or channels: two K groups of two waves that take half of every K tile each.  (Two groups
// of four waves of 64 x 128, two waves per SIMD, 10.5 instructions of conversion: a K tile of 256 codes takes 1.30 us, here
// 1.05.  T = 2048, N = 4096, K = 4096 27.5 -> 25.3 us, K = 11008 59.9 -> 53.2; T = 333, K = 5120, N = 13824 28.5 -> 25.9.)
//   128 x 192 and 256 x 192 tiles (waves of 128 x 96, 8.2 instructions of conversion): a K tile takes 0.86 and 0.85 of the time of
// the wider ones, so they pay where they fill the CUs better (T = 333, K = 5120, N = 13824, 216 or 162 tiles: 25.9 -> 23.5 us;
// T = 1001, K = 3072, N = 9216, 192 or 144 tiles: 29.3 -> 26.2).
// The conversion is done in registers, by every wave for itself: one that is shared through LDS (24 bytes per 32 codes
// written once and read by all) moves 1.5 times the bytes out of LDS, writes them at a quarter of the read rate, and was
// 10 - 15 % slower.  T = 8192, K = 8192, N = 28672: int8 instruction 1359 us, here 980 - 1005.
//   The times above are of launches one behind the other on the same operands.  With operands and outputs out of a ring beyond the
// caches the same calls take up to 8 % longer (T = 2048, N = 4096: K = 4096 25.9 / 26.9 us, K = 11008 54.3 / 55.1; T = 333,
// K = 5120, N = 13824 23.5 / 25.4; T = 1001, K = 3072, N = 9216 26.6 / 29.0), and with other kernels between them T = 2048, K = N = 4096 takes 28.4.
#include "sq_fp6_store.h"
#include "sq_gemm_tile.h"
#include "sq_w4a4_fp6.h"

namespace sq {

namespace {

typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));

// Sixteen codes of two dwords w0, w1 and the sixteen 6-bit fields of three dwords d0, d1, d2.  With r = w1 rotated
// left by two, every nibble of w0 and of r lies where a field begins, or straddles two dwords as a field does:
//   d0 takes nibbles 0, 3, 6 of w0 and 1, 4 and the lower half of 7 of r;  d1: 1, 4, 7 of w0, the upper half of 7 and
//   2, 5 of r;  d2: 2, 5 of w0 and 0, 3, 6 of r.
// The order of the codes within an operand changes, in the same way for both.  The code's top bit is flipped (code + 8).
constexpr uint32_t kM0 = 0x0F00F00Fu, kM1 = 0xF00F00F0u, kM2 = 0x00F00F00u;   // fields taken from the first dword
constexpr uint32_t kN0 = 0xC03C03C0u, kN1 = 0x03C03C03u, kN2 = 0x3C03C03Cu;   // fields taken from the rotated second

struct FieldMasks {
    uint32_t m0, m1, m2, n0, n1, n2, f0, f1, f2;
};

__device__ __forceinline__ FieldMasks field_masks()
{
    FieldMasks k;
    auto in_vgpr = [](uint32_t c) {
        uint32_t v;
        asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(c));
        return v;
    };
    k.m0 = in_vgpr(kM0), k.m1 = in_vgpr(kM1), k.m2 = in_vgpr(kM2);
    k.n0 = in_vgpr(kN0), k.n1 = in_vgpr(kN1), k.n2 = in_vgpr(kN2);
    k.f0 = in_vgpr((0x88888888u & kM0) | (0x22222222u & kN0));
    k.f1 = in_vgpr((0x88888888u & kM1) | (0x22222222u & kN1));
    k.f2 = in_vgpr((0x88888888u & kM2) | (0x22222222u & kN2));
    return k;
}

// sixteen codes (two dwords of nibbles) -> sixteen six-bit fields (three dwords), seven instructions.  The masks sit
// in vector registers: the three-operand bit operation issues every 2.4 cycles then, and every 4.4 with a scalar one.
__device__ __forceinline__ void to_fp6(uint32_t w0, uint32_t w1, const FieldMasks &k, int &d0, int &d1, int &d2)
{
    // bitop3 0x6A: (a & b) ^ c;  0x78: a ^ (b & c)
    const uint32_t r = __builtin_amdgcn_alignbit(w1, w1, 30);
    const uint32_t t0 = __builtin_amdgcn_bitop3_b32(w0, k.m0, k.f0, 0x6A);
    const uint32_t t1 = __builtin_amdgcn_bitop3_b32(w0, k.m1, k.f1, 0x6A);
    const uint32_t t2 = __builtin_amdgcn_bitop3_b32(w0, k.m2, k.f2, 0x6A);
    d0 = (int)__builtin_amdgcn_bitop3_b32(t0, r, k.n0, 0x78);
    d1 = (int)__builtin_amdgcn_bitop3_b32(t1, r, k.n1, 0x78);
    d2 = (int)__builtin_amdgcn_bitop3_b32(t2, r, k.n2, 0x78);
}

__device__ __forceinline__ v16f mfma_fp6(const v6i a, const v6i b, const v16f c)
{
    const v8i x = {a[0], a[1], a[2], a[3], a[4], a[5], 0, 0}, y = {b[0], b[1], b[2], b[3], b[4], b[5], 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 2, 2, 0, 0, 0, 0);   // both operands E2M3
}

// Where the next global -> LDS load goes.  Nothing else in this kernel uses M0 (the LDS instructions of this part do
// not), so it is set once per K tile and moved on behind every load.
__device__ __forceinline__ void dma_begin(uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0" ::"s"(lds_addr) : "memory", "m0");
}

// global -> LDS: BYTES per lane from base + off (base wave-uniform) to M0 + BYTES * lane; M0 moves on by STEP
template <int STEP>
__device__ __forceinline__ void dma_16(const void *base, uint32_t off)
{
    asm volatile("global_load_lds_dwordx4 %0, %1\n\t"
                 "s_add_u32 m0, m0, %2"
                 :
                 : "v"(off), "s"(base), "n"(STEP)
                 : "memory", "m0", "scc");
}

template <int STEP>
__device__ __forceinline__ void dma_4(const void *base, uint32_t off)
{
    asm volatile("global_load_lds_dword %0, %1\n\t"
                 "s_add_u32 m0, m0, %2"
                 :
                 : "v"(off), "s"(base), "n"(STEP)
                 : "memory", "m0", "scc");
}

// fp16(x0 w0) and fp16(x1 w1) in one dword, each product rounded once, on its way to fp16, as the other GEMM kernels do
// (their compiler finds this instruction; for two results in one dword it finds two products and a packed conversion,
// which round twice): Y is the same bit for bit whichever kernel a call takes.
__device__ __forceinline__ uint32_t scaled_pair(float x0, float w0, float x1, float w1)
{
    uint32_t d;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(d) : "v"(x0), "v"(w0));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(d) : "v"(x1), "v"(w1));
    return d;
}

// Output tile WM FM 32 tokens x 2 FN 32 channels; KG groups of WM x 2 waves share it and split every K tile.
template <int WM, int FM, int FN, int KG>
struct Fp6Shape {
    static constexpr int WN = 2, NW = WM * WN * KG, NT = NW * kWave;
    static constexpr int BM = WM * FM * 32, BN = WN * FN * 32;
    static constexpr int BKB = 128, STEPS = 4 / KG;                 // bytes of a tile row; steps per wave and tile
    static constexpr int A_BYTES = BM * BKB, STAGE = (BM + BN) * BKB;
    static constexpr int NS = STAGE > 49152 ? 2 : 3;
    static constexpr int SCALE_BYTE = NS * STAGE, SUM_BYTE = SCALE_BYTE + 2 * (BM + BN) * 4;
    static constexpr int LDS_BYTES = SUM_BYTE + KG * (BM + BN) * 4;
    static_assert(LDS_BYTES <= kMaxDynamicLds, "ring does not fit in LDS");
};

// Row sums on the matrix cores.  The 16 x 16 x 128 instruction reads the same registers as rows l % 16 with the
// contraction index in block l / 16: a fragment's rows 16 .. 31 look like blocks 1 and 3 of rows 0 .. 15.  Against a
// second operand whose column 0 is one in blocks 0 and 2 and whose column 1 is one in blocks 1 and 3 (zero elsewhere),
// the product's first two columns are the sums of the 32 rows.
// (In assembly, to keep these accumulators in ordinary vector registers: the 256 x 256 tile fills all accumulation
// registers.  The operands were written at least one MFMA earlier, and the epilogue waits before it reads the result.)
__device__ __forceinline__ void mfma_fp6_16(const v6i a, const v6i b, v4f &c)
{
    asm("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:2 blgp:2" : "+v"(c) : "v"(a), "v"(b));
}

__device__ __forceinline__ v6i sum_selector(int lane)
{
    // sixteen fields of 1.0 (0b001000) are the dwords below
    const bool one = (lane & 15) == ((lane >> 4) & 1);
    const int d0 = one ? 0x08208208 : 0, d1 = one ? (int)0x82082082 : 0, d2 = one ? 0x20820820 : 0;
    return v6i{d0, d1, d2, d0, d1, d2};
}

}  // namespace

template <int WM, int FM, int FN, int KG>
__global__ __launch_bounds__(WM * 2 * KG * kWave, WM * KG / 2) void w4a4_gemm_fp6_kernel(
    const uint8_t *__restrict__ Qx, const float *__restrict__ sx, int T, int Kb, const uint8_t *__restrict__ Qw,
    const float *__restrict__ sw, int N, __half *__restrict__ Y, int64_t ldy, int32_t *__restrict__ acc_dbg,
    int tiles_m, int tiles_n, int rows_aligned)
{
    using G = Fp6Shape<WM, FM, FN, KG>;
    constexpr int WN = G::WN, BM = G::BM, BN = G::BN, NS = G::NS, NW = G::NW, BKB = G::BKB, STEPS = G::STEPS;
    constexpr int NM = FM * FN, NF = FM + FN, FMO = FM / KG, FRAG_BYTES = 32 * BKB;
    constexpr int A_LOADS = BM / 8 / NW, B_LOADS = BN / 8 / NW, LOADS = A_LOADS + B_LOADS;
    // the waves that share a row block share its sums, if its blocks are so many
    constexpr int SHARE_B = FN % WM == 0 ? WM : 1;
    constexpr int NSUM_A = FM / WN, NSUM = NSUM_A + FN / SHARE_B;     // fragments a wave sums
    static_assert(FM % WN == 0, "the waves that share a row block share its sums");
    static_assert(KG == 1 || (KG == 2 && FM % 2 == 0), "each of two K groups finishes half of the rows of fragments");
    static_assert(NW == 4, "one wave per SIMD: issue slots are short, registers are not");
    extern __shared__ uint4 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)smem;

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int kg = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
    const int frow = lane & 31, fhalf = lane >> 5;
    const int ktiles = Kb / BKB, tiles = tiles_m * tiles_n;

    // ---- requests: global -> LDS, a stream of K tiles that runs on from one output tile into the next.  One wave-wide
    // load fills 8 tile rows of 128 bytes, whole cache lines; lane l lands in row l / 8, physical chunk l % 8, which
    // holds the logical chunk (l % 8) ^ ((row / 2) % 8).
    // (the last tile of a row or column of tiles ends with the matrix and overlaps its neighbour: the entries that
    // both compute are the same.)
    const uint8_t *a_next, *b_next;
    int req_tile = blockIdx.x, req_parity = 0;
    const uint32_t dma_off = (uint32_t)(lane >> 3) * Kb + ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) * 16;
    static_assert(NW % 2 == 0, "the swizzle is the same for all loads of a wave");
    // (one workgroup of four waves per CU issues too few instructions to spend scalar ones on addresses: offsets kept)
    constexpr int KEPT = A_LOADS > B_LOADS ? A_LOADS : B_LOADS;
    uint32_t load_off[KEPT];
#pragma unroll
    for (int g = 0; g < KEPT; ++g) load_off[g] = dma_off + (uint32_t)(g * 8 * NW) * Kb;
    auto origin = [&](int tile, int &row0, int &col0) {
        int bm, bn;
        tile_of_index(tile, tiles_m, tiles_n, bm, bn);
        row0 = fp6_tile_origin(bm, BM, T);
        col0 = fp6_tile_origin(bn, BN, N);
    };
    // first request of an output tile: where its rows lie; its dequantization steps go to LDS too (two sets alternate)
    auto open_tile = [&]() {
        int row0, col0;
        origin(req_tile, row0, col0);
        a_next = Qx + (int64_t)(row0 + 8 * wave) * Kb;
        b_next = Qw + (int64_t)(col0 + 8 * wave) * Kb;
        dma_begin(lds_base + G::SCALE_BYTE + req_parity * ((BM + BN) * 4) + wave * 256);
        for (int p = wave * kWave; p < BM + BN; p += NW * kWave)
            dma_4<NW * 256>(p < BM ? sx + row0 + p : sw + col0 + p - BM, lane * 4);
        req_parity ^= 1;
    };
    // loads of a K tile go to consecutive pieces of NW KB: its rows of tokens, then of weights
    auto issue_one = [&](int idx) {
        const uint8_t *base = idx < A_LOADS ? a_next : b_next;
        const int g = idx < A_LOADS ? idx : idx - A_LOADS;
        dma_16<NW * 1024>(base, load_off[g]);
    };
    auto start_requests = [&](int stage) { dma_begin(lds_base + (uint32_t)stage * G::STAGE + wave * 1024); };
    auto end_requests = [&]() {
        a_next += BKB;
        b_next += BKB;
    };
    // A walk over output tiles: past the last one of this workgroup that one is requested again, into dead stages, so
    // that the count of outstanding loads stays constant.
    auto next_tile = [&]() {
        if (req_tile + (int)gridDim.x < tiles) req_tile += gridDim.x;
        open_tile();
    };

    // Fragment c (0 .. FM - 1: tokens, then the weights) of this wave is row block c ^ wn of its tokens, block
    // (c - FM) ^ wm of its weights: the WN (WM) waves that share a row block hold it at different places, and each
    // sums the codes of the fragments at places that are multiples of WN (WM).
    // Byte offset in LDS: the lane's part (row, and chunk fhalf of the first step of this K group; a later step flips
    // bits of the chunk number above that one, which the swizzle passes through) plus a wave-uniform part.
    const int lane_off = lds_chunk_slot<BKB>(frow, 2 * kg * STEPS + fhalf) * 16;
    auto token_block = [&](int c) { return c ^ wn ^ (kg * FMO); };
    auto channel_block = [&](int j) { return SHARE_B == 1 ? j : j ^ wm; };
    auto part = [&](int c) {
        return c < FM ? (wm * FM + token_block(c)) * FRAG_BYTES : G::A_BYTES + (wn * FN + channel_block(c - FM)) * FRAG_BYTES;
    };
    const FieldMasks masks = field_masks();

    v16f acc[FM][FN];
    constexpr int RB = NF % 4 == 0 ? 4 : NF;      // chunks on their way from LDS
    static_assert(NF % RB == 0, "a chunk keeps its place from step to step");
    uint4 raw[RB];
    v6i frag[2][NF];
    v4f sum_acc[NSUM];                   // sums of the codes + 8, divided by 8
    const v6i sum_sel = sum_selector(lane);
    auto read_chunk = [&](int stage_byte, int s, int c) {
        raw[c % RB] = *reinterpret_cast<const uint4 *>(lds + ((lane_off ^ (32 * s)) + (stage_byte + part(c))));
    };
    // place of a fragment among those this wave sums, or -1
    auto sum_slot = [](int c) { return c < FM ? (c % WN == 0 ? c / WN : -1) : ((c - FM) % SHARE_B == 0 ? NSUM_A + (c - FM) / SHARE_B : -1); };
    auto convert_half = [&](int set, int c, int h) {
        const uint4 r = raw[c % RB];
        const uint32_t w0 = h ? r.z : r.x, w1 = h ? r.w : r.y;
        int d0, d1, d2;
        to_fp6(w0, w1, masks, d0, d1, d2);
        frag[set][c][3 * h] = d0, frag[set][c][3 * h + 1] = d1, frag[set][c][3 * h + 2] = d2;
    };
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll
        for (int u = 0; u < NSUM; ++u) sum_acc[u] = v4f{0.f, 0.f, 0.f, 0.f};
    };

    // One step of 64 codes, written in the order it should issue: every MFMA on frag[C] is followed by its share of
    // the conversion of raw (the next step, at N_BYTE, N_STEP) into frag[1 - C], and the place of a converted chunk is
    // refilled RB chunks ahead, in that step or the one behind it (A_BYTE, A_STEP).  LOAD0 .. LOAD1: the loads of a K
    // tile this step issues, from MFMA M0 on.  TURN: the turn between two K tiles, ahead of the first read of the next (the
    // K tiles that may still be on their way), or -1.  CONVERT, AHEAD: whether there is a next step, and one behind it.
    // (The row sums' instruction waits for the matrix core behind an MFMA: 256 x 256 tiles 0 - 1.5 % faster with it at the
    // end of a slot, 128 x 256 tiles 1 % slower.)
#define SQ_FP6_STEP(C, N_BYTE, N_STEP, A_BYTE, A_STEP, M0, LOAD0, LOAD1, TURN, CONVERT, AHEAD)                      \
    do {                                                                                                            \
        _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                                            \
            const int j = m / FM, i = m % FM;                                                                       \
            if ((TURN) >= 0 && m == (M0)) SQ_FP6_TURN(TURN);                                                        \
            acc[i][j] = mfma_fp6(frag[C][FM + j], frag[C][i], acc[i][j]);                                           \
            _Pragma("unroll") for (int c = 0; KG == 2 && c < NF; ++c)                                               \
                if (sum_slot(c) >= 0 && m == (2 * c + 1) * NM / (2 * NF)) mfma_fp6_16(frag[C][c], sum_sel, sum_acc[sum_slot(c)]); \
            _Pragma("unroll") for (int h = m * 2 * NF / NM; (CONVERT) && h < (m + 1) * 2 * NF / NM; ++h) {          \
                convert_half(1 - (C), h >> 1, h & 1);                                                               \
                if (h & 1) {                                                                                        \
                    const int t = (h >> 1) + RB;                                                                    \
                    if (t < NF) read_chunk(N_BYTE, N_STEP, t);                                                      \
                    else if (AHEAD) read_chunk(A_BYTE, A_STEP, t - NF);                                             \
                }                                                                                                   \
            }                                                                                                       \
            _Pragma("unroll") for (int q = (LOAD0); q < (LOAD1); ++q)                                               \
                if (m == (M0) + (q - (LOAD0)) * (NM - (M0)) / ((LOAD1) > (LOAD0) ? (LOAD1) - (LOAD0) : 1)) issue_one(q);   \
            if (KG == 1) __builtin_amdgcn_sched_barrier(0);                                                         \
            _Pragma("unroll") for (int c = 0; KG == 1 && c < NF; ++c)                                               \
                if (sum_slot(c) >= 0 && m == (2 * c + 1) * NM / (2 * NF)) mfma_fp6_16(frag[C][c], sum_sel, sum_acc[sum_slot(c)]); \
            __builtin_amdgcn_sched_barrier(0);                                                                      \
        }                                                                                                           \
    } while (0)
    // Between K tiles.  Loads complete in order: the next K tile has landed once only the LATER behind it are
    // outstanding.  All reads of this one have been issued and are drained here: its stage takes the one NS ahead.
#define SQ_FP6_TURN(LATER)                                                                                          \
    do {                                                                                                            \
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((LATER) * LOADS) : "memory");              \
        start_requests(cur);                                                                                        \
    } while (0)
    // One K tile.  The conversion runs ahead of the MFMAs: the last step converts the first step of the next K tile,
    // and stops behind the last one of the workgroup (LAST, two K groups).
    // LATER: K tiles requested beyond the next one; REQUEST: this K tile's turn requests another one.
#define SQ_FP6_TILE(LAST, LATER, REQUEST)                                                                           \
    do {                                                                                                            \
        const int next = cur + 1 == NS ? 0 : cur + 1;                                                               \
        const int cb = cur * G::STAGE, nb = next * G::STAGE;                                                        \
        constexpr int TURN_AT = ((2 * (NF - RB) + 2) * NM + 2 * NF - 1) / (2 * NF) - 1, FIRST = STEPS == 4 ? LOADS / 4 : LOADS / 6;                      \
        constexpr bool END = KG == 2 && (LAST);                                                                     \
        if constexpr (STEPS == 4) {                                                                                 \
            SQ_FP6_STEP(0, cb, 1 % STEPS, cb, 2 % STEPS, 0, 0, 0, -1, true, true);                                  \
            SQ_FP6_STEP(1, cb, 2 % STEPS, cb, 3 % STEPS, 0, 0, 0, -1, true, true);                                  \
        }                                                                                                           \
        SQ_FP6_STEP(0, cb, STEPS - 1, nb, 0, TURN_AT, 0, (REQUEST) ? FIRST : 0, END ? -1 : (LATER), true, !END);    \
        SQ_FP6_STEP(1, nb, 0, nb, 1, 0, (REQUEST) ? FIRST : 0, (REQUEST) ? LOADS : 0, -1, !END, true);              \
        if (REQUEST) end_requests();                                                                                \
        cur = next;                                                                                                 \
    } while (0)

    open_tile();
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        start_requests(t);
#pragma unroll
        for (int q = 0; q < LOADS; ++q) issue_one(q);
        end_requests();
    }
    wait_vmcnt<(NS - 1) * LOADS>();
    block_barrier();
#pragma unroll
    for (int c = 0; c < RB; ++c) read_chunk(0, 0, c);
#pragma unroll
    for (int c = 0; c < NF; ++c) {
        convert_half(0, c, 0);
        convert_half(0, c, 1);
        if (c + RB < NF) read_chunk(0, 0, c + RB);
        else read_chunk(0, 1, c + RB - NF);
    }

    int cur = 0, parity = 0;     // ring stage of the K tile being multiplied; set of dequantization steps
    for (int tile = blockIdx.x;;) {
        clear();
        for (int kt = NS; kt < ktiles; ++kt) SQ_FP6_TILE(false, NS - 2, true);
        if constexpr (KG == 1) {
            next_tile();
#pragma unroll
            for (int u = 1; u < NS; ++u) SQ_FP6_TILE(false, NS - 2, true);
            SQ_FP6_TILE(true, NS - 2, true);
        } else {                  // one output tile: nothing is requested behind it
            static_assert(KG == 1 || NS == 3, "two K tiles are left");
            SQ_FP6_TILE(false, 1, false);
            SQ_FP6_TILE(false, 0, false);
            SQ_FP6_TILE(true, 0, false);
        }

        // ---- epilogue.  The row sums meet in LDS, then every lane stores runs of eight channels of its token row
        // straight from registers.  The weights are the first MFMA operand: the 32 x 32 accumulator has the token in
        // the lane, and register e holds channel 8 (e / 4) + 4 (lane / 32) + e % 4.
        // (the lane's place is made opaque here, so that what only the epilogue needs of it does not sit in registers
        // through the loop above)
        int el = lane;
        asm volatile("" : "+v"(el));
        const int frow = el & 31, fhalf = el >> 5;
        float *sums = reinterpret_cast<float *>(lds + G::SUM_BYTE);
        const float *steps = reinterpret_cast<const float *>(lds + G::SCALE_BYTE) + parity * (BM + BN);
        typedef uint32_t v2u __attribute__((ext_vector_type(2)));
        // the results of the last matrix instructions: seven passes at most
#pragma unroll
        for (int u = 0; u < NSUM; ++u) asm volatile("s_nop 15" : "+v"(sum_acc[u]));
        // In LDS a row's share of the correction, a whole number: -8 sum b of a channel (its codes are 8 less than the fields)
        // and -8 sum a - 64 K of a token.
#pragma unroll
        for (int c = 0; c < NF; ++c) {
            const int u = sum_slot(c);
            if (u < 0) continue;
            const int row = c < FM ? (wm * FM + token_block(c)) * 32 : BM + (wn * FN + channel_block(c - FM)) * 32;
            const float codes8 = c < FM ? 0.f : (float)(128 / KG * Kb);      // 64 times the codes of this K group
            // accumulator of the 16 x 16 instruction: column l % 16, rows 4 (l / 16) + register; columns 0 and 1
            // hold the sums of rows 0 .. 15 and 16 .. 31 of the block
            if ((el & 15) < 2)
                *reinterpret_cast<float4 *>(sums + kg * (BM + BN) + row + 16 * (el & 15) + 4 * (el >> 4)) =
                    float4{fmaf(-64.f, sum_acc[u][0], codes8), fmaf(-64.f, sum_acc[u][1], codes8),
                           fmaf(-64.f, sum_acc[u][2], codes8), fmaf(-64.f, sum_acc[u][3], codes8)};
        }
        block_barrier();
        // The correction is c + t for channel c and token t: one matrix instruction of rank four per fragment adds it, in place of
        // two additions per entry.  A number below 2^23 is 4096 hi + lo, both whole and exact in fp16; the sums stay
        // multiples of 1/64 below 2^18, exact in fp32 in any order.
        auto halves = [&](int row) {
            const float x = KG == 2 ? sums[row] + sums[BM + BN + row] : sums[row], hi = rintf(x * (1.f / 4096.f));
            const uint32_t d = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(hi, fmaf(-4096.f, hi, x)));
            return fhalf == 0 ? d : 0u;
        };
        const uint32_t ones = fhalf == 0 ? 0x24005400u : 0u;         // 4096 / 64 and 1 / 64
        uint32_t token_halves[FMO];
#pragma unroll
        for (int i = 0; i < FMO; ++i) token_halves[i] = halves((wm * FM + token_block(i)) * 32 + frow);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const v4i channels = {(int)halves(BM + (wn * FN + channel_block(j)) * 32 + frow), (int)ones, 0, 0};
#pragma unroll
            for (int i = 0; i < FMO; ++i) {
                const v4i tokens = {(int)ones, (int)token_halves[i], 0, 0};
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, channels), __builtin_bit_cast(v8h, tokens),
                                                                   acc[i][j], 0, 0, 0);
            }
        }
        // A wave finishes its first FMO fragment rows, with the other K group's share of the sums (its last ones), which
        // comes through the ring (dead: one output tile per workgroup).
        float4 *part = reinterpret_cast<float4 *>(lds) + (wave % (WM * WN)) * (FMO * FN * 4 * kWave) + el;
        constexpr int HALF = WM * WN * FMO * FN * 4 * kWave;
        if constexpr (KG == 2) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FMO; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v16f &x = acc[FMO + i][j];
                        part[kg * HALF + ((j * FMO + i) * 4 + q) * kWave] = float4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
                    }
            block_barrier();
            part += (1 - kg) * HALF;
        }
        int row0, col0;
        origin(tile, row0, col0);
        const bool vector_stores = fp6_vector_stores(rows_aligned != 0, col0);
        float sxt[FMO];
        __half *ydst[FMO];
#pragma unroll
        for (int i = 0; i < FMO; ++i) {
            const int tl = (wm * FM + token_block(i)) * 32 + frow;
            sxt[i] = 64.f * steps[tl];
            ydst[i] = Y + (int64_t)(row0 + tl) * ldy + col0 + wn * (FN * 32) + 8 * fhalf + (vector_stores && (el & 16) ? 16 - 16 * ldy : 0);
        }
        // PLAIN: 16-byte stores and no accumulators asked for: no branch, so that the reads from LDS run ahead
        auto finish = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int nj = channel_block(j) * 32;                 // first channel of the fragment within this wave's
                float swn[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n4 = BM + wn * (FN * 32) + nj + 8 * q + 4 * fhalf;
                    const float4 s4 = *reinterpret_cast<const float4 *>(steps + n4);
                    swn[4 * q] = s4.x, swn[4 * q + 1] = s4.y, swn[4 * q + 2] = s4.z, swn[4 * q + 3] = s4.w;
                }
#pragma unroll
                for (int i = 0; i < FMO; ++i) {
                    v16f x = acc[i][j];
                    if constexpr (KG == 2) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4 p = part[((j * FMO + i) * 4 + q) * kWave];
                            x[4 * q] += p.x, x[4 * q + 1] += p.y, x[4 * q + 2] += p.z, x[4 * q + 3] += p.w;
                        }
                    }
                    uint4 w[2];                               // channels nj + 16 h + 8 fhalf ..
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint32_t run[2][2];
#pragma unroll
                        for (int e = 8 * h; e < 8 * h + 8; e += 2) {
                            run[(e / 4) & 1][(e / 2) & 1] = scaled_pair(x[e] * sxt[i], swn[e], x[e + 1] * sxt[i], swn[e + 1]);
                        }
                        // The swaps read a register two wait states behind the instruction that writes it at the earliest.  The
                        // compiler keeps that distance from the instructions it knows, not from those in assembly.
                        asm("s_nop 1" : "+v"(run[0][0]), "+v"(run[0][1]), "+v"(run[1][0]), "+v"(run[1][1]));
                        // lower half-wave: both halves of the first run; upper half-wave: of the second
                        const v2u s0 = __builtin_amdgcn_permlane32_swap(run[0][0], run[1][0], false, false);
                        const v2u s1 = __builtin_amdgcn_permlane32_swap(run[0][1], run[1][1], false, false);
                        w[h] = uint4{s0[0], s1[0], s0[1], s1[1]};
                    }
                    if (PLAIN || vector_stores) {
                        // sixteen rows of 64 bytes a store: rows l % 16, then the other sixteen (ydst is the lane's place)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            uint32_t &x0 = reinterpret_cast<uint32_t *>(&w[0])[r], &x1 = reinterpret_cast<uint32_t *>(&w[1])[r];
                            const v2u sw16 = __builtin_amdgcn_permlane16_swap(x0, x1, false, false);
                            x0 = sw16[0], x1 = sw16[1];
                        }
                        *reinterpret_cast<uint4 *>(ydst[i] + nj) = w[0];
                        *reinterpret_cast<uint4 *>(ydst[i] + 16 * ldy + nj) = w[1];
                    } else {
#pragma unroll
                        for (int e = 0; e < 16; ++e) {           // register-only: no addressable copy of the chunks
                            const uint32_t d[8] = {w[0].x, w[0].y, w[0].z, w[0].w, w[1].x, w[1].y, w[1].z, w[1].w};
                            reinterpret_cast<uint16_t *>(ydst[i] + nj + 8 * (e / 8))[e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
                        }
                    }
                    if (!PLAIN && acc_dbg != nullptr) {
                        const int t = row0 + (wm * FM + token_block(i)) * 32 + frow;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int n = col0 + wn * (FN * 32) + nj + 8 * (e / 4) + 4 * fhalf + (e % 4);
                            acc_dbg[(int64_t)t * N + n] = (int)(64.f * x[e]);
                        }
                    }
                }
            }
        };
        if constexpr (KG == 1) finish(std::false_type{});
        else if (vector_stores && acc_dbg == nullptr) finish(std::true_type{});
        else finish(std::false_type{});
        if (KG == 2 || tile + (int)gridDim.x >= tiles) break;
        tile += gridDim.x;
        parity ^= 1;
    }
    wait_vmcnt<0>();             // the requests past the end write to this workgroup's LDS
#undef SQ_FP6_TILE
#undef SQ_FP6_TURN
#undef SQ_FP6_STEP
}

template <int WM, int FM, int FN, int KG>
static sq_status launch(const uint8_t *Qx, const float *sx, int T, int K, const uint8_t *Qw, const float *sw, int N,
                        __half *Y, int64_t ldy, int32_t *acc_dbg, hipStream_t st)
{
    using G = Fp6Shape<WM, FM, FN, KG>;
    auto kernel = w4a4_gemm_fp6_kernel<WM, FM, FN, KG>;
    if (!allow_large_lds(reinterpret_cast<const void *>(kernel))) return SQ_ERR_LAUNCH;
    const int tiles_m = (T + G::BM - 1) / G::BM, tiles_n = (N + G::BN - 1) / G::BN, tiles = tiles_m * tiles_n;
    const int rows_aligned = fp6_rows_aligned((uintptr_t)Y, ldy) ? 1 : 0;
    static_assert(G::NS * 256 <= 768, "the requests run at most one output tile ahead");
    // One workgroup per CU walks over its output tiles: the loads of the next one run behind the epilogue (T = 8192,
    // K = 8192, N = 28672: 1060 -> 1037 us).  (Two K groups exchange their sums through the ring: one
    // output tile each.)
    const bool walk = KG == 1 && tiles > 256;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(walk ? 256 : tiles)), dim3(G::NT), G::LDS_BYTES, st, Qx, sx, T, K / 2, Qw,
                       sw, N, Y, ldy, acc_dbg, tiles_m, tiles_n, rows_aligned);
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

sq_status launch_w4a4_fp6(Fp6Tile tile, const uint8_t *Qx, const float *sx, int T, int K, const uint8_t *Qw,
                          const float *sw, int N, __half *Y, int64_t ldy, int32_t *acc_dbg, hipStream_t st)
{
    if (!w4a4_fp6_takes(tile, T, K, N)) return SQ_ERR_SHAPE;
    switch (tile) {
        case Fp6Tile::k128x192: return launch<1, 4, 3, 2>(Qx, sx, T, K, Qw, sw, N, Y, ldy, acc_dbg, st);
        case Fp6Tile::k128x256: return launch<1, 4, 4, 2>(Qx, sx, T, K, Qw, sw, N, Y, ldy, acc_dbg, st);
        case Fp6Tile::k256x192: return launch<2, 4, 3, 1>(Qx, sx, T, K, Qw, sw, N, Y, ldy, acc_dbg, st);
        default: return launch<2, 4, 4, 1>(Qx, sx, T, K, Qw, sw, N, Y, ldy, acc_dbg, st);
    }
}

}  // namespace sq
