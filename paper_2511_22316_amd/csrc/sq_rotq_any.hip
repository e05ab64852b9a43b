// The matrix-core kernel of sq_rotate_quantize for any number of rows: 8 <= n1 <= 128 with n2 = 32, 64 or 128.
//
// What Alg. 1 makes of a layer width K is nearly always such a pair (K = 3072: 48 x 64, K = 10880: 85 x 128), and a
// width without an instantiation of its own in sq_rotq_mfma.hip used to take the plain-FMA kernel, which is bound by
// its LDS reads: one per two fp32 FMAs.  Here the rows of a token are padded to the 32-row blocks of the
// matrix instruction, as they are there, and only their number is an argument; padding rows are zeros in LDS
// that nothing is ever loaded over.  R1 has rows of n1 halves, so its chunks start at any even byte.
// 48 x 64 at T = 1001: 45.9 us there, 10.7 us here (layer with N = 9216: 78.4 -> 38.5 us).
//
// The plain-FMA kernel holds everything as fp32; the split Z and the Givens values carry scales here that keep the error
// below that kernel's (rotate_quantize_mfma_body, ANY_N1; they cost 2 - 4 % of the kernel).  Error against 64 bits, relative
// to the norm, P = 64 (plain-FMA kernel / here):
//                                  48 x 64            85 x 128           20 x 32
//   outliers of 1000, body of 1    1.8e-7 / 1.2e-7    2.5e-7 / 1.5e-7    1.3e-7 / 1.2e-7
//   rows of 0.02 (weights)         1.8e-7 / 1.1e-7    2.5e-7 / 1.4e-7    1.3e-7 / 1.0e-7
//   rows of 0.001                  1.8e-7 / 1.1e-7    2.5e-7 / 1.4e-7    1.3e-7 / 1.0e-7
// and, with R2 in blocks, on columns smaller than the others of the same wave by
//   10^-3                          1.4e-7 / 0.9e-7    1.8e-7 / 1.1e-7    1.1e-7 / 0.8e-7
//   10^-4                          1.4e-7 / 0.9e-7    1.8e-7 / 1.1e-7    1.0e-7 / 0.8e-7
//   10^-5                          1.4e-7 / 2.4e-7    1.8e-7 / 2.7e-7    1.0e-7 / 2.3e-7
//
// The operands are R1 and R2 as they are, also behind a prepared rotation (it holds copies of both): its
// layout for these pairs stays what it was.
#include "sq_rotq_body.h"

namespace sq {

namespace {

template <int N1P, int N2, int OCC, int QS_MAX, int NSX, bool R1LDS, bool CLIP>
__global__ __launch_bounds__(256, OCC) void rotate_quantize_any_kernel(
    const __half *__restrict__ X, int64_t ldx, int T, RotqPlan plan, const __half *__restrict__ R1,
    const __half *__restrict__ R2, uint8_t *__restrict__ Q, float *__restrict__ scales, float *__restrict__ xrot,
    int sides, int n1)
{
    extern __shared__ uint4 smem_u4[];
    rotate_quantize_mfma_body<N1P, N2, QS_MAX, NSX, R1LDS, false, false, CLIP, true>(
        X, ldx, T, plan, R1, R2, Q, scales, xrot, (int)blockIdx.x, (int)gridDim.x, smem_u4, sides, nullptr, 0, n1);
}

template <int N1P, int N2, int OCC, int QS_MAX, int NSX, bool R1LDS>
__global__ __launch_bounds__(256, OCC) void rotate_fp16_any_kernel(
    const __half *__restrict__ X, int64_t ldx, int T, RotqPlan plan, const __half *__restrict__ R1,
    const __half *__restrict__ R2, __half *__restrict__ xout, int64_t ldo, int sides, int n1)
{
    extern __shared__ uint4 smem_u4[];
    rotate_quantize_mfma_body<N1P, N2, QS_MAX, NSX, R1LDS, false, true, false, true>(
        X, ldx, T, plan, R1, R2, nullptr, nullptr, nullptr, (int)blockIdx.x, (int)gridDim.x, smem_u4, sides, xout, ldo,
        n1);
}

struct AnyArgs {
    const __half *X;
    int64_t ldx;
    int T, n1;
    const __half *R1, *R2;
    uint8_t *Q;
    float *scales, *xrot;
    __half *xout;          // not null: the rotated rows leave as fp16, no quantizer
    int64_t ldo;
};

template <int N1P, int N2, int QS_MAX, int NSX, int OCC, bool R1LDS>
sq_status launch_ring(const AnyArgs &a, const RotqPlan &plan, hipStream_t st)
{
    using S = RotqShape<N1P, N2, NSX, R1LDS>;
    const int qsteps = (plan.n_qslots + 15) / 16;
    const int sides = S::side_tiles(qsteps, OCC), lds = S::lds_bytes(qsteps, sides);
    if (lds > kMaxDynamicLds) return SQ_ERR_SHAPE;
    const int groups = (a.T + S::TPP - 1) / S::TPP, by_lds = (160 * 1024) / lds;
    const int resident = 256 * (by_lds < OCC ? by_lds : OCC);
    const dim3 grid((unsigned)(groups < resident ? groups : resident));
    if (a.xout != nullptr) {
        auto kernel = rotate_fp16_any_kernel<N1P, N2, OCC, QS_MAX, NSX, R1LDS>;
        if (!allow_large_lds(reinterpret_cast<const void *>(kernel))) return SQ_ERR_LAUNCH;
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, a.X, a.ldx, a.T, plan, a.R1, a.R2, a.xout, a.ldo, sides, a.n1);
    } else {
        auto kernel = plan.clip < 1.0f ? rotate_quantize_any_kernel<N1P, N2, OCC, QS_MAX, NSX, R1LDS, true>
                                       : rotate_quantize_any_kernel<N1P, N2, OCC, QS_MAX, NSX, R1LDS, false>;
        if (!allow_large_lds(reinterpret_cast<const void *>(kernel))) return SQ_ERR_LAUNCH;
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, a.X, a.ldx, a.T, plan, a.R1, a.R2, a.Q, a.scales, a.xrot, sides,
                           a.n1);
    }
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

// The ring and the place of R1 as in sq_rotq_mfma.hip: two workgroups per CU where the registers and LDS allow it.
template <int N1P, int N2, int QS_MAX>
sq_status launch_qs(const AnyArgs &a, const RotqPlan &plan, hipStream_t st)
{
    if constexpr (N1P == 96 && QS_MAX == 4) {
        using S2 = RotqShape<N1P, N2, 2, true>;
        if (2 * S2::lds_bytes((plan.n_qslots + 15) / 16, 1) <= 160 * 1024)
            return launch_ring<N1P, N2, QS_MAX, 2, 2, true>(a, plan, st);
    }
    return launch_ring<N1P, N2, QS_MAX, 3, (N1P <= 64) ? 2 : 1, false>(a, plan, st);
}

template <int N2>
sq_status launch_rows(const AnyArgs &a, const RotqPlan &plan, hipStream_t st)
{
    if constexpr (N2 == 128) {
        if (plan.n_qslots > 64) {
            if (a.n1 <= 32) return launch_qs<32, N2, 8>(a, plan, st);
            if (a.n1 <= 64) return launch_qs<64, N2, 8>(a, plan, st);
            if (a.n1 <= 96) return launch_qs<96, N2, 8>(a, plan, st);
            return launch_qs<128, N2, 8>(a, plan, st);
        }
    }
    if (a.n1 <= 32) return launch_qs<32, N2, 4>(a, plan, st);
    if (a.n1 <= 64) return launch_qs<64, N2, 4>(a, plan, st);
    if (a.n1 <= 96) return launch_qs<96, N2, 4>(a, plan, st);
    return launch_qs<128, N2, 4>(a, plan, st);
}

}  // namespace

bool rotq_any_covers(int n1, int n2) { return n1 >= 8 && n1 <= 128 && (n2 == 32 || n2 == 64 || n2 == 128); }

sq_status rotq_any_launch(const __half *X, int64_t ldx, int T, int n1, int n2, const RotqPlan &plan, const __half *R1,
                          const __half *R2, uint8_t *Q, float *scales, float *xrot, __half *xout, int64_t ldo,
                          hipStream_t st)
{
    if (!rotq_any_covers(n1, n2)) return SQ_ERR_SHAPE;
    const AnyArgs a = {X, ldx, T, n1, R1, R2, Q, scales, xrot, xout, ldo};
    return n2 == 32 ? launch_rows<32>(a, plan, st) : n2 == 64 ? launch_rows<64>(a, plan, st) : launch_rows<128>(a, plan, st);
}

}  // namespace sq
