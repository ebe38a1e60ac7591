// pair_mixed.hip -- mixed-precision all-pairs Lienard-Wiechert evaluation
// (Secs. 2.1-2.2 of arXiv 2605.05543 with the precision split below).
//
// The pass is the FP64 kernel's (pair_body in pair_kernel.h): the same
// LDS-staged FP64 history tiles and the same FP64 sign tests, so the bracket
// index is bit-identical to the FP64 path.  On gfx950 an FP32 and an FP64
// vector instruction issue at the same rate, so FP32 sign tests (which need
// a rounding band and an FP64 re-test inside it) would cost more than the
// exact test they stand in for.  The precision split is in the field
// evaluation of each pair (lw_pair_mixed):
//  * FP64: the offset r - w_1 to the bracket sample, the light-cone residual
//    at the root C0 = L1^2 - |r - w_1|^2 and the other coefficients of the
//    quadratic, the velocity at the root, the vector eta - |eta| v/c whose
//    length is the cancellation-prone 1 - eta_hat.beta, and the root
//    whenever the FP32 root fails its residual test (a rescue);
//  * FP32: the root, the reconstruction and the LW terms; the field sum is
//    accumulated with Knuth's two-sum into an FP32 (sum, error) pair.
#include "pair_kernel.h"

namespace empp {

extern const bool kHaveMixed = true;

template <bool KSTAR, bool COUNT, int GUESS, bool DB>
__global__ __launch_bounds__(kBlockFp64, 4) void pair_mixed_kernel(PairParams p)
{
    pair_body<true, KSTAR, COUNT, GUESS, false, false, DB>(p);
}

namespace {

template <bool K, bool C, int G, bool DB>
void launch_kernel(const PairParams &p, dim3 grid, hipStream_t stream)
{
    const size_t lds = pair_lds_bytes(p.D);
    (void)hipFuncSetAttribute((const void *)pair_mixed_kernel<K, C, G, DB>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((pair_mixed_kernel<K, C, G, DB>), grid, dim3(kBlockFp64), lds, stream, p);
}

template <bool K, bool C, int G>
void launch_mode(const PairParams &p, dim3 grid, hipStream_t stream)
{
    if (pair_two_buffers(p.D))
        launch_kernel<K, C, G, true>(p, grid, stream);
    else
        launch_kernel<K, C, G, false>(p, grid, stream);
}

}  // namespace

hipError_t launch_pair_mixed(const PairParams &p, hipStream_t stream, bool kstar, bool count)
{
    // fixed step, no warm start, linear reconstruction, one wavefront per target
    if (p.guess > 3 || p.ad || p.recon == 1 || p.sg_log2 != 0)
        return hipErrorInvalidValue;
    const int64_t nblocks = (p.m + kBlockFp64 - 1) / kBlockFp64 * p.nsplit;
    if (nblocks < 1 || nblocks > INT32_MAX)
        return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)nblocks);
#define EMPP_BY_GUESS(K, C)                                                                                  \
    do {                                                                                                    \
        if (p.guess == 3) launch_mode<K, C, 3>(p, grid, stream);                                             \
        else if (p.guess == 2) launch_mode<K, C, 2>(p, grid, stream);                                        \
        else if (p.guess == 1) launch_mode<K, C, 1>(p, grid, stream);                                        \
        else launch_mode<K, C, 0>(p, grid, stream);                                                          \
    } while (0)
    if (kstar) {
        if (count) EMPP_BY_GUESS(true, true); else EMPP_BY_GUESS(true, false);
    } else {
        if (count) EMPP_BY_GUESS(false, true); else EMPP_BY_GUESS(false, false);
    }
#undef EMPP_BY_GUESS
    return hipGetLastError();
}

}  // namespace empp
