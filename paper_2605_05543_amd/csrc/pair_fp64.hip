// pair_fp64.hip -- all-pairs Lienard-Wiechert field evaluation in double
// precision (Secs. 2.1-2.2 of arXiv 2605.05543): the plain path, its
// adaptive-step reductions, the warm-started search and the midpoint
// ablation.  The pass itself is pair_body in pair_kernel.h.
#include "pair_kernel.h"

namespace empp {

template <bool KSTAR, bool COUNT, int GUESS, bool ADAPT, bool MID, bool DB>
__global__ __launch_bounds__(kBlockFp64, 4) void pair_fp64_kernel(PairParams p)
{
    pair_body<false, KSTAR, COUNT, GUESS, ADAPT, MID, DB>(p);
}

// Sources per staged LDS tile.
int pair_fp64_tile(int D) { return pair_staged_tile(D); }

namespace {

template <bool K, bool C, int G, bool A, bool MID, bool DB>
void launch_kernel(const PairParams &p, dim3 grid, hipStream_t stream)
{
    const size_t lds = pair_lds_bytes(p.D);
    (void)hipFuncSetAttribute((const void *)pair_fp64_kernel<K, C, G, A, MID, DB>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((pair_fp64_kernel<K, C, G, A, MID, DB>), grid, dim3(kBlockFp64), lds, stream, p);
}

template <bool K, bool C, int G, bool A, bool MID = false>
void launch_mode(const PairParams &p, dim3 grid, hipStream_t stream)
{
    if (pair_two_buffers(p.D))
        launch_kernel<K, C, G, A, MID, true>(p, grid, stream);
    else
        launch_kernel<K, C, G, A, MID, false>(p, grid, stream);
}

}  // namespace

// Host-side launcher (called from the C ABI layer).
hipError_t launch_pair_fp64(const PairParams &p, hipStream_t stream, bool kstar, bool count)
{
    const int64_t targets = kBlockFp64 >> p.sg_log2;
    const int64_t nblocks = (p.m + targets - 1) / targets * p.nsplit;
    if (nblocks < 1 || nblocks > INT32_MAX)
        return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)nblocks);
#define EMPP_MODE(K, C, G, A) launch_mode<K, C, G, A>(p, grid, stream)
#define EMPP_BY_COUNT(K, G) \
    do { if (count) EMPP_MODE(K, true, G, false); else EMPP_MODE(K, false, G, false); } while (0)
#define EMPP_BY_ADAPT(C, G) \
    do { if (p.ad) EMPP_MODE(false, C, G, true); else EMPP_MODE(false, C, G, false); } while (0)
    if (p.ad && (kstar || p.x || p.guess == 1 || p.guess == 3))
        return hipErrorInvalidValue;  // the adaptive step is taken in step mode
    if (p.recon == 1) {
        // midpoint ablation: the paper's bisection, fixed step, any target mode
        if (p.ad || count)
            return hipErrorInvalidValue;
        if (kstar)
            launch_mode<true, false, 0, false, true>(p, grid, stream);
        else
            launch_mode<false, false, 0, false, true>(p, grid, stream);
        return hipGetLastError();
    }
    if (p.guess == 4) {
        // warm start: step mode only (no per-pair k* output); the first
        // step of a run searches afresh and fills the cache (search mode 5)
        if (kstar || !p.kc || p.x)
            return hipErrorInvalidValue;
        if (p.kc_cold) {
            if (count) EMPP_BY_ADAPT(true, 5); else EMPP_BY_ADAPT(false, 5);
        } else {
            if (count) EMPP_BY_ADAPT(true, 4); else EMPP_BY_ADAPT(false, 4);
        }
    } else if (kstar) {
        if (p.guess == 2) EMPP_BY_COUNT(true, 2);
        else if (p.guess == 3) EMPP_BY_COUNT(true, 3);
        else if (p.guess == 1) EMPP_BY_COUNT(true, 1);
        else EMPP_BY_COUNT(true, 0);
    } else if (p.guess == 3) {
        EMPP_BY_COUNT(false, 3);
    } else if (p.guess == 1) {
        EMPP_BY_COUNT(false, 1);
    } else if (p.guess == 2) {
        if (count) EMPP_BY_ADAPT(true, 2); else EMPP_BY_ADAPT(false, 2);
    } else {
        if (count) EMPP_BY_ADAPT(true, 0); else EMPP_BY_ADAPT(false, 0);
    }
#undef EMPP_BY_ADAPT
#undef EMPP_BY_COUNT
#undef EMPP_MODE
    return hipGetLastError();
}

}  // namespace empp
