// ea_half_c2.hip -- fused-round and split-call kernels for buckets of 512 elements
// (2 chunks per tile) with the worker quantizer fixed at compile time: scaled
// sign, stochastic uniform with 1, 2, 4 or 8 bits and an L2 or max-norm
// scale, top-k, random-k, Example 1 with 2 or 3 bits, and (with no bucket,
// so at any tile size) Example 2 with 4-bit codes and full precision.  The
// server quantizer and the Adam placement are read at run time.  The
// workers' per-element work is N times the server's, so these kernels run
// close to the fully specialized ones.
#include "ea_round.hpp"

namespace ea {

namespace {

// MW: minimum waves per SIMD, 0 for the tile's own.  Top-k fits 72 registers,
// three 8-wave blocks a CU instead of two (40M parameters, 8 workers, top-16
// of 512 under a sign server 1063 -> 900 us).
template <class QW, int MW = 0>
constexpr HalfKernel half()
{
    return HalfKernel{2, QW::kind(QDev{}), QW::bits(QDev{}), QW::norm(QDev{}), QW::cpb(QDev{}),
                      step_kernel<2, QW, QRt, -1, MW>, kernel_tiles(2, -1, true),
                      worker_kernel<2, QW>, aggregate_kernel<2, QW>,
                      server_kernel<2, QW>, apply_kernel<2, QW>};
}

const HalfKernel kHalf[] = {
    half<QCt<Q_SCALED_SIGN, 1, S_L1, 2>>(),
    half<QCt<Q_STOCH, 1, S_L2, 2>>(),
    half<QCt<Q_STOCH, 1, S_MAX, 2>>(),
    half<QCt<Q_STOCH, 2, S_L2, 2>>(),
    half<QCt<Q_STOCH, 2, S_MAX, 2>>(),
    half<QCt<Q_STOCH, 4, S_L2, 2>>(),
    half<QCt<Q_STOCH, 4, S_MAX, 2>>(),
    half<QCt<Q_STOCH, 8, S_L2, 2>>(),
    half<QCt<Q_STOCH, 8, S_MAX, 2>>(),
    half<QCt<Q_TOPK, 1, S_MAX, 2>, 7>(),
    half<QCt<Q_RANDK, 1, S_MAX, 2>>(),
    half<QCt<Q_DET, 2, S_MAX, 2>>(),
    half<QCt<Q_DET, 3, S_MAX, 2>>(),
    half<QCt<Q_POW2, 4, S_MAX, 0>>(),
    half<QCt<Q_NONE, 32, S_MAX, 0>>(),
    // one bucket over the vector: the scale is given, whichever norm it is
    half<QCt<Q_SCALED_SIGN, 1, S_MAX, 0>>(),
    half<QCt<Q_STOCH, 1, S_MAX, 0>>(),
    half<QCt<Q_STOCH, 2, S_MAX, 0>>(),
    half<QCt<Q_STOCH, 4, S_MAX, 0>>(),
    half<QCt<Q_STOCH, 8, S_MAX, 0>>(),
    half<QCt<Q_DET, 2, S_MAX, 0>>(),
    half<QCt<Q_DET, 3, S_MAX, 0>>(),
};

}  // namespace

const HalfKernel* half_kernels_c2(int* n)
{
    *n = (int)(sizeof(kHalf) / sizeof(kHalf[0]));
    return kHalf;
}

}  // namespace ea
