// ea_half_wide_c12.hip -- fused-round and split-call kernels with the worker
// quantizer fixed at compile time, as in ea_half_c*.hip, for the wider
// deterministic codes: Example 1 with 4 to 8 bits in buckets of 256 and 512
// elements, and Example 2 with 5-bit codes on tiles of those sizes. Example 1 with 4 to 8 bits also with one
// bucket over the vector.
#include "ea_round.hpp"

namespace ea {

namespace {

template <int C, class QW>
constexpr HalfKernel half()
{
    return HalfKernel{C, QW::kind(QDev{}), QW::bits(QDev{}), QW::norm(QDev{}), QW::cpb(QDev{}),
                      step_kernel<C, QW, QRt, -1>, kernel_tiles(C, -1, true),
                      worker_kernel<C, QW>, aggregate_kernel<C, QW>,
                      server_kernel<C, QW>, apply_kernel<C, QW>};
}

const HalfKernel kHalf[] = {
    half<1, QCt<Q_DET, 4, S_MAX, 1>>(),
    half<1, QCt<Q_DET, 5, S_MAX, 1>>(),
    half<1, QCt<Q_DET, 6, S_MAX, 1>>(),
    half<1, QCt<Q_DET, 7, S_MAX, 1>>(),
    half<1, QCt<Q_DET, 8, S_MAX, 1>>(),
    half<1, QCt<Q_POW2, 5, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 4, S_MAX, 2>>(),
    half<2, QCt<Q_DET, 5, S_MAX, 2>>(),
    half<2, QCt<Q_DET, 6, S_MAX, 2>>(),
    half<2, QCt<Q_DET, 7, S_MAX, 2>>(),
    half<2, QCt<Q_DET, 8, S_MAX, 2>>(),
    half<2, QCt<Q_POW2, 5, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 4, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 5, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 6, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 7, S_MAX, 0>>(),
    half<2, QCt<Q_DET, 8, S_MAX, 0>>(),
};

}  // namespace

const HalfKernel* half_kernels_wide_c12(int* n)
{
    *n = (int)(sizeof(kHalf) / sizeof(kHalf[0]));
    return kHalf;
}

}  // namespace ea
