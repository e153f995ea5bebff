// The tile pass writing a dense root (see accum.h), without node sizes.
#include "accum.h"

namespace sparcml {

hipError_t acc_dense_info_launch(const AccArgs& a, hipStream_t s);  // accum_info.hip

hipError_t acc_dense_launch(const AccArgs& a, uint32_t nb, bool info, hipStream_t s)
{
    if (info) return acc_dense_info_launch(a, s);
    if (nb == 2u)
        return a.qbits ? acc_launch_p<2, kAccDense, false, true>(a, s) : acc_launch_p<2, kAccDense, false, false>(a, s);
    if (nb == 4u)
        return a.qbits ? acc_launch_p<4, kAccDense, false, true>(a, s) : acc_launch_p<4, kAccDense, false, false>(a, s);
    return a.qbits ? acc_launch_p<8, kAccDense, false, true>(a, s) : acc_launch_p<8, kAccDense, false, false>(a, s);
}

}  // namespace sparcml
