// The tile pass writing a sparse root (accum.h).
#include "accum.h"

namespace sparcml {

hipError_t acc_write_launch(const AccArgs& a, uint32_t nb, hipStream_t s)
{
    if (nb == 2u)
        return a.qbits ? acc_launch_p<2, kAccWrite, false, true>(a, s) : acc_launch_p<2, kAccWrite, false, false>(a, s);
    if (nb == 4u)
        return a.qbits ? acc_launch_p<4, kAccWrite, false, true>(a, s) : acc_launch_p<4, kAccWrite, false, false>(a, s);
    return a.qbits ? acc_launch_p<8, kAccWrite, false, true>(a, s) : acc_launch_p<8, kAccWrite, false, false>(a, s);
}

}  // namespace sparcml
