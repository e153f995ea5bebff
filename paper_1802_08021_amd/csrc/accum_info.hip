// The tile pass writing a dense root and counting the node sizes (accum.h).
#include "accum.h"

namespace sparcml {

hipError_t acc_dense_info_launch(const AccArgs& a, hipStream_t s)
{
    return a.qbits ? acc_launch_p<8, kAccDense, true, true>(a, s) : acc_launch_p<8, kAccDense, true, false>(a, s);
}

}  // namespace sparcml
