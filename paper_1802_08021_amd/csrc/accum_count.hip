// The tile pass that counts the root's union, with or without the node sizes
// (accum.h).  It reads no values.
#include "accum.h"

namespace sparcml {

hipError_t acc_count_launch(const AccArgs& a, bool info, hipStream_t s)
{
    return info ? acc_launch_p<8, kAccCount, true, false>(a, s) : acc_launch_p<2, kAccCount, false, false>(a, s);
}

}  // namespace sparcml
