// The packed expansion in double (a file of its own: every degree, nmax and
// chunk is a kernel, and the two precisions compile side by side).
#include "expansion_packed.hpp"

namespace soap {

hipError_t launch_packed_f64(const FeatureArgs& a, const PackLayout& W, hipStream_t st)
{
    return launch_packed<double>(a, W, st);
}

}  // namespace soap
