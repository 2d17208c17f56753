// Row-marching kernel instantiations without the point lists.
#include "rowfuse.h"

namespace fz {

hipError_t launch_rowfuse_direct(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s)
{
    return pick_rowfuse<false>(rp, K, rgb, diff, s);
}

}  // namespace fz
