// ocd_gram_backward.hip -- the adjoint in the Gram form (ocd_gram_grad.h).
#include "ocd_gram_grad.h"

namespace ocd {

hipError_t launch_gram_backward(bool f16, const Params &p, int max_blocks, size_t limit,
                                hipStream_t s)
{
    return launch_grad<false>(f16, p, max_blocks, limit, s);
}

}  // namespace ocd
