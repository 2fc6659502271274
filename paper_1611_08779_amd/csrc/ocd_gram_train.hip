// ocd_gram_train.hip -- the training step in the Gram form (ocd_gram_grad.h).
#include "ocd_gram_grad.h"

namespace ocd {

hipError_t launch_gram_train(bool f16, const Params &p, int max_blocks, size_t limit, hipStream_t s)
{
    return launch_grad<true>(f16, p, max_blocks, limit, s);
}

}  // namespace ocd
