// The sample-block kernel (dn_block.h) for tanh hidden layers.
#include "dn_block.h"

namespace dn {

hipError_t block_tanh(int units, int n2, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream)
{
    return block_dispatch<DN_ACT_TANH>(units, n2, g, plan, stream);
}

}  // namespace dn
