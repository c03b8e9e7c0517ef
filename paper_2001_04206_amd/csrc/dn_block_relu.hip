// The sample-block kernel (dn_block.h) for relu hidden layers.
#include "dn_block.h"

namespace dn {

hipError_t block_relu(int units, int n2, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream)
{
    return block_dispatch<DN_ACT_RELU>(units, n2, g, plan, stream);
}

}  // namespace dn
