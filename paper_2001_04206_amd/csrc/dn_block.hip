// Host side of the sample-block kernel (dn_block.h), and its compilation for linear and sigmoid hidden layers; the other
// activation functions are sources of their own, so that they compile beside each other.
#include "dn_block.h"

namespace dn {

hipError_t block_tanh(int units, int n2, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream);
hipError_t block_relu(int units, int n2, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream);

static hipError_t block_act(int units, int n2, int act, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream)
{
    switch (act) {
    case DN_ACT_SIGMOID: return block_dispatch<DN_ACT_SIGMOID>(units, n2, g, plan, stream);
    case DN_ACT_TANH: return block_tanh(units, n2, g, plan, stream);
    case DN_ACT_RELU: return block_relu(units, n2, g, plan, stream);
    default: return block_dispatch<DN_ACT_LINEAR>(units, n2, g, plan, stream);
    }
}

bool block_geometry(const int32_t *n, int L, BlockGeom &g)
{
    g = BlockGeom{};
    // (layers of at most 64: one wavefront's, whose arena need not hold the blocks' inner products)
    if (L != 2 || (n[0] <= 64 && n[1] <= 64 && n[2] <= 64)) return false;
    if (n[0] < 4 || n[0] > 1024 || n[1] < 1 || n[2] < 1 || n[2] > 64) return false;
    g.units_per_lane = n[2] <= 16 ? (n[1] <= 64 ? 1 : (n[1] <= 512 ? 2 : 4)) : (n[1] <= 256 ? 1 : 2);
    g.chain_waves = (n[1] + 64 * g.units_per_lane - 1) / (64 * g.units_per_lane);
    if (g.chain_waves > 4) return false;
    g.grid = 1 + BLOCK_GRAM_GROUPS + (n[1] + 3) / 4;
    return g.grid <= ON_MAX_WG;
}

size_t block_exchange_bytes(const int32_t *n, int L)
{
    BlockGeom g;
    if (!block_geometry(n, L, g)) return 0;
    const size_t words = 2 * (size_t)TB * (n[1] + (size_t)g.chain_waves * g.units_per_lane * 64);
    return (words + (size_t)(BLOCK_LAUNCH_SAMPLES / TB) * kRecord) * sizeof(u64);
}

hipError_t block_prepare(const int32_t *n, int act)
{
    BlockGeom g;
    if (!block_geometry(n, 2, g)) return hipErrorInvalidValue;
    return block_act(g.units_per_lane, n[2], act, nullptr, nullptr, nullptr);
}

hipError_t launch_block_epoch(const BlockGeom &g, BlockPlan plan, unsigned long long *exchange, hipStream_t stream)
{
    if (plan.n_samples < 1 || plan.n_samples > BLOCK_LAUNCH_SAMPLES) return hipErrorInvalidValue;
    if (!plan.arrived || !plan.settled) return hipErrorInvalidValue;
    plan.chain_waves = g.chain_waves;
    plan.d_stride = g.chain_waves * g.units_per_lane * 64;
    plan.z_x = exchange;
    plan.d_x = plan.z_x + 2 * (size_t)TB * plan.n1;
    plan.gram_x = plan.d_x + 2 * (size_t)TB * plan.d_stride;
    return block_act(g.units_per_lane, plan.n2, plan.act1, &g, &plan, stream);
}

}  // namespace dn
