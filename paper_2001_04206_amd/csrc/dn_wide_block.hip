// Per-sample (batch 1) training of two-layer nets whose hidden layer is too wide for one compute unit -- the network the paper
// trains, 340 inputs, 100000 hidden units, 10 outputs (section "Experimental Evaluation") -- plain gradient descent, the
// samples in blocks of 32 as in dn_block.h: W_1 is read and written once per block.
//
// Every workgroup owns a block of hidden units.  Four of its eight waves take the steps (run_steps of dn_block.h: the output
// layer's sums over all workgroups are the one thing a step waits for), the other four meanwhile sweep the workgroup's rows of
// W_1 through the matrix cores: a tile of 32 units x 32 inputs comes from memory, takes the last block's 32 rank-1 updates
// (W^T += X^T (-lr Delta), sixteen v_mfma_f32_32x32x2_f32 with the tile as accumulator), goes back, and meets the features
// of the block after next (sixteen more; the accumulator's registers are operand B of that product as they are, with the
// inputs paired 8 q + e and 8 q + 4 + e).  Net inputs of a block and its deltas share their place in LDS.
//
// What bounds it: the exchange.  340-100000-10, 256 samples, workgroup 0, cycles per step: activations and own sums 980, exchange
// 10700 (two hops of 3900 and waiting for the slowest of sixteen workgroups), output layer 690, deltas and corrections 590;
// a block's sweep is 30 us of matrix instructions beside 180 us of steps.  us per step, a pass with it divided by its samples:
// 340-100000-10, 256 samples 20.8 -> 5.5 to 6.5 on several cards (a pass 5335 -> 1410 to 1651; one card repeats itself within
// 0.6 %), 512 samples 5.1 to 5.9; 340-60001-10 15.6 -> 6.3 and 384-40000-3 14.3 -> 6.0 in passes of 130 and 96 samples.  Exchanges tried: every workgroup reads
// all 2560 words, by workgroup 12.3 us a step, by output (whole lines) 9.0; two levels 7.7, with three looks on their way at a
// time 8.7 (the looks hold up the words), with eight copies of the upper level 6.9; steps before the sweep (s_setprio) 6.8.
// The sweep is not what a step waits for: with one long sum instead of one per tile, or without the loads of a tile ahead, a pass
// takes the same time on one card (6.51, 6.53 and 6.53 in turn).
// Two waves on a SIMD leave a lane 256 registers: 66 to 68 of its numbers live in scratch memory for up to 10 outputs, 94 for 16
// (340-100000-k, 512 samples: 5.4 us a step for 3 outputs, 5.6 for 10, 6.2 to 6.8 for 11 to 16).
#define DN_PERSIST_THREADS 512   // four waves for the steps, four for the sweep
#include "dn_block.h"

namespace dn {
namespace {

constexpr int kStepThreads = 256;

// This wave's share of the sweep: groups of 32 units, each whole or (one group left over) every fourth tile of it.
struct Share {
    int groups, whole0, extra;   // whole groups whole0 .. whole0 + groups - 1; extra: a group to share, or -1
};
__device__ __forceinline__ Share share_of(int count, int sweeper)
{
    const int g = (count + 31) / 32, each = g / 4, rest = g % 4;
    Share s;
    s.groups = each + (rest > 1 && sweeper < rest ? 1 : 0);
    s.whole0 = each * sweeper + (rest > 1 ? min(sweeper, rest) : 0);
    s.extra = rest == 1 ? g - 1 : -1;
    return s;
}

struct TileOperands {
    v4f w[4];       // lane 32 h + c: unit c, inputs 8 q + 4 h ..
    float xu[16];   // lane 32 h + i: sample 2 s + h of the block whose update is due, input i
    v4f xf[4];      // lane 32 h + i: sample i of the block whose net inputs are due, inputs 8 q + 4 h ..
};

// update: block whose deltas W_1 takes (their net inputs' place in LDS holds them), -1 for none; products: block whose net
// inputs are formed, -1 for none; velocity: leave the last step's change as velocity.
__device__ __forceinline__ void sweep(const BlockPlan &p, const ChainLds &l, int update, int products, bool velocity)
{
    const int lane = threadIdx.x & 63, sweeper = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) - 4;
    const int c = lane & 31, h = lane >> 5;
    const int n0 = p.n0, stride = p.d_stride, base = (int)blockIdx.x * p.per, count = min(p.per, p.n1 - base), n = (int)p.n_samples;
    const int tiles = (n0 + 31) / 32;
    const Share sh = share_of(count, sweeper);
    const float *deltas = l.zc + (update & 1) * TB * stride;
    float *to = l.zc + (products & 1) * TB * stride;
    const float *xf_row = p.X + (size_t)min(max(products, 0) * TB + c, n - 1) * n0;
    const int last = n - 1;
    for (int i = 0; i < sh.groups + (sh.extra >= 0 ? 1 : 0); ++i) {
        const bool shared = i == sh.groups;
        const int g = shared ? sh.extra : sh.whole0 + i, unit = 32 * g + c;
        const size_t row = (size_t)(base + min(unit, count - 1)) * n0;
        float nld[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) nld[s] = update >= 0 ? deltas[(2 * s + h) * stride + unit] : 0.f;
        v16f total;
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] = 0.f;
        auto load = [&](TileOperands &t, int tile) {
            const int f0 = 32 * tile;
#pragma unroll
            for (int q = 0; q < 4; ++q) t.w[q] = *(const v4f *)(p.W1 + row + min(f0 + 8 * q + 4 * h, n0 - 4));
            if (update >= 0) {
                const int f = min(f0 + c, n0 - 1);
#pragma unroll
                for (int s = 0; s < 16; ++s) t.xu[s] = p.X[(uint32_t)(min(update * TB + 2 * s + h, last) * n0 + f)];
            }
            if (products >= 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) t.xf[q] = *(const v4f *)(xf_row + min(f0 + 8 * q + 4 * h, n0 - 4));
            }
        };
        auto take = [&](TileOperands &t, int tile) {
            const int f0 = 32 * tile;
            v16f w;
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = t.w[r / 4][r % 4];
            if (update >= 0) {
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const bool in = update * TB + 2 * s + h <= last;   // (a short last block: no infinity may meet its missing deltas)
                    w = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? t.xu[s] : 0.f, nld[s], w, 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int f = f0 + 8 * q + 4 * h;
                    if (unit < count && f < n0) *(v4f *)(p.W1 + row + f) = (v4f){w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
                }
                if (velocity) {
                    const float v = deltas[(last - update * TB) * stride + unit];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int f = f0 + 8 * q + 4 * h;
                        if (unit < count && f < n0) *(v4f *)(p.VW1 + row + f) = *(const v4f *)(p.X + (size_t)last * n0 + f) * v;
                    }
                }
            }
            if (products >= 0) {
                // (a sum per tile: one of 340 terms in a row left the net inputs, and W_2 with them, 11 % further from 64 bits than
                // the sixteen short ones of the kernel that sweeps every step)
                v16f acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = f0 + 8 * q + 4 * h < n0;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? t.xf[q][e] : 0.f, in ? w[4 * q + e] : 0.f, acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) total[r] += acc[r];
            }
        };
        const int step = shared ? 4 : 1;
        TileOperands a, b;
        int t = shared ? sweeper : 0;
        if (t < tiles) load(a, t);
        for (; t < tiles; t += 2 * step) {
            if (t + step < tiles) load(b, t + step);
            take(a, t);
            if (t + step >= tiles) break;
            if (t + 2 * step < tiles) load(a, t + 2 * step);
            take(b, t + step);
        }
        if (products >= 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int sample = 8 * (r / 4) + 4 * h + r % 4;
                if (shared) l.parts[(sweeper * TB + sample) * 32 + c] = total[r];
                else to[sample * stride + unit] = total[r];
            }
        }
    }
}

// The waves that sweep.  (Their barriers are those of run_steps.)
__device__ __forceinline__ void run_sweep(const BlockPlan &p, const ChainLds &l)
{
    const int blocks = (int)((p.n_samples + TB - 1) / TB);
    sweep(p, l, -1, 0, false);
    for (int b = 0; b < blocks; ++b) {
        __syncthreads();
        if (*l.abort) break;
        __syncthreads();
        const int products = b + 1 < blocks ? b + 1 : -1;
        if (b > 0 || products >= 0) sweep(p, l, b - 1, products, false);
    }
    __syncthreads();
    sweep(p, l, blocks - 1, -1, p.keep_v != 0);
}

template <int NK, int ACT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void wide_block_epoch_kernel(BlockPlan p)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_abort;
    // (inner products beyond fp32: the pass is another kernel's, which is launched behind this one)
    const int blocks = (int)((p.n_samples + TB - 1) / TB);
    bool bad = false;
    for (int b = threadIdx.x; b < blocks; b += kThreads) bad = bad || (uint32_t)p.gram_x[(size_t)b * kRecord + kFlagWord] != 0;
    if (threadIdx.x == 0) s_abort = 0;
    if (__syncthreads_or(bad)) return;
    ChainLds l;
    l.gs = lds;
    l.gx = l.gs + TB * TB;
    l.zp = (u64 *)(l.gx + TB * TB);
    l.zq = l.zp + 2 * 64 * 4;
    l.zc = (float *)(l.zq + 2 * 16);
    l.parts = l.zc + 2 * TB * p.d_stride;
    const int groups = (min(p.per, p.n1 - (int)blockIdx.x * p.per) + 31) / 32;
    l.shared_from = groups % 4 == 1 ? 32 * (groups - 1) : 1 << 30;
    l.abort = (lds_int *)&s_abort;
    l.flags = nullptr;
    for (int i = threadIdx.x; i < 2 * 64 * 4 + 2 * 16; i += kThreads) l.zp[i] = 0;
    for (int i = threadIdx.x; i < 2 * TB * p.d_stride; i += kThreads) l.zc[i] = 0.f;
    __syncthreads();
    if (threadIdx.x < kStepThreads) run_steps<2, NK, ACT, true>(p, l);
    else run_sweep(p, l);
}

__global__ __launch_bounds__(kThreads) void block_gram_kernel(BlockPlan p)
{
    extern __shared__ __align__(16) float lds[];
    run_gram(p, lds, (int)blockIdx.x, (int)gridDim.x);
}
constexpr size_t kGramLds = 2 * kWaves * 16 * 64 * sizeof(float);

size_t wide_block_lds(int stride, bool shared)
{
    return (2 * TB * TB + 2 * (size_t)TB * stride + (shared ? 4 * TB * 32 : 0)) * sizeof(float) + (2 * 64 * 4 + 2 * 16) * sizeof(u64);
}

template <int NK, int ACT>
hipError_t wide_block_one(const BlockPlan *plan, int grid, size_t lds, hipStream_t stream)   // plan == nullptr: raise the LDS limit only
{
    const auto kernel = wide_block_epoch_kernel<NK, ACT>;
    if (!plan) return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ON_MAX_LDS_BYTES);
    return launch_resident(kernel, *plan, grid, lds, stream);
}

template <int NK>
hipError_t wide_block_act(int act, const BlockPlan *plan, int grid, size_t lds, hipStream_t stream)
{
    switch (act) {
    case DN_ACT_SIGMOID: return wide_block_one<NK, DN_ACT_SIGMOID>(plan, grid, lds, stream);
    case DN_ACT_TANH: return wide_block_one<NK, DN_ACT_TANH>(plan, grid, lds, stream);
    case DN_ACT_RELU: return wide_block_one<NK, DN_ACT_RELU>(plan, grid, lds, stream);
    default: return wide_block_one<NK, DN_ACT_LINEAR>(plan, grid, lds, stream);
    }
}

hipError_t wide_block_dispatch(int n2, int act, const BlockPlan *plan, int grid, size_t lds, hipStream_t stream)
{
    return n2 <= 10 ? wide_block_act<10>(act, plan, grid, lds, stream) : wide_block_act<16>(act, plan, grid, lds, stream);
}

}  // namespace

// per (units of a workgroup) and grid from wide_geometry; false where the units or the buffers do not fit.
bool wide_block_fits(int n1, int per)
{
    if (per > 2 * kStepThreads) return false;
    const int groups = (per + 31) / 32, tail = (n1 - (n1 - 1) / per * per + 31) / 32;
    return wide_block_lds(32 * groups, groups % 4 == 1 || tail % 4 == 1) <= ON_MAX_LDS_BYTES;
}

constexpr size_t kAllWords = 2 * 4096 + 2 * 8 * 256;
static_assert(ON_MAX_WG <= 256, "sixteen groups of sixteen workgroups");

size_t wide_block_exchange_bytes(const int32_t *n, int L)
{
    bool fits = false;   // on a device of some size
    WideGeom g;
    for (int units = ON_MAX_WG; units > 0 && !fits; --units) fits = wide_geometry(n, L, units, false, g) && wide_block_fits(n[1], g.per);
    return !fits ? 0 : (kAllWords + (size_t)(BLOCK_LAUNCH_SAMPLES / TB) * kRecord) * sizeof(u64);
}

hipError_t wide_block_prepare(int n2, int act)
{
    hipError_t e = hipFuncSetAttribute((const void *)block_gram_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGramLds);
    return e != hipSuccess ? e : wide_block_dispatch(n2, act, nullptr, 0, 0, nullptr);
}

// The blocks' inner products, then the pass; *gram: the records, whose flags tell whether the pass was taken.
hipError_t launch_wide_block_epoch(BlockPlan plan, int grid, unsigned long long *exchange, const unsigned long long **gram, hipStream_t stream)
{
    if (plan.n_samples < 1 || plan.n_samples > BLOCK_LAUNCH_SAMPLES || !wide_block_fits(plan.n1, plan.per)) return hipErrorInvalidValue;
    const int groups = (plan.per + 31) / 32, tail = (plan.n1 - (grid - 1) * plan.per + 31) / 32;
    plan.chain_waves = 4;
    plan.d_stride = 32 * groups;
    plan.all_x = exchange;
    plan.gram_x = plan.all_x + kAllWords;
    *gram = plan.gram_x;
    const int blocks = (int)((plan.n_samples + TB - 1) / TB);
    hipLaunchKernelGGL(block_gram_kernel, dim3(blocks), dim3(kThreads), kGramLds, stream, plan);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return wide_block_dispatch(plan.n2, plan.act1, &plan, grid, wide_block_lds(plan.d_stride, groups % 4 == 1 || tail % 4 == 1), stream);
}

}  // namespace dn
