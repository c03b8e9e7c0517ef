// Per-sample (batch 1) training of two-layer nets, plain gradient descent, with the samples taken in blocks of 32: one
// persistent kernel in which W_1 is read and written once per block instead of once per step.
//
// Within a block the first layer's net inputs do not need the updated W_1.  With W the matrix at the block's start,
//     W_1 x_i  at step i  =  W x_i  -  sum over the block's steps j < i of  lr delta_j (x_j . x_i),
// so a step needs the products W x_i (one 32-column product per block), the inner products x_j . x_i of the block's samples
// and, of every step before it, one multiply-add per hidden unit; W_1 itself takes the block's 32 rank-1 updates as one
// product.  (The bias of layer 1 is a further input of 1: x_j . x_i + 1.)  The arithmetic per weight is the same; what is
// gone is the sweep over W_1 inside every step, and with it every wait but those of a block's end.  Errors against 64 bits
// are those of the kernels that sweep every step: 4000 steps of 784-128-10, mean of twelve seeds, before and now, W_1 2.49e-7 and
// 2.49e-7 of its norm, b_1 2.49e-7 and 2.49e-7, W_2 2.33e-7 and 2.37e-7, b_2 7.9e-7 and 8.2e-7 (2e-7 either way from seed to seed).
//
// Roles, one workgroup each, 256 threads (one wave per SIMD: a lane may hold 512 registers):
//   chain   (workgroup 0) runs the steps.  A lane of the first NW waves keeps U hidden units: their net inputs for the
//           block's remaining samples (32 registers a unit), their column of W_2 and bias.  The output layer's sums over the
//           units meet by lane swaps and, with several waves, in stamped words in LDS; a step has no barrier, a block has two.
//   Gram    (workgroups 1 to 4) the blocks' inner products, running ahead of the steps.
//   rows    (the others) four rows of W_1 each, in registers in the lane layout of v_mfma_f32_4x4x1_16b_f32, which serves
//           both products: as operand A of W x (lane 4 b + i: row i, columns 4 b .. 4 b + 3 of a group of 64) and as the
//           accumulator of W - lr delta x.  The four waves split the columns.
// All of a launch's workgroups have to be on the device at once; launch_counts() below says what happens if they cannot.
// What crosses workgroups goes in stamped words (dn_persist.h): net inputs from the rows to the chain and deltas back,
// 32 per unit and block each, and the inner products.
//
// Numbers that the direct sums hold and an inner product does not (|x|^2 beyond fp32, infinities, NaN): the Gram workgroup marks
// such a block, and its samples are then taken one by one, each as a block of its own.
//
// The rows take a block's update and form the net inputs of the block after next while the steps take the one between: what is
// missing in those, the deltas of that block, comes from the inner products of the two blocks' samples, as a matrix product
// of two steps at a time beside the steps.  So at a block's end the steps wait for LDS only.
//
// What bounds it: the instructions of the waves that take the steps, about 260 a step for 784-128-10 and five to six cycles each
// (one wave on its SIMD), and their dependent chain: 1600 of 1700 cycles; a block's end costs 3400 cycles once in 32 steps.
// us per step, before (the kernels that sweep W_1 every step) and now: 784-128-10, 4000 samples 3.18 -> 0.72 (one
// workgroup); 256-256-10 3.5 -> 1.2; 1021-97-16 10.1 -> 1.5 (odd width); 784-500-33 5.8 -> 2.8; 128-1000-16 5.5 -> 2.5;
// 5-999-2 25.7 -> 2.3; 64-128-10 in passes of 96 samples 2.1 -> 1.3 (about 30 us of each pass are start and end).
// With four units a lane, or two and more than 32 outputs, a lane's numbers are more than its 512 registers: 7, 43 and 144 of them
// live in scratch memory for 4, 10 and 16 outputs, 150 for 64 (128-1000-k 1.9, 2.3 and 2.7 us a step, 784-500-64 2.5).
// Tried on the way: corrections within the block as a register file that moves up by one every step (62 copies a step, 1.48 us);
// without the look-ahead over the block's end 1.33.
#pragma once
#include <algorithm>
#include <cfloat>

#ifndef DN_PERSIST_THREADS
#define DN_PERSIST_THREADS 256   // one wave per SIMD: a lane may hold 512 registers
#endif
#include "dn_internal.h"
#include "dn_persist.h"
#include "dn_wave.h"

namespace dn {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
constexpr int TB = BLOCK_SAMPLES;
static_assert(TB == 32, "the lane layouts below are for 32 samples");

__device__ __forceinline__ float bits_to_float(unsigned v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ unsigned float_to_bits(float v) { return __builtin_bit_cast(unsigned, v); }

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// v in a vector register proper (the lane swaps cannot take sums of the matrix instructions from where those may be kept).
__device__ __forceinline__ float in_vector(float v)
{
    asm("" : "+v"(v));
    return v;
}

// a's lower half and b's lower half meet their upper halves: lanes below 32 get a[l] + a[l + 32], the others b[l - 32] + b[l].
__device__ __forceinline__ float add_halves(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(float_to_bits(in_vector(a)), float_to_bits(in_vector(b)), false, false);
    return bits_to_float(r[0]) + bits_to_float(r[1]);
}
// ... and the same for rows of 16 lanes: even rows get a's sum of two rows, odd rows b's.
__device__ __forceinline__ float add_rows(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(float_to_bits(in_vector(a)), float_to_bits(in_vector(b)), false, false);
    return bits_to_float(r[0]) + bits_to_float(r[1]);
}

typedef volatile int __attribute__((address_space(3))) lds_int;

// The lane that the permutation CTRL pairs this one with (every lane of the wave is active and has a partner).
template <int CTRL>
__device__ __forceinline__ float partner(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kMirror = 0x140, kHalfMirror = 0x141, kQuad2 = 0x4E, kQuad1 = 0xB1;   // lane i with 15 - i, 7 - i, i ^ 2, i ^ 1 of its row

__device__ __forceinline__ float larger(float a, float b)   // (fmaxf would quiet its operands first)
{
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
    return m;
}

constexpr int log2_up(int k) { return k <= 1 ? 0 : 1 + log2_up((k + 1) / 2); }

// Sums over the 64 lanes of each of N values.  Level by level the lanes split in two by one bit of their number, from the
// highest on, one half going on with the first ceil(n / 2) of the n values that are left and the other with the rest; with one
// value left all lanes add their partner's.  So lanes that agree in their first log2_up(N) bits hold the same sum.
template <int CTRL, int BIT, int N, int A>
__device__ __forceinline__ void row_level(float (&p)[A], int lane)
{
    constexpr int H = (N + 1) / 2;
    if constexpr (N > 1) {
        const bool up = (lane & BIT) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const float second = i + H < N ? p[i + H < A ? i + H : 0] : 0.f;
            const float keep = up ? second : p[i], send = up ? p[i] : second;
            p[i] = keep + partner<CTRL>(send);
        }
    } else {
        p[0] += partner<CTRL>(p[0]);
    }
}

template <int N>
__device__ __forceinline__ float sums_over_lanes(float (&p)[N], int lane)
{
    static_assert(N >= 3 && N <= 64, "three to 64 values");
    constexpr int H1 = (N + 1) / 2, H2 = (H1 + 1) / 2, H3 = (H2 + 1) / 2, H4 = (H3 + 1) / 2, H5 = (H4 + 1) / 2;
#pragma unroll
    for (int i = 0; i < H1; ++i) p[i] = add_halves(p[i], i + H1 < N ? p[i + H1 < N ? i + H1 : 0] : 0.f);
#pragma unroll
    for (int i = 0; i < H2; ++i) p[i] = add_rows(p[i], i + H2 < H1 ? p[i + H2 < N ? i + H2 : 0] : 0.f);
    row_level<kMirror, 8, H2>(p, lane);
    row_level<kHalfMirror, 4, H3>(p, lane);
    row_level<kQuad2, 2, H4>(p, lane);
    row_level<kQuad1, 1, H5>(p, lane);
    return p[0];
}

// Which of the N sums a lane ends up with (-1: none), and the first lane that holds sum k.
__device__ __forceinline__ int sum_of_lane(int n, int lane)
{
    int k = 0, left = n, half[6];
    bool in = true;
    for (int l = 0; l < 6; ++l) half[l] = left > 1 ? (left + 1) / 2 : 0, left = (left + 1) / 2;
    int size[6];
    left = n;
    for (int l = 0; l < 6; ++l) size[l] = left, left = (left + 1) / 2;
    for (int l = 5; l >= 0; --l) {
        if (half[l] == 0 || !(lane & (32 >> l))) continue;
        k += half[l];
        in = in && k < size[l];
    }
    return in ? k : -1;
}
__host__ __device__ constexpr int lane_of_sum(int n, int k)
{
    int lane = 0;
    for (int bit = 32; bit > 0 && n > 1; bit >>= 1) {
        const int half = (n + 1) / 2;
        if (k >= half) lane |= bit, k -= half;
        n = half;
    }
    return lane;
}

// Maximum / sum over the values of all groups of lanes that hold the same one (LEVELS bits tell the groups apart).
template <int LEVELS, class Op>
__device__ __forceinline__ float over_groups(float v, Op op)
{
    if constexpr (LEVELS >= 6) v = op(v, partner<kQuad1>(v));
    if constexpr (LEVELS >= 5) v = op(v, partner<kQuad2>(v));
    if constexpr (LEVELS >= 4) v = op(v, partner<kHalfMirror>(v));
    if constexpr (LEVELS >= 3) v = op(v, partner<kMirror>(v));
    const auto r = __builtin_amdgcn_permlane16_swap(float_to_bits(v), float_to_bits(v), false, false);
    v = op(bits_to_float(r[0]), bits_to_float(r[1]));
    const auto h = __builtin_amdgcn_permlane32_swap(float_to_bits(v), float_to_bits(v), false, false);
    return op(bits_to_float(h[0]), bits_to_float(h[1]));
}

template <int ACT>
__device__ __forceinline__ float activation(float z) { return act_fn(ACT, z); }
template <int ACT>
__device__ __forceinline__ float activation_slope(float a) { return act_deriv(ACT, a); }

// A zero that the compiler cannot see through: addresses that contain it are formed where they are used, not once for all and kept
// in registers through the loop around them.
__device__ __forceinline__ int hidden_zero()
{
    int z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

// One wave's bounded wait for N words per lane, word i at addr(i, 0) (need(i): this lane's word i exists); false after a timeout.
template <int N, class Addr, class Need>
__device__ __forceinline__ bool wave_poll(u64 (&v)[N], uint32_t seq, Addr addr, Need need, int *abort_flag)
{
    int spins = 0;
    for (;;) {
        const int o = hidden_zero();
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = ll_load(addr(i, o));
        bool wait = false;
#pragma unroll
        for (int i = 0; i < N; ++i) wait = wait || (need(i) && (uint32_t)(v[i] >> 32) != seq);
        if (!__any(wait)) return true;
        ++spins;
        if (spins > kSpinLimit) {
            __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        if ((spins & 255) == 0 && __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
        __builtin_amdgcn_s_sleep(1);
    }
}

// A launch counts only if all of its workgroups are on the device at once, which other work may prevent.  Nobody writes a parameter
// before the matter is settled, and whoever settles it first settles it for all: the first Gram workgroup, which waits for nobody
// else, after its products (kPlacePolls polls for those that are missing), or a wave that is about to write or has timed out.
// patience: polls to wait for the missing ones.  (Looked at in every wait instead, it cost the steps of 784-128-10 3.5 %.)
constexpr int kPlacePolls = 1 << 16;   // of about a microsecond
__device__ __forceinline__ bool launch_counts(const BlockPlan &p, int patience)
{
    for (int spins = 0;; ++spins) {
        const int settled = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p.settled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (settled != p.launch) return settled == p.launch + 1;
        const unsigned there = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p.arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (spins >= patience || there == p.expected) {
            int seen = p.launch;
            const int word = patience > 0 && there == p.expected ? p.launch + 1 : -1 - p.launch;
            if ((threadIdx.x & 63) == 0)
                __hip_atomic_compare_exchange_strong(p.settled, &seen, word, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            __builtin_amdgcn_s_sleep(1);
        }
    }
}
// Before a wave writes parameters; ok: its own waits have come to their end.  (One that timed out takes the launch back.)
__device__ __forceinline__ bool may_write(const BlockPlan &p, bool ok) { return launch_counts(p, ok ? kPlacePolls : 0) && ok; }

constexpr int kRecord = 2 * TB * TB;   // words of a block's record: its own inner products, then those with the next block's samples
constexpr int kFlagWord = TB - 1;      // (own products of sample 0 end one word earlier)
constexpr int OWN_BAD = 1, NEXT_BAD = 2;

__device__ __forceinline__ int block_flags(const BlockPlan &p, int64_t block, bool &ok)
{
    u64 v[1];
    const u64 *flag = p.gram_x + (size_t)block * kRecord + kFlagWord;
    ok = wave_poll(v, p.seq0 + 1u, [&](int, int) { return flag; }, [](int) { return true; }, p.abort_flag) && ok;
    return __builtin_amdgcn_readfirstlane((int)(uint32_t)v[0]);
}

// Whether the net inputs of block b + 1 are formed without block b's update (flags f and fnext): only then are they corrected
// through the inner products of the two blocks.
__device__ __forceinline__ bool next_is_ahead(int f, int fnext) { return (f & (OWN_BAD | NEXT_BAD)) == 0 && (fnext & OWN_BAD) == 0; }

// The parts of a sum that the workgroup's first nw <= N waves leave in LDS (every wave leaves one before it waits here), in
// wave order.
template <int N>
__device__ __forceinline__ float gather(const u64 *parts, int nw, uint32_t stamp)
{
    u64 v[N];
    bool wait;
    do {
        wait = false;
#pragma unroll
        for (int w = 0; w < N; ++w) v[w] = __hip_atomic_load(parts + min(w, nw - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
        for (int w = 0; w < N; ++w) wait = wait || (uint32_t)(v[w] >> 32) != stamp;
        if (N == 1 && __any(wait)) __builtin_amdgcn_s_sleep(1);
    } while (__any(wait));
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < N; ++w) sum += w < nw ? bits_to_float((uint32_t)v[w]) : 0.f;
    return sum;
}

// ---- the steps' workgroup ----
struct ChainLds;
template <int NK>
__device__ __forceinline__ float over_workgroups(const BlockPlan &p, const ChainLds &l, float z2, uint32_t stamp, int par, bool first, int group, int my_k);

struct ChainLds {
    float *gs;   // [2][32][32]: row j: inner products of sample j with samples j0, j0 + 1, .. (j0 = j rounded down to 4)
    float *gx;   // [2][32][32]: row j: inner products of sample j with the next block's samples
    u64 *zp;     // [2][64][4]: the waves' parts of the output layer's sums, stamped
    float *zc;   // [32][d_stride]: net inputs of the next block as they came from the rows.  WIDE: [2][32][d_stride], by block
                 // parity: a block's net inputs, then -lr delta in their place
    u64 *zq;     // WIDE: [2][16]: the sums over all workgroups, stamped
    float *parts;   // WIDE: [4][32][32]: four parts of the net inputs of units shared_from .. shared_from + 31
    int shared_from;
    lds_int *abort;
    lds_int *flags;   // [2]: the blocks' flags
};

// What the piece that begins with sample s needs (a block, or one sample of a block that is taken sample by sample), into
// LDS; this wave does a share of it, fetcher of fetchers.
__device__ __forceinline__ void fetch_piece(const BlockPlan &p, const ChainLds &l, int64_t s, bool with_record, int fetcher, int fetchers)
{
    const int lane = threadIdx.x & 63, n1 = p.n1;
    const int64_t n = p.n_samples, block = s / TB;
    bool ok = true;
    if (with_record) {
        const u64 *rec = p.gram_x + (size_t)block * kRecord;
        float *to_s = l.gs + (block & 1) * TB * TB, *to_x = l.gx + (block & 1) * TB * TB;
        const int m = (int)min((int64_t)TB, n - block * TB), mx = (int)min((int64_t)TB, n - block * TB - m);
        for (int q0 = fetcher * 256; q0 < kRecord && ok; q0 += fetchers * 256) {
            auto inside = [&](int i) {
                const int q = (q0 + i * 64 + lane) % (TB * TB), j = q / TB, t = q % TB;
                return q0 < TB * TB ? j + t + 1 < m : (j < m && t < mx);
            };
            u64 v[4];
            ok = wave_poll(v, p.seq0 + 1u, [&](int i, int) { return rec + (inside(i) ? q0 + i * 64 + lane : kFlagWord); }, inside,
                           p.abort_flag);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = (q0 + i * 64 + lane) % (TB * TB), j = q / TB, t = q % TB;
                const float val = inside(i) ? bits_to_float((uint32_t)v[i]) : 0.f;
                if (q0 < TB * TB) to_s[j * TB + (t + 1 + j % 4) % TB] = val;   // (what wraps is not used)
                else to_x[j * TB + t] = val;
            }
        }
        if (fetcher == 0) {
            const int f = block_flags(p, block, ok);
            if (lane == 0) l.flags[block & 1] = f;
        }
    }
    const u64 *src = p.z_x + (size_t)(block & 1) * TB * n1;
    const int total = (int)min((int64_t)TB, n - s) * n1;   // (a single sample's piece uses the first n1)
    constexpr int PER = 16;
    for (int q0 = fetcher * 64 * PER; q0 < total && ok; q0 += fetchers * 64 * PER) {
        u64 v[PER];
        ok = wave_poll(v, p.seq0 + 1u + (uint32_t)s, [&](int i, int) { return src + min(q0 + i * 64 + lane, total - 1); },
                       [&](int i) { return q0 + i * 64 + lane < total; }, p.abort_flag);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = q0 + i * 64 + lane, j = q / n1;
            if (q < total) l.zc[j * p.d_stride + (q - j * n1)] = bits_to_float((uint32_t)v[i]);
        }
    }
    if (!ok) *l.abort = 1;
}

// The waves that take no steps fetch while the steps run; with no such wave all fetch after the steps.
__device__ __forceinline__ bool fetch_beside(const BlockPlan &p) { return p.chain_waves < kWaves; }

// A wave of the workgroup that takes no steps.  (Its barriers are those of run_steps.)
__device__ __forceinline__ void run_fetcher(const BlockPlan &p, const ChainLds &l)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fetchers = kWaves - p.chain_waves, fetcher = wave - p.chain_waves;
    const int64_t n = p.n_samples;
    fetch_piece(p, l, 0, true, fetcher, fetchers);
    for (int64_t s0 = 0; s0 < n;) {
        const int64_t block = s0 / TB;
        __syncthreads();
        if (*l.abort) break;
        const bool serial = (l.flags[block & 1] & OWN_BAD) != 0;
        const int64_t next = s0 + (serial ? 1 : min((int64_t)TB, n - s0));
        __syncthreads();   // zc is free
        if (next < n) fetch_piece(p, l, next, next / TB != block, fetcher, fetchers);
        s0 = next;
    }
}

// The output layer's sums over the units of all workgroups, in two levels of sixteen: the four waves' parts meet in LDS, the
// workgroup's go out as words, one workgroup of every sixteen adds those of its sixteen and sends the sums on, and every
// workgroup adds the sixteen sums.  (Two short hops: with everybody reading everybody's words, 5 MB a look, a step waited 6 us.)
// Words: [2][16 groups][16 outputs][16 members], then [2][8 copies][16 outputs][16 groups] (a word that all workgroups ask for
// keeps its writer waiting).  Every sum is formed in the same order.
// Workgroups w, w + 16, w + 32, .. are a group: by the usual round-robin placement they share an XCD, where a hop is 0.9 instead of 1.2 us.
__device__ __forceinline__ int members_of_group(int g, int grid) { return (grid - g + 15) >> 4; }
__device__ __forceinline__ int reader_of_group(int g, int grid) { return 16 * min(g, members_of_group(g, grid) - 1) + g; }

template <int NK>
__device__ __forceinline__ float over_workgroups(const BlockPlan &p, const ChainLds &l, float z2, uint32_t stamp, int par, bool first, int group, int my_k)
{
    static_assert(NK <= 16, "a workgroup's words");
    constexpr int R = (NK + 3) / 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), grid = (int)gridDim.x, w = (int)blockIdx.x;
    u64 *mine = l.zp + (par * 64 + group) * 4, *sums = l.zq + par * 16;
    if (first) __hip_atomic_store(mine + wave, ((u64)stamp << 32) | float_to_bits(z2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (wave == 0) {
        u64 *words = p.all_x + par * 4096, *tops = p.all_x + 2 * 4096 + par * 8 * 256;
        const float own = gather<4>(mine, 4, stamp);
        if (first && my_k >= 0) ll_store(words + (w & 15) * 256 + my_k * 16 + (w >> 4), own, stamp);
        const int member = lane & 15, kq = lane >> 4;   // lane's word of round r: output 4 r + kq
        bool ok = true;
        u64 v[R];
        if (w == reader_of_group(w & 15, grid)) {
            const int there = members_of_group(w & 15, grid);
            const u64 *from = words + (w & 15) * 256 + min(member, there - 1);
            ok = wave_poll(v, stamp, [&](int r, int) { return from + min(4 * r + kq, NK - 1) * 16; }, [](int) { return true; }, p.abort_flag);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float sum = row16_sum(member < there ? bits_to_float((uint32_t)v[r]) : 0.f);
                if (member < 8 && 4 * r + kq < NK) ll_store(tops + member * 256 + (4 * r + kq) * 16 + (w & 15), sum, stamp);
            }
        }
        const int groups = min(grid, 16);
        const u64 *from = tops + (w & 7) * 256 + min(member, groups - 1);
        ok = wave_poll(v, stamp, [&](int r, int) { return from + min(4 * r + kq, NK - 1) * 16; }, [](int) { return true; }, p.abort_flag) && ok;
        if (!ok) *l.abort = 1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float sum = row16_sum(member < groups ? bits_to_float((uint32_t)v[r]) : 0.f);
            if (member == 0) __hip_atomic_store(sums + 4 * r + kq, ((u64)stamp << 32) | float_to_bits(sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    } else {
        __builtin_amdgcn_s_sleep(32);   // (nothing to find before the words have travelled; the sweep has the SIMD meanwhile)
    }
    return gather<1>(sums + max(my_k, 0), 1, stamp);
}

// WIDE: the hidden layer is spread over the workgroups of the launch (dn_wide_block.hip), p.per units each; the output
// layer's sums meet in exchanged words once a step, and the rows are updated by other waves of this workgroup, through LDS.
template <int U, int NK, int ACT, bool WIDE = false>
__device__ __forceinline__ void run_steps(const BlockPlan &p, const ChainLds &l)
{
    constexpr int LEVELS = log2_up(NK), SH = 6 - LEVELS;
    if (WIDE) __builtin_amdgcn_s_setprio(3);   // before the waves that sweep: every workgroup waits for the slowest step
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n1 = p.n1, n2 = p.n2, nw = p.chain_waves, stride = p.d_stride;
    const int base = WIDE ? (int)blockIdx.x * p.per : 0, count = WIDE ? min(p.per, n1 - base) : n1;
    const int my_k = sum_of_lane(NK, lane), group = lane >> SH;
    const int lane_first = group << SH;   // of the lanes with the same sum
    const bool outl = my_k >= 0 && my_k < n2, first = lane == lane_first;
    const float lr = p.lr;

    float w2[U][NK], b1[U];
    int unit[U];
    bool hid[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        unit[u] = (wave * U + u) * 64 + lane;
        hid[u] = unit[u] < count;
        b1[u] = hid[u] ? p.b1[base + unit[u]] : 0.f;
#pragma unroll
        for (int k = 0; k < NK; ++k) w2[u][k] = (hid[u] && k < n2) ? p.W2[(size_t)k * n1 + base + unit[u]] : 0.f;
    }
    float b2 = outl ? p.b2[my_k] : 0.f;
    double loss_acc = 0.0;
    float loss_sum = 1.f, loss_z = 0.f;   // lane j: softmax sum of step j and its label's distance from the maximum

    const int64_t n = p.n_samples;
    if (!WIDE && !fetch_beside(p)) fetch_piece(p, l, 0, true, wave, kWaves);

    v16f ahead[U][2];   // corrections of the next block's net inputs: units 0 .. 31 and 32 .. 63 of the wave's 64
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) ahead[u][0][r] = ahead[u][1][r] = 0.f;
    int before = OWN_BAD;   // the previous block's flags
    for (int64_t s0 = 0; s0 < n;) {
        const int64_t block = s0 / TB;
        __syncthreads();
        if (*l.abort) break;
        const int flags = WIDE ? 0 : __builtin_amdgcn_readfirstlane(l.flags[block & 1]);
        const bool serial = (flags & OWN_BAD) != 0;
        const int at = (int)(s0 - block * TB);            // the piece's first sample within its block
        const int m = serial ? 1 : (int)min((int64_t)TB, n - s0);
        const uint32_t seq = p.seq0 + 1u + (uint32_t)(block * TB);
        float z[U][TB];
        float *zd = l.zc + (size_t)(WIDE ? block & 1 : 0) * TB * stride;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                if constexpr (WIDE) z[u][i] = zd[i * stride + min(unit[u], stride - 1)];
                else z[u][i] = l.zc[i * stride + unit[u]];
            }
        if constexpr (WIDE) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = unit[u] - l.shared_from;
                if (c < 0 || c >= 32) continue;
#pragma unroll
                for (int i = 0; i < TB; ++i)
                    z[u][i] = (l.parts[i * 32 + c] + l.parts[(TB + i) * 32 + c]) + (l.parts[(2 * TB + i) * 32 + c] + l.parts[(3 * TB + i) * 32 + c]);
            }
            // the block's inner products
            const u64 *rec = p.gram_x + (size_t)block * kRecord;
            const int mx = (int)min((int64_t)TB, n - s0 - m);
#pragma unroll
            for (int i = 0; i < kRecord / 256; ++i) {
                const int q = (i * 256 + tid) % (TB * TB), j = q / TB, t = q % TB;
                const bool own = i < kRecord / 512, inside = own ? j + t + 1 < m : (j < m && t < mx);
                const float v = inside ? bits_to_float((uint32_t)rec[i * 256 + tid]) : 0.f;
                if (own) l.gs[j * TB + (t + 1 + j % 4) % TB] = v;
                else l.gx[j * TB + t] = v;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < TB; ++i) z[u][i] = !WIDE || hid[u] ? z[u][i] + b1[u] : 0.f;   // (WIDE: the rows past a workgroup's last repeat it)
        if (next_is_ahead(before, flags)) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const auto x = __builtin_amdgcn_permlane32_swap(float_to_bits(in_vector(ahead[u][0][r])), float_to_bits(in_vector(ahead[u][1][r])), false, false);
                    z[u][8 * (r / 4) + r % 4] += bits_to_float(x[0]);
                    z[u][8 * (r / 4) + 4 + r % 4] += bits_to_float(x[1]);
                }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) ahead[u][0][r] = ahead[u][1][r] = 0.f;
        int label = p.labels[s0 + min(lane, m - 1)];
        label = lane_of_sum(NK, label < 0 ? 0 : (label >= n2 ? n2 - 1 : label));
        __syncthreads();   // zc is free
        const int64_t next = s0 + m;
        const float *gsb = l.gs + (WIDE ? 0 : block & 1) * TB * TB, *gxb = l.gx + (WIDE ? 0 : block & 1) * TB * TB;
        u64 *out = p.d_x + (size_t)((block & 1) * TB + at) * stride;
        const int last = p.keep_v && next == n ? m - 1 : -1;   // the pass's last step also leaves the applied change as velocity
        // steps j0 .. j0 + 3 use net inputs 0 .. 3 of the registers, which then move up
        for (int j0 = 0; j0 < m; j0 += 4) {
            float nld[U][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = j0 + q;
                if (j >= m) break;
                // ---- activations of the own units, their part of the output layer's net inputs ----
                float a[U], part[NK];
#pragma unroll
                for (int u = 0; u < U; ++u) a[u] = activation<ACT>(z[u][q]);
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    part[k] = w2[0][k] * a[0];
#pragma unroll
                    for (int u = 1; u < U; ++u) part[k] = __builtin_fmaf(w2[u][k], a[u], part[k]);
                }
                float z2 = sums_over_lanes<NK>(part, lane);
                if constexpr (WIDE) {
                    z2 = over_workgroups<NK>(p, l, z2, seq + (uint32_t)j, j & 1, first, group, my_k);
                } else if (nw > 1) {   // the waves' parts, added in wave order
                    const uint32_t stamp = seq + (uint32_t)(at + j);
                    u64 *zq = l.zp + ((q & 1) * 64 + group) * 4;
                    if (first) __hip_atomic_store(zq + wave, ((u64)stamp << 32) | float_to_bits(z2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    z2 = nw <= 2 ? gather<2>(zq, nw, stamp) : gather<4>(zq, nw, stamp);
                }
                z2 += b2;
                // ---- output error and loss (every wave alike) ----
                const int y = __builtin_amdgcn_readlane(label, j);
                const float t1 = lane_first == y ? 1.0f : 0.0f;
                float d2;
                if (p.loss == DN_LOSS_CROSS_ENTROPY) {
                    const float zz = outl ? z2 : -INFINITY;
                    const float mx = over_groups<LEVELS>(zz, [](float x, float w) { return larger(x, w); });
                    const float below = zz - mx;
                    const float ex = exp_below_zero(below);
                    const float sum = over_groups<LEVELS>(ex, [](float x, float w) { return x + w; });
                    d2 = __builtin_fmaf(ex, inverse(sum), -t1);
                    loss_sum = lane == j ? sum : loss_sum;
                    const float by = lane_value(below, y);
                    loss_z = lane == j ? by : loss_z;
                } else {
                    const float a2 = outl ? act_fn(p.act2, z2) : 0.f;
                    const float f = outl ? a2 - t1 : 0.f;
                    d2 = f * act_deriv(p.act2, a2);
                    loss_acc += (double)(0.5f * f * f);   // this lane's share, counted once per group at the end
                }
                v4f g[TB / 4];
#pragma unroll
                for (int i = 0; i < TB / 4; ++i) g[i] = *(const v4f *)(gsb + j * TB + 4 * i);
                // ---- deltas of the own units through W_2 as it was, W_2's update ----
                // (both take -lr delta_2, rounded anew every step.  Rounding lr a instead leaves the same error in a weight step
                // after step where a unit's activation hardly changes: W_2 of the wide net 4.4e-7 off instead of 3.9e-7.)
                const float nld2 = -(lr * d2);
                float d1[U], d1b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    d1[u] = d1b[u] = 0.f;
                    if (ACT == DN_ACT_SIGMOID) a[u] = hid[u] ? a[u] : 0.f;   // (lanes past the layer's end keep zeros; f(0) = 0 elsewhere)
                }
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    const float dk = lane_value(nld2, lane_of_sum(NK, k));
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        (k & 1 ? d1b[u] : d1[u]) = __builtin_fmaf(w2[u][k], dk, k & 1 ? d1b[u] : d1[u]);
                        w2[u][k] = __builtin_fmaf(dk, a[u], w2[u][k]);
                    }
                }
                // ---- -lr delta to the rows, into the net inputs of the samples to come, and the biases ----
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float v = (d1[u] + d1b[u]) * activation_slope<ACT>(a[u]);
                    if constexpr (!WIDE) ll_store(out + (uint32_t)(j * stride + unit[u]), v, seq);
                    else if (unit[u] < stride) zd[j * stride + unit[u]] = v;
                    b1[u] += v;
                    nld[u][q] = v;
                }
#pragma unroll
                for (int c = 0; c < TB / 8; ++c) {
                    if (c > 0 && j0 >= TB - 8 * c) break;   // past the block's end
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int i = 8 * c; i < 8 * c + 8; ++i)
                            if (i > q) z[u][i] = __builtin_fmaf(g[i / 4][i % 4], nld[u][q], z[u][i]);
                }
                b2 += nld2;
                if (q % 2 == 1) {   // two steps' part of the next block's corrections: k = 0 and 1 of the product
                    const float gk = gxb[(j - 1 + (lane >> 5)) * TB + (lane & 31)];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const auto x = __builtin_amdgcn_permlane32_swap(float_to_bits(in_vector(nld[u][q - 1])), float_to_bits(in_vector(nld[u][q])), false, false);
                        ahead[u][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(gk, bits_to_float(x[0]), ahead[u][0], 0, 0, 0);
                        ahead[u][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(gk, bits_to_float(x[1]), ahead[u][1], 0, 0, 0);
                    }
                }
                if (j == last) {
                    int n2v = n2;
                    asm volatile("" : "+s"(n2v));   // (else the tests below are formed once and kept in registers through all steps)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (!hid[u]) continue;
                        p.Vb1[base + unit[u]] = nld[u][q];
#pragma unroll
                        for (int k = 0; k < NK; ++k)
                            if (k < n2v) p.VW2[(size_t)k * n1 + base + unit[u]] = a[u] * lane_value(nld2, lane_of_sum(NK, k));
                    }
                    if (wave == 0 && (!WIDE || blockIdx.x == 0) && outl && first) p.Vb2[my_k] = nld2;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i + 4 < TB; ++i) z[u][i] = z[u][i + 4];
        }
        if (p.loss == DN_LOSS_CROSS_ENTROPY && lane < m) loss_acc += (double)(logf(loss_sum) - loss_z);
        if constexpr (WIDE) {   // a short last block: no deltas in the rest of it
            for (int j = m; j < TB; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (unit[u] < stride) zd[j * stride + unit[u]] = 0.f;
        } else if (next < n && !fetch_beside(p)) fetch_piece(p, l, next, next / TB != block, wave, kWaves);
        if (next / TB != block) before = flags;
        s0 = next;
    }
    if constexpr (WIDE) __syncthreads();   // the last block's deltas

    // ---- epilogue ----
    if (!WIDE && !may_write(p, *l.abort == 0)) return;
    int n2e = n2;
    asm volatile("" : "+s"(n2e));
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!hid[u]) continue;
        p.b1[base + unit[u]] = b1[u];
#pragma unroll
        for (int k = 0; k < NK; ++k)
            if (k < n2e) p.W2[(size_t)k * n1 + base + unit[u]] = w2[u][k];
    }
    if (wave != 0 || (WIDE && blockIdx.x != 0)) return;
    if (outl && first) p.b2[my_k] = b2;
    if (p.loss != DN_LOSS_CROSS_ENTROPY && !(outl && first)) loss_acc = 0.0;
    for (int off = 32; off > 0; off >>= 1) loss_acc += __shfl_xor(loss_acc, off, 64);
    if (lane == 0) *p.loss_acc += loss_acc;
}

// ---- the blocks' inner products ----
// Two 32 x 32 products over the n0 features on v_mfma_f32_32x32x2_f32: the block's samples with themselves (both operands are
// the same registers) and with the next block's; the features split among the waves in groups of eight.
__device__ __forceinline__ void run_gram(const BlockPlan &p, float *lds, int first, int step)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, idx = lane & 31, h = lane >> 5;
    const int n0 = p.n0, groups = (n0 + 7) / 8;
    const int64_t n = p.n_samples;
    for (int64_t block = first; block * TB < n; block += step) {
        const int64_t s0 = block * TB;
        const int m = (int)min((int64_t)TB, n - s0), mx = (int)min((int64_t)TB, n - s0 - m);
        const float *row[2] = {p.X + (size_t)(s0 + min(idx, m - 1)) * n0, p.X + (size_t)(s0 + min(TB + idx, m + mx - 1)) * n0};
        v16f acc[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
        constexpr int F = 4;   // groups whose loads travel together (twelve started a pass no faster)
        for (int g0 = wave; g0 < groups; g0 += kWaves * F) {
            v4f x[2][F];
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int k = 8 * (g0 + f * kWaves) + 4 * h;
                    if (p.vec) {
                        x[c][f] = *(const v4f *)(row[c] + min(k, n0 - 4));
                        if (k >= n0) x[c][f] = (v4f){0.f, 0.f, 0.f, 0.f};
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            x[c][f][e] = row[c][min(k + e, n0 - 1)];
                            if (k + e >= n0) x[c][f][e] = 0.f;
                        }
                    }
                }
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[0][f][e], x[c][f][e], acc[c], 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) lds[((c * kWaves + wave) * 16 + r) * 64 + lane] = acc[c][r];
        __syncthreads();
        u64 *rec = p.gram_x + (size_t)block * kRecord;
        bool bad[2] = {false, false};
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 16 / kWaves; ++q) {
                const int r = wave + kWaves * q, j = 8 * (r / 4) + 4 * h + (r % 4);
                float v = c == 0 ? 1.0f : 0.f;   // within a block the bias moves too, an input of one
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v += lds[((c * kWaves + w) * 16 + r) * 64 + lane];
                if (c == 0 ? (idx > j && idx < m) : (j < m && idx < mx)) {
                    ll_store(rec + c * TB * TB + j * TB + (c == 0 ? idx - j - 1 : idx), v, p.seq0 + 1u);
                    bad[c] = bad[c] || !(fabsf(v) <= FLT_MAX);
                }
            }
        const int own = __syncthreads_or(bad[0]), next = __syncthreads_or(bad[1]);
        if (tid == 0) {
            const u64 word = ((u64)(p.seq0 + 1u) << 32) | (u64)((own ? OWN_BAD : 0) | (next ? NEXT_BAD : 0));
            __hip_atomic_store(rec + kFlagWord, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---- rows of W_1 ----
// Lane 4 b + i of wave w keeps row i of its workgroup's four, columns 64 (w + 4 t) + 4 b + e (t < 4, e < 4).
__device__ __forceinline__ void run_rows(const BlockPlan &p, float *lds, lds_int *s_abort, int w)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = lane >> 2, i4 = lane & 3;
    const int n0 = p.n0, n1 = p.n1, row0 = w * 4;
    const int64_t n = p.n_samples;
    constexpr int TCH = 4;
    int col[TCH];
    const int rowc = min(row0 + i4, n1 - 1);
#pragma unroll
    for (int t = 0; t < TCH; ++t) col[t] = 64 * (wave + kWaves * t);

    // four consecutive columns of a row of a matrix with n0 columns, zeros past the end
    auto quad = [&](const float *row, int k, bool vec) {
        v4f v;
        if (vec) {
            v = *(const v4f *)(row + min(k, n0 - 4));
            if (k >= n0) v = (v4f){0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = row[min(k + e, n0 - 1)];
                if (k + e >= n0) v[e] = 0.f;
            }
        }
        return v;
    };
    const bool wvec = n0 % 4 == 0;
    v4f W[TCH];
#pragma unroll
    for (int t = 0; t < TCH; ++t) W[t] = quad(p.W1 + (size_t)rowc * n0, col[t] + 4 * b, wvec);

    v4f xf[TCH][TB / 4];     // lane 4 b + j: sample 4 c + j, columns 4 b .. 4 b + 3
    auto load_xf = [&](int64_t s) {
        const int o = hidden_zero();
#pragma unroll
        for (int c = 0; c < TB / 4; ++c) {
            const float *row = p.X + (uint32_t)(min((int)s + 4 * c + i4, (int)n - 1) * (n0 + o));
#pragma unroll
            for (int t = 0; t < TCH; ++t) xf[t][c] = quad(row, col[t] + 4 * b, p.vec);
        }
    };
    float last = 0.f;

    // net inputs of the samples from s on; false after a timeout anywhere in the workgroup
    auto publish = [&](int64_t s) {
        load_xf(s);
        const uint32_t seq = p.seq0 + 1u + (uint32_t)s;
        u64 *to = p.z_x + (size_t)((s / TB) & 1) * TB * n1;
        v4f acc[TB / 4];
#pragma unroll
        for (int c = 0; c < TB / 4; ++c) acc[c] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < TCH; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < TB / 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(W[t][e], xf[t][c][e], acc[c], 0, 0, 0);
        // value v = 4 c + r of lane 4 b + j: sample 4 c + j, row r.  Bits 5 and 4 of the lane take over bits 4 and 3 of v;
        // the other sums over b and those over the waves are taken on the way out of LDS.
        float h16[16], h8[8];
#pragma unroll
        for (int v = 0; v < 16; ++v) h16[v] = add_halves(acc[v / 4][v % 4], acc[v / 4 + 4][v % 4]);
#pragma unroll
        for (int v = 0; v < 8; ++v) h8[v] = add_rows(h16[v], h16[v + 8]);
#pragma unroll
        for (int v = 0; v < 8; ++v) lds[(wave * 8 + v) * 64 + lane] = h8[v];
        __syncthreads();
        const bool ok = *s_abort == 0;
#pragma unroll
        for (int v = wave; v < 8; v += kWaves) {
            float sum = 0.f;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) sum += lds[(q * 8 + v) * 64 + lane];
            sum += partner<0x128>(sum);   // row_ror:8
            sum += partner<0x124>(sum);   // row_ror:4
            const int c = 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + (v >> 2), sample = 4 * c + i4, row = row0 + (v & 3);
            if ((lane & 12) == 0 && row < n1 && s + sample < n) ll_store(to + (size_t)sample * n1 + row, sum, seq);
        }
        __syncthreads();
        return ok;
    };
    // the update of m samples from sample `at` of block `block` on, eight at a time as their deltas come
    auto update = [&](int64_t block, int at, int m) {
        const uint32_t seq = p.seq0 + 1u + (uint32_t)(block * TB);
        const u64 *from = p.d_x + (size_t)((block & 1) * TB + at) * p.d_stride;
        bool ok = true;
#pragma unroll
        for (int c0 = 0; c0 < TB; c0 += 8) {
            if (c0 >= m || !ok) continue;
            float xu[TCH][8];   // lane l: column l of the eight samples
            const int s = (int)block * TB + at + c0, o = hidden_zero();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float *row = p.X + (uint32_t)(min(s + i, (int)n - 1) * (n0 + o));
#pragma unroll
                for (int t = 0; t < TCH; ++t) {
                    xu[t][i] = row[min(col[t] + lane, n0 - 1)];
                    if (col[t] + lane >= n0) xu[t][i] = 0.f;
                }
            }
            u64 v[8];
            ok = wave_poll(v, seq, [&](int i, int o) { return from + (uint32_t)(min(c0 + i, m - 1) * (p.d_stride + o) + rowc); },
                           [](int) { return true; }, p.abort_flag);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (c0 + i >= m) continue;
                last = bits_to_float((uint32_t)v[i]);
#pragma unroll
                for (int t = 0; t < TCH; ++t) W[t] = __builtin_amdgcn_mfma_f32_4x4x1f32(xu[t][i], last, W[t], 0, 0, 0);
            }
        }
        if (!ok) *s_abort = 1;
    };

    bool ok = publish(0);
    int flags = block_flags(p, 0, ok);
    for (int64_t s0 = 0; s0 < n && ok; s0 += TB) {   // while the steps take block s0
        const int64_t block = s0 / TB;
        const int m = (int)min((int64_t)TB, n - s0);
        const bool more = s0 + TB < n;
        bool got = true;
        const int fnext = more ? block_flags(p, block + 1, got) : OWN_BAD;
        if (!got) *s_abort = 1;
        const bool ahead = more && next_is_ahead(flags, fnext);
        if (ahead) ok = publish(s0 + TB);
        if (!(flags & OWN_BAD)) {
            update(block, 0, m);
        } else {   // sample by sample
            for (int i = 0; i < m && ok; ++i) {
                if (i > 0) ok = publish(s0 + i);
                update(block, i, 1);
            }
        }
        if (more && !ahead) ok = publish(s0 + TB) && ok;
        flags = fnext;
    }

    // ---- epilogue ----
    if (!may_write(p, ok && *s_abort == 0)) return;
    const int row = row0 + i4;
    if (row >= n1) return;
#pragma unroll
    for (int t = 0; t < TCH; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = col[t] + 4 * b + e;
            if (k >= n0) continue;
            p.W1[(size_t)row * n0 + k] = W[t][e];
            if (p.keep_v) p.VW1[(size_t)row * n0 + k] = last * p.X[(size_t)(n - 1) * n0 + k];
        }
}

template <int U, int NK, int ACT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void block_epoch_kernel(BlockPlan p)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_abort, s_flags[2];
    if (threadIdx.x == 0) {
        s_abort = 0;
        __hip_atomic_fetch_add(p.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const int w = (int)blockIdx.x;
    if (w == 0) {
        ChainLds l;
        l.gs = lds;
        l.gx = l.gs + 2 * TB * TB;
        l.zp = (u64 *)(l.gx + 2 * TB * TB);
        l.zc = (float *)(l.zp + 2 * 64 * 4);
        l.abort = (lds_int *)&s_abort;
        l.flags = (lds_int *)s_flags;
        for (int i = threadIdx.x; i < 2 * 64 * 4; i += kThreads) l.zp[i] = 0;
        for (int i = threadIdx.x; i < TB * p.d_stride; i += kThreads) l.zc[i] = 0.f;
        __syncthreads();
        if ((int)threadIdx.x < 64 * p.chain_waves) run_steps<U, NK, ACT>(p, l);
        else run_fetcher(p, l);
    } else if (w <= BLOCK_GRAM_GROUPS) {
        run_gram(p, lds, w - 1, BLOCK_GRAM_GROUPS);
        if (w == 1 && threadIdx.x < 64 && !launch_counts(p, kPlacePolls))
            __hip_atomic_store(p.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // (whoever waits need not any longer)
    } else run_rows(p, lds, (lds_int *)&s_abort, w - 1 - BLOCK_GRAM_GROUPS);
}

// LDS of the workgroup that runs the steps; the others' partial sums need less.  More than half of a compute unit's: one
// workgroup on each.
constexpr size_t chain_lds(int stride) { return (4 * TB * TB + (size_t)TB * stride) * sizeof(float) + 2 * 64 * 4 * sizeof(u64); }
constexpr size_t kBlockLds = 84 * 1024;
static_assert(kBlockLds >= 2 * 4 * 16 * 64 * sizeof(float), "the Gram workgroups' and the rows' partial sums");
static_assert(chain_lds(1024) <= ON_MAX_LDS_BYTES, "the widest layer");

template <int U, int NK, int ACT>
hipError_t block_one(const BlockGeom *g, const BlockPlan *plan, hipStream_t stream)
{
    const auto kernel = block_epoch_kernel<U, NK, ACT>;
    if (!g) return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ON_MAX_LDS_BYTES);
    return launch_resident(kernel, *plan, g->grid, std::max(kBlockLds, chain_lds(plan->d_stride)), stream);
}

// Launches (g == nullptr: raises the LDS limit of) the kernel for a net with one activation function: compiled for 4, 10, 16,
// 32 and 64 outputs, as a step's multiply-adds and lane swaps grow with that number whether the net has as many or not (us a step
// of 784-128-k 0.66, 0.79, 0.90, 1.03, 1.51; of 784-500-k 1.15, 1.28, 1.42, 1.71, 2.54).  10 rather than 8: the next step up from ten
// classes would cost 0.11 to 0.41 us, and the library's data sets have three or ten.
template <int ACT>
hipError_t block_dispatch(int units, int n2, const BlockGeom *g, const BlockPlan *plan, hipStream_t stream)
{
    if (units == 4) {
        if (n2 <= 4) return block_one<4, 4, ACT>(g, plan, stream);
        if (n2 <= 10) return block_one<4, 10, ACT>(g, plan, stream);
        return block_one<4, 16, ACT>(g, plan, stream);
    }
    if (units == 2) {
        if (n2 <= 4) return block_one<2, 4, ACT>(g, plan, stream);
        if (n2 <= 10) return block_one<2, 10, ACT>(g, plan, stream);
        if (n2 <= 16) return block_one<2, 16, ACT>(g, plan, stream);
        if (n2 <= 32) return block_one<2, 32, ACT>(g, plan, stream);
        return block_one<2, 64, ACT>(g, plan, stream);
    }
    if (n2 <= 4) return block_one<1, 4, ACT>(g, plan, stream);
    if (n2 <= 10) return block_one<1, 10, ACT>(g, plan, stream);
    if (n2 <= 16) return block_one<1, 16, ACT>(g, plan, stream);
    if (n2 <= 32) return block_one<1, 32, ACT>(g, plan, stream);
    return block_one<1, 64, ACT>(g, plan, stream);
}

}  // namespace
}  // namespace dn
