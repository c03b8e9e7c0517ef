// Minibatch training as ONE persistent kernel per epoch, every layer cut into square tiles.
//
// A step of a small or medium net is a chain of 2L short products, and with a launch per product it is bound by the chain's
// launches.  Here up to 256 workgroups (one per compute unit) stay on the device for the whole epoch; workgroup t keeps tile t of
// every layer's matrix in LDS, T x T weights W_l[i][j] (row block i of the layer's units, column block j of its inputs).  Per step
//
//   forward    tile (i, j) multiplies its weights with column block j of A_{l-1} and publishes a partial B x T block of net inputs;
//              the C tiles of row block i each add up a share of that block over all C, apply the activation and publish it; the
//              tiles of the next layer that need the block read it.
//   output     the last layer's tiles share the samples: net inputs summed, softmax or activation, loss, Delta_L.
//   backward   the same with rows and columns exchanged: a partial B x T block of Delta_l W_l, summed over the R tiles of column
//              block j, times f'.  W_l -= lr/B Delta_l^T A_{l-1} needs what the workgroup already holds in LDS, and is done while
//              the next block is on its way.
//
// So a layer costs two hops each way, but a hop moves B x T numbers into each workgroup where whole rows per workgroup
// (deep_batch_epoch_kernel) move B x n: 16 KB against 128 KB for 1024-wide layers at batch 32, and every weight is kept once.
//
// A last layer of at most 64 outputs is no layer of tiles (FUSED): whoever forms a run of sixteen units of A_{L-1} also publishes
// what they give to the outputs' net inputs, and every workgroup with a tile of layer L-1 keeps the columns of W_L that its row block
// feeds, forms Delta_{L-1} of the block from the outputs' Delta, and updates its copy -- during the next step's first hop.  All
// copies take the same numbers in the same order and stay equal.  This saves three hops of a step.
//
// What bounds it is latency: a hop is 1.2 us within an XCD to 2 us, of 35 us for a step of 1024-1024-1024-1024-10 at batch 32 (58.5
// before) eleven hops; the products of a hop take 0.4 us on the matrix cores, the instructions around them as much again.
// Polls that put a load behind a branch, and an update rule or activation tested per number, cost 60 us a step in the first version.
// us a step, before (one launch per product, or the kernels that own rows) / now: 784-128-10 batch 128 18.6 / 16.6, 300-500-200-300
// batch 33 52 / 27, 1348-128-1056-113 batch 10 74 / 28, 64-96-80-10 batch 8 30 / 17.
//
// Values cross workgroups as 64-bit words {value, phase number}, written and read with relaxed device-scope atomics; a consumer
// polls until the number is that of its phase (see dn_online.hip).  Partial blocks lie in one slot per workgroup and phase parity:
// a workgroup writes its slot again two phases later, and by then it has taken in a block that every reader of the slot
// contributed to after it had read.  Blocks of A_l and Delta_l have places of their own, by layer and step parity.
//
// All sums are taken in a fixed order.  Products run on v_mfma_f32_16x16x4_f32.  Parameters (and velocities that nothing reads
// before) are written at the end of the launch, so a launch whose workgroups do not all find room is taken back: workgroup 0
// waits for all of them, for a bounded time, before it publishes anything, and every step depends on it.
#include <type_traits>

#include "dn_persist.h"

namespace dn {
namespace {

constexpr int kVmcntZero = 0x0f70;   // s_waitcnt vmcnt(0), the other counters free
constexpr int kGateSpins = 1 << 17;   // polls of ~0.7 us: about 0.1 s, less than kSpinLimit polls of those that wait meanwhile

// Where element (m, c) of a B x T block or T x T tile lies in LDS.  The rows' columns are exchanged in groups of four, so that the
// matrix instruction's operands are free of bank conflicts in both directions: sixteen rows at one group of four columns, and
// rows 4q + s (q = 0..3) at sixteen consecutive columns.
template <int T>
__device__ __forceinline__ int at(int m, int c)
{
    if (T == 64) return m * 64 + (c ^ ((((m >> 2) & 3) << 4) | ((m & 3) << 2)));
    const int slot = (m & ~5) | ((m & 1) << 2) | ((m >> 2) & 1);
    return slot * 32 + (c ^ ((((m >> 3) & 1) << 4) | ((m & 3) << 2)));
}

__device__ __forceinline__ v4f mfma(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ void put(u64 *ex, uint32_t byte, float v, uint32_t seq) { ll_store((u64 *)((char *)ex + byte), v, seq); }

// Waits until all words whose bit in `need` is set carry `seq`, asking for all again until they do.  False: this or another
// workgroup gave up.
template <int N, class Again>
__device__ __forceinline__ bool wait_for(unsigned need, uint32_t seq, u64 (&w)[N], Again again, int *abort_flag, volatile int *s_abort)
{
    int spins = 0;
    for (;;) {
        unsigned missing = need;
#pragma unroll
        for (int u = 0; u < N; ++u)
            if ((uint32_t)(w[u] >> 32) == seq) missing &= ~(1u << u);
        if (!missing) return true;
        ++spins;
        if (spins > kSpinLimit) {
            __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *s_abort = 1;
            return false;
        }
        if ((spins & 255) == 0 && __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            *s_abort = 1;
            return false;
        }
        again();
    }
}
// d f'(a) for four numbers, one branch.
__device__ __forceinline__ void through_act(int act, const float (&a)[4], v4f &d)
{
    if (act == DN_ACT_TANH) {
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] *= 1.0f - a[s] * a[s];
    } else if (act == DN_ACT_SIGMOID) {
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] *= a[s] * (1.0f - a[s]);
    } else if (act == DN_ACT_RELU) {
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] = a[s] > 0.0f ? d[s] : d[s] * 0.0f;
    }
}

// What a workgroup knows about its tile of a layer, one number per lane of a register: a phase reads them with one LDS load.
enum Field : int {
    F_HAS,                                  // there is one
    F_IN, F_OUT,                            // columns and rows of the tile that are weights (the others are zero)
    F_ROW0, F_COL0,                         // its first row and column
    F_R, F_C, F_I, F_J,
    F_W, F_A, F_B,                          // LDS: tile, block of A_{l-1} (layer 1: two of them), biases
    F_ACT, F_ACT_IN,
    F_SRC_A, F_SRC_D, F_PUB_A, F_PUB_D,     // published blocks: A_{l-1}, Delta_l (to read); A_l, Delta_{l-1} (to write), step parity 0
    F_PAR_IN, F_PAR_OUT,                    // ... from parity 0 to parity 1, of layer l - 1's and layer l's blocks
    F_FWD0, F_FWD_STRIDE, F_BWD0, F_BWD_STRIDE,   // partial blocks to add up: the first, and from one to the next (phase parity 0)
    F_COUNT
};

template <int T, bool FUSED>
__global__ __launch_bounds__(TILE_THREADS) void tile_epoch_kernel(TilePlan p)
{
    static_assert(kThreads == TILE_THREADS, "eight waves");
    constexpr int G = T / 16;
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_abort;
    __shared__ int s_field[TILE_MAX_L + 1][64];
    __shared__ double s_loss[TILE_MAX_WG];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, q = lane >> 4;
    const int wid = blockIdx.x, L = p.tiled, Bp = p.rows;   // L: layers in tiles; with p.fused one more follows
    const uint32_t slot = (uint32_t)Bp * T * 8u;                   // bytes of a block
    const uint32_t part0 = p.part, part1 = slot * (uint32_t)p.grid;   // partial blocks; from one phase parity to the other
    u64 *const ex = p.ex;
    float *const Dl = lds + p.lds_d, *const tmp = lds + p.lds_tmp;
    if (tid == 0) {
        s_abort = 0;
        __hip_atomic_fetch_add(p.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int l = 1 + tid; l <= L; l += kThreads) {
        const TileLayer &y = p.layer[l], &x = p.layer[l - 1];   // (x is not read for layer 1)
        int *f = s_field[l];
        f[F_HAS] = wid < y.R * y.C;
        const int i = y.map ? wid % y.R : wid / y.C, j = y.map ? wid / y.R : wid % y.C;
        f[F_I] = i; f[F_J] = j; f[F_R] = y.R; f[F_C] = y.C;
        f[F_ROW0] = i * T; f[F_COL0] = j * T;
        f[F_OUT] = min(T, y.n_out - i * T); f[F_IN] = min(T, y.n_in - j * T);
        f[F_W] = y.lds_w; f[F_A] = y.lds_a; f[F_B] = y.lds_b;
        f[F_ACT] = y.act; f[F_ACT_IN] = l > 1 ? x.act : 0;
        f[F_SRC_A] = l > 1 ? (int)(x.pub_a + (uint32_t)j * slot) : 0;
        f[F_PUB_D] = l > 1 ? (int)(x.pub_d + (uint32_t)j * slot) : 0;
        f[F_PAR_IN] = l > 1 ? (int)((uint32_t)x.R * slot) : 0;
        f[F_SRC_D] = (int)(y.pub_d + (uint32_t)i * slot);
        f[F_PUB_A] = (int)(y.pub_a + (uint32_t)i * slot);
        f[F_PAR_OUT] = (int)((uint32_t)y.R * slot);
        f[F_FWD0] = (int)(part0 + (uint32_t)(y.map ? i : i * y.C) * slot);
        f[F_FWD_STRIDE] = (int)((uint32_t)(y.map ? y.R : 1) * slot);
        f[F_BWD0] = (int)(part0 + (uint32_t)(y.map ? j * y.R : j) * slot);
        f[F_BWD_STRIDE] = (int)((uint32_t)(y.map ? 1 : y.C) * slot);
    }
    for (int e = tid; e < p.lds_tmp; e += kThreads) lds[e] = 0.f;   // padding of tiles and blocks stays zero
    __syncthreads();

    // ---- own tiles into LDS ----
    for (int l = 1; l <= L; ++l) {
        const int *f = s_field[l];
        if (!f[F_HAS]) continue;
        const TileLayer &y = p.layer[l];
        const float *src = y.W + (size_t)f[F_ROW0] * y.n_in + f[F_COL0];
        const int h = f[F_OUT], w = f[F_IN];
        for (int e = tid; e < h * T; e += kThreads) {
            const int r = e / T, c = e % T;
            if (c < w) lds[f[F_W] + at<T>(r, c)] = src[(size_t)r * y.n_in + c];
        }
        if (f[F_J] == 0 && tid < h) {
            lds[f[F_B] + tid] = y.b[f[F_ROW0] + tid];
            lds[f[F_B] + T + tid] = y.Vb[f[F_ROW0] + tid];
        }
    }

    // Operand positions of this lane (see at()): rows n of sixteen, columns 16 g + 4 q ..; rows 4 q + s, column n (^ column block).
    int kc[G], mc[4];
    const int qx = T == 64 ? q : q >> 1;
#pragma unroll
    for (int g = 0; g < G; ++g) kc[g] = at<T>(n, 16 * g + 4 * q);
#pragma unroll
    for (int s = 0; s < 4; ++s) mc[s] = at<T>(4 * q + s, n) - (qx << 4);
    auto column = [&](int block) { return (block ^ qx) << 4; };

    // A thread moves element (row0 + u * kRows, tid % T) of a block, u = 0, 1, ..
    constexpr int kRows = kThreads / T;
    const int row0 = tid / T;
    const int spot0 = at<T>(row0, tid % T), spot1 = at<T>(row0 + kRows, tid % T) - kRows * T;   // where in LDS, for even and odd u (T = 32: the same)
    auto spot = [&](int u) { return (u & 1 ? spot1 : spot0) + u * kThreads; };

    // Sends a block of the features to LDS, rows beyond the batch zero; it is there once the wave's memory counter has been zero.
    auto load_x = [&](int64_t s0, int Bs, int par) {
        const int *f = s_field[1];
        const int n0 = p.layer[1].n_in, w = f[F_IN];
        float *dst = lds + __builtin_amdgcn_readfirstlane(f[F_A] + par * Bp * T);
        const float *src = p.X + (size_t)s0 * n0 + f[F_COL0];
        for (int r = wave; r * (64 / T) < Bp; r += kWaves) {   // sixty-four places of LDS in a row
            const int place = r * 64 + lane, slot_of = place / T;
            const int m = T == 64 ? slot_of : (slot_of & ~5) | ((slot_of & 1) << 2) | ((slot_of >> 2) & 1);
            const int c = (place % T) ^ (at<T>(m, 0) % T);
            if (m < Bs) {
                if (c < w)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (size_t)m * n0 + c),
                                                     (__attribute__((address_space(3))) void *)(dst + r * 64), 4, 0, 0);
            } else {
                dst[place] = 0.f;
            }
        }
    };
    // A published block into LDS, rows beyond the batch zero.  Its first four words may be asked for ahead of time; meet: other waves
    // may still be reading what the block replaces.  (A block is followed by as many words that can be read.)
    auto gather_ask = [&](uint32_t src, u64 (&w)[4]) {
        const u64 *from = (const u64 *)((const char *)ex + src);
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = ll_load(from + tid + u * kThreads);
    };
    auto gather_take = [&](u64 (&first)[4], uint32_t src, int Bs, uint32_t seq, float *dst, bool meet) {
        auto part = [&](auto words, int u0, auto &w, auto again) {
            constexpr int N = decltype(words)::value;
            unsigned need = 0;
#pragma unroll
            for (int u = 0; u < N; ++u) need |= row0 + (u0 + u) * kRows < Bs ? 1u << u : 0u;
            const bool ok = wait_for<N>(need, seq, w, again, p.abort_flag, &s_abort);
            if (meet && u0 == 0) __syncthreads();
            if (ok)
#pragma unroll
                for (int u = 0; u < N; ++u)
                    if (row0 + (u0 + u) * kRows < Bp) dst[spot(u) + u0 * kThreads] = need >> u & 1 ? __uint_as_float((uint32_t)w[u]) : 0.f;
            return ok;
        };
        if (!part(std::integral_constant<int, 4>{}, 0, first, [&]() { gather_ask(src, first); })) return;
        for (int u0 = 4; u0 * kRows < Bp; u0 += 8) {
            u64 w[8];
            auto ask = [&]() {
                const u64 *from = (const u64 *)((const char *)ex + src) + u0 * kThreads;
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = ll_load(from + tid + u * kThreads);
            };
            ask();
            if (!part(std::integral_constant<int, 8>{}, u0, w, ask)) return;
        }
    };
    auto gather = [&](uint32_t src, int Bs, uint32_t seq, float *dst) {
        u64 w[4];
        gather_ask(src, w);
        gather_take(w, src, Bs, seq, dst, false);
    };

    // Sums over P published numbers, `stride` bytes apart, of the runs of sixteen numbers rank, rank + every, .. below total, a number
    // per lane of a row: place(run) is where the run's numbers begin in the first block.  A wave takes K runs at a time; its four
    // rows of lanes take every fourth number each, V at once.  fin(run, sum) on all lanes.
    auto sum_runs = [&](auto runs, auto at_once, int rank, int every, int total, uint32_t stride, int P, uint32_t seq, auto place, auto fin) {
        constexpr int K = decltype(runs)::value, V = decltype(at_once)::value, N = K * V;
        const int groups = (P + 3) >> 2;
        const uint32_t lane_at = (uint32_t)q * stride + (uint32_t)n * 8u;
        const uint32_t over = (uint32_t)min(q, P - 1 - 4 * (groups - 1)) * stride + (uint32_t)n * 8u;   // (P not a multiple of four)
        for (int r0 = rank + every * wave; r0 < total; r0 += 8 * K * every) {
            float s[K];
#pragma unroll
            for (int k = 0; k < K; ++k) s[k] = 0.f;
            for (int g0 = 0; g0 < groups; g0 += V) {
                u64 w[N];
                auto ask_all = [&]() {
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const int run = r0 + 8 * (u / V) * every, g = min(g0 + u % V, groups - 1);
                        const uint32_t first = place(run < total ? run : r0) + 4u * (uint32_t)g * stride;
                        w[u] = ll_load((const u64 *)((const char *)ex + first + (g == groups - 1 ? over : lane_at)));
                    }
                };
                ask_all();
                unsigned need = 0;
#pragma unroll
                for (int u = 0; u < N; ++u) need |= r0 + 8 * (u / V) * every < total && 4 * (g0 + u % V) + q < P ? 1u << u : 0u;
                if (!wait_for<N>(need, seq, w, ask_all, p.abort_flag, &s_abort)) return;
#pragma unroll
                for (int u = 0; u < N; ++u) s[u / V] += need >> u & 1 ? __uint_as_float((uint32_t)w[u]) : 0.f;
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float sum = add_rows(s[k]);
                if (r0 + 8 * k * every < total) fin(r0 + 8 * k * every, sum);
            }
        }
    };
    // This workgroup's share (rank of P) of the sum of P partial blocks, Bs rows: fin(m, first column of the run, sum) on all lanes.
    auto reduce = [&](uint32_t first, uint32_t stride, int P, int rank, int Bs, uint32_t seq, auto fin) {
        auto place = [&](int run) { return first + (uint32_t)run * 128u; };   // (run = row * G + column / 16)
        auto end = [&](int run, float sum) { fin(run / G, run % G * 16, sum); };
        if (Bs * G <= 8 * P && P <= 16) sum_runs(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{}, rank, P, Bs * G, stride, P, seq, place, end);
        else sum_runs(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{}, rank, P, Bs * G, stride, P, seq, place, end);
    };

    // Products of a B x T block with the tile, K = 16 groups: store(tm, tj, acc) per 16 x 16 numbers.
    constexpr int kStripes = kWaves / G;
    const int tj = wave % G;
    auto forward = [&](const float *A, const float *W, int mt, float bias, auto store) {
        v4f w[G];
#pragma unroll
        for (int g = 0; g < G; ++g) w[g] = *(const v4f *)(W + tj * 16 * T + kc[g]);
        for (int tm = wave / G; tm < mt; tm += kStripes) {
            v4f a[G], acc = {bias, bias, bias, bias};
#pragma unroll
            for (int g = 0; g < G; ++g) a[g] = *(const v4f *)(A + tm * 16 * T + kc[g]);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = mfma(a[g][s], w[g][s], acc);
            store(tm, acc);
        }
    };
    // ... K = 16 NG times `pieces`; D goes on a block further where its T columns end.
    auto backward = [&](auto groups, const float *D, const float *W, int mt, int pieces, auto store) {
        constexpr int NG = decltype(groups)::value;
        for (int tm = wave / G; tm < mt; tm += kStripes) {
            v4f acc = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < pieces; ++k) {
                const int g0 = k * NG;
                const float *Wc = W + column(tj) + g0 * 16 * T, *Dp = D + g0 / G * Bp * T + tm * 16 * T;
                v4f d[NG];
                float w[NG][4];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    d[g] = *(const v4f *)(Dp + kc[(NG == G ? 0 : (G == 4 && (k & 1)) ? 2 : 0) + g]);
#pragma unroll
                    for (int s = 0; s < 4; ++s) w[g][s] = Wc[mc[s] + g * 16 * T];
                }
#pragma unroll
                for (int g = 0; g < NG; ++g)
#pragma unroll
                    for (int s = 0; s < 4; ++s) acc = mfma(d[g][s], w[g][s], acc);
            }
            store(tm, acc);
        }
    };

    // W -= scale D^T A for the sixteenths (tr, tj0 + k) of a tile with `rows` x `cols` weights, where D is B x rows and A is B x cols;
    // vel: their velocities (V: where they go in device memory, n_in a row; null: nowhere).
    // (One rule without branches: plain descent is momentum 0 from velocity 0.)
    const bool momentum = p.mu != 0.f;
    constexpr int NT = T == 64 ? 2 : 1;
    const int tr = wave >> 1, tj0 = (wave & 1) * NT;
    auto update = [&](int k, const float *D, const float *A, float *W, int rows, int cols, int mt, float scale, float (&vel)[4],
                      float *V, int n_in) {
        if (tr * 16 >= rows || (tj0 + k) * 16 >= cols) return;
        const int col = column(tj0 + k);
        float *Wt = W + tr * 16 * T + col;
        float w[4];
        v4f sums[4];   // (a quarter of the chain each, and closer to 64 bits)
#pragma unroll
        for (int s = 0; s < 4; ++s) sums[s] = (v4f){0.f, 0.f, 0.f, 0.f};
        D += column(tr % G);
        A += col;
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s] = Wt[mc[s]];
        int b = 0;
        for (; b + 2 <= mt; b += 2, D += 32 * T, A += 32 * T) {
            float d[8], a[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                d[s] = D[mc[s & 3] + (s >> 2) * 16 * T];
                a[s] = A[mc[s & 3] + (s >> 2) * 16 * T];
            }
            __builtin_amdgcn_sched_barrier(0);   // (all loads, then all products)
#pragma unroll
            for (int s = 0; s < 8; ++s) sums[s & 3] = mfma(d[s], a[s], sums[s & 3]);
        }
        if (b < mt) {
            float d[4], a[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                d[s] = D[mc[s]];
                a[s] = A[mc[s]];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) sums[s] = mfma(d[s], a[s], sums[s]);
        }
        const v4f g = (sums[0] + sums[1]) + (sums[2] + sums[3]);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool in = tr * 16 + 4 * q + s < rows && (tj0 + k) * 16 + n < cols;
            vel[s] = (momentum ? p.mu * vel[s] : 0.f) - scale * g[s];
            Wt[mc[s]] = in ? w[s] + vel[s] : 0.f;   // (padding stays zero beside infinities too)
        }
        if (V)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (tr * 16 + 4 * q + s < rows && (tj0 + k) * 16 + n < cols) V[(size_t)s * n_in + k * 16] = vel[s];
    };

    // ---- nothing is published before all workgroups are here ----
    if (wid == 0 && tid == 0) {
        int spins = 0;
        while (__hip_atomic_load(p.arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < p.expected)
            if (++spins > kGateSpins) {
                __hip_atomic_store(p.settled, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                drain_device_scope_stores();
                __hip_atomic_store(p.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_abort = 1;
                break;
            }
    }
    const int64_t nsteps = (p.n_samples + p.batch - 1) / p.batch;
    if (s_field[1][F_HAS]) load_x(0, (int)min((int64_t)p.batch, p.n_samples), 0);
    __builtin_amdgcn_s_waitcnt(kVmcntZero);

    // The narrow last layer that follows the tiles (p.fused): every workgroup with a tile of layer L keeps the columns of W that its row
    // block's units feed, and all biases; each copy takes the same update.
    constexpr bool fused = FUSED;
    const bool last_tile = s_field[L][F_HAS] != 0;
    const int PO = (p.out.n_out + 15) & ~15;   // words a sample in what is published of that layer
    float *const WL = lds + p.out.lds_w, *const AL = lds + p.out.lds_a, *const DL = lds + p.lds_dl, *const bL = lds + p.out.lds_b;
    float vel_out[NT][4], vel_bias = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) vel_out[k][s] = 0.f;
    auto each_out = [&](auto run) {   // run(weight in device memory, its place in LDS, its velocity) of the sixteenths this lane updates
        const int rows = p.out.n_out, cols = s_field[L][F_OUT], c0 = s_field[L][F_ROW0];
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int r = tr * 16 + 4 * q + s, c = (tj0 + k) * 16 + n;
                if (r < rows && c < cols) run((size_t)r * p.out.n_in + c0 + c, at<T>(r, c), vel_out[k][s]);
            }
    };
    if (fused && last_tile) {
        each_out([&](size_t e, int pos, float &v) {
            WL[pos] = p.out.W[e];
            v = p.out.VW[e];
        });
        if (tid < p.out.n_out) bL[tid] = p.out.b[tid];
        if (wave >= 4 && (wave - 4) * 16 + n < p.out.n_out) vel_bias = p.out.Vb[(wave - 4) * 16 + n];
    }
    __syncthreads();
    int prev_rows = 0;   // of the step whose update of that layer is still to be done
    float prev_scale = 0.f;
    auto update_out = [&]() {
        const int mt = (prev_rows + 15) >> 4;
#pragma unroll
        for (int k = 0; k < NT; ++k) update(k, DL + tr / G * Bp * T, AL, WL, p.out.n_out, s_field[L][F_OUT], mt, prev_scale, vel_out[k], nullptr, 0);
        if (wave >= 4 && (wave - 4) * 16 < p.out.n_out) {   // the biases: sixteen a wave
            const int t = wave - 4;
            const float *D = DL + t / G * Bp * T + column(t % G);
            float g = 0.f;
            for (int b = 0; b < mt; ++b, D += 16 * T) g += (D[mc[0]] + D[mc[1]]) + (D[mc[2]] + D[mc[3]]);
            g = add_rows(g);
            vel_bias = (momentum ? p.mu * vel_bias : 0.f) - prev_scale * g;
            if (q == 0 && t * 16 + n < p.out.n_out) bL[t * 16 + n] += vel_bias;
        }
    };

    double loss = 0.0;
    const uint32_t out_blocks = (uint32_t)((p.out.n_out + T - 1) / T);   // of outputs, 16 G each
    const int nL = p.out.n_out, PT = (nL + T - 1) / T * T, runs_out = PO >> 4, runs_in = (p.out.n_in + 15) >> 4;
    int64_t step = 0;
    if (!s_abort)
        for (; step < nsteps + (fused ? 1 : 0); ++step) {   // (one turn more: the last update of the narrow layer)
            const bool more = step < nsteps;
            const int64_t s0 = step * p.batch;
            const int Bs = (int)min((int64_t)p.batch, p.n_samples - s0);   // the last batch may be short
            const int mt = (Bs + 15) >> 4, par = (int)(step & 1);
            const uint32_t seq0 = p.seq0 + 1u + (uint32_t)step * (uint32_t)(2 * L - 1);
            const float scale = p.lr / (float)Bs;
            const uint32_t zp = p.zp + (par ? (uint32_t)(Bp * runs_in * PO) * 8u : 0u);   // [sample][run of 16 units][output]
            const uint32_t dp = p.dp + (par ? out_blocks * slot : 0u);                      // [sample][output], in blocks

            // ---- forward ----
            for (int l = 1; l <= L; ++l) {
                const int fields = s_field[l][lane];
                auto f = [&](int k) { return __builtin_amdgcn_readlane(fields, k); };
                const bool has = f(F_HAS) != 0;
                const uint32_t seq = seq0 + (uint32_t)(l - 1), phase = (seq & 1) ? part1 : 0u;
                const int valid = f(F_OUT), act = f(F_ACT);
                const uint32_t pub = (uint32_t)f(F_PUB_A) + (par ? (uint32_t)f(F_PAR_OUT) : 0u);
                const bool whole = f(F_C) == 1 && l < L;   // no partial blocks: this tile's is the sum
                if (has && more) {
                    float *A = lds + f(F_A) + (l == 1 ? par * Bp * T : 0);
                    if (l > 1) {
                        gather((uint32_t)f(F_SRC_A) + (par ? (uint32_t)f(F_PAR_IN) : 0u), Bs, seq - 1, A);
                        __syncthreads();
                        if (s_abort) break;
                    }
                    const uint32_t to = (whole ? pub : part0 + phase + (uint32_t)wid * slot) + (uint32_t)(4 * q * T + tj * 16 + n) * 8u;
                    forward(A, lds + f(F_W), mt, f(F_J) == 0 ? lds[f(F_B) + tj * 16 + n] : 0.f, [&](int tm, v4f acc) {
                        if (whole) {
#pragma unroll
                            for (int s = 0; s < 4; ++s) acc[s] = tj * 16 + n < valid ? act_fn(act, acc[s]) : 0.f;
                        }
#pragma unroll
                        for (int s = 0; s < 4; ++s) put(ex, to + (uint32_t)((tm * 16 + s) * T * 8), acc[s], seq);   // (rows beyond Bs are not read)
                    });
                }
                if (fused && l == 1) {   // the last step's update of the narrow layer, while these blocks are on their way
                    if (step > 0 && last_tile) update_out();
                    if (!more) break;
                    if (L == 1) __syncthreads();   // (else a gather's barrier comes before the layer is used)
                }
                if (has && (l < L || fused) && !whole) {
                    const int run0 = f(F_ROW0) >> 4;
                    reduce((uint32_t)f(F_FWD0) + phase, (uint32_t)f(F_FWD_STRIDE), f(F_C), f(F_J), Bs, seq, [&](int m, int c0, float z) {
                        const float a = c0 + n < valid ? act_fn(act, z) : 0.f;
                        if (q == 0) put(ex, pub + (uint32_t)(m * T + c0 + n) * 8u, a, seq);
                        if (fused && l == L && c0 < valid) {   // what these sixteen units give to the outputs' net inputs
                            const uint32_t at_z = zp + (uint32_t)((m * runs_in + run0 + (c0 >> 4)) * PO) * 8u;
                            for (int o = q; o < PO; o += 4) {
                                const float z2 = row16_sum(a * WL[at<T>(o, c0 + n)]);
                                if (n == 0) put(ex, at_z + (uint32_t)o * 8u, z2, seq);
                            }
                        }
                    });
                }
            }
            if (s_abort || !more) break;   // (the flag is set before a barrier that all waves have passed, or noticed at the next one)

            // ---- output: net inputs, loss and Delta of this workgroup's samples wid, wid + NR, .. ----
            const int NR = fused ? s_field[L][F_R] * s_field[L][F_C] : p.grid;
            const int ns = wid < NR && wid < Bs ? (Bs - wid + NR - 1) / NR : 0;
            const uint32_t seq_out = seq0 + (uint32_t)(L - 1);
            u64 early[4];   // the first words of a block that will be needed
            uint32_t src_al = 0;
            if (fused && last_tile) {
                src_al = (uint32_t)__builtin_amdgcn_readfirstlane(s_field[L][F_PUB_A] + (par ? s_field[L][F_PAR_OUT] : 0));
                gather_ask(src_al, early);
            }
            if (ns > 0) {
                int lab = p.labels[s0 + wid + NR * min(wave, ns - 1)];   // (before the words that take longer)
                const int total = ns * runs_out;
                float *const z = Dl;   // (free until Delta comes)
                auto end = [&](int run, float sum) {
                    if (q == 0) z[run * 16 + n] = sum;   // (run = sample * runs_out + run of outputs)
                };
                if (fused) {
                    auto place = [&](int run) {
                        const int sm = runs_out == 1 ? run : run / runs_out;
                        return zp + (uint32_t)((wid + NR * sm) * runs_in * PO + (run - sm * runs_out) * 16) * 8u;
                    };
                    if (total <= 8 && runs_in > 16) sum_runs(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{}, 0, 1, total, (uint32_t)PO * 8u, runs_in, seq_out, place, end);
                    else sum_runs(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{}, 0, 1, total, (uint32_t)PO * 8u, runs_in, seq_out, place, end);
                } else {
                    const uint32_t phase = part0 + ((seq_out & 1) ? part1 : 0u);
                    auto place = [&](int run) {
                        const int sm = run / runs_out, o = (run - sm * runs_out) * 16, block = o / T;
                        return phase + (uint32_t)(p.out.map ? block : block * p.out.C) * slot + (uint32_t)((wid + NR * sm) * T + o % T) * 8u;
                    };
                    sum_runs(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{}, 0, 1, total, (uint32_t)(p.out.map ? p.out.R : 1) * slot, p.out.C, seq_out, place, end);
                }
                __syncthreads();
                if (s_abort) break;
                for (int sm = wave; sm < ns; sm += kWaves) {
                    const int m = wid + NR * sm;
                    float *zr = z + sm * PO;
                    if (sm >= kWaves) lab = p.labels[s0 + m];
                    lab = lab < 0 ? 0 : lab >= nL ? nL - 1 : lab;
                    if (fused) {
                        for (int o = lane; o < nL; o += 64) zr[o] += bL[o];
                    }
                    const uint32_t dst = fused ? dp + (uint32_t)(m * T) * 8u : p.out.pub_d + (par ? (uint32_t)p.out.R * slot : 0u) + (uint32_t)(m * T) * 8u;
                    float e, top = -INFINITY, inv = 0.f;
                    if (p.loss == DN_LOSS_CROSS_ENTROPY) {
                        float sum = 0.f;
                        for (int o = lane; o < nL; o += 64) top = fmaxf(top, zr[o]);
                        top = wave_max(top);
                        for (int o = lane; o < nL; o += 64) sum += expf(zr[o] - top);
                        sum = wave_sum(sum);
                        inv = 1.0f / sum;
                        e = logf(sum) - (zr[lab] - top);
                    } else {
                        e = 0.f;
                        for (int o = lane; o < nL; o += 64) {
                            zr[o] = act_fn(p.out.act, zr[o]);
                            const float d = zr[o] - (o == lab ? 1.0f : 0.0f);
                            e += 0.5f * d * d;
                        }
                        e = wave_sum(e);
                    }
                    for (int o = lane; o < PT; o += 64) {   // (all columns of the blocks)
                        const float target = o == lab ? 1.0f : 0.0f;
                        float d = 0.f;
                        if (o < nL) d = p.loss == DN_LOSS_CROSS_ENTROPY ? expf(zr[o] - top) * inv - target : (zr[o] - target) * act_deriv(p.out.act, zr[o]);
                        put(ex, dst + (uint32_t)(o / T) * slot + (uint32_t)(o % T) * 8u, d, seq_out);
                    }
                    loss += (double)e;
                }
                __syncthreads();   // z gives way to Delta
            }
            if (fused && last_tile) gather_take(early, src_al, Bs, seq_out, AL, false);

            // the next batch's features, while Delta is on its way
            if (step + 1 < nsteps && s_field[1][F_HAS])
                load_x(s0 + p.batch, (int)min((int64_t)p.batch, p.n_samples - s0 - p.batch), par ^ 1);

            // ---- backward and update ----
            bool asked = false;
            for (int l = L; l >= 1; --l) {
                const int fields = s_field[l][lane];
                auto f = [&](int k) { return __builtin_amdgcn_readlane(fields, k); };
                if (!f(F_HAS)) continue;
                const uint32_t seq = seq0 + (uint32_t)(2 * L - l), phase = (seq & 1) ? part1 : 0u;   // of this layer's partial blocks
                float *A = lds + f(F_A) + (l == 1 ? par * Bp * T : 0), *W = lds + f(F_W);
                const int rows = f(F_OUT), cols = f(F_IN);
                // velocities of the weights this lane will update
                float vel[NT][4];
                float *V = nullptr;
                int n_in = 0;
#pragma unroll
                for (int k = 0; k < NT; ++k)
#pragma unroll
                    for (int s = 0; s < 4; ++s) vel[k][s] = 0.f;
                if (momentum || (p.keep_v && step == nsteps - 1)) {
                    n_in = p.layer[l].n_in;
                    V = p.layer[l].VW + (size_t)(f(F_ROW0) + tr * 16 + 4 * q) * n_in + f(F_COL0) + tj0 * 16 + n;
                    if (momentum)
#pragma unroll
                        for (int k = 0; k < NT; ++k)
#pragma unroll
                            for (int s = 0; s < 4; ++s)
                                if (tr * 16 + 4 * q + s < rows && (tj0 + k) * 16 + n < cols) vel[k][s] = V[(size_t)s * n_in + k * 16];
                }
                if (fused && l == L) {
                    // Delta_L of the row block from the outputs' Delta
                    for (uint32_t b = 0; b < out_blocks; ++b) gather(dp + b * slot, Bs, seq_out, DL + b * Bp * T);
                    __syncthreads();
                    if (s_abort) break;
                    const int act = f(F_ACT);
                    auto keep = [&](int tm, v4f acc) {
                        const int pos = tm * 16 * T + column(tj);
                        float a[4];
#pragma unroll
                        for (int s = 0; s < 4; ++s) a[s] = AL[mc[s] + pos];
                        through_act(act, a, acc);
#pragma unroll
                        for (int s = 0; s < 4; ++s) Dl[mc[s] + pos] = tj * 16 + n < rows ? acc[s] : 0.f;
                    };
                    if (PO == 16) backward(std::integral_constant<int, 1>{}, DL, WL, mt, 1, keep);
                    else backward(std::integral_constant<int, 2>{}, DL, WL, mt, (PO + 31) >> 5, keep);
                    __syncthreads();
                } else {
                    const uint32_t src = (uint32_t)f(F_SRC_D) + (par ? (uint32_t)f(F_PAR_OUT) : 0u);
                    if (!asked) gather_ask(src, early);
                    gather_take(early, src, Bs, seq - 1, Dl, asked);
                    asked = false;
                    __syncthreads();
                    if (s_abort) break;
                }
                const uint32_t pub = (uint32_t)f(F_PUB_D) + (par ? (uint32_t)f(F_PAR_IN) : 0u);
                const bool whole = f(F_R) == 1;
                const int act_in = f(F_ACT_IN);
                if (l > 1) {
                    const uint32_t to = (whole ? pub : part0 + phase + (uint32_t)wid * slot) + (uint32_t)(4 * q * T + tj * 16 + n) * 8u;
                    backward(std::integral_constant<int, G>{}, Dl, W, mt, 1, [&](int tm, v4f acc) {
                        if (whole) {
                            float a[4];
#pragma unroll
                            for (int s = 0; s < 4; ++s) a[s] = A[mc[s] + tm * 16 * T + column(tj)];
                            through_act(act_in, a, acc);
#pragma unroll
                            for (int s = 0; s < 4; ++s) acc[s] = tj * 16 + n < cols ? acc[s] : 0.f;
                        }
#pragma unroll
                        for (int s = 0; s < 4; ++s) put(ex, to + (uint32_t)((tm * 16 + s) * T * 8), acc[s], seq);
                    });
                }
                const bool biased = f(F_J) == 0;
                if (biased) {   // column sums of Delta_l, in 512 / T parts
                    float g = 0.f;   // (rows beyond the batch are zero, up to a multiple of sixteen)
                    for (int u = 0; u * kRows < 16 * mt; u += 2) g += Dl[spot0 + u * kThreads] + ((u + 1) * kRows < 16 * mt ? Dl[spot1 + (u + 1) * kThreads] : 0.f);
                    tmp[tid] = g;
                }
                if (l == 1) __builtin_amdgcn_s_waitcnt(kVmcntZero);   // (features that load_x sent for are in LDS)
                __syncthreads();
                // the update, between the words that are waited for
                if (NT == 2 || l == 1) update(0, Dl, A, W, rows, cols, mt, scale, vel[0], V, n_in);
                if (l > 1 && !whole)
                    reduce((uint32_t)f(F_BWD0) + phase, (uint32_t)f(F_BWD_STRIDE), f(F_R), f(F_I), Bs, seq, [&](int m, int c0, float s) {
                        if (q == 0) put(ex, pub + (uint32_t)(m * T + c0 + n) * 8u, c0 + n < cols ? s * act_deriv(act_in, A[at<T>(m, c0 + n)]) : 0.f, seq);
                    });
                if (l > 1) {
                    const int *x = s_field[l - 1];
                    if (x[F_HAS]) {
                        asked = true;
                        gather_ask((uint32_t)__builtin_amdgcn_readfirstlane(x[F_SRC_D] + (par ? x[F_PAR_OUT] : 0)), early);
                    }
                }
                if (NT == 2) update(NT - 1, Dl, A, W, rows, cols, mt, scale, vel[NT - 1], V, n_in);
                else if (l > 1) update(0, Dl, A, W, rows, cols, mt, scale, vel[0], V, n_in);
                if (biased && tid < rows) {
                    float g = 0.f;
#pragma unroll
                    for (int k = 0; k < kRows; ++k) g += tmp[k * T + tid];
                    float *b = lds + f(F_B) + tid;
                    const float v = (momentum ? p.mu * b[T] : 0.f) - scale * g;
                    *b += v;
                    b[T] = v;
                }
                if (!asked) __syncthreads();
            }
            if (s_abort) break;
            prev_rows = Bs;
            prev_scale = scale;
        }
    __syncthreads();
    if (s_abort || step < nsteps) return;
    if (fused && last_tile) {
        if (s_field[L][F_J] == 0) {
            const bool v_too = p.mu != 0.f || p.keep_v;
            each_out([&](size_t e, int pos, float &v) {
                p.out.W[e] = WL[pos];
                if (v_too) p.out.VW[e] = v;
            });
            if (wid == 0) {
                if (tid < nL) p.out.b[tid] = bL[tid];
                const int o = (wave - 4) * 16 + n;
                if (v_too && wave >= 4 && q == 0 && o < nL) p.out.Vb[o] = vel_bias;
            }
        }
    }

    // ---- own tiles back ----
    for (int l = 1; l <= L; ++l) {
        const int *f = s_field[l];
        if (!f[F_HAS]) continue;
        const TileLayer &y = p.layer[l];
        float *dst = y.W + (size_t)f[F_ROW0] * y.n_in + f[F_COL0];
        const int h = f[F_OUT], w = f[F_IN];
        for (int e = tid; e < h * T; e += kThreads) {
            const int r = e / T, c = e % T;
            if (c < w) dst[(size_t)r * y.n_in + c] = lds[f[F_W] + at<T>(r, c)];
        }
        if (f[F_J] == 0 && tid < h) {
            y.b[f[F_ROW0] + tid] = lds[f[F_B] + tid];
            if (p.mu != 0.f || p.keep_v) y.Vb[f[F_ROW0] + tid] = lds[f[F_B] + T + tid];
        }
    }
    // ---- losses: a sum per workgroup, added up by the first ----
    if (lane == 0) s_loss[wave] = loss;
    __syncthreads();
    const uint32_t seq = p.seq0 + (uint32_t)nsteps * (uint32_t)(2 * L - 1) + 1u;
    if (tid == 0) {
        double sum = 0.0;
        for (int k = 0; k < kWaves; ++k) sum += s_loss[k];
        const u64 bits = (u64)__double_as_longlong(sum);
        put(ex, (uint32_t)wid * 16u, __uint_as_float((uint32_t)bits), seq);
        put(ex, (uint32_t)wid * 16u + 8u, __uint_as_float((uint32_t)(bits >> 32)), seq);
    }
    if (wid != 0) return;
    __syncthreads();
    if (tid < p.grid) {
        u64 w[2];
        auto ask = [&]() {
            w[0] = ll_load(ex + 2 * tid);
            w[1] = ll_load(ex + 2 * tid + 1);
        };
        ask();
        wait_for<2>(3u, seq, w, ask, p.abort_flag, &s_abort);
        s_loss[tid] = __longlong_as_double((long long)((u64)(uint32_t)w[0] | (w[1] << 32)));
    }
    __syncthreads();
    if (tid == 0 && !s_abort) {
        double sum = 0.0;
        for (int k = 0; k < p.grid; ++k) sum += s_loss[k];
        *p.loss_acc += sum;
    }
}

bool geometry_of(const int32_t *n, int L, int T, int batch, int max_wg, TileGeom &g)
{
    g = TileGeom{};
    g.T = T;
    g.rows = (batch + 15) / 16 * 16;
    g.fused = L > 1 && n[L] <= 64;   // a narrow last layer rides with the tiles of the one before
    g.tiled = L - g.fused;
    int at = 0;
    const int block = g.rows * T, out16 = (n[L] + 15) / 16 * 16;
    for (int l = 1; l <= g.tiled; ++l) {
        const int64_t R = ((int64_t)n[l] + T - 1) / T, C = ((int64_t)n[l - 1] + T - 1) / T;
        if (R * C > max_wg) return false;
        g.R[l] = (int)R;
        g.C[l] = (int)C;
        g.map[l] = l & 1;
        if ((int)(R * C) > g.grid) g.grid = (int)(R * C);
        g.lds_w[l] = at;
        at += T * T;
        g.lds_a[l] = at;
        at += block * (l == 1 ? 2 : 1);
        g.lds_b[l] = at;
        at += 2 * T;
    }
    int samples = (g.rows + g.grid - 1) / g.grid;   // of a workgroup, in the output stage
    if (g.fused) {
        const int h = g.tiled, groups = g.R[h] * g.C[h];
        samples = (g.rows + groups - 1) / groups;
        g.lds_w[L] = at;
        at += (out16 == 16 ? 16 : (out16 + 31) / 32 * 32) * T;   // (products take 16 or 32 outputs at a time)
        g.lds_a[L] = at;
        at += block;
        g.lds_b[L] = at;
        at += 64;
        g.lds_dl = at;
        at += (n[L] + T - 1) / T * block;
    }
    g.lds_d = at;   // Delta_l, and before it the net inputs of a workgroup's samples
    at += block > samples * out16 ? block : samples * out16;
    g.lds_tmp = at;
    at += TILE_THREADS;
    g.lds_floats = at;
    if ((size_t)at * sizeof(float) > TILE_MAX_LDS_BYTES) return false;
    // exchange region, in 64-bit words
    size_t w = (size_t)2 * TILE_MAX_WG;   // losses
    g.off_part = w;
    w += (size_t)2 * g.grid * block;
    for (int l = 1; l <= g.tiled; ++l) {
        g.off_a[l] = w;
        if (l < L) w += (size_t)2 * g.R[l] * block;
        g.off_d[l] = w;
        w += (size_t)2 * g.R[l] * block;
    }
    if (g.fused) {
        g.off_z = w;
        w += (size_t)2 * g.rows * ((n[L - 1] + 15) / 16) * out16;
        g.off_dp = w;
        w += (size_t)2 * ((n[L] + T - 1) / T) * block;
    }
    w += (size_t)8 * TILE_THREADS;   // (blocks are read in pieces of this many words)
    g.words = w;
    return true;
}

}  // namespace

namespace {

// Microseconds a step takes, from what it consists of; the numbers fit 337 nets (two to five layers of 8 to 4096 units, batch 2 to 256,
// tiles of 32 and of 64) to 10 %: a round of waiting for up to sixteen words a lane 1.4 in a sum and 0.8 in the output stage, a
// block read 1.2 and as much for every eight further words a thread, sixteen rows times a tile of 64 1.0 in a product and 1.4 in an
// update, eight samples of a workgroup through the output stage 2.5, eight runs of sixteen units into a narrow layer's sums 0.06 an
// output, everything else 3.7.
float step_us(const int32_t *n, int L, int batch, const TileGeom &g)
{
    const int T = g.T, G = T / 16, h = g.tiled, mt = g.rows / 16;
    auto up = [](int a, int b) { return (a + b - 1) / b; };
    auto sum_rounds = [&](int P) {   // of a workgroup's share of a block, P partial blocks
        const int runs = batch * G;
        return runs <= 8 * P && P <= 16 ? 1 : up(up(runs, P), 16) * up(up(P, 4), 8);
    };
    const int words = g.rows * T / TILE_THREADS, reads = 1 + (words > 4 ? up(words - 4, 8) : 0);
    const float product = (float)up(mt, 8 / G) * (float)T / 64.f;
    int sums = 0, blocks = 0;
    float products = 0.f;
    for (int l = 1; l <= h; ++l) {
        blocks += l > 1 ? 2 * reads : reads;
        products += l > 1 ? 2.f * product : product;
        if ((l < h || g.fused) && !(g.C[l] == 1 && l < h)) sums += sum_rounds(g.C[l]);
        if (l > 1 && g.R[l] > 1) sums += sum_rounds(g.R[l]);
    }
    const int groups = g.fused ? g.R[h] * g.C[h] : g.grid, samples = up(batch, groups), out16 = up(n[L], 16);
    const int from = g.fused ? up(n[L - 1], 16) : g.C[h];
    const int out_rounds = g.fused && samples * out16 <= 8 && from > 16 ? up(from, 64) : up(samples * out16, 16) * up(up(from, 4), 4);
    const float narrow = g.fused ? (float)up(up(batch * G, g.C[h]), 8) * (float)out16 / 4.f : 0.f;
    return 3.7f + 1.38f * (float)sums + 1.15f * (float)blocks + 1.03f * products + 0.84f * (float)out_rounds + 2.5f * (float)up(samples, 8) +
           3.7f * narrow + 1.39f * (float)(h * mt) * (float)T / 64.f;
}

}  // namespace

bool tile_geometry(const int32_t *n, int L, int batch, int max_wg, TileGeom &g)
{
    if (L < 1 || L > TILE_MAX_L || n[L] > TILE_MAX_NL || batch < 1 || batch > TILE_MAX_BATCH) return false;
    if (max_wg > TILE_MAX_WG) max_wg = TILE_MAX_WG;
    // The smaller tile where it fits: more workgroups, each with less to move.  us a step, 32 / 64: 64-96-80-10 batch 8 17.0 / 22.6;
    // 300-500-200-300 batch 33 26.6 / 49; 784-128-10 batch 128 16.6 / (LDS).  1024-1024-1024-1024-10 is 256 tiles of 64.
    for (int T : {32, 64})
        if (geometry_of(n, L, T, batch, max_wg, g)) {
            g.step_us = step_us(n, L, batch, g);
            return true;
        }
    return false;
}

size_t tile_exchange_bytes(const int32_t *n, int L, int max_batch)
{
    size_t most = 0;
    if (L < 1 || L > TILE_MAX_L || n[L] > TILE_MAX_NL) return 0;
    for (int T : {32, 64})
        for (int rows = max_batch < TILE_MAX_BATCH ? (max_batch + 15) / 16 * 16 : TILE_MAX_BATCH; rows >= 16; rows -= 16) {
            TileGeom g;
            if (!geometry_of(n, L, T, rows, TILE_MAX_WG, g)) continue;
            if (g.words * sizeof(u64) > most) most = g.words * sizeof(u64);
            break;   // fewer rows need less
        }
    return most;
}

hipError_t tile_prepare()
{
    for (const void *k : {reinterpret_cast<const void *>(tile_epoch_kernel<32, false>), reinterpret_cast<const void *>(tile_epoch_kernel<32, true>),
                          reinterpret_cast<const void *>(tile_epoch_kernel<64, false>), reinterpret_cast<const void *>(tile_epoch_kernel<64, true>)}) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TILE_MAX_LDS_BYTES);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_tile_epoch(const TileGeom &g, TilePlan plan, int L, hipStream_t stream)
{
    plan.grid = g.grid;
    plan.rows = g.rows;
    plan.lds_d = g.lds_d;
    plan.lds_tmp = g.lds_tmp;
    plan.part = (uint32_t)(g.off_part * sizeof(u64));
    plan.tiled = g.tiled;
    plan.fused = g.fused;
    plan.lds_dl = g.lds_dl;
    plan.zp = (uint32_t)(g.off_z * sizeof(u64));
    plan.dp = (uint32_t)(g.off_dp * sizeof(u64));
    for (int l = 1; l <= L; ++l) {
        TileLayer &y = plan.layer[l];
        y.R = g.R[l]; y.C = g.C[l]; y.map = g.map[l];
        y.lds_w = g.lds_w[l]; y.lds_a = g.lds_a[l]; y.lds_b = g.lds_b[l];
        y.pub_a = (uint32_t)(g.off_a[l] * sizeof(u64));
        y.pub_d = (uint32_t)(g.off_d[l] * sizeof(u64));
    }
    plan.out = plan.layer[L];
    const size_t bytes = (size_t)g.lds_floats * sizeof(float);
    if (g.T == 32)
        return g.fused ? launch_resident(tile_epoch_kernel<32, true>, plan, g.grid, bytes, stream)
                       : launch_resident(tile_epoch_kernel<32, false>, plan, g.grid, bytes, stream);
    return g.fused ? launch_resident(tile_epoch_kernel<64, true>, plan, g.grid, bytes, stream)
                   : launch_resident(tile_epoch_kernel<64, false>, plan, g.grid, bytes, stream);
}

}  // namespace dn
