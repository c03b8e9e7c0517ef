// Per-sample training of nets whose layers fit the LDS of a few workgroups.
//
// The kernels that spread every layer over as many workgroups as there are (dn_online.hip, dn_twin.hip) pay an exchange through
// memory per layer and direction, 1.9 us with 256 workgroups, and instructions for partial sums over all of them: 14 to 25 us a step
// for three and four layers, however small.  Here a net takes as few workgroups as hold it: one, if its weights (and velocities) fit
// one LDS, which then has no exchange at all, or P of up to 32 on one XCD, where an exchange takes 0.9 us, and more beyond.
//
// Workgroup w owns `per` rows of every hidden layer's matrix and the columns of the last layer's that its units of layer L-1 feed.
// Per step: the hidden layers' activations in turn (own rows times all of a_{l-1}; published and gathered unless P = 1), the
// outputs' net inputs (partial sums over own units), loss and Delta_L (every wave for itself), then backward: one pass over the
// own slice multiplies it with delta_l and updates it; what it gives to the units of layer l-1 is published and each
// workgroup adds up its own units' P numbers.  2L - 3 exchanges a step.  Words {value, step number}, two copies by step parity, as
// in dn_online.hip.
//
// A word is written again two steps later, and by then everyone has read it: every workgroup of the P has units of some hidden layer,
// so each step it publishes either activations that all workgroups wait for (layers 1 to L-2) or a share of the outputs' net inputs
// that all wait for (layer L-1), and does so after it has read all it needs of the step before.  So nobody gets two steps ahead of
// anybody.  (A workgroup without units would publish nothing, be waited for by nobody and find its words overwritten: geometry_of
// counts none, and what a launch has beyond the P ends at once.)
//
// What bounds it: the chain of phases, each 0.5 to 1 us for its reads of LDS (80 to 150 cycles each, so several rows and pieces of
// a row are in flight together) and some hundred instructions of one wave, and the exchanges.  us a step, the kernels above / this one:
// 37-116-21-61 21.5 / 6.8, 96-64-160-440-37 26 / 16 (three workgroups), 192-68-7 with momentum 8.6 / 4.6, 1000-1000-33 with momentum
// 19.0 / 7.2 (63).  Four waves instead of eight: 8.2 for the first net; sums over the parts of a column without reads in flight
// together: 1 us more.  Where two copies of the inner weights fit (dn_twin.hip) and one workgroup does not, that kernel stays:
// 1024-1024-1024-1024-10 12.7 there, 19.7 here.
#include "dn_persist.h"

namespace dn {
namespace {

// Sum over the wave, in every lane.
__device__ __forceinline__ float whole_wave_sum(float v) { return add_rows(row16_sum(v)); }

// LANES (sixteen or sixty-four) a row, RU rows and CU pieces of a row in flight together (a phase is a few such rounds, and a round
// takes as long as its slowest read of LDS): fin(row, sum) on one lane per row.  Rows of `pitch` floats (a multiple of four, padding
// zero, as is x's).  zero: four zeros, which pieces beyond a row's end take in place of numbers of both (an infinity times zero is none).
template <int LANES, int RU, int CU, class Fin>
__device__ __forceinline__ void rows_times_n(const float *W, int rows, int pitch, const float *x, const float *zero, Fin fin)
{
    constexpr int kAtOnce = kThreads / LANES;   // rows side by side
    const int lane = threadIdx.x & (LANES - 1), first = threadIdx.x / LANES;
    for (int r0 = 0; r0 < rows; r0 += kAtOnce * RU) {
        v4f s[RU];
        const float *w[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            s[u] = (v4f){0.f, 0.f, 0.f, 0.f};
            w[u] = W + min(r0 + first + u * kAtOnce, rows - 1) * pitch;
        }
        for (int c0 = 0; c0 < pitch; c0 += 4 * LANES * CU) {
            v4f xv[CU], a[RU][CU];
#pragma unroll
            for (int k = 0; k < CU; ++k) {
                const int c = c0 + 4 * (lane + LANES * k);
                const bool in = c < pitch;
                xv[k] = *(const v4f *)(in ? x + c : zero);
#pragma unroll
                for (int u = 0; u < RU; ++u) a[u][k] = *(const v4f *)(in ? w[u] + c : zero);
            }
#pragma unroll
            for (int k = 0; k < CU; ++k)
#pragma unroll
                for (int u = 0; u < RU; ++u) s[u] += a[u][k] * xv[k];
        }
        float v = 0.f;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const float t = (s[u].x + s[u].y) + (s[u].z + s[u].w);
            const float sum = LANES == 16 ? row16_sum(t) : whole_wave_sum(t);
            v = lane == u ? sum : v;
        }
        const int r = r0 + first + lane * kAtOnce;
        if (lane < RU && r < rows) fin(r, v);
    }
}
template <class Fin>
__device__ __forceinline__ void rows_times(const float *W, int rows, int pitch, const float *x, const float *zero, Fin fin)
{
    if (rows > 64) rows_times_n<16, 4, 2>(W, rows, pitch, x, zero, fin);
    else if (rows > 16) rows_times_n<16, 2, 4>(W, rows, pitch, x, zero, fin);
    else if (pitch > 128) rows_times_n<64, 2, 4>(W, rows, pitch, x, zero, fin);
    else rows_times_n<16, 1, 2>(W, rows, pitch, x, zero, fin);
}

// One pass over a slice: W[r][c] -= (lr d[r]) a[c] by the rule of MOM, and with SUM s[c] = sum over the rows of d[r] W[r][c] from the
// weights before: red holds `subs` parts of it afterwards, part k at red + k * 4 * groups (a barrier must follow).  Four rows in
// flight together.  Padding, columns `cols` to pitch - 1, stays zero beside infinities too.
template <bool MOM, bool SUM>
__device__ __forceinline__ void rank_one(float *W, float *V, int rows, int cols, int pitch, const float *d, const float *a, float lr, float mu,
                                         float *red, int shift, int subs)
{
    constexpr int RU = 4;
    const int g = threadIdx.x & ((1 << shift) - 1), sub = threadIdx.x >> shift;   // four columns, every subs-th row
    if (sub >= subs) return;
    v4f s = {0.f, 0.f, 0.f, 0.f};
    if (4 * g < pitch) {
        const int c = 4 * g;
        const v4f av = *(const v4f *)(a + c);
        float no_number = 0.f;   // NaN once a delta is not finite
        for (int r0 = sub; r0 < rows; r0 += RU * subs) {
            float *w[RU];
            v4f wv[RU], vv[RU];
            float dv[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const int r = min(r0 + u * subs, rows - 1);
                w[u] = W + r * pitch + c;
                wv[u] = *(v4f *)w[u];
                if (MOM) vv[u] = *(v4f *)(V + r * pitch + c);
                dv[u] = d[r];
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const bool on = r0 + u * subs < rows;
                const float gv = lr * dv[u];
                no_number = fmaf(gv, 0.f, no_number);
                if (SUM)
#pragma unroll
                    for (int k = 0; k < 4; ++k) s[k] = on ? fmaf(dv[u], wv[u][k], s[k]) : s[k];
                if (MOM) {
                    const v4f v = mu * vv[u] - gv * av;
                    if (on) {
                        *(v4f *)(V + (r0 + u * subs) * pitch + c) = v;
                        *(v4f *)w[u] = wv[u] + v;
                    }
                } else if (on) {
                    *(v4f *)w[u] = wv[u] - gv * av;
                }
            }
        }
        if (no_number != 0.f && c + 4 > cols)
            for (int r = sub; r < rows; r += subs)
                for (int k = max(c, cols); k < c + 4; ++k) {
                    W[r * pitch + k] = 0.f;
                    if (MOM) V[r * pitch + k] = 0.f;
                }
    }
    if (SUM) *(v4f *)(red + (sub << shift) * 4 + 4 * g) = s;
}

// The parts that rank_one left, added up for column c (at most eight).
__device__ __forceinline__ float parts_of(const float *red, int part, int subs, int c)
{
    float v[8], s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = red[min(k, subs - 1) * part + c];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += k < subs ? v[k] : 0.f;
    return s;
}

template <int L, bool MOM>
__global__ __launch_bounds__(SLICE_THREADS) void slice_epoch_kernel(SlicePlan p)
{
    static_assert(kThreads == SLICE_THREADS, "eight waves");
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_abort;
    if (blockIdx.x % p.spread != 0) return;   // (the others are one XCD's, by the usual round-robin placement)
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, w = p.spread > 1 ? (int)blockIdx.x / p.spread : owner_index(), P = p.P;
    if (w >= P) return;
    const int nL = p.layer[L].n_out, n0 = p.layer[1].n_in;
    const float *const zero = lds + p.lds_zero;
    float *const red = lds + p.lds_red, *const z = lds + p.lds_z, *const dL = lds + p.lds_dL, *const bL = lds + p.lds_bL;
    int row0[L + 1], nr[L + 1];   // own units of the hidden layers
#pragma unroll
    for (int l = 1; l < L; ++l) {
        row0[l] = w * p.layer[l].per;
        nr[l] = max(0, min(p.layer[l].per, p.layer[l].n_out - row0[l]));
    }
    if (tid == 0) s_abort = 0;
    for (int e = tid; e < p.lds_floats; e += kThreads) lds[e] = 0.f;
    __syncthreads();
#pragma unroll
    for (int l = 1; l <= L; ++l) {
        const SliceLayer &y = p.layer[l];
        const int rows = l < L ? nr[l] : nL, cols = l < L ? y.n_in : nr[L - 1];
        const size_t at = l < L ? (size_t)row0[l] * y.n_in : (size_t)row0[L - 1];
        for (int r = wave; r < rows; r += kWaves)
            for (int c = lane; c < cols; c += 64) {
                lds[y.lds_w + r * y.pitch + c] = y.W[at + (size_t)r * y.n_in + c];
                if (MOM) lds[y.lds_v + r * y.pitch + c] = y.VW[at + (size_t)r * y.n_in + c];
            }
        if (l < L)
            for (int r = tid; r < rows; r += kThreads) {
                lds[y.lds_b + r] = y.b[row0[l] + r];
                lds[y.lds_b + y.per + r] = y.Vb[row0[l] + r];
            }
    }
    for (int k = tid; k < nL; k += kThreads) {
        bL[k] = p.layer[L].b[k];
        bL[ON_MAX_NL + k] = p.layer[L].Vb[k];
    }
    for (int c = tid; c < n0; c += kThreads) lds[p.lds_x + c] = p.X[c];
    double loss = 0.0;
    __syncthreads();

    // velocity and weight of a bias
    auto bias_step = [&](float *b, float *v, float g) {
        if (MOM) {
            *v = p.mu * *v - g;
            *b += *v;
        } else {
            *v = -g;
            *b -= g;
        }
    };
    constexpr int NX = SLICE_MAX_IN / kThreads;
    int next_label = p.labels[tid >> 9];   // (a vector load: a scalar one would be waited for by the next read of LDS)
    for (int64_t step = 0; step < p.n_samples; ++step) {
        const uint32_t seq = p.seq0 + 1u + (uint32_t)step;
        const int par = (int)(seq & 1u), buf = (int)(step & 1);
        const float *x = lds + p.lds_x + buf * p.x_pitch;
        int lab = __builtin_amdgcn_readfirstlane(next_label);
        lab = lab < 0 ? 0 : lab >= nL ? nL - 1 : lab;

        // ---- hidden layers ----
        float next[NX];   // the next sample's features, on their way
#pragma unroll
        for (int l = 1; l < L; ++l) {
            const SliceLayer &y = p.layer[l];
            const float *in = l == 1 ? x : lds + p.layer[l - 1].lds_a;
            float *out = lds + y.lds_a + (l < L - 1 ? row0[l] : 0);   // (of the last one only the own units are kept)
            const float *b = lds + y.lds_b;
            u64 *ax = p.ex + y.act_x + (size_t)par * y.n_out + row0[l];
            const bool publish = l < L - 1 && P > 1;
            rows_times(lds + y.lds_w, nr[l], y.pitch, in, zero, [&](int r, float s) {
                const float a = act_fn(y.act, s + b[r]);
                out[r] = a;
                if (publish) ll_store(ax + r, a, seq);
            });
            if (l == 1 && step + 1 < p.n_samples) next_label = p.labels[step + 1 + (tid >> 9)];
            if (l == 1 && step + 1 < p.n_samples)
#pragma unroll
                for (int u = 0; u < NX; ++u) next[u] = tid + u * kThreads < n0 ? p.X[(size_t)(step + 1) * n0 + tid + u * kThreads] : 0.f;
            if (publish) {
                float *a = lds + y.lds_a;
                const u64 *src = p.ex + y.act_x + (size_t)par * y.n_out;
                poll_words(y.n_out, seq, [&](int q) { return src + q; }, [&](int q, float v) { a[q] = v; }, p.abort_flag, &s_abort);
            }
            __syncthreads();
            if (publish && s_abort) break;
        }
        if (P > 1 && s_abort) break;

        // ---- net inputs of the outputs, loss, Delta_L ----
        {
            const SliceLayer &y = p.layer[L];
            u64 *zx = p.ex + p.z_x + ((size_t)par * P + w) * nL;
            rows_times(lds + y.lds_w, nL, y.pitch, lds + p.layer[L - 1].lds_a, zero, [&](int r, float s) {
                if (P == 1) z[r] = s + bL[r];
                else if (nr[L - 1] > 0) ll_store(zx + r, s, seq);
            });
            if (P > 1) {
                const u64 *src = p.ex + p.z_x + (size_t)par * P * nL;
                const int parts = p.layer[L - 1].P;
                for (int o0 = 0; o0 < nL; o0 += kThreads / 16) {
                    const int o = o0 + (tid >> 4);
                    float s = 0.f;
                    for (int q0 = tid & 15; q0 < parts && o < nL; q0 += 64) {
                        u64 v[4];
                        int spins = 0;
                        for (;;) {
                            bool ok = true;
#pragma unroll
                            for (int u = 0; u < 4; ++u) v[u] = ll_load(src + (size_t)min(q0 + 16 * u, parts - 1) * nL + o);
#pragma unroll
                            for (int u = 0; u < 4; ++u) ok = ok && (uint32_t)(v[u] >> 32) == seq;
                            if (ok) break;
                            if (give_up(++spins, p.abort_flag, &s_abort)) break;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) s += q0 + 16 * u < parts ? __uint_as_float((uint32_t)v[u]) : 0.f;
                    }
                    s = row16_sum(s);
                    if ((tid & 15) == 0 && o < nL) z[o] = s + bL[o];
                }
            }
            __syncthreads();
            if (P > 1 && s_abort) break;
            const float z0 = lane < nL ? z[lane] : -INFINITY, z1 = lane + 64 < nL ? z[lane + 64] : -INFINITY;
            float d0, d1, e;
            if (p.loss == DN_LOSS_CROSS_ENTROPY) {
                const float top = wave_max(fmaxf(z0, z1));
                const float e0 = lane < nL ? expf(z0 - top) : 0.f, e1 = lane + 64 < nL ? expf(z1 - top) : 0.f;
                const float sum = wave_sum(e0 + e1), inv = 1.0f / sum;
                d0 = e0 * inv - (lane == lab ? 1.0f : 0.0f);
                d1 = e1 * inv - (lane + 64 == lab ? 1.0f : 0.0f);
                e = w == 0 && wave == 0 ? logf(sum) - (z[lab] - top) : 0.f;
            } else {
                const float a0 = act_fn(y.act, z0), a1 = act_fn(y.act, z1);
                const float f0 = a0 - (lane == lab ? 1.0f : 0.0f), f1 = a1 - (lane + 64 == lab ? 1.0f : 0.0f);
                d0 = f0 * act_deriv(y.act, a0);
                d1 = f1 * act_deriv(y.act, a1);
                e = w == 0 && wave == 0 ? wave_sum((lane < nL ? 0.5f * f0 * f0 : 0.f) + (lane + 64 < nL ? 0.5f * f1 * f1 : 0.f)) : 0.f;
            }
            // (every wave writes the same numbers and reads what it wrote)
            if (lane < nL) dL[lane] = d0;
            if (lane + 64 < nL) dL[lane + 64] = d1;
            loss += (double)e;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

            // ---- backward through the last layer ----
            rank_one<MOM, true>(lds + y.lds_w, lds + y.lds_v, nL, nr[L - 1], y.pitch, dL, lds + p.layer[L - 1].lds_a, p.lr, p.mu, red, y.shift, y.subs);
            __syncthreads();
            const SliceLayer &h = p.layer[L - 1];
            for (int r = tid; r < nr[L - 1]; r += kThreads) {
                const float s = parts_of(red, 4 << y.shift, y.subs, r);
                const float d = s * act_deriv(h.act, lds[h.lds_a + r]);
                lds[h.lds_d + r] = d;
                bias_step(lds + h.lds_b + r, lds + h.lds_b + h.per + r, p.lr * d);
            }
            for (int k = tid - kThreads / 2; k >= 0 && k < nL; k += kThreads) bias_step(bL + k, bL + ON_MAX_NL + k, p.lr * dL[k]);
            __syncthreads();
        }

        // ---- backward through the other layers ----
#pragma unroll
        for (int l = L - 1; l >= 2; --l) {
            const SliceLayer &y = p.layer[l], &h = p.layer[l - 1];
            const float *a = lds + h.lds_a;
            rank_one<MOM, true>(lds + y.lds_w, lds + y.lds_v, nr[l], y.n_in, y.pitch, lds + y.lds_d, a, p.lr, p.mu, red, y.shift, y.subs);
            __syncthreads();
            u64 *px = p.ex + y.part_x + ((size_t)par * P + w) * y.n_in;
            for (int c = tid; c < y.n_in; c += kThreads) {
                const float s = parts_of(red, 4 << y.shift, y.subs, c);
                if (P == 1) {
                    const float d = s * act_deriv(h.act, a[c]);
                    lds[h.lds_d + c] = d;
                    bias_step(lds + h.lds_b + c, lds + h.lds_b + h.per + c, p.lr * d);
                } else if (nr[l] > 0) {
                    ll_store(px + c, s, seq);
                }
            }
            if (P > 1) {
                // own units' numbers from every workgroup with rows of this layer
                const int width = 1 << h.fold, r = tid & (width - 1), parts = y.P, every = kThreads >> h.fold;
                const u64 *src = p.ex + y.part_x + (size_t)par * P * y.n_in + row0[l - 1] + min(r, max(nr[l - 1] - 1, 0));
                float s = 0.f;
                if (nr[l - 1] > 0)
                    for (int q0 = tid >> h.fold; q0 < parts; q0 += 4 * every) {
                        u64 v[4];
                        int spins = 0;
                        for (;;) {
                            bool ok = true;
#pragma unroll
                            for (int u = 0; u < 4; ++u) v[u] = ll_load(src + (size_t)min(q0 + u * every, parts - 1) * y.n_in);
#pragma unroll
                            for (int u = 0; u < 4; ++u) ok = ok && (uint32_t)(v[u] >> 32) == seq;
                            if (ok) break;
                            if (give_up(++spins, p.abort_flag, &s_abort)) break;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) s += q0 + u * every < parts ? __uint_as_float((uint32_t)v[u]) : 0.f;
                    }
                for (int o = width; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
                __syncthreads();   // (red has been read)
                const int kept = width < 64 ? kWaves : every;   // parts left
                if (width >= 64 || lane < width) red[(width < 64 ? wave << h.fold : (tid >> h.fold) << h.fold) + r] = s;
                __syncthreads();
                if (s_abort) break;
                for (int c = tid; c < nr[l - 1]; c += kThreads) {
                    const float t = parts_of(red, 1 << h.fold, kept, c);
                    const float d = t * act_deriv(h.act, a[row0[l - 1] + c]);
                    lds[h.lds_d + c] = d;
                    bias_step(lds + h.lds_b + c, lds + h.lds_b + h.per + c, p.lr * d);
                }
            }
            __syncthreads();
        }
        if (P > 1 && s_abort) break;

        // ---- layer 1 ----
        rank_one<MOM, false>(lds + p.layer[1].lds_w, lds + p.layer[1].lds_v, nr[1], n0, p.layer[1].pitch, lds + p.layer[1].lds_d, x, p.lr, p.mu, red,
                             p.layer[1].shift, p.layer[1].subs);
        if (step + 1 < p.n_samples) {
            float *xn = lds + p.lds_x + (buf ^ 1) * p.x_pitch;
#pragma unroll
            for (int u = 0; u < NX; ++u)
                if (tid + u * kThreads < n0) xn[tid + u * kThreads] = next[u];
        }
        __syncthreads();
    }
    __syncthreads();
    if (P > 1 && s_abort) return;

    // ---- slices back; without momentum the velocities are the last step's change ----
    const float *x = lds + p.lds_x + (int)((p.n_samples - 1) & 1) * p.x_pitch;
#pragma unroll
    for (int l = 1; l <= L; ++l) {
        const SliceLayer &y = p.layer[l];
        const int rows = l < L ? nr[l] : nL, cols = l < L ? y.n_in : nr[L - 1];
        const size_t at = l < L ? (size_t)row0[l] * y.n_in : (size_t)row0[L - 1];
        const float *d = l < L ? lds + y.lds_d : dL, *a = l == 1 ? x : lds + p.layer[l - 1].lds_a;
        for (int r = wave; r < rows; r += kWaves)
            for (int c = lane; c < cols; c += 64) {
                y.W[at + (size_t)r * y.n_in + c] = lds[y.lds_w + r * y.pitch + c];
                if (MOM) y.VW[at + (size_t)r * y.n_in + c] = lds[y.lds_v + r * y.pitch + c];
                else if (p.keep_v) y.VW[at + (size_t)r * y.n_in + c] = -(p.lr * d[r] * a[c]);
            }
        if (l < L)
            for (int r = tid; r < rows; r += kThreads) {
                y.b[row0[l] + r] = lds[y.lds_b + r];
                if (MOM || p.keep_v) y.Vb[row0[l] + r] = lds[y.lds_b + y.per + r];
            }
    }
    if (w == 0) {
        for (int k = tid; k < nL; k += kThreads) {
            p.layer[L].b[k] = bL[k];
            if (MOM || p.keep_v) p.layer[L].Vb[k] = bL[ON_MAX_NL + k];
        }
        if (tid == 0) *p.loss_acc += loss;
    }
}

int log2_up(int n)
{
    int s = 0;
    while ((1 << s) < n) ++s;
    return s;
}

bool geometry_of(const int32_t *n, int L, bool momentum, int P, SliceGeom &g)
{
    g = SliceGeom{};
    g.P = 1;   // workgroups with units (1000 units on 64 are 16 each for 63 of them)
    auto four = [](int k) { return (k + 3) & ~3; };
    int at = 0;
    auto take = [&](int k) { const int here = at; at += four(k); return here; };
    g.x_pitch = four(n[0]);
    g.lds_x = take(2 * g.x_pitch);
    for (int l = 1; l < L; ++l) {
        g.per[l] = (n[l] + P - 1) / P;
        g.owners[l] = (n[l] + g.per[l] - 1) / g.per[l];
        if (g.owners[l] > g.P) g.P = g.owners[l];
        g.lds_a[l] = take(l < L - 1 ? n[l] : g.per[l]);
        g.lds_d[l] = take(g.per[l]);
        g.lds_b[l] = take(2 * g.per[l]);
        g.fold[l] = log2_up(g.per[l]);
    }
    g.lds_z = take(ON_MAX_NL);
    g.lds_dL = take(ON_MAX_NL);
    g.lds_bL = take(2 * ON_MAX_NL);
    g.lds_red = take(4 * SLICE_THREADS);
    g.lds_zero = take(4);
    for (int l = 1; l <= L; ++l) {
        const int rows = l < L ? g.per[l] : n[L], cols = l < L ? n[l - 1] : g.per[L - 1];
        g.pitch[l] = four(cols);
        const int groups = g.pitch[l] / 4;
        g.shift[l] = log2_up(groups);
        if ((1 << g.shift[l]) > SLICE_THREADS || (l < L && g.per[l] > SLICE_THREADS && g.P > 1)) return false;
        g.subs[l] = SLICE_THREADS >> g.shift[l];
        if (g.subs[l] > 8) g.subs[l] = 8;
        if ((size_t)rows * g.pitch[l] > (size_t)1 << 20) return false;
        g.lds_w[l] = take(rows * g.pitch[l]);
        if (momentum) g.lds_v[l] = take(rows * g.pitch[l]);
        if ((size_t)at * sizeof(float) > SLICE_MAX_LDS_BYTES) return false;
    }
    g.lds_floats = at;
    size_t words = 0;
    if (g.P > 1) {
        for (int l = 1; l < L - 1; ++l) {
            g.act_x[l] = words;
            words += (size_t)2 * n[l];
        }
        for (int l = 2; l < L; ++l) {
            g.part_x[l] = words;
            words += (size_t)2 * g.P * n[l - 1];
        }
        g.z_x = words;
        words += (size_t)2 * g.P * n[L];
    }
    g.words = words;
    return true;
}

template <int L>
hipError_t launch(const SlicePlan &plan, bool momentum, int grid, size_t bytes, hipStream_t stream)
{
    return momentum ? launch_resident(slice_epoch_kernel<L, true>, plan, grid, bytes, stream)
                    : launch_resident(slice_epoch_kernel<L, false>, plan, grid, bytes, stream);
}

}  // namespace

bool slice_geometry(const int32_t *n, int L, bool momentum, int max_wg, SliceGeom &g)
{
    if (L < 2 || L > SLICE_MAX_L || n[L] > ON_MAX_NL || n[0] > SLICE_MAX_IN) return false;
    for (int l = 1; l < L; ++l)
        if (n[l] > SLICE_MAX_IN) return false;
    for (int P : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256})
        if (P <= max_wg && geometry_of(n, L, momentum, P, g)) return true;
    return false;
}

size_t slice_exchange_bytes(const int32_t *n, int L)
{
    size_t most = 0;
    for (int m = 0; m < 2; ++m) {
        SliceGeom g;
        if (slice_geometry(n, L, m != 0, ON_MAX_WG, g) && g.words * sizeof(u64) > most) most = g.words * sizeof(u64);
    }
    return most;
}

hipError_t slice_prepare(int L)
{
    const void *k[2] = {nullptr, nullptr};
    switch (L) {
    case 2: k[0] = (const void *)slice_epoch_kernel<2, false>; k[1] = (const void *)slice_epoch_kernel<2, true>; break;
    case 3: k[0] = (const void *)slice_epoch_kernel<3, false>; k[1] = (const void *)slice_epoch_kernel<3, true>; break;
    case 4: k[0] = (const void *)slice_epoch_kernel<4, false>; k[1] = (const void *)slice_epoch_kernel<4, true>; break;
    default: return hipErrorInvalidValue;
    }
    for (const void *f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLICE_MAX_LDS_BYTES);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_slice_epoch(const SliceGeom &g, SlicePlan plan, int L, bool momentum, int device_cus, hipStream_t stream)
{
    plan.P = g.P;
    plan.lds_x = g.lds_x; plan.x_pitch = g.x_pitch; plan.lds_z = g.lds_z; plan.lds_dL = g.lds_dL; plan.lds_bL = g.lds_bL;
    plan.lds_red = g.lds_red; plan.lds_zero = g.lds_zero; plan.lds_floats = g.lds_floats;
    plan.z_x = g.z_x;
    for (int l = 1; l <= L; ++l) {
        SliceLayer &y = plan.layer[l];
        y.per = g.per[l]; y.P = g.owners[l]; y.pitch = g.pitch[l]; y.shift = g.shift[l]; y.subs = g.subs[l]; y.fold = g.fold[l];
        y.lds_w = g.lds_w[l]; y.lds_v = g.lds_v[l]; y.lds_a = g.lds_a[l]; y.lds_d = g.lds_d[l]; y.lds_b = g.lds_b[l];
        y.act_x = g.act_x[l]; y.part_x = g.part_x[l];
    }
    // Up to 32 workgroups go to one XCD: every eighth one, the others end at once.  More: a multiple of eight, for owner_index.
    plan.spread = g.P > 1 && g.P <= 32 && 8 * g.P <= device_cus ? 8 : 1;
    const size_t bytes = (size_t)g.lds_floats * sizeof(float);
    const int eights = (g.P + 7) / 8 * 8;
    const int grid = plan.spread > 1 ? g.P * plan.spread : g.P > 1 && eights <= device_cus ? eights : g.P;
    switch (L) {
    case 2: return launch<2>(plan, momentum, grid, bytes, stream);
    case 3: return launch<3>(plan, momentum, grid, bytes, stream);
    case 4: return launch<4>(plan, momentum, grid, bytes, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dn
