// Host side of libdn: argument validation, arena layout, the schedule of
// kernel launches for each entry point of include/dn.h, and launch timing.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "dn_internal.h"

using namespace dn;

namespace {

constexpr size_t kAlign = 256;
constexpr int kMaxTimed = 16384;

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Offsets (bytes) of everything the arena holds.
struct Layout {
    std::vector<size_t> W, b;   // per layer, relative to the start of a parameter-shaped region
    size_t region = 0;          // bytes of one parameter-shaped region (params / velocity / gradients)
    std::vector<size_t> A, D;   // activations / deltas of layers 1..L, absolute
    size_t off_params = 0, off_vel = 0, off_grads = 0;
    size_t off_loss_rows = 0, off_hit_rows = 0, off_loss_sums = 0, off_scalars = 0;
    size_t off_online = 0, online_bytes = 0;   // exchange buffers of the persistent batch-1 kernel
    size_t off_gemm_ws = 0, off_gemm_counters = 0;   // partial tiles / arrival counters of k-split contractions
    size_t off_batch = 0, batch_bytes = 0;           // exchange buffers of the persistent minibatch kernel
    size_t off_deep = 0, deep_bytes = 0;             // exchange buffers of the persistent minibatch kernel for deeper nets
    size_t off_tile = 0, tile_bytes = 0;             // exchange buffers of the minibatch kernel whose layers are cut into tiles
    size_t total = 0;
};

bool compute_layout(const int32_t *widths, int32_t n_widths, int32_t max_batch, Layout &lo)
{
    if (!widths || n_widths < 2 || max_batch <= 0) return false;
    const int L = n_widths - 1;
    for (int i = 0; i < n_widths; ++i)
        if (widths[i] <= 0) return false;
    lo.W.assign(L + 1, 0);
    lo.b.assign(L + 1, 0);
    lo.A.assign(L + 1, 0);
    lo.D.assign(L + 1, 0);
    const size_t lim = (size_t)1 << 46;  // refuse absurd sizes before they overflow
    size_t p = 0;
    for (int l = 1; l <= L; ++l) {
        const size_t nw = (size_t)widths[l] * (size_t)widths[l - 1];
        if (nw > lim / 4) return false;
        lo.W[l] = p;
        p += align_up(nw * sizeof(float));
        lo.b[l] = p;
        p += align_up((size_t)widths[l] * sizeof(float));
        if (p > lim) return false;
    }
    lo.region = p;
    size_t o = 0;
    lo.off_params = o; o += lo.region;
    lo.off_vel = o; o += lo.region;
    lo.off_grads = o; o += lo.region;
    for (int l = 1; l <= L; ++l) {
        const size_t na = align_up((size_t)max_batch * (size_t)widths[l] * sizeof(float));
        if (na > lim) return false;
        lo.A[l] = o; o += na;
        lo.D[l] = o; o += na;
        if (o > lim) return false;
    }
    lo.off_loss_rows = o; o += align_up((size_t)max_batch * sizeof(float));
    lo.off_hit_rows = o; o += align_up((size_t)max_batch * sizeof(float));
    lo.off_loss_sums = o; o += align_up((size_t)max_batch * sizeof(double));
    lo.off_scalars = o; o += kAlign;
    lo.online_bytes = std::max({online_exchange_bytes_bound(widths, L), twin_exchange_bytes_bound(widths, L),
                                wide_exchange_bytes_bound(widths, L), block_exchange_bytes(widths, L),
                                wide_block_exchange_bytes(widths, L), slice_exchange_bytes(widths, L)});
    lo.off_online = o; o += align_up(lo.online_bytes);
    lo.off_gemm_ws = o; o += align_up(GEMM_WS_FLOATS * sizeof(float));
    lo.off_gemm_counters = o; o += align_up(GEMM_COUNTERS * sizeof(unsigned));
    lo.batch_bytes = batch_exchange_bytes_bound(widths, L, max_batch);
    lo.off_batch = o; o += align_up(lo.batch_bytes);
    lo.deep_bytes = deep_exchange_bytes_bound(widths, L, max_batch);
    lo.off_deep = o; o += align_up(lo.deep_bytes);
    lo.tile_bytes = max_batch > 1 ? tile_exchange_bytes(widths, L, max_batch) : 0;
    lo.off_tile = o; o += align_up(lo.tile_bytes);
    lo.total = o;
    return true;
}

// Page-locked host memory that the one-wave kernels write a pass's summed loss to, one slot per net: 4 KB, allocated once per
// process; a net gives its slot back when it goes.  A net without a slot (all taken, none to be had) copies the sum from its arena.
class ResultSlots {
public:
    double *take()
    {
        std::lock_guard<std::mutex> lock(m_);
        if (!tried_) {
            tried_ = true;
            void *p = nullptr;
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // (another thread's capture may be under way)
            const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
            if (hipHostMalloc(&p, kSlots * kStride, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) base_ = (char *)p;
            else (void)hipGetLastError();
            if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
        }
        for (int i = 0; base_ && i < kSlots; ++i)
            if (!used_[i]) {
                used_[i] = true;
                return (double *)(base_ + i * kStride);
            }
        return nullptr;
    }
    void give(double *slot)
    {
        if (!slot) return;
        std::lock_guard<std::mutex> lock(m_);
        used_[((char *)slot - base_) / kStride] = false;
    }

private:
    static constexpr int kSlots = 64, kStride = 64;
    std::mutex m_;
    char *base_ = nullptr;
    bool tried_ = false, used_[kSlots] = {};
};
ResultSlots result_slots;

struct TimedLaunch {
    hipEvent_t start, stop;
    int cls;
    double flop;   // algorithmic flops of the launch (2 M N K per product)
};

}  // namespace

struct dn_net {
    int L = 0;
    std::vector<int32_t> n;     // widths n_0..n_L
    std::vector<int32_t> act;   // act[l], l = 1..L (index 0 unused)
    int loss = 0;
    int max_batch = 0;
    char *arena = nullptr;
    Layout lo;
    hipStream_t stream = nullptr;
    // state of the split API
    const float *X = nullptr;
    int fwd_batch = 0;
    bool have_fwd = false, have_bwd = false;
    bool w1_as_in_bwd = false;   // W_1 is still the matrix the last dn_backward propagated through
    // options
    int time_kernels = 0, gemm_variant = -1, online_mode = 0, online_min_tile = ON_DEFAULT_MIN_TILE,
        online_resident = 1, online_twin = 1, online_tiny = 1, online_solo = 1, online_wide = 1, online_blocks = 1, split_k_on = 1, merge_launches = 1;
    // persistent batch-1 kernel
    OnlineGeom geom{};
    bool online_ok = false;
    bool online_prepared = false, batch_prepared = false, deep_prepared = false;   // LDS limits raised at creation
    bool twin_ready = false;   // the two-copy batch-1 kernel's LDS limit is raised
    bool tiny_ready = false;   // the one-wave batch-1 kernel's LDS limit is raised
    bool wide_ready = false;   // the wide-hidden-layer batch-1 kernel's LDS limit is raised
    bool wide_ok = false;      // ... and the net suits it
    bool wide_block_ready = false;   // ... and the sample-block form of the wide-hidden-layer kernel
    bool slice_ready = false;  // the few-workgroup batch-1 kernel's LDS limit is raised
    int online_slices = 1;
    bool block_ready = false;  // the sample-block batch-1 kernel's LDS limit is raised and the net suits it
    int last_schedule = DN_SCHED_NONE;   // how the last dn_train_epoch ran
    double *result = nullptr;   // a slot of result_slots
    uint32_t online_seq = 0;   // last step number stamped into the exchange buffers
    // persistent minibatch kernel (one- and two-layer nets)
    bool batch_ok = false, deep_ok = false;
    int batch_mode = 0;
    uint32_t batch_seq = 0, deep_seq = 0, tile_seq = 0;
    bool tile_ready = false;   // the tiled minibatch kernel's LDS limit is raised
    int batch_tiles = 1;
    bool last_tiles = false;   // it ran the last dn_train_epoch
    int tile_pause = 0, tile_rest = 0;   // passes without it after a launch that was taken back; how many of them are left
    int device_cus = 0;
    // timing
    hipEvent_t ev_epoch0 = nullptr, ev_epoch1 = nullptr;
    std::vector<TimedLaunch> pool;
    int timed = 0;
    float epoch_ms = 0.f;
    double cls_ms[DN_K_CLASSES] = {0};
    double cls_flop[DN_K_CLASSES] = {0};
    int64_t cls_launches[DN_K_CLASSES] = {0};

    float *W(int l) const { return (float *)(arena + lo.off_params + lo.W[l]); }
    float *b(int l) const { return (float *)(arena + lo.off_params + lo.b[l]); }
    float *VW(int l) const { return (float *)(arena + lo.off_vel + lo.W[l]); }
    float *Vb(int l) const { return (float *)(arena + lo.off_vel + lo.b[l]); }
    float *GW(int l) const { return (float *)(arena + lo.off_grads + lo.W[l]); }
    float *Gb(int l) const { return (float *)(arena + lo.off_grads + lo.b[l]); }
    float *A(int l) const { return (float *)(arena + lo.A[l]); }
    float *D(int l) const { return (float *)(arena + lo.D[l]); }
    float *loss_rows() const { return (float *)(arena + lo.off_loss_rows); }
    float *hit_rows() const { return (float *)(arena + lo.off_hit_rows); }
    double *loss_sums() const { return (double *)(arena + lo.off_loss_sums); }
    double *hit_acc() const { return (double *)(arena + lo.off_scalars + 16); }   // after epoch_acc and the abort flag
    double *epoch_acc() const { return (double *)(arena + lo.off_scalars); }
    int *abort_flag() const { return (int *)(arena + lo.off_scalars + sizeof(double)); }
    int *swept() const { return (int *)(arena + lo.off_scalars + 12); }   // see WidePlan
    unsigned *arrived() const { return (unsigned *)(arena + lo.off_scalars + 24); }   // launches of sample blocks: see BlockPlan
    int *settled() const { return (int *)(arena + lo.off_scalars + 28); }
    unsigned long long *exchange() const { return (unsigned long long *)(arena + lo.off_online); }
    unsigned long long *batch_exchange() const { return (unsigned long long *)(arena + lo.off_batch); }
    char *deep_exchange() const { return arena + lo.off_deep; }
    unsigned long long *tile_exchange() const { return (unsigned long long *)(arena + lo.off_tile); }
    void split_k(GemmArgs &g) const
    {
        g.ws = split_k_on ? (float *)(arena + lo.off_gemm_ws) : nullptr;
        g.counters = (unsigned *)(arena + lo.off_gemm_counters);
        g.ws_floats = GEMM_WS_FLOATS;
        g.n_counters = GEMM_COUNTERS;
    }
};

LaunchEvents &dn::launch_events()
{
    static thread_local LaunchEvents ev;
    return ev;
}

namespace {

#define DN_HIP(expr)                                   \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return DN_ERR_DEVICE;    \
    } while (0)

// Which persistent kernels this net fits with the current tile option ("online_min_tile").
void refresh_persistent(dn_net *net)
{
    const int L = net->L;
    net->online_ok = net->batch_ok = net->deep_ok = net->wide_ok = false;
    if (net->device_cus <= 0) return;
    if (net->wide_ready) {
        WideGeom wg;
        net->wide_ok = wide_geometry(net->n.data(), L, net->device_cus, false, wg) &&
                       wg.words * sizeof(unsigned long long) <= net->lo.online_bytes;
    }
    if (net->online_prepared && online_geometry(net->n.data(), L, net->online_min_tile, false, net->geom))
        net->online_ok = net->geom.grid <= net->device_cus;
    if (net->batch_prepared) {
        BatchGeom bg;   // with velocities: the larger of the two LDS layouts
        net->batch_ok = batch_geometry(net->n.data(), L, net->max_batch, net->online_min_tile, true, bg) &&
                        bg.grid <= net->device_cus;
    }
    if (net->deep_prepared) {
        DeepGeom dg;
        net->deep_ok = deep_geometry(net->n.data(), L, net->max_batch, net->online_min_tile, dg) &&
                       dg.grid <= net->device_cus;
    }
}

// Whether dn_forward takes a narrow last layer in one launch (product, softmax or activation, copy to the caller) or as a product and
// what follows it.  A workgroup of the one launch reads all of W_L for one row (four beyond 1024 rows), so it loses where W_L is
// large or the rows are many, and without a softmax there is less to save.  us for a whole dn_forward of 16-n-m, product and the
// rest / one launch -- softmax: 64-16, 1 row 10.0 / 8.0; 4096-3, 64 and 512 rows 16.3 / 10.3, 26.9 / 17.4; 2048-16 (32768 weights),
// 1 and 768 rows 14.3 / 10.7, 21.6 / 18.1; beyond it 4096-16, 1 and 1024 rows 16.1 / 14.7, 33.8 / 40.9, 8192-10, 1 row 17.1 / 18.2,
// 16384-16, 1 row 19.2 / 38.4, 100000-10, 1 and 1024 rows 45.7 / 289, 389 / 983; 1025 to 2048 rows: 1024-10 22.3 / 20.0, 2048-6 34.1 /
// 28.6, 512-10 16.1 / 15.3, but 256-16 12.7 / 14.4, 2048-16 1025 rows 24.5 / 24.2, 4096-10 44.6 / 47.3; 4096 rows: 256-10 15.4 /
// 22.8, 1024-10 31.8 / 35.6.  Squared error, where the product's launch may be all there is (no copy asked for): 1024-10, 1 and 768
// rows 10.2 / 8.1, 13.6 / 11.4; 4096-3, 1 row 14.1 / 9.4; 256-10, 1 and 512 rows 8.5 / 8.0, 9.0 / 9.0 (and with the copy 300-10, 64 rows
// 13.2 / 10.0); but 64-16, 1 row 6.9 / 8.8, 256-16, 768 rows 9.0 / 10.5, 1536-16, 768 rows 16.6 / 17.1, 1024-16, 1025 rows 14.9 / 18.5.
bool one_launch_forward(const dn_net *net, int rows)
{
    const int n_out = net->n[net->L], n_in = net->n[net->L - 1];
    if (net->gemm_variant >= 0 || !narrow_layer(n_out)) return false;
    const size_t weights = (size_t)n_out * n_in;
    if (net->loss != DN_LOSS_CROSS_ENTROPY)
        return weights <= 16384 && rows <= (n_in >= 1024 ? 768 : n_in >= (n_out <= 10 ? 256 : 512) ? 512 : 0);
    return rows <= 768 ? weights <= 32768 : rows <= 2048 && n_in >= 512 && weights <= 16384;
}

double product_flop(const GemmArgs &g) { return 2.0 * (double)g.M * (double)g.N * (double)g.K; }

bool rate_ok(float lr, float mu)
{
    return std::isfinite(lr) && std::isfinite(mu) && lr >= 0.f && mu >= 0.f && mu < 1.f;
}

// Times one launch when per-launch timing is on.  bind: the scope holds exactly one kernel launch
// made through launch_kernel, which takes the event pair along (the kernel's own start and end);
// otherwise the events are recorded around whatever the scope enqueues.
struct ScopedTimer {
    dn_net *net;
    TimedLaunch *t = nullptr;
    bool bind;
    ScopedTimer(dn_net *n, int cls, bool enabled, double flop = 0.0, bool bind_to_launch = false) : net(n), bind(bind_to_launch)
    {
        if (!enabled || net->timed >= kMaxTimed) return;
        if ((int)net->pool.size() <= net->timed) {
            TimedLaunch tl{};
            if (hipEventCreate(&tl.start) != hipSuccess) return;
            if (hipEventCreate(&tl.stop) != hipSuccess) {
                (void)hipEventDestroy(tl.start);
                return;
            }
            net->pool.push_back(tl);
        }
        t = &net->pool[net->timed++];
        t->cls = cls;
        t->flop = flop;
        if (bind) {
            LaunchEvents &ev = launch_events();
            ev.start = t->start;
            ev.stop = t->stop;
            ev.bound = false;
        } else {
            (void)hipEventRecord(t->start, net->stream);
        }
    }
    ~ScopedTimer()
    {
        if (!t) return;
        if (bind) {
            LaunchEvents &ev = launch_events();
            if (!ev.bound) --net->timed;   // nothing was launched (an error on the way): the pair stays unused
            ev = LaunchEvents{};
        } else {
            (void)hipEventRecord(t->stop, net->stream);
        }
    }
};

// Forward pass of one batch; leaves A_1..A_L in the arena.  The softmax layer's
// row normalisation is left to the caller (it is fused with the loss in training).
dn_status run_forward(dn_net *net, const float *X, int B, bool timing, int last_layer = -1)
{
    if (last_layer < 0) last_layer = net->L;
    for (int l = 1; l <= last_layer; ++l) {
        GemmArgs g{};
        g.A = (l == 1) ? X : net->A(l - 1);
        g.lda = net->n[l - 1];
        g.B = net->W(l);
        g.ldb = net->n[l - 1];
        g.M = B; g.N = net->n[l]; g.K = net->n[l - 1];
        g.C = net->A(l); g.ldc = net->n[l];
        g.bias = net->b(l);
        g.act = net->act[l];
        net->split_k(g);
        ScopedTimer st(net, DN_K_FORWARD, timing, product_flop(g), true);
        DN_HIP(launch_gemm(GEMM_FWD, g, net->gemm_variant, net->stream));
    }
    return DN_OK;
}

// Back propagation of one batch from Delta_L.  mode GRAD_STORE leaves gradients in the gradient
// region; the other modes update parameters in place.  With T_l the delta product through W_l
// (giving Delta_{l-1}) and G_l the gradient / update of layer l, the order is
//     T_L, T_{L-1}, ..., T_2 (each needs the one before), then G_L .. G_1:
// every T_l has read W_l before any G writes it, and once all deltas exist the G_l are independent
// of one another, so those whose shapes allow share ONE launch (launch_gemm_grads).  A narrow last
// layer's G_L rides with T_{L-1} instead (launch_delta_with_narrow_grad): its vector-unit work fits
// beside the few tiles of a delta product.  merge_launches = 0: one launch per product.
// have_top_delta: Delta_{L-1} came with the output error already (narrow last layer).
dn_status run_backward(dn_net *net, const float *X, int B, int mode, float lr, float mu, bool timing,
                       bool have_top_delta = false)
{
    const float scale = (mode == GRAD_STORE) ? 1.0f / (float)B : lr / (float)B;
    const int L = net->L;
    const bool merge = net->merge_launches != 0;
    auto delta_args = [&](int l) {   // T_l, l >= 2
        GemmArgs g{};
        g.A = net->D(l); g.lda = net->n[l];
        g.B = net->W(l); g.ldb = net->n[l - 1];
        g.M = B; g.N = net->n[l - 1]; g.K = net->n[l];
        g.C = net->D(l - 1); g.ldc = net->n[l - 1];
        g.aux = net->A(l - 1);
        g.act = net->act[l - 1];
        net->split_k(g);
        return g;
    };
    auto grad_args = [&](int l) {    // G_l
        GemmArgs g{};
        g.A = net->D(l); g.lda = net->n[l];
        g.B = (l == 1) ? X : net->A(l - 1); g.ldb = net->n[l - 1];
        g.M = net->n[l]; g.N = net->n[l - 1]; g.K = B;
        g.C = (mode == GRAD_STORE) ? net->GW(l) : net->W(l);
        g.ldc = net->n[l - 1];
        g.V = net->VW(l);
        g.gb = (mode == GRAD_STORE) ? net->Gb(l) : net->b(l);   // bias gradient / update rides along
        g.vb = net->Vb(l);
        g.scale = scale; g.mu = mu; g.mode = mode;
        return g;
    };
    if (L > ON_MAX_L + 56) return DN_ERR_UNSUPPORTED;
    int top_grad = L;                // gradients L .. 1 are still to do
    for (int l = L; l >= 2; --l) {
        if (l == L && have_top_delta) continue;
        const GemmArgs d = delta_args(l);
        if (merge && l == L - 1 && top_grad == L) {
            const GemmArgs gl = grad_args(L);
            if (delta_narrow_grad_fits(d, gl, net->gemm_variant)) {
                ScopedTimer st(net, DN_K_DELTA, timing, product_flop(d) + product_flop(gl), true);
                DN_HIP(launch_delta_with_narrow_grad(d, gl, net->stream));
                top_grad = L - 1;
                continue;
            }
        }
        ScopedTimer st(net, DN_K_DELTA, timing, product_flop(d), true);
        DN_HIP(launch_gemm(GEMM_DELTA, d, net->gemm_variant, net->stream));
    }
    GemmArgs grads[ON_MAX_L + 56];
    int n = 0;
    for (int l = top_grad; l >= 1; --l) grads[n++] = grad_args(l);
    if (!timing) {
        DN_HIP(launch_gemm_grads(grads, n, net->gemm_variant, merge, net->stream, nullptr));
        return DN_OK;
    }
    // timed: the shared launch (if any) and every single launch get an event pair of their own
    int merged = 0;
    {
        // a dry run tells which products share the launch: they are timed together, the others one by one
        bool in_shared[ON_MAX_L + 56];
        gemm_grads_plan(grads, n, net->gemm_variant, merge, in_shared, &merged);
        if (merged >= 2) {
            GemmArgs shared[ON_MAX_L + 56];
            int ns = 0;
            double fs = 0.0;
            for (int i = 0; i < n; ++i)
                if (in_shared[i]) { shared[ns++] = grads[i]; fs += product_flop(grads[i]); }
            ScopedTimer st(net, DN_K_GRAD_UPDATE, timing, fs, true);
            DN_HIP(launch_gemm_grads(shared, ns, net->gemm_variant, true, net->stream, nullptr));
        }
        for (int i = 0; i < n; ++i) {
            if (merged >= 2 && in_shared[i]) continue;
            ScopedTimer st(net, DN_K_GRAD_UPDATE, timing, product_flop(grads[i]), true);
            DN_HIP(launch_gemm(GEMM_GRAD, grads[i], net->gemm_variant, net->stream));
        }
    }
    return DN_OK;
}

// One wavefront can run a batch-1 pass of this net: every layer at most 64 wide.
bool one_wave(dn_net *net, float mu, TinyPlan &p)
{
    return net->online_tiny && net->tiny_ready && tiny_plan(net->n.data(), net->L, mu != 0.f, p);
}

// A whole batch-1 epoch of a very small net on one wavefront.
dn_status run_tiny(dn_net *net, TinyPlan &p, const float *X, const int32_t *labels, int64_t n_samples, float lr, float mu,
                   bool timing)
{
    for (int l = 1; l <= net->L; ++l) {
        TinyLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.act = net->act[l];
    }
    p.loss_acc = net->result ? net->result : net->epoch_acc();
    p.X = X; p.labels = labels; p.n_samples = n_samples;
    p.lr = lr; p.mu = mu; p.loss = net->loss; p.keep_v = 1;
    p.in_registers = (net->online_tiny == 1 && net->L == 2 && mu == 0.f) ? 1 : 0;
    net->last_schedule = p.in_registers ? DN_SCHED_ONE_WAVE_REGISTERS : DN_SCHED_ONE_WAVE;
    ScopedTimer st(net, DN_K_ONLINE, timing);
    DN_HIP(launch_tiny_epoch(p, net->stream));
    return DN_OK;
}

// A whole batch-1 epoch of plain gradient descent with the two-copy kernel (same exchange region
// and step numbering as run_online, so either may follow the other).
dn_status run_twin(dn_net *net, const TwinGeom &g, const float *X, const int32_t *labels, int64_t n_samples, float lr,
                   bool timing)
{
    const int L = net->L;
    TwinPlan p{};
    p.L = L;
    for (int l = 1; l <= L; ++l) {
        TwinLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.n_in = net->n[l - 1]; y.n_out = net->n[l]; y.act = net->act[l];
        y.per = g.per[l]; y.P = g.P[l];
        y.r_kshift = g.r_kshift[l]; y.r_seg = g.r_seg[l]; y.c_kshift = g.c_kshift[l]; y.c_seg = g.c_seg[l];
        const int stride = ON_THREADS * 4;
        y.inv_in = 1.0f / (float)y.n_in; y.r_rs = stride / y.n_in; y.r_ks = stride % y.n_in;
        y.inv_out = 1.0f / (float)y.n_out; y.c_rs = stride / y.n_out; y.c_ks = stride % y.n_out;
        p.act_x[l] = net->exchange() + g.off_act[l];
        p.dl_x[l] = net->exchange() + g.off_dl[l];
        p.lds_a[l] = g.lds_a[l]; p.lds_own_a[l] = g.lds_own_a[l]; p.lds_own_d[l] = g.lds_own_d[l];
        p.lds_b[l] = g.lds_b[l]; p.lds_r[l] = g.lds_r[l]; p.lds_c[l] = g.lds_c[l];
    }
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.lr = lr; p.loss = net->loss;
    p.lds_x = g.lds_x; p.lds_d = g.lds_d; p.lds_wL = g.lds_wL; p.lds_out = g.lds_out; p.lds_kpart = g.lds_kpart;
    const int64_t chunk = (int64_t)1 << 30;
    for (int64_t s0 = 0; s0 < n_samples; s0 += chunk) {
        const int64_t n = (n_samples - s0) < chunk ? (n_samples - s0) : chunk;
        if ((uint64_t)net->online_seq + (uint64_t)n + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->exchange(), 0, net->lo.online_bytes, net->stream));
            net->online_seq = 0;
        }
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (s0 + n >= n_samples) ? 1 : 0;
        p.seq0 = net->online_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_twin_epoch(g, p, net->stream));
        net->online_seq += (uint32_t)n;
    }
    return DN_OK;
}

// Samples of a pass for them to be taken in blocks.  us a pass of 64, the kernels before / blocks: 65-4-2 146 / 74; 784-4-2 212 / 87;
// 64-128-10 141 / 89; 784-128-10 378 / 104; 256-256-10 308 / 108; 340-200-40 389 / 153; 1024-512-64 484 / 230; 5-999-2 1649 / 165;
// 1024-1004-16 347 / 234; hidden layers beyond LDS 340-38000-3 945 / 355, 340-100000-10 1511 / 550, 64-131072-16 1585 / 430.  (The line is
// where nothing measured lost; it may lie lower.)
constexpr int64_t kBlocksMinSamples = 64;

// Batch-1 epochs of a two-layer net with a wide hidden layer: most of W_1 stays in LDS and registers.
dn_status run_wide(dn_net *net, const WideGeom &g, const float *X, const int32_t *labels, int64_t n_samples, float lr,
                   float mu, bool timing)
{
    WidePlan p{};
    p.W1 = net->W(1); p.b1 = net->b(1); p.VW1 = net->VW(1); p.Vb1 = net->Vb(1);
    p.W2 = net->W(2); p.b2 = net->b(2); p.VW2 = net->VW(2); p.Vb2 = net->Vb(2);
    p.z_x = net->exchange();
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.n0 = net->n[0]; p.n1 = net->n[1]; p.nL = net->n[2];
    p.act1 = net->act[1]; p.actL = net->act[2]; p.loss = net->loss;
    p.per = g.per; p.lds_rows = g.lds_rows;
    p.lr = lr; p.mu = mu;
    p.lds_x = g.lds_x; p.lds_a = g.lds_a; p.lds_d = g.lds_d; p.lds_b = g.lds_b; p.lds_z = g.lds_z; p.lds_w2 = g.lds_w2;
    p.lds_vb = g.lds_vb; p.lds_vw2 = g.lds_vw2;
    p.lds_zall = g.lds_zall; p.lds_out = g.lds_out; p.lds_w1 = g.lds_w1;
    // Without momentum the samples go in blocks, W_1 read and written once per block; the kernel that sweeps it every step is
    // launched behind and ends at once unless a block's inner products left fp32.
    const bool blocks = mu == 0.f && net->online_blocks && net->wide_block_ready && n_samples >= kBlocksMinSamples &&
                        (reinterpret_cast<uintptr_t>(X) & 15) == 0;   // (it reads the samples in sixteen-byte pieces)
    if (blocks) net->last_schedule = DN_SCHED_WIDE_BLOCKS;
    p.swept = net->swept();
    const int64_t chunk = blocks ? BLOCK_LAUNCH_SAMPLES : (int64_t)1 << 30;
    for (int64_t s0 = 0; s0 < n_samples; s0 += chunk) {
        const int64_t n = (n_samples - s0) < chunk ? (n_samples - s0) : chunk;
        if ((uint64_t)net->online_seq + 2 * (uint64_t)n + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->exchange(), 0, net->lo.online_bytes, net->stream));
            net->online_seq = 0;
        }
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (s0 + n >= n_samples) ? 1 : 0;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        if (blocks) {
            BlockPlan b{};
            b.W1 = p.W1; b.b1 = p.b1; b.VW1 = p.VW1; b.Vb1 = p.Vb1; b.W2 = p.W2; b.b2 = p.b2; b.VW2 = p.VW2; b.Vb2 = p.Vb2;
            b.abort_flag = p.abort_flag; b.loss_acc = p.loss_acc;
            b.X = p.X; b.labels = p.labels; b.n_samples = n; b.keep_v = p.keep_v;
            b.n0 = p.n0; b.n1 = p.n1; b.n2 = p.nL; b.act1 = p.act1; b.act2 = p.actL; b.loss = p.loss;
            b.per = g.per; b.lr = lr;
            b.vec = (reinterpret_cast<uintptr_t>(p.X) & 15) == 0;
            b.seq0 = net->online_seq;
            DN_HIP(launch_wide_block_epoch(b, g.grid, net->exchange(), &p.gram, net->stream));
            p.gram_blocks = (int)((n + BLOCK_SAMPLES - 1) / BLOCK_SAMPLES);
            net->online_seq += (uint32_t)n;
        }
        p.seq0 = net->online_seq;
        DN_HIP(launch_wide_epoch(g, p, net->stream));
        net->online_seq += (uint32_t)n;
    }
    return DN_OK;
}

// Batch-1 steps of a two-layer net on one workgroup that keeps W_1 in its registers (plain gradient descent).
dn_status run_solo(dn_net *net, const SoloGeom &g, const float *X, const int32_t *labels, int64_t n_samples, float lr,
                   bool keep_v, bool timing)
{
    SoloPlan p{};
    p.W1 = net->W(1); p.b1 = net->b(1); p.VW1 = net->VW(1); p.Vb1 = net->Vb(1);
    p.W2 = net->W(2); p.b2 = net->b(2); p.VW2 = net->VW(2); p.Vb2 = net->Vb(2);
    p.loss_acc = net->epoch_acc();
    p.n0 = net->n[0]; p.n1 = net->n[1]; p.n2 = net->n[2];
    p.act1 = net->act[1]; p.act2 = net->act[2]; p.loss = net->loss;
    p.lr = lr;
    const int64_t chunk = (int64_t)1 << 30;   // the kernel counts its steps in 32 bits
    for (int64_t s0 = 0; s0 < n_samples; s0 += chunk) {
        const int64_t n = (n_samples - s0) < chunk ? (n_samples - s0) : chunk;
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (keep_v && s0 + n >= n_samples) ? 1 : 0;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_solo_epoch(g, p, net->stream));
    }
    return DN_OK;
}

dn_status run_online_shared(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, float lr, float mu,
                            bool timing);

// Batch-1 steps of a two-layer net with the samples in blocks of 32 (plain gradient descent).
dn_status run_blocks(dn_net *net, const BlockGeom &g, const float *X, const int32_t *labels, int64_t n_samples, float lr,
                     bool timing)
{
    BlockPlan p{};
    p.W1 = net->W(1); p.b1 = net->b(1); p.VW1 = net->VW(1); p.Vb1 = net->Vb(1);
    p.W2 = net->W(2); p.b2 = net->b(2); p.VW2 = net->VW(2); p.Vb2 = net->Vb(2);
    p.n0 = net->n[0]; p.n1 = net->n[1]; p.n2 = net->n[2];
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.act1 = net->act[1]; p.act2 = net->act[2]; p.loss = net->loss;
    p.lr = lr;
    p.arrived = net->arrived();
    p.settled = net->settled();
    for (int64_t s0 = 0; s0 < n_samples; s0 += BLOCK_LAUNCH_SAMPLES, ++p.launch) {
        p.expected = (unsigned)(p.launch + 1) * (unsigned)g.grid;
        if (net->online_blocks >= 2 && p.launch == net->online_blocks - 2) ++p.expected;   // (one more than will come)
        const int64_t n = std::min<int64_t>(n_samples - s0, BLOCK_LAUNCH_SAMPLES);
        if ((uint64_t)net->online_seq + (uint64_t)n + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->exchange(), 0, net->lo.online_bytes, net->stream));
            net->online_seq = 0;
        }
        p.X = X + (size_t)s0 * p.n0;
        p.labels = labels + s0;
        p.vec = p.n0 % 4 == 0 && (reinterpret_cast<uintptr_t>(p.X) & 15) == 0;
        p.n_samples = n;
        p.keep_v = (s0 + n >= n_samples) ? 1 : 0;
        p.seq0 = net->online_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_block_epoch(g, p, net->exchange(), net->stream));
        net->online_seq += (uint32_t)n;
    }
    return DN_OK;
}

// Whether a pass of a two-layer net takes its samples in blocks, on workgroups that the device can hold all at once.  (One wavefront
// goes first.)
bool takes_blocks(const dn_net *net, int64_t n_samples, float mu, BlockGeom &g)
{
    return net->block_ready && net->online_blocks && mu == 0.f && n_samples >= kBlocksMinSamples &&
           block_geometry(net->n.data(), net->L, g) && g.grid <= net->device_cus;
}

// Batch-1 steps of a net on as few workgroups as hold it in LDS.
dn_status run_slices(dn_net *net, const SliceGeom &g, const float *X, const int32_t *labels, int64_t n_samples, float lr, float mu,
                     bool timing)
{
    const int L = net->L;
    SlicePlan p{};
    for (int l = 1; l <= L; ++l) {
        SliceLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.n_in = net->n[l - 1]; y.n_out = net->n[l]; y.act = net->act[l];
    }
    p.ex = net->exchange();
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.lr = lr; p.mu = mu; p.loss = net->loss;
    const int64_t chunk = (int64_t)1 << 30;
    for (int64_t s0 = 0; s0 < n_samples; s0 += chunk) {
        const int64_t n = std::min(n_samples - s0, chunk);
        if ((uint64_t)net->online_seq + (uint64_t)n + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->exchange(), 0, net->lo.online_bytes, net->stream));
            net->online_seq = 0;
        }
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (s0 + n >= n_samples) ? 1 : 0;
        p.seq0 = net->online_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_slice_epoch(g, p, L, mu != 0.f, net->device_cus, net->stream));
        net->online_seq += (uint32_t)n;
    }
    return DN_OK;
}

// Whether n_samples samples take less there than on the kernel that would run them otherwise.  Both take what a step costs and, once,
// what a call costs; a call costs more here the more rows a workgroup has to load (34 us, and 0.035 a row), so short passes stay where they
// were: one sample of 9-16-64-3 30 there / 44 here, of 124-748-476-504-10 67 / 84, of 40-8-1384-4 67 / 117.  Steps are estimated, the other kernel
// on the low side, by what was measured on 450 nets (1 to 192 samples; the estimates fit to 8 % in the mean): a step on the general kernel
// grows with the units of its busiest workgroups and, from three layers on, with the partial sums these add up (3-1322-410-38 with momentum
// 246, 16-832-3 12.9), here with the rows of a workgroup (13 and 16.9).  On nets that the estimates had not seen, 1 to 120 samples: of
// 2611 passes taken five are slower than 0.97 times the other kernel's, the slowest 0.94.
bool slices_pay(const dn_net *net, const SliceGeom &g, int64_t n_samples, bool two_copies)
{
    const int L = net->L;
    const int32_t *n = net->n.data();
    double rows = 0, runs = 0;              // of a workgroup here: rows of the hidden layers, runs of 64 weights in them
    double units = 0, far = 0, partial = 0; // there: units of a workgroup, the same by the 256 inputs, partial sums it adds up
    bool many = false;                      // there: several workgroups
    int owned_below = 0;
    for (int l = 1; l < L; ++l) {
        rows += g.per[l];
        runs += (double)g.per[l] * ((n[l - 1] + 63) / 64);
        const int owned = std::min(n[l], std::max((n[l] + 255) / 256, (4095 + n[l - 1]) / n[l - 1])), owners = (n[l] + owned - 1) / owned;
        units += owned;
        far += (double)owned * ((n[l - 1] + 255) / 256);
        partial += (double)owners * owned_below;
        many = many || owners > 1;
        owned_below = owned;
    }
    const double outputs = n[L], deep = L - 3, spread = g.P > 1;
    double there, here, call;
    if (two_copies) {
        there = 0.88 * (4.3 + 2.9 * deep + (many ? 2.0 : 0.0) + 0.04 * units + 0.036 * outputs);
        here = 4.2 + 1.5 * deep + 0.014 * rows + 0.0086 * outputs + 0.0039 * n[0];
        call = 0.5 + 0.028 * runs;
    } else if (L == 2) {
        there = 0.9 * (5.0 + (many ? 1.9 : 0.0) + 0.0285 * far + 0.166 * outputs);
        here = 3.4 + 1.1 * spread + 0.0157 * rows + 0.027 * outputs;
        call = 0.039 * runs - 5.3;
    } else {
        there = 0.9 * (11.5 + 6.3 * deep + 0.031 * far + 0.0012 * partial + 0.12 * outputs);
        here = 5.3 + 1.1 * deep + 4.5 * spread * (L - 2) + 0.012 * rows + 0.012 * outputs;
        call = 0.039 * runs - 5.3;
    }
    return (double)n_samples * (there - here) > call;
}

// Whether a batch-1 pass runs on that kernel.  us a step, before / there (200 and 214 samples): against the general kernel, 4-32-643-7 16.2 /
// 14.6, 96-64-160-440-37 26 / 16, 37-116-21-61 21.5 / 6.8, with momentum 192-68-7 8.6 / 4.6, 1000-1000-33 19.0 / 7.2 and 1024-1024-1024-1024-10
// 25.4 / 22.7.  Against the kernel with two copies on one workgroup 28-16-32-188-19 15.9 / 9.5, 532-44-20-9 (24468 weights) 7.6 / 7.6,
// 68-16-676-23 (27 thousand) 17.8 / 15.8, but 4-32-736-10 (31 thousand) 13.5 / 15.8, 544-44-224-2 (34 thousand) 10.0 / 10.4, and on two and
// more workgroups 376-156-32-5 8.1 / 9.6, 868-544-896-640-3 12.9 / 17.9.  Against one wavefront 18-10-21-7-23 (698 weights) 6.8 / 6.8,
// 8-33-10-19-14 with momentum (1050) 8.1 / 7.8, 36-54-15-32 13.6 / 5.8.
bool takes_slices(dn_net *net, float mu, int64_t n_samples, SliceGeom &g)
{
    if (!net->slice_ready || !net->online_slices || net->online_mode != 0) return false;
    const int L = net->L;
    if (!slice_geometry(net->n.data(), L, mu != 0.f, net->device_cus, g) || g.words * sizeof(unsigned long long) > net->lo.online_bytes) return false;
    if (net->online_slices == 2) return true;
    if (L == 2 && mu == 0.f) return false;
    // (a caller that sets one of these means the general kernel)
    if (net->online_min_tile != ON_DEFAULT_MIN_TILE || net->online_resident == 0) return false;
    // (on a device of few compute units a net may fit no other persistent kernel: its passes stay launches, which wait for nobody)
    if (g.P > 1 && !net->online_ok) return false;
    int64_t weights = 0;
    for (int l = 1; l <= L; ++l) weights += (int64_t)net->n[l] * net->n[l - 1];
    // One wavefront: a step gains by the net's size, a call costs up to 16 us more (54 nets of 1050 to 7200 weights, the first faster
    // pass: 1050 64 samples, 1350 8, 2000 6, 2400 3 or 4, 2800 2 or 3, 3600 one).
    TinyPlan tiny;
    if (one_wave(net, mu, tiny)) return weights > 1024 && ((double)n_samples + 1.2) * (double)(weights - 900) > 6300.0;
    TwinGeom tg;
    if (mu == 0.f && net->online_twin && net->twin_ready && twin_geometry(net->n.data(), L, net->online_min_tile, tg) && tg.grid <= net->device_cus)
        return g.P == 1 && weights <= 24576 && slices_pay(net, g, n_samples, true);
    WideGeom wg;
    if (net->online_wide && net->wide_ok && wide_geometry(net->n.data(), L, net->device_cus, mu != 0.f, wg)) return false;
    return !net->online_ok || slices_pay(net, g, n_samples, false);
}

// A whole batch-1 epoch on the persistent kernel that suits the net.
dn_status run_online(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, float lr, float mu,
                     bool blocks, bool timing)
{
    SliceGeom slices;
    if (takes_slices(net, mu, n_samples, slices)) {
        net->last_schedule = DN_SCHED_SLICES;
        return run_slices(net, slices, X, labels, n_samples, lr, mu, timing);
    }
    const int L = net->L;
    TinyPlan tp;
    if (one_wave(net, mu, tp)) return run_tiny(net, tp, X, labels, n_samples, lr, mu, timing);
    BlockGeom bg;
    if (blocks && takes_blocks(net, n_samples, mu, bg)) {
        net->last_schedule = DN_SCHED_SAMPLE_BLOCKS;
        return run_blocks(net, bg, X, labels, n_samples, lr, timing);
    }
    bool solo_ran = false;
    if (mu == 0.f && net->online_solo) {
        // two layers, W_1 within one compute unit's registers: one workgroup, no exchange through memory.
        // Its scalar reads of a sample may run past the row's end; the last tail_steps samples, where
        // that would leave the array, go to the kernels below (which must then be known to fit).
        SoloGeom sg;
        if (solo_geometry(net->n.data(), L, sg) && n_samples > sg.tail_steps && (sg.tail_steps == 0 || net->online_ok)) {
            const int64_t n_solo = n_samples - sg.tail_steps;
            dn_status st = run_solo(net, sg, X, labels, n_solo, lr, sg.tail_steps == 0, timing);
            if (st != DN_OK) return st;
            net->last_schedule = DN_SCHED_ONE_WORKGROUP;
            if (sg.tail_steps == 0) return DN_OK;
            X += (size_t)n_solo * net->n[0];
            labels += n_solo;
            n_samples = sg.tail_steps;
            solo_ran = true;
        }
    }
    dn_status st = run_online_shared(net, X, labels, n_samples, lr, mu, timing);
    if (solo_ran && st == DN_OK) net->last_schedule = DN_SCHED_ONE_WORKGROUP;
    return st;
}

// ... on the kernels whose workgroups exchange through device memory, in launches of at most 2^30 steps each.
dn_status run_online_shared(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, float lr, float mu,
                            bool timing)
{
    const int L = net->L;
    if (mu == 0.f && net->online_twin && net->twin_ready) {
        // slices that fit in LDS with a second copy of the inner layers: no partial sums cross workgroups
        TwinGeom tg;
        if (twin_geometry(net->n.data(), L, net->online_min_tile, tg) && tg.grid <= net->device_cus) {
            net->last_schedule = DN_SCHED_TWO_COPY;
            return run_twin(net, tg, X, labels, n_samples, lr, timing);
        }
    }
    if (net->online_wide && net->wide_ok) {
        // two layers, the hidden one too wide for LDS: most of its rows stay in LDS and registers
        WideGeom wg;
        if (wide_geometry(net->n.data(), L, net->device_cus, mu != 0.f, wg)) {
            net->last_schedule = DN_SCHED_WIDE_HIDDEN;
            return run_wide(net, wg, X, labels, n_samples, lr, mu, timing);
        }
    }
    OnlineGeom g;   // same slices as net->geom; LDS residency depends on whether velocities are read
    if (!online_geometry(net->n.data(), L, net->online_min_tile, mu != 0.f, g) || g.grid > net->device_cus) return DN_ERR_UNSUPPORTED;
    OnlinePlan p{};
    p.L = L;
    for (int l = 1; l <= L; ++l) {
        OnlineLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.n_in = net->n[l - 1]; y.n_out = net->n[l]; y.act = net->act[l];
        y.per = g.per[l]; y.P = g.P[l]; y.kshift = g.kshift[l]; y.seg = g.seg[l]; y.vec4 = g.vec4[l];
        p.act_x[l] = net->exchange() + g.off_act[l];
        p.part_x[l] = net->exchange() + g.off_part[l];
        p.lds_a[l] = g.lds_a[l]; p.lds_own_a[l] = g.lds_own_a[l]; p.lds_own_d[l] = g.lds_own_d[l];
        p.lds_b[l] = g.lds_b[l]; p.lds_w[l] = g.lds_w[l]; p.lds_v[l] = g.lds_v[l];
    }
    p.z_x = net->exchange() + g.off_z;
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.lr = lr; p.mu = mu; p.loss = net->loss;
    p.resident = g.resident;
    p.part_rows = g.part_rows;
    if (net->online_resident == 0) {   // slice images are laid out last: drop them
        p.resident = 0;
        p.part_rows = 0;
        g.lds_floats = g.lds_work_floats;
    }
    p.lds_x = g.lds_x; p.lds_out = g.lds_out; p.lds_kpart = g.lds_kpart; p.lds_tmp = g.lds_tmp;
    const int64_t chunk = (int64_t)1 << 30;
    for (int64_t s0 = 0; s0 < n_samples; s0 += chunk) {
        const int64_t n = (n_samples - s0) < chunk ? (n_samples - s0) : chunk;
        if ((uint64_t)net->online_seq + (uint64_t)n + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->exchange(), 0, net->lo.online_bytes, net->stream));
            net->online_seq = 0;
        }
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (s0 + n >= n_samples) ? 1 : 0;
        p.seq0 = net->online_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_online_epoch(g, p, net->stream));
        net->online_seq += (uint32_t)n;
    }
    return DN_OK;
}

// Automatic choice between the persistent minibatch kernel and one launch per product: the
// persistent kernel does its products on the vector units, so it only pays while a step is
// launch bound, i.e. while the step's contraction work is small.  us/step with momentum, persistent against launches:
// 784-128-10 batch 32 11.9 / 25.4, batch 128 19.5 / 27.7, batch 256 30.7 / 28.8; 784-256-10 batch 128 22.4 / 28.2, batch 256
// 32.9 / 29.5; 1024-512-10 batch 64 21.3 / 24.5, batch 128 (above the line) 29.8 / 25.9; 2048-1024-10 batch 16 24.6 / 34.5,
// batch 32 28.7 / 34.7, batch 64 (above) 42.0 / 35.3; 784-1024-10 batch 64 27.7 / 27.8.  The line is where it was set before
// the launches became faster; at batch 256 they are now up to a tenth faster below it.
bool batch_pays(const dn_net *net, int batch)
{
    double flop = 0.0;
    for (int l = 1; l <= net->L; ++l) flop += 6.0 * batch * (double)net->n[l] * (double)net->n[l - 1];
    return flop <= 4.0e8;
}

// The same question for the deeper-net kernel, which reads whole activation / delta matrices of
// the batch past the L2 in every phase: it pays while those matrices are small.
bool deep_pays(const dn_net *net, int batch)
{
    (void)net;
    // 1024-1024-1024-1024-10, us/step persistent against one launch per product (7 launches): batch 4: 38 / 66,
    // batch 8: 38 / 66, batch 16: 44 / 65, batch 24: 58 / 66, batch 32: 60 / 65, batch 48: 79 / 70, batch 64: 87 / 71;
    // 512-512-512-10: batch 8: 24 / 34, batch 16: 27 / 34, batch 32: 30 / 34, batch 48: 37 / 35
    return batch <= 32;
}

// A whole minibatch epoch of a one- or two-layer net in persistent-kernel launches.
dn_status run_batch_persistent(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, int batch,
                               float lr, float mu, bool timing)
{
    const int L = net->L;
    BatchGeom g;
    if (!batch_geometry(net->n.data(), L, net->max_batch, net->online_min_tile, mu != 0.f, g)) return DN_ERR_UNSUPPORTED;
    BatchPlan p{};
    p.L = L;
    if (L == 2) { p.W1 = net->W(1); p.b1 = net->b(1); p.VW1 = net->VW(1); p.Vb1 = net->Vb(1); p.act1 = net->act[1]; }
    p.W2 = net->W(L); p.b2 = net->b(L); p.VW2 = net->VW(L); p.Vb2 = net->Vb(L); p.actL = net->act[L];
    p.n0 = net->n[0]; p.n_mid = net->n[L - 1]; p.nL = net->n[L];
    p.per = g.per; p.P = g.P; p.spw = g.spw; p.max_batch = net->max_batch;
    p.z_x = net->batch_exchange() + g.off_z;
    p.d_x = net->batch_exchange() + g.off_d;
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.batch = batch;
    p.lr = lr; p.mu = mu; p.loss = net->loss; p.with_v = (mu != 0.f) ? 1 : 0;
    p.lds_w1 = g.lds_w1; p.lds_v1 = g.lds_v1; p.lds_b1 = g.lds_b1; p.lds_w2 = g.lds_w2; p.lds_v2 = g.lds_v2;
    p.lds_bL = g.lds_bL; p.lds_a1 = g.lds_a1; p.lds_d1 = g.lds_d1; p.lds_d2 = g.lds_d2; p.lds_zs = g.lds_zs;
    p.lds_tmp = g.lds_tmp;
    const int64_t chunk_steps = (int64_t)1 << 30;
    const int64_t total_steps = (n_samples + batch - 1) / batch;
    for (int64_t t0 = 0; t0 < total_steps; t0 += chunk_steps) {
        const int64_t nt = (total_steps - t0) < chunk_steps ? (total_steps - t0) : chunk_steps;
        if ((uint64_t)net->batch_seq + (uint64_t)nt + 2 > 0xffffffffull) {   // step numbers would wrap
            DN_HIP(hipMemsetAsync(net->batch_exchange(), 0, net->lo.batch_bytes, net->stream));
            net->batch_seq = 0;
        }
        const int64_t s0 = t0 * batch;
        const int64_t n = ((t0 + nt) * batch < n_samples ? (t0 + nt) * batch : n_samples) - s0;
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (t0 + nt >= total_steps) ? 1 : 0;
        p.seq0 = net->batch_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_batch_epoch(g, p, net->stream));
        net->batch_seq += (uint32_t)nt;
    }
    return DN_OK;
}

// A whole plain-gradient-descent minibatch epoch of a net of three or more layers in
// persistent-kernel launches.
dn_status run_deep_persistent(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, int batch,
                              float lr, bool timing)
{
    const int L = net->L;
    DeepGeom g;
    if (!deep_geometry(net->n.data(), L, net->max_batch, net->online_min_tile, g)) return DN_ERR_UNSUPPORTED;
    DeepPlan p{};
    p.L = L;
    char *ex = net->deep_exchange();
    for (int l = 1; l <= L; ++l) {
        DeepLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.n_in = net->n[l - 1]; y.n_out = net->n[l]; y.act = net->act[l];
        y.per = g.per[l]; y.P = g.P[l];
        p.ea[l] = (float *)(ex + g.off_ea[l]); p.ed[l] = (float *)(ex + g.off_ed[l]);
        p.fa[l] = (unsigned long long *)(ex + g.off_fa[l]); p.fd[l] = (unsigned long long *)(ex + g.off_fd[l]);
        p.lds_r[l] = g.lds_r[l]; p.lds_ct[l] = g.lds_ct[l]; p.lds_b[l] = g.lds_b[l]; p.lds_a[l] = g.lds_a[l];
        p.lds_dl[l] = g.lds_dl[l];
    }
    p.grid = g.grid; p.spw = g.spw; p.max_batch = net->max_batch; p.halves = g.halves;
    p.z_x = (unsigned long long *)(ex + g.off_z);
    p.d_x = (unsigned long long *)(ex + g.off_d);
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.batch = batch;
    p.lr = lr; p.loss = net->loss;
    p.lds_w2 = g.lds_w2; p.lds_bL = g.lds_bL; p.lds_d2 = g.lds_d2; p.lds_zs = g.lds_zs; p.lds_tmp = g.lds_tmp;
    const int64_t chunk_steps = (int64_t)1 << 30;
    const int64_t total_steps = (n_samples + batch - 1) / batch;
    for (int64_t t0 = 0; t0 < total_steps; t0 += chunk_steps) {
        const int64_t nt = (total_steps - t0) < chunk_steps ? (total_steps - t0) : chunk_steps;
        if ((uint64_t)net->deep_seq + (uint64_t)nt + 2 > 0xffffffffull) {
            DN_HIP(hipMemsetAsync(net->deep_exchange(), 0, net->lo.deep_bytes, net->stream));
            net->deep_seq = 0;
        }
        const int64_t s0 = t0 * batch;
        const int64_t n = ((t0 + nt) * batch < n_samples ? (t0 + nt) * batch : n_samples) - s0;
        p.X = X + (size_t)s0 * net->n[0];
        p.labels = labels + s0;
        p.n_samples = n;
        p.keep_v = (t0 + nt >= total_steps) ? 1 : 0;
        p.seq0 = net->deep_seq;
        ScopedTimer st(net, DN_K_ONLINE, timing);
        DN_HIP(launch_deep_epoch(g, p, net->stream));
        net->deep_seq += (uint32_t)nt;
    }
    return DN_OK;
}

// Microseconds a step takes on the schedules that a minibatch pass would run on without tiles: the low side of what was measured, so
// that tiles are not taken where they could lose.  The kernel for one and two layers (62 nets of 64 and more inputs, 20 %; 61 nets of
// fewer, which cost it more, the fewer the more: 24-888-4 batch 43 22, 8-512-6 batch 109 44): with the first layer's rows in few workgroups 784-128-10 batch 128 18.6 and 1288-19-4 batch 4 10.1,
// but 64-106-3 batch 12 21, 44-424-127 batch 3 72.  Launches, 124 nets, 15 %: 12.7 a layer for the launches themselves, then by flops,
// parameters read and written, and a launch for a last layer of more than 16 outputs.
float step_us_without_tiles(const dn_net *net, int batch)
{
    const int L = net->L, n0 = net->n[0], nL = net->n[L];
    if (net->batch_ok && batch_pays(net, batch)) {
        const int n1 = L == 2 ? net->n[1] : n0, per = std::min(std::min(n1, PB_MAX_ROWS), std::max((n1 + 255) / 256, (4095 + n0) / n0));
        if (n0 >= 64)
            return 0.85f * (9.4f + 0.079f * (float)batch + 0.0116f * (float)n1 + 0.146f * (float)nL + 0.0144f * (float)((n1 + per - 1) / per) +
                            4.27e-5f * (float)batch * (float)n0);
        return (n0 < 20 ? 0.8f : 0.62f) * (21.9f + 0.017f * (float)n1 + 0.0184f * (float)(per * nL));
    }
    double weights = 0.0;
    for (int l = 1; l <= L; ++l) weights += (double)net->n[l] * (double)net->n[l - 1];
    return 0.88f * (11.4f * (float)L + (float)(weights * (6e-8 * batch + 3e-6)) + (nL > 16 ? 3.f : 0.f));
}

// A net of one layer: microseconds that a step on tiles takes less than on batch_epoch_kernel, the low side.  There it has no exchange
// but the outputs', here the workgroups of a row of tiles wait for one another and share the samples among them: nets of few inputs and
// outputs lose (us a step, batch_epoch_kernel / tiles: 16-21 batch 234 14 / 78, 304-3 batch 157 7.2 / 10.9, 12-3 batch 19 5.8 / 9.3), many
// outputs gain (392-112 batch 19 37 / 6.7, 480-27 batch 12 10 / 6.0).  121 nets, both estimates to 12 and 5 % in the mean.
float one_layer_gain(const dn_net *net, int batch, const TileGeom &g)
{
    auto up = [](int a, int b) { return (a + b - 1) / b; };
    const int n0 = net->n[0], nL = net->n[1], samples = up(batch, g.grid), out16 = up(nL, 16);
    const float there = 4.9f + 0.0212f * (float)batch + 0.0856f * (float)nL + 0.00086f * (float)batch * (float)nL + 1.27e-4f * (float)n0 * (float)nL;
    const float here = 3.3f + 1.3f * (float)up(samples, 8) + 0.92f * (float)(up(samples * out16, 16) * up(up(g.C[1], 4), 4)) +
                       0.48f * (float)(g.rows / 16) * (float)g.T / 32.f;
    return 0.83f * there - here;
}

// Whether a minibatch pass runs on the kernel that cuts every layer into tiles.  (A caller that sets "online_min_tile" means the
// kernels that own rows.)  A call there costs 3 to 7 us more than one on batch_epoch_kernel, so a pass of few steps may stay on that: us a
// call of 1, 2, 4 and 8 steps, batch_epoch_kernel / tiles: 784-128-10 batch 128 53.7 / 58.5, 72.4 / 75.3, 109 / 107, 186 / 172.
// (Launches and the kernel for deeper nets lose with one step already: 32 samples of 1024-1024-1024-1024-10 at batch 32 115 / 95.)
bool takes_tiles(const dn_net *net, int64_t n_samples, int batch, TileGeom &g)
{
    if (!net->tile_ready || !net->batch_tiles || net->online_min_tile != ON_DEFAULT_MIN_TILE || batch < 2) return false;
    if ((n_samples + batch - 1) / batch > ((int64_t)1 << 31) / (2 * net->L)) return false;   // (phases are counted in 32 bits)
    if (!tile_geometry(net->n.data(), net->L, batch, net->device_cus, g) || g.words * sizeof(unsigned long long) > net->lo.tile_bytes) return false;
    if (net->batch_tiles >= 2) return true;
    const float steps = (float)((n_samples + batch - 1) / batch);
    const bool rows = net->batch_ok && batch_pays(net, batch);   // batch_epoch_kernel runs the pass without tiles
    if (rows && net->L == 1) return one_layer_gain(net, batch, g) * steps > 3.f;
    const float without = step_us_without_tiles(net, batch);
    return g.step_us < without && (!rows || (1.18f * without - g.step_us) * steps > 8.f);
}

// A whole minibatch epoch in one launch of that kernel.
dn_status run_tiles(dn_net *net, const TileGeom &g, const float *X, const int32_t *labels, int64_t n_samples, int batch, float lr,
                    float mu, bool timing)
{
    const int L = net->L;
    TilePlan p{};
    for (int l = 1; l <= L; ++l) {
        TileLayer &y = p.layer[l];
        y.W = net->W(l); y.b = net->b(l); y.VW = net->VW(l); y.Vb = net->Vb(l);
        y.n_in = net->n[l - 1]; y.n_out = net->n[l]; y.act = net->act[l];
    }
    p.abort_flag = net->abort_flag();
    p.loss_acc = net->epoch_acc();
    p.arrived = net->arrived();
    p.settled = net->settled();
    p.expected = (unsigned)g.grid + (net->batch_tiles == 3 ? 1u : 0u);   // (3: one more than will come)
    p.X = X; p.labels = labels; p.n_samples = n_samples; p.batch = batch;
    p.lr = lr; p.mu = mu; p.loss = net->loss; p.keep_v = 1;
    const uint64_t phases = (uint64_t)((n_samples + batch - 1) / batch) * (uint64_t)(2 * L - 1) + 1;
    if ((uint64_t)net->tile_seq + phases + 2 > 0xffffffffull) {   // phase numbers would wrap
        DN_HIP(hipMemsetAsync(net->tile_exchange(), 0, net->lo.tile_bytes, net->stream));
        net->tile_seq = 0;
    }
    p.seq0 = net->tile_seq;
    p.ex = net->tile_exchange();
    ScopedTimer st(net, DN_K_ONLINE, timing);
    DN_HIP(launch_tile_epoch(g, p, L, net->stream));
    net->tile_seq += (uint32_t)phases;
    return DN_OK;
}

// Launch-per-product path: every step enqueued on the net's stream.
dn_status run_launches(dn_net *net, const float *X, const int32_t *labels, int64_t n_samples, int32_t batch, float lr, float momentum,
                       bool timing)
{
    const int L = net->L;
    // The epoch's loss is kept as one running sum per batch row, added
    // to by the output kernel of each step, and reduced once after the last step.
    const int rows_used = (int)(n_samples < batch ? n_samples : batch);
    DN_HIP(hipMemsetAsync(net->loss_sums(), 0, (size_t)rows_used * sizeof(double), net->stream));
    for (int64_t s0 = 0; s0 < n_samples; s0 += batch) {
        const int B = (int)((n_samples - s0) < batch ? (n_samples - s0) : batch);
        const float *Xb = X + (size_t)s0 * net->n[0];
        const bool last = s0 + batch >= n_samples;
        const int mode = (momentum != 0.f) ? GRAD_MOMENTUM : (last ? GRAD_SGD_KEEPV : GRAD_SGD);
        // a last layer of at most 16 outputs: its forward product and the output error in one launch
        const bool fused_out = net->gemm_variant < 0 && narrow_layer(net->n[L]);
        dn_status st = run_forward(net, Xb, B, timing, fused_out ? L - 1 : L);
        if (st != DN_OK) return st;
        {
            // with a narrow last layer the launch also holds that layer's forward product and its delta product
            const double out_flop = fused_out ? 2.0 * B * (double)net->n[L] * net->n[L - 1] * (L > 1 ? 2.0 : 1.0) : 0.0;
            ScopedTimer t(net, DN_K_OUTPUT, timing, out_flop, true);
            if (fused_out)
                DN_HIP(launch_narrow_output(L == 1 ? Xb : net->A(L - 1), net->W(L), net->b(L), labels + s0, net->A(L),
                                            net->D(L), net->loss_rows(), net->loss_sums(), B, net->n[L], net->n[L - 1],
                                            net->act[L], net->loss, net->stream, L > 1 ? net->D(L - 1) : nullptr,
                                            L > 1 ? net->act[L - 1] : 0));
            else
                DN_HIP(launch_output_delta(net->A(L), net->D(L), labels + s0, net->loss_rows(), B, net->n[L],
                                           net->act[L], net->loss, OUT_FUSED, net->stream, nullptr, net->loss_sums()));
        }
        st = run_backward(net, Xb, B, mode, lr, momentum, timing, fused_out && L > 1);
        if (st != DN_OK) return st;
    }
    DN_HIP(launch_loss_sums_reduce(net->loss_sums(), rows_used, net->epoch_acc(), net->stream));
    return DN_OK;
}

void collect_times(dn_net *net)
{
    for (int c = 0; c < DN_K_CLASSES; ++c) {
        net->cls_ms[c] = 0.0;
        net->cls_flop[c] = 0.0;
        net->cls_launches[c] = 0;
    }
    for (int i = 0; i < net->timed; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, net->pool[i].start, net->pool[i].stop) == hipSuccess) {
            net->cls_ms[net->pool[i].cls] += ms;
            net->cls_flop[net->pool[i].cls] += net->pool[i].flop;
            net->cls_launches[net->pool[i].cls] += 1;
        }
    }
}

}  // namespace

extern "C" {

const char *dn_status_string(dn_status s)
{
    switch (s) {
    case DN_OK: return "ok";
    case DN_ERR_INVALID_ARG: return "invalid argument";
    case DN_ERR_SHAPE: return "shape mismatch";
    case DN_ERR_UNSUPPORTED: return "unsupported activation/loss combination";
    case DN_ERR_OOM: return "out of host memory";
    case DN_ERR_DEVICE: return "device error";
    default: return "unknown status";
    }
}

size_t dn_net_arena_bytes(const int32_t *widths, int32_t n_widths, int32_t max_batch)
{
    Layout lo;
    return compute_layout(widths, n_widths, max_batch, lo) ? lo.total : 0;
}

dn_status dn_net_create(const int32_t *widths, int32_t n_widths, const dn_act *acts, dn_loss loss,
                        int32_t max_batch, void *arena_dev, size_t arena_bytes, void *hip_stream,
                        dn_net **out)
{
    if (!out) return DN_ERR_INVALID_ARG;
    *out = nullptr;
    if (!widths || !acts || !arena_dev) return DN_ERR_INVALID_ARG;
    if (n_widths < 2 || max_batch <= 0) return DN_ERR_SHAPE;
    for (int i = 0; i < n_widths; ++i)
        if (widths[i] <= 0) return DN_ERR_SHAPE;
    if (loss != DN_LOSS_MSE && loss != DN_LOSS_CROSS_ENTROPY) return DN_ERR_INVALID_ARG;
    const int L = n_widths - 1;
    for (int l = 0; l < L; ++l) {
        if ((int)acts[l] < DN_ACT_LINEAR || (int)acts[l] > DN_ACT_SOFTMAX) return DN_ERR_INVALID_ARG;
        if (acts[l] == DN_ACT_SOFTMAX && l != L - 1) return DN_ERR_UNSUPPORTED;
    }
    const bool softmax_last = acts[L - 1] == DN_ACT_SOFTMAX;
    if (softmax_last != (loss == DN_LOSS_CROSS_ENTROPY)) return DN_ERR_UNSUPPORTED;
    if (reinterpret_cast<uintptr_t>(arena_dev) % kAlign != 0) return DN_ERR_INVALID_ARG;
    Layout lo;
    if (!compute_layout(widths, n_widths, max_batch, lo)) return DN_ERR_SHAPE;
    if (arena_bytes < lo.total) return DN_ERR_SHAPE;

    dn_net *net = new (std::nothrow) dn_net();
    if (!net) return DN_ERR_OOM;
    try {
        net->n.assign(widths, widths + n_widths);
        net->act.assign(L + 1, 0);
        for (int l = 1; l <= L; ++l) net->act[l] = (int)acts[l - 1];
        net->lo = lo;
    } catch (...) {
        delete net;
        return DN_ERR_OOM;
    }
    net->L = L;
    net->loss = (int)loss;
    net->max_batch = max_batch;
    net->arena = (char *)arena_dev;
    net->stream = (hipStream_t)hip_stream;
    // persistent kernels: slices per workgroup, if the net fits them and the device has the units
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&net->device_cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            net->device_cus = 0;
        (void)hipGetLastError();
    }
    if (net->device_cus > 0) {
        // the kernels' LDS limits are raised once; whether a net fits follows the tile option
        net->online_prepared = lo.online_bytes > 0 && online_prepare() == hipSuccess;
        net->twin_ready = lo.online_bytes > 0 && twin_exchange_bytes_bound(net->n.data(), L) > 0 && twin_prepare() == hipSuccess;
        net->tiny_ready = tiny_prepare() == hipSuccess;
        net->wide_ready = lo.online_bytes > 0 && wide_exchange_bytes_bound(net->n.data(), L) > 0 && wide_prepare() == hipSuccess;
        WideGeom wg;
        net->wide_block_ready = net->wide_ready && wide_geometry(net->n.data(), L, net->device_cus, false, wg) &&
                                wide_block_fits(net->n[1], wg.per) && wide_block_prepare(net->n[2], net->act[1]) == hipSuccess;
        net->block_ready = block_exchange_bytes(net->n.data(), L) > 0 && block_prepare(net->n.data(), net->act[1]) == hipSuccess;
        net->slice_ready = L >= 2 && L <= SLICE_MAX_L && slice_prepare(L) == hipSuccess;
        net->batch_prepared = lo.batch_bytes > 0 && batch_prepare() == hipSuccess;
        net->deep_prepared = lo.deep_bytes > 0 && deep_prepare() == hipSuccess;
        net->tile_ready = lo.tile_bytes > 0 && tile_prepare() == hipSuccess;
        (void)hipGetLastError();
    }
    refresh_persistent(net);
    // parameters, velocities and gradients start at zero; exchange words start unstamped
    if (hipMemsetAsync(net->arena, 0, 3 * lo.region, net->stream) != hipSuccess ||
        hipMemsetAsync(net->arena + lo.off_scalars, 0, kAlign, net->stream) != hipSuccess ||
        (lo.online_bytes > 0 &&
         hipMemsetAsync(net->arena + lo.off_online, 0, lo.online_bytes, net->stream) != hipSuccess) ||
        hipMemsetAsync(net->arena + lo.off_gemm_counters, 0, GEMM_COUNTERS * sizeof(unsigned), net->stream) != hipSuccess ||
        (lo.batch_bytes > 0 &&
         hipMemsetAsync(net->arena + lo.off_batch, 0, lo.batch_bytes, net->stream) != hipSuccess) ||
        (lo.deep_bytes > 0 &&
         hipMemsetAsync(net->arena + lo.off_deep, 0, lo.deep_bytes, net->stream) != hipSuccess) ||
        (lo.tile_bytes > 0 &&
         hipMemsetAsync(net->arena + lo.off_tile, 0, lo.tile_bytes, net->stream) != hipSuccess) ||
        hipEventCreate(&net->ev_epoch0) != hipSuccess || hipEventCreate(&net->ev_epoch1) != hipSuccess ||
        hipStreamSynchronize(net->stream) != hipSuccess) {
        if (net->ev_epoch0) (void)hipEventDestroy(net->ev_epoch0);
        if (net->ev_epoch1) (void)hipEventDestroy(net->ev_epoch1);
        delete net;
        return DN_ERR_DEVICE;
    }
    TinyPlan tiny;
    if (one_wave(net, 0.f, tiny)) net->result = result_slots.take();
    *out = net;
    return DN_OK;
}

dn_status dn_net_destroy(dn_net *net)
{
    if (!net) return DN_ERR_INVALID_ARG;
    dn_status st = DN_OK;
    if (hipStreamSynchronize(net->stream) != hipSuccess) st = DN_ERR_DEVICE;
    for (auto &t : net->pool) {
        (void)hipEventDestroy(t.start);
        (void)hipEventDestroy(t.stop);
    }
    (void)hipEventDestroy(net->ev_epoch0);
    (void)hipEventDestroy(net->ev_epoch1);
    result_slots.give(net->result);
    delete net;
    return st;
}

dn_status dn_set_params(dn_net *net, int32_t layer, const float *W_host, const float *b_host)
{
    if (!net || layer < 1 || layer > net->L) return DN_ERR_INVALID_ARG;
    if (layer == 1 && W_host) net->w1_as_in_bwd = false;
    const size_t nw = (size_t)net->n[layer] * net->n[layer - 1], nb = (size_t)net->n[layer];
    if (W_host) {
        DN_HIP(hipMemcpyAsync(net->W(layer), W_host, nw * sizeof(float), hipMemcpyHostToDevice, net->stream));
        DN_HIP(hipMemsetAsync(net->VW(layer), 0, nw * sizeof(float), net->stream));
    }
    if (b_host) {
        DN_HIP(hipMemcpyAsync(net->b(layer), b_host, nb * sizeof(float), hipMemcpyHostToDevice, net->stream));
        DN_HIP(hipMemsetAsync(net->Vb(layer), 0, nb * sizeof(float), net->stream));
    }
    DN_HIP(hipStreamSynchronize(net->stream));
    return DN_OK;
}

static dn_status read_pair(dn_net *net, int32_t layer, const float *Wd, const float *bd, float *W_host,
                           float *b_host)
{
    const size_t nw = (size_t)net->n[layer] * net->n[layer - 1], nb = (size_t)net->n[layer];
    if (W_host) DN_HIP(hipMemcpyAsync(W_host, Wd, nw * sizeof(float), hipMemcpyDeviceToHost, net->stream));
    if (b_host) DN_HIP(hipMemcpyAsync(b_host, bd, nb * sizeof(float), hipMemcpyDeviceToHost, net->stream));
    DN_HIP(hipStreamSynchronize(net->stream));
    return DN_OK;
}

dn_status dn_get_params(dn_net *net, int32_t layer, float *W_host, float *b_host)
{
    if (!net || layer < 1 || layer > net->L) return DN_ERR_INVALID_ARG;
    return read_pair(net, layer, net->W(layer), net->b(layer), W_host, b_host);
}

dn_status dn_get_grads(dn_net *net, int32_t layer, float *G_host, float *g_host)
{
    if (!net || layer < 1 || layer > net->L) return DN_ERR_INVALID_ARG;
    if (!net->have_bwd) return DN_ERR_INVALID_ARG;
    return read_pair(net, layer, net->GW(layer), net->Gb(layer), G_host, g_host);
}

dn_status dn_forward(dn_net *net, const float *X_dev, int32_t batch, float *out_dev)
{
    if (!net || !X_dev) return DN_ERR_INVALID_ARG;
    if (batch < 1 || batch > net->max_batch) return DN_ERR_SHAPE;
    net->have_fwd = false;
    net->have_bwd = false;
    net->w1_as_in_bwd = false;
    // A narrow last layer's product, softmax and the copy to the caller are one launch, other softmax layers' last two.  (Not the
    // copy of a single layer's narrow outputs: the product reads X, which a caller may ask to be overwritten.)
    const int L = net->L;
    const bool narrow = one_launch_forward(net, batch);
    dn_status st = run_forward(net, X_dev, batch, false, narrow ? L - 1 : L);
    if (st != DN_OK) return st;
    if (narrow)
        DN_HIP(launch_narrow_output(L == 1 ? X_dev : net->A(L - 1), net->W(L), net->b(L), nullptr, net->A(L), nullptr, nullptr,
                                    nullptr, batch, net->n[L], net->n[L - 1], net->act[L], net->loss, net->stream, nullptr, 0,
                                    L > 1 ? out_dev : nullptr));
    else if (net->loss == DN_LOSS_CROSS_ENTROPY)
        DN_HIP(launch_output_delta(net->A(L), net->D(L), nullptr, net->loss_rows(), batch, net->n[L],
                                   net->act[L], net->loss, OUT_SOFTMAX_ONLY, net->stream, nullptr, nullptr, out_dev));
    if (out_dev && (narrow ? L == 1 : net->loss != DN_LOSS_CROSS_ENTROPY))
        DN_HIP(launch_copy(out_dev, net->A(L), (size_t)batch * net->n[L], net->stream));
    net->X = X_dev;
    net->fwd_batch = batch;
    net->have_fwd = true;
    return DN_OK;
}

dn_status dn_backward(dn_net *net, const int32_t *labels_dev, int32_t batch, float *loss_dev)
{
    if (!net || !labels_dev) return DN_ERR_INVALID_ARG;
    if (!net->have_fwd) return DN_ERR_INVALID_ARG;
    if (batch != net->fwd_batch) return DN_ERR_SHAPE;
    const int L = net->L;
    DN_HIP(launch_output_delta(net->A(L), net->D(L), labels_dev, net->loss_rows(), batch, net->n[L],
                               net->act[L], net->loss, OUT_FROM_P, net->stream));
    if (loss_dev) DN_HIP(launch_loss_reduce(net->loss_rows(), batch, loss_dev, nullptr, net->stream));
    dn_status st = run_backward(net, net->X, batch, GRAD_STORE, 0.f, 0.f, false);
    if (st != DN_OK) return st;
    net->have_bwd = true;
    net->w1_as_in_bwd = true;
    return DN_OK;
}

dn_status dn_input_gradient(dn_net *net, int32_t batch, float *dX_dev)
{
    if (!net || !dX_dev) return DN_ERR_INVALID_ARG;
    if (!net->have_bwd || !net->w1_as_in_bwd) return DN_ERR_INVALID_ARG;
    if (batch != net->fwd_batch) return DN_ERR_SHAPE;
    // the delta propagation of the hidden layers, one layer further: the input has no activation,
    // so the derivative factor is that of the identity (the kernel still reads an operand of the
    // output's shape for it, whose values the identity's derivative ignores: the output buffer
    // itself, so that the caller's X need not outlive dn_backward)
    GemmArgs g{};
    g.A = net->D(1); g.lda = net->n[1];
    g.B = net->W(1); g.ldb = net->n[0];
    g.M = batch; g.N = net->n[0]; g.K = net->n[1];
    g.C = dX_dev; g.ldc = net->n[0];
    g.aux = dX_dev;
    g.act = DN_ACT_LINEAR;
    net->split_k(g);
    DN_HIP(launch_gemm(GEMM_DELTA, g, net->gemm_variant, net->stream));
    return DN_OK;
}

dn_status dn_update(dn_net *net, float lr, float momentum)
{
    if (!net || !rate_ok(lr, momentum)) return DN_ERR_INVALID_ARG;
    if (!net->have_bwd) return DN_ERR_INVALID_ARG;
    net->w1_as_in_bwd = false;
    // parameters, velocities and gradients are three regions of one shape (padding holds zeros)
    DN_HIP(launch_update((float *)(net->arena + net->lo.off_params), (float *)(net->arena + net->lo.off_vel),
                         (const float *)(net->arena + net->lo.off_grads), net->lo.region / sizeof(float), lr,
                         momentum, net->stream));
    return DN_OK;
}

dn_status dn_sgd_step(float *param_dev, const float *grad_dev, float *velocity_dev, int64_t count, float lr,
                      float momentum, void *hip_stream)
{
    if (!param_dev || !grad_dev || !rate_ok(lr, momentum)) return DN_ERR_INVALID_ARG;
    if (momentum != 0.f && !velocity_dev) return DN_ERR_INVALID_ARG;
    if (count < 1) return DN_ERR_SHAPE;
    DN_HIP(launch_update(param_dev, velocity_dev, grad_dev, (size_t)count, lr, momentum, (hipStream_t)hip_stream));
    return DN_OK;
}

dn_status dn_train_epoch(dn_net *net, const float *X_dev, const int32_t *labels_dev, int64_t n_samples,
                         int32_t batch, float lr, float momentum, float *mean_loss_host)
{
    if (!net || !X_dev || !labels_dev || n_samples <= 0 || !rate_ok(lr, momentum)) return DN_ERR_INVALID_ARG;
    if (batch < 1 || batch > net->max_batch) return DN_ERR_SHAPE;
    net->have_fwd = net->have_bwd = net->w1_as_in_bwd = false;  // activations / gradients of the split API are overwritten
    const bool timing = net->time_kernels != 0;
    net->timed = 0;
    // (a two-layer net with a very wide hidden layer may suit only the kernel for such nets)
    bool wide_fit = false;
    if (net->online_wide && net->wide_ok) {
        WideGeom wg;
        wide_fit = wide_geometry(net->n.data(), net->L, net->device_cus, momentum != 0.f, wg);
    }
    const bool online_fit = net->online_ok || wide_fit;
    if (batch == 1 && net->online_mode == 2 && !online_fit) return DN_ERR_UNSUPPORTED;
    const bool pbatch = batch > 1 && net->batch_mode != 1 && net->batch_ok &&
                        (net->batch_mode == 2 || batch_pays(net, batch));
    const bool pdeep = batch > 1 && net->batch_mode != 1 && net->deep_ok && momentum == 0.f &&
                       (net->batch_mode == 2 || deep_pays(net, batch));
    if (batch > 1 && net->batch_mode == 2 && !pbatch && !pdeep) return DN_ERR_UNSUPPORTED;
    // One wavefront runs the whole pass and hands the loss over itself: no memset before it and no copy after it (iris 4-16-3,
    // 150 samples, us a pass: 119.3 with both, 102.8 without).
    BlockGeom bg;
    TinyPlan tiny;
    TileGeom tg;
    // Samples may be taken in blocks, layers in tiles.  A launch of tiles that is taken back has cost a tenth of a second, some fifty times a
    // small pass: whatever kept its workgroups apart is given 8 passes to go away, then 16, up to 1024.
    bool blocks = true, tiles = batch > 1 && net->tile_rest == 0;
    if (batch > 1 && net->tile_rest > 0) --net->tile_rest;
    int64_t first = 0;    // samples that are done
    SliceGeom slices;
    const bool few = batch == 1 && takes_slices(net, momentum, n_samples, slices);
    const bool direct = batch == 1 && net->online_mode != 1 && online_fit && net->result && !few && one_wave(net, momentum, tiny);
    // what the kernels of a whole pass leave beside the parameters: off_scalars
    struct { double acc; int aborted, swept; double hits; unsigned arrived; int settled; } res{};
    static_assert(sizeof(res) == 32, "the scalars of the arena");
    if (!direct) DN_HIP(hipMemsetAsync(net->epoch_acc(), 0, sizeof(res), net->stream));
    DN_HIP(hipEventRecord(net->ev_epoch0, net->stream));
    for (;;) {
        const float *X = X_dev + (size_t)first * net->n[0];
        const int32_t *labels = labels_dev + first;
        const int64_t n = n_samples - first;
        bool persistent = batch == 1 && net->online_mode != 1 && (online_fit || few || (blocks && takes_blocks(net, n, momentum, bg)));
        // A persistent path that turns out not to fit (its geometry is recomputed for this call's momentum
        // and the current tile option) reports DN_ERR_UNSUPPORTED before it launches anything: in automatic
        // mode the epoch then runs with one launch per product instead.
        net->last_schedule = DN_SCHED_LAUNCHES;
        net->last_tiles = false;
        if (persistent) {
            net->last_schedule = DN_SCHED_PER_SAMPLE;   // run_online changes it if another kernel takes the pass
            dn_status st = run_online(net, X, labels, n, lr, momentum, blocks, timing);
            if (st == DN_ERR_UNSUPPORTED && net->online_mode == 0) persistent = false;
            else if (st != DN_OK) return st;
        } else if (tiles && net->batch_mode == 0 && takes_tiles(net, n, batch, tg)) {
            net->last_schedule = net->L <= 2 ? DN_SCHED_MINIBATCH : DN_SCHED_MINIBATCH_DEEP;
            net->last_tiles = true;
            dn_status st = run_tiles(net, tg, X, labels, n, batch, lr, momentum, timing);
            if (st != DN_OK) return st;
            persistent = true;
        } else if (pbatch) {
            net->last_schedule = DN_SCHED_MINIBATCH;
            dn_status st = run_batch_persistent(net, X, labels, n, batch, lr, momentum, timing);
            if (st == DN_OK) persistent = true;
            else if (st != DN_ERR_UNSUPPORTED || net->batch_mode != 0) return st;
        } else if (pdeep) {
            net->last_schedule = DN_SCHED_MINIBATCH_DEEP;
            dn_status st = run_deep_persistent(net, X, labels, n, batch, lr, timing);
            if (st == DN_OK) persistent = true;
            else if (st != DN_ERR_UNSUPPORTED || net->batch_mode != 0) return st;
        }
        if (!persistent) {
            net->last_schedule = DN_SCHED_LAUNCHES;
            dn_status st = run_launches(net, X, labels, n, batch, lr, momentum, timing);
            if (st != DN_OK) return st;
        }
        DN_HIP(hipEventRecord(net->ev_epoch1, net->stream));
        if (!direct) DN_HIP(hipMemcpyAsync(&res, net->epoch_acc(), sizeof(res), hipMemcpyDeviceToHost, net->stream));
        DN_HIP(hipStreamSynchronize(net->stream));
        if (direct) res.acc = *(volatile double *)net->result;
        if (res.settled >= 0) {
            if (net->last_tiles) net->tile_pause = 0;
            break;
        }
        // A launch of sample blocks or tiles whose workgroups did not all find room has changed nothing, nor have those behind it: the
        // samples from its first on go to another kernel.
        first += (int64_t)(-1 - res.settled) * BLOCK_LAUNCH_SAMPLES;
        blocks = tiles = false;
        if (net->last_tiles) net->tile_rest = net->tile_pause = std::min(std::max(8, 2 * net->tile_pause), 1024);
        DN_HIP(hipMemsetAsync(net->abort_flag(), 0, sizeof(res) - sizeof(double), net->stream));
    }
    if (res.swept) net->last_schedule = DN_SCHED_WIDE_HIDDEN;   // some or all of the samples were not the block kernel's after all
    DN_HIP(hipEventElapsedTime(&net->epoch_ms, net->ev_epoch0, net->ev_epoch1));
    collect_times(net);
    if (res.aborted) return DN_ERR_DEVICE;   // a workgroup of the persistent kernel gave up waiting
    const double acc = res.acc;
    if (mean_loss_host) *mean_loss_host = (float)(acc / (double)n_samples);
    return DN_OK;
}

dn_status dn_train(dn_net *net, const float *X_dev, const int32_t *labels_dev, int64_t n_samples, int32_t batch,
                   float lr, float momentum, float max_error, int32_t max_epochs, int32_t *epochs_run_host,
                   float *last_loss_host)
{
    if (!net || max_epochs <= 0 || std::isnan(max_error)) return DN_ERR_INVALID_ARG;
    float loss = 0.f;
    int32_t e = 0;
    while (e < max_epochs) {
        dn_status st = dn_train_epoch(net, X_dev, labels_dev, n_samples, batch, lr, momentum, &loss);
        if (st != DN_OK) return st;
        ++e;
        if (loss <= max_error) break;
    }
    if (epochs_run_host) *epochs_run_host = e;
    if (last_loss_host) *last_loss_host = loss;
    return DN_OK;
}

dn_status dn_evaluate(dn_net *net, const float *X_dev, const int32_t *labels_dev, int64_t n_samples, int32_t batch,
                      float *mean_loss_host, int64_t *correct_host)
{
    if (!net || !X_dev || !labels_dev || n_samples <= 0) return DN_ERR_INVALID_ARG;
    if (batch < 1 || batch > net->max_batch) return DN_ERR_SHAPE;
    net->have_fwd = net->have_bwd = net->w1_as_in_bwd = false;  // the activations of the split API are overwritten
    const int L = net->L;
    DN_HIP(hipMemsetAsync(net->epoch_acc(), 0, 24, net->stream));
    for (int64_t s0 = 0; s0 < n_samples; s0 += batch) {
        const int B = (int)((n_samples - s0) < batch ? (n_samples - s0) : batch);
        dn_status st = run_forward(net, X_dev + (size_t)s0 * net->n[0], B, false);
        if (st != DN_OK) return st;
        DN_HIP(launch_output_delta(net->A(L), net->D(L), labels_dev + s0, net->loss_rows(), B, net->n[L],
                                   net->act[L], net->loss, OUT_EVAL, net->stream, net->hit_rows()));
        DN_HIP(launch_loss_reduce(net->loss_rows(), B, nullptr, net->epoch_acc(), net->stream));
        DN_HIP(launch_loss_reduce(net->hit_rows(), B, nullptr, net->hit_acc(), net->stream));
    }
    struct { double loss; int aborted; int pad; double hits; } res = {0.0, 0, 0, 0.0};
    DN_HIP(hipMemcpyAsync(&res, net->epoch_acc(), 24, hipMemcpyDeviceToHost, net->stream));
    DN_HIP(hipStreamSynchronize(net->stream));
    if (mean_loss_host) *mean_loss_host = (float)(res.loss / (double)n_samples);
    if (correct_host) *correct_host = (int64_t)(res.hits + 0.5);
    return DN_OK;
}

size_t dn_layer_backward_workspace_bytes(int32_t cols_out, int32_t cols_input)
{
    if (cols_out <= 0 || cols_input <= 0) return 0;
    const size_t nw = (size_t)cols_out * (size_t)cols_input;
    if (nw > ((size_t)1 << 31)) return 0;
    return align_up((size_t)cols_out * 4) * 2 + align_up((size_t)cols_input * 4) + 2 * align_up(nw * 4);
}

dn_status dn_layer_backward_host(const float *deltas_host, const float *inputs_host, float learning_rate,
                                 int32_t cols_out, int32_t cols_input, float *gradients_host,
                                 float *delta_weights_host, float *delta_biases_host, void *workspace_dev,
                                 size_t workspace_bytes, void *hip_stream, float *ms_copy_in, float *ms_kernel,
                                 float *ms_copy_out)
{
    if (!deltas_host || !inputs_host || !gradients_host || !delta_weights_host || !delta_biases_host ||
        !workspace_dev || !std::isfinite(learning_rate))
        return DN_ERR_INVALID_ARG;
    const size_t need = dn_layer_backward_workspace_bytes(cols_out, cols_input);
    if (need == 0 || workspace_bytes < need) return DN_ERR_SHAPE;
    if (reinterpret_cast<uintptr_t>(workspace_dev) % kAlign != 0) return DN_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    const size_t nw = (size_t)cols_out * (size_t)cols_input;
    char *w = (char *)workspace_dev;
    float *d_dev = (float *)w; w += align_up((size_t)cols_out * 4);
    float *db_dev = (float *)w; w += align_up((size_t)cols_out * 4);
    float *x_dev = (float *)w; w += align_up((size_t)cols_input * 4);
    float *g_dev = (float *)w; w += align_up(nw * 4);
    float *dw_dev = (float *)w;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    dn_status st = DN_OK;
    for (auto &e : ev)
        if (hipEventCreate(&e) != hipSuccess) st = DN_ERR_DEVICE;
    auto ok = [&](hipError_t e) { if (e != hipSuccess) st = DN_ERR_DEVICE; return st == DN_OK; };
    if (st == DN_OK) {
        // the task schedule of the paper: stream in, run the task, stream out
        ok(hipEventRecord(ev[0], stream)) &&
        ok(hipMemcpyAsync(d_dev, deltas_host, (size_t)cols_out * 4, hipMemcpyHostToDevice, stream)) &&
        ok(hipMemcpyAsync(x_dev, inputs_host, (size_t)cols_input * 4, hipMemcpyHostToDevice, stream)) &&
        ok(hipEventRecord(ev[1], stream)) &&
        ok(launch_layer_backward(d_dev, x_dev, learning_rate, cols_out, cols_input, g_dev, dw_dev, db_dev, stream)) &&
        ok(hipEventRecord(ev[2], stream)) &&
        ok(hipMemcpyAsync(gradients_host, g_dev, nw * 4, hipMemcpyDeviceToHost, stream)) &&
        ok(hipMemcpyAsync(delta_weights_host, dw_dev, nw * 4, hipMemcpyDeviceToHost, stream)) &&
        ok(hipMemcpyAsync(delta_biases_host, db_dev, (size_t)cols_out * 4, hipMemcpyDeviceToHost, stream)) &&
        ok(hipEventRecord(ev[3], stream)) &&
        ok(hipStreamSynchronize(stream));
    }
    if (st == DN_OK) {
        float a = 0.f, b = 0.f, c = 0.f;
        if (hipEventElapsedTime(&a, ev[0], ev[1]) != hipSuccess || hipEventElapsedTime(&b, ev[1], ev[2]) != hipSuccess ||
            hipEventElapsedTime(&c, ev[2], ev[3]) != hipSuccess)
            st = DN_ERR_DEVICE;
        if (ms_copy_in) *ms_copy_in = a;
        if (ms_kernel) *ms_kernel = b;
        if (ms_copy_out) *ms_copy_out = c;
    }
    for (auto &e : ev)
        if (e) (void)hipEventDestroy(e);
    return st;
}

dn_status dn_last_epoch_ms(dn_net *net, float *epoch_ms)
{
    if (!net || !epoch_ms) return DN_ERR_INVALID_ARG;
    *epoch_ms = net->epoch_ms;
    return DN_OK;
}

dn_status dn_last_schedule(dn_net *net, int32_t *schedule)
{
    if (!net || !schedule) return DN_ERR_INVALID_ARG;
    *schedule = net->last_schedule;
    return DN_OK;
}

dn_status dn_last_kernel(dn_net *net, const char **name)
{
    if (!net || !name) return DN_ERR_INVALID_ARG;
    switch (net->last_schedule) {
    case DN_SCHED_PER_SAMPLE: *name = "online_epoch_kernel"; break;
    case DN_SCHED_TWO_COPY: *name = "twin_epoch_kernel"; break;
    case DN_SCHED_MINIBATCH: *name = net->last_tiles ? "tile_epoch_kernel" : "batch_epoch_kernel"; break;
    case DN_SCHED_MINIBATCH_DEEP: *name = net->last_tiles ? "tile_epoch_kernel" : "deep_batch_epoch_kernel"; break;
    case DN_SCHED_ONE_WAVE: *name = "tiny_epoch_kernel"; break;
    case DN_SCHED_WIDE_HIDDEN: *name = "wide_epoch_kernel"; break;
    case DN_SCHED_ONE_WAVE_REGISTERS: *name = "tiny_regs_epoch_kernel"; break;
    case DN_SCHED_ONE_WORKGROUP: *name = "solo_epoch_kernel"; break;
    case DN_SCHED_SAMPLE_BLOCKS: *name = "block_epoch_kernel"; break;
    case DN_SCHED_WIDE_BLOCKS: *name = "wide_block_epoch_kernel"; break;
    case DN_SCHED_SLICES: *name = "slice_epoch_kernel"; break;
    default: *name = ""; break;
    }
    return DN_OK;
}

dn_status dn_kernel_time(dn_net *net, int32_t kernel_class, float *ms_total, int64_t *launches)
{
    if (!net || kernel_class < 0 || kernel_class >= DN_K_CLASSES) return DN_ERR_INVALID_ARG;
    if (ms_total) *ms_total = (float)net->cls_ms[kernel_class];
    if (launches) *launches = net->cls_launches[kernel_class];
    return DN_OK;
}

dn_status dn_kernel_flops(dn_net *net, int32_t kernel_class, double *flops)
{
    if (!net || !flops || kernel_class < 0 || kernel_class >= DN_K_CLASSES) return DN_ERR_INVALID_ARG;
    *flops = net->cls_flop[kernel_class];
    return DN_OK;
}

dn_status dn_set_option(dn_net *net, const char *name, int64_t value)
{
    if (!net || !name) return DN_ERR_INVALID_ARG;
    if (!strcmp(name, "time_kernels")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->time_kernels = (int)value;
    } else if (!strcmp(name, "gemm_variant")) {
        if (value < -1 || value >= gemm_variant_count()) return DN_ERR_INVALID_ARG;
        net->gemm_variant = (int)value;
    } else if (!strcmp(name, "online_mode")) {
        if (value < 0 || value > 2) return DN_ERR_INVALID_ARG;
        net->online_mode = (int)value;
    } else if (!strcmp(name, "online_min_tile")) {
        if (value < 1 || value > ((int64_t)1 << 30) || net->lo.online_bytes == 0) return DN_ERR_INVALID_ARG;
        OnlineGeom g;
        if (!online_geometry(net->n.data(), net->L, (int)value, false, g) || g.grid > net->device_cus)
            return DN_ERR_INVALID_ARG;
        if (hipStreamSynchronize(net->stream) != hipSuccess) return DN_ERR_DEVICE;
        net->online_min_tile = (int)value;
        refresh_persistent(net);   // the minibatch kernels cut their slices by the same option
    } else if (!strcmp(name, "batch_mode")) {
        if (value < 0 || value > 2) return DN_ERR_INVALID_ARG;
        net->batch_mode = (int)value;
    } else if (!strcmp(name, "batch_tiles")) {
        if (value < 0 || value > 3) return DN_ERR_INVALID_ARG;
        net->batch_tiles = (int)value;
        net->tile_pause = net->tile_rest = 0;
    } else if (!strcmp(name, "merge_launches")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->merge_launches = (int)value;
    } else if (!strcmp(name, "split_k")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->split_k_on = (int)value;
    } else if (!strcmp(name, "online_resident")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->online_resident = (int)value;
    } else if (!strcmp(name, "online_tiny")) {
        if (value < 0 || value > 2) return DN_ERR_INVALID_ARG;
        net->online_tiny = (int)value;
    } else if (!strcmp(name, "online_solo")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->online_solo = (int)value;
    } else if (!strcmp(name, "online_twin")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->online_twin = (int)value;
    } else if (!strcmp(name, "online_slices")) {
        if (value < 0 || value > 2) return DN_ERR_INVALID_ARG;
        net->online_slices = (int)value;
    } else if (!strcmp(name, "online_blocks")) {
        if (value < 0 || value > 1 << 20) return DN_ERR_INVALID_ARG;
        net->online_blocks = (int)value;
    } else if (!strcmp(name, "online_wide")) {
        if (value != 0 && value != 1) return DN_ERR_INVALID_ARG;
        net->online_wide = (int)value;
    } else {
        return DN_ERR_INVALID_ARG;
    }
    return DN_OK;
}

}  // extern "C"
