"""Per-sample epochs on as few workgroups as hold the net in LDS, against the CPU checker (fp32 storage, fp64 sums) on the same seeded
inputs.

Tolerance 2e-5 (2-norm and largest, per tensor): a step rounds a weight, its velocity and what moves it by 6e-8 of themselves, sums of up
to a thousand terms by a few times that; 40 steps of random signs come to about 1e-6, the largest error of a tensor to a few times
its 2-norm's."""
import numpy as np
import pytest

from oracle.dn_oracle import Oracle
from paper_2001_04206_amd import synth
from parity_util import announce, assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LIN, SIG, TANH, RELU, SOFTMAX = 0, 1, 2, 3, 4
MSE, CE = 0, 1
TOL = 2e-5
WHEREVER_IT_FITS = 2


@pytest.fixture(scope="module")
def dnlib():
    from paper_2001_04206_amd import dn
    assert torch.cuda.is_available(), "these tests need the GPU"
    dn.lib()
    return dn


def train(dn, w, passes, option=WHEREVER_IT_FITS):
    net = dn.Net(w.widths, w.acts, w.loss, 1)
    net.set_all(w.W, w.b)
    net.dn_set_option("online_slices", option)
    net.dn_set_option("online_blocks", 0)
    X = torch.from_numpy(w.X).to("cuda:0")
    y = torch.from_numpy(w.labels).to("cuda:0")
    losses = [net.dn_train_epoch(X, y, 1, w.lr, mu) for mu in passes]
    out = losses, net.get_all(), net.dn_last_schedule()
    net.close()
    return out


def workload(widths, act, loss, n):
    L = len(widths) - 1
    w = synth.make("slices", widths, [act] * (L - 1) + [SOFTMAX if loss == CE else SIG], loss, n_samples=n, features="normal",
                   init="xavier_uniform", batch=1, lr=0.01, momentum=0.0, seed=6)
    rng = np.random.default_rng(13)
    w.b = [rng.standard_normal(k).astype(np.float32) * 0.1 for k in w.widths[1:]]
    return w


# widths, hidden activation, loss, samples
NETS = [
    ([3, 1, 2], TANH, CE, 5),                   # the smallest of everything
    ([1, 5, 1], SIG, MSE, 9),
    ([37, 116, 21, 61], TANH, CE, 40),          # one workgroup
    ([61, 17, 65, 18, 3], SIG, MSE, 40),        # rows on either side of what sixteen and sixty-four lanes take at once
    ([192, 68, 7], LIN, CE, 40),
    ([129, 64, 128, 128], TANH, MSE, 24),       # the widest output
    ([96, 64, 160, 440, 37], TANH, CE, 30),     # three workgroups, six with momentum
    ([2048, 33, 16], TANH, CE, 12),             # the widest input: as many columns as threads times four
    ([40, 2047, 30, 9], TANH, CE, 12),          # a wide layer on a few workgroups, the next on fewer than there are
    ([500, 400, 300, 20], TANH, CE, 16),
    ([1000, 1000, 33], TANH, MSE, 16),
    ([1021, 1023, 1000, 1022, 10], TANH, CE, 10),   # on half the device and more, rows of no multiple of four
    ([300, 700, 5, 650, 6], RELU, CE, 16),      # a layer of fewer units than workgroups
]


@pytest.mark.parametrize("widths,act,loss,n", NETS)
def test_slices_match_checker(dnlib, widths, act, loss, n):
    announce("slices widths=%s" % widths)
    w = workload(widths, act, loss, n)
    passes = (0.0, 0.6, 0.6)      # plain (leaves the last step's velocity), then momentum on top of it
    losses, (W, b), schedule = train(dnlib, w, passes)
    assert schedule == dnlib.DN_SCHED_SLICES
    o = Oracle("o32", w.widths, w.acts, w.loss)
    o.set_params(w.W, w.b)
    for got, mu in zip(losses, passes):
        ref, _ = o.train_epoch(w.X, w.labels, 1, w.lr, mu)
        assert abs(got - ref) <= TOL * max(abs(ref), 0.1), (got, ref)   # (a small loss is a difference of net inputs of up to 10, 6e-7 each)
    Wr, br = o.get_params()
    tol = 1e-3 if act == RELU else TOL     # (a net input within rounding of zero may fall on either side)
    for l in range(len(widths) - 1):
        assert_close(W[l], Wr[l], tol, "W_%d" % (l + 1))
        assert_close(b[l], br[l], tol, "b_%d" % (l + 1))


@pytest.mark.parametrize("widths", [[37, 116, 21, 61], [96, 64, 160, 440, 37], [500, 400, 300, 20]])
def test_slices_repeat_bit_for_bit(dnlib, widths):
    announce("slices determinism widths=%s" % widths)
    w = workload(widths, TANH, CE, 50)
    a, b = train(dnlib, w, (0.0, 0.9)), train(dnlib, w, (0.0, 0.9))
    assert a[0] == b[0] and all(np.array_equal(x, y) for x, y in zip(a[1][0] + a[1][1], b[1][0] + b[1][1]))


def test_not_a_number_stays_one(dnlib):
    announce("slices, NaN")
    w = workload([40, 50, 33, 12], TANH, CE, 6)
    w.X[2, 7] = np.nan
    got, (W, b), _ = train(dnlib, w, (0.0,))
    ref, (Wr, br), schedule = train(dnlib, w, (0.0,), option=0)
    assert schedule != dnlib.DN_SCHED_SLICES and np.isnan(got[0]) and np.isnan(ref[0])
    for x, y in zip(W + b, Wr + br):
        assert np.array_equal(np.isnan(x), np.isnan(y))


@pytest.mark.parametrize("widths", [[5, 6, 2], [1021, 501, 2]])
@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_infinite_deltas(dnlib, widths, mu):
    """Rows of no multiple of four.  The first sample's first output is infinite, and so is its delta, which makes all weights below it and
    their row of the last layer -inf.  The second sample's net inputs are then -inf in the hidden layer and, through weights of one sign, infinite
    in the second output, whose row of the last layer becomes infinite: a NaN in the padding of a row, or from a weight beside the padding,
    would show there."""
    announce("slices, infinite deltas widths=%s mu=%g" % (widths, mu))
    w = synth.make("slices", widths, [LIN, LIN], MSE, n_samples=2, features="normal", init="xavier_uniform", batch=1, lr=0.0001, momentum=0.0, seed=6)
    w.X = np.abs(w.X) + np.float32(0.1)
    w.W = [np.abs(W) + np.float32(0.1) for W in w.W]
    w.W[-1][0], w.W[-1][1] = 3e38, -1.0
    w.b = [np.full(k, 0.1, np.float32) for k in widths[1:]]
    losses, (W, b), schedule = train(dnlib, w, (mu,))
    assert schedule == dnlib.DN_SCHED_SLICES
    ref = dnlib.Net(w.widths, w.acts, w.loss, 1)
    ref.set_all(w.W, w.b)
    ref.dn_set_option("online_mode", 1)
    ref.dn_train_epoch(torch.from_numpy(w.X).to("cuda:0"), torch.from_numpy(w.labels).to("cuda:0"), 1, w.lr, mu)
    Wr, br = ref.get_all()
    ref.close()
    assert np.isinf(W[1][1]).all()
    for got, want in zip(W + b, Wr + br):
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(got), kind(want))
