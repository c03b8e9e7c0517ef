"""Per-sample training with a feature that is NaN or infinite, on the kernels whose exponentials and products of sample blocks do
not follow the plain order of operations: the same numbers are NaN as in the CPU checker, and the others are right.  (In the
last sample, the first layer loses the feature's column; earlier, everything that depends on it.)"""
import numpy as np
import pytest

from oracle.dn_oracle import Oracle
from paper_2001_04206_amd import synth
from parity_util import announce, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIG, TANH, RELU, SOFTMAX = 1, 2, 3, 4
MSE, CE = 0, 1
TOL = 2e-5   # as for sample blocks without such features: a sum in another order, one pass of a few dozen steps


# one wavefront (a net in registers; one of its widest), sample blocks on one to four waves of steps, with and without waves
# that fetch beside them, and over the whole chip
@pytest.mark.parametrize("widths,n", [([4, 16, 3], 70), ([64, 60, 10], 70), ([66, 70, 10], 97), ([40, 200, 5], 97), ([40, 300, 5], 70),
                                      ([40, 500, 5], 97), ([41, 1000, 16], 70), ([384, 30000, 3], 70)])
@pytest.mark.parametrize("act,loss", [(TANH, CE), (SIG, MSE), (RELU, CE)])
@pytest.mark.parametrize("value,sample", [(np.nan, 40), (np.nan, -1), (np.inf, -1), (-np.inf, 33)])
def test_features_that_are_not_finite(widths, n, act, loss, value, sample):
    from paper_2001_04206_amd import dn
    announce("feature %s in sample %d, widths=%s act=%d" % (value, sample, widths, act))
    w = synth.make("nonfinite", widths, [act, SOFTMAX if loss == CE else SIG], loss, n_samples=n, features="normal", init="xavier_uniform",
                   batch=1, lr=0.001, momentum=0.0, seed=21)
    w.X[sample, 2] = value
    net = dn.Net(w.widths, w.acts, w.loss, 1)
    net.set_all(w.W, w.b)
    got_loss = net.dn_train_epoch(torch.from_numpy(w.X).to("cuda:0"), torch.from_numpy(w.labels).to("cuda:0"), 1, w.lr, 0.0)
    ran = net.dn_last_schedule()
    assert ran == (dn.DN_SCHED_ONE_WAVE_REGISTERS if max(widths) <= 64 else dn.DN_SCHED_WIDE_HIDDEN if widths[1] > 1004 else dn.DN_SCHED_SAMPLE_BLOCKS)
    o = Oracle("o32", w.widths, w.acts, w.loss)
    o.set_params(w.W, w.b)
    with np.errstate(all="ignore"):
        ref_loss, _ = o.train_epoch(w.X, w.labels, 1, w.lr, 0.0)
    if loss == MSE:   # (the checker bounds a probability before its logarithm, NaN included)
        assert np.isnan(got_loss) == np.isnan(ref_loss)
    for got, ref, name in zip(sum(zip(*net.get_all()), ()), sum(zip(*o.get_params()), ()), ("W_1", "b_1", "W_2", "b_2")):
        finite = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), finite), (name, np.isfinite(got).mean(), finite.mean())
        if finite.any():
            assert rel_err(got[finite], ref[finite])[0] <= TOL, (name, rel_err(got[finite], ref[finite]))
    net.close()
