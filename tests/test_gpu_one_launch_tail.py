"""What used to be several small operations around a call: the last layer of a forward pass whose outputs are few is one launch
(product, softmax or activation, the copy to the caller), and the kernels of one wavefront hand a pass's loss to the host
themselves."""
import numpy as np
import pytest

from test_gpu_parity import CE, LIN, MSE, SIG, SOFTMAX, TANH, dnlib, torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def forward_bound(X, W, b, acts, loss):
    """Outputs in 64 bits and a bound on an fp32 pass: a sum of k terms is off by at most k + 2 roundings and 2^-21 for operands
    held in 22 bits, each of the sum of its terms' magnitudes; tanh and sigmoid have slopes of at most 1 and cost 8 roundings."""
    a, e = X.astype(np.float64), np.zeros(X.shape)
    for l in range(len(W)):
        k, w = W[l].shape[1], np.abs(W[l].astype(np.float64))
        e = e @ w.T + ((k + 2) * U + 2.0 ** -21) * ((np.abs(a) + e) @ w.T + np.abs(b[l]))
        z = a @ W[l].T.astype(np.float64) + b[l]
        last = l == len(W) - 1
        if last and loss == CE:
            p = np.exp(z - z.max(1, keepdims=True))
            p /= p.sum(1, keepdims=True)
            return p, p * np.expm1(2 * e.max(1, keepdims=True) + 64 * U)   # both parts of the quotient, ten terms, exp and division
        a = {LIN: z, SIG: 1 / (1 + np.exp(-z)), TANH: np.tanh(z)}[acts[l]]
        if acts[l] != LIN:
            e = e + 8 * U
    return a, e


def build(dn, widths, acts, loss, batch, seed):
    rng = np.random.default_rng(seed)
    W = [(rng.standard_normal((o, i)) / np.sqrt(i)).astype(np.float32) for i, o in zip(widths, widths[1:])]
    b = [rng.standard_normal(o).astype(np.float32) for o in widths[1:]]
    net = dn.Net(widths, acts, loss, batch)
    net.set_all(W, b)
    return net, W, b, rng.standard_normal((batch, widths[0])).astype(np.float32)


# one to four rows a workgroup (up to 1024 rows and above), rows of whole and ragged groups of four, the widest narrow layer and one
# more than that; one layer, whose product reads X itself
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("widths,batch,loss", [([64, 96, 10], 128, CE), ([30, 61, 16], 1025, CE), ([30, 61, 17], 65, CE),
                                               ([40, 64, 3], 1027, MSE), ([52, 7], 300, CE), ([33, 16], 1030, MSE), ([33, 20], 70, CE)])
def test_forward_tail(dnlib, widths, batch, loss, in_place):
    acts = [TANH] * (len(widths) - 2) + [SOFTMAX if loss == CE else SIG]
    net, W, b, X = build(dnlib, widths, acts, loss, batch, 3)
    Xd = torch.from_numpy(X).cuda()
    out = Xd.view(-1)[:batch * widths[-1]].view(batch, widths[-1]) if in_place else torch.empty(batch, widths[-1], device="cuda")
    net.dn_forward(Xd, out)
    want, bound = forward_bound(X, W, b, acts, loss)
    err = np.abs(out.cpu().numpy() - want)
    assert np.all(err <= bound), float((err / bound).max())
    net.close()


# either side of the lines between one launch and several: four rows a workgroup (whole and ragged groups, rows of odd length, one
# layer), the largest last layers of one row a workgroup, squared error
@pytest.mark.parametrize("widths,batch,loss", [([24, 512, 10], 1025, CE), ([20, 1021, 16], 1030, CE), ([20, 1024, 16], 2048, CE), ([520, 7], 1101, CE),
                                               ([24, 511, 10], 1025, CE), ([12, 2048, 16], 768, CE), ([12, 2049, 16], 5, CE), ([8, 10923, 3], 3, CE),
                                               ([9, 1025, 3], 767, MSE), ([9, 257, 10], 512, MSE), ([9, 255, 10], 64, MSE), ([9, 1024, 16], 769, MSE)])
def test_forward_tail_lines(dnlib, widths, batch, loss):
    test_forward_tail(dnlib, widths, batch, loss, False)


# (more nets at once than there are places for their results; both forms of the kernel; after passes of another schedule)
def test_losses_of_many_small_nets(dnlib):
    nets = [build(dnlib, [4, 10, 3], [TANH, SOFTMAX], CE, 150, 5) for _ in range(70)]
    X = torch.from_numpy(nets[0][3]).cuda()
    y = torch.from_numpy((np.arange(150) % 3).astype(np.int32)).cuda()
    for lr, mu in ((0.05, 0.0), (0.05, 0.9)):
        losses = {(n[0].dn_train_epoch(X, y, 1, lr, mu), n[0].dn_train_epoch(X, y, 32, lr, mu), n[0].dn_evaluate(X, y, 50)[0])
                  for n in nets}
        assert len(losses) == 1
    assert len({n[0].dn_train_epoch(X, y, 1, 0.05, 0.0) for n in nets}) == 1
    for n in nets:
        n[0].close()
    again = [build(dnlib, [4, 10, 3], [TANH, SOFTMAX], CE, 150, 5)[0] for _ in range(2)]
    assert len({n.dn_train_epoch(X, y, 1, 0.05, 0.0) for n in again}) == 1
