"""The classifier's joined launches (pooling backward with the convolution's delta, all filter updates at once) give the
bits of the separate calls: windows of two and three that tile the image, windows that do not, no pooling; every
activation; with and without momentum; more vectors than one update launch holds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LINEAR, SIGMOID, TANH, RELU, SOFTMAX = 0, 1, 2, 3, 4


@pytest.fixture(scope="module")
def dn():
    from paper_2001_04206_amd import dn
    assert torch.cuda.is_available(), "these tests need the GPU"
    dn.lib()
    return dn


@pytest.mark.parametrize("momentum", [0.0, 0.9])
@pytest.mark.parametrize("h,w,blocks", [
    (12, 16, [(9, 3, 1, 1, RELU, 2, 2)]),                                   # pairs
    (18, 9, [(5, 3, 1, 1, TANH, 3, 3)]),                                    # windows of three
    (11, 13, [(6, 3, 1, 1, SIGMOID, 2, 2)]),                                # a row and a column left over: separate calls
    (16, 14, [(7, 3, 1, 1, RELU, 2, 2), (40, 3, 1, 1, TANH, 0, 0), (33, 3, 1, 1, RELU, 2, 1)]),
    (6, 6, [(3, 1, 1, 0, LINEAR, 0, 0)] * 9),                               # eighteen vectors
])
def test_epoch_is_the_separate_calls(dn, h, w, blocks, momentum):
    B, c, lr, classes = 5, 3, 0.05, 4
    rng = np.random.default_rng(h * 100 + w)
    X = torch.from_numpy(rng.standard_normal((2 * B, c, h, w), dtype=np.float32)).cuda()
    y = torch.from_numpy(rng.integers(0, classes, 2 * B).astype(np.int32)).cuda()
    cnn = dn.Cnn(c, h, w, blocks, [classes], [SOFTMAX], 1, B)
    params, cin = [], c
    for i, blk in enumerate(blocks):
        W = (rng.standard_normal((blk[0], cin, blk[1], blk[1])) * 0.4).astype(np.float32)
        b = (rng.standard_normal(blk[0]) * 0.1).astype(np.float32)
        cnn.dn_cnn_set_filters(i, W, b)
        params.append([torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda()])
        cin = blk[0]
    Wd, bd = (rng.standard_normal((classes, cnn.flat)) * 0.1).astype(np.float32), np.zeros(classes, np.float32)
    cnn.dense.set_all([Wd], [bd])
    dense = dn.Net([cnn.flat, classes], [SOFTMAX], 1, B)
    dense.set_all([Wd], [bd])
    vel = [[torch.zeros_like(t) for t in p] for p in params]
    cnn.dn_cnn_train_epoch(X, y, B, lr, momentum)
    for s in (0, B):
        a, kept = X[s:s + B].contiguous(), []
        for blk, (W, b) in zip(blocks, params):
            side = lambda n: n + 2 * blk[3] - blk[1] + 1
            Y = torch.empty((B, blk[0], side(a.shape[2]), side(a.shape[3])), device="cuda")
            dn.dn_conv_forward(a, W, b, Y, 1, blk[3], blk[4])
            P = Y
            if blk[5]:
                P = torch.empty((B, blk[0], (Y.shape[2] - blk[5]) // blk[6] + 1, (Y.shape[3] - blk[5]) // blk[6] + 1), device="cuda")
                dn.dn_maxpool_forward(Y, P, blk[5], blk[6])
            kept.append((a, Y, P))
            a = P
        dense.dn_forward(a.reshape(B, -1))
        dense.dn_backward(y[s:s + B].contiguous())
        back = torch.empty_like(a)
        dense.dn_input_gradient(back.view(B, -1))
        grads = []
        for i in range(len(blocks) - 1, -1, -1):
            (a, Y, P), blk, (W, b) = kept[i], blocks[i], params[i]
            dY = back
            if blk[5]:
                dY = torch.empty_like(Y)
                dn.dn_maxpool_backward(Y, back, dY, blk[5], blk[6])
            delta, dX, dW, db = torch.empty_like(Y), torch.empty_like(a), torch.empty_like(W), torch.empty_like(b)
            dn.dn_conv_backward(a, W, Y, dY, delta, dX if i else None, dW, db, 1, blk[3], blk[4])
            back, grads = dX, [(dW, db)] + grads
        dense.dn_update(lr, momentum)
        for p, g, v in zip(params, grads, vel):
            for k in range(2):
                dn.dn_sgd_step(p[k], g[k], v[k] if momentum else None, lr, momentum)
    for i, p in enumerate(params):
        W, b = cnn.dn_cnn_get_filters(i)
        assert np.array_equal(W, p[0].cpu().numpy()) and np.array_equal(b, p[1].cpu().numpy()), "block %d" % i
