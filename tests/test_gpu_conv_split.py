"""3 x 3 convolutions on the f16 matrix instruction: edges of pixel tiles, channel stages and output-channel tiles,
numbers of very different magnitudes, infinities and NaN.  Reference: torch's CPU convolution in 64 bits; the bound on
every element follows from the roundings of its own terms (one or two per sixteen channels and tap; sixteen times as many
where stages are left to the fp32 instruction) and the 22 bits an operand keeps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LINEAR = 0


@pytest.fixture(scope="module")
def dnlib():
    from paper_2001_04206_amd import dn
    assert torch.cuda.is_available(), "these tests need the GPU"
    dn.lib()
    return dn


def run(dn, X, W, dA, pad):
    dev = [torch.from_numpy(a).cuda() for a in (X, W, dA)]
    bias = torch.zeros(W.shape[0], device="cuda")
    Y = torch.empty(dA.shape, device="cuda")
    delta, dX, dW, db = torch.empty_like(Y), torch.empty_like(dev[0]), torch.empty_like(dev[1]), torch.empty_like(bias)
    dn.dn_conv_forward(dev[0], dev[1], bias, Y, 1, pad, LINEAR)
    dn.dn_conv_backward(dev[0], dev[1], Y, dev[2], delta, dX, dW, db, 1, pad, LINEAR)
    return Y.cpu().numpy(), dX.cpu().numpy()


def reference(X, W, dA, pad):
    X, W, dA = (torch.from_numpy(a).double() for a in (X, W, dA))
    conv, back = torch.nn.functional.conv2d, torch.nn.functional.conv_transpose2d
    return conv(X, W, padding=pad).numpy(), back(dA, W, padding=pad).numpy()


def close(got, want, magnitude, terms, floor, what):
    err, bound = np.abs(got - want), (2 * (terms / 16 + 9) * 2.0 ** -24 + 2.0 ** -21) * magnitude + floor
    assert np.all(err <= bound), "%s: %g times the bound" % (what, np.max(err / bound))


def check(dn, X, W, dA, pad):
    Y, dX = run(dn, X, W, dA, pad)
    wantY, wantdX = reference(X, W, dA, pad)
    magY, magdX = reference(np.abs(X), np.abs(W), np.abs(dA), pad)
    close(Y, wantY, magY, 9 * X.shape[1], 0.0, "forward")
    close(dX, wantdX, magdX, 9 * W.shape[0], 0.0, "input gradient")


def draw(B, ci, h, w, co, pad, seed=3):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((B, ci, h, w), dtype=np.float32), rng.standard_normal((co, ci, 3, 3), dtype=np.float32),
            rng.standard_normal((B, co, h + 2 * pad - 2, w + 2 * pad - 2), dtype=np.float32))


@pytest.mark.parametrize("B,ci,h,w,co,pad", [(2, 32, 32, 32, 64, 1), (3, 33, 33, 35, 70, 1), (2, 47, 9, 31, 32, 0),
                                             (130, 32, 16, 16, 32, 1), (2, 32, 16, 16, 48, 2), (1, 40, 17, 14, 97, 1)])
def test_sizes(dnlib, B, ci, h, w, co, pad):
    check(dnlib, *draw(B, ci, h, w, co, pad), pad)


@pytest.mark.parametrize("case", ["tiny", "huge", "stages of growing size", "one large pixel", "one pixel beyond all others"])
def test_magnitudes(dnlib, case):
    X, W, dA = draw(2, 64, 18, 34, 40, 1)
    if case == "tiny":
        X *= np.float32(1e-25)
        dA *= np.float32(1e-20)
    elif case == "huge":
        X *= np.float32(1e25)
        W *= np.float32(1e-20)
    elif case == "stages of growing size":
        X *= np.exp2(np.arange(64) // 16 * 12).astype(np.float32)[None, :, None, None]
    elif case == "one large pixel":
        X[0, 5, 9, 9] = 1e5
    else:   # every other number of the tile would lose its bits: summed in fp32 again
        X[0, 5, 9, 9], dA[1, 3, 4, 20] = 1e30, 1e28
    Y, dX = run(dnlib, X, W, dA, 1)
    wantY, wantdX = reference(X, W, dA, 1)
    magY, magdX = reference(np.abs(X), np.abs(W), np.abs(dA), 1)
    close(Y, wantY, magY, 9 * 64 * 16, 0.0, "forward")
    close(dX, wantdX, magdX, 9 * 40 * 16, 0.0, "input gradient")


def test_infinities_and_nan(dnlib):
    X, W, dA = draw(2, 40, 18, 34, 40, 1)
    X[0, 5, 9, 9], X[1, 0, 0, 0], X[1, 39, 17, 33] = np.inf, np.nan, -np.inf
    Y, _ = run(dnlib, X, W, dA, 1)
    want, _ = reference(X, W, dA, 1)
    assert np.array_equal(np.isnan(Y), np.isnan(want)) and np.array_equal(np.isposinf(Y), np.isposinf(want))
    fine = np.isfinite(want)
    assert np.array_equal(np.isfinite(Y), fine) and np.allclose(Y[fine], want[fine], rtol=0, atol=1e-4)


@pytest.mark.parametrize("small", [1e-8, 1e-11, 1e-13, 1e-16, 1e-30])
@pytest.mark.parametrize("case", ["later channels", "part of an image", "one output channel", "one input channel's filters",
                                  "beside one weight", "beside one pixel"])
def test_small_numbers_beside_large_ones(dnlib, case, small):
    """Every output is within the roundings of its own terms, however small they are beside other numbers of the tile."""
    X, W, dA = draw(2, 64, 18, 34, 40, 1)
    small = np.float32(small)
    if case == "later channels":          # the large channels meet zero weights, the first one's weights meet zeros
        X[:, 16:] *= small
        X[:, 0] = 0.0
        W[:, 1:16] = 0.0
        dA[:, 16:] *= small
        dA[:, 0] = 0.0
        W[1:16] = 0.0
    elif case == "part of an image":
        X[:, :, :, :12] *= small
        dA[:, :, :, :12] *= small
    elif case == "one output channel":    # and, in the input gradient, its part of every sum alone
        W[7] *= small
        dA[0] = 0.0
        dA[0, 7] = draw(1, 64, 18, 34, 40, 1, seed=4)[2][0, 7]
    elif case == "beside one weight":     # of a later stage, which meets zeros
        W[37, 20], X[:, 20], dA[:, 37] = 1.0 / small, 0.0, 0.0
    elif case == "beside one pixel":
        X[0, 20, 9, 9], W[:, 20] = 1.0 / small, 0.0
        dA[1, 18, 3, 30], W[18] = 1.0 / small, 0.0
    else:
        W[:, 9] *= small
        X[1] = 0.0
        X[1, 9] = draw(1, 64, 18, 34, 40, 1, seed=4)[0][0, 9]
    Y, dX = run(dnlib, X, W, dA, 1)
    wantY, wantdX = reference(X, W, dA, 1)
    magY, magdX = reference(np.abs(X), np.abs(W), np.abs(dA), 1)
    close(Y, wantY, magY, 9 * 64 * 16, 1e-44, "forward")
    close(dX, wantdX, magdX, 9 * 40 * 16, 1e-44, "input gradient")


def test_more_stages_than_are_counted_one_by_one(dnlib):
    """1040 and 1060 channels are 65 and 67 stages, counted in pairs: some are left alone, some with the one after them, and
    from the last quarter on all of them."""
    X, W, dA = draw(1, 1040, 9, 14, 1060, 1)
    for c in (20, 320, 336, 700):
        X[:, c] *= np.float32(1e-12)
        dA[:, c] *= np.float32(1e-12)
    check(dnlib, X, W, dA, 1)
    X[:, 100::16] *= np.float32(1e-12)
    dA[:, 100::16] *= np.float32(1e-12)
    Y, dX = run(dnlib, X, W, dA, 1)
    wantY, wantdX = reference(X, W, dA, 1)
    magY, magdX = reference(np.abs(X), np.abs(W), np.abs(dA), 1)
    close(Y, wantY, magY, 9 * 1040 * 16, 0.0, "forward")
    close(dX, wantdX, magdX, 9 * 1060 * 16, 0.0, "input gradient")
