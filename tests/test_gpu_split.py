"""The contraction kernels that split fp32 operands into pairs of f16 numbers (tile shapes 13 to 16; 17 and 18 run the
same slices on the fp32 instruction): edges of tiles and slices, alignment, magnitudes far from one, operands whose
magnitude grows along k, large numbers beside small ones, infinities and NaN; every activation and update on them, and the
gradients of several layers of odd widths in one launch.  Reference: the same products in 64 bits, the bound on every
element following from the fp32 roundings of its own terms and the bits an operand keeps; the CPU checker for whole steps."""
import numpy as np
import pytest

import test_gpu_parity as parity
from paper_2001_04206_amd import synth

pytestmark = pytest.mark.gpu

LINEAR, MSE = 0, 0


@pytest.fixture(scope="module")
def dnlib():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2001_04206_amd import dn
    return dn


def products(dn, X, W, variant):
    """One linear layer: its outputs X W^T, gradient Delta^T X / B and input gradient Delta W, with the Delta they belong to."""
    import torch
    B, K = X.shape
    N = W.shape[0]
    net = dn.Net([K, N], [LINEAR], MSE, B)
    net.dn_set_params(1, W, np.zeros(N, np.float32))
    net.dn_set_option("gemm_variant", variant)
    Xd, y = torch.from_numpy(X).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda")
    out, dX = torch.empty((B, N), device="cuda"), torch.empty((B, K), device="cuda")
    net.dn_forward(Xd, out)
    net.dn_backward(y)
    net.dn_input_gradient(dX)
    G, g = net.dn_get_grads(1)
    delta = out.cpu().numpy().copy()
    delta[:, 0] -= 1.0
    return out.cpu().numpy(), G, g, dX.cpu().numpy(), delta


def close(got, A, B, scale, what):
    """got against scale * A B in 64 bits, every element within the roundings of its own terms: at most one per pair of
    terms and one per addition of at most 32 partial sums, 2^-22 for either operand.  Nothing is allowed for the largest
    numbers of its row or column."""
    A, B = A.astype(np.float64), B.astype(np.float64)
    bound = abs(scale) * ((A.shape[1] / 2 + 44) * 2.0 ** -24 + 2.0 ** -21) * (np.abs(A) @ np.abs(B))
    err = np.abs(got - scale * (A @ B))
    assert np.all(err <= bound + 1e-44), "%s: %g times the bound" % (what, np.max(err / (bound + 1e-44)))


def check(dn, X, W, variant):
    out, G, g, dX, delta = products(dn, X, W, variant)
    close(out, X, W.T, 1.0, "forward")
    close(G, delta.T, X, 1.0 / X.shape[0], "gradient")
    close(g[:, None], delta.T, np.ones((X.shape[0], 1), np.float32), 1.0 / X.shape[0], "bias gradient")
    close(dX, delta, W, 1.0, "input gradient")


# batch, inputs, outputs: whole tiles; one past and one short of tiles and slices; less than one slice; a long sum that
# workgroups share; 16-byte pieces that end inside a slice
SHAPES = [(64, 128, 64), (65, 129, 33), (63, 127, 95), (3, 5, 17), (1, 40, 32), (128, 2064, 96), (70, 2051, 130), (36, 20, 68)]


@pytest.mark.parametrize("variant", [13, 14, 15, 16, 17, 18])
@pytest.mark.parametrize("shape", SHAPES)
def test_products_match_64_bits(dnlib, shape, variant):
    B, K, N = shape
    rng = np.random.default_rng(B * 1000 + K)
    check(dnlib, rng.standard_normal((B, K), dtype=np.float32), rng.standard_normal((N, K), dtype=np.float32), variant)


@pytest.mark.parametrize("variant", [13, 15])
@pytest.mark.parametrize("sx,sw", [(1e-30, 1e25), (1e30, 1e-30), (1e-20, 1e-10), (3e4, 7e4), (1e-7, 1.0)])
def test_magnitudes(dnlib, sx, sw, variant):
    rng = np.random.default_rng(5)
    X = (rng.standard_normal((66, 260)) * sx).astype(np.float32)
    W = (rng.standard_normal((70, 260)) * sw).astype(np.float32)
    check(dnlib, X, W, variant)


@pytest.mark.parametrize("variant", [13, 14, 15, 16])
@pytest.mark.parametrize("order", ["zeros first", "growing", "shrinking", "one large row"])
def test_magnitude_changes_along_k(dnlib, order, variant):
    rng = np.random.default_rng(6)
    X = rng.standard_normal((40, 600)).astype(np.float32)
    W = rng.standard_normal((72, 600)).astype(np.float32)
    if order == "zeros first":
        X[:, :300] = 0.0
        X[:, 300:] *= np.float32(1e-6)
    elif order == "one large row":
        X[7] *= np.float32(1e12)
    else:
        steps = np.exp2(np.linspace(-40, 40, 600)).astype(np.float32)
        X *= steps if order == "growing" else steps[::-1]
    check(dnlib, X, W, variant)


@pytest.mark.parametrize("variant", [13, 14, 15, 16, 17])
def test_infinities_and_nan(dnlib, variant):
    rng = np.random.default_rng(7)
    X = rng.standard_normal((70, 100)).astype(np.float32)
    W = rng.standard_normal((40, 100)).astype(np.float32)
    X[3, 10], X[65, 99], X[20, 0], X[5, 50] = np.inf, -np.inf, np.nan, np.float32(3.4e38)
    W[:, 50] = np.sign(W[:, 50]) * np.float32(0.5)
    out, G, _, _, _ = products(dnlib, X, W, variant)
    with np.errstate(invalid="ignore", over="ignore"):
        want = X.astype(np.float64) @ W.astype(np.float64).T
    assert np.array_equal(np.isnan(out), np.isnan(want)) and np.array_equal(np.isinf(out), np.isinf(want))
    assert np.array_equal(np.sign(out[[3, 65]]), np.sign(want[[3, 65]]))
    rows = [r for r in range(70) if r not in (3, 65, 20, 5)]
    assert np.allclose(out[rows], want[rows], rtol=0, atol=2e-4) and np.allclose(out[5] / want[5], 1.0, rtol=1e-5)
    assert np.isnan(G).all()   # every gradient has sample 20, whose deltas are NaN


def wide_products(dn, big, variant):
    """Numbers `big` that meet only zeros, so no result holds them: feature 9 has zero weights, sample 4 has feature 30 large
    and a delta of zero in every output but one, output 70 has zero weights and a large bias."""
    import torch
    B, K, N = 130, 200, 110
    rng = np.random.default_rng(11)
    X, W = rng.standard_normal((B, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    bias = np.zeros(N, np.float32)
    W[:, 9] = 0.0
    X[:, 9] = big
    X[4] = 0.0
    X[4, 30] = big
    W[:, 30] = 0.0
    W[70] = 0.0
    bias[70] = big
    net = dn.Net([K, N], [LINEAR], MSE, B)
    net.dn_set_params(1, W, bias)
    net.dn_set_option("gemm_variant", variant)
    Xd, y = torch.from_numpy(X).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda")
    out, dX = torch.empty((B, N), device="cuda"), torch.empty((B, K), device="cuda")
    net.dn_forward(Xd, out)
    net.dn_backward(y)
    net.dn_input_gradient(dX)
    G, _ = net.dn_get_grads(1)
    out, dX = out.cpu().numpy(), dX.cpu().numpy()
    delta = out.copy()
    delta[:, 0] -= 1.0
    return X, W, bias, out, G, dX, delta


@pytest.mark.parametrize("variant", [-1, 13, 14, 15, 16, 17])
@pytest.mark.parametrize("big", [1e9, 1e12, 1e15, 1e22, 1e30])
def test_large_numbers_against_zeros(dnlib, big, variant):
    X, W, bias, out, G, dX, delta = wide_products(dnlib, np.float32(big), variant)
    others = np.arange(110) != 70
    close(out[:, others], X, W[others].T, 1.0, "forward")
    assert np.all(out[:, 70] == bias[70])
    close(G[others], delta[:, others].T, X, 1.0 / X.shape[0], "gradient")   # (row 70 overflows)
    close(dX, delta, W, 1.0, "input gradient")


@pytest.mark.parametrize("variant", [13, 14, 15, 16])
@pytest.mark.parametrize("shape", [(130, 200, 110), (129, 203, 111), (1300, 64, 40), (2100, 131, 33)])
def test_slices_left_for_fp32(dnlib, shape, variant):
    """Numbers of very different size along k: some slices, a run of them, or from one on all go to the fp32 instruction;
    more slices than a wave counts one by one."""
    B, K, N = shape
    rng = np.random.default_rng(B)
    for part in ("one sample in forty", "a tenth", "the second half", "all"):
        X, W = rng.standard_normal((B, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
        rows = {"one sample in forty": slice(5, None, 40), "a tenth": slice(B // 3, B // 3 + B // 10),
                "the second half": slice(B // 2, None), "all": slice(None)}[part]
        X[rows] *= (10.0 ** rng.uniform(-14, 0, X[rows].shape)).astype(np.float32)
        out, G, g, dX, delta = products(dnlib, X, W, variant)
        close(out, X, W.T, 1.0, part + ": forward")
        close(G, delta.T, X, 1.0 / B, part + ": gradient")
        close(g[:, None], delta.T, np.ones((B, 1), np.float32), 1.0 / B, part + ": bias gradient")
        close(dX, delta, W, 1.0, part + ": input gradient")


@pytest.mark.parametrize("variant", [13, 14, 15, 16, 17, 18])
@pytest.mark.parametrize("widths,acts,loss,B", parity.SMALL_CASES)
def test_one_step_small_and_ragged(dnlib, widths, acts, loss, B, variant):
    parity.test_one_step_small_and_ragged(dnlib, widths, acts, loss, B, variant)


@pytest.mark.parametrize("variant", [13, 14, 15, 17])
@pytest.mark.parametrize("widths,acts,loss,B", parity.SPLIT_K_CASES)
def test_one_step_split_k(dnlib, widths, acts, loss, B, variant):
    parity.test_one_step_split_k(dnlib, widths, acts, loss, B, variant, 1)


@pytest.mark.parametrize("variant", [13, 14, 15, 16, 17, 18])
@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_updates_in_the_epilogue(dnlib, mu, variant):
    """Plain, last-step and momentum updates with a forced tile shape, ragged in every direction and with a short last batch."""
    B = 101
    w = synth.make("forced", [203, 131, 97, 5], [parity.TANH, parity.SIG, parity.SOFTMAX], parity.CE, n_samples=3 * B - 7,
                   features="normal", init="xavier_uniform", batch=B, lr=0.05, momentum=mu, seed=31)
    net, o = parity.make_pair(dnlib, w, B)
    net.dn_set_option("gemm_variant", variant)
    X, y = parity.to_dev(w)
    for _ in range(2):
        got = net.dn_train_epoch(X, y, B, w.lr, mu)
        ref, _ = o.train_epoch(w.X, w.labels, B, w.lr, mu)
        assert abs(got - ref) <= parity.EPOCH_TOL * abs(ref)
    for got, ref in zip(net.get_all(), o.get_params()):
        for l in range(net.L):
            parity.assert_close(got[l], ref[l], parity.EPOCH_TOL, "layer %d" % (l + 1))
    net.close()


# odd widths, read through registers: 306 tiles of 64 x 64 (four waves) and 910 (two), for sums in f16 pairs and short ones
@pytest.mark.parametrize("widths", [[517, 1029, 519, 21], [1621, 1623, 517, 37]])
@pytest.mark.parametrize("B,mu", [(101, 0.9), (101, 0.0), (41, 0.9)])
def test_merged_gradients_of_odd_widths(dnlib, widths, B, mu):
    parity.test_merged_backward_launches(dnlib, widths, [parity.TANH, parity.TANH, parity.SOFTMAX], parity.CE, B, mu, 1)


# either side of the line between the fp32 instruction and pairs, as the library picks: one k split and several, gradients
# small and large, the launches that join a narrow layer's gradient with a delta product and several gradients
@pytest.mark.parametrize("B,K,N", [(100, 184, 300), (100, 185, 300), (40, 1288, 520), (40, 1289, 520), (184, 96, 300), (185, 97, 300),
                                   (92, 2560, 1024), (93, 2560, 1024), (2048, 96, 384), (2048, 95, 384)])
def test_either_side_of_the_line(dnlib, B, K, N):
    rng = np.random.default_rng(B + K)
    check(dnlib, rng.standard_normal((B, K), dtype=np.float32), rng.standard_normal((N, K), dtype=np.float32), -1)


@pytest.mark.parametrize("widths,B", [([516, 1040, 184, 12], 184), ([516, 1040, 188, 12], 188), ([1028, 1040, 1100, 24], 184), ([1028, 1040, 1100, 24], 188)])
def test_joined_launches_either_side_of_the_line(dnlib, widths, B):
    parity.test_merged_backward_launches(dnlib, widths, [parity.TANH, parity.RELU, parity.SOFTMAX], parity.CE, B, 0.9, 1)


def test_short_sums_lose_nothing(dnlib):
    """Fewer than 184 terms a run of one tile: no further from 64 bits than fp32 sums in 8 runs of 23 terms (pairs are: 1.0e-7)."""
    import torch
    torch.manual_seed(0)
    X, W = torch.randn(512, 128, device="cuda").relu_(), torch.randn(1024, 128) * 0.125
    net = dnlib.Net([128, 1024], [LINEAR], MSE, 512)
    net.dn_set_params(1, W.numpy(), np.zeros(1024, np.float32))
    out = torch.empty(512, 1024, device="cuda")
    net.dn_forward(X, out)
    want = X.double() @ W.cuda().double().t()
    assert ((out.double() - want).norm() / want.norm()).item() < 8.5e-8
