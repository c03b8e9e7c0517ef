"""The filter gradient that takes eight images to a lane, at the edges of its tiles, against sums in 64 bits of the same deltas."""
import numpy as np
import pytest
import torch

from paper_2001_04206_amd import dn
from parity_util import announce

pytestmark = pytest.mark.gpu

# A product is off by the terms its three-part numbers leave out, below 2^-22 of it; a sum of k terms rounds once a term, and the
# roundings of such sums grow with sqrt(k) (8 covers their spread over all elements); every element is held to
#   2^-22 sum|terms| + 8 2^-24 sqrt(k) rms(sum over the terms).
# (tests/test_schedule.py sees to it that conv_dw_images_kernel is what these run)
ODD = (121, 31, 30, 30, 63, 0)
LONG = (256, 64, 48, 24, 128, 1)
SHAPES = [   # B, Cin, H, W, Cout, pad
    (128, 32, 32, 32, 64, 1),    # whole tiles
    (133, 33, 21, 35, 65, 1),    # one channel in a second group on both sides, five of eight images, three of 16 columns
    ODD,                         # one channel short on both sides, one image in the last group, no padding
    (128, 64, 14, 14, 64, 1),    # strips of 14 columns, chunks that begin inside an image
    (40, 128, 23, 19, 128, 1),   # eight pairs of channel groups
    (264, 16, 28, 28, 60, 0),    # half of the input channels of a tile
]


def run(X, delta, pad):
    """dW, dbias of a linear layer: delta is dA."""
    (B, c_in, _, _), c_out = X.shape, delta.shape[1]
    W = torch.zeros(c_out, c_in, 3, 3, device="cuda")
    need = int(dn.lib().dn_conv_backward_workspace_bytes(B, c_in, X.shape[2], X.shape[3], c_out, 3, 3, 1, pad))
    dW, db, d = torch.full_like(W, np.nan), torch.full((c_out,), np.nan, device="cuda"), torch.empty_like(delta)
    dn.dn_conv_backward(X, W, delta, delta, d, None, dW, db, 1, pad, 0, workspace=torch.full((need,), 255, dtype=torch.uint8, device="cuda"))
    return dW, db


def sums(X, delta, pad):
    X, delta = X.double(), delta.double()
    out = torch.empty(delta.shape[1], X.shape[1], 3, 3, dtype=torch.float64, device="cuda")
    ho, wo = delta.shape[2:]
    P = torch.nn.functional.pad(X, (pad, pad, pad, pad))
    flat = delta.transpose(0, 1).reshape(delta.shape[1], -1)
    for u in range(3):
        for v in range(3):
            out[:, :, u, v] = flat @ P[:, :, u:u + ho, v:v + wo].transpose(0, 1).reshape(X.shape[1], -1).t().contiguous()
    return out


def check(X, delta, pad, dW, db):
    B, k = X.shape[0], delta.shape[0] * delta.shape[2] * delta.shape[3]
    want, size = sums(X, delta, pad) / B, sums(X.abs(), delta.abs(), pad) / B
    spread = (sums(X.double() ** 2, delta.double() ** 2, pad)).sqrt() / B
    bound = 2.0 ** -22 * size + 8 * 2.0 ** -24 * k ** 0.5 * spread
    assert ((dW.double() - want).abs() <= bound).all(), ((dW.double() - want).abs() / bound).max().item()
    d = delta.double()
    bias = 2.0 ** -22 * d.abs().sum((0, 2, 3)) / B + 8 * 2.0 ** -24 * k ** 0.5 * d.pow(2).sum((0, 2, 3)).sqrt() / B
    assert ((db.double() - d.sum((0, 2, 3)) / B).abs() <= bias).all()


def make(B, c_in, H, W, c_out, pad, seed=5):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(B, c_in, H, W, generator=gen, device="cuda"),
            torch.randn(B, c_out, H + 2 * pad - 2, W + 2 * pad - 2, generator=gen, device="cuda"))


@pytest.mark.parametrize("B,Cin,H,W,Cout,pad", SHAPES)
def test_filter_gradient(B, Cin, H, W, Cout, pad):
    announce("conv dW B=%d Cin=%d %dx%d Cout=%d pad=%d" % (B, Cin, H, W, Cout, pad))
    X, delta = make(B, Cin, H, W, Cout, pad)
    dW, db = run(X, delta, pad)
    check(X, delta, pad, dW, db)
    again = run(X, delta, pad)
    assert torch.equal(dW, again[0]) and torch.equal(db, again[1])


@pytest.mark.parametrize("shape", [LONG, SHAPES[0]])
def test_sums_of_one_sign(shape):
    """Sums of products of one sign, up to 3e5 of them: what an instruction that rounds its sums downwards loses adds up.  Here each sum of
    sixteen products begins at zero.  It is off by the roundings of its two or three last additions, 2^-23 of it at most (half of that in
    the mean, and for every other four pixels to the other side), and by the terms left out, 2^-25; additions to nearest do the rest.
    Bound: 2^-22 of the sum.  (Long sums on the instruction were 1.2e-6 off.)"""
    announce("conv dW of one sign %s" % (shape,))
    gen = torch.Generator(device="cuda").manual_seed(3)
    X, delta = (torch.rand(t.shape, generator=gen, device="cuda") for t in make(*shape))
    dW, _ = run(X, delta, shape[5])
    want = sums(X, delta, shape[5]) / shape[0]
    assert ((dW.double() - want).norm() / want.norm()).item() <= 2.0 ** -22


@pytest.mark.parametrize("scale_x,scale_d", [(1e-30, 1e30), (1e17, 1e18), (1e-12, 1e-10), (1e30, 1e-35)])
def test_numbers_of_all_sizes(scale_x, scale_d):
    """Also far apart in one image, and too small for three parts."""
    announce("conv dW scales %g %g" % (scale_x, scale_d))
    X, delta = make(*ODD)
    X, delta = X * scale_x, delta * scale_d
    delta[:, 7] *= 1e-4
    X[:, 3] *= 1e-6
    check(X, delta, 0, *run(X, delta, 0))


@pytest.mark.parametrize("exponent,last_bits", [(-109, 63), (-107, 15), (-106, 7), (-104, 1)])
@pytest.mark.parametrize("small", ["delta", "X"])
def test_numbers_whose_last_bits_are_subnormal(exponent, last_bits, small):
    """2^exponent (1 + j 2^-7 + last_bits 2^-23): the last bits by themselves are below 2^-126.  Taken for zero, they would make every product,
    all of one sign, 2^-17 too small at 2^-109, 2^-19 at 2^-107, 2^-20 at 2^-106."""
    announce("conv dW, %s of 2^%d" % (small, exponent))
    X, delta = (t.abs() + 0.5 for t in make(*ODD))
    tiny = lambda t: 2.0 ** exponent * (1 + (t * 100 % 128).floor() * 2.0 ** -7 + last_bits * 2.0 ** -23)
    X, delta = (X * 2.0 ** 70, tiny(delta)) if small == "delta" else (tiny(X), delta * 2.0 ** 70)
    check(X, delta, 0, *run(X, delta, 0))


@pytest.mark.parametrize("image,y,small", [(0, 0, "delta"), (60, 13, "X"), (120, 27, "delta"), (120, 29, "X")])
def test_one_number_too_small(image, y, small):
    """The workgroup that meets it begins again, wherever in its rows that is; all others keep their sums."""
    announce("conv dW, image %d row %d of %s too small" % (image, y, small))
    X, delta = make(*ODD)
    (delta if small == "delta" else X)[image, 5, y, 7] = 2.0 ** -115
    dW, db = run(X, delta, 0)
    check(X, delta, 0, dW, db)
    again = run(X, delta, 0)
    assert torch.equal(dW, again[0]) and torch.equal(db, again[1])


def test_not_finite():
    """A number that is not finite reaches the filters it meets, as it does on the fp32 instruction, and no other."""
    announce("conv dW not finite")
    X, delta = make(*ODD)
    delta, clean = delta.abs(), delta.abs()
    X[3, 5, 10, 10], X[40, 9, 12, 12], X[120, 20, 3, 11] = float("inf"), float("nan"), float("-inf")   # (meeting no column outside)
    dW, db = run(X, delta, 0)
    kind = lambda t: torch.stack([torch.isnan(t), t == float("inf"), t == float("-inf")])
    want = sums(X, delta, 0)
    assert torch.equal(kind(dW), kind(want))
    Y = X.clone()
    Y[:, [5, 9, 20]] = 0
    dW[:, [5, 9, 20]] = 0
    check(Y, clean, 0, dW, db)
    X, delta = make(*ODD)
    dW, _ = run(X.abs() * 3e19, delta.abs() * 3e19, 0)      # every product 1e39
    assert torch.isinf(dW).all()
