"""The 64 x 64 tile of eight waves (tile shape 19) and the sizes at which the automatic choice turns to it: the checks of
test_gpu_split on it, products against 64 bits with the bound on every element that follows from its own terms."""
import numpy as np
import pytest

import test_gpu_split as split
from test_gpu_split import dnlib  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", split.SHAPES + [(64, 1024, 64), (65, 1153, 190)])
def test_products_match_64_bits(dnlib, shape):
    split.test_products_match_64_bits(dnlib, shape, 19)


# batch, inputs, outputs: forward products of 128, 129, 256 and 257 tiles; of 65 and more over k = 3071 and 3072; gradients of
# 127, 128, 256 and 257 tiles over k = 256 and 257
@pytest.mark.parametrize("shape", [(512, 200, 1024), (130, 96, 2752), (1024, 300, 1024), (64, 100, 16448), (320, 3071, 830), (320, 3072, 830),
                                   (257, 1024, 507), (256, 1024, 512), (257, 1024, 512), (257, 1023, 1021), (300, 1028, 1030)])
def test_the_rule(dnlib, shape):
    split.test_products_match_64_bits(dnlib, shape, -1)


@pytest.mark.parametrize("order", ["zeros first", "growing", "shrinking", "one large row"])
def test_magnitude_changes_along_k(dnlib, order):
    split.test_magnitude_changes_along_k(dnlib, order, 19)


def test_infinities_and_nan(dnlib):
    split.test_infinities_and_nan(dnlib, 19)


@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_updates_in_the_epilogue(dnlib, mu):
    split.test_updates_in_the_epilogue(dnlib, mu, 19)
