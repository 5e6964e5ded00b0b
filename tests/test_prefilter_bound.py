"""The error constants of the assignment's pre-filter (csrc/cluster.h) against what its two-term bf16 splits and its
additions can lose, element by element (CPU only): a label it settles is proved only if the constants cover that."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U = 2.0 ** -24          # one float32 addition, relative to the sum of magnitudes


def to_bf16(x):
    """float32 -> nearest bf16 (ties to even), as float32."""
    u = x.view(np.uint32)
    return ((u + np.uint32(0x7fff) + ((u >> np.uint32(16)) & np.uint32(1))) & np.uint32(0xffff0000)).view(np.float32)


def two_terms():
    """Largest lower term and largest remainder of the two-term split, relative to the element: one whole binade."""
    x = (np.uint32(0x3f800000) + np.arange(1 << 23, dtype=np.uint32)).view(np.float32)
    hi = to_bf16(x)
    lo = to_bf16(x - hi)
    return float((np.abs(lo) / x).max()), float((np.abs((x - hi) - lo) / x).max())


def fast_eps(token_type):
    text = open(os.path.join(ROOT, "paper_2603_18636_amd", "csrc", "cluster.h")).read()
    return float(re.search(r"fast_eps<%s>\(\) \{ return ([-+.0-9e]+)f; \}" % token_type, text).group(1))


@pytest.mark.parametrize("token_type,products", [("uint16_t", 2), ("float", 3)])
def test_margin_constant_covers_the_split_and_the_additions(token_type, products):
    low, left = two_terms()
    assert 0.9 * 2.0 ** -8 < low <= 2.0 ** -8 and 0.9 * 2.0 ** -17 < left <= 2.0 ** -17
    error = left                                                # of W, bf16 tokens being exact
    if token_type == "float":
        error += left * (1.0 + 2 * low) + low * low             # of the token; the product of the lower terms is left out
    error += products * 128 * U                                 # d <= 128
    error += 15 * 2.0 ** -23                                    # the place in a score's last four bits
    norms = 1.0 + 2.0 ** -15                                    # 128 squares and a root in float32
    assert error * norms <= fast_eps(token_type), (error, fast_eps(token_type))
