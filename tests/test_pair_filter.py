"""The bounds of the pair search's matrix products (csrc/pairs.hpp, home_operand and
group_pairs): every pair within reach has to come out a hit.

In units of the reach, a home particle at distance at most H from its leaf's centre
with reach T and a candidate within T of it (H + T at most kHalfFar; beyond, every
candidate is listed).  Taken to halves towards zero a coordinate loses up to 2^-10 of
itself, or 2^-14 where it has no normal half, so the two are up to
d = 2^-10 (2 H + T) + 2 sqrt(3) 2^-14 further apart; the sums are single precision,
each addition wrong by up to one unit in the last place (2^-23 of its result, however
the matrix cores round).  The widened threshold has to hold both.
"""
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_04488_amd", "csrc",
                   "pairs.hpp")


def _constants():
    text = open(SRC).read()
    m = re.search(r"constexpr float kHalfRel = ([\d.e-]+)f, kHalfAbs = ([\d.e-]+)f, kHalfFar = ([\d.]+)f", text)
    return (float(v) for v in m.groups())


@pytest.mark.parametrize("criterion", ["home particle's reach", "candidate's reach"])
def test_thresholds_cover_halves_and_single_precision(criterion):
    rel, ab, far = _constants()
    H, T = np.meshgrid(np.r_[0, np.logspace(-4, np.log10(far), 400)], np.r_[0, np.logspace(-6, np.log10(far), 400)],
                       indexing="ij")
    inside = H + T <= far
    u = 2.0 ** -23
    d = 2.0 ** -10 * (2 * H + T) + 2 * np.sqrt(3) * 2.0 ** -14
    xj = H + T
    if criterion == "home particle's reach":
        Tw = T * (1 + rel) + 2 * rel * H + ab
        room = Tw ** 2 - (T + d) ** 2
        wrong = 0.0
    else:   # |x_j|^2 - T_j^2 goes through a half, rounded towards zero
        Tw = T * (1 + 2 * rel) + 2 * rel * H + ab
        W = Tw ** 2 * (1 + rel)
        room = W * (1 - 2.0 ** -10) - (T + d) ** 2
        wrong = 3 * u * xj ** 2
    # |x_i|^2 (three sums), Tw^2 from a square root and four products, their
    # difference, and the four sums of the product
    largest = xj ** 2 + 2 * H * xj + np.maximum(H ** 2, Tw ** 2)
    wrong = wrong + 3 * u * H ** 2 + 9 * u * Tw ** 2 + u * np.maximum(H ** 2, Tw ** 2) + 4 * u * largest
    assert np.all((room > wrong)[inside])


def test_halves_hold_what_is_tested():
    """-2 x_i and the largest |x_j|^2 that is not dropped are finite halves."""
    rel, ab, far = _constants()
    assert np.isfinite(np.float16(2 * far)) and far ** 2 <= 4e4 and np.isfinite(np.float16(4e4))
