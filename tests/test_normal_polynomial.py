"""The a-trous levels' polynomial for the normal weight's logarithm."""

import os
import re

import numpy as np

from paper_2312_06827_amd import _build as B


def test_polynomial_against_the_logarithm():
    """kNormalPoly against log2(1 - s2/2) / s2 in binary64, at the bound that
    its comment states (below half a unit of binary32, 3e-8)."""
    text = open(os.path.join(B.CSRC, "sv_internal.h")).read()
    q = [float(v) for v in re.search(r"kNormalPoly\[5\] = \{([^}]*)\}", text).group(1).split(",")]
    assert len(q) == 5 and all(v < 0 for v in q)  # all negative: no clamp needed
    s2 = np.linspace(0.0, 0.22, 100001)[1:]
    exact = np.log1p(-s2 / 2) / np.log(2) / s2
    err = np.abs(np.polyval(q[::-1], s2) / exact - 1)
    assert err.max() <= 1.4e-8
    # what 0.22 means as a weight, for the two exponents the comment names
    assert abs((1 - 0.11) ** 128 / 3.3e-7 - 1) < 0.02
    assert abs((1 - 0.11) ** 96 / 1.4e-5 - 1) < 0.02
