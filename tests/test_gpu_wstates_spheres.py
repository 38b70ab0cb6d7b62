"""Transformed states at both ends of the radii that one orbital window takes, on the
36 and 40 grids: the smallest and the largest sphere of the largest index K.
Tolerance as in tests/test_gpu_wstates_forms.py.
"""
import math

import pytest

from tests import test_gpu_wstates_forms as forms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ko,r2", [(36, 11, 121), (36, 11, 143), (36, 12, 144), (36, 12, 168),
                                     (40, 13, 169), (40, 13, 195)])
def test_spheres_of_a_window(n, ko, r2):
    L = 0.55 * n
    half_b2 = 0.5 * (2 * math.pi / L) ** 2
    forms.test_orbital_windows_vs_oracle(n, L, half_b2 * (r2 + 0.5), half_b2 * 100.25, ko)
