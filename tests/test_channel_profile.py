"""The channel profile's velocity of a node, j / rho - gx / 2, is rounded once."""
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_2504_14494_amd import lbm


@pytest.mark.gpu
def test_velocity_of_one_column_is_rounded_once():
    gen = np.random.default_rng(11)
    n, gx = 4096, np.float32(2e-4)
    g = np.zeros((n, 9, 1), np.float32)
    g[:, 0, 0], g[:, 1, 0] = gen.uniform(-0.1, 0.1, n), gen.uniform(-0.05, 0.05, n)
    prof = lbm.lbm_channel_profile(torch.as_tensor(g, device="cuda"), float(gx)).cpu().numpy()
    j = g[:, 1, 0].astype(np.float64)
    inv = 1.0 / (1.0 + (g[:, 0, 0].astype(np.float64) + j))
    half = Fraction(float(gx)) / 2
    ref = np.array([float(Fraction(a) * Fraction(b) - half) for a, b in zip(j, inv)])
    assert (prof == ref).all(), np.mean(prof == ref)
