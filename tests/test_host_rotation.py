"""The per-segment rotations of a plan at widths around the blocks that they
are built in (8 columns, 256 entries of a row): M's rows are orthonormal, the
rows of a segment span its eigenvectors, and the rotation is not the identity.
An FP32 entry of M is within 2^-25 of the FP64 one (|entry| <= 1), so a product
of two rows of D entries is within D 2^-25 2 / sqrt(D) by Cauchy-Schwarz of the
rounding errors against a unit row: 2 sqrt(D) 2^-25, and FP64 adds nothing
visible."""
import numpy as np
import pytest

import paper_2509_12086_amd as saq


@pytest.mark.parametrize("D,granularity", [(1, 1), (7, 7), (8, 8), (9, 9), (17, 1), (255, 16),
                                           (256, 64), (257, 257), (333, 16)])
def test_rotated_rows(D, granularity):
    rng = np.random.default_rng(D)
    V = np.linalg.qr(rng.standard_normal((D, D)))[0]
    lam = 4.0 * (1 - np.arange(D) / D) ** 2
    params = saq.PlanParams(bits_per_dim=4.0, granularity=granularity, max_width=0)
    p = saq.Plan.from_basis(np.zeros(D), V, lam, params)
    M = p.arrays()[0].astype(np.float64)
    tol = 2 * np.sqrt(D) * 2.0 ** -25 + 1e-12
    assert np.max(np.abs(M @ M.T - np.eye(M.shape[0]))) <= tol
    pos = row = 0
    for w, b in zip(p.widths, p.bits):
        if b > 0:
            R = M[row:row + w] @ V[:, pos:pos + w]      # the rotation itself
            assert np.max(np.abs(R @ R.T - np.eye(w))) <= 2 * tol
            if w > 1:
                assert np.max(np.abs(R - np.eye(w))) > 1e-3
            row += w
        pos += w
    assert row == M.shape[0]
