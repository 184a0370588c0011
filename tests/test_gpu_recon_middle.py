"""The middle cell of an odd number of theta cells is its own partner (q = Q - 1 - q)
in the series products; its value comes from one place only.

For Q = 49 a Gamma with the single element (49, 49) makes it visible: cos(49 theta)
vanishes at every midpoint, and what is left of the table's cosine at the middle is
2/pi cospi(fl(49 fl(1/98))) = 2^-53 (49 fl(1/98) is half an ulp short of 1/2), which
enters E + O with its sign and E - O with the other one.  The difference of the sums
at two chemical potentials inside the middle cell holds that cell alone; all cells
have terms of the same size, 48 of them, so the difference is exact to some 1e-14 of
it (1e-9 allowed).  Several energies (frequencies) and repeats: every one gives the
same bits.
"""
import numpy as np
import pytest

from oracle import cond as ocond

pytestmark = pytest.mark.gpu

Q = M0 = 49
E0, E1, ETA, OPN = -7.0, 9.0, 0.3, 30.0
DE = 8.0


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _setup():
    G = np.zeros((M0 + 1, M0 + 1), dtype=complex)
    G[M0, M0] = 1.0
    x = M0 * (1.0 / (2.0 * Q))
    assert 0.5 - x == 2.0 ** -54
    D = 2.0 / np.pi * np.sin(np.pi * (0.5 - x))
    h = np.pi / Q
    mu = np.cos(h * np.array([24.1, 24.9])) * DE + 0.5 * (E0 + E1)
    return G, D, h, mu


def test_bastin_middle_cell(K):
    G, D, h, mu = _setup()
    g = ocond.cpgf_derivative(M0 + 1, np.array([0.0]), ETA / DE, +1)[0, M0]
    want = 2.0 * np.pi * OPN / DE ** 2 * 0.8 * h * 2.0 * D * g.imag
    runs = [K.reconstruct_sigma_bastin(G, np.tile(mu, 8), E0, E1, ETA, OPN, n_theta=Q) for _ in range(5)]
    for s in runs:
        assert np.array_equal(s, runs[0])
    assert abs((runs[0][0] - runs[0][1]) - want) <= 1e-9 * abs(want)


def test_optical_middle_cell(K):
    G, D, h, mu = _setup()
    om = np.array([0.4, 1.1, 2.5, 0.9, 3.3])
    g1 = np.zeros(M0 + 1, dtype=complex)
    a, b = ([K.reconstruct_sigma_optical(G, g1, om, m, E0, E1, ETA, OPN, n_theta=Q) for _ in range(5)] for m in mu)
    for r in a:
        assert np.array_equal(r, a[0])
    for i, w in enumerate(om):
        gR = ocond.cpgf_coefficients(M0 + 1, np.array([(w + 1j * ETA) / DE]), +1)[0, M0]
        gA = ocond.cpgf_coefficients(M0 + 1, np.array([(-w - 1j * ETA) / DE]), -1)[0, M0]
        want = -2j * np.pi * OPN / w * 0.8 * h * D * (gR + gA) / DE
        assert abs((a[0][i] - b[0][i]) - want) <= 1e-9 * abs(want)
