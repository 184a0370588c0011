"""The exact-mode Gamma product at the edges of its tiles (32 x 32 per workgroup, K
blocks of 256 values, at most 64 chunks of them) against the oracle.

Tolerance: 1e-10 of the largest element in FP64, as for the other exact-mode tests (the
chains' rounding grows as n^1.5 2^-53, 1e-12 at the orders here; the product adds sums
of at most 3 10^4 terms, below 1e-14).  In FP32 the chains' own bound,
fp32_chain_bound, relative to the sum of magnitudes, with the product exact.
"""
import numpy as np
import pytest

import workload as wl
from oracle import cond as ocond
from _bounds import fp32_chain_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


# (L1, L2, R): one K block, a few, more than 64 with a ragged last chunk.
@pytest.mark.parametrize("L1,L2,R", [(6, 5, 1), (13, 11, 3), (97, 53, 3)])
@pytest.mark.parametrize("M", [2, 3, 16, 31, 32, 33, 65])
def test_gamma_fp64_tiles(K, L1, L2, R, M):
    print(f"gamma fp64 {L1}x{L2} R={R} M={M}", flush=True)
    lat = wl.Lattice(kind=wl.HONEYCOMB, L1=L1, L2=L2, t=-2.7, anderson_w=1.0, vacancy_p=0.02, disorder_seed=4,
                     e_min=-9.0, e_max=9.5)
    par = wl.CondParams(num_moments=M, num_random=R, vector_seed=9, alpha=0, beta=1, gamma_mode=wl.GAMMA_FP64)
    (ref, B), _ = ocond.cond_gamma(lat, par, with_bound=True)
    G = K.moments_cond(lat, par, precision=wl.FP64)
    assert np.max(np.abs(G - ref)) <= 1e-10 * np.max(np.abs(ref))
    G32 = K.moments_cond(lat, par, precision=wl.FP32)
    n = np.arange(M)
    assert np.all(np.abs(G32 - ref) <= np.sqrt(2) * fp32_chain_bound(n[:, None], n[None, :]) * B)
