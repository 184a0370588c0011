"""Chain patches (small spinless lattices) against the chain sweeps by rows
(KPM_CHAIN_STEPS = 2) at the edges of their shapes: one patch and many, halos that wrap
more than once, padded vectors, ragged K blocks, orders around a launch's levels.

Tolerance: 1e-12 of the largest element, in FP64 as between the row sweeps and single
steps (sums in another order), in FP32 because both paths round each site alike (the
vectors are the same to the bit).  Split BF16: the same planes, so the same product.
"""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

KINDS = {
    "square": dict(kind=wl.SQUARE, t=-2.7, anderson_w=2.0, vacancy_p=0.05, disorder_seed=8, e_min=-12.0, e_max=12.5),
    "honeycomb": dict(kind=wl.HONEYCOMB, t=-2.7, e_min=-9.0, e_max=9.0),
    "honeycomb-flux": dict(kind=wl.HONEYCOMB, t=-2.7, anderson_w=1.0, vacancy_p=0.05, disorder_seed=4, e_min=-9.0,
                           e_max=9.5),
}


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


@pytest.mark.parametrize("L1,L2,R", [(4, 3, 1), (9, 16, 2), (33, 40, 3), (61, 59, 9)])
@pytest.mark.parametrize("kind", list(KINDS))
def test_chain_patches_match_rows(K, monkeypatch, kind, L1, L2, R):
    print(f"{kind} {L1}x{L2} R={R}", flush=True)
    lat = wl.Lattice(L1=L1, L2=L2, flux=1.0 / L1 if kind.endswith("flux") else 0.0, **KINDS[kind])
    for M in (2, 3, 8, 9, 10, 17, 33):
        for mode, prec in ((wl.GAMMA_FP64, wl.FP64), (wl.GAMMA_FP64, wl.FP32), (wl.GAMMA_SPLIT_BF16, wl.FP32)):
            par = wl.CondParams(num_moments=M, num_random=R, vector_seed=9, alpha=0, beta=M % 2, gamma_mode=mode)
            monkeypatch.delenv("KPM_CHAIN_STEPS", raising=False)
            a = K.moments_cond(lat, par, precision=prec)
            monkeypatch.setenv("KPM_CHAIN_STEPS", "2")
            b = K.moments_cond(lat, par, precision=prec)
            assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b)), (M, mode, prec, np.max(np.abs(a - b)))
