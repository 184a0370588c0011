"""Chain sweeps whose groups of vector chunks share 128-byte lines, against single steps.

Sums in another order, in FP64: 1e-12 of the largest element (as the other chain tests).
"""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


@pytest.mark.parametrize("kind,prec,R", [(wl.HONEYCOMB, wl.FP64, 13), (wl.SQUARE, wl.FP64, 9), (wl.HONEYCOMB, wl.FP32, 26),
                                         (wl.HONEYCOMB_SPIN, wl.FP64, 5), (wl.HONEYCOMB_SPIN, wl.FP32, 11)])
def test_shared_lines(K, monkeypatch, kind, prec, R):
    lat = wl.Lattice(kind=kind, L1=70, L2=50, t=-2.7, rashba=0.2 if kind == wl.HONEYCOMB_SPIN else 0.0, anderson_w=0.5,
                     vacancy_p=0.03, disorder_seed=4, e_min=-13.0, e_max=13.0)
    par = wl.CondParams(num_moments=17, num_random=R, vector_seed=9, alpha=0, beta=1, gamma_mode=wl.GAMMA_FP64)
    steps = "2" if kind != wl.HONEYCOMB_SPIN else "3"
    monkeypatch.setenv("KPM_CHAIN_STEPS", steps)
    a = K.moments_cond(lat, par, precision=prec)
    monkeypatch.setenv("KPM_CHAIN_STEPS", "1")
    b = K.moments_cond(lat, par, precision=prec)
    tol = 1e-12 if prec == wl.FP64 else 1e-5   # FP32 chains round differently in the two forms
    assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))
