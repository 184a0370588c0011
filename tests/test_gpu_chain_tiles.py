"""Chain sweeps whose groups of vector chunks share 128-byte lines, and the rows per tile
in FP64: results against single steps, and the time of the library's rows against given
ones.

Sums in another order, in FP64: 1e-12 of the largest element (as the other chain tests).
Rows: the library's choice takes no more than 1.15 times the best of 8, 16 and 32 rows on
sizes where tiles of five rows, two per CU, took up to 1.18 times as long as 8 rows (7 to
11 % longer than the former choice).
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


def test_rows_in_fp64(K, monkeypatch):
    for kind, L1, L2, R in ((wl.HONEYCOMB, 236, 926, 2), (wl.HONEYCOMB, 400, 500, 2), (wl.SQUARE, 400, 900, 2)):
        lat = wl.Lattice(kind=kind, L1=L1, L2=L2, t=-2.7, vacancy_p=0.02, e_min=-13.0, e_max=13.0)
        par = wl.CondParams(num_moments=48, num_random=R, gamma_mode=wl.GAMMA_FP64)
        ms = {r: np.inf for r in (0, 8, 16, 32)}
        for _ in range(5):
            for r in ms:
                monkeypatch.setenv("KPM_CHAIN_STEPS", "2")
                monkeypatch.setenv("KPM_CHAIN_ROWS", str(r))
                K.moments_cond(lat, par, precision=wl.FP64)
                ms[r] = min(ms[r], K.cond_last_stats()["chain_ms"])
        print(f"{L1}x{L2}: chains {ms} ms", flush=True)
        assert ms[0] <= 1.15 * min(ms[8], ms[16], ms[32])
