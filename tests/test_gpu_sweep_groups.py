"""Sweeps over several groups of vector chunks that share 128-byte lines (a site's chunks
are not a multiple of 8): the groups run on neighbouring tiles.

Moments: a vector's start depends on its index only, so the first 13 of 16 vectors (two
groups of whole lines) and 13 vectors alone (lines shared) have the same moments up to
the order of FP64 sums of values <= 1 over n orbitals: 1e-12.  Time: 13 vectors move less
than 16; with the groups apart they took 1.85 times as long a step (every shared line
fetched twice), together 1.03 times.  1.35 divides the two.
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


def _plan(K, lats, R, prec, M=64):
    return K.Plan(lats, wl.DosParams(num_moments=M, num_random=R, vector_seed=3, precision=prec), kernel=5)


HC = wl.Lattice(kind=wl.HONEYCOMB, L1=200, L2=170, t=-2.7, anderson_w=0.5, vacancy_p=0.02, disorder_seed=5, e_min=-9.0,
                e_max=9.5)
SQ = wl.Lattice(kind=wl.SQUARE, L1=333, L2=90, t=-1.0, anderson_w=0.5, disorder_seed=5, e_min=-6.0, e_max=6.5)


@pytest.mark.parametrize("lat", [HC, SQ], ids=["honeycomb", "square"])
@pytest.mark.parametrize("prec,n_few,n_full", [(wl.FP64, 9, 16), (wl.FP64, 13, 16), (wl.FP64, 21, 24), (wl.FP32, 25, 32)])
def test_groups_of_shared_lines(K, lat, prec, n_few, n_full):
    lats = [lat, lat.replace(L1=lat.L1 - 67, disorder_seed=6)]
    mu = {}
    for R in (n_few, n_full):
        p = _plan(K, lats, R, prec, 41)
        mu[R] = np.empty((2, R, 41))
        p.run(mu_per_vector=mu[R])
        p.close()
    assert np.max(np.abs(mu[n_few] - mu[n_full][:, :n_few])) <= 1e-12


def test_shared_lines_are_fetched_once(K):
    import torch
    lat = HC.replace(L1=1000, L2=1000)
    t = {}
    for R in (13, 16):
        p = _plan(K, [lat], R, wl.FP64)
        mu = torch.empty((1, R, 64), dtype=torch.float64, device="cuda")
        ms = []
        for _ in range(6):
            p.run(mu_per_vector=mu)
            ms.append(p.info()["last_loop_ms"])
        p.close()
        t[R] = min(ms[1:])
    print(f"loop of 32 steps: 13 vectors {t[13]:.2f} ms, 16 vectors {t[16]:.2f} ms", flush=True)
    assert t[13] <= 1.35 * t[16]
