"""The single-shot accumulation at the edges of its tiles (16 packs of elements x 16
energies, vectors in groups of 32, flushes of 64) against the oracle.

FP64 against the oracle with the tolerance of the other single-shot tests, 1e-10 of the
largest value (they reach M = 150; the FP64 sums over at most 97 vectors add 1e-14).
FP32 by structure: an energy's sums are formed independently of the energies beside it,
so its value is the same to the bit in any group (the FP32 recursion's own error, which
is not bounded relative to a single, cancelled value, drops out).
"""
import numpy as np
import pytest

import workload as wl
from oracle import cond as ocond
from oracle import kpm as okpm
from oracle import lattice as olat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


@pytest.mark.parametrize("L1,L2,R", [(3, 3, 1), (7, 5, 3), (23, 17, 4)])
@pytest.mark.parametrize("M", [2, 3, 31, 32, 33, 64, 65, 97])
def test_singleshot_tiles(K, L1, L2, R, M):
    print(f"single-shot {L1}x{L2} R={R} M={M}", flush=True)
    lat = wl.Lattice(kind=wl.HONEYCOMB, L1=L1, L2=L2, t=-2.7, anderson_w=1.0, disorder_seed=4, e_min=-9.0, e_max=9.5)
    par = wl.CondParams(num_moments=M, num_random=R, vector_seed=29, alpha=0, beta=0)
    m = olat.build(lat)
    vecs = okpm.random_phase_vectors(m, R, par.vector_seed, 0)
    for n_e in (1, 15, 16, 17, 33):
        E = np.linspace(-6.0, 5.0, n_e)
        ref = ocond.sigma_singleshot(m, lat.e_min, lat.e_max, E, 0.2, M, vecs, 0, 0)
        s = K.sigma_singleshot(lat, par, E, 0.2, precision=wl.FP64)
        assert np.max(np.abs(s - ref)) <= 1e-10 * np.max(np.abs(ref)), (n_e, np.max(np.abs(s - ref)))
        s32 = np.asarray(K.sigma_singleshot(lat, par, E, 0.2, precision=wl.FP32))
        for k in {0, n_e // 2, n_e - 1}:
            one = np.asarray(K.sigma_singleshot(lat, par, E[k:k + 1], 0.2, precision=wl.FP32))
            assert one[0] == s32[k], (n_e, k, one[0], s32[k])
