"""Which kernels the library chooses, on the lattices that the patch tests use: they
compare patches with rows only where the patches are in fact taken."""
import numpy as np
import pytest

import workload as wl
from test_gpu_patch import KINDS, SIZES, _lattice
from test_gpu_patch_chain import KINDS as CHAIN_KINDS

pytestmark = pytest.mark.gpu

PATCH, CHAIN_PATCH, ROWS, STEP = range(4)


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _counts(K):
    return np.array([K.debug_launches(k) for k in range(4)])


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_small_lattices_take_patches(K, kind, prec):
    for L1, L2, R in SIZES:
        lat = _lattice(kind, L1, L2)
        rows = 2 if lat.kind == wl.HONEYCOMB_SPIN else 5
        for kernel, want in ((0, True), (rows, False)):
            c = _counts(K)
            p = K.Plan([lat], wl.DosParams(num_moments=16, num_random=R, vector_seed=11, precision=prec), kernel=kernel)
            p.run(mu_per_vector=np.empty((1, R, 16)))
            p.close()
            assert ((_counts(K) - c)[PATCH] > 0) == want, (L1, L2, R, kernel)
        c = _counts(K)
        K.time_evolve(lat, np.ones((R, lat.n_orbitals), dtype=complex), 0.5, 9, 2, precision=prec)
        d = _counts(K) - c
        # (With a spin the larger ones keep single steps where those are modelled as fast.)
        patches = lat.kind != wl.HONEYCOMB_SPIN or L1 * L2 * R < 8192
        assert d[ROWS] == 0 and (d[PATCH] > 0 or not patches) and (d[STEP] == 0 or not patches), (L1, L2, R, d)


@pytest.mark.parametrize("L1,L2,R", [(4, 3, 1), (9, 16, 2), (33, 40, 3), (61, 59, 9)])
@pytest.mark.parametrize("kind", list(CHAIN_KINDS))
def test_small_chains_take_patches(K, monkeypatch, kind, L1, L2, R):
    lat = wl.Lattice(L1=L1, L2=L2, flux=1.0 / L1 if kind.endswith("flux") else 0.0, **CHAIN_KINDS[kind])
    for mode, prec in ((wl.GAMMA_FP64, wl.FP64), (wl.GAMMA_FP64, wl.FP32), (wl.GAMMA_SPLIT_BF16, wl.FP32)):
        par = wl.CondParams(num_moments=17, num_random=R, vector_seed=9, alpha=0, beta=0, gamma_mode=mode)
        for steps in (None, "2"):
            if steps is None:
                monkeypatch.delenv("KPM_CHAIN_STEPS", raising=False)
            else:
                monkeypatch.setenv("KPM_CHAIN_STEPS", steps)
            c = _counts(K)
            K.moments_cond(lat, par, precision=prec)
            assert ((_counts(K) - c)[CHAIN_PATCH] > 0) == (steps is None)
