"""Patch kernels (several recursion steps per launch on small lattices) at the edges
of their shapes, against the row kernels and the oracle: lattices of one patch and
many, narrower than the halo (it wraps more than once), ragged last patches, chunks
that do not fill a group, batches of unequal lattices, step counts on both sides of a
launch.

Tolerances.  Against the row kernels: the vectors are the same to the bit, the moments
differ by the order of FP64 sums of n terms of size <= 1 over n orbitals: 1e-12.  A
wrong site shows as 1/n >= 1e-5.  States against the oracle: fp32_chain_bound's
argument, as for the history sweeps.
"""
import numpy as np
import pytest

import workload as wl
from oracle import evolve as oev
from oracle import lattice as olat

pytestmark = pytest.mark.gpu

U = {wl.FP32: 2.0 ** -24, wl.FP64: 2.0 ** -50}
KINDS = {
    "square": dict(kind=wl.SQUARE, t=-1.0, anderson_w=1.0, vacancy_p=0.1, disorder_seed=3, e_min=-6.0, e_max=6.5),
    "honeycomb": dict(kind=wl.HONEYCOMB, t=-2.7, e_min=-9.0, e_max=9.0),
    "honeycomb-flux": dict(kind=wl.HONEYCOMB, t=-2.7, anderson_w=1.0, vacancy_p=0.05, disorder_seed=4, e_min=-9.0,
                           e_max=9.5),
    "spin": dict(kind=wl.HONEYCOMB_SPIN, t=-2.7, rashba=0.3, exchange=0.2, vacancy_p=0.1, disorder_seed=5, e_min=-10.5,
                 e_max=10.0),
    "spin-flux": dict(kind=wl.HONEYCOMB_SPIN, t=-2.7, rashba=0.3, anderson_w=1.0, disorder_seed=6, e_min=-10.5,
                      e_max=10.5),
}
SIZES = [(2, 2, 1), (3, 5, 2), (8, 8, 3), (16, 3, 7), (33, 40, 5), (61, 59, 9), (97, 130, 4)]


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _lattice(kind, L1, L2):
    return wl.Lattice(L1=L1, L2=L2, flux=1.0 / L1 if kind.endswith("flux") else 0.0, **KINDS[kind])


def _moments(K, lats, M, R, prec, **tune):
    par = wl.DosParams(num_moments=M, num_random=R, vector_seed=11, precision=prec)
    plan = K.Plan(lats, par, **tune)
    mu = np.empty((len(lats), R, M))
    plan.run(mu_per_vector=mu)
    plan.close()
    return mu


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("L1,L2,R", SIZES)
@pytest.mark.parametrize("kind", list(KINDS))
def test_patch_moments_match_rows(K, kind, L1, L2, R, prec):
    print(f"{kind} {L1}x{L2} R={R} prec={prec}", flush=True)
    lat = _lattice(kind, L1, L2)
    rows = 2 if lat.kind == wl.HONEYCOMB_SPIN else 5
    for M in (2, 3, 9, 15, 16, 17, 18, 41):
        a = _moments(K, [lat], M, R, prec)
        b = _moments(K, [lat], M, R, prec, kernel=rows)
        assert np.max(np.abs(a - b)) <= 1e-12, (M, np.max(np.abs(a - b)))


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_patch_batch_of_unequal_lattices(K, kind, prec):
    print(f"batch {kind} prec={prec}", flush=True)
    lats = [_lattice(kind, a, b).replace(disorder_seed=20 + i)
            for i, (a, b) in enumerate([(5, 40), (64, 7), (12, 12), (90, 33), (2, 9)])]
    rows = 2 if lats[0].kind == wl.HONEYCOMB_SPIN else 5
    a = _moments(K, lats, 27, 3, prec)
    b = _moments(K, lats, 27, 3, prec, kernel=rows)
    assert np.max(np.abs(a - b)) <= 1e-12


def _check_states(K, lat, R, steps, prec):
    m = olat.build(lat)
    n_orb = lat.L1 * lat.L2 * {wl.SQUARE: 1, wl.HONEYCOMB: 2, wl.HONEYCOMB_SPIN: 4}[lat.kind]
    rng = np.random.default_rng(lat.L1 * 100 + R)
    x = rng.standard_normal((R, m.orb_index.size)) + 1j * rng.standard_normal((R, m.orb_index.size))
    x /= np.linalg.norm(x, axis=1)[:, None]
    psi0 = np.zeros((R, n_orb), dtype=np.complex128)
    psi0[:, m.orb_index] = x
    for M in steps:
        _, coef, _ = oev.step_operator(lat, m, 1.0, M)
        got = np.asarray(K.time_evolve(lat, psi0, 1.0, M, 2, precision=prec)[0]).reshape(R, n_orb)
        # A spinful site adds 7 terms of 2 x 2 blocks (14 products) where the bound counts 6.
        chain = 3 * (np.arange(M) + 1.0) ** 1.5 * 6 * U[prec] * 8 / np.sqrt(3)
        tol = 2 * U[prec] * (1 + np.sum(np.abs(coef))) + np.sum(np.abs(coef) * chain)
        for r in range(R):
            ref = np.zeros(n_orb, dtype=np.complex128)
            ref[m.orb_index] = oev.evolve(lat, m, x[r], 1.0, M, 2)[0]
            assert np.max(np.abs(got[r] - ref)) <= tol, (M, r, np.max(np.abs(got[r] - ref)), tol)


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("L1,L2,R", SIZES)
@pytest.mark.parametrize("kind", ["spin", "spin-flux"])
def test_patch_states_with_spin(K, kind, L1, L2, R, prec):
    """Every T_n x stored (the ring of three vectors and more)."""
    print(f"{kind} {L1}x{L2} R={R} prec={prec}", flush=True)
    _check_states(K, _lattice(kind, L1, L2), R, (2, 3, 4, 5, 6, 9, 33, 38), prec)


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["square", "honeycomb-flux"])
def test_row_history_above_the_patches(K, kind, prec):
    """A lattice with too many cells x chunks for patches: history sweeps by rows."""
    print(f"rows {kind} prec={prec}", flush=True)
    _check_states(K, _lattice(kind, 331, 411).replace(flux=2.0 / 331 if kind.endswith("flux") else 0.0), 16, (6, 39), prec)
