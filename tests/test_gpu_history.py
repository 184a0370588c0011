"""History sweeps (four recursion steps per launch, every T_n x stored) against the
oracle at the edges of their shapes: lattices narrower and shorter than a tile's
halo, ragged tiles, one and several groups of vector chunks, padded vectors, counts
of steps on both sides of a sweep and of the history ring.

Tolerance: fp32_chain_bound's argument for one chain.  An element of T_n x is off by
at most 6 u lambda / sqrt(3) n^1.5 (lambda = 8) of the largest element the recursion
meets, taken as the vector's 2-norm times 1 (|T_n(H~)| <= 1); a state is a sum of
them with known coefficients, Gamma_n a product with h~ r.  u = 2^-24 or 2^-53; in
FP64 2^-50 covers the oracle's own roundings too.  A site, a neighbour or a level
taken wrongly is an error of the order of the elements themselves.
"""
import numpy as np
import pytest

import workload as wl
from oracle import cond as ocond
from oracle import evolve as oev
from oracle import lattice as olat

pytestmark = pytest.mark.gpu

U = {wl.FP32: 2.0 ** -24, wl.FP64: 2.0 ** -50}
KINDS = {
    "square": dict(kind=wl.SQUARE, t=-1.0, e_min=-6.0, e_max=6.0),
    "square-dis": dict(kind=wl.SQUARE, t=-1.0, anderson_w=1.0, vacancy_p=0.1, disorder_seed=3, e_min=-6.0, e_max=6.5),
    "honeycomb": dict(kind=wl.HONEYCOMB, t=-2.7, e_min=-9.0, e_max=9.0),
    "honeycomb-on": dict(kind=wl.HONEYCOMB, t=-2.7, anderson_w=1.0, disorder_seed=5, e_min=-9.0, e_max=9.5),
    "honeycomb-vac": dict(kind=wl.HONEYCOMB, t=-2.7, vacancy_p=0.1, disorder_seed=6, e_min=-9.0, e_max=9.0),
    "honeycomb-flux": dict(kind=wl.HONEYCOMB, t=-2.7, anderson_w=1.0, vacancy_p=0.05, disorder_seed=4,
                           e_min=-9.0, e_max=9.5),
}
SIZES = [(2, 2, 1), (3, 5, 2), (7, 4, 3), (58, 9, 4), (59, 11, 5), (61, 3, 8), (33, 40, 17), (130, 37, 1)]
STEPS = [2, 3, 4, 5, 6, 7, 10, 33, 38]


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _lattice(kind, L1, L2):
    return wl.Lattice(L1=L1, L2=L2, flux=1.0 / L1 if kind.endswith("flux") else 0.0, **KINDS[kind])


def _chain(n, u):
    return n ** 1.5 * 6 * u * 8 / np.sqrt(3)


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("L1,L2,R", SIZES)
@pytest.mark.parametrize("kind", list(KINDS))
def test_evolve_history_edges(K, kind, L1, L2, R, prec):
    print(f"{kind} {L1}x{L2} R={R} prec={prec}", flush=True)
    lat = _lattice(kind, L1, L2)
    m = olat.build(lat)
    n_orb = L1 * L2 * (1 if lat.kind == wl.SQUARE else 2)
    rng = np.random.default_rng(L1 * 100 + R)
    x = rng.standard_normal((R, m.orb_index.size)) + 1j * rng.standard_normal((R, m.orb_index.size))
    x /= np.linalg.norm(x, axis=1)[:, None]
    psi0 = np.zeros((R, n_orb), dtype=np.complex128)
    psi0[:, m.orb_index] = x
    for M in STEPS:
        Ht, coef, _ = oev.step_operator(lat, m, 1.0, M)
        got, _ = K.time_evolve(lat, psi0, 1.0, M, 2, precision=prec)
        got = np.asarray(got).reshape(R, n_orb)
        # The stored state and the start are rounded to the vectors' type once each.
        tol = 2 * U[prec] * (1 + np.sum(np.abs(coef))) + np.sum(np.abs(coef) * _chain(np.arange(M) + 1.0, U[prec]))
        for r in range(R):
            ref = np.zeros(n_orb, dtype=np.complex128)
            ref[m.orb_index] = oev.evolve(lat, m, x[r], 1.0, M, 2)[0]
            assert np.max(np.abs(got[r] - ref)) <= tol, (M, r, np.max(np.abs(got[r] - ref)), tol)


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("L1,L2,R", SIZES)
@pytest.mark.parametrize("kind", ["square-dis", "honeycomb", "honeycomb-flux"])
def test_gamma1_ring_edges(K, kind, L1, L2, R, prec):
    """M around the ring of 8 vectors and its minimum of 6 (in place below it)."""
    if min(L1, L2) < 3:
        pytest.skip("second-order velocity needs distinct neighbours")
    print(f"{kind} {L1}x{L2} R={R} prec={prec}", flush=True)
    lat = _lattice(kind, L1, L2)
    for M in (1, 5, 6, 7, 8, 9, 12, 16, 19):
        par = wl.CondParams(num_moments=M, num_random=R, vector_seed=17, alpha=0, beta=M % 2)
        ref, _ = ocond.cond_gamma1(lat, par)
        got = K.moments_gamma1(lat, par, precision=prec)
        # |Gamma_n| <= mean |T_n r| |h~ r| / N: |r| = sqrt(N), |h~| <= sum of |bond second moments|
        # <= 4 bonds x |t| x a^2 (nm) each.
        h2 = 4 * abs(lat.t) * 0.25 ** 2 * 4
        tol = h2 * _chain(M + 1.0, U[prec])
        assert np.max(np.abs(got - ref)) <= tol, (M, np.max(np.abs(got - ref)), tol)
