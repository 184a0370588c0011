"""Row history sweeps (several recursion steps per launch by rows, every T_n x stored),
asked for with KPM_HISTORY_STEPS so that lattices of every size run them, at the edges
of their shapes: narrower and shorter than a tile's halo, ragged tiles, one and several
groups of vector chunks, padded vectors, every instance of on-site terms, vacancies and
phases, launches of one to four levels.

Against single steps: the sweeps' arithmetic is that of the single-step kernels to the
bit, so the states are equal.  Against the oracle: the tolerance of the history tests,
6 u lambda / sqrt(3) n^1.5 of the norm per T_n x (lambda = 8, u = 2^-24 or 2^-50).
"""
import numpy as np
import pytest

import workload as wl
from oracle import evolve as oev
from oracle import lattice as olat

pytestmark = pytest.mark.gpu

U = {wl.FP32: 2.0 ** -24, wl.FP64: 2.0 ** -50}
PATCH, CHAIN_PATCH, ROWS, STEP = range(4)
SQ = dict(kind=wl.SQUARE, t=-1.0, e_min=-6.0, e_max=6.5)
HC = dict(kind=wl.HONEYCOMB, t=-2.7, e_min=-9.0, e_max=9.5)
DIS = dict(anderson_w=1.0, disorder_seed=3)
VAC = dict(vacancy_p=0.1, disorder_seed=6)
KINDS = {
    "square": SQ, "square-on": dict(SQ, **DIS), "square-vac": dict(SQ, **VAC), "square-on-vac": dict(SQ, **DIS, vacancy_p=0.1),
    "honeycomb": HC, "honeycomb-on": dict(HC, **DIS), "honeycomb-vac": dict(HC, **VAC),
    "honeycomb-on-vac": dict(HC, **DIS, vacancy_p=0.1), "honeycomb-flux": HC, "honeycomb-on-flux": dict(HC, **DIS),
    "honeycomb-vac-flux": dict(HC, **VAC), "honeycomb-on-vac-flux": dict(HC, **DIS, vacancy_p=0.1),
}
SIZES = [(2, 2, 1), (3, 5, 2), (7, 4, 3), (58, 9, 4), (59, 11, 5), (61, 3, 8), (33, 40, 17), (130, 37, 1)]


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _lattice(kind, L1, L2):
    return wl.Lattice(L1=L1, L2=L2, flux=1.0 / L1 if kind.endswith("flux") else 0.0, **KINDS[kind])


def _states(K, monkeypatch, steps, lat, psi0, M, prec):
    """The states after one time step, and the launches of each kind."""
    if steps is None:
        monkeypatch.delenv("KPM_HISTORY_STEPS", raising=False)
    else:
        monkeypatch.setenv("KPM_HISTORY_STEPS", str(steps))
    before = [K.debug_launches(k) for k in range(4)]
    psi = np.asarray(K.time_evolve(lat, psi0, 1.0, M, 2, precision=prec)[0]).reshape(psi0.shape)
    return psi, [K.debug_launches(k) - b for k, b in zip(range(4), before)]


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("L1,L2,R", SIZES)
@pytest.mark.parametrize("kind", list(KINDS))
def test_rows_match_single_steps(K, monkeypatch, kind, L1, L2, R, prec):
    print(f"{kind} {L1}x{L2} R={R} prec={prec}", flush=True)
    lat = _lattice(kind, L1, L2)
    m = olat.build(lat)
    rng = np.random.default_rng(L1 * 100 + R)
    x = rng.standard_normal((R, m.orb_index.size)) + 1j * rng.standard_normal((R, m.orb_index.size))
    x /= np.linalg.norm(x, axis=1)[:, None]
    psi0 = np.zeros((R, L1 * L2 * (1 if lat.kind == wl.SQUARE else 2)), dtype=np.complex128)
    psi0[:, m.orb_index] = x
    for M in (3, 4, 5, 6, 7, 10, 38):
        one, n = _states(K, monkeypatch, 1, lat, psi0, M, prec)
        assert n[STEP] == M - 1 and n[ROWS] == n[PATCH] == 0
        for steps in (4, 3, 2) if M in (7, 38) else (4,):
            got, n = _states(K, monkeypatch, steps, lat, psi0, M, prec)
            assert n[ROWS] >= (M - 1) // steps and n[STEP] == n[PATCH] == 0
            assert np.array_equal(got, one), (M, steps, np.max(np.abs(got - one)))
    _, coef, _ = oev.step_operator(lat, m, 1.0, 10)
    chain = (np.arange(10) + 1.0) ** 1.5 * 6 * U[prec] * 8 / np.sqrt(3)
    tol = 2 * U[prec] * (1 + np.sum(np.abs(coef))) + np.sum(np.abs(coef) * chain)
    got, _ = _states(K, monkeypatch, 4, lat, psi0, 10, prec)
    for r in range(R):
        ref = np.zeros(psi0.shape[1], dtype=np.complex128)
        ref[m.orb_index] = oev.evolve(lat, m, x[r], 1.0, 10, 2)[0]
        assert np.max(np.abs(got[r] - ref)) <= tol, (r, np.max(np.abs(got[r] - ref)), tol)


@pytest.mark.parametrize("kind,prec", [("square", wl.FP64), ("square-on", wl.FP32), ("honeycomb-on-vac", wl.FP32),
                                       ("honeycomb-flux", wl.FP64)])
@pytest.mark.parametrize("L1,L2,R", [(5, 100000, 1), (100000, 5, 1), (700, 600, 9)])
def test_rows_on_long_lattices(K, monkeypatch, kind, L1, L2, R, prec):
    """Above the patches' limit, very narrow or very flat, and with two groups of chunks."""
    print(f"{kind} {L1}x{L2} R={R}", flush=True)
    lat = _lattice(kind, L1, L2)
    rng = np.random.default_rng(3)
    n_orb = L1 * L2 * (1 if lat.kind == wl.SQUARE else 2)
    psi0 = (rng.standard_normal((R, n_orb)) + 1j * rng.standard_normal((R, n_orb))) / np.sqrt(2 * n_orb)
    one, _ = _states(K, monkeypatch, 1, lat, psi0, 9, prec)
    got, n = _states(K, monkeypatch, 4, lat, psi0, 9, prec)
    assert n[ROWS] > 0 and n[PATCH] == 0
    assert np.array_equal(got, one)


@pytest.mark.parametrize("kind", ["square-on-vac", "honeycomb", "honeycomb-on-vac-flux"])
def test_gamma1_and_singleshot_on_rows(K, monkeypatch, kind):
    """The two other callers: the same vectors, so the same products and sums."""
    lat = _lattice(kind, 61, 30)
    E = np.linspace(-1.0, 1.0, 5)
    for prec in (wl.FP32, wl.FP64):
        par = wl.CondParams(num_moments=21, num_random=5, vector_seed=17, alpha=0, beta=0)
        ref = None
        for steps in (1, 4):
            monkeypatch.setenv("KPM_HISTORY_STEPS", str(steps))
            before = K.debug_launches(ROWS)
            got = (K.moments_gamma1(lat, par, precision=prec), K.sigma_singleshot(lat, par, E, 0.3, precision=prec))
            assert (K.debug_launches(ROWS) > before) == (steps > 1)
            if ref is None:
                ref = got
        assert np.array_equal(ref[0], got[0]) and np.array_equal(ref[1], got[1])


@pytest.mark.parametrize("kind,prec", [("square", wl.FP64), ("honeycomb-on-vac-flux", wl.FP32)])
def test_few_levels_run_as_single_steps(K, monkeypatch, kind, prec):
    """Above the patches: M history vectors allow M - 2 levels per launch, and the last
    launch of a run may have fewer left.  One or two levels are single steps."""
    lat = _lattice(kind, 700, 600)
    psi0 = np.ones((9, lat.n_orbitals), dtype=complex) / np.sqrt(lat.n_orbitals)
    for M, rows, single in ((3, 0, 2), (4, 0, 3), (7, 1, 2), (38, 9, 2)):
        got, n = _states(K, monkeypatch, None, lat, psi0, M, prec)
        assert (n[PATCH], n[ROWS], n[STEP]) == (0, rows, single), (M, n)
        one, _ = _states(K, monkeypatch, 1, lat, psi0, M, prec)
        assert np.array_equal(got, one)


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["square", "honeycomb-on-vac"])
def test_stats_count_the_launches_made(K, monkeypatch, kind, prec):
    """kpm_evolve_stats_t.bytes: two vectors in and one per level out for each launch.
    M = 38 with 32 history vectors: runs of 31 and 6 steps."""
    lat = _lattice(kind, 40, 30)
    psi0 = np.ones((2, lat.n_orbitals), dtype=complex) / np.sqrt(lat.n_orbitals)
    size = 4 if prec == wl.FP32 else 8
    vec = lat.n_orbitals * 2 * 2 * size
    site = 0 if kind == "square" else lat.n_orbitals * (size + 1)
    for steps, launches in ((1, [1] * 37), (4, [4] * 7 + [3, 4, 2]), (2, [2] * 15 + [1, 2, 2, 2])):
        _states(K, monkeypatch, steps, lat, psi0, 38, prec)
        want = sum((2 + n) * vec + site for n in launches) + (38 + 2 * 2 - 1) * vec
        assert K.evolve_last_stats()["bytes"] == pytest.approx(want, rel=1e-12), steps
