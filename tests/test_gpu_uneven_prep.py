"""Model and start vectors of a batch with one large and many small lattices: each
lattice gets its own workgroups.

Moments: LDOS starts do not depend on the lattice's place in the batch, and the random
starts of the first lattices not on how many follow; the sums over n orbitals of values
<= 1 may run in another order: 1e-12.  Time of everything around the recursion: 2000
lattices of 16 cells beside one of 10^6 add 1 % to the elements; workgroups for 2001
lattices of the largest size took hundreds of times longer.  Four times (and 0.3 ms for
the reductions of 2001 lattices) divides the two.
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


KINDS = {
    "honeycomb": dict(kind=wl.HONEYCOMB, t=-2.7, anderson_w=0.7, vacancy_p=0.03, e_min=-9.0, e_max=9.5),
    "honeycomb-clean": dict(kind=wl.HONEYCOMB, t=-2.7, e_min=-9.0, e_max=9.5),
    "spin": dict(kind=wl.HONEYCOMB_SPIN, t=-2.7, rashba=0.2, vacancy_p=0.02, e_min=-10.5, e_max=10.5),
    "square": dict(kind=wl.SQUARE, t=-1.0, anderson_w=0.5, e_min=-6.0, e_max=6.5),
}


def _batch(kind, n_small, big=(150, 131)):
    rng = np.random.default_rng(5)
    sizes = [big] + [(int(rng.integers(2, 30)), int(rng.integers(2, 30))) for _ in range(n_small)]
    at = n_small // 2
    sizes[0], sizes[at] = sizes[at], sizes[0]   # the large one in the middle
    return [wl.Lattice(L1=a, L2=b, disorder_seed=7 + i, **KINDS[kind]) for i, (a, b) in enumerate(sizes)]


@pytest.mark.parametrize("prec", [wl.FP32, wl.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_batch_of_one_large_and_many_small(K, kind, prec):
    lats = _batch(kind, 300)
    par = wl.DosParams(num_moments=12, num_random=5, vector_seed=4, precision=prec)
    full, _ = K.moments_dos(lats, par)
    part, _ = K.moments_dos(lats[:160], par)
    assert np.max(np.abs(full[:160] - part)) <= 1e-12
    rng = np.random.default_rng(1)
    sites = [int(s) for s in rng.integers(0, 4, 3)]
    clean = [l.replace(vacancy_p=0.0) for l in lats]   # (a start site must not be vacant)
    ldos = wl.DosParams(num_moments=12, precision=prec, start=wl.START_SITES, sites=sites)
    mu, _ = K.moments_dos(clean, ldos)
    for i in (0, 1, 149, 150, 151, 299, 300):
        one, _ = K.moments_dos([clean[i]], ldos)
        assert np.max(np.abs(mu[i] - one[0])) <= 1e-12, i


def test_small_lattices_cost_little_beside_a_large_one(K):
    import torch
    big = wl.Lattice(kind=wl.HONEYCOMB, L1=1000, L2=1000, t=-2.7, anderson_w=0.5, disorder_seed=1, e_min=-9.0, e_max=9.0)
    lats = [big] + [big.replace(L1=4, L2=4, disorder_seed=2 + i) for i in range(2000)]
    par = wl.DosParams(num_moments=4, num_random=16, vector_seed=4, precision=wl.FP32)
    around = []
    for batch in ([big], lats):
        p = K.Plan(batch, par)
        mu = torch.empty((len(batch), 16, 4), dtype=torch.float64, device="cuda")
        t = []
        for _ in range(4):
            p.run(mu_per_vector=mu)
            i = p.info()
            t.append(i["last_run_ms"] - i["last_loop_ms"])
        p.close()
        around.append(min(t[1:]))
    print(f"around the recursion: {around[0]:.3f} ms alone, {around[1]:.3f} ms with 2000 small lattices", flush=True)
    assert around[1] <= 4 * around[0] + 0.3


def test_ldos_batch_beyond_2_32_elements(K):
    """Five lattices of 1024 x 1024 with 256 vectors: 5.4e9 numbers to clear, more than one
    launch has threads; each lattice alone has fewer."""
    lat = wl.Lattice(kind=wl.HONEYCOMB, L1=1024, L2=1024, t=-2.7, anderson_w=0.5, e_min=-9.0, e_max=9.0)
    lats = [lat.replace(disorder_seed=i) for i in range(5)]
    sites = [int(s) for s in np.random.default_rng(2).integers(0, lat.n_orbitals, 256)]
    par = wl.DosParams(num_moments=4, precision=wl.FP32, start=wl.START_SITES, sites=sites)
    K.release_workspace()
    mu, _ = K.moments_dos(lats, par)
    for i in (0, 4):
        one, _ = K.moments_dos([lats[i]], par)
        assert np.max(np.abs(mu[i] - one[0])) <= 1e-12
    K.release_workspace()
