"""The autotuner measures the shape that the library chooses by itself: with a tuned
shape, or a cache line, a lattice is not slower than without.

Times are the loops of the plans in turn, the smallest of several; 15 % covers what two
runs of a short loop differ by (without the default among the candidates the tuned
shapes took 1.3 to 2.7 times as long).
"""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

PATCH = 0


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _loop_ms(K, lat, par, shapes):
    import torch
    mu = torch.empty((1, par.num_random, par.num_moments), dtype=torch.float64, device="cuda")
    plans = [K.Plan([lat], par, **s) for s in shapes]
    t = np.full(len(plans), np.inf)
    for rep in range(8):
        for i, p in enumerate(plans):
            p.run(mu_per_vector=mu)
            if rep:
                t[i] = min(t[i], p.info()["last_loop_ms"])
    infos = [p.info() for p in plans]
    for p in plans:
        p.close()
    return t, infos


@pytest.mark.parametrize("kind,L1,L2,R,prec", [(wl.HONEYCOMB, 64, 64, 4, wl.FP64), (wl.SQUARE, 100, 90, 2, wl.FP32),
                                               (wl.HONEYCOMB_SPIN, 60, 50, 4, wl.FP32),
                                               (wl.HONEYCOMB, 1000, 1000, 4, wl.FP32)])
def test_tuned_shape_is_not_slower_than_the_default(K, tmp_path, monkeypatch, kind, L1, L2, R, prec):
    lat = wl.Lattice(kind=kind, L1=L1, L2=L2, t=-2.7, anderson_w=0.3, e_min=-13.0, e_max=13.0)
    par = wl.DosParams(num_moments=128, num_random=R, vector_seed=1, precision=prec)
    cache = tmp_path / "tune.txt"
    # A stale line for the same key (single steps by direct loads): the tuner must not measure it as the default.
    n_orb = lat.n_orbitals
    rp = R if prec == wl.FP64 else (R + 1) // 2 * 2
    cache.write_text(f"{kind} {prec} {rp} {int(np.floor(np.log2(n_orb)))} 1 256 128 1024 0 1.0\n")
    monkeypatch.setenv("KPM_TUNE_CACHE", str(cache))
    best = K.autotune([lat], par, probe_steps=16, cache_path=str(cache))
    best.pop("GBs")
    lines = cache.read_text().strip().splitlines()
    assert len(lines) == 2
    monkeypatch.delenv("KPM_TUNE_CACHE")
    (default, tuned), (i0, i1) = _loop_ms(K, lat, par, [{}, best])
    print(f"default {default:.3f} ms, tuned {tuned:.3f} ms {best} {lines[1]}", flush=True)
    assert tuned <= 1.15 * default
    if lines[1].endswith(" auto"):
        keys = ("kernel", "block", "rows", "grid", "tile_cells_x", "tile_chunks")
        assert [i0[k] for k in keys] == [i1[k] for k in keys]
    monkeypatch.setenv("KPM_TUNE_CACHE", str(cache))
    (cached,), _ = _loop_ms(K, lat, par, [{}])
    assert cached <= 1.15 * default


def test_cached_default_serves_other_lattices_of_its_key(K, tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    cache.write_text("0 1 4 13 5 512 12 136 1 5.0 auto\n")
    monkeypatch.setenv("KPM_TUNE_CACHE", str(cache))
    for L1, L2 in ((64, 64), (60, 70), (90, 80)):
        lat = wl.Lattice(kind=wl.HONEYCOMB, L1=L1, L2=L2, t=-2.7, e_min=-9.0, e_max=9.0)
        before = K.debug_launches(PATCH)
        K.moments_dos([lat], wl.DosParams(num_moments=16, num_random=4, precision=wl.FP64))
        assert K.debug_launches(PATCH) > before
