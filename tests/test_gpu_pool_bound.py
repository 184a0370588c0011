"""The bound on the pool's idle blocks holds for small blocks too: a program that closes
many plans whose buffers are all below 16 MB keeps no more idle than stays free."""
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

GIB = 1 << 30


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def test_many_small_blocks_stay_within_the_bound(K):
    """120 plans of four 14 MB vectors (6.6 GB) on a card with 9 GB free: when all are
    closed, at least as much as the idle blocks is free for others (they then share the
    9 GB, so at most half of it idles; 128 MB for the memory looked at only after each
    16 MB and for rounding)."""
    import torch
    torch.cuda.empty_cache()
    K.release_workspace()
    free, total = torch.cuda.mem_get_info()
    fill = torch.empty(free - 9 * GIB, dtype=torch.uint8, device="cuda")
    lat = wl.Lattice(kind=wl.HONEYCOMB, L1=200, L2=256, t=-2.7, e_min=-9.0, e_max=9.0)
    par = wl.DosParams(num_moments=4, num_random=8, vector_seed=1, precision=wl.FP64)
    plans = [K.Plan([lat], par) for _ in range(120)]
    mu = torch.empty((1, 8, 4), dtype=torch.float64, device="cuda")
    for p in plans:
        p.run(mu_per_vector=mu)
    first = mu.clone()
    full, _ = torch.cuda.mem_get_info()
    assert full < 4 * GIB
    for p in plans:
        p.close()
    left, _ = torch.cuda.mem_get_info()
    held = K.release_workspace()
    print(f"idle {held / GIB:.2f} GB, free beside it {left / GIB:.2f} GB", flush=True)
    assert 0 < held <= left + (128 << 20)
    del fill
    torch.cuda.empty_cache()
    with_room = K.Plan([lat], par)
    with_room.run(mu_per_vector=mu)
    with_room.close()
    assert torch.equal(mu, first)


def test_blocks_of_a_failed_run_are_not_reused(K):
    """A run that fails before its wait may leave work on its stream, and a later run on
    another stream waits for that one only: the plan's blocks go back to the device."""
    import torch
    lat = wl.Lattice(kind=wl.HONEYCOMB, L1=64, L2=64, t=-2.7, e_min=-9.0, e_max=9.0)
    par = wl.DosParams(num_moments=16, num_random=4, vector_seed=1, precision=wl.FP64)
    mu = torch.empty((1, 4, 16), dtype=torch.float64, device="cuda")
    for fails in (False, True):
        plan = K.Plan([lat], par, use_graph=False)
        K.release_workspace()
        if fails:
            K.debug_inject_failure(2, 1)   # the second checked operation of the run
            with pytest.raises(K.KPMError):
                plan.run(mu_per_vector=mu)
            assert K.debug_inject_failure(0) == 1
        plan.run(mu_per_vector=mu)
        with torch.cuda.stream(torch.cuda.Stream()):
            plan.run(mu_per_vector=mu)
        torch.cuda.synchronize()
        plan.close()
        assert (K.release_workspace() == 0) == fails
