"""Many energies or frequencies on a fine theta grid: the workspace does not grow with
their product, so a call that once fitted the card still does.  The values do not depend
on how the frequencies are split: equal bits to calls of their own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GIB = 1 << 30


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _gamma(M, dev):
    import torch
    g = torch.Generator(device=dev)
    g.manual_seed(M)
    return torch.randn(M, M, 2, generator=g, device=dev, dtype=torch.float64) * 1e-3


@pytest.mark.parametrize("M,Q,n,left", [(2, 1 << 20, 600, 6), (1500, 22500, 2990, None)])
def test_optical_blocks_of_frequencies(K, M, Q, n, left):
    """2^20 cells: 16.8 MB of sums per frequency, 10 GB for 600 of them on a card with 6 GB
    free, in blocks of 64.  1500 orders: several blocks of cells and of frequencies
    (2980 of these fill one)."""
    import torch
    K.release_workspace()
    torch.cuda.empty_cache()
    fill = torch.empty(torch.cuda.mem_get_info()[0] - left * GIB, dtype=torch.uint8, device="cuda") if left else None
    G = _gamma(M, "cuda")
    om = torch.linspace(0.2, 6.0, n, device="cuda", dtype=torch.float64)
    args = dict(mu=0.8, e_min=-7.0, e_max=9.0, eta=0.3, orbitals_per_nm2=30.0, n_theta=Q, kT=0.0)
    print(f"M={M} Q={Q} {n} frequencies", flush=True)
    got = K.reconstruct_sigma_optical(G, G[0].contiguous(), om, **args)
    for i in (0, 1, 63, 64, 70, n - 11, n - 10, n - 1):
        one = K.reconstruct_sigma_optical(G, G[0].contiguous(), om[i:i + 1], **args)
        assert torch.equal(one[0], got[i]), i
    del fill
    torch.cuda.empty_cache()


def test_bastin_blocks_of_energies(K):
    """2^20 cells: 32 KB of partial sums per energy, 3.3 GB for 100000 on a card with 3 GB free."""
    import torch
    K.release_workspace()
    torch.cuda.empty_cache()
    fill = torch.empty(torch.cuda.mem_get_info()[0] - 3 * GIB, dtype=torch.uint8, device="cuda")
    G = _gamma(2, "cuda")
    E = torch.linspace(-6.9, 8.9, 100000, device="cuda", dtype=torch.float64)
    args = dict(e_min=-7.0, e_max=9.0, eta=0.3, orbitals_per_nm2=30.0, n_theta=1 << 20)
    got = K.reconstruct_sigma_bastin(G, E, **args)
    idx = torch.tensor([0, 1, 8190, 8191, 8192, 8193, 65535, 99999], device="cuda")
    assert torch.equal(K.reconstruct_sigma_bastin(G, E[idx], **args), got[idx])
    del fill
    torch.cuda.empty_cache()


def test_gamma_aligned_to_its_doubles(K):
    """A device Gamma whose first element lies 8 bytes past a 16-byte boundary."""
    import torch
    M = 70
    G = _gamma(M, "cuda")
    buf = torch.zeros(2 * M * M + 1, device="cuda", dtype=torch.float64)
    buf[1:] = G.flatten()
    odd = buf[1:].view(M, M, 2)
    assert G.data_ptr() % 16 == 0 and odd.data_ptr() % 16 == 8
    E = torch.linspace(-3.0, 3.0, 9, device="cuda", dtype=torch.float64)
    args = dict(e_min=-7.0, e_max=9.0, eta=0.3, orbitals_per_nm2=30.0)
    assert torch.equal(K.reconstruct_sigma_bastin(odd, E, **args), K.reconstruct_sigma_bastin(G, E, **args))
    om = torch.linspace(0.3, 3.0, 5, device="cuda", dtype=torch.float64)
    assert torch.equal(K.reconstruct_sigma_optical(odd, odd[0].contiguous(), om, 0.4, **args),
                       K.reconstruct_sigma_optical(G, G[0].contiguous(), om, 0.4, **args))
