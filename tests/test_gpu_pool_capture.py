"""Calls that take blocks from the pool and give them back while another thread captures
a stream: the pool makes no device-wide wait (which would fail, and end the capture)."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def _calls(K):
    g = np.random.default_rng(3)
    G = (g.standard_normal((64, 64)) + 1j * g.standard_normal((64, 64))) * 1e-2
    big = (g.standard_normal((900, 900)) + 1j * g.standard_normal((900, 900))) * 1e-2   # blocks above 16 MB
    E, mu = np.linspace(-2, 2, 7), g.standard_normal(64)
    return {
        "jackson": lambda: K.reconstruct_jackson(mu, E, -9.0, 9.0),
        "sigma": lambda: K.reconstruct_sigma(G, E, -9.0, 9.0, 30.0),
        "bastin": lambda: K.reconstruct_sigma_bastin(G, E, -9.0, 9.0, 0.2, 30.0, kT=0.1),
        "bastin, large": lambda: K.reconstruct_sigma_bastin(big, E, -9.0, 9.0, 0.2, 30.0),
        "optical": lambda: K.reconstruct_sigma_optical(G, G[0], np.array([0.5, 1.0]), 0.1, -9.0, 9.0, 0.2, 30.0),
    }


@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_calls_beside_another_threads_capture(K, mode):
    import torch
    calls = _calls(K)
    for name, f in calls.items():
        f()
        want = f()   # (its blocks are idle now)
        x = torch.zeros(1024, device="cuda")
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph, got = torch.cuda.CUDAGraph(), []

        def work():
            try:
                got.extend(f() for _ in range(3))
            except BaseException as e:   # noqa: BLE001 (reported by the main thread)
                got.append(e)

        print(f"{name} beside a capture ({mode})", flush=True)
        with torch.cuda.stream(s):
            graph.capture_begin(capture_error_mode=mode)
            x.add_(1)
            t = threading.Thread(target=work)
            t.start()
            t.join()
            graph.capture_end()
        assert len(got) == 3 and all(np.array_equal(r, want) for r in got), (name, got)
        for n in (1, 2):
            graph.replay()
            torch.cuda.synchronize()
            assert float(x.min()) == float(x.max()) == n
