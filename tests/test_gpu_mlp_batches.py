"""FP32 products of large batches (64 x 64 tiles with short stages from 384 tiles on)
against the small batches' tiles: the sums run in the same order, so a row's outputs are
equal to the bit however many rows go with it.  Gradients are means over rows: those of
the whole batch against the mean over parts, 1e-4 (the gradient tolerance of the other
network tests), the loss 1e-6 (FP64 sums of squares of equal values, in parts)."""
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


# 97 x 4 and 97 x 5 tiles with a ragged last row of them; aligned and unaligned widths;
# contractions shorter than a stage and with a remainder; one tile short of the rule.
@pytest.mark.parametrize("n_in,n_hid,n_out,B", [(100, 252, 304, 6145), (101, 250, 303, 6145), (7, 193, 255, 6150),
                                                (101, 250, 303, 6080), (33, 70, 50, 24577)])
@pytest.mark.parametrize("scaled", [False, True], ids=["plain", "scaled"])
def test_rows_do_not_depend_on_the_batch(K, n_in, n_hid, n_out, B, scaled):
    import torch
    print(f"{n_in}-{n_hid}-{n_out} batch {B}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(B)
    net = K.MLP(n_in, n_hid, n_out, seed=4)
    x = torch.randn(B, n_in, generator=g, device="cuda")
    t = torch.randn(B, n_out, generator=g, device="cuda") + 0.2
    w = torch.rand(n_out, generator=g, device="cuda") + 0.1
    if scaled:
        net.fit_scaling(x[:500], t[:500])
    y = net.forward(x)
    parts = [slice(i, min(i + 512, B)) for i in range(0, B, 512)]
    for p in parts:
        assert torch.equal(net.forward(x[p]), y[p]), p
    grads, loss = net.gradients(x, t, w)
    mean, mean_loss = [np.zeros(a.shape) for a in grads], 0.0
    for p in parts:
        gp, lp = net.gradients(x[p].contiguous(), t[p].contiguous(), w)
        share = (p.stop - p.start) / B
        mean_loss += lp * share
        for a, b in zip(mean, gp):
            a += b * share
    assert abs(loss - mean_loss) <= 1e-6 * mean_loss
    for a, b in zip(grads, mean):
        assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b)
    net.close()
