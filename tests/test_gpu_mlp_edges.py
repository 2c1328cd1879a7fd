"""The training kernels at the edges of their tiles and launches: a row on each
side of a 16-row tile, of a workgroup's four tiles and of the grid's first
turn; the loss on each side of its one-workgroup limit and of its chunks.
Against the float64 oracle; bounds as for the kernels' other tests."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def inputs(B, seed):
    rng = np.random.default_rng(seed)
    p = rng.uniform(-0.4, 0.4, mlp.NPAR).astype(np.float32)
    x = rng.uniform(0, 1, (B, 12)).astype(np.float32)
    d = (rng.normal(0, 1, (B, 5)) / B).astype(np.float32)
    return p, x, d


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 129])
def test_forward_and_backward(B):
    p, x, d = inputs(B, B)
    pd, xd, dd = (torch.tensor(a, device="cuda") for a in (p, x, d))
    logits, act = llp.mlp_forward(pd, xd)
    grad = torch.zeros(mlp.NPAR, dtype=torch.float32, device="cuda")
    llp.mlp_backward(pd, xd, act, dd, grad)
    torch.cuda.synchronize()
    a = (act.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    h1, h2 = a[:, :64], a[:, 64:]
    for got, want in ((h1, mlp.layer1(p, x)), (h2, mlp.layer2(p, h1))):
        assert np.all(np.abs(got - want) <= np.maximum(np.abs(want), 1e-30) * 2.0 ** -7 + 1e-30)
    want = mlp.layer3(p, h2)
    assert np.allclose(logits.cpu().numpy(), want, rtol=1e-4, atol=1e-5 * np.abs(want).max())
    want = mlp.backward(p, x, h1, h2, d)
    assert np.allclose(grad.cpu().numpy(), want, rtol=1e-4, atol=1e-6 * np.abs(want).max())


# 32768 rows are one tile for each wave of 512 workgroups of the backward pass,
# 65536 for each of the forward pass
@pytest.mark.parametrize("B", [32767, 32785, 65553])
def test_rows_of_a_large_batch(B):
    """A row's outputs don't depend on the batch it is in: bit for bit those of
    batches of 128 rows, and the batch's gradient is the oracle's."""
    p, x, d = inputs(B, B)
    pd, xd, dd = (torch.tensor(a, device="cuda") for a in (p, x, d))
    logits, act = llp.mlp_forward(pd, xd)
    for r in (0, 32640, B - 128):
        part, pact = llp.mlp_forward(pd, xd[r:r + 128].contiguous())
        assert torch.equal(part, logits[r:r + 128]) and torch.equal(pact, act[r:r + 128])
    grad = torch.zeros(mlp.NPAR, dtype=torch.float32, device="cuda")
    llp.mlp_backward(pd, xd, act, dd, grad)
    torch.cuda.synchronize()
    a = (act.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    want = mlp.backward(p, x, a[:, :64], a[:, 64:], d)
    assert np.allclose(grad.cpu().numpy(), want, rtol=1e-4, atol=1e-6 * np.abs(want).max())


@pytest.mark.parametrize("over", [False, True])
@pytest.mark.parametrize("B", [1, 1023, 4096, 4097, 5119, 5120, 5121])
def test_loss(B, over):
    """`over`: the gradients written over the logits."""
    rng = np.random.default_rng(B)
    z = rng.normal(0, 3, (B, 5)).astype(np.float32)
    labels = (rng.integers(0, 3, B) | (rng.integers(0, 3, B) << 8)).astype(np.int32)
    zd, yd = torch.tensor(z, device="cuda"), torch.tensor(labels, device="cuda")
    if over:
        dl, loss = zd, torch.zeros(1, device="cuda")
        assert llp.lib().llp_mlp_loss(B, zd.data_ptr(), yd.data_ptr(), zd.data_ptr(), loss.data_ptr(), llp._stream()) == 0
    else:
        loss, dl = llp.mlp_loss(zd, yd)
    torch.cuda.synchronize()
    want_l, want_d = mlp.loss(z, labels)
    assert abs(float(loss.item()) - want_l) <= 1e-5 * max(abs(want_l), 1.0)
    assert np.allclose(dl.cpu().numpy(), want_d, rtol=1e-4, atol=1e-6 / B)   # a few units in the last place of a probability
