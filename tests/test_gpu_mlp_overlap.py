"""Predictions written over their own inputs: a serving loop that keeps one buffer
passes an ``out`` that shares memory with ``x``.  All of x counts as read before the
first output is written, whatever the overlap, as with separate buffers; the same
bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from test_gpu_mlp import device_net, random_net  # noqa: E402


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n_in,n_hidden,n_out", [(130, 128, 40), (40, 64, 130), (96, 256, 96), (70, 576, 30)])
@pytest.mark.parametrize("batch", [1, 17, 1000, 4500])
def test_out_over_x(n_in, n_hidden, n_out, batch, noalloc):
    if noalloc and n_hidden == 576 and batch == 4500:
        batch = 4096  # the fixed workspace's rows at this width
    rng = np.random.default_rng(n_in + batch)
    net = random_net(rng, n_in, n_hidden, n_out)
    d = device_net(net, batch)
    x = torch.as_tensor(rng.normal(0, 2, (batch, n_in)).astype(np.float32), device="cuda")
    want = d.forward(x)
    size = batch * max(n_in, n_out)
    # out at the start of x, x at the start of out's second half, and one float apart
    for xo, yo in ((0, 0), (size // 2, 0), (0, size // 2), (1, 0)):
        buf = torch.zeros(2 * size + 1, dtype=torch.float32, device="cuda")
        xv = buf[xo:xo + batch * n_in].view(batch, n_in)
        yv = buf[yo:yo + batch * n_out].view(batch, n_out)
        xv.copy_(x)
        (d.forward_noalloc if noalloc else d.forward)(xv, out=yv)
        assert torch.equal(yv, want), (xo, yo)
    d.close()
