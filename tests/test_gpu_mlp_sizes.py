"""The network's row kernel and its one-launch gradients at the sizes where their
tiling changes: hidden layers that leave waves without a column tile (64), end in
the middle of a wave's tiles (192, 320), fill them (512) and are too wide (576: one
product per layer); inputs and outputs at and past a 64-column edge; batches
around 16-row blocks, 32-row operands and the slices of the weight gradients, and
one of 32-row workgroups.  Outputs, loss and gradients against the FP64 reference
with the same BF16 rounding points, the gradients again after an update (the update
writes the BF16 copies, transposed ones included); the bar of the network's other
tests, 2e-3 of each tensor's largest magnitude (the BF16 unit is 3.9e-3)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import mlp as M  # noqa: E402

from test_gpu_mlp import TOL, device_net, random_net, rel  # noqa: E402


def check_gradients(d, net, x, t, what):
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    d.train_step(x, t, 1e-3, loss=loss)
    g = d.gradients().cpu().numpy()
    ref, grads = M.loss_and_grads(net, x.astype(np.float64), t.astype(np.float64), bf16=True)
    assert abs(loss.item() - ref) <= 1e-4 * ref
    k = 0
    worst = 0.0
    for gr in grads:
        worst = max(worst, rel(g[k:k + gr.size].reshape(gr.shape), gr))
        k += gr.size
    print(f"{what}: gradients off by {worst:.1e}", flush=True)
    assert worst < TOL


@pytest.mark.parametrize("n_in,n_hidden,n_out,batch", [
    (1, 64, 1, 1), (64, 64, 64, 16), (65, 128, 65, 17), (100, 192, 130, 64), (130, 320, 40, 65), (300, 512, 100, 257),
    (70, 576, 30, 130), (1300, 64, 20, 33), (40, 256, 600, 100), (667, 256, 224, 1000)])
def test_network_sizes(n_in, n_hidden, n_out, batch):
    rng = np.random.default_rng(n_in + n_hidden)
    net = random_net(rng, n_in, n_hidden, n_out)
    d = device_net(net, batch)
    x = rng.normal(0, 2, (batch, n_in)).astype(np.float32)
    t = (net.mu_out[:n_out] + net.sigma_out[:n_out] * rng.normal(0, 1, (batch, n_out))).astype(np.float32)
    y = d.forward(x).cpu().numpy()
    ref, _ = M.forward(net, x.astype(np.float64), bf16=True)
    print(f"\n{n_in}-{n_hidden}-{n_out}, batch {batch}: outputs off by {rel(y, ref):.1e}", flush=True)
    assert rel(y, ref) < TOL
    check_gradients(d, net, x, t, "first step")
    w = d.weights().cpu().numpy().astype(np.float64)
    k = 0
    for p in net.params():
        p[...] = w[k:k + p.size].reshape(p.shape)
        k += p.size
    check_gradients(d, net, x, t, "second step")
    d.close()


@pytest.mark.parametrize("n_in,n_hidden", [(130, 128), (1300, 256)])
def test_rows_do_not_depend_on_the_batch(n_in, n_hidden):
    """Workgroups of 32 rows (large batches; past 64 KB of LDS for the wider network)
    and of 16 give a row the same bits."""
    rng = np.random.default_rng(5)
    net = random_net(rng, n_in, n_hidden, 70)
    n = 20000
    d = device_net(net, n)
    x = torch.as_tensor(rng.normal(0, 2, (n, n_in)).astype(np.float32), device="cuda")
    y = d.forward(x)
    for lo, hi in ((0, 1000), (9999, 11000), (n - 17, n)):
        assert torch.equal(y[lo:hi], d.forward(x[lo:hi].contiguous()))
    d.close()
