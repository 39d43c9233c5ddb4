"""The step's own inference on networks of either weight order (the row kernel's blocks,
and row-major above 512 hidden columns): a learned step equals one warm started
from outside with the network's prediction, bit for bit, before and after a training
step has rewritten the BF16 weights."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2603_16536_amd import kamx  # noqa: E402

from test_gpu_mlp import BIPED, biped_model, device_net, random_net, slots_to_rows  # noqa: E402


@pytest.mark.parametrize("hidden", [64, 512, 576])
def test_learned_step_equals_external(hidden):
    n = 6
    _, cold = biped_model(n, BIPED)
    nf, ns = cold.feature_dims()
    rng = np.random.default_rng(hidden)
    net = device_net(random_net(rng, nf, hidden, ns), n)
    x = torch.as_tensor(rng.normal(0, 1, (n, nf)).astype(np.float32), device="cuda")
    t = torch.as_tensor(rng.normal(0, 1, (n, ns)).astype(np.float32), device="cuda")
    for trained in (False, True):
        if trained:
            net.train_step(x, t, 1e-2)
        scene, A = biped_model(n, BIPED)
        _, B = biped_model(n, BIPED)
        _, C = biped_model(n, BIPED)
        pred = net.forward(A.features()).cpu().numpy()
        A.attach_mlp(net)
        A.set_params(**dict(BIPED, warmstart=kamx.WARM_LEARNED, max_iters=50))
        A.step(1)
        C.step(1)  # reveals the contact order
        B.set_params(**dict(BIPED, warmstart=kamx.WARM_EXTERNAL, max_iters=50))
        B.set_warmstart(slots_to_rows(pred, C, scene)[0])
        B.step(1)
        for a, b in zip((*A.state(), A.impulses(), A.stats()["iters"]), (*B.state(), B.impulses(), B.stats()["iters"])):
            assert torch.equal(a, b), trained
        for m in (A, B, C):
            m.close()
    net.close()
    cold.close()


@pytest.mark.parametrize("n_in,hidden,n_out", [(20, 320, 60), (20, 448, 130), (64, 512, 64), (64, 384, 64), (128, 448, 65),
                                               (20, 256, 20)])
def test_large_batches(n_in, hidden, n_out):
    """Above 32768 rows wide hidden layers between narrow ends predict through one product
    per layer: the bits of the row kernel on a part of the rows, in place too."""
    rng = np.random.default_rng(n_in + hidden)
    n = 33000
    net = device_net(random_net(rng, n_in, hidden, n_out), n)
    x = torch.as_tensor(rng.normal(0, 2, (n, n_in)).astype(np.float32), device="cuda")
    y = net.forward(x)
    for lo, hi in ((0, 1000), (20000, 32768), (n - 300, n)):
        assert torch.equal(y[lo:hi], net.forward(x[lo:hi].contiguous()))
    buf = torch.zeros(n * max(n_in, n_out), dtype=torch.float32, device="cuda")
    xv, yv = buf[:n * n_in].view(n, n_in), buf[:n * n_out].view(n, n_out)
    xv.copy_(x)
    assert torch.equal(net.forward(xv, out=yv), y)
    net.close()
