"""Worlds without a single row in a step (bodies that touch nothing, no joints): there
is no triangle to factor, whatever earlier steps and other worlds left in LDS, so
the step is status OK with zero residuals and u+ = u_f, the oracle's velocity (FP32 of
a sum of three terms: 4 2^-24 of its largest)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2603_16536_amd import kamx, scenes  # noqa: E402

P = dict(dt=1e-3, eta=1e-4, rho_bilateral=1e-4, rho_contact=0.3, eps=1e-6, max_iters=50)
WORLDS = 600  # more than the compute units hold


def boxes(points, seed):
    rng = np.random.default_rng(seed)
    one = [scenes.box_point_contacts(rng, points, mu=0.5) for _ in range(20)]
    return scenes.round_to_f32(scenes.concat([one[w % 20] for w in range(WORLDS)]))


def without_contacts(scene, keep=lambda w: False):
    k = np.array([keep(w) for w in scene.contact_world], bool)
    names = [n for n in vars(scene) if n.startswith("contact_")]
    return scene.replace(**{n: getattr(scene, n)[k] for n in names})


def check(m, u0, free):
    """The free worlds' last step, from the twists u0."""
    st = {k: v.cpu().numpy() for k, v in m.stats().items()}
    u = m.state()[1].cpu().numpy().astype(np.float64)
    assert np.all(st["rows"][free] == 0)
    print("\nstatus of worlds without rows:", np.bincount(st["status"][free], minlength=1), flush=True)
    assert np.all(st["status"][free] == 0) and np.all(st["resid"][free] == 0)
    assert np.all(st["iters"][free] <= 1)
    return np.abs(u[free] - u0[free]).max()


def reference(scene):
    ref = oracle.step(scene, oracle.Params(dt=1e-3, eta=1e-4, rho_bil=1e-4, rho_c=0.3, max_iters=50, eps=1e-6))["u"]
    return ref, 4 * 2.0 ** -24 * np.abs(ref).max()


@pytest.mark.parametrize("points", [3, 10, 20, 60])
def test_after_a_model_with_contacts(points):
    scene = boxes(points, 700 + points)
    m = kamx.Model(scene, params=P, max_contacts=points)
    m.upload_contacts(scene)
    m.step(1)
    m.close()
    free = without_contacts(scene)
    m = kamx.Model(free, params=P, max_contacts=points)
    m.upload_contacts(free)
    m.step(1)
    ref, bound = reference(free)
    assert check(m, ref, np.arange(WORLDS)) <= bound
    m.step(3)  # one launch, its steps one after the other on a world
    check(m, ref, np.arange(WORLDS))
    m.close()


@pytest.mark.parametrize("points", [10, 20])
def test_beside_and_after_contacts(points):
    """Every second world free in a batch, then the others too on the same model."""
    scene = boxes(points, 800 + points)
    half = without_contacts(scene, keep=lambda w: w % 2 == 0)
    odd = np.arange(1, WORLDS, 2)
    m = kamx.Model(half, params=P, max_contacts=points)
    m.upload_contacts(half)
    m.step(1)
    ref, bound = reference(without_contacts(scene))
    assert check(m, ref, odd) <= bound
    m.upload_contacts(without_contacts(scene))
    m.step(1)
    check(m, ref, np.arange(WORLDS))
    m.close()


@pytest.mark.parametrize("solver", ["dense", "sparse"])
@pytest.mark.parametrize("over,iters,status,log", [
    (dict(), 1, 0, [0]),
    (dict(eps=0.0, max_iters=7), 7, 1, [0, 1, 1, 1, 1, 1, 1]),
    (dict(fixed_iters=4, max_iters=6), 4, 0, [0, 1, 1, 1]),
    (dict(fixed_iters=4, max_iters=3, accel=0), 4, 0, [0, 0, 0]),
    (dict(fixed_iters=3, max_iters=3, warmstart=1), 3, 0, [0, 1, 1])])
def test_what_the_iteration_would_report(solver, over, iters, status, log):
    """Iterations, status and restart log of worlds without rows are those of the loop on
    zero residuals: out at the first iteration, unless eps or a fixed count keep it
    going; every later one restarts the acceleration."""
    scene = without_contacts(boxes(5, 900))
    p = dict(P, log_restarts=1, linear_solver=kamx.SOLVER_SPARSE if solver == "sparse" else kamx.SOLVER_DENSE)
    p.update(over)
    m = kamx.Model(scene, params=p, max_contacts=5)
    m.upload_contacts(scene)
    m.step(2)
    st = {k: v.cpu().numpy() for k, v in m.stats().items()}
    assert np.all(st["rows"] == 0) and np.all(st["resid"] == 0)
    assert np.all(st["iters"] == iters) and np.all(st["status"] == status)
    got = m.restart_log().cpu().numpy()[:, :len(log)]
    assert np.array_equal(got, np.tile(np.array(log, np.uint8), (WORLDS, 1)))
    assert np.all(m.impulses().cpu().numpy() == 0)
    m.close()
