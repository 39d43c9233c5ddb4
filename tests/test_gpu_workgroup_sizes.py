"""Every workgroup size a row bucket is built for, at row counts next to the tile
edges of the bucket: the factorization, both passes over the triangle and the
reductions are laid out for the size (one wave alone at 32 rows; more thread groups
than row pairs at 32, 64, 96 and 160 rows), and give the default size's bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2603_16536_amd import kamx, scenes  # noqa: E402

P = dict(dt=1e-3, eta=1e-4, rho_bilateral=1e-4, rho_contact=0.3, eps=1e-6, max_iters=60)


def outputs(scene, contacts, variant):
    m = kamx.Model(scene, params=P, max_contacts=contacts)
    if contacts:
        m.upload_contacts(scene)
    sizes = m.buckets()[0]["variants"]
    if variant:
        m.set_bucket_threads(0, sizes[variant])
    m.step(2)
    st = m.stats()
    out = [t.cpu().numpy() for t in (*m.state(), m.impulses(), st["iters"], st["resid"], st["status"], st["rows"])]
    m.close()
    return out, sizes


def check(scene, contacts, rows):
    print(f"\n{rows} rows", flush=True)
    want, sizes = outputs(scene, contacts, 0)
    assert want[-1].tolist() == [rows] * scene.n_worlds and np.isfinite(want[1]).all()
    for v in range(1, len(sizes)):
        for k, (a, b) in enumerate(zip(outputs(scene, contacts, v)[0], want)):
            assert np.array_equal(a, b), (sizes[v], k)


@pytest.mark.parametrize("joints", [1, 3, 6, 7, 9, 10, 13, 16, 19, 20, 22, 25, 26, 29, 32, 35, 38])
def test_joint_rows(joints):
    rng = np.random.default_rng(500 + joints)
    one = [scenes.random_chain_world(rng, joints, with_limits=False, on_manifold=True) for _ in range(3)]
    check(scenes.round_to_f32(scenes.concat(one)), 0, 5 * joints)


@pytest.mark.parametrize("points", [1, 5, 11, 16, 21, 32, 43, 53, 64])
def test_contact_rows(points):
    rng = np.random.default_rng(600 + points)
    one = [scenes.box_point_contacts(rng, points, mu=0.5, gap_scale=1e-3) for _ in range(3)]
    check(scenes.round_to_f32(scenes.concat(one)), points, 3 * points)
