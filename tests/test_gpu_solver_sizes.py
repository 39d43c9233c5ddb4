"""The dense solve at the sizes where its tiling changes: one step of worlds
whose row counts sit at the edges of 4-row quads, 16-row tiles and size
buckets, against the oracle with the GPU's restart decisions replayed.  The
bar is the parity tests' 1e-4 relative per world on u+ and the net impulses per
body (FP32 rows and factors, FP64 products)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2603_16536_amd import kamx, scenes  # noqa: E402

from parity_util import compare_worlds, gpu_step, summary  # noqa: E402

TOL = 1e-4
ITERS = 25


def check(scene, rows, name):
    p = dict(dt=1e-3, eta=1e-4, rho_bilateral=1e-4, rho_contact=0.3, fixed_iters=ITERS, max_iters=ITERS, log_restarts=1)
    g = gpu_step(scene, p)
    assert g["rows"].tolist() == rows
    assert np.all(g["status"] == 0) and np.all(g["iters"] == ITERS)
    rs = compare_worlds(scene, kamx.make_params(**p), g, list(range(scene.n_worlds)), mode="replay")
    print(summary(name, rs), flush=True)
    assert max(r["e_imp"] for r in rs) < TOL
    assert max(r["e_u"] for r in rs) < TOL


@pytest.mark.parametrize("joints", [1, 3, 4, 6, 7, 12, 13, 16, 19, 20, 25, 26, 32, 38, 39, 44])
def test_joint_rows_at_tile_edges(joints):
    """Chains of 1 to 44 links: 5 to 220 rows, every size bucket, with the
    rows ending before, at and after multiples of 4, 16 and 32."""
    rng = np.random.default_rng(100 + joints)
    one = [scenes.random_chain_world(rng, joints, with_limits=False, on_manifold=True) for _ in range(3)]
    check(scenes.round_to_f32(scenes.concat(one)), [5 * joints] * 3, f"{joints} joints")


@pytest.mark.parametrize("points", [1, 2, 5, 10, 11, 16, 21, 32, 43, 64])
def test_contact_rows_on_one_body(points):
    """One body carrying every row (3 to 192): the longest gather lists, and
    contacts whose rows lie in two wavefronts (from 11 points on)."""
    rng = np.random.default_rng(200 + points)
    one = [scenes.box_point_contacts(rng, points, mu=0.5, gap_scale=1e-3) for _ in range(3)]
    check(scenes.round_to_f32(scenes.concat(one)), [3 * points] * 3, f"{points} contacts")
