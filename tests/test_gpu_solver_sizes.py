"""The dense solve at the sizes where its tiling changes: one step (and forward
kinematics, which shares the factorization) of worlds
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

import oracle  # noqa: E402
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


@pytest.mark.parametrize("joints", [1, 2, 3, 8, 11, 16, 21, 24, 32, 37])
def test_kinematics_at_tile_edges(joints):
    """Chains with every joint targeted (6 to 222 rows).  The iteration stops at
    |F| <= 3e-7 in FP64; the poses it returns are rounded to FP32, half an ulp
    of the largest coordinate R per component and of 1 per quaternion entry, and a
    constraint sees four such roundings over levers of at most R."""
    tol = 3e-7
    rng = np.random.default_rng(300 + joints)
    one = [scenes.random_chain_world(rng, joints, with_limits=False, on_manifold=True) for _ in range(3)]
    scene = scenes.round_to_f32(scenes.concat(one))
    targets = rng.uniform(-0.2, 0.2, scene.n_joints).astype(np.float32)
    m = kamx.Model(scene)
    it, res = m.forward_kinematics(targets, max_iters=50, tol=tol)
    q = m.state()[0].cpu().numpy().astype(np.float64)
    it, res = it.cpu().numpy(), res.cpu().numpy()
    m.close()
    assert np.all(res <= tol) and np.all(it < 50)
    sg = scene.replace(q=q)
    R = np.abs(q[:, :3]).max()
    bound = tol + 4 * 2.0 ** -24 * (R + 2.0 * max(R, 1.0))
    f = max(np.abs(oracle.world_system(sg, oracle.Params(dt=scene.dt), w)["f"]).max() for w in range(3))
    c = max(abs(oracle.joint_coordinate(sg, q, j)[0] - targets[j]) for j in range(scene.n_joints))
    print(f"\n{joints} joints: {it.max()} iterations, constraints {f:.1e}, targets {c:.1e} (bound {bound:.1e})", flush=True)
    assert f < bound and c < bound


@pytest.mark.parametrize("kind,n", [("points", 1), ("points", 3), ("points", 4), ("points", 6), ("points", 7),
                                    ("points", 64), ("joints", 42), ("joints", 43), ("joints", 44)])
def test_matrix_free_gather_lists(kind, n):
    """The matrix-free product where a body's list goes past the rows its tasks hold
    in registers (3 to 192 rows on one body; ten are held, the rest is read in eights),
    and where there are more gather tasks than threads (more than 42 bodies on 256).
    The residuals come from the last product D~ x: against FP64 at the returned
    iterate, on the FP32 Jacobian.  J~ is rounded to FP32 after three operations and the
    sums are FP64, so with |J~| <= 1 per side and k rows on a body an entry of D~ x is off
    by at most 8 2^-24 2 k |x|, and v~_f and z by as many roundings of their own."""
    rng = np.random.default_rng(400 + n)
    if kind == "points":
        one, rows = [scenes.box_point_contacts(rng, n, mu=0.5, gap_scale=1e-3) for _ in range(2)], 3 * n
    else:
        one, rows = [scenes.random_chain_world(rng, n, with_limits=False, on_manifold=True) for _ in range(2)], 5 * n
    scene = scenes.round_to_f32(scenes.concat(one))
    p = dict(dt=1e-3, eta=1e-4, rho_bilateral=1e-4, rho_contact=0.3, fixed_iters=ITERS, max_iters=ITERS, log_restarts=1,
             linear_solver=kamx.SOLVER_SPARSE, cr_iters=9)
    g = gpu_step(scene, p)
    assert g["rows"].tolist() == [rows] * 2
    assert np.all(g["status"] == 0) and np.all(g["iters"] == ITERS)
    rs = compare_worlds(scene, kamx.make_params(**p), g, [0, 1], mode="replay", oracle_over=dict(cr_iters=9))
    it = np.abs(g["iterate"]).max(0)
    k = rows if kind == "points" else 10
    bound = 2.0 ** -21 * (2 * k * it[0] + 2 * it[2])
    d = max(np.abs(r["gpu_resid"][:3] - r["fp64_resid"])[:2].max() for r in rs)
    print(f"\n{n} {kind}, matrix-free: residuals off by {d:.1e} (bound {bound:.1e})", flush=True)
    assert d < bound
