"""Products with the dense blocks of point skeletons at the batch widths where their columns
(bodies of a shape x right-hand sides) are grouped differently: solves of a batch against the
solves of its columns one by one, and against the full system."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    ctx = Context(0)
    k, rng = 2.0, np.random.default_rng(3)
    sph, pro = geo.sphere(1.0, 4, 10), geo.prolate(0.8, 1.3, 4, 9)
    for b in range(5):
        c = pro if b in (1, 4) else sph
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, k, k, 10, np.array([5.0 * b, 0.3 * b, 0.0]),
                       geo.random_rotation(rng))
    ctx.precompute_scattering()
    ctx.skeletonize_points(1e-10)
    dirs = geo.fibonacci_directions(40)
    v = ctx.incident_plane_waves(dirs)
    from paper_1406_0236_amd import SOLVE_FP64
    single = [ctx.solve_skeleton(v[c:c + 1].contiguous(), mode=SOLVE_FP64, tol=1e-12)[0] for c in range(12)]
    full, _ = ctx.solve(v, mode=SOLVE_FP64, tol=1e-12)
    yield ctx, v, single, full
    ctx.close()


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 6, 11, 16, 40])
@pytest.mark.parametrize("mixed", [False, True])
def test_batches_of_every_width(scene, nrhs, mixed):
    from paper_1406_0236_amd import SOLVE_FP64, SOLVE_MIXED
    ctx, v, single, full = scene
    x = v[:nrhs].contiguous()
    got, info = ctx.solve_skeleton(x, mode=SOLVE_MIXED if mixed else SOLVE_FP64, tol=1e-11)
    assert all(i["converged"] for i in info)
    for c in range(min(nrhs, 12)):
        # both solved to 1e-11 (1e-12): the second-kind system's condition number times that
        e = float((got[c] - single[c][0]).norm() / single[c].norm())
        assert e < 1e-9, (c, e)
    # the IDs at 1e-10 leave a few 1e-9 at most on separated bodies
    e = float((got - full[:nrhs]).norm() / full[:nrhs].norm())
    assert e < 1e-8, e
