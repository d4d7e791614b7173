"""Precomputation at the sizes where its kernels change shape: the inverses of the modal
matrices against LAPACK's, at matrix sizes around the blocks of 16 columns and the workgroup
sizes of the elimination."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context(shapes, kappa, M):
    """One body per (contour, ...) along x, far apart."""
    from paper_1406_0236_amd import Context
    ctx = Context(0)
    for k, c in enumerate(shapes):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, kappa, M, np.array([6.0 * k, 0.0, 0.0]), np.eye(3))
    ctx.precompute_scattering()
    return ctx


def _check_inverse(ctx, body, M, NG):
    A = ctx.modal_matrices(body, 0, M=M, NG=NG).cpu().numpy()
    S = ctx.modal_matrices(body, 1, M=M, NG=NG).cpu().numpy()
    for m in range(M + 1):
        ref = np.linalg.inv(A[m])
        cond = np.linalg.norm(A[m], 2) * np.linalg.norm(ref, 2)
        # elimination with partial pivoting: a backward error of about n eps, on either side
        tol = 2.0 * NG * np.finfo(np.float64).eps * cond
        err = np.linalg.norm(S[m] - ref, 2) / np.linalg.norm(ref, 2)
        assert err < tol, (NG, m, err, tol)


@pytest.mark.parametrize("n_panels,p", [(1, 2), (1, 15), (1, 16), (3, 11), (4, 16), (5, 13), (16, 16), (20, 13),
                                        (32, 16), (57, 9), (64, 16), (65, 16)])
def test_inverse_at_edges_of_blocks(n_panels, p):
    from workloads import geometry as geo
    M = 1 if n_panels * p > 512 else 3
    c = geo.sphere(1.0, n_panels, p)
    ctx = _context([c], 2.0, M)
    _check_inverse(ctx, 0, M, c.NG)
    ctx.close()


def test_inverse_of_shapes_of_different_sizes_together():
    from workloads import geometry as geo
    shapes = [geo.sphere(1.0, 2, 8), geo.prolate(0.8, 1.3, 7, 9), geo.sphere(0.9, 27, 10), geo.bowl(3, 2, 4, 10)]
    ctx = _context(shapes, 1.5, 2)
    for b, c in enumerate(shapes):
        _check_inverse(ctx, b, 2, c.NG)
    ctx.close()
