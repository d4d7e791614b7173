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


@pytest.mark.parametrize("M,kappa", [(0, 1.0), (1, 0.0), (20, 3.0), (40, 0.5)])
def test_node_geometry_at_small_and_ragged_sizes(M, kappa):
    """Node positions, normals and weights of rotated bodies of different shapes against their
    closed form in numpy; positions of mirrored azimuths of an unrotated body mirror exactly."""
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    rng = np.random.default_rng(2)
    shapes = [geo.sphere(1.0, 1, 3), geo.prolate(0.7, 1.4, 7, 11), geo.bowl(2, 2, 3, 8)]
    poses = [(np.array([5.0 * k, -1.0, 0.3]), np.eye(3) if k == 0 else geo.random_rotation(rng)) for k in range(3)]
    ctx = Context(0)
    for c, (x0, rot) in zip(shapes, poses):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, 1.0, M, x0, rot)
    ctx.precompute_scattering()
    got = ctx.node_geometry()
    NF, rows = 2 * M + 1, []
    for c, (x0, rot) in zip(shapes, poses):
        th = 2 * math.pi * np.arange(NF) / NF
        r, z = c.rz[:, :1], c.rz[:, 1:]
        sp = np.hypot(c.drz[:, :1], c.drz[:, 1:])
        nr, nz = -c.drz[:, 1:] / sp, c.drz[:, :1] / sp
        one = np.ones((1, NF))
        loc = np.stack([r * np.cos(th), r * np.sin(th), z * one], -1).reshape(-1, 3)
        nl = np.stack([nr * np.cos(th), nr * np.sin(th), nz * one], -1).reshape(-1, 3)
        w = ((2 * math.pi / NF) * r * sp * c.gw[:, None] * one).reshape(-1, 1)
        rows.append(np.concatenate([loc @ rot.T + x0, nl @ rot.T, w], 1))
    ref = np.concatenate(rows)
    # a handful of roundings at the size of the coordinates (up to 12)
    assert np.max(np.abs(got - ref)) < 12 * 8 * np.finfo(np.float64).eps
    first = got[:shapes[0].NG * NF].reshape(-1, NF, 7)
    if M:
        assert np.array_equal(first[:, 1:, 0], first[:, :0:-1, 0])
    ctx.close()


@pytest.mark.parametrize("kind,kappa,eta,M", [("sphere2", 1.0, 1.0, 20), ("bowl", 2 * math.pi, 2 * math.pi, 12),
                                              ("prolate", 0.0, 1.0, 20), ("prolate16", 3.0, 3.0, 10)])
def test_modal_matrices_against_the_reference(kind, kappa, eta, M):
    """A~_m with the graded rules of own and neighbouring panels against the reference's
    tanh-sinh product integrals, on a few target rows.  The reference refines until two steps agree to
    2e-12 of the largest entry at worst; the bound is five times that."""
    from oracle.nystrom import Shape
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    c = {"sphere2": lambda: geo.sphere(1.0, 2, 10), "bowl": lambda: geo.bowl(3, 2, 4, 10),
         "prolate": lambda: geo.prolate(0.5, 1.0, 5, 10),
         "prolate16": lambda: geo.prolate(0.8, 1.3, 3, 16)}[kind]()
    ctx = Context(0)
    ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, eta, M, np.zeros(3), np.eye(3))
    ctx.precompute_scattering()
    A = ctx.modal_matrices(0, 0, M=M, NG=c.NG).cpu().numpy()
    ref = Shape(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, eta, M, Nt=128)
    for i in sorted({0, c.p - 1, c.p, c.NG // 2, c.NG - 1}):
        row = ref.modal_row(i)
        row[:, i] += 0.5
        err = np.max(np.abs(A[:, i, :] - row)) / np.max(np.abs(row))
        assert err < 1e-11, (kind, i, err)
    ctx.close()


@pytest.mark.parametrize("panels,kappa,eta,M", [(3, 1.0, 1.0, 0), (3, 2.0, 2.0, 31), (3, 1.0, 1.0, 32), (3, 1.0, 1.0, 47),
                                                (3, 1.0, 1.0, 50), (2, 0.0, 1.0, 40), (2, 0.0, 1.0, 64),
                                                (16, 45.0, 45.0, 70)])
def test_modal_values_at_edges(panels, kappa, eta, M):
    """The modal kernel at the numbers of modes and samples where its split changes, with more modes
    than series terms, and with four points a workgroup; bound as above."""
    from oracle.nystrom import Shape
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    c = geo.sphere(1.0, panels, 10)
    ctx = Context(0)
    ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, eta, M, np.zeros(3), np.eye(3))
    ctx.precompute_scattering()
    A = ctx.modal_matrices(0, 0, M=M, NG=c.NG).cpu().numpy()
    ref = Shape(c.rz, c.drz, c.gw, c.n_panels, c.p, kappa, eta, M, Nt=512 if kappa > 10 else 256)
    for i in (0, c.NG // 2 + 3):
        row = ref.modal_row(i)
        row[:, i] += 0.5
        err = np.max(np.abs(A[:, i, :] - row)) / np.max(np.abs(row))
        assert err < 1e-11, (i, err)
    ctx.close()


@pytest.mark.parametrize("M", [3, 20])
def test_shapes_together_as_alone(M):
    """Shapes of one p, M and number of samples are set up in common launches: the same bits as
    each of them by itself, matrices and inverses."""
    from workloads import geometry as geo
    shapes = [geo.sphere(1.0, 1, 10), geo.prolate(0.8, 1.3, 7, 10), geo.sphere(0.9, 4, 10), geo.prolate(0.5, 1.0, 3, 9),
              geo.bowl(3, 2, 4, 10)]
    ctx = _context(shapes, 1.5, M)
    for b, c in enumerate(shapes):
        one = _context([c], 1.5, M)
        for which in (0, 1):
            got = ctx.modal_matrices(b, which, M=M, NG=c.NG).cpu().numpy()
            assert np.array_equal(got, one.modal_matrices(0, which, M=M, NG=c.NG).cpu().numpy()), (b, which)
        one.close()
    ctx.close()


def test_inverses_as_exact_as_row_by_row_elimination():
    """Rounding of the blocked elimination: the inverses' errors (against inverses refined with residuals
    in extended precision), averaged over shapes and modes, are no larger than those of an ordinary
    Gauss-Jordan elimination of one column at a time with partial pivoting."""
    from workloads import geometry as geo

    def refined(A):
        R, A2 = np.linalg.inv(A), A.astype(np.clongdouble)
        for _ in range(2):
            R = R + np.linalg.solve(A, (np.eye(len(A)) - A2 @ R.astype(np.clongdouble)).astype(np.complex128))
        return R

    def by_columns(A):
        n = len(A)
        w = np.concatenate([A, np.eye(n)], 1).astype(np.complex128)
        for k in range(n):
            i = k + int(np.argmax(np.abs(w[k:, k])))
            w[[k, i]] = w[[i, k]]
            w[k] *= 1.0 / w[k, k]
            f = w[:, k].copy()
            f[k] = 0.0
            w -= np.outer(f, w[k])
        return w[:, n:]

    M, got, ref = 9, [], []
    for c, kappa in ((geo.sphere(1.0, 1, 16), 1.0), (geo.sphere(1.0, 4, 10), 2.0), (geo.prolate(0.8, 1.3, 7, 9), 3.0),
                     (geo.bowl(3, 2, 4, 10), 6.0), (geo.sphere(1.0, 12, 10), 6.0)):
        ctx = _context([c], kappa, M)
        A = ctx.modal_matrices(0, 0, M=M, NG=c.NG).cpu().numpy()
        S = ctx.modal_matrices(0, 1, M=M, NG=c.NG).cpu().numpy()
        ctx.close()
        for m in range(0, M + 1, 3):
            R = refined(A[m])
            got.append(np.log(np.linalg.norm(S[m] - R)))
            ref.append(np.log(np.linalg.norm(by_columns(A[m]) - R)))
    ratio = math.exp(np.mean(got) - np.mean(ref))
    print(f"error of the inverses, blocked over column by column: {ratio:.3f}")
    assert ratio <= 1.0, ratio


def test_refused_wavenumber_leaves_nothing_behind():
    """A wavenumber beyond the modal kernel's LDS is refused before anything is allocated or
    queued, every time, and the device is as it was for another context."""
    import torch
    from paper_1406_0236_amd import AxsError, Context
    from workloads import geometry as geo
    ctx = Context(0)
    c = geo.sphere(1.0, 4, 10)
    for b in range(2):     # a shape that is taken beside one that is not
        f = 0.01 if b == 0 else 1.0
        ctx.build_body(c.rz * f, c.drz * f, c.gw, c.n_panels, c.p, 400.0, 400.0, 20, np.array([6.0 * b, 0.0, 0.0]),
                       np.eye(3))
    before = torch.cuda.memory_allocated()
    for _ in range(2):
        with pytest.raises(AxsError, match="EINVAL.*too large for the modal kernel"):
            ctx.precompute_scattering()
        assert torch.cuda.memory_allocated() == before
    ctx.close()
    ok = _context([geo.sphere(1.0, 2, 8)], 1.0, 2)
    _check_inverse(ok, 0, 2, 16)
    ok.close()


def test_shapes_of_long_and_short_panels_together_as_alone():
    """Panels of more than 5 / kappa take more points a level; the shapes beside them do not."""
    from workloads import geometry as geo
    M, kappa = 6, 4.0     # kappa times the longest panel: 6.3, 3.1 and 12.6
    shapes = [geo.sphere(1.0, 2, 10), geo.sphere(1.0, 4, 10), geo.sphere(0.99, 1, 10)]
    ctx = _context(shapes, kappa, M)
    for b, c in enumerate(shapes):
        one = _context([c], kappa, M)
        for which in (0, 1):
            got = ctx.modal_matrices(b, which, M=M, NG=c.NG).cpu().numpy()
            diff = float(np.max(np.abs(got - one.modal_matrices(0, which, M=M, NG=c.NG).cpu().numpy())))
            assert diff == 0.0, (b, which, diff)
        one.close()
    ctx.close()
