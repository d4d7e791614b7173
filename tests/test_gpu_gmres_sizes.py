"""GMRES at the sizes where its Gram-Schmidt kernels change shape (entries per workgroup, partial
sums added up by their readers or ahead of them, more vectors than one pass holds), against the
minimal residual over the same Krylov space by numpy's QR and least squares, with the library's
own operator; and the augmented inner runs of mixed mode by their FP64 residual."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _krylov_residuals(op, b, steps):
    """min ||b - A y|| / ||b|| over span(b, ..., A^(k-1) b), k = 1..steps, per row of b"""
    V = [b / np.linalg.norm(b, axis=1, keepdims=True)]
    W = []
    for _ in range(steps):
        w = op(V[-1])
        W.append(w.copy())
        for _ in range(2):
            for v in V:
                w = w - v * np.sum(v.conj() * w, axis=1, keepdims=True)
        V.append(w / np.maximum(np.linalg.norm(w, axis=1, keepdims=True), 1e-300))
    out = np.empty((b.shape[0], steps))
    for c in range(b.shape[0]):
        for k in range(1, steps + 1):
            Q = np.linalg.qr(np.stack([w[c] for w in W[:k]], axis=1))[0]
            r = b[c] - Q @ (Q.conj().T @ b[c])
            out[c, k - 1] = np.linalg.norm(r) / np.linalg.norm(b[c])
    return out


# (panels, p, M, bodies, rhs): 4, 510, 576, 5740 and 48,600 nodes in all
@pytest.mark.parametrize("panels,p,M,nb,nrhs", [(1, 2, 0, 2, 1), (1, 15, 8, 2, 3), (2, 16, 4, 2, 1), (7, 10, 20, 2, 1),
                                                (7, 10, 20, 2, 50), (7, 10, 20, 2, 100), (7, 10, 20, 2, 200),
                                                (20, 10, 40, 3, 1)])
def test_gmres_at_edges(panels, p, M, nb, nrhs):
    import torch
    from paper_1406_0236_amd import FP64, SOLVE_FP64, SOLVE_MIXED, Context
    from workloads import geometry as geo
    c = geo.sphere(1.0, panels, p)
    ctx = Context(0)
    for k in range(nb):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, 1.5, 1.5, M, np.array([2.4 * k, 0.3 * k, 0.0]), np.eye(3))
    ctx.precompute_scattering()
    rng = np.random.default_rng(panels + nrhs)
    v = rng.standard_normal((nrhs, ctx.N)) + 1j * rng.standard_normal((nrhs, ctx.N))
    v = torch.from_numpy(v).to("cuda:0")
    b = -ctx.apply_precond(v, FP64).cpu().numpy()

    def op(x):
        return ctx.apply_matvec(torch.from_numpy(x).to("cuda:0"), FP64).cpu().numpy()

    x, info = ctx.solve(v, mode=SOLVE_FP64, tol=1e-9, max_iters=40)
    steps = max(i["iterations"] for i in info)
    # both sides carry rounding of about steps x sqrt(N) x eps relative to ||b||
    slack = 40 * np.sqrt(ctx.N) * np.finfo(np.float64).eps
    some = list(range(nrhs))[::max(1, nrhs // 4)]
    ref = _krylov_residuals(op, b[some], steps)
    res = np.linalg.norm(b - op(x.cpu().numpy()), axis=1) / np.linalg.norm(b, axis=1)
    for c_, i in enumerate(info):
        assert i["converged"] and abs(res[c_] - i["rel_residual"]) < slack, (c_, res[c_], i)
    for row, c_ in enumerate(some):
        k = info[c_]["iterations"]
        assert abs(ref[row, k - 1] - info[c_]["rel_residual"]) < slack, (c_, ref[row], info[c_])
    x, info = ctx.solve(v, mode=SOLVE_MIXED, tol=1e-10, max_iters=40)
    res = np.linalg.norm(b - op(x.cpu().numpy()), axis=1) / np.linalg.norm(b, axis=1)
    assert all(i["converged"] for i in info) and np.max(res) < 1e-10 + slack, np.max(res)
    # more steps than one pass over the coefficients holds
    if ctx.N > 1000 and nrhs == 1:
        x2, info = ctx.solve(v, mode=SOLVE_FP64, tol=1e-300, max_iters=45)
        res = np.linalg.norm(b - op(x2.cpu().numpy()), axis=1) / np.linalg.norm(b, axis=1)
        assert np.max(res) < slack, (np.max(res), info)
    ctx.close()
