"""The block-diagonal preconditioner D^{-1} at the sizes where its kernels change shape (contour
nodes per DFT block, the split of the per-mode products' inner dimension, ragged shapes together),
against the same steps in numpy's FP64 from the library's own S_m."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(ctx, bodies, x):
    out, off = np.empty_like(x), 0
    for k, (c, M) in enumerate(bodies):
        NF = 2 * M + 1
        S = ctx.modal_matrices(k, 1, M=M, NG=c.NG).cpu().numpy()
        w = x[:, off:off + c.NG * NF].reshape(-1, c.NG, NF)
        W = np.fft.fft(w, axis=2)
        Y = np.empty_like(W)
        for f in range(NF):
            m = min(f, NF - f)
            Y[:, :, f] = W[:, :, f] @ S[m].T
        out[:, off:off + c.NG * NF] = np.fft.ifft(Y, axis=2).reshape(x.shape[0], -1)
        off += c.NG * NF
    return out


@pytest.mark.parametrize("M", [0, 1, 7, 20])
@pytest.mark.parametrize("nrhs", [1, 2, 5, 33, 70])
def test_precond_at_edges(M, nrhs):
    import torch
    from paper_1406_0236_amd import FP32, FP64, Context
    from workloads import geometry as geo
    # 2, 15, 16, 17 (of 1 panel: at most 16), 64, 70 and 117 contour nodes
    shapes = [geo.sphere(1.0, 1, 2), geo.sphere(0.9, 1, 15), geo.prolate(0.8, 1.2, 1, 16), geo.sphere(1.0, 4, 16),
              geo.prolate(0.7, 1.3, 7, 10), geo.sphere(0.8, 9, 13)]
    ctx = Context(0)
    bodies = []
    for k, c in enumerate(shapes):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, 1.5, 1.5, M, np.array([4.0 * k, 0.0, 0.0]), np.eye(3))
        bodies.append((c, M))
    ctx.precompute_scattering()
    rng = np.random.default_rng(M + nrhs)
    x = rng.standard_normal((nrhs, ctx.N)) + 1j * rng.standard_normal((nrhs, ctx.N))
    ref = _reference(ctx, bodies, x)
    dev = torch.from_numpy(x).to("cuda:0")
    # sums over up to 117 x 41 terms of |S_m| <= a few: n eps with the growth of the two transforms
    # (N_F) and the products (N_G), relative to the largest entry
    grow = 4 * (117 + 41)
    for prec, eps in ((FP64, np.finfo(np.float64).eps), (FP32, np.finfo(np.float32).eps)):
        got = ctx.apply_precond(dev, prec).cpu().numpy()
        err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
        assert err < grow * eps, (prec, err)
    ctx.close()
