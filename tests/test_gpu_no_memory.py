"""Calls that find no device memory fail with AXS_ENOMEM, and the same context serves later calls
as if they had not been made: whatever allocation it is that fails."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@contextlib.contextmanager
def _failing_at(n):
    """The n-th allocation from now on fails (and those after it succeed)."""
    real, count = torch.cuda.caching_allocator_alloc, [0]

    def alloc(*a):
        count[0] += 1
        if count[0] == n + 1:
            raise torch.OutOfMemoryError("none left")
        return real(*a)

    torch.cuda.caching_allocator_alloc = alloc
    try:
        yield count
    finally:
        torch.cuda.caching_allocator_alloc = real


def _check(fresh, small, large):
    """fresh(): a new state; small(state), large(state): calls of growing size.  Every allocation of
    the large call after a small one fails in turn; small and large calls afterwards are right."""
    from paper_1406_0236_amd import AxsError
    s = fresh()
    want_small, want_large = small(s), large(s)
    n = 0
    while True:
        s = fresh()
        small(s)
        with _failing_at(n) as count:
            try:
                large(s)
                assert count[0] <= n
                return n
            except AxsError as e:
                assert e.status == -3, e
        assert torch.equal(small(s), want_small), n
        assert torch.equal(large(s), want_large), n
        n += 1


@pytest.fixture(scope="module")
def contexts():
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    made = []

    def fresh():
        ctx = Context(0)
        for k, c in enumerate((geo.sphere(1.0, 2, 10), geo.prolate(0.8, 1.3, 3, 9))):
            ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, 2.0, 2.0, 8, np.array([3.0 * k, 0.0, 0.0]), np.eye(3))
        ctx.precompute_scattering()
        made.append(ctx)
        return ctx

    yield fresh
    for c in made:
        c.close()


def _vec(ctx, nrhs):
    g = torch.Generator(device="cuda:0").manual_seed(nrhs)
    return torch.randn((nrhs, ctx.N), dtype=torch.complex128, device="cuda:0", generator=g)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("sizes", [(1, 5), (16, 48), (3, 20)])
def test_operator(contexts, prec, sizes):
    n = _check(contexts, lambda c: c.apply_matvec(_vec(c, sizes[0]), prec), lambda c: c.apply_matvec(_vec(c, sizes[1]), prec))
    assert n >= 4


def test_fields(contexts):
    t = np.random.default_rng(0).uniform(5, 9, (700, 3))
    assert _check(contexts, lambda c: c.eval_field(_vec(c, 1), t[:20]), lambda c: c.eval_field(_vec(c, 40), t)) >= 2


def test_solves(contexts):
    from paper_1406_0236_amd import SOLVE_FP64, SOLVE_MIXED
    for mode in (SOLVE_FP64, SOLVE_MIXED):
        assert _check(contexts, lambda c: c.solve(_vec(c, 1), mode=mode, tol=1e-6)[0],
                      lambda c: c.solve(_vec(c, 4), mode=mode, tol=1e-8)[0]) >= 4


def test_training(contexts):
    from paper_1406_0236_amd import Mlp
    ctx = contexts()
    g = torch.Generator().manual_seed(0)
    X, T = torch.randn(64, 4, generator=g).cuda(), torch.randn(64, 40, generator=g).cuda()
    order = np.arange(64, dtype=np.int32)
    nets = []

    def fresh():
        net = Mlp(ctx, 4, 32, 2, 40)
        net.set_params(np.random.default_rng(1).standard_normal(net.nparams).astype(np.float32) * 0.1)
        nets.append(net)
        return net

    def epoch(batch, steps):
        # learning rates that leave the parameters as they are: the calls do not depend on those before
        return lambda net: torch.tensor([net.train_epoch(X, T, order[:batch * steps], batch, [1e-30] * steps)],
                                        dtype=torch.float64)

    assert _check(fresh, epoch(4, 2), epoch(16, 4)) >= 4
    for net in nets:
        net.close()
