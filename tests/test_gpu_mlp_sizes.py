"""The network's products at the sizes where their tiles, K splits and edges change (one to 257
rows, rows of odd length, so that nothing is 16-byte aligned), layer by layer against the FP64
reference."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("width,depth,n_out,B", [
    (24, 1, 1, 1), (31, 3, 33, 5),       # 32 x 32 tiles
    (33, 1, 32771, 32),                  # 32 x 128 forward, 64 x 64 weights' gradient
    (512, 2, 70001, 20),                 # 32 x 128 both ways, K split
    (64, 1, 6001, 130),                  # 64 x 64 forward
    (512, 1, 8203, 250),                 # 64 x 64 with K split
    (130, 2, 16390, 257),                # 128 x 128 forward, 32 x 32 with K split
    (512, 1, 32770, 255),                # 128 x 128 throughout
])
def test_products_at_edges(width, depth, n_out, B):
    from oracle import mlp as ref
    from paper_1406_0236_amd import Context, Mlp
    print(f"[gpu] {width} x {depth} -> {n_out}, batch {B}", flush=True)
    ctx = Context(0)
    rng = np.random.default_rng(width + B)
    sizes = ref.layer_sizes(4, width, depth, n_out)
    p = ref.init_params(sizes, rng).astype(np.float32).astype(np.float64)
    p += (0.05 * rng.standard_normal(p.size)).astype(np.float32)
    p = p.astype(np.float32).astype(np.float64)
    net = Mlp(ctx, 4, width, depth, n_out)
    net.set_params(p)
    X = rng.standard_normal((B, 4)).astype(np.float32)
    T = rng.standard_normal((B, n_out)).astype(np.float32)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    # rounding of sums of up to max(sizes, B) terms of random sign, relative in the 2-norm,
    # through at most depth + 1 layers each way
    tol = 4 * (depth + 1) * np.finfo(np.float32).eps * np.sqrt(max(max(sizes), B))
    Yr, _ = ref.forward(p, sizes, X.astype(np.float64))
    Y = net.forward(Xd).cpu().numpy()
    assert np.linalg.norm(Y - Yr) <= tol * np.linalg.norm(Yr)
    lr, gr = ref.loss_and_grad(p, sizes, X.astype(np.float64), T.astype(np.float64))
    loss, g = net.gradient(Xd, Td)
    g = g.cpu().numpy()
    assert abs(loss - lr) <= tol * lr
    o = 0
    for a, b in zip(sizes, sizes[1:]):
        for n in (a * b, b):
            e = np.linalg.norm(g[o:o + n] - gr[o:o + n]) / np.linalg.norm(gr[o:o + n])
            assert e <= tol, (a, b, n, e, tol)
            o += n
    # the rows of a batch taken from a larger set on the device
    order = rng.permutation(B).astype(np.int32)
    l2 = net.train_epoch(Xd, Td, order, B, [1e-12])
    assert abs(l2 - lr) <= tol * lr
    net.close()
    ctx.close()


def test_gradient_that_fails_leaves_the_callers_array_alone():
    """No device memory for the workspace of a split product: the call fails before it writes."""
    import ctypes
    from paper_1406_0236_amd import Context, Mlp
    ctx = Context(0)
    net = Mlp(ctx, 4, 512, 1, 70001)
    B = 20
    X, T = torch.randn(B, 4, device="cuda:0"), torch.randn(B, 70001, device="cuda:0")
    net.forward(X)                  # the activations are there
    grad = torch.full((net.nparams,), 7.0, device="cuda:0")
    real = torch.cuda.caching_allocator_alloc
    try:
        # everything but large blocks: the partial sums of the loss, not the split product's workspace
        torch.cuda.caching_allocator_alloc = lambda n, *a: real(n, *a) if n < (1 << 20) else 1 // 0
        st = net.lib.axs_mlp_gradient(net.h, ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(T.data_ptr()), B, None,
                                      ctypes.c_void_p(grad.data_ptr()))
    finally:
        torch.cuda.caching_allocator_alloc = real
    torch.cuda.synchronize()
    assert st == -3, st
    assert bool((grad == 7.0).all())
    loss, g = net.gradient(X, T)    # and succeeds once there is memory
    assert np.isfinite(loss) and bool(torch.isfinite(g).all())
    net.close()
    ctx.close()


def test_parameters_set_while_the_stream_is_busy():
    """On a stream of its own that has not come to an earlier forward pass yet, new parameters take
    their turn: the pass before them uses the old ones, the pass after them the new ones."""
    from paper_1406_0236_amd import Context, Mlp
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = Context(0)
        net = Mlp(ctx, 4, 24, 2, 33)
        X = torch.randn(7, 4, device="cuda:0")
        p = [np.random.default_rng(k).standard_normal(net.nparams).astype(np.float32) for k in range(2)]
        want = []
        for q in p:
            net.set_params(q)
            want.append(net.forward(X).clone())
        net.set_params(p[0])
        torch.cuda.synchronize()
        torch.cuda._sleep(50_000_000)
        got0 = net.forward(X)
        net.set_params(p[1])
        got1 = net.forward(X)
        torch.cuda.synchronize()
        assert torch.equal(got0, want[0]) and torch.equal(got1, want[1])
        net.close()
        ctx.close()
