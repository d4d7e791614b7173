"""Source chunks of the FP32 MFMA orders.  interbody_mfma_kernel adds up a whole chunk in FP32 and the
chunks meet in FP64, so its chunks are never longer than 4,096 workgroups of 128 targets (at most
64 chunks) make them, whatever the number of right-hand sides."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[2, 8])
def scene(request):
    import torch
    import numpy as np
    from paper_1406_0236_amd import Context
    from workloads import geometry as geo
    ctx = Context(0)
    nb, k = request.param, 3.0
    c = geo.sphere(1.0, 10 if nb == 2 else 6, 10)
    for b in range(nb):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, k, k, 20,
                       np.array([2.6 * (b % 2), 2.6 * (b // 2 % 2), 2.6 * (b // 4)]), np.eye(3))
    ctx.precompute_scattering()
    gen = torch.Generator(device="cuda:0").manual_seed(nb)
    x = torch.randn((64, ctx.N), dtype=torch.complex128, device="cuda:0", generator=gen)
    tiles, splits = nb * -(-c.NG * 41 // 128), 1
    while tiles * splits < 4096 and splits < 64:
        splits *= 2
    yield ctx, x, splits
    ctx.close()


@pytest.mark.parametrize("variant,nrhs", [(3, 16), (3, 31), (3, 32), (3, 64), (0, 17), (0, 20), (0, 31), (0, 50)])
def test_fp32_mfma_order_adds_up_no_longer_chunks(scene, variant, nrhs):
    """The default chunks give the bits of the chunks by that rule (empty ones are left out)."""
    from paper_1406_0236_amd import FP32
    ctx, x, splits = scene
    x = x[:nrhs].contiguous()
    try:
        ctx.set_interbody_config(FP32, variant, 0, 0, 0)
        shape = ctx.interbody_launch_shape(FP32, nrhs)
        got = ctx.apply_interbody(x, FP32)
        ctx.set_interbody_config(FP32, shape[0], shape[1], shape[2], splits)
        ref = ctx.apply_interbody(x, FP32)
    finally:
        ctx.set_interbody_config(FP32, 0, 0, 0, 0)
    diff = float((got - ref).abs().max())
    assert diff == 0.0, (shape, splits, diff)


def test_fp16_multiply_accumulate_sums_any_chunk_alike():
    """Sums of 19,680 terms of nearly one sign: the error against FP64 with all sources in one chunk
    is that with 64 chunks.  What a longer FP32 sum may add is the rounding of its last
    addition, 2^-24 / sqrt(3) of the result against about 5 * 2^-24 in all: within 3 %."""
    import numpy as np
    import torch
    from paper_1406_0236_amd import Context, FP32, FP64
    from workloads import geometry as geo
    ctx = Context(0)
    c = geo.sphere(1.0, 6, 10)
    for b in range(8):
        ctx.build_body(c.rz, c.drz, c.gw, c.n_panels, c.p, 1.0, 1.0, 20,
                       np.array([2.6 * (b % 3), 2.6 * (b // 3), 0.0]), np.eye(3))
    ctx.precompute_scattering()
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    x = 1 + 0.2 * torch.rand((16, ctx.N), dtype=torch.float64, device="cuda:0", generator=gen) + 0j
    ref = ctx.apply_interbody(x, FP64)
    err = {}
    for splits in (1, 3, 64):
        ctx.set_interbody_config(FP32, 4, 2, 256, splits)
        err[splits] = float((ctx.apply_interbody(x, FP32) - ref).norm() / ref.norm())
    ctx.close()
    assert max(err[1], err[3]) < 1.03 * err[64], err
