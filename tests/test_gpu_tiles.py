"""GPU: the tile kernels at the edges of their tiles, against the CPU oracle, bit for bit.

A tile holds 16 x 16 x 16 tile_z owned points (16 x 64 in a field of one x plane) with a +1 face per axis; a thread
works on quads of eight z. The shapes end one point short of, on and past those edges; the values reach what the
arithmetic treats apart: reconstruction errors equal to the bound, zeros of both signs, numbers near the denormals.
"""
import numpy as np
import pytest

import fieldgen as G
import oracle as O
from test_gpu_parity import CFGS, check_case, ctx  # noqa: F401  (ctx: the shared context fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(16, 16, 32), (17, 17, 33), (18, 16, 34), (16, 18, 31), (33, 31, 63), (32, 17, 65), (15, 34, 129), (5, 9, 7),
          (1, 16, 64), (1, 17, 65), (1, 18, 63), (1, 33, 130), (1, 5, 9), (34, 1, 20)]


@pytest.mark.parametrize("tile_z", [1, 2, 4])
@pytest.mark.parametrize("si", range(len(SHAPES)))
def test_tile_edges(ctx, si, tile_z):
    x = G.grf(SHAPES[si], 3.0, 900 + si)
    check_case(ctx, x, O.REL, 1e-3, tune=False, cfg=CFGS[(si + 3 * tile_z) % len(CFGS)], chunk=256, tile_z=tile_z)


@pytest.mark.parametrize("ci", range(len(CFGS)))
@pytest.mark.parametrize("shape", [(33, 34, 67), (1, 50, 131)])
def test_errors_equal_to_the_bound(ctx, shape, ci):
    # halves of integers under the bound 1/2: every second residual is a tie whose error is the bound itself
    rng = np.random.default_rng(ci)
    x = (rng.integers(-60, 60, size=shape) * 0.5).astype(np.float32)
    check_case(ctx, x, O.ABS, 0.5, tune=False, cfg=CFGS[ci], chunk=512, tile_z=2)


@pytest.mark.parametrize("scale", [1e-37, 1e-40])
@pytest.mark.parametrize("ci", [0, 1, 7, 8])
def test_tiny_values(ctx, ci, scale):
    x = (G.grf((20, 35, 40), 3.0, 77) * np.float32(scale)).astype(np.float32)
    check_case(ctx, x, O.REL, 1e-2, tune=False, cfg=CFGS[ci], chunk=256, tile_z=2)


@pytest.mark.parametrize("ci", [0, 1, 7, 9])
def test_zeros_of_both_signs(ctx, ci):
    rng = np.random.default_rng(5)
    x = np.where(rng.random((34, 20, 50)) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
    x[10:20, 5:9, 3:40] = G.grf((10, 4, 37), 3.0, 6)
    check_case(ctx, x, O.ABS, 1e-3, tune=False, cfg=CFGS[ci], chunk=256, tile_z=1)


@pytest.mark.parametrize("shape", [(33, 20, 64), (18, 35, 47), (1, 40, 66)])
def test_fields_at_any_multiple_of_four_bytes(ctx, shape):
    from paper_2507_11165_amd import hiz
    x = G.grf(shape, 3.0, 55)
    n = x.size
    ref = O.compress(x, O.REL, 1e-3, tune=True, chunk=256, debug=False)
    want = O.decompress(ref.stream)
    p = hiz.make_params(tune=True, chunk=256)
    sh = hiz.C.c_void_p(torch.cuda.current_stream().cuda_stream)
    out = torch.zeros(hiz.compress_bound(shape), dtype=torch.uint8, device="cuda:0")
    for shift in (1, 2, 3):
        buf = torch.zeros(n + shift, device="cuda:0")
        buf[shift:] = torch.from_numpy(x).reshape(-1).to("cuda:0")
        size = ctx.compress_ptr(buf.data_ptr() + 4 * shift, shape, "rel", 1e-3, out.data_ptr(), out.numel(), p, sh)
        assert np.array_equal(out[:size].cpu().numpy(), ref.stream)
        back = torch.zeros(n + shift, device="cuda:0")
        ctx.decompress_ptr(out.data_ptr(), size, back.data_ptr() + 4 * shift, n, sh)
        torch.cuda.synchronize()
        assert np.array_equal(back[shift:].cpu().numpy().view(np.uint32), want.reshape(-1).view(np.uint32))
