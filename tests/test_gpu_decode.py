"""GPU: the decoders of several lanes per chunk and of one, against the CPU oracle, bit for bit.

How many lanes read a chunk follows from the number of chunks; the sizes fall on either side of each change. The codes
reach from one bit (a field of one symbol) over flat codebooks (noise) to codes longer than the lookup table.
"""
import numpy as np
import pytest

import fieldgen as G
import oracle as O
from test_gpu_parity import check_case, ctx  # noqa: F401  (ctx: the shared context fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _field(kind, shape):
    rng = np.random.default_rng(31)
    if kind == "flat":  # codes of nearly equal length
        return rng.uniform(-1, 1, size=shape).astype(np.float32)
    if kind == "one":  # all codes 128: one symbol
        return G.multilinear(shape)
    if kind == "rare":  # one symbol nearly everywhere: codes from one bit up to far past the table
        x = G.multilinear(shape).astype(np.float64)
        at = rng.integers(0, x.size, size=max(8, x.size // 300))
        x.reshape(-1)[at] += 2.0 * np.round(np.exp(rng.uniform(0, 4.8, at.size))) * rng.choice([-1, 1], at.size)
        return x.astype(np.float32)
    return G.grf(shape, 3.0, 33)


@pytest.mark.parametrize("chunk", [256, 512, 1024, 2048])
@pytest.mark.parametrize("kind", ["flat", "one", "rare", "grf"])
def test_codes_of_all_lengths(ctx, kind, chunk):
    x = _field(kind, (23, 31, 45))
    check_case(ctx, x, O.ABS, 1.0 if kind in ("one", "rare") else 5e-3, tune=False, chunk=chunk)


# chunks of 256 codes: 16, 17, 32, 33, 256 and 258 sub-blocks of 256 chunks (the count per field is even)
@pytest.mark.parametrize("points", [16 * 65536, 16 * 65536 + 1, 32 * 65536, 32 * 65536 + 1, 256 * 65536, 256 * 65536 + 1])
@pytest.mark.parametrize("kind", ["grf", "rare"])
def test_either_side_of_each_change_of_lanes(ctx, points, kind):
    dz = 4096 if points % 2 == 0 else points // 4096
    shape = (1, points // dz, dz) if points % 2 == 0 else (1, 1, points)
    x = np.zeros(shape, np.float32)
    part = _field(kind, (8, 32, 256)).reshape(-1)
    flat = x.reshape(-1)
    for i in range(0, points, part.size):
        flat[i:i + part.size] = part[:min(part.size, points - i)]
    check_case(ctx, x, O.ABS, 1.0 if kind == "rare" else 1e-2, tune=False, chunk=256)


def test_a_batch_of_mixed_chunk_lengths(ctx):
    from paper_2507_11165_amd import hiz
    zs, want = [], []
    for i, chunk in enumerate((256, 1024, 4096, 512)):
        x = G.grf((20 + i, 33, 50), 3.0, 60 + i)
        ref = O.compress(x, O.REL, 1e-3, tune=True, chunk=chunk, debug=False)
        want.append(O.decompress(ref.stream))
        zs.append(torch.from_numpy(ref.stream.copy()).to("cuda:0"))
    for sel in ([0, 1, 3], [0, 1, 2, 3]):  # without and with chunks longer than the split decoder takes
        ys = ctx.decompress_batch([zs[i] for i in sel])
        for i, y in zip(sel, ys):
            assert np.array_equal(y.cpu().numpy().view(np.uint32), want[i].view(np.uint32)), (sel, i)
