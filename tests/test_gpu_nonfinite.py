"""GPU: fields that hold NaN or Inf in a batch with absolute bounds, where the tile kernel itself finds them.

Such a field is refused, and its neighbours in the batch are not touched by it: their streams are the oracle's byte for
byte. The tiles are more than the chip holds workgroups, so that workgroups walk from one field into the next, and
values that are not finite are met by some workgroups while others are at that field's first tile.
"""
import numpy as np
import pytest

import fieldgen as G
import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hz():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_11165_amd import hiz
    return hiz


def _plant(x, how):
    v = x.view(-1)
    if how == "first":
        v[0] = float("nan")
    elif how == "last":
        v[-1] = float("-inf")
    elif how == "inside":
        v.view(torch.int32)[v.numel() // 2] = -1  # a NaN with the sign set
    else:
        v.fill_(float("inf"))
    return x


@pytest.mark.parametrize("pipeline", [0, 1])
@pytest.mark.parametrize("tile_z", [1, 2, 4, "flat"])
def test_sound_fields_beside_nonfinite_ones(hz, tile_z, pipeline):
    flat = tile_z == "flat"
    sound = ([(1, 70, 90), (1, 33, 257), (1, 16, 16), (1, 100, 64), (1, 17, 130)] if flat else
             [(40, 33, 50), (17, 17, 17), (33, 48, 31), (16, 64, 70), (65, 20, 90)])
    big = (1, 1024, 1088) if flat else (128, 128, 272)
    xs = [G.random_small(s, 4100 + i) for i, s in enumerate(sound)]
    g = torch.Generator(device=DEV).manual_seed(4200)
    bad = [_plant(torch.randn(big, generator=g, device=DEV), how) for how in ("first", "everywhere", "last", "inside")]
    fields, refs = [], []
    for i, x in enumerate(xs):
        fields.append(torch.from_numpy(x).to(DEV))
        refs.append(x)
        if i < len(bad):
            fields.append(bad[i])
            refs.append(None)
    caps = [hz.compress_bound(f.shape) if r is not None else 4096 for f, r in zip(fields, refs)]
    outs = [torch.zeros(c, dtype=torch.uint8, device=DEV) for c in caps]
    p = hz.make_params(tune=True, chunk=256, tile_z=0 if flat else tile_z, pipeline=pipeline)
    ctx = hz.Context(0)
    print(f"tile_z {tile_z}, pipeline {pipeline}", flush=True)
    sizes, st = ctx.compress_batch_ptr([f.data_ptr() for f in fields], [f.shape for f in fields],
                                       ["abs"] * len(fields), [1e-3] * len(fields), [o.data_ptr() for o in outs], caps,
                                       p, hz._stream_handle(None))
    assert st == [hz.OK if r is not None else hz.ERR_NONFINITE for r in refs]
    for x, z, n in zip(refs, outs, sizes):
        if x is None:
            continue
        ref = O.compress(x, O.ABS, 1e-3, tune=True, chunk=256, debug=False, pipeline=pipeline).stream
        assert n == ref.size and np.array_equal(z[:n].cpu().numpy(), ref), x.shape
    ctx.close()
