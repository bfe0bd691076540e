"""GPU: decompression whose headers are read by one launch gives what reading each through its tensor gives.

The launch is taken when the decoding runs on the device's current stream; with that stream named by the caller the
headers are read through the tensors. Both have to agree on fields and on errors: short, empty, misaligned and
damaged streams, constant ones (shorter than a header's tables), outputs that do not fit, and a context that is busy.
"""
import numpy as np
import pytest

import fieldgen as G
from test_gpu_parity import ctx  # noqa: F401  (the shared context fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def outcome(f):
    from paper_2507_11165_amd import hiz
    try:
        y = f()
        return [t.cpu().numpy().copy() for t in y] if isinstance(y, list) else y.cpu().numpy().copy()
    except hiz.HizError as e:
        return e.status, str(e)


def same(a, b):
    if isinstance(a, list):
        return isinstance(b, list) and len(a) == len(b) and all(same(x, y) for x, y in zip(a, b))
    return a == b if isinstance(a, tuple) else isinstance(b, np.ndarray) and np.array_equal(a, b)


def streams(ctx):
    z = [ctx.compress(torch.from_numpy(G.grf(s, 3.0, i)).to("cuda:0"), "rel", 1e-3).clone()
         for i, s in enumerate([(20, 35, 40), (1, 40, 50), (5, 6, 7)])]
    const = ctx.compress(torch.full((3, 4, 5), 1.5, device="cuda:0"), "rel", 1e-3).clone()
    bad = z[0].clone()
    bad[0] ^= 1
    wide = torch.zeros(z[0].numel() + 16, dtype=torch.uint8, device="cuda:0")
    moved = []
    for k in (1, 4, 8):
        wide[k:k + z[0].numel()] = z[0]
        moved.append(wide.clone()[k:k + z[0].numel()])
    return dict(whole=z[0], flat=z[1], small=z[2], const=const, bad=bad, moved1=moved[0], moved4=moved[1],
                moved8=moved[2], empty=z[0][:0], short=z[0][:10], header=z[0][:100].clone(), tables=z[0][:384].clone(),
                cut=z[0][:z[0].numel() - 4].clone(), strided=torch.stack([z[0], z[0]], dim=1)[:, 0])


def test_single(ctx):
    now = torch.cuda.current_stream()
    for name, z in streams(ctx).items():
        assert same(outcome(lambda: ctx.decompress(z)), outcome(lambda: ctx.decompress(z, stream=now))), name
    z = streams(ctx)["whole"]
    for n in (0, 27999, 28000, 28001):
        out = [torch.zeros(n, device="cuda:0") for _ in range(2)]
        assert same(outcome(lambda: ctx.decompress(z, out=out[0])),
                    outcome(lambda: ctx.decompress(z, out=out[1], stream=now))), n
        assert torch.equal(out[0], out[1])


def test_batches(ctx):
    now = torch.cuda.current_stream()
    z = streams(ctx)
    for names in ([], ["whole"], ["const"], ["whole", "flat", "const", "small"], ["whole", "bad"], ["cut", "whole"],
                  ["flat", "moved4"], ["small", "empty"], ["const", "short"], ["whole"] * 100):
        batch = [z[k] for k in names]
        assert same(outcome(lambda: ctx.decompress_batch(batch)),
                    outcome(lambda: ctx.decompress_batch(batch, stream=now))), names


def test_busy_context(ctx):
    now = torch.cuda.current_stream()
    x = torch.from_numpy(G.grf((20, 35, 40), 3.0, 0)).to("cuda:0")
    z = ctx.compress(x, "rel", 1e-3).clone()
    out = torch.zeros(4 * x.numel() + 4096, dtype=torch.uint8, device="cuda:0")
    ctx.compress_batch_ptr([x.data_ptr()], [x.shape], ["rel"], [1e-3], [out.data_ptr()], [out.numel()],
                           submit_only=True)
    a, b = outcome(lambda: ctx.decompress(z)), outcome(lambda: ctx.decompress(z, stream=now))
    sizes, _, st = ctx.batch_finish(1)
    assert isinstance(a, tuple) and a == b
    assert st == [0] and torch.equal(out[:sizes[0]], z)


def test_headers_follow_the_stream(ctx):
    # the header is read behind what the stream still has to write
    s = torch.cuda.Stream()
    fields = [torch.from_numpy(G.grf((20 + k, 35, 40), 3.0, k)).to("cuda:0") for k in range(3)]
    zs = [ctx.compress(f, "rel", 1e-3).clone() for f in fields]
    want = [ctx.decompress(z).clone() for z in zs]
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for z, w in zip(zs, want):
            big = torch.zeros(64 << 20, device="cuda:0")
            buf = torch.zeros(z.numel(), dtype=torch.uint8, device="cuda:0")
            for _ in range(8):
                big += 1.0
            buf.copy_(z)
            assert torch.equal(ctx.decompress(buf), w)
