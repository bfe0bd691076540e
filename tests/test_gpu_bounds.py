"""GPU: where a field's bound and configuration come from, against the CPU oracle, byte for byte.

An absolute bound and a configuration without a sample are set as the call begins, a relative bound by the tuner's
launch or, for a field too small to be sampled, by one of its own. One batch holds them all, constant fields too, so
that no launch may take another field's place; the same batch is replayed as a graph. A field of several times the
min/max launch's reach makes its workgroups take more than one unit.
"""
import numpy as np
import pytest

import fieldgen as G
import oracle as O
from test_gpu_parity import ctx  # noqa: F401  (the shared context fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def mixed():
    const = np.full((20, 21, 22), 2.5, dtype=np.float32)
    return [(G.grf((20, 35, 40), 3.0, 1), "rel", 1e-3), (G.grf((9, 10, 30), 3.0, 2), "rel", 1e-2),
            (G.grf((33, 18, 20), 3.0, 3), "abs", 1e-2), (const, "rel", 1e-3), (G.grf((5, 6, 7), 3.0, 4), "abs", 1e-2),
            (const[:9, :9, :9].copy(), "rel", 1e-3), (const, "abs", 1e-3), (G.grf((1, 40, 50), 3.0, 5), "rel", 1e-4)]


def oracle_stream(x, mode, eb, tune):
    return O.compress(x, O.REL if mode == "rel" else O.ABS, eb, tune=tune, chunk=256).stream


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("tune", [True, False])
def test_mixed_batch(ctx, tune, graphs):
    from paper_2507_11165_amd import hiz
    cases = mixed()
    want = [oracle_stream(*c, tune) for c in cases]
    p = hiz.make_params(tune=tune, chunk=256)
    ctx.set_graphs(graphs)
    try:
        for k in range(3):
            order = [(i + k) % len(cases) for i in range(len(cases))]
            fields = [torch.from_numpy(cases[i][0]).to("cuda:0") for i in order]
            out = ctx.compress_batch(fields, [cases[i][1] for i in order], [cases[i][2] for i in order], params=p)
            torch.cuda.synchronize()
            for i, z in zip(order, out):
                assert np.array_equal(z.cpu().numpy(), want[i]), (k, i)
    finally:
        ctx.set_graphs(False)


def test_extremes_of_a_large_field(ctx):
    # units past the launch's first round hold them, and the last, short one
    n = 16384 * 8 * torch.cuda.get_device_properties(0).multi_processor_count
    x = torch.zeros(1, 1, n + 16384 * 5 + 7, device="cuda:0")
    for at, v in ((n + 3 * 16384 + 5, 8.0), (x.numel() - 1, -24.0)):
        x.zero_()
        x[0, 0, 100] = 1.0
        x[0, 0, at] = v
        z = ctx.compress(x, "rel", 0.125)
        from paper_2507_11165_amd import hiz
        info = hiz.inspect(z)
        assert (info["vmin"], info["vmax"]) == (min(v, 0.0), max(v, 1.0))
        assert info["eps"] == 0.125 * (max(v, 1.0) - min(v, 0.0))
        assert float((ctx.decompress(z) - x).abs().max()) <= info["eps"]


@pytest.mark.parametrize("first", [False, True])
def test_graphs_tell_reordered_streams_apart(ctx, first):
    from paper_2507_11165_amd import hiz
    x = G.grf((20, 35, 40), 3.0, 9)
    f = torch.from_numpy(x).to("cuda:0")
    z = {r: ctx.compress(f, "rel", 1e-3, hiz.make_params(tune=False, chunk=256, reorder=r)).clone()
         for r in (False, True)}
    plain = {r: ctx.decompress(z[r]).clone() for r in z}
    ctx.set_graphs(True)
    try:
        for r in (first, not first, first, not first):
            assert torch.equal(ctx.decompress(z[r]), plain[r])
    finally:
        ctx.set_graphs(False)
