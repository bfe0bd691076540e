"""GPU: which fields hiz_compress_noalloc takes does not depend on the tiles that the launch table picks.

The limit counts tiles of the depth asked for, or of two blocks along z. The shapes refused here need a little more than
the scratch array holds that way, and less with the launch table's tiles of four blocks.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,pipeline,fits", [((550, 560, 128), 2, False), ((546, 560, 128), 2, True),
                                                 ((1, 16320, 16000), 0, False), ((1, 16200, 16000), 0, True)])
def test_noalloc_limit(shape, pipeline, fits):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_11165_amd import hiz
    dev = torch.device("cuda:0")
    x = torch.zeros(shape, dtype=torch.float32, device=dev)
    x[:, ::3] = 1.0
    out = torch.empty(x.numel(), dtype=torch.uint8, device=dev)
    ctx = hiz.Context(0)
    params = hiz.make_params(tune=False, pipeline=pipeline)
    args = (x.data_ptr(), shape, "rel", 1e-1, out.data_ptr(), out.numel(), params, hiz._stream_handle(None))
    print(shape, pipeline, flush=True)
    if fits:
        n = ctx.compress_noalloc_ptr(*args)
        y = ctx.decompress(out[:n])
        assert float((y - x).abs().amax()) <= 0.1
    else:
        with pytest.raises(hiz.HizError) as e:
            ctx.compress_noalloc_ptr(*args)
        assert e.value.status == hiz.ERR_ARG and "allocation-free" in str(e.value)
    ctx.close()
