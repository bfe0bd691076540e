"""GPU: single fields on either side of the count of sub-blocks (256 chunks each) up to which several lanes read a chunk.

The count is lower for fields with few outliers than for those with many. Each stream is read alone and as one of two in
a batch, whose chunks are more than either count, so that one lane per chunk reads it: the fields are the same bits.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("outliers", [False, True])
@pytest.mark.parametrize("sub_blocks", [190, 192, 194, 256, 258])
def test_alone_as_in_a_batch(sub_blocks, outliers):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_11165_amd import hiz
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(17)
    shape = (16, 256, 16 * sub_blocks)  # 256 chunks of 256 codes per sub-block
    x = torch.randn(shape, generator=g, device=dev)
    ctx = hiz.Context(0)
    z = ctx.compress(x, "abs", 0.004 if outliers else 0.05, hiz.make_params(tune=False, chunk=256))
    info = hiz.inspect(z[:384])
    assert info["n_chunks"] == 256 * sub_blocks
    assert (info["n_outliers"] >= 256 * sub_blocks) == outliers
    print(sub_blocks, outliers, flush=True)
    alone = ctx.decompress(z)
    assert float((alone.double() - x.double()).abs().amax()) <= info["eps"]
    for y in ctx.decompress_batch([z, z]):
        assert torch.equal(alone.view(torch.int32), y.view(torch.int32))
    ctx.close()
