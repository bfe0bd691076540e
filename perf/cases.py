"""The work that users of the compressor have it do, as cases that can be timed.

Every case goes through the package's torch-facing calls (compress, decompress, decompress_batch; a batch is
compressed into the program's own buffers) on one default context, the way a simulation's output step or an analysis
reader calls them: the field (or the stream) is in GPU memory; streams go to buffers that the program keeps,
decompressed fields are new tensors. Fields are seeded Gaussian random fields made on the GPU, the repository's own
kinds: `turb` (spectrum k^-11/3 plus 1 % white noise), `smooth` (k^-3 scaled to [0, 1]) and `front` (k^-3 plus a
tanh front across a random plane).
"""
import math

import numpy
import torch

from paper_2507_11165_amd import hiz

PIPES = {"huffman": hiz.PIPE_HUFFMAN, "tp": hiz.PIPE_TP, "cr": hiz.PIPE_CR}


def _case(name, op, dims, field="turb", mode="rel", eb=1e-3, pipe="huffman", spline="tuned", batch=0):
    c = {"op": op, "dx": dims[0], "dy": dims[1], "dz": dims[2], "field": field, "mode": mode, "eb": eb,
         "pipe": pipe, "spline": spline, "batch": batch}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest fields of the serving trace, one by one: launches and latency are what a caller waits for
        _case("compress 64^3", "compress", (64, 64, 64), field="smooth"),
        _case("decompress 64^3", "decompress", (64, 64, 64), field="smooth"),
        # a turbulence snapshot, the largest single field: written at each output step, read back for analysis
        _case("compress 512^3", "compress", (512, 512, 512)),
        _case("decompress 512^3", "decompress", (512, 512, 512)),
        # an anisotropic field with a sharp front at a tight bound: rows that are no multiple of a block, many outliers
        _case("compress front", "compress", (100, 500, 500), field="front", eb=1e-4),
        _case("decompress front", "decompress", (100, 500, 500), field="front", eb=1e-4),
        # odd sides under an absolute bound, with the interpolation fixed by the program (no tuner, no range pass)
        _case("compress odd", "compress", (193, 301, 277), mode="abs", eb=5e-3, spline="cubic"),
        _case("decompress odd", "decompress", (193, 301, 277), mode="abs", eb=5e-3, spline="cubic"),
        # a climate-sized 2-D field, written and checked by reading it back
        _case("2-D there and back", "roundtrip", (1, 1800, 3600), field="smooth"),
        # the two other lossless pipelines: ratio mode for an archive, throughput mode for a loose bound
        _case("ratio mode there and back", "roundtrip", (256, 256, 256), pipe="cr"),
        _case("throughput mode there and back", "roundtrip", (256, 256, 256), eb=1e-2, pipe="tp"),
        # many uneven fields in one call per direction (an adaptive mesh's patches)
        _case("batch there and back", "roundtrip", (160, 160, 160), batch=24),
    ]


def draw(rng):
    """A case of the same ranges: sides and volumes spread over their logarithm, mostly not multiples of a block."""
    form = rng.choice(["single"] * 5 + ["pipe", "2d", "batch"])
    field = rng.choice(["turb", "smooth", "front"])
    mode = rng.choice(["rel", "rel", "rel", "abs"])
    eb = 10.0 ** rng.uniform(-4.0, -2.0)
    spline = rng.choice(["tuned", "tuned", "tuned", "cubic"])
    op = rng.choice(["compress", "decompress"])
    if form == "2d":
        h, w = (int(round(math.exp(rng.uniform(math.log(500), math.log(3600))))) for _ in range(2))
        return _case(None, "roundtrip", (1, h, w), field, mode, eb, "huffman", spline)
    if form == "batch":
        hi = rng.randint(48, 160)
        return _case(None, "roundtrip", (hi, hi, hi), field, "rel", eb, "huffman", spline, rng.randint(2, 24))
    pipe = rng.choice(["cr", "tp"]) if form == "pipe" else "huffman"
    n = math.exp(rng.uniform(math.log(64 ** 3), math.log((256 if form == "pipe" else 400) ** 3)))
    a, b = rng.uniform(-0.7, 0.7), rng.uniform(-0.7, 0.7)
    side = n ** (1.0 / 3.0)
    dims = [max(17, int(round(side * math.exp(v)))) for v in (a, b, -a - b)]
    if rng.random() < 0.25:
        dims[2] = max(32, dims[2] // 16 * 16)
    return _case(None, "roundtrip" if form == "pipe" else op, dims, field, mode, eb, pipe, spline)


def _shapes(case, seed):
    """The field's shape, or those of a batch's fields: sides uniform from 32 up."""
    if not case["batch"]:
        return [(case["dx"], case["dy"], case["dz"])]
    g = torch.Generator().manual_seed(1000003 * case["batch"] + case["dx"])  # the same sizes for every seed
    return [tuple(int(v) for v in torch.randint(32, case["dx"] + 1, (3,), generator=g)) for _ in range(case["batch"])]


def _field(kind, shape, g):
    """One Gaussian random field on the GPU: white noise, shaped in the Fourier domain to a density k^-beta."""
    dev = torch.device("cuda")
    beta = 11.0 / 3.0 if kind == "turb" else 3.0
    f = torch.fft.rfftn(torch.randn(shape, generator=g, device=dev))
    k2 = torch.zeros((1, 1, 1), device=dev)
    for axis, n in enumerate(shape):
        k = (torch.fft.rfftfreq(n, 1.0 / n, device=dev) if axis == 2 else torch.fft.fftfreq(n, 1.0 / n, device=dev))
        k2 = k2 + (k * k).reshape([-1 if a == axis else 1 for a in range(3)])
    f *= torch.where(k2 > 0, k2.clamp(min=1e-20).pow(-beta / 4.0), torch.zeros_like(k2))
    del k2
    x = torch.fft.irfftn(f, s=shape)
    del f
    x -= x.mean()
    x /= x.std()
    if kind == "turb":
        x += 0.01 * torch.randn(shape, generator=g, device=dev)
    elif kind == "smooth":
        lo, hi = x.amin(), x.amax()
        x = (x - lo) / (hi - lo)
    else:
        n = torch.randn(3, generator=g, device=dev)
        n = n / n.norm()
        at = [torch.arange(s, device=dev, dtype=torch.float32) - 0.5 * (s - 1) for s in shape]
        d = at[0][:, None, None] * n[0] + at[1][None, :, None] * n[1] + at[2][None, None, :] * n[2]
        x += 2.0 * torch.tanh(d / 2.0)
    return x.contiguous()


def _fields(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    xs = [_field(case["field"], s, g) for s in _shapes(case, seed)]
    if not case["batch"] and case["dx"] == 1:
        xs = [xs[0][0]]  # a 2-D field is passed as one
    return xs


def _params(case):
    return hiz.make_params(tune=case["spline"] == "tuned", pipeline=PIPES[case["pipe"]])


def _buffers(xs):
    """A stream buffer for each field, as a program that writes fields again and again keeps them."""
    return [torch.zeros(min(hiz.compress_bound(x.shape if x.dim() == 3 else (1, *x.shape)), 5 * x.numel() + (1 << 16)),
                        dtype=torch.uint8, device=x.device) for x in xs]


def prepare(case, seed):
    xs = _fields(case, seed)
    params = _params(case)
    if case["op"] == "decompress":
        # a reader holds the stream alone
        return {"case": case, "stream": hiz.compress(xs[0], case["mode"], case["eb"], params).clone()}
    return {"case": case, "params": params, "fields": xs, "buffers": _buffers(xs)}


def run(state):
    case = state["case"]
    if case["op"] == "decompress":
        return hiz.decompress(state["stream"])
    xs, bufs, params = state["fields"], state["buffers"], state["params"]
    if case["batch"]:
        ctx = hiz.default_context()
        sizes, _ = ctx.compress_batch_ptr([x.data_ptr() for x in xs], [x.shape for x in xs], [case["mode"]] * len(xs),
                                          [case["eb"]] * len(xs), [b.data_ptr() for b in bufs],
                                          [b.numel() for b in bufs], params)
        ys = ctx.decompress_batch([b[:n] for b, n in zip(bufs, sizes)])
        return {"streams": bufs, "sizes": numpy.array(sizes), "fields": ys}
    z = hiz.compress(xs[0], case["mode"], case["eb"], params, out=bufs[0])
    if case["op"] == "compress":
        return {"streams": bufs, "sizes": z.numel()}
    return {"streams": bufs, "sizes": z.numel(), "fields": [hiz.decompress(z, squeeze=xs[0].dim() == 2)]}


def work(case):
    """The field read or written once and the stream written or read once, at about 5 bits a value for a bound of
    1e-3 and log2(10) more for each tighter decade; a stencil and a quantization are some 30 operations a value."""
    n = sum(a * b * c for a, b, c in _shapes(case, 0))
    bits = min(32.0, max(1.0, 5.0 - math.log2(10.0) * (math.log10(case["eb"]) + 3.0)))
    ways = 2 if case["op"] == "roundtrip" else 1
    return {"bytes": ways * n * (4.0 + bits / 8.0), "flops": ways * 30.0 * n}


def exact(case, seed):
    """A decompressed field stands for the original, from which it may be off by the bound: the original in 64
    bits. Streams are bytes and have no such value."""
    if case["op"] == "compress":
        return None
    xs = [x.double() for x in _fields(case, seed)]
    if case["op"] == "decompress":
        return xs[0]
    return {"streams": None, "sizes": None, "fields": xs}
