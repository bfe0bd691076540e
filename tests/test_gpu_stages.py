"""GPU: the bitwise-redundancy stages and the reordering at the edges of their pieces, against the CPU oracle, byte for
byte.

A thread of the stages works on 16 or 32 bytes of a 16384-byte chunk, four groups of eight bytes at a time where the
planes allow it; a bitmap has one to four levels. The lengths end short of, on and past those edges in the last chunk.
The fields leave few marks, many, all of them (chunks stored as they are) and outliers. The reordering takes 16 points
of a row at a time, of rows on every level.
"""
import numpy as np
import pytest

import fieldgen as G
import oracle as O
from test_gpu_pipelines import check, ctx, hz  # noqa: F401  (hz, ctx: the shared fixtures)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 65, 511, 513, 520, 4096, 4104, 4097, 8200, 16383, 16384, 16385,
           16392, 16384 + 31, 16384 + 48, 3 * 16384 - 8]


def line(kind, n):
    rng = np.random.default_rng(n)
    z = np.arange(n, dtype=np.float64)
    if kind == "smooth":
        x = np.sin(z / 300.0)
    elif kind == "noise":
        x = rng.normal(size=n)
    elif kind == "steps":
        x = np.floor(z / 700.0) + 0.001 * (rng.random(n) < 0.01)
    else: # spikes far past the bound: outliers
        x = np.sin(z / 300.0) + 1e4 * (rng.random(n) < 0.03)
    return x.astype(np.float32).reshape(1, 1, n)


@pytest.mark.parametrize("pipeline", [O.PIPE_TP, O.PIPE_CR])
@pytest.mark.parametrize("kind", ["smooth", "noise", "steps", "spikes"])
def test_lengths(hz, ctx, kind, pipeline):
    for n in LENGTHS:
        check(hz, ctx, line(kind, n), pipeline, False, eb=1e-5 if kind == "spikes" else 1e-3, chunk=256)


@pytest.mark.parametrize("dz", [1, 7, 15, 16, 17, 31, 32, 33, 47, 50])
@pytest.mark.parametrize("dxy", [(1, 1), (2, 3), (5, 6), (17, 18), (34, 9)])
def test_reordered_rows(hz, ctx, dxy, dz):
    x = G.grf(dxy + (dz,), 3.0, 100 * dxy[0] + dz)
    check(hz, ctx, x, O.PIPE_TP, True, eb=1e-4)
