"""GPU: codebooks of chosen code counts, against the CPU oracle, byte for byte.

In a 1-D field whose even points are zero every odd point is predicted as zero, so an odd point of q * 2 eb gets
code 128 + q: the counts can be laid out at will. They are chosen for the rounds in which nodes are merged: ties
throughout, sums that fall between the leaves, one merge per round (Fibonacci counts, the deepest tree), odd ones left
over in a round, and alphabets of two symbols up to all of them.
"""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import CFGS, check_case, ctx  # noqa: F401  (ctx: the shared context fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def fib(n):
    f = [1, 1]
    while len(f) < n:
        f.append(f[-1] + f[-2])
    return f[:n]


COUNTS = {
    "two": [3],
    "three": [1, 1],
    "fibonacci": fib(24),
    "powers": [1 << i for i in range(16)],
    "ties": [7] * 253,
    "ties and one": [7] * 252 + [8],
    "ramp": list(range(1, 254)),
    "steps": [1 << (i // 16) for i in range(253)],
    "threes": [3 ** (i // 28) for i in range(253)],
    "sums between leaves": sorted([2 * i + 1 for i in range(60)] + [4 * i + 2 for i in range(60)]),
}


@pytest.mark.parametrize("name", list(COUNTS))
def test_counts(ctx, name):
    counts = COUNTS[name]
    # codes 1..255 without 128 (the even points' own)
    q = [v for k in range(1, 128) for v in (k, -k)][:len(counts)]
    odd = np.repeat(np.array(q, dtype=np.float32), counts)
    x = np.zeros((1, 1, 2 * odd.size + 3), dtype=np.float32)
    x[0, 0, 1:2 * odd.size:2] = np.random.default_rng(1).permutation(odd)
    check_case(ctx, x, O.ABS, 0.5, tune=False, cfg=CFGS[0], chunk=1024, tile_z=1)
