"""The softmax row sums of long rows.  One key has weight 1 and every other key
the same weight w, so that rounding errors of a sum over n keys don't cancel:
taken one key at a time, the sum is off by up to n 2^-24 of itself (n: the keys
that one lane adds).  With the keys of a 64-key block summed apart it is off by
at most (32 + n / 32) 2^-24."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 16384   # tokens of the document


def _qk(xs, dtype):
    """q and k of len(xs) heads of size 64 over one kv head: at the scale 1/8,
    key 0 has score 0 and the others -x, exactly."""
    import torch
    q = torch.zeros(L, len(xs), 64, dtype=dtype, device="cuda")
    q[:, :, 0] = torch.tensor([8 * x for x in xs], dtype=dtype, device="cuda")
    k = torch.zeros(L, 1, 64, dtype=dtype, device="cuda")
    k[1:, 0, 0] = -1
    return q, k


# weights for which one-at-a-time sums are off by more than a row
@pytest.mark.parametrize("x", [0.5, 0.75, 2.5, 3.0])
def test_extraction(x):
    """beta lies between the probability w / (1 + p w) of rows p = r - 1 and
    p = r.  A page's count of cells above it is that of the rows before r, or 16
    less or more where r is off by a row; gamma lies 8 below and 8 above it.
    The sum's error, (32 + 256) 2^-24, and that of the threshold's three
    additions, each of half an ulp of 16, come to 0.3 rows at row 15,000, and r
    tolerates 0.5."""
    import torch
    from paper_2606_09441_amd import extract_bits
    T, r, w = 16, 15000, np.exp(-x)
    q, k = _qk([x], torch.bfloat16)
    keys = np.arange(T, 2 * T)                    # page 1
    count, cells = int((r - keys).sum()), int((L - keys).sum())
    beta = w / (1 + (r - 0.5) * w)
    for step, want in ((-8, 1), (8, 0)):
        _, ca = extract_bits(q, k, [0, L], tile=T, alpha=0.5, beta=beta, gamma=(count + step) / cells)
        assert int(ca[0]) >> 6 & 1 == want, (x, step)
