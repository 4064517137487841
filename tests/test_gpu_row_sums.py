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


@pytest.mark.parametrize("kernel", ["units", "lists"])
def test_fp32_attention(kernel):
    """Every tile marked, v zero but for key 0: row p is 1 / (1 + p w), whose
    error is that of the row sum: (32 + 256) 2^-24, and 8 roundings of the
    weights and the quotient."""
    import torch
    from paper_2606_09441_amd import Plan
    xs = (0.75, 1.5, 2.5)
    q, k = _qk(xs, torch.float32)
    v = torch.zeros_like(k)
    v[0] = 1
    with Plan([0, L, L], [0, 2], len(xs), 1, 64, 64) as plan:
        la, ca = (torch.full((plan.info[n],), 255, dtype=torch.uint8, device="cuda")
                  for n in ("la_bytes", "ca_bytes"))
        if kernel == "units":
            out = plan.run(q, k, v, la, ca)
        else:
            out = plan.attention(q, k, v, *plan.decode(la, ca))
        torch.cuda.synchronize()
    w = np.exp(-np.asarray(xs))
    want = 1 / (1 + np.arange(L)[:, None] * w)
    err = np.abs(out.cpu().numpy().astype(np.float64) / want[:, :, None] - 1).max((0, 2))
    print(f"{kernel}: relative error {err}", flush=True)
    assert err.max() <= (32 + 256 + 8) * 2.0 ** -24
