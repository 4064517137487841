"""Extraction where the row maxima of a document's key blocks fit LDS, partly
fit, and where blocks need no count, some, or all: every bit against the fp64
oracle."""

import numpy as np
import pytest

from oracle import extract_oracle as X
from test_gpu_extract import _gpu_bits

pytestmark = pytest.mark.gpu


def _inputs(lens, hq, hkv, d, seed):
    """Documents with heavy key blocks along a direction the queries share."""
    import workloads as W
    rng = np.random.default_rng(seed)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(offs[-1])
    u = rng.standard_normal((hkv, d))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    heavy = np.repeat(rng.random((n // 64 + 1, hkv)) < 0.2, 64, axis=0)[:n] & (rng.random((n, hkv)) < 0.4)
    q = rng.standard_normal((n, hq, d)) + 6.0 * np.repeat(u, hq // hkv, axis=0)
    k = rng.standard_normal((n, hkv, d)) + 16.0 * heavy[:, :, None] * u
    return offs, W.bf16_round(q.astype(np.float32)), W.bf16_round(k.astype(np.float32))


@pytest.mark.parametrize("tile", [16, 32, 64, 128])
@pytest.mark.parametrize("d,lens", [
    (64, [1, 63, 65, 130, 700]),
    (128, [1700, 64]),          # T = 16: blocks past the first 24 are formed again
    (64, [6400]),               # every T: past the stored blocks
])
@pytest.mark.parametrize("alpha,beta,gamma", [(0.001, 0.01, 0.1), (0.002, 1e-7, 0.5), (0.0, 0.9, 0.0)])
def test_bits(alpha, beta, gamma, d, lens, tile):
    hq, hkv = (1, 1) if max(lens) > 4000 else (2, 1)
    offs, q, k = _inputs(lens, hq, hkv, d, tile + d)
    got = _gpu_bits(offs, q, k, tile, alpha, beta, gamma)
    want = X.extract_bits(offs, q, k, hq, hkv, tile, alpha, beta, gamma)
    for g, w, ambiguous in zip(got, want[:2], want[2:]):
        assert g.shape == w.shape
        assert not np.any((g ^ w) & ~ambiguous)


@pytest.mark.parametrize("d", [64, 128])
def test_storage_off_a_16_byte_line(d):
    import torch
    from paper_2606_09441_amd import extract_bits
    offs, q, k = _inputs([300, 65, 1], 2, 1, d, 3)

    def skew(x):
        buf = torch.empty(x.size + 1, dtype=torch.bfloat16, device="cuda")
        buf[1:] = torch.from_numpy(x).flatten()
        return buf[1:].view(x.shape)

    got = extract_bits(skew(q), skew(k), offs, tile=32, alpha=0.002, beta=0.004, gamma=0.1)
    want = _gpu_bits(offs, q, k, 32, 0.002, 0.004, 0.1)
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w)
