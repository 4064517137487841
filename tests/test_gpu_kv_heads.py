"""kv head counts whose work the launch order cuts across XCDs (not a multiple
of 8) and one that it does not: every work unit runs once, whatever the cut."""

import pytest

import gpu_helpers as G
import workloads as W
from oracle import sift_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hkv", [1, 2, 3, 6, 8, 12])
def test_matches_oracle(hkv, dtype):
    import torch
    wl = W.custom([[500, 64, 130, 257, 90], [1], [65, 300]], tile=64, hq=2 * hkv, hkv=hkv, d=128,
                  dtype=dtype, seed=hkv)
    dw = G.DevWorkload(wl)
    out = dw.run(torch.float32)
    err = G.max_abs(out.cpu().numpy(), O.attention(G.oracle_layout(wl), wl.q, wl.k, wl.v, wl.la, wl.ca))
    G.say(f"hkv={hkv} {dtype}: max-abs {err:.2e}")
    assert err <= (G.F32_TOL if dtype == "f32" else G.BF16_TOL)
    dw.close()
