"""Plans with and without a schedule pass, at the work unit counts where the
rule changes (512, 1536): short segments, one work unit each per head; the last
workgroups' empty records; and calls of both types on one plan, which order its
work units differently."""

import pytest

import gpu_helpers as G
import workloads as W
from oracle import sift_oracle as O

pytestmark = pytest.mark.gpu


def _wl(segs, hq, hkv, tile, dtype, seed=1):
    # prompts of at most 16 segments: no query unit is long enough for pieces
    prompts = [[9] * (n - 1) + [3] for n in [16] * (segs // 16) + [segs % 16] if n]
    return W.custom(prompts, tile=tile, hq=hq, hkv=hkv, d=128, dtype=dtype, seed=seed)


def _ref(wl):
    return O.attention(G.oracle_layout(wl), wl.q, wl.k, wl.v, wl.la, wl.ca)


# (segments, hq, hkv): 512, 520, 1536 and 1544 units, of 8 kv heads; 1040 of 16;
# 18 and 513, whose chunks are not whole
@pytest.mark.parametrize("segs,hq,hkv", [(64, 8, 8), (65, 8, 8), (192, 8, 8), (193, 8, 8),
                                         (65, 16, 16), (6, 3, 1), (171, 3, 1)])
@pytest.mark.parametrize("tile,dtype", [(64, "bf16"), (128, "bf16"), (32, "bf16"), (64, "f32")])
def test_unit_counts(segs, hq, hkv, tile, dtype):
    import torch
    wl = _wl(segs, hq, hkv, tile, dtype)
    dw = G.DevWorkload(wl)
    assert dw.plan.info["num_work_units"] == segs * hq
    out = dw.run(torch.float32)
    err = G.max_abs(out.cpu().numpy(), _ref(wl))
    rp, ci = dw.plan.decode(dw.la, dw.ca)
    over = dw.plan.attention(dw.q, dw.k, dw.v, rp, ci, out_dtype=torch.float32)
    err2 = G.max_abs(over.cpu().numpy(), _ref(wl))
    G.say(f"{segs * hq} units, T={tile} {dtype}: max-abs {err:.2e}, over lists {err2:.2e}")
    assert max(err, err2) <= (G.F32_TOL if dtype == "f32" else G.BF16_TOL)
    dw.close()


def test_types_share_a_plan():
    """An fp32 call sorts the work units, a bf16 one of the same plan does not,
    and each decodes other bits; then attention alone, of both types."""
    import torch
    a, b = (_wl(100, 8, 8, 64, "f32", seed) for seed in (1, 2))
    da, db = G.DevWorkload(a), G.DevWorkload(b)
    ra, rb = _ref(a), _ref(b)
    x = [t.to(torch.bfloat16) for t in (da.q, da.k, da.v)]
    y = [t.to(torch.bfloat16) for t in (db.q, db.k, db.v)]
    p, f32 = da.plan, torch.float32
    for _ in range(2):
        got = [(p.run(da.q, da.k, da.v, da.la, da.ca), ra, G.F32_TOL),
               (p.run(*y, db.la, db.ca, out_dtype=f32), rb, G.BF16_TOL),
               (p.attention_internal(db.q, db.k, db.v), rb, G.F32_TOL)]
        p.decode_internal(da.la, da.ca)
        got += [(p.attention_internal(da.q, da.k, da.v), ra, G.F32_TOL),
                (p.attention_internal(*x, out_dtype=f32), ra, G.BF16_TOL)]
        torch.cuda.synchronize()
        errs = [G.max_abs(o.cpu().numpy(), r) for o, r, _ in got]
        G.say("max-abs " + " ".join(f"{e:.1e}" for e in errs))
        assert all(e <= t for e, (_, _, t) in zip(errs, got))
    da.close()
    db.close()
