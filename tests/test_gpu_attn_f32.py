"""fp32 attention: the work-unit kernel (large calls) and the list kernel
(small calls, caller-given lists) at the edges of their 16-row, 64-row and
64-key blocks, against the fp64 oracle; packed, paged and over lists; and
which lists an attention call on a plan uses after each kind of decode.

The tolerance is the project's fp32 bar: scores of |s| <= 8 carry an error of
about 128 * 2^-24 * |s| and as much again in the weights, 1e-6 in all for
values of order one."""

import numpy as np
import pytest

import gpu_helpers as G
import workloads as W
from oracle import sift_oracle as O

pytestmark = pytest.mark.gpu

# (prompts, hq, hkv): groups of 64 rows over all heads below and above 512
SMALL = ([[130, 17, 1, 40], [64, 16, 33]], 4, 2)
UNITS = ([[200, 65, 1, 129, 30], [16, 48, 300, 64, 0]], 40, 5)
SPLIT = ([[300] * 7 + [90]], 24, 8)     # a query long enough for pieces: 35 steps


def _ref(wl):
    return O.attention(G.oracle_layout(wl), wl.q, wl.k, wl.v, wl.la, wl.ca)


@pytest.mark.parametrize("tile", [16, 32, 64])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [SMALL, UNITS, SPLIT], ids=["small", "units", "split"])
def test_against_oracle(shape, d, tile):
    import torch
    prompts, hq, hkv = shape
    wl = W.custom(prompts, tile=tile, hq=hq, hkv=hkv, d=d, dtype="f32", seed=tile + d)
    dw = G.DevWorkload(wl)
    ref = _ref(wl)
    out = dw.run()
    err = G.max_abs(out.cpu().numpy(), ref)
    kp, vp, table = G.page_pool(wl, dw.k, dw.v)
    paged = dw.plan.run_paged(dw.q, kp, vp, table, dw.la, dw.ca)
    # packed K and V again over that decode, then over lists in the caller's buffers
    after = dw.plan.attention_internal(dw.q, dw.k, dw.v)
    rp, ci = dw.plan.decode(dw.la, dw.ca)
    own = dw.plan.attention_internal(dw.q, dw.k, dw.v)
    lists = dw.plan.attention(dw.q, dw.k, dw.v, rp, ci)
    torch.cuda.synchronize()
    errs = [G.max_abs(x.cpu().numpy(), ref) for x in (after, own, lists)]
    G.say(f"f32 T={tile} D={d} {len(prompts)} prompts: max-abs {err:.2e}, after paged / own / lists "
          + " ".join(f"{e:.2e}" for e in errs))
    assert err <= G.F32_TOL and max(errs) <= G.F32_TOL
    assert torch.equal(paged, out)
    dw.close()


def test_caller_lists_leave_the_decode_in_place():
    """Attention over caller lists, then over the plan's decode: each its own."""
    import torch
    prompts, hq, hkv = UNITS
    wl = W.custom(prompts, tile=32, hq=hq, hkv=hkv, d=64, dtype="f32", seed=3)
    dw = G.DevWorkload(wl)
    out = dw.run()
    # lists of the diagonal tiles alone
    M, rows = dw.plan.info["num_tiles"], dw.plan.info["num_rows"]
    rp = torch.arange(rows + 1, dtype=torch.int32, device="cuda")
    ci = torch.arange(M, dtype=torch.int32, device="cuda").repeat(hq)
    diag = dw.plan.attention(dw.q, dw.k, dw.v, rp, ci)
    again = dw.plan.attention_internal(dw.q, dw.k, dw.v)
    torch.cuda.synchronize()
    assert torch.equal(again, out) and not torch.equal(diag, out)
    dw.close()


def test_nan_reaches_only_rows_that_list_its_tile():
    """A NaN key row: rows whose lists hold its tile become NaN, the others
    stay as they were, in either kernel."""
    import torch
    for prompts, hq, hkv in (SMALL, UNITS):
        wl = W.custom(prompts, tile=16, hq=hq, hkv=hkv, d=64, dtype="f32", seed=9)
        dw = G.DevWorkload(wl)
        rp, ci = dw.lists()
        out = dw.run().cpu().numpy()
        lay = G.oracle_layout(wl)
        n = 2
        _, _, a, cnt = lay.tile_span(n)
        dw.k[a + cnt - 1] = float("nan")       # the tile's last key
        got = dw.run().cpu().numpy()
        for h in range(hq):
            for m in range(lay.num_tiles):
                _, _, b, c = lay.tile_span(m)
                row = ci[rp[h * lay.num_tiles + m]: rp[h * lay.num_tiles + m + 1]]
                if n not in row:
                    assert np.array_equal(got[b:b + c, h], out[b:b + c, h]), (h, m)
                elif m > n:
                    assert np.isnan(got[b:b + c, h]).all(), (h, m)
        dw.close()


@pytest.mark.parametrize("shape", [SMALL, UNITS], ids=["small", "units"])
def test_storage_off_a_16_byte_line(shape):
    import torch
    prompts, hq, hkv = shape
    wl = W.custom(prompts, tile=32, hq=hq, hkv=hkv, d=64, dtype="f32", seed=4)
    dw = G.DevWorkload(wl)
    ref = dw.run()

    def skew(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.flatten()
        return buf[1:].view(t.shape)

    q, k, v, out = (skew(t) for t in (dw.q, dw.k, dw.v, ref))
    out.zero_()
    dw.plan.run(q, k, v, dw.la, dw.ca, out=out)
    torch.cuda.synchronize()
    assert out.data_ptr() % 16 == 4
    assert G.max_abs(out.cpu(), ref.cpu()) <= 2 * G.F32_TOL
    dw.close()


def _skewed(t):
    """t on storage 4 bytes off a 16-byte line."""
    import torch
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t.flatten()
    return buf[1:].view(t.shape)


@pytest.mark.parametrize("tile,d", [(16, 64), (32, 128), (64, 64), (64, 128)])
@pytest.mark.parametrize("shape", [SMALL, UNITS, SPLIT], ids=["small", "units", "split"])
def test_lists_in_caller_buffers_and_skewed_storage(shape, tile, d):
    """A decode into the caller's buffers leaves the plan's own lists those of
    an older decode, of other bits here: attention on the plan uses the new
    ones, also where K or V is off a 16-byte line (or in a pool that is)."""
    import torch
    prompts, hq, hkv = shape
    wl = W.custom(prompts, tile=tile, hq=hq, hkv=hkv, d=d, dtype="f32", seed=tile + d)
    dw = G.DevWorkload(wl)
    ref = _ref(wl)
    dw.plan.run(dw.q, dw.k, dw.v, ~dw.la, ~dw.ca)
    dw.plan.decode(dw.la, dw.ca)
    k, v = _skewed(dw.k), _skewed(dw.v)
    outs = [dw.plan.attention_internal(*x) for x in
            ((dw.q, dw.k, dw.v), (dw.q, k, dw.v), (dw.q, dw.k, v), (_skewed(dw.q), k, v))]
    packed = dw.plan.run(dw.q, k, v, dw.la, dw.ca)
    kp, vp, table = G.page_pool(wl, dw.k, dw.v)
    paged = dw.plan.run_paged(dw.q, _skewed(kp), _skewed(vp), table, dw.la, dw.ca)
    torch.cuda.synchronize()
    assert k.data_ptr() % 16 == 4
    errs = [G.max_abs(o.cpu().numpy(), ref) for o in outs + [packed, paged]]
    G.say(f"f32 T={tile} D={d}: max-abs " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) <= G.F32_TOL
    # staged by DMA or through registers, the same sums
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
    assert torch.equal(paged, packed)
    dw.close()


def test_no_lists_of_the_last_decode():
    """No decode yet, or one into the caller's buffers whose steps a bf16 call
    over lists has replaced: refused, until the next decode."""
    import torch

    from paper_2606_09441_amd import SiftError
    prompts, hq, hkv = SMALL
    wl = W.custom(prompts, tile=32, hq=hq, hkv=hkv, d=128, dtype="f32", seed=7)
    dw = G.DevWorkload(wl)
    out = torch.full_like(dw.q, 3.0)

    def refused():
        with pytest.raises(SiftError) as e:
            dw.plan.attention_internal(dw.q, dw.k, dw.v, out=out)
        assert e.value.status == 7
        torch.cuda.synchronize()
        assert bool((out == 3.0).all())

    refused()
    rp, ci = dw.plan.decode(dw.la, dw.ca)
    dw.plan.attention(*(t.to(torch.bfloat16) for t in (dw.q, dw.k, dw.v)), rp, ci)
    refused()
    got = [dw.plan.attention(dw.q, dw.k, dw.v, rp, ci)]
    dw.plan.decode_internal(dw.la, dw.ca)
    dw.plan.attention(*(t.to(torch.bfloat16) for t in (dw.q, dw.k, dw.v)), rp, ci)
    got.append(dw.plan.attention_internal(dw.q, dw.k, dw.v))
    ref = _ref(wl)
    assert all(G.max_abs(o.cpu().numpy(), ref) <= G.F32_TOL for o in got)
    dw.close()


@pytest.mark.parametrize("prompts", [(1 << 17) - 1, 1 << 17])
def test_work_units_at_the_limit_of_a_launch(prompts):
    """Prompts of one token and 64 heads: 2^23 - 64 work units, whose workgroups
    of 512 threads a grid just holds, and 2^23, which the list kernel takes.
    Each row's only key is its own, so it is its V row, but for the rounding of
    the weight and of its reciprocal."""
    import torch

    from paper_2606_09441_amd import Plan, SiftError
    hq = 64
    so = np.arange(prompts + 1)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(prompts, hq, 64, generator=gen, device="cuda")
    k, v = (torch.randn(prompts, 1, 64, generator=gen, device="cuda") for _ in range(2))
    none = torch.zeros(1, dtype=torch.uint8, device="cuda")
    with Plan(so, so, hq, 1, 64, 64) as plan:
        assert plan.info["num_work_units"] == prompts * hq
        out = plan.run(q, k, v, none, none)
        err = float((out - v).abs().max())
        out.zero_()
        rp, ci = plan.decode(none, none)
        if prompts * hq < 1 << 23:
            plan.attention_internal(q, k, v, out=out)
        else:
            with pytest.raises(SiftError) as e:
                plan.attention_internal(q, k, v, out=out)
            assert e.value.status == 5
            plan.attention(q, k, v, rp, ci, out=out)
        err = max(err, float((out - v).abs().max()))
    G.say(f"{prompts * hq} units: max-abs {err:.2e}")
    assert err <= 8 * 2.0 ** -24 * float(v.abs().max())


@pytest.mark.parametrize("shape", [SMALL, UNITS], ids=["small", "units"])
def test_captured_attention(shape):
    """fp32 attention in a graph, with and without the decode in it: replays
    after bf16 calls over other lists, which replace the plan's steps, give the
    eager result."""
    import torch
    prompts, hq, hkv = shape
    wl = W.custom(prompts, tile=64, hq=hq, hkv=hkv, d=128, dtype="f32", seed=11)
    dw = G.DevWorkload(wl)
    p, io = dw.plan, (dw.q, dw.k, dw.v)
    half = tuple(t.to(torch.bfloat16) for t in io)
    rows = p.info["num_rows"]
    rp = torch.arange(rows + 1, dtype=torch.int32, device="cuda")
    ci = torch.arange(p.info["num_tiles"], dtype=torch.int32, device="cuda").repeat(hq)
    p.attention(*half, rp, ci)
    want = dw.run()
    assert G.max_abs(want.cpu(), _ref(wl)) <= G.F32_TOL
    outs = [torch.empty_like(dw.q) for _ in range(3)]

    def alone():
        p.attention_internal(*io, out=outs[0])

    def decode_first():
        p.decode_internal(dw.la, dw.ca)
        p.attention_internal(*io, out=outs[1])

    def run():
        p.run(*io, dw.la, dw.ca, out=outs[2])

    for fn, out in zip((alone, decode_first, run), outs):
        p.decode_internal(dw.la, dw.ca)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            fn()
        for _ in range(3):
            out.zero_()
            p.attention(*half, rp, ci)     # other lists
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert G.max_abs(out.cpu(), want.cpu()) <= 2 * G.F32_TOL, fn.__name__
            p.decode_internal(dw.la, dw.ca)
            g.replay()
            torch.cuda.synchronize()
            assert G.max_abs(out.cpu(), want.cpu()) <= 2 * G.F32_TOL, fn.__name__
    dw.close()
