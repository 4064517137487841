"""Attention over caller-given lists (bf16): the merge of the lists into steps,
at window edges (64 tiles), with entries to skip, and with lists that do not
ascend strictly, which one lane merges."""

import numpy as np
import pytest

import gpu_helpers as G
import workloads as W

pytestmark = pytest.mark.gpu


def _attend(dw, rp, ci):
    import torch
    out = dw.plan.attention(dw.q, dw.k, dw.v, torch.from_numpy(rp.astype(np.int32)).cuda(),
                            torch.from_numpy(np.concatenate([ci, [0]]).astype(np.int32)).cuda())
    torch.cuda.synchronize()
    return out


def _rebuild(rp, ci, edit):
    rows = [edit(r, ci[rp[r]:rp[r + 1]]) for r in range(len(rp) - 1)]
    return np.concatenate([[0], np.cumsum([len(x) for x in rows])]), np.concatenate(rows)


@pytest.mark.parametrize("tile", [16, 32, 64, 128])
def test_merge(tile):
    import torch
    T = tile
    # prompts of 63, 64, 65 and 130 tiles, and one that spans many windows
    prompts = [[40 * T, 22 * T, 5], [63 * T, T], [64 * T + 1], [100 * T, 29 * T - 3, T + 7],
               [30 * T, 7, 90 * T, 1, 64 * T, 3 * T]]
    wl = W.custom(prompts, tile=T, hq=4, hkv=2, d=128, dtype="bf16", seed=T, p_la=0.1, p_ca=0.2)
    dw = G.DevWorkload(wl)
    rp, ci = dw.lists()
    run = dw.run()
    clean = _attend(dw, rp, ci)
    # T < 64: the decode gathers pages, so the sums run in another order
    if T >= 64:
        assert torch.equal(clean, run)
    else:
        assert G.max_abs(clean.float().cpu(), run.float().cpu()) <= G.BF16_TOL
    far = 1 << 30
    pad = _rebuild(rp, ci, lambda r, x: np.concatenate([np.arange(-70 * (r % 3), 0), x,
                                                        far + np.arange(65 * (r % 2))]))
    assert torch.equal(_attend(dw, *pad), clean)
    # the same entries in lists that do not ascend strictly
    same = _rebuild(rp, ci, lambda r, x: np.concatenate([[-1, -1], x, [-5, far, far, -7]]))
    assert torch.equal(_attend(dw, *same), clean)
    # the first entry last, behind entries to skip: in lists short enough that
    # a tile listed twice in a unit's union leaves it within its room
    M = dw.plan.info["num_tiles"]
    late = _rebuild(rp, ci, lambda r, x: np.concatenate([x[1:], np.full(70, far), x[:1]])
                    if r % 7 == 3 and 128 // T * 2 * len(x) <= r % M - x[0] else x)
    assert len(late[1]) > len(ci) or T < 64
    assert G.max_abs(_attend(dw, *late).float().cpu(), clean.float().cpu()) <= G.BF16_TOL
    # empty lists give zeros
    none = _rebuild(rp, ci, lambda r, x: x[:0] if r % 2 else x)
    out = _attend(dw, *none).float().cpu().numpy()
    lay = G.oracle_layout(wl)
    for m in (0, 1, 62, 63):
        for h in range(wl.hq):
            _, _, a, c = lay.tile_span(m)
            want = clean.float().cpu().numpy()[a:a + c, h]
            if (h * lay.num_tiles + m) % 2:
                assert not out[a:a + c, h].any()
            else:
                assert np.max(np.abs(out[a:a + c, h] - want)) <= G.BF16_TOL
    dw.close()


@pytest.mark.parametrize("tile", [16, 32, 64, 128])
def test_sparse_lists(tile):
    """Lists with gaps of whole windows and segments, which the merge steps
    over: the diagonals alone, the prompt's first tile and the diagonal, and a
    few tiles at a stride that meets every place of a window and of a step."""
    import torch
    T = tile
    prompts = [[3 * T + 1] * 70 + [T], [200 * T, 5, 63 * T, 7 * T, 130 * T + 3, 2 * T + 9], [150 * T],
               [T] * 66 + [40 * T]]
    wl = W.custom(prompts, tile=T, hq=2, hkv=1, d=128, dtype="bf16", seed=T)
    dw = G.DevWorkload(wl)
    lay = G.oracle_layout(wl)
    M = lay.num_tiles
    first = np.zeros(M, np.int64)
    at = 0
    for p in prompts:
        n = sum(-(-x // T) for x in p)
        first[at:at + n] = at
        at += n
    rows = np.tile(np.arange(M), wl.hq)
    for tiles in (lambda r, a, m: [m], lambda r, a, m: sorted({a, m}),
                  lambda r, a, m: sorted({*range(m, a - 1, -(67 + r % 3)), m}),
                  lambda r, a, m: [x for x in range(a, m + 1) if (x - a) % 97 < 2]):
        lists = [np.asarray(tiles(r, first[m], m), np.int64) for r, m in enumerate(rows)]
        rp = np.concatenate([[0], np.cumsum([len(x) for x in lists])])
        ci = np.concatenate(lists)
        got = _attend(dw, rp, ci)
        # the same entries, merged by one lane
        want = _attend(dw, *_rebuild(rp, ci, lambda r, x: np.concatenate([x, [-5, -5]])))
        assert torch.equal(got, want)
        # the fp32 list kernel, which merges nothing
        f32 = dw.plan.attention(dw.q.float(), dw.k.float(), dw.v.float(),
                                torch.from_numpy(rp.astype(np.int32)).cuda(),
                                torch.from_numpy(ci.astype(np.int32)).cuda()) if T < 128 else None
        if f32 is not None:
            assert G.max_abs(got.float().cpu(), f32.cpu()) <= G.BF16_TOL
    dw.close()
