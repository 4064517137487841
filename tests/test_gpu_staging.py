"""The one-shot forms and the extraction return once their work is enqueued,
however many calls wait on the stream: each has its tables in a pinned buffer of
its own until its copy has read them."""

import time

import numpy as np
import pytest

import gpu_helpers as G

pytestmark = pytest.mark.gpu

CALLS = 150   # more than twice the buffers that the library keeps for good


def test_calls_behind_long_work_do_not_wait():
    import torch

    from paper_2606_09441_amd import (Plan, extract_bits, extract_sizes, sparse_prefill_ex,
                                      workspace_bytes)
    hq, hkv, d, tile = 4, 2, 128, 64
    # a layout of its own for every call
    segs = [np.cumsum([0, 65 + i, 130 - i % 3, 1 + i]).tolist() for i in range(CALLS)]
    top = segs[-1]
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(top[-1], h, d, generator=gen, device="cuda").to(torch.bfloat16)
               for h in (hq, hkv, hkv))
    la, ca = (torch.randint(0, 256, (256,), generator=gen, device="cuda").to(torch.uint8)
              for _ in range(2))
    ws = torch.empty(max(workspace_bytes(s, [0, 3], hq, hkv, d, tile) for s in segs),
                     dtype=torch.uint8, device="cuda")
    ews = torch.empty(max(extract_sizes(s[:3], hq, tile)[2] for s in segs), dtype=torch.uint8,
                      device="cuda")
    outs = [torch.empty_like(q[:s[-1]]) for s in segs]

    def one(i):
        s = segs[i]
        n, docs = s[-1], s[2]
        if i % 3 == 2:
            return extract_bits(q[:docs], k[:docs], s[:3], tile=tile, alpha=0.01, beta=0.01,
                                workspace=ews)
        return (sparse_prefill_ex(q[:n], k[:n], v[:n], s, [0, 3], la, ca, tile=tile, workspace=ws,
                                  out=outs[i]),)

    one(0), one(2)   # code objects loaded
    a = torch.randn(8192, 8192, generator=gen, device="cuda").to(torch.bfloat16)
    b = torch.empty_like(a)
    for turn in range(2):
        torch.cuda.synchronize()
        for _ in range(1000):   # about a second of work
            torch.mm(a, a, out=b)
        behind = torch.cuda.Event()
        behind.record()
        start = time.perf_counter()
        got = [one(i) for i in range(CALLS)]
        waited, took = behind.query(), time.perf_counter() - start
        torch.cuda.synchronize()
        G.say(f"{CALLS} calls enqueued in {1e3 * took:.1f} ms")
        assert not waited
        for i, s in enumerate(segs):
            if i % 3 == 2:
                want = one(i)
            else:
                # a plan's destruction gives spare buffers back
                with Plan(s, [0, 3], hq, hkv, d, tile) as plan:
                    n = s[-1]
                    want = (plan.run(q[:n], k[:n], v[:n], la, ca),)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(got[i], want)), (turn, i)
    G.say(f"{CALLS} calls queued behind other work: none waited, outputs equal")
