"""Benchmark of the SIFT sparse prefill hot path on one MI355X.

A step is one layer of the online path for one batch of synthetic input:
decode the bit vectors into tile lists, then sparse attention over them
(sift_plan_run).  The default workload is the 64K long-context layer:
48 query heads / 8 kv heads, head_dim 128, bf16, 32 documents x 2048 tokens
plus a 512-token query, tile 64, bit vectors at 15% tile density.

Prints one JSON line: useful attention TFLOP/s (4*D flop per computed
query-key cell), the fraction of the bf16 MFMA peak reached by the attention
kernel, the speedup over the same kernels with all-ones bit vectors (dense
causal attention), and the fp64 oracle timed on a sample on the host.
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

BF16_PEAK_TFLOPS = 2516.6   # MI355X dense bf16 MFMA: 256 CU x 2.4 GHz x 4096 flop/clk
HBM_PEAK_GBS = 8000.0


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def attn_source_digest(csrc):
    """sha256 over the attention kernel's source: attn_bf16.hip, then the
    unit body it includes."""
    import hashlib
    h = hashlib.sha256()
    for name in ("attn_bf16.hip", "attn_bf16_unit.inc"):
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def measured_traffic():
    """HBM bytes per attention launch from the committed rocprofv3 counter
    summary (FETCH_SIZE and WRITE_SIZE, scaled by the copy-kernel factors), or
    None when the attention kernel source has changed since it was taken."""
    import re
    path = os.path.join(ROOT, "profiles", "attn_bf16_long64k_hbm_traffic.md")
    csrc = os.path.join(ROOT, "paper_2606_09441_amd", "csrc")
    try:
        text = open(path).read()
        m = re.search(r"```json\s*(\{.*?\})\s*```", text, re.S)
        info = json.loads(m.group(1))
        digest = attn_source_digest(csrc)
    except (OSError, AttributeError, ValueError):
        return None
    return info["hbm_bytes_per_launch"] if info.get("source_sha256") == digest else None


def tile_tables(seg_offsets, prompt_seg_ptr, tile):
    """Per global tile: token count and first tile of its prompt (segment-local tiling)."""
    lens, lo = [], []
    for b in range(len(prompt_seg_ptr) - 1):
        first = len(lens)
        for s in range(prompt_seg_ptr[b], prompt_seg_ptr[b + 1]):
            n = int(seg_offsets[s + 1] - seg_offsets[s])
            for i in range(-(-n // tile)):
                lens.append(min(tile, n - i * tile))
                lo.append(first)
    return np.asarray(lens, np.int64), np.asarray(lo, np.int64)


def useful_flops(row_ptr, col_idx, tlen, M, D):
    """4*D per causal in-range cell of every listed (head, M-block, N-block)."""
    counts = np.diff(row_ptr)
    m = np.repeat(np.arange(len(counts)) % M, counts)
    n = col_idx[: len(m)]
    qn, kn = tlen[m], tlen[n]
    cells = np.where(n == m, qn * (qn + 1) // 2, qn * kn)
    return 4 * D * int(cells.sum())


def row_cells(rows, heads, row_ptr, col_idx, tlen, tok_tile, tok_local, M):
    """Computed cells of given (row, head) pairs, from the lists."""
    total = 0
    for r in rows:
        m = tok_tile[r]
        for h in heads:
            lst = col_idx[row_ptr[h * M + m]: row_ptr[h * M + m + 1]]
            total += int(tlen[lst[lst != m]].sum()) + int(tok_local[r]) + 1
    return total


def extract_leg(wl, q, k, dev, args):
    """The offline metadata extraction of the workload's documents, each
    prefilled alone (Sections 4.1, 4.2, 4.4), with the paper's thresholds.
    Work: QK^T over every causal cell, 2 D flop per cell and query head (scores
    that the kernel forms again are not counted).  Time: wall clock per call,
    including its table upload."""
    import torch

    from paper_2606_09441_amd import extract_bits, extract_sizes
    docs = []
    for b in range(len(wl.prompt_seg_ptr) - 1):
        for s in range(int(wl.prompt_seg_ptr[b]), int(wl.prompt_seg_ptr[b + 1]) - 1):
            docs.append((int(wl.seg_offsets[s]), int(wl.seg_offsets[s + 1])))
    if not docs:
        return None
    idx = torch.from_numpy(np.concatenate([np.arange(a, b) for a, b in docs])).to(dev)
    qe, ke = q.index_select(0, idx).contiguous(), k.index_select(0, idx).contiguous()
    lens = [b - a for a, b in docs]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    _, _, ws_n = extract_sizes(offs, wl.hq, wl.tile)
    ws = torch.empty(ws_n, dtype=torch.uint8, device=dev)
    for _ in range(2):
        la_e, ca_e = extract_bits(qe, ke, offs, tile=wl.tile, workspace=ws)
    torch.cuda.synchronize()
    n = max(3, args.steps)
    t0 = time.perf_counter()
    for _ in range(n):
        la_e, ca_e = extract_bits(qe, ke, offs, tile=wl.tile, workspace=ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / n
    cells = sum(L * (L + 1) // 2 for L in lens)
    work = 2 * wl.d * cells * wl.hq
    la_bits = np.unpackbits(la_e.cpu().numpy()).mean() if la_e.numel() else 0.0
    ca_bits = np.unpackbits(ca_e.cpu().numpy()).mean() if ca_e.numel() else 0.0
    log(f"extract: {len(docs)} documents, {sum(lens)} tokens: {ms:.3f} ms per call, "
        f"{work / ms / 1e9:.1f} TFLOP/s")
    return {"ms_per_call": round(ms, 4), "tflops": round(work / ms / 1e9, 2),
            "documents": len(docs), "tokens": int(sum(lens)),
            "thresholds": [0.001, 0.01, 0.1],
            "la_bits_set": round(float(la_bits), 4), "ca_bits_set": round(float(ca_bits), 4),
            "work": "QK^T over the causal cells, 2*D flop per cell and head"}


def layer_leg(wl, plan, la, ca, dev, args):
    """Per-layer prefill time of one decoder layer of the workload's shape
    (hidden = Hq D; the MLP of Llama-3.1-8B, 14336 wide for hidden 4096, else
    3.5 x hidden), random-init weights: the attention block (norm, q/k/v
    GEMMs, RoPE, decode + attention, o_proj) and the whole layer (with the
    SwiGLU MLP), over the workload's bits and over all-ones bits (dense
    causal attention, the paper's full recompute)."""
    import torch

    import workloads as W
    from paper_2606_09441_amd.layer import PrefillLayer
    hidden = wl.hq * wl.d
    inter = 14336 if hidden == 4096 else int(3.5 * hidden)
    w = W.layer_weights(hidden, wl.hq, wl.hkv, wl.d, inter, seed=1)
    layer = PrefillLayer({k: torch.from_numpy(v).to(dev).bfloat16() for k, v in w.items()},
                         wl.hq, wl.hkv, wl.d, torch.from_numpy(W.rope_inv_freq(wl.d)).to(dev))
    x = torch.from_numpy(W.layer_input(wl.tokens, hidden, seed=2)).to(dev).bfloat16()
    pos = torch.from_numpy(W.prompt_positions(wl.seg_offsets, wl.prompt_seg_ptr)).to(dev)
    wd = W.all_ones(wl)
    la_d, ca_d = torch.from_numpy(wd.la).to(dev), torch.from_numpy(wd.ca).to(dev)
    res = {"hidden": hidden, "intermediate": inter}
    n = max(3, args.steps // 2)
    for tag, bits in (("sparse", (la, ca)), ("dense", (la_d, ca_d))):
        for part, mlp in (("attention_block", False), ("layer", True)):
            fn = lambda: layer.forward(x, plan, pos, bits[0], bits[1], mlp=mlp)
            for _ in range(2):
                fn()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(n):
                fn()
            e1.record()
            torch.cuda.synchronize()
            res[f"{part}_ms_{tag}"] = round(e0.elapsed_time(e1) / n, 4)
    res["attention_block_speedup"] = round(res["attention_block_ms_dense"] /
                                           res["attention_block_ms_sparse"], 3)
    res["layer_speedup"] = round(res["layer_ms_dense"] / res["layer_ms_sparse"], 3)
    log(f"layer (hidden {hidden}): attention block {res['attention_block_ms_sparse']:.3f} vs "
        f"{res['attention_block_ms_dense']:.3f} ms dense, whole layer {res['layer_ms_sparse']:.3f} vs "
        f"{res['layer_ms_dense']:.3f} ms dense: {res['layer_speedup']:.2f}x")
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="long64k")
    ap.add_argument("--rho", type=float, default=None)
    ap.add_argument("--layer", action="store_true",
                    help="also time the decoder-layer prefill slice, sparse vs dense bits")
    ap.add_argument("--heads", default=None,
                    help="HQ,HKV for the long64k workload (default 48,8; 32,8 is Llama-3.1-8B)")
    ap.add_argument("--tile", type=int, default=None,
                    help="tile size of the RAG workloads (64 or 128; default 64)")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-dense", action="store_true")
    ap.add_argument("--no-hh8", action="store_true",
                    help="skip the heavy-hitter x8 leg (long64k only)")
    ap.add_argument("--no-low-toggle", action="store_true",
                    help="skip timing the attention on mantissa-cleared inputs")
    ap.add_argument("--no-extract", action="store_true",
                    help="skip the offline metadata extraction leg")
    ap.add_argument("--only-extract", action="store_true",
                    help="run the extraction leg only (for profiler runs)")
    ap.add_argument("--paged", action="store_true",
                    help="also time the step with K/V in a page pool (random page order)")
    ap.add_argument("--only-steps", action="store_true",
                    help="run warmup + timed steps only (for profiler runs)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only: the path has no multi-GPU part "
              f"(--gpus {args.gpus} requested)", file=sys.stderr)
        sys.exit(2)

    import torch

    import workloads as W
    from paper_2606_09441_amd import Plan

    assert torch.cuda.is_available(), "bench.py needs the GPU"
    dev = torch.device("cuda:0")
    kw = {} if args.rho is None else {"rho": args.rho}
    if args.tile is not None:
        kw["tile"] = args.tile
    if args.heads is not None:
        kw["hq"], kw["hkv"] = (int(x) for x in args.heads.split(","))
    t0 = time.time()
    wl = W.make(args.workload, **kw)
    log(f"workload {wl.name}: {wl.tokens} tokens, hq={wl.hq} hkv={wl.hkv} D={wl.d} "
        f"T={wl.tile} (generated in {time.time() - t0:.1f}s)")
    dt = torch.bfloat16 if wl.dtype == "bf16" else torch.float32
    q = torch.from_numpy(wl.q).to(dev).to(dt)
    k = torch.from_numpy(wl.k).to(dev).to(dt)
    v = torch.from_numpy(wl.v).to(dev).to(dt)
    la = torch.from_numpy(wl.la).to(dev)
    ca = torch.from_numpy(wl.ca).to(dev)
    out = torch.empty_like(q)
    torch.cuda.synchronize()

    if args.only_extract:
        extract_leg(wl, q, k, dev, args)
        return

    tp = time.perf_counter()
    plan = Plan(wl.seg_offsets, wl.prompt_seg_ptr, wl.hq, wl.hkv, wl.d, wl.tile)
    plan_ms = (time.perf_counter() - tp) * 1e3
    M = plan.info["num_tiles"]
    stream = torch.cuda.current_stream()

    def timed(fn, steps):
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(steps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / steps

    def per_launch(fn, steps):
        """Average duration of one launch of fn, events around each launch."""
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
              for _ in range(steps)]
        torch.cuda.synchronize()
        for a, b in ev:
            a.record(stream)
            fn()
            b.record(stream)
        torch.cuda.synchronize()
        return float(np.mean([a.elapsed_time(b) for a, b in ev]))

    step = lambda: plan.run(q, k, v, la, ca, out=out)
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    log(f"warmup done ({args.warmup} steps)")
    ms_step = timed(step, args.steps)
    log(f"timed {args.steps} steps: {ms_step:.3f} ms/step")
    if args.only_steps:
        return

    # lists and useful work of this input
    rp_t, ci_t = plan.decode(la, ca)
    torch.cuda.synchronize()
    rp = rp_t.cpu().numpy().astype(np.int64)
    ci = ci_t[: int(rp[-1])].cpu().numpy().astype(np.int64)
    tlen, _ = tile_tables(wl.seg_offsets, wl.prompt_seg_ptr, wl.tile)
    flops = useful_flops(rp, ci, tlen, M, wl.d)
    nnz = int(rp[-1])
    density = nnz / plan.info["list_capacity"]
    # the two kernels of the path, each timed alone: decode (Section 5.1) and
    # attention over the decoded lists (Section 5.2)
    ms_decode = per_launch(lambda: plan.decode_internal(la, ca), args.steps)
    plan.decode_internal(la, ca)
    ms_attn = per_launch(lambda: plan.attention_internal(q, k, v, out=out), args.steps)
    log(f"decode {ms_decode * 1e3:.1f} us, attention {ms_attn:.3f} ms, nnz {nnz}, "
        f"density {density:.4f}, useful {flops / 1e12:.3f} TFLOP")

    dense = {}
    if not args.no_dense:
        wd = W.all_ones(wl)
        la_d = torch.from_numpy(wd.la).to(dev)
        ca_d = torch.from_numpy(wd.ca).to(dev)
        step_d = lambda: plan.run(q, k, v, la_d, ca_d, out=out)
        for _ in range(max(1, args.warmup)):
            step_d()
        ms_step_d = timed(step_d, max(2, args.steps // 2))
        rpd, cid = plan.decode(la_d, ca_d)
        plan.decode_internal(la_d, ca_d)
        ms_attn_d = per_launch(lambda: plan.attention_internal(q, k, v, out=out),
                               max(2, args.steps // 2))
        torch.cuda.synchronize()
        rpd_h = rpd.cpu().numpy().astype(np.int64)
        flops_d = useful_flops(rpd_h, cid[: int(rpd_h[-1])].cpu().numpy().astype(np.int64),
                               tlen, M, wl.d)
        dense = {
            "ms_per_step": round(ms_step_d, 4),
            "attention_ms": round(ms_attn_d, 4),
            "useful_tflops": round(flops_d / ms_attn_d / 1e9, 2),
            "speedup_step": round(ms_step_d / ms_step, 3),
            "speedup_attention": round(ms_attn_d / ms_attn, 3),
            "inverse_density": round(1.0 / density, 3),
        }
        log(f"dense: step {ms_step_d:.3f} ms, attention {ms_attn_d:.3f} ms "
            f"({flops_d / ms_attn_d / 1e9:.1f} TFLOP/s); speedup {ms_step_d / ms_step:.2f}x "
            f"vs 1/density {1 / density:.2f}")

    paged = None
    if args.paged:
        # K/V in a pool of T-row pages, one page per tile, in a random order
        tl = torch.from_numpy(tlen).to(dev)
        T = wl.tile
        perm = np.random.default_rng(1).permutation(M).astype(np.int32)
        kp = torch.zeros((M * T, wl.hkv, wl.d), dtype=dt, device=dev)
        vp = torch.zeros_like(kp)
        tok0 = np.concatenate([[0], np.cumsum(tlen)[:-1]]).astype(np.int64)
        for m in range(M):
            p, a, n = int(perm[m]), int(tok0[m]), int(tlen[m])
            kp[p * T: p * T + n] = k[a: a + n]
            vp[p * T: p * T + n] = v[a: a + n]
        table = torch.from_numpy(perm).to(dev)
        step_p = lambda: plan.run_paged(q, kp, vp, table, la, ca, out=out)
        for _ in range(args.warmup):
            step_p()
        ms_step_p = timed(step_p, args.steps)
        paged = {"ms_per_step": round(ms_step_p, 4),
                 "useful_tflops_step": round(flops / ms_step_p / 1e9, 2)}
        log(f"paged K/V: step {ms_step_p:.3f} ms ({flops / ms_step_p / 1e9:.1f} TFLOP/s)")
        del kp, vp, tl

    # launches whose attention needed the exact second pass, over every
    # attention launch so far on this plan
    exact = {"launches_with_exact_pass": plan.exact_passes(), "note":
             "count of bf16 attention launches on this input whose first pass flagged a weight "
             "bound or a non-finite output, so that the second launch redid every unit"}

    heavy = None
    if args.workload == "long64k" and args.rho is None and wl.dtype == "bf16" and not args.no_hh8:
        # heavy-hitter keys scaled x8 instead of x4: scores rise further above
        # a row's first tile, the case the exact second pass exists for
        t0 = time.time()
        wh = W.make(args.workload, hh=8.0, **kw)
        log(f"heavy-hitter x8 input generated in {time.time() - t0:.1f}s")
        kh = torch.from_numpy(wh.k).to(dev).to(dt)
        lah, cah = torch.from_numpy(wh.la).to(dev), torch.from_numpy(wh.ca).to(dev)
        qh, vh = torch.from_numpy(wh.q).to(dev).to(dt), torch.from_numpy(wh.v).to(dev).to(dt)
        before = plan.exact_passes()
        plan.decode_internal(lah, cah)
        n_h = max(2, args.steps // 2)
        ms_attn_h = per_launch(lambda: plan.attention_internal(qh, kh, vh, out=out), n_h)
        ran = plan.exact_passes() - before
        rph, cih = plan.decode(lah, cah)
        torch.cuda.synchronize()
        rph_h = rph.cpu().numpy().astype(np.int64)
        flops_h = useful_flops(rph_h, cih[: int(rph_h[-1])].cpu().numpy().astype(np.int64), tlen,
                               M, wl.d)
        heavy = {"attention_ms": round(ms_attn_h, 4),
                 "useful_tflops": round(flops_h / ms_attn_h / 1e9, 2),
                 "launches": n_h, "launches_with_exact_pass": int(ran),
                 "note": "same layout and shapes, heavy-hitter K rows x8"}
        log(f"heavy-hitter x8: attention {ms_attn_h:.3f} ms, exact pass in {ran} of {n_h} launches")
        del kh, qh, vh, lah, cah, wh

    low_toggle = None
    if wl.dtype == "bf16" and not args.no_low_toggle:
        # the same lists and instruction stream on inputs whose bits switch
        # less: Q, K and V with their mantissas cleared (sign and exponent
        # kept), timed in turn with the inputs themselves
        clear = lambda x: (x.view(torch.int16) & -128).view(torch.bfloat16)
        ql, kl, vl = clear(q), clear(k), clear(v)
        plan.decode_internal(la, ca)
        n_l = max(2, args.steps // 2)
        ms_l, ms_r = [], []
        for _ in range(2):
            ms_l.append(per_launch(lambda: plan.attention_internal(ql, kl, vl, out=out), n_l))
            ms_r.append(per_launch(lambda: plan.attention_internal(q, k, v, out=out), n_l))
        low_toggle = {"attention_ms": round(float(np.mean(ms_l)), 4),
                      "attention_ms_unmodified": round(float(np.mean(ms_r)), 4),
                      "note": "Q, K, V with their bf16 mantissas cleared, same lists and "
                              "launches, interleaved with the unmodified inputs: the speed "
                              "depends on how many operand bits switch"}
        log(f"mantissas cleared: attention {np.mean(ms_l):.3f} ms against {np.mean(ms_r):.3f} ms")
        del ql, kl, vl

    one_shot = None
    if wl.dtype == "bf16":
        from paper_2606_09441_amd import sparse_prefill
        call = lambda: sparse_prefill(q, k, v, wl.seg_offsets, wl.prompt_seg_ptr, la, ca,
                                      tile=wl.tile, out=out)
        # the same warm-up and count as the step: the first calls after the
        # plan-based runs read their tables from cold caches
        for _ in range(args.warmup):
            call()
        torch.cuda.synchronize()
        n1 = args.steps
        t_h = time.perf_counter()
        ms_gpu = timed(call, n1)
        wall = (time.perf_counter() - t_h) * 1e3 / n1
        one_shot = {"ms_per_call": round(ms_gpu, 4), "wall_ms_per_call": round(wall, 4),
                    "note": "sift_sparse_prefill: host plan, stream-ordered scratch and table "
                            "upload, decode, attention, free; events on the stream / host wall "
                            "clock around back-to-back calls"}
        log(f"one-shot sift_sparse_prefill: {ms_gpu:.3f} ms per call (wall {wall:.3f} ms)")

    layer = None
    if args.layer and wl.dtype == "bf16":
        layer = layer_leg(wl, plan, la, ca, dev, args)

    extract = None
    if wl.dtype == "bf16" and not args.no_extract:
        extract = extract_leg(wl, q, k, dev, args)

    cpu = None
    if not args.no_cpu_baseline:
        from oracle import sift_oracle as O
        cores = len(os.sched_getaffinity(0))
        model = None
        try:
            with open("/proc/cpuinfo") as f:
                model = next((ln.split(":", 1)[1].strip() for ln in f if ln.startswith("model name")),
                             None)
        except OSError:
            pass
        lay = O.Layout(wl.seg_offsets, wl.prompt_seg_ptr, wl.tile, wl.hq)
        tok_tile = np.zeros(wl.tokens, np.int64)
        tok_local = np.zeros(wl.tokens, np.int64)
        for s_ in lay.segs:
            loc = np.arange(s_.length)
            tok_tile[s_.start:s_.start + s_.length] = s_.tile_base + loc // wl.tile
            tok_local[s_.start:s_.start + s_.length] = loc % wl.tile
        # whole query tiles (M-blocks) in a random order, all heads, the
        # oracle spread over (head, row group) on every core this process has
        rng = np.random.default_rng(0)
        order = rng.permutation(M)
        done_tiles, rows_done, cells, t_cpu = 0, 0, 0, 0.0
        while t_cpu < args.cpu_seconds and done_tiles < M:
            tiles = np.sort(order[done_tiles:done_tiles + 4])
            rows = np.concatenate([np.nonzero(tok_tile == m)[0] for m in tiles])
            tc = time.perf_counter()
            O.attention(lay, wl.q, wl.k, wl.v, wl.la, wl.ca, rows=rows, workers=cores)
            t_cpu += time.perf_counter() - tc
            cells += row_cells(rows, range(wl.hq), rp, ci, tlen, tok_tile, tok_local, M)
            done_tiles += len(tiles)
            rows_done += len(rows)
        cpu = {
            "value": round(4 * wl.d * cells / t_cpu / 1e12, 6),
            "unit": "TFLOP/s",
            "cores": int(cores),
            "kind": "oracle",
            "cpu_model": model,
            "sample": f"{done_tiles} random query tiles ({rows_done} rows) x all {wl.hq} heads of "
                      f"the same input, fp64 numpy, {cores} worker threads ({t_cpu:.1f}s)",
        }
        log(f"cpu oracle: {cpu['value']} TFLOP/s on {rows_done} rows in {t_cpu:.1f}s, {cores} threads")

    achieved = flops / ms_attn / 1e9
    res = {
        "metric": "useful attention TFLOP/s (sparse prefill, decode + attention)",
        "value": round(flops / ms_step / 1e9, 3),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16" if wl.dtype == "bf16" else "f32",
        "data": "synthetic",
        "config": {
            "workload": f"{wl.name}: {wl.tokens} tokens ({len(wl.seg_offsets) - 2} docs + query), "
                        f"{wl.hq}/{wl.hkv} heads, D={wl.d}, T={wl.tile}",
            "tokens": wl.tokens, "q_heads": wl.hq, "kv_heads": wl.hkv, "head_dim": wl.d,
            "tile": wl.tile, "rho": wl.meta.get("rho"),
        },
        "density": round(density, 5),
        "nnz_tiles": nnz,
        "useful_tflop_per_step": round(flops / 1e12, 4),
        "decode_us": round(ms_decode * 1e3, 2),
        "attention_ms": round(ms_attn, 4),
        "plan_ms": round(plan_ms, 3),
        "pct_bf16_peak_attention": round(100 * achieved / BF16_PEAK_TFLOPS, 2),
        "dense": dense or None,
        "paged": paged,
        "extract": extract,
        "layer": layer,
        "exact_pass": exact,
        "heavy_hitters_x8": heavy,
        "one_shot": one_shot,
        "low_toggle": low_toggle,
        "roofline": {
            "bound": "mfma",
            "achieved": round(achieved, 2),
            "peak": BF16_PEAK_TFLOPS,
            "unit": "TFLOP/s",
            "frac": round(achieved / BF16_PEAK_TFLOPS, 4),
            # HBM bytes per launch (rocprofv3 counters), only for the long64k
            # workload they were taken on
            "traffic": measured_traffic() if args.workload == "long64k" and args.rho is None
                       and args.tile in (None, 64) else None,
        },
        "cpu_baseline": cpu,
    }
    plan.close()
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
