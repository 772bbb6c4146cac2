#!/usr/bin/env python3
"""Benchmark of the KV offloading hot path on one MI355X.

One step = one pass of the whole path over a synthetic KV cache already resident in HBM:
  offload  (plan lookups, pack kernels, chunked D2H, page-cache-path memcpy hop) of every layer, then
  reload   (memcpy hop, chunked H2D, unpack kernels) + decode attention of every layer.
Prints one JSON line: offload+reload GB/s over the step, with the dominant kernel's roofline, the
measured host-link ceiling, decode-attention microseconds per layer and a CPU baseline (the plain
checker timed on a bounded sample of the same workload).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0  # MI355X published HBM3E bandwidth

# HBM bytes per launch from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of `bench.py --leg kernels` on each
# workload (profiles/pmc_traffic_<workload>.md), each counter scaled by what it reads for a plain device-to-device
# copy of known size in the same run.  Valid only for the sources they were taken with: the hash below covers the
# two kernel files, what cuts and launches their work, and the compiler's flags; a mismatch reports traffic as null.
PMC_TRAFFIC = {"sha": "90a2c03dd0da1a3a",
               "llama8b_32k": {"kv_layout_kernel<pack>": 268458307, "kv_layout_kernel<unpack>": 268454775, "kv_attn_partial_kernel+kv_attn_combine_kernel": 135563990},
               "llama8b_4k": {"kv_layout_kernel<pack>": 268468511, "kv_layout_kernel<unpack>": 268463344, "kv_attn_partial_kernel+kv_attn_combine_kernel": 18137246},
               "llama8b_ragged_paged": {"kv_layout_kernel<pack>": 282080321, "kv_layout_kernel<unpack>": 282054250, "kv_attn_partial_kernel+kv_attn_combine_kernel": 142712142},
               "gemma7b_mha_8k": {"kv_layout_kernel<pack>": 536894812, "kv_layout_kernel<unpack>": 536883735, "kv_attn_partial_kernel+kv_attn_combine_kernel": 537767573}}


def kernel_sources_hash() -> str:
    import hashlib
    from paper_2604_26557_amd.build import FLAGS
    h = hashlib.sha256()
    for fn in ("layout_kernels.hip", "attn_kernels.hip", "attn_splits.hpp", "launch.hpp"):
        with open(os.path.join(ROOT, "paper_2604_26557_amd", "csrc", fn), "rb") as f:
            h.update(f.read())
    h.update(" ".join(f for f in FLAGS if not os.path.isabs(f)).encode())   # without this tree's own folders
    return h.hexdigest()[:16]


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def measure_link(torch, total_bytes: int, piece: int = 64 << 20, min_s: float = 1.0, max_s: float = 3.0):
    """Back-to-back pinned copies in >= 64 MiB pieces, each direction, no kernels: the host-link ceiling.
    Passes repeat for at least min_s per direction and then until one comes within 2 % of the best so far
    (at most max_s): when another process has just left the GPU, the first second or so of transfers has
    been seen to run at about half rate, and the ceiling is the settled rate.  Every pass is logged."""
    n = max(1, total_bytes // piece)
    host = torch.empty(piece, dtype=torch.uint8, pin_memory=True)
    host.fill_(1)
    dev = torch.empty(piece, dtype=torch.uint8, device="cuda")
    out = {}
    for name, (dst, src) in {"h2d": (dev, host), "d2h": (host, dev)}.items():
        dst.copy_(src, non_blocking=True)
        torch.cuda.synchronize()
        rates = []
        begin = time.perf_counter()
        while time.perf_counter() - begin < max_s:
            t0 = time.perf_counter()
            for _ in range(n):
                dst.copy_(src, non_blocking=True)
            torch.cuda.synchronize()
            rates.append(n * piece / (time.perf_counter() - t0) / 1e9)
            if time.perf_counter() - begin >= min_s and rates[-1] >= 0.98 * max(rates[:-1]):
                break
        out[name] = max(rates)
        log(f"[bench] link {name}, GB/s per pass: " + " ".join(f"{r:.1f}" for r in rates))
    return out


def host_memcpy_rate(dst_addr: int, src_addr: int, nbytes: int, threads: int) -> float:
    """GB/s of `threads` host threads copying disjoint pieces (the third hop of the page-cache path)."""
    import ctypes
    import threading
    piece = nbytes // threads

    def work(i):
        ctypes.memmove(dst_addr + i * piece, src_addr + i * piece, piece)   # releases the GIL

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    t0 = time.perf_counter()
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    return piece * threads / (time.perf_counter() - t0) / 1e9


def cpu_baseline(cfg, W, budget_s: float = 24.0, gpu_attn=None):
    """The CPU checker, as it stands, on whole layers of the same workload: pack K and V into extent images,
    unpack them back, one decode attention per layer.  Two builds of the same C file are timed, each on as many
    layers as fit its share of budget_s: the defining one-thread build, and the -fopenmp build on all host
    cores.  Only the checker's calls are timed, not the input generation.  The checker is imported here and
    nowhere else in this script."""
    import numpy as np
    from oracle import kv_oracle as o
    lens = W.seq_lens(cfg)
    plan = o.layout_plan(cfg.n_layers, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, lens, 2, cfg.sector_bytes,
                         cfg.extent_mode == W.PER_SEQ, cfg.pc_budget_bytes, cfg.lba_start)
    nbytes = plan.n_blocks_tensor * plan.lba_size
    paged = cfg.layout == W.PAGED
    if paged:
        table, n_pool = W.block_table(cfg, lens)

    def layer_inputs(layer):
        if paged:
            K = W.paged_layer(cfg, layer, 0, n_pool, "cpu")
            V = W.paged_layer(cfg, layer, 1, n_pool, "cpu")
            src = o.Source(H=cfg.n_kv_heads, D=cfg.head_dim, paged=True, block_table=table.numpy(),
                           block_tokens=cfg.block_tokens)
        else:
            K = W.bhsd_layer(cfg, layer, 0, "cpu")
            V = W.bhsd_layer(cfg, layer, 1, "cpu")
            src = o.bhsd_source(K.shape)
        return K, V, W.query(cfg, layer, "cpu"), src

    def leg(omp: bool, budget: float, parity_hook):
        moved, layers, move_s, attn_s, parity = 0, 0, 0.0, 0.0, None
        for layer in range(cfg.n_layers):
            K, V, q, src = layer_inputs(layer)
            ext = np.empty(nbytes, dtype=np.uint8)
            back = np.empty_like(o.u16(K))
            t0 = time.perf_counter()
            for t in (K, V):
                o.pack(src, o.u16(t), plan.per_seq, lens, plan.seq_base, plan.n_blocks_tensor, plan.lba_size, ext, omp=omp)
                o.unpack(src, back, plan.per_seq, lens, plan.seq_base, plan.lba_size, ext, omp=omp)
                moved += 2 * nbytes  # extent bytes once out (pack) and once back (unpack)
            t1 = time.perf_counter()
            ref = o.attention(src, o.u16(K), o.u16(V), o.u16(q), cfg.dtype == W.BF16, lens, cfg.n_q_heads, omp=omp)
            t2 = time.perf_counter()
            if layer == 0 and parity_hook is not None:   # the same bits through the GPU path, against the checker's output
                got = parity_hook(K, V, q)
                parity = {"layer": 0, "max_abs_err": float(np.abs(got - ref).max()),
                          "reference_max_abs": float(np.abs(ref).max())}
            move_s += t1 - t0
            attn_s += t2 - t1
            layers += 1
            if (move_s + attn_s) * (layers + 1) / layers > budget:
                break
        return {"cores": o.threads(omp), "layers": layers, "seconds": round(move_s + attn_s, 2),
                "pack_unpack_GBps": round(moved / move_s / 1e9, 3),
                "decode_attn_us_per_layer": round(attn_s / layers * 1e6, 1)}, parity

    one, parity = leg(False, budget_s / 2, gpu_attn)
    many, _ = leg(True, budget_s / 2, None)
    return {"value": many["pack_unpack_GBps"], "unit": "GB/s", "cores": many["cores"], "kind": "oracle",
            "sample": f"whole layers of the same workload (pack and unpack of K and V: extent bytes moved per second of "
                      f"pack+unpack time; one decode attention per layer, timed apart): {many['layers']} of "
                      f"{cfg.n_layers} layers in {many['seconds']} s on {many['cores']} threads (-fopenmp build of the "
                      f"plain C checker, loops over tokens and over (b, h_q) shared, no pinning), {one['layers']} layers "
                      f"in {one['seconds']} s on 1 thread (the defining build)",
            "decode_attn_us_per_layer": many["decode_attn_us_per_layer"],
            "one_thread": one, "all_cores": many,
            "gpu_attention_vs_checker": parity}


def kernel_leg(torch, kv, cfg, plan, info, src_view, dst_view, k, qs, outs, lens, reps: int):
    """Resident-KV leg: every kernel of the path launched back to back in the launch configuration the pipeline
    uses (K and V of a layer in one launch up to 256 MiB; consecutive layers of one path together while their
    images stay within 128 MiB), rotating over all layers (so each launch touches memory no earlier launch left
    in the last-level cache), no DMA in flight.  Each kind is bracketed by events on the stream it is launched on
    (the default stream, which is also PyTorch's current stream here); the figure is the average per launch,
    gaps included."""
    L = cfg.n_layers
    n1 = int(info.n_pagecache_layers)
    tensor_image = int(info.tensor_blocks) * cfg.sector_bytes
    pair = 2 * tensor_image <= (256 << 20)
    group = min(16, max(1, (128 << 20) // (2 * tensor_image))) if pair else 1
    runs = []                                             # (first layer, layers) of every launch; a run keeps to one path
    for lo, hi in ((0, n1), (n1, L)):
        runs += [(l, min(group, hi - l)) for l in range(lo, hi, group)]
    image = (2 * group if pair else 1) * tensor_image
    n_img = max(2, min(len(runs) * (1 if pair else 2), (1 << 30) // image))   # rotating extent images, about 1 GiB
    imgs = [torch.empty(image, dtype=torch.uint8, device="cuda") for _ in range(n_img)]
    max_len = max(lens)
    ws = torch.empty(kv.kv_decode_attn_workspace(plan, 0, max_len), dtype=torch.uint8, device="cuda")
    ev = lambda: torch.cuda.Event(enable_timing=True)

    def timed(fn, n_launches):
        fn()                                              # warm
        torch.cuda.synchronize()
        e0, e1 = ev(), ev()
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / (reps * n_launches)   # microseconds per launch

    def pack_all():
        i = 0
        for l, n in runs:
            if n > 1:
                kv.kv_offload_pack_layers(plan, l, l + n, src_view, imgs[i % n_img])
                i += 1
            else:
                for kind in ([kv.KV_KV] if pair else [kv.KV_K, kv.KV_V]):
                    kv.kv_offload_pack(plan, l, kind, src_view, kv.KV_SEQ_ALL, 0, 0, imgs[i % n_img])
                    i += 1

    def unpack_all():
        i = 0
        for l, n in runs:
            if n > 1:
                kv.kv_reload_unpack_layers(plan, l, l + n, imgs[i % n_img], dst_view)
                i += 1
            else:
                for kind in ([kv.KV_KV] if pair else [kv.KV_K, kv.KV_V]):
                    kv.kv_reload_unpack(plan, l, kind, imgs[i % n_img], dst_view, kv.KV_SEQ_ALL, 0, 0)
                    i += 1

    def attn_all():
        for l in range(L):
            kv.kv_decode_attn(plan, src_view, l, qs[l], outs[l], kv.KV_OUT_F32, 0, ws)

    def copy_ref():
        # plain device-to-device copies of one extent image each: the known-size reference that hardware
        # byte counters of the kernels above are scaled by
        for i in range(8):
            imgs[(i + 1) % n_img].copy_(imgs[i % n_img])

    def attn_graph_us():
        # the same launches for all layers recorded once in a HIP graph and replayed: through the entry point that
        # allocates nothing (split partials in the library's static device array), which capture requires
        def static_all():
            for l in range(L):
                kv.kv_decode_attn_static(plan, src_view, l, qs[l], outs[l], kv.KV_OUT_F32, 0)
        static_all()                                      # resolves the array's address before capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            static_all()
        return timed(g.replay, L)

    n = len(runs) * (1 if pair else 2)
    res = {"pack_us": timed(pack_all, n), "unpack_us": timed(unpack_all, n), "attn_us": timed(attn_all, L),
           "copy_ref_bytes": image, "tensors_per_launch": 2 * L / n, "layout_launches": n}
    try:
        res["attn_graph_us"] = attn_graph_us()
    except Exception as e:                                # reported, never fatal: the eager figure is the metric
        res["attn_graph_us"] = None
        res["attn_graph_error"] = f"{type(e).__name__}: {e}"
    res["copy_ref_us"] = timed(copy_ref, 8)               # last: these copies end the profiled command
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", default="llama8b_32k")
    ap.add_argument("--leg", choices=["both", "pipeline", "kernels"], default="both",
                    help="pipeline: the timed steps only; kernels: the resident-KV kernel leg only")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--host-workers", type=int, default=0)
    ap.add_argument("--span-chunks", type=int, default=0)
    ap.add_argument("--attn-from-extent", action="store_true",
                    help="reload: decode attention reads the staged extent images, nothing is unpacked")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this library runs on one GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2604_26557_amd import binding as kv
    from paper_2604_26557_amd import workloads as W

    from paper_2604_26557_amd import build as native_build
    native_build.build_if_missing()   # a harness may build; the binding itself never does
    kv.lib()  # fails loudly if the HIP library is missing
    torch.cuda.set_device(0)
    cfg = W.config(args.config)
    lens = W.seq_lens(cfg)
    plan = kv.kv_layout_plan(cfg.n_layers, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, lens,
                             kv.KV_F16 if cfg.dtype == W.F16 else kv.KV_BF16, cfg.sector_bytes, cfg.chunk_tokens,
                             kv.KV_PER_SEQ if cfg.extent_mode == W.PER_SEQ else kv.KV_TOKEN_MAJOR,
                             cfg.lba_start, kv.KV_UNBOUNDED, cfg.pc_budget_bytes, kv.KV_UNBOUNDED)
    info = plan.info
    L = cfg.n_layers
    n1 = int(info.n_pagecache_layers)
    log(f"[bench] {cfg.name}: L={L} H={cfg.n_kv_heads} Hq={cfg.n_q_heads} D={cfg.head_dim} B={cfg.batch} "
        f"lens={lens if len(set(lens)) > 1 else lens[0]} chunk={cfg.chunk_tokens} depth={cfg.depth} "
        f"pagecache_layers={n1}")

    # ---- synthetic KV resident in HBM (seeded N(0,1) in the config's 16-bit dtype)
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    if cfg.layout == W.PAGED:
        table, n_pool = W.block_table(cfg, lens)
        table_dev = table.cuda()
        k = [W.paged_layer(cfg, l, 0, n_pool, "cuda") for l in range(L)]
        v = [W.paged_layer(cfg, l, 1, n_pool, "cuda") for l in range(L)]
        mk = lambda kk, vv, ln=lens, ld=lens_dev: kv.paged_view(kk, vv, table_dev, ln, ld)
    else:
        k = [W.bhsd_layer(cfg, l, 0, "cuda") for l in range(L)]
        v = [W.bhsd_layer(cfg, l, 1, "cuda") for l in range(L)]
        mk = lambda kk, vv, ln=lens, ld=lens_dev: kv.bhsd_view(kk, vv, ln, ld)
    src_view = mk(k, v)
    k2 = [torch.zeros_like(t) for t in k]
    v2 = [torch.zeros_like(t) for t in v]
    dst_view = mk(k2, v2)
    qs = [W.query(cfg, l, "cuda") for l in range(L)]
    outs = [torch.zeros((cfg.batch, cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda") for _ in range(L)]

    payload = 2 * L * int(info.tensor_blocks) * cfg.sector_bytes  # bytes over the link per direction
    tensor_payload = int(info.tensor_payload_bytes)
    tensor_image = int(info.tensor_blocks) * cfg.sector_bytes
    res = {
        "metric": "KV offload+reload GB/s and decode-attn us/layer, 8B-shape KV at 32K ctx",
        "value": None, "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": None, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": f"{cfg.name}: {L} layers, {cfg.n_kv_heads} KV heads, {cfg.n_q_heads} query heads, "
                               f"head_dim {cfg.head_dim}, batch {cfg.batch}, context {max(lens)}, {cfg.dtype} K/V, "
                               f"{cfg.sector_bytes} B sectors",
                   "chunk_tokens": cfg.chunk_tokens, "depth": cfg.depth, "pagecache_layers": n1,
                   "span_chunks": args.span_chunks, "layout": cfg.layout, "extent_mode": cfg.extent_mode,
                   "leg": args.leg, "attn_from_extent": args.attn_from_extent},
    }

    def roof(name, us, per_launch, where):
        ach = per_launch / (us * 1e-6) / 1e9 if us > 0 else 0.0
        return {"kernel": name, "bound": "hbm", "achieved": round(ach, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                "frac": round(ach / HBM_PEAK_GBPS, 4), "traffic": None, "us_per_launch": round(us, 2),
                "bytes_per_launch": int(per_launch), "where": where}

    if args.leg in ("both", "pipeline"):
        # ---- storage model: pinned LBA region (direct path) + pageable arena (page-cache path)
        region = torch.empty(max(int(info.region_bytes_needed), 1), dtype=torch.uint8, pin_memory=True)
        region.zero_()
        arena = np.zeros(max(int(info.pageable_bytes_needed), 1), dtype=np.uint8)
        arena[::4096] = 1  # touch every page before timing
        torch.cuda.synchronize()

        def step(timed: bool):
            a = kv.kv_pipeline_run(plan, kv.KV_DIR_OFFLOAD, 0, L, src_view, region, arena, depth=cfg.depth,
                                   span_chunks=args.span_chunks, host_workers=args.host_workers, time_kernels=timed)
            b = kv.kv_pipeline_run(plan, kv.KV_DIR_RELOAD_ATTN, 0, L, dst_view, region, arena, depth=cfg.depth,
                                   q_layers=qs, out_layers=outs, span_chunks=args.span_chunks,
                                   host_workers=args.host_workers, time_kernels=timed,
                                   attn_from_extent=args.attn_from_extent)
            return a, b

        # the link ceiling first: its passes also bring an idle link up to its settled rate before the steps
        link = measure_link(torch, min(payload, 2 << 30))
        for _ in range(args.warmup):
            step(False)
        torch.cuda.synchronize()
        stats = []
        t0 = time.perf_counter()
        for _ in range(args.steps):
            stats.append(step(True))
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0
        res["ms_per_step"] = round(elapsed / args.steps * 1e3, 3)
        res["value"] = round(2 * payload * args.steps / elapsed / 1e9, 3)
        log("[bench] per step, offload / reload+attention GB/s: " +
            ", ".join(f"{payload / a.wall_s / 1e9:.1f} / {payload / b.wall_s / 1e9:.1f}" for a, b in stats) +
            "; issuing thread waited for host copies / transfers, ms: " +
            ", ".join(f"{(a.host_copy_wait_s + b.host_copy_wait_s) * 1e3:.1f} / "
                      f"{(a.harvest_wait_s + b.harvest_wait_s) * 1e3:.1f}" for a, b in stats))

        # the timed work's result: the reloaded cache must equal the source bit for bit
        if cfg.layout == W.PAGED:   # slots past a sequence's length are not part of the cache
            bt = cfg.block_tokens
            valid = torch.zeros((n_pool, bt), dtype=torch.bool)
            for b, n in enumerate(lens):
                nb = -(-n // bt)
                valid[table[b, :nb].long()] = True
                if n % bt:
                    valid[table[b, nb - 1].long(), n % bt:] = False
            mask = valid.cuda()[:, None, :, None]
        else:
            mask = None
        for l in (() if args.attn_from_extent else (0, L - 1)):
            for a, b_ in ((k[l], k2[l]), (v[l], v2[l])):
                a, b_ = a.view(torch.int16), b_.view(torch.int16)
                if mask is not None:
                    a, b_ = torch.where(mask, a, 0), torch.where(mask, b_, 0)
                assert torch.equal(a, b_), "reload differs from source"

        off_s = sum(a.wall_s for a, _ in stats) / args.steps
        rel_s = sum(b.wall_s for _, b in stats) / args.steps

        def kstat(kind, which):
            ms = sum(s[which].kernel_ms[kind] for s in stats)
            n = sum(s[which].kernel_launches[kind] for s in stats)
            return (ms / n * 1e3 if n else 0.0), n  # microseconds per launch

        pack_us, pack_n = kstat(kv.KV_KERNEL_PACK, 0)
        unpack_us, unpack_n = kstat(kv.KV_KERNEL_UNPACK, 1)
        attn_us, attn_n = kstat(kv.KV_KERNEL_ATTN_PARTIAL, 1)
        per_t_pack = pack_n / (2 * L * args.steps)
        per_t_unpack = max(unpack_n, 1) / (2 * L * args.steps)
        where = "inside the pipeline steps (chunk commands in flight next to the kernels)"
        res["rooflines_in_pipeline"] = [
            roof("kv_layout_kernel<pack>", pack_us, (tensor_payload + tensor_image) / per_t_pack, where),
            roof("kv_layout_kernel<unpack>", unpack_us, 2 * tensor_payload / per_t_unpack, where),
            roof("kv_attn_partial_kernel+kv_attn_combine_kernel", attn_us, 2 * tensor_payload, where)]

        off_gbps = payload / off_s / 1e9
        rel_gbps = payload / rel_s / 1e9
        res["lba_seq_breaks"] = {"offload": int(stats[-1][0].lba_seq_breaks), "reload": int(stats[-1][1].lba_seq_breaks)}
        res["offload_GBps"] = round(off_gbps, 2)
        res["reload_attn_GBps"] = round(rel_gbps, 2)
        res["host_link"] = {"h2d_GBps": round(link["h2d"], 2), "d2h_GBps": round(link["d2h"], 2),
                            "offload_frac": round(off_gbps / link["d2h"], 3),
                            "reload_frac": round(rel_gbps / link["h2d"], 3),
                            "how": "back-to-back pinned 64 MiB copies, no kernels, same run before the steps, best pass"}

        # per-path throughput (outside the timed region): page-cache-path layers and direct-path layers alone
        per_path = {}
        for label, lo, hi in (("pagecache", 0, n1), ("direct", n1, L)):
            if hi > lo:
                a = kv.kv_pipeline_run(plan, kv.KV_DIR_OFFLOAD, lo, hi, src_view, region, arena, depth=cfg.depth,
                                       span_chunks=args.span_chunks, host_workers=args.host_workers)
                b = kv.kv_pipeline_run(plan, kv.KV_DIR_RELOAD, lo, hi, dst_view, region, arena, depth=cfg.depth,
                                       span_chunks=args.span_chunks, host_workers=args.host_workers)
                nb = a.bytes_direct + a.bytes_pagecache
                per_path[label] = {"offload_GBps": round(nb / a.wall_s / 1e9, 2),
                                   "reload_GBps": round(nb / b.wall_s / 1e9, 2),
                                   "offload_frac_of_link": round(nb / a.wall_s / 1e9 / link["d2h"], 3),
                                   "reload_frac_of_link": round(nb / b.wall_s / 1e9 / link["h2d"], 3)}
        if n1 > 0:
            # the extra ceiling of the page-cache path: pinned bounce memory <-> pageable arena by the host threads
            nthr = args.host_workers or 8
            nb = min(int(info.pageable_bytes_needed), 1 << 30)
            pin = torch.empty(nb, dtype=torch.uint8, pin_memory=True)
            pin.zero_()
            rates = {"from_arena": 0.0, "to_arena": 0.0}
            for _ in range(3):   # arena -> pinned, then the same bytes back: the arena keeps its contents
                rates["from_arena"] = max(rates["from_arena"], host_memcpy_rate(pin.data_ptr(), arena.ctypes.data, nb, nthr))
                rates["to_arena"] = max(rates["to_arena"], host_memcpy_rate(arena.ctypes.data, pin.data_ptr(), nb, nthr))
            rates = {k_: round(v_, 1) for k_, v_ in rates.items()}
            per_path["pagecache"]["host_memcpy_GBps"] = dict(rates, threads=nthr)
            del pin
        res["per_path"] = per_path

        # the two overlap strategies of the adaptive pipeline, one reload each, per path group
        orders = {}
        for name, code in (("intra", kv.KV_ORDER_INTRA), ("cross", kv.KV_ORDER_CROSS)):
            st = kv.kv_pipeline_run(plan, kv.KV_DIR_RELOAD, 0, L, dst_view, region, arena, depth=cfg.depth,
                                    span_chunks=args.span_chunks, host_workers=args.host_workers,
                                    order_pagecache=code, order_direct=code)
            orders[name] = {g: round(b / s_ / 1e9, 2) if s_ > 0 else None
                            for g, b, s_ in (("pagecache_GBps", st.bytes_pagecache, st.group_seconds[0]),
                                             ("direct_GBps", st.bytes_direct, st.group_seconds[1]))}
        res["reload_overlap_orders"] = orders

        # overlap fraction = (T_serial - T_pipe) / (T_serial - T_link): T_serial is one step with every
        # stage run to completion before the next starts, T_link the same bytes at the measured link rate
        sa = kv.kv_pipeline_run(plan, kv.KV_DIR_OFFLOAD, 0, L, src_view, region, arena, depth=1, serialize=True,
                                span_chunks=args.span_chunks, host_workers=args.host_workers)
        sb = kv.kv_pipeline_run(plan, kv.KV_DIR_RELOAD_ATTN, 0, L, dst_view, region, arena, depth=1, serialize=True,
                                q_layers=qs, out_layers=outs, span_chunks=args.span_chunks,
                                host_workers=args.host_workers)
        t_serial = sa.wall_s + sb.wall_s
        t_link = payload / (link["d2h"] * 1e9) + payload / (link["h2d"] * 1e9)
        t_pipe = off_s + rel_s
        res["overlap"] = {"serial_s": round(t_serial, 5), "pipeline_s": round(t_pipe, 5), "link_s": round(t_link, 5),
                          "fraction": round((t_serial - t_pipe) / (t_serial - t_link), 3) if t_serial > t_link else None}
        res["decode_attn_us_per_layer_in_pipeline"] = round(attn_us, 2)

        # the decode step's other two forms (outside the timed region): reload with attention straight from the
        # staged extent images (no unpack), and the append of one new token row to every tensor
        if not args.attn_from_extent and args.span_chunks == 0:
            fe = kv.kv_pipeline_run(plan, kv.KV_DIR_RELOAD_ATTN, 0, L, dst_view, region, arena, depth=cfg.depth,
                                    q_layers=qs, out_layers=outs, host_workers=args.host_workers, attn_from_extent=True)
            res["reload_attn_from_extent_GBps"] = round(payload / fe.wall_s / 1e9, 2)
        if min(lens) >= 2:
            short = [n - 1 for n in lens]   # store all but the last token, then append it
            short_dev = torch.tensor(short, dtype=torch.int32, device="cuda")
            short_view = mk(k, v, short, short_dev)
            for timed in (False, True):      # the first round creates the library's append buffers
                kv.kv_pipeline_run(plan, kv.KV_DIR_OFFLOAD, 0, L, short_view, region, arena, depth=cfg.depth,
                                   host_workers=args.host_workers)
                t0 = time.perf_counter()
                ap_st = kv.kv_append_tokens(plan, 0, L, src_view, region, arena)
                ap_s = time.perf_counter() - t0
            res["decode_append"] = {"us_all_layers": round(ap_s * 1e6, 1), "write_cmds": int(ap_st.n_cmds),
                                    "rmw_sector_reads": int(ap_st.n_rmw_reads), "sectors_written": int(ap_st.blocks_written)}
        del region, arena

    if args.leg in ("both", "kernels"):
        kl = kernel_leg(torch, kv, cfg, plan, info, src_view, dst_view, k, qs, outs, lens, reps=max(3, args.steps))
        where = "resident-KV leg: whole-tensor launches back to back, rotating over all layers"
        tpl = kl["tensors_per_launch"]
        rl = [roof("kv_layout_kernel<pack>", kl["pack_us"], tpl * (tensor_payload + tensor_image), where),
              roof("kv_layout_kernel<unpack>", kl["unpack_us"], tpl * 2 * tensor_payload, where),
              roof("kv_attn_partial_kernel+kv_attn_combine_kernel", kl["attn_us"], 2 * tensor_payload, where)]
        if cfg.name in PMC_TRAFFIC and kernel_sources_hash() == PMC_TRAFFIC["sha"]:
            for r in rl:
                r["traffic"] = PMC_TRAFFIC[cfg.name].get(r["kernel"])
        res["rooflines"] = rl
        res["decode_attn_us_per_layer"] = round(kl["attn_us"], 2)
        res["decode_attn_graph"] = {"us_per_layer": None if kl["attn_graph_us"] is None else round(kl["attn_graph_us"], 2),
                                    "how": "the launches of all layers recorded in one HIP graph and replayed "
                                           "(kv_decode_attn_static: no workspace, no allocation)",
                                    **({"error": kl["attn_graph_error"]} if "attn_graph_error" in kl else {})}
        # the dominant kernel of a step: the one with the most GPU time over its launches
        tot = [kl["pack_us"] * kl["layout_launches"], kl["unpack_us"] * kl["layout_launches"], kl["attn_us"] * L]
        dom = rl[max(range(3), key=lambda i: tot[i])]
        res["roofline"] = {key: dom[key] for key in ("bound", "achieved", "peak", "unit", "frac", "traffic", "kernel", "where")}
    else:
        dom = max(res["rooflines_in_pipeline"], key=lambda r: r["us_per_launch"])
        res["roofline"] = {key: dom[key] for key in ("bound", "achieved", "peak", "unit", "frac", "traffic", "kernel", "where")}

    if not args.no_cpu_baseline:
        log("[bench] timing the CPU checker on a bounded sample ...")
        def gpu_attn(K, V, q):
            Kd, Vd, qd = K.cuda(), V.cuda(), q.cuda()
            view = mk([Kd], [Vd])
            out = torch.empty((cfg.batch, cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(plan, 0, max(lens)), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(plan, view, 0, qd, out, kv.KV_OUT_F32, 0, ws)
            torch.cuda.synchronize()
            return out.double().cpu().numpy()

        res["cpu_baseline"] = cpu_baseline(cfg, W, gpu_attn=gpu_attn)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
