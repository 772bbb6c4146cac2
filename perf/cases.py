"""The work that is timed: what a program that offloads its KV cache has this library do, through the binding's
public calls, from a two-layer toy to gigabytes per pass.

A case is a dict of plain values.  `kind` says which calls one pass makes:
  decode   decode attention of every layer over resident KV (one decode step of a model)
  pack     attention-side KV -> extent images of whole layers (`per` = "layer": a call per layer as prefill
           finishes it; "all": one call for all layers; "chunk": a call per layer for one chunk of token rows)
  unpack   the inverse
  step     the pipeline: offload all layers to host memory, reload them and attend (write after prefill, read in decode)
  append   one new token row of every sequence and tensor to its extent

Lengths, block tables and everything else that fixes the amount of work come from the case; values come from the seed.
K, V and Q are N(0,1) rounded to 16 bits, as in the tests and the benchmark.
"""
import math
import random

import numpy as np
import torch

from paper_2604_26557_amd import binding as kv

MiB = 1 << 20
SECTOR = 4096


def _case(kind, L, H, G, D, B, lo, hi, dtype, layout, **more):
    c = {"kind": kind, "L": L, "H": H, "G": G, "D": D, "B": B, "lo": lo, "hi": hi, "dtype": dtype, "layout": layout,
         "bt": 16, "lens_seed": 3, "out": "f32", "graph": False, "per": "layer", "chunk": 1024, "depth": 4, "pc_layers": 0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: two layers, 256 tokens, latency and launches only
        _case("decode", 2, 2, 2, 64, 1, 256, 256, "f16", "bhsd", name="decode_tiny"),
        # one interactive sequence at 4K context, 8B shape; a serving loop replays the step as a HIP graph
        _case("decode", 32, 8, 4, 128, 1, 4096, 4096, "f16", "bhsd", graph=True, name="decode_4k_graph"),
        # one long sequence, 8B shape at 32K (the benchmark's headline shape), half of the layers
        _case("decode", 16, 8, 4, 128, 1, 32768, 32768, "bf16", "bhsd", name="decode_32k"),
        # a ragged batch over a paged cache, 8B shape
        _case("decode", 16, 8, 4, 128, 8, 1024, 8192, "f16", "paged", name="decode_ragged_paged"),
        # the paper's own workload: batch 32, prompts of 512 plus up to 32 generated tokens, 32 KV heads without grouping
        _case("decode", 8, 32, 1, 128, 32, 512, 544, "f16", "bhsd", out="same", name="decode_batch32_mha"),
        # wide heads without grouping, batch 4 at 8K: the most bytes per layer
        _case("decode", 4, 16, 1, 256, 4, 8192, 8192, "bf16", "bhsd", name="decode_mha_8k"),
        # a serving batch of many ragged sequences over a paged cache, an odd number of query heads per KV head
        _case("decode", 8, 4, 7, 128, 48, 200, 4000, "bf16", "paged", out="same", name="decode_serving_paged"),
        # offload after prefill, all layers of a 4K context in one call
        _case("pack", 32, 8, 4, 128, 1, 4096, 4096, "f16", "bhsd", per="all", name="pack_4k"),
        # chunked prefill: the newest 256 token rows of every layer, a small call per layer
        _case("pack", 32, 8, 4, 128, 1, 4096, 4096, "f16", "bhsd", per="chunk", chunk=256, name="pack_chunk"),
        # reload of a ragged batch into a paged cache, a call per layer as its images land
        _case("unpack", 8, 8, 4, 128, 8, 1024, 8192, "f16", "paged", name="unpack_ragged_paged"),
        # the benchmark's step at 32K: both paths, 2 MiB commands
        _case("step", 4, 8, 4, 128, 1, 32768, 32768, "bf16", "bhsd", pc_layers=2, name="step_32k"),
        # a decode step's write-back: one row per layer, kind and sequence
        _case("append", 32, 8, 4, 128, 8, 33, 200, "f16", "paged", pc_layers=16, name="append_ragged"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 6 + ["pack"] * 2 + ["unpack"] * 2 + ["step", "append"])
    D = rng.choice([64, 128, 128, 256])
    H = rng.choice([1, 2, 3, 4, 5, 8, 8, 16, 32])
    G = rng.choice([1, 1, 2, 3, 4, 4, 5, 6, 7, 8])
    B = _log_int(rng, 1, 96)
    hi = _log_int(rng, 48, 32768)
    lo = hi if rng.random() < 0.3 else rng.randint(max(1, hi // 8), hi)
    dtype, layout = rng.choice(["f16", "bf16"]), rng.choice(["bhsd", "paged"])
    more = {"lens_seed": rng.randrange(1 << 30), "out": rng.choice(["f32", "same"])}
    if layout == "paged":
        more["bt"] = rng.choice([16, 16, 16, 32, 64])
    if kind in ("pack", "unpack"):
        more["per"] = rng.choice(["layer", "all"] + (["chunk"] if kind == "pack" else []))
    if kind == "append":  # the cost does not depend on the context: short extents keep the host buffers small
        B, hi = min(B, 32), min(hi, 400)
        lo = min(lo, hi)
    if kind == "step":  # one sequence, or a uniform or ragged batch
        B = min(B, 16)
    limit = (96 if kind == "step" else 512) * MiB  # K and V of one layer
    while B * hi * H * D * 4 > limit:
        if hi > 512 and (B == 1 or rng.random() < 0.5):
            hi = max(48, hi // 2)
            lo = max(1, min(lo // 2, hi))
        elif B > 1:
            B = max(1, B // 2)
        else:
            H = max(1, H // 2)
    total = {"decode": 1600, "pack": 768, "unpack": 768, "step": 384, "append": 128}[kind] * MiB
    L = max(1, min(32, total // (B * hi * H * D * 4)))
    if kind == "step":
        more["pc_layers"] = rng.choice([0, L // 2, L])
        more["depth"] = rng.choice([3, 4])
    if kind == "append":
        more["pc_layers"] = L // 2
    row = (H * D * 2) * (B if lo == hi else 1)
    unit = SECTOR // math.gcd(row, SECTOR)  # token rows whose bytes are whole sectors
    want = _log_int(rng, 512 * 1024, 8 * MiB) if kind == "step" else _log_int(rng, 64 * 1024, 4 * MiB)
    more["chunk"] = unit * max(1, want // row // unit)
    if more.get("per") == "chunk" and more["chunk"] > lo:
        more["per"] = "layer"
    if kind == "decode" and rng.random() < 0.2 and B * H * G * D <= 65536 and hi <= 8192:
        more["graph"] = True
    return _case(kind, L, H, G, D, B, lo, hi, dtype, layout, **more)


def _lens(c):
    r = random.Random(c["lens_seed"])
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["B"])]


def _plan(c, lens):
    uniform = c["lo"] == c["hi"]
    row = c["H"] * c["D"] * 2
    blocks = (len(lens) * lens[0] * row + SECTOR - 1) // SECTOR if uniform else sum((n * row + SECTOR - 1) // SECTOR for n in lens)
    # a chunk is whole sectors of token rows
    unit = SECTOR // math.gcd(row * (c["B"] if uniform else 1), SECTOR)
    chunk = max(unit, c["chunk"] // unit * unit)
    return kv.kv_layout_plan(c["L"], c["H"], c["H"] * c["G"], c["D"], lens, kv.KV_F16 if c["dtype"] == "f16" else kv.KV_BF16,
                             SECTOR, chunk, kv.KV_TOKEN_MAJOR if uniform else kv.KV_PER_SEQ,
                             lba_start=2048, pc_budget_bytes=c["pc_layers"] * 2 * blocks * SECTOR)


def _normal(shape, dtype, gen):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    for i in range(shape[0]):
        t[i] = torch.randn(shape[1:], generator=gen, device="cuda", dtype=torch.float32)
    return t


def _table(c, lens):
    """Block table of a pool in which every sequence owns blocks at random places."""
    per = [(n + c["bt"] - 1) // c["bt"] for n in lens]
    ids = list(range(sum(per)))
    random.Random(c["lens_seed"] + 1).shuffle(ids)
    t, base = np.full((len(lens), max(per)), -1, dtype=np.int32), 0
    for b, n in enumerate(per):
        t[b, :n] = ids[base:base + n]
        base += n
    return torch.from_numpy(t), len(ids)


def _dtype(c):
    return torch.float16 if c["dtype"] == "f16" else torch.bfloat16


def _kv_shape(c, lens, n_pool):
    if c["layout"] == "paged":
        return (c["L"], n_pool, c["H"], c["bt"], c["D"])
    return (c["L"], c["B"], c["H"], max(lens), c["D"])


def _view(c, s, k, v):
    ks, vs = [k[i] for i in range(c["L"])], [v[i] for i in range(c["L"])]
    if c["layout"] == "paged":
        return kv.paged_view(ks, vs, s["table"], s["lens"], s["lens_dev"])
    return kv.bhsd_view(ks, vs, s["lens"], s["lens_dev"])


def prepare(case, seed):
    c, kind = case, case["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    lens = _lens(c)
    s = {"case": c, "lens": lens, "lens_dev": torch.tensor(lens, dtype=torch.int32, device="cuda"), "plan": _plan(c, lens)}
    info = s["plan"].info
    n_pool = 0
    if c["layout"] == "paged":
        table, n_pool = _table(c, lens)
        s["table"] = table.cuda()
    shape, dt = _kv_shape(c, lens, n_pool), _dtype(c)
    image = int(info.tensor_blocks) * SECTOR

    if kind == "unpack":
        s["src"] = torch.randint(0, 256, (c["L"], 2 * image), dtype=torch.uint8, device="cuda", generator=gen)
        s["k"], s["v"] = torch.zeros(shape, dtype=dt, device="cuda"), torch.zeros(shape, dtype=dt, device="cuda")
        s["view"] = _view(c, s, s["k"], s["v"])
        return s
    s["k"], s["v"] = _normal(shape, dt, gen), _normal(shape, dt, gen)
    s["view"] = _view(c, s, s["k"], s["v"])
    if kind == "pack":
        if c["per"] == "chunk":
            # the last whole chunk of the shortest sequence
            C = int(info.chunk_tokens)
            tok0 = max(0, (min(lens) // C - 1) * C)
            n = min(C, min(lens) - tok0)
            s["tok0"], s["ntok"] = tok0, n
            req = kv.kv_plan_translate(s["plan"], 0, kv.KV_K, 0, tok0, n)[1]
            s["dst"] = torch.zeros((c["L"], 2 * req), dtype=torch.uint8, device="cuda")
        else:
            s["dst"] = torch.zeros((c["L"], 2 * image), dtype=torch.uint8, device="cuda")
    if kind in ("decode", "step"):
        odt = torch.float32 if c["out"] == "f32" else dt
        s["q"] = _normal((c["L"], c["B"], c["H"] * c["G"], c["D"]), dt, gen)
        s["out"] = torch.zeros((c["L"], c["B"], c["H"] * c["G"], c["D"]), dtype=odt, device="cuda")
        s["odt"] = kv.KV_OUT_F32 if c["out"] == "f32" else kv.KV_OUT_SAME
    if kind == "decode":
        if c["graph"]:
            _decode(s)  # the library resolves its own scratch memory outside the capture
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                _decode(s)
            s["graph"] = g
        else:
            s["ws"] = torch.empty(kv.kv_decode_attn_workspace(s["plan"], 0, max(lens)), dtype=torch.uint8, device="cuda")
    if kind in ("step", "append"):
        s["region"] = torch.empty(max(1, int(info.region_bytes_needed)), dtype=torch.uint8, pin_memory=True).zero_()
        s["arena"] = torch.zeros(max(1, int(info.pageable_bytes_needed)), dtype=torch.uint8)
    if kind == "step":
        s["k2"], s["v2"] = torch.zeros_like(s["k"]), torch.zeros_like(s["v"])
        s["view2"] = _view(c, s, s["k2"], s["v2"])
    return s


def _decode(s):
    c = s["case"]
    for l in range(c["L"]):
        if c["graph"]:
            kv.kv_decode_attn_static(s["plan"], s["view"], l, s["q"][l], s["out"][l], s["odt"])
        else:
            kv.kv_decode_attn(s["plan"], s["view"], l, s["q"][l], s["out"][l], s["odt"], 0, s["ws"])


def run(state):
    s = state
    c, L = s["case"], s["case"]["L"]
    kind = c["kind"]
    if kind == "decode":
        if c["graph"]:
            s["graph"].replay()
        else:
            _decode(s)
        return s["out"]
    if kind == "pack":
        if c["per"] == "all":
            kv.kv_offload_pack_layers(s["plan"], 0, L, s["view"], s["dst"])
        elif c["per"] == "layer":
            for l in range(L):
                kv.kv_offload_pack(s["plan"], l, kv.KV_KV, s["view"], kv.KV_SEQ_ALL, 0, 0, s["dst"][l])
        else:
            for l in range(L):
                kv.kv_offload_pack(s["plan"], l, kv.KV_KV, s["view"], 0, s["tok0"], s["ntok"], s["dst"][l])
        return s["dst"]
    if kind == "unpack":
        if c["per"] == "all":
            kv.kv_reload_unpack_layers(s["plan"], 0, L, s["src"], s["view"])
        else:
            for l in range(L):
                kv.kv_reload_unpack(s["plan"], l, kv.KV_KV, s["src"][l], s["view"], kv.KV_SEQ_ALL, 0, 0)
        return {"k": s["k"].view(torch.int16), "v": s["v"].view(torch.int16)}
    if kind == "step":
        kv.kv_pipeline_run(s["plan"], kv.KV_DIR_OFFLOAD, 0, L, s["view"], s["region"], s["arena"], depth=c["depth"])
        kv.kv_pipeline_run(s["plan"], kv.KV_DIR_RELOAD_ATTN, 0, L, s["view2"], s["region"], s["arena"], depth=c["depth"],
                           q_layers=list(s["q"].unbind(0)), out_layers=list(s["out"].unbind(0)), out_dtype=s["odt"])
        return {"out": s["out"], "k": s["k2"].view(torch.int16), "v": s["v2"].view(torch.int16), "region": s["region"], "arena": s["arena"]}
    st = kv.kv_append_tokens(s["plan"], 0, L, s["view"], s["region"], s["arena"])
    return {"region": s["region"], "arena": s["arena"], "commands": int(st.n_cmds), "blocks": int(st.blocks_written)}


def work(case):
    c = case
    tokens = sum(_lens(c))
    kv_bytes = c["L"] * 2 * tokens * c["H"] * c["D"] * 2
    qo = c["L"] * c["B"] * c["H"] * c["G"] * c["D"] * (2 + (4 if c["out"] == "f32" else 2))
    flops = 4.0 * c["L"] * tokens * c["H"] * c["G"] * c["D"]
    if c["kind"] == "decode":
        return {"bytes": kv_bytes + qo, "flops": flops}
    if c["kind"] == "step":  # every byte out over the link, back, and into the attention-side buffers
        return {"bytes": 4 * kv_bytes + qo, "flops": flops}
    if c["kind"] == "append":
        return {"bytes": 2 * c["L"] * 2 * c["B"] * c["H"] * c["D"] * 2, "flops": 0}
    if c["kind"] == "pack" and c["per"] == "chunk":
        n = min(c["chunk"], c["lo"]) * (c["B"] if c["lo"] == c["hi"] else 1)
        return {"bytes": 2 * c["L"] * 2 * n * c["H"] * c["D"] * 2, "flops": 0}
    return {"bytes": 2 * kv_bytes, "flops": 0}


def tolerance(case):
    if case["kind"] not in ("decode", "step"):
        return "exact"
    if case["out"] == "f32":
        return {"rel": 1.2e-6}  # 16-bit products are exact, sums are 32-bit: 1.8e-7 to 2.9e-7 from 64 bits as measured
    return {"rel": 8.4e-4} if case["dtype"] == "f16" else {"rel": 6.8e-3}  # one rounding to 11 or 8 bits: 2.1e-4, 1.7e-3


def exact(case, seed):
    if case["kind"] not in ("decode", "step"):
        return None
    c = case
    s = prepare(c, seed)
    out = torch.zeros((c["L"], c["B"], c["H"] * c["G"], c["D"]), dtype=torch.float64, device="cuda")
    for l in range(c["L"]):
        for b, n in enumerate(s["lens"]):
            K, V = (_rows(c, s, t[l], b, n) for t in (s["k"], s["v"]))  # [H, n, D]
            q = s["q"][l, b].view(c["H"], c["G"], c["D"]).double().transpose(1, 2).contiguous()
            p = torch.softmax(torch.matmul(K, q) / math.sqrt(c["D"]), dim=1).transpose(1, 2).contiguous()
            out[l, b] = torch.matmul(p, V).reshape(c["H"] * c["G"], c["D"])
    return out if c["kind"] == "decode" else {"out": out, "k": None, "v": None, "region": None, "arena": None}


def _rows(c, s, t, b, n):
    if c["layout"] == "bhsd":
        return t[b, :, :n].double()
    ids = s["table"][b, :(n + c["bt"] - 1) // c["bt"]].long()
    return t[ids].transpose(0, 1).reshape(c["H"], -1, c["D"])[:, :n].double()
