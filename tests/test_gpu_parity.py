"""GPU parity: the HIP path (through the C ABI) against the CPU checker, element by element, on
reduced shapes of the five evaluation configs that still span several tiles and a ragged tail.
Pack / unpack / host-region bytes must be bit-exact; attention within 2e-3 max abs error of the fp64
reference (and 1e-2 of the reference's own max magnitude, so the check is not vacuous)."""
import os

import numpy as np
import pytest
import torch

from oracle import kv_oracle as o
from paper_2604_26557_amd import binding as kv
from paper_2604_26557_amd import workloads as W
from kvcase import Case, bits, pinned_bytes

pytestmark = pytest.mark.gpu

ATTN_ATOL = 2e-3
ATTN_REL_OF_MAX = 1e-2
GUARD = 4096
CANARY = 0xA5


def small_configs():
    c = W.CONFIGS
    return [
        c[0],
        W.shrink(c[1], n_layers=3, seq_len=1001),
        W.shrink(c[2], n_layers=4, seq_len=3000, pc_budget_bytes=2 * 2 * 3000 * 2048),
        W.shrink(c[3], n_layers=3, batch=4, len_range=(100, 1500)),
        W.shrink(c[4], n_layers=3, seq_len=600, pc_budget_bytes=1 * 2 * 600 * 32768),
        # shapes outside the five: odd head count (row of 5*8 vectors), B=3 token-major, 512 B sectors
        W.KVConfig("odd_heads", 7, 2, 5, 10, 64, 3, W.F16, 512, 4, 2, W.TOKEN_MAJOR, W.BHSD, 203),
        # token-major extent from a paged source, G = 8
        W.KVConfig("paged_token_major", 8, 2, 1, 8, 128, 2, W.BF16, 4096, 32, 2, W.TOKEN_MAJOR, W.PAGED, 320),
    ]


SMALL = small_configs()
IDS = [c.name for c in SMALL]


@pytest.fixture(scope="module", params=SMALL, ids=IDS)
def case(request):
    torch.cuda.set_device(0)
    return Case(request.param, "cuda", gen_device="cpu")


def _guarded(nbytes):
    buf = torch.full((nbytes + 2 * GUARD,), CANARY, dtype=torch.uint8, device="cuda")
    return buf, buf[GUARD:GUARD + nbytes]


def _guards_intact(buf, nbytes):
    b = buf.cpu().numpy()
    return (b[:GUARD] == CANARY).all() and (b[GUARD + nbytes:] == CANARY).all()


# ------------------------------------------------------------------------------------------ pack
def test_pack_whole_tensor(case):
    r = case.ref
    nbytes = r.n_blocks_tensor * r.lba_size
    for layer in sorted({0, case.cfg.n_layers - 1}):
        for kind in (0, 1):
            buf, dst = _guarded(nbytes)
            kv.kv_offload_pack(case.plan, layer, kind, case.view, kv.KV_SEQ_ALL, 0, 0, dst)
            torch.cuda.synchronize()
            assert np.array_equal(dst.cpu().numpy(), case.expected_extent(layer, kind)), (layer, kind)
            assert _guards_intact(buf, nbytes)


def test_pack_chunk_ranges(case):
    r = case.ref
    layer, kind = case.cfg.n_layers - 1, 1
    want = case.expected_extent(layer, kind)
    nseq = len(case.lens) if r.per_seq else 1
    for b in range(nseq):
        base = int(r.seq_base[b]) * r.lba_size
        for c in kv.kv_plan_chunk_cmds(case.plan, layer, kind, b):
            nbytes = (c.nlb + 1) * r.lba_size
            buf, dst = _guarded(nbytes)
            kv.kv_offload_pack(case.plan, layer, kind, case.view, b, c.tok0, c.ntok, dst)
            torch.cuda.synchronize()
            got = dst.cpu().numpy()
            assert np.array_equal(got, want[base + c.buf_off: base + c.buf_off + nbytes]), (b, c.tok0)
            assert _guards_intact(buf, nbytes)


def test_pack_unpack_both_tensors_in_one_launch(case):
    """kind = KV_KV: K's image, then V's, from one launch; whole extents and one chunk range."""
    r = case.ref
    ext_bytes = r.n_blocks_tensor * r.lba_size
    layer = case.cfg.n_layers - 1
    buf, dst = _guarded(2 * ext_bytes)
    kv.kv_offload_pack(case.plan, layer, kv.KV_KV, case.view, kv.KV_SEQ_ALL, 0, 0, dst)
    torch.cuda.synchronize()
    want_k, want_v = case.expected_extent(layer, 0), case.expected_extent(layer, 1)
    got = dst.cpu().numpy()
    assert np.array_equal(got[:ext_bytes], want_k) and np.array_equal(got[ext_bytes:], want_v)
    assert _guards_intact(buf, 2 * ext_bytes)

    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    kv.kv_reload_unpack(case.plan, layer, kv.KV_KV, dst, view, kv.KV_SEQ_ALL, 0, 0)
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, [layer])

    c = kv.kv_plan_chunk_cmds(case.plan, layer, 0, 0)[-1]          # the ragged tail chunk of sequence 0
    nbytes = (c.nlb + 1) * r.lba_size
    buf, dst = _guarded(2 * nbytes)
    kv.kv_offload_pack(case.plan, layer, kv.KV_KV, case.view, 0, c.tok0, c.ntok, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    assert np.array_equal(got[:nbytes], want_k[c.buf_off:c.buf_off + nbytes])
    assert np.array_equal(got[nbytes:], want_v[c.buf_off:c.buf_off + nbytes])
    assert _guards_intact(buf, 2 * nbytes)


# ------------------------------------------------------------------------------------------ unpack
def test_pack_unpack_several_layers_in_one_call(case):
    """kv_offload_pack_layers / kv_reload_unpack_layers: the images of K and V of a run of layers, back to back in
    tensor-id order, equal the single-tensor images; the inverse restores every layer of the run and no other."""
    r, L = case.ref, case.cfg.n_layers
    image = r.n_blocks_tensor * r.lba_size
    for lb, le in ((0, L), (L - 1, L), (1, 1)):
        n = le - lb
        buf, dst = _guarded(2 * n * image)
        if n == 0:
            dst = buf                                      # an empty run writes nothing anywhere
        kv.kv_offload_pack_layers(case.plan, lb, le, case.view, dst)
        torch.cuda.synchronize()
        got = dst.cpu().numpy()
        for l in range(lb, le):
            for kind in (0, 1):
                j = (l - lb) * 2 + kind
                assert np.array_equal(got[j * image:(j + 1) * image], case.expected_extent(l, kind)), (lb, le, l, kind)
        assert _guards_intact(buf, 2 * n * image) and (n > 0 or (buf.cpu().numpy() == CANARY).all())
        k_new, v_new = case.blank_like_source()
        kv.kv_reload_unpack_layers(case.plan, lb, le, dst, case.make_view(k_new, v_new))
        torch.cuda.synchronize()
        _check_restored(case, k_new, v_new, range(lb, le))
        for l in set(range(L)) - set(range(lb, le)):       # layers outside the run keep their fill
            assert (bits(k_new[l]) == 0x7E7E).all() and (bits(v_new[l]) == 0x7E7E).all()
    small = torch.empty(2 * L * image - 16, dtype=torch.uint8, device="cuda")
    for f, args in ((kv.kv_offload_pack_layers, (case.plan, 0, L, case.view, small)),
                    (kv.kv_reload_unpack_layers, (case.plan, 0, L, small, case.view))):
        with pytest.raises(kv.KVError) as e:
            f(*args)
        assert e.value.code == kv.KV_ENOSPC
    with pytest.raises(kv.KVError) as e:
        kv.kv_offload_pack_layers(case.plan, 0, L + 1, case.view, small)
    assert e.value.code == kv.KV_ERANGE


def _check_restored(case, k_new, v_new, layers, fill=0x7E7E):
    cfg = case.cfg
    for layer in layers:
        for kind, new in ((0, k_new), (1, v_new)):
            got, src = bits(new[layer]), bits(case.tensor_cpu(layer, kind))
            if case.paged:
                bt = cfg.block_tokens
                table = case.table_cpu.numpy()
                touched = np.zeros(got.shape[:1] + got.shape[2:3], dtype=bool)   # [n_pool, bt]
                for b, n in enumerate(case.lens):
                    for s in range(n):
                        touched[table[b, s // bt], s % bt] = True
                m = touched[:, None, :, None]
                assert np.array_equal(np.where(m, got, 0), np.where(m, src, 0))
                assert (np.where(m, fill, got) == fill).all()                     # other slots untouched
            else:
                for b, n in enumerate(case.lens):
                    assert np.array_equal(got[b, :, :n], src[b, :, :n])
                    assert (got[b, :, n:] == fill).all()


def test_unpack_whole_tensor(case):
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    layers = sorted({0, case.cfg.n_layers - 1})
    for layer in layers:
        for kind in (0, 1):
            ext = torch.from_numpy(case.expected_extent(layer, kind)).cuda()
            kv.kv_reload_unpack(case.plan, layer, kind, ext, view, kv.KV_SEQ_ALL, 0, 0)
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, layers)


def test_unpack_chunk_ranges(case):
    r = case.ref
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    layer = 0
    nseq = len(case.lens) if r.per_seq else 1
    for kind in (0, 1):
        ext = case.expected_extent(layer, kind)
        for b in range(nseq):
            base = int(r.seq_base[b]) * r.lba_size
            for c in kv.kv_plan_chunk_cmds(case.plan, layer, kind, b):
                nbytes = (c.nlb + 1) * r.lba_size
                img = torch.from_numpy(ext[base + c.buf_off: base + c.buf_off + nbytes].copy()).cuda()
                kv.kv_reload_unpack(case.plan, layer, kind, img, view, b, c.tok0, c.ntok)
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, [layer])


@pytest.mark.parametrize("cfg", [SMALL[0], SMALL[3], SMALL[5]], ids=lambda c: c.name)
def test_round_trip_raw_bit_patterns(cfg):
    """Pack is a byte move: NaN / Inf / denormal payloads must survive unchanged."""
    case = Case(cfg, "cuda", raw=True, gen_device="cpu", s_extra=3)
    r = case.ref
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    nbytes = r.n_blocks_tensor * r.lba_size
    for layer in range(cfg.n_layers):
        for kind in (0, 1):
            buf, dst = _guarded(nbytes)
            kv.kv_offload_pack(case.plan, layer, kind, case.view, kv.KV_SEQ_ALL, 0, 0, dst)
            torch.cuda.synchronize()
            assert np.array_equal(dst.cpu().numpy(), case.expected_extent(layer, kind))
            kv.kv_reload_unpack(case.plan, layer, kind, dst, view, kv.KV_SEQ_ALL, 0, 0)
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, range(cfg.n_layers))


def test_pack_shorter_than_capacity_zero_fills():
    """Valid length below the extent capacity: rows [0,len) then zeros to the end of the extent."""
    cfg = W.shrink(W.CONFIGS[0], seq_len=256)
    case = Case(cfg, "cuda", gen_device="cpu")
    lens = [100]
    view = kv.bhsd_view(case.k, case.v, lens, case.lens_dev)
    r = case.ref
    nbytes = r.n_blocks_tensor * r.lba_size
    buf, dst = _guarded(nbytes)
    kv.kv_offload_pack(case.plan, 1, 0, view, kv.KV_SEQ_ALL, 0, 0, dst)
    torch.cuda.synchronize()
    want = np.zeros(nbytes, dtype=np.uint8)
    t = case.k_cpu[1]
    o.pack(case.source(t), o.u16(t), False, lens, r.seq_base, r.n_blocks_tensor, r.lba_size, want)
    assert np.array_equal(dst.cpu().numpy(), want) and not want[100 * 256:].any()
    assert _guards_intact(buf, nbytes)


def test_kernel_argument_errors(case):
    """Bad arguments are rejected on the host before anything is launched."""
    r = case.ref
    dst = torch.zeros(r.n_blocks_tensor * r.lba_size, dtype=torch.uint8, device="cuda")

    def code(fn):
        with pytest.raises(kv.KVError) as e:
            fn()
        return e.value.code

    cap = case.lens[0]
    assert code(lambda: kv.kv_offload_pack(case.plan, 99, 0, case.view, kv.KV_SEQ_ALL, 0, 0, dst)) == kv.KV_ERANGE
    assert code(lambda: kv.kv_offload_pack(case.plan, 0, 3, case.view, kv.KV_SEQ_ALL, 0, 0, dst)) == kv.KV_EINVAL
    assert code(lambda: kv.kv_offload_pack(case.plan, 0, 0, case.view, 0, 0, cap + 1, dst)) == kv.KV_ERANGE
    assert code(lambda: kv.kv_offload_pack(case.plan, 0, 0, case.view, kv.KV_SEQ_ALL, 0, 0, dst[:4096])) == kv.KV_ENOSPC
    assert code(lambda: kv.kv_offload_pack(case.plan, 0, 0, case.view, kv.KV_SEQ_ALL, 0, 0, dst[8:])) == kv.KV_EINVAL
    if (r.row_bytes % r.lba_size) != 0 and cap > 2:
        assert code(lambda: kv.kv_offload_pack(case.plan, 0, 0, case.view, 0, 1, 1, dst)) == kv.KV_EALIGN
    assert code(lambda: kv.kv_reload_unpack(case.plan, 0, 0, dst[:4096], case.view, kv.KV_SEQ_ALL, 0, 0)) == kv.KV_ENOSPC
    assert code(lambda: kv.kv_reload_unpack(case.plan, -1, 0, dst, case.view, kv.KV_SEQ_ALL, 0, 0)) == kv.KV_ERANGE

    # decode attention
    cfg = case.cfg
    q = W.query(cfg, 0, "cuda")
    out = torch.zeros((len(case.lens), cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, 0, max(case.lens)), dtype=torch.uint8, device="cuda")
    attn = lambda **kw: kv.kv_decode_attn(**dict(dict(plan=case.plan, kv=case.view, layer=0, q=q, out=out,
                                                      out_dtype=kv.KV_OUT_F32, n_splits=0, workspace=ws), **kw))
    attn()
    torch.cuda.synchronize()
    assert code(lambda: attn(layer=99)) == kv.KV_ERANGE
    assert code(lambda: attn(out_dtype=5)) == kv.KV_EINVAL
    assert code(lambda: attn(n_splits=1025)) == kv.KV_EINVAL
    assert code(lambda: attn(n_splits=-1)) == kv.KV_EINVAL
    assert code(lambda: attn(workspace=ws[:64])) == kv.KV_ENOSPC
    misaligned = torch.zeros(q.numel() * 2 + 16, dtype=torch.uint8, device="cuda")[2:]
    assert code(lambda: attn(q=misaligned)) == kv.KV_EINVAL


# ------------------------------------------------------------------------------------------ attention
def _attn_check(got: torch.Tensor, want: np.ndarray):
    g = got.double().cpu().numpy()
    err = np.abs(g - want).max()
    scale = np.abs(want).max()
    assert err <= ATTN_ATOL, err
    assert err <= ATTN_REL_OF_MAX * scale, (err, scale)


@pytest.mark.parametrize("n_splits", [0, 1, 3, 70, 200])
def test_decode_attention(case, n_splits):
    cfg = case.cfg
    max_len = max(case.lens)
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max_len), dtype=torch.uint8, device="cuda")
    for layer in sorted({0, cfg.n_layers - 1}):
        q = W.query(cfg, layer, "cpu")
        qd = q.cuda()
        out = torch.full((len(case.lens), cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")
        kv.kv_decode_attn(case.plan, case.view, layer, qd, out, kv.KV_OUT_F32, n_splits, ws)
        torch.cuda.synchronize()
        _attn_check(out, case.expected_attention(layer, q))


def test_decode_attention_16bit_output_and_short_lengths(case):
    """Output in the KV dtype is the fp32 result rounded to nearest even; a zero-length sequence gives zeros."""
    cfg = case.cfg
    lens = list(case.lens)
    lens[0] = 1
    if len(lens) > 1:
        lens[1] = 0
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    view = (kv.paged_view(case.k, case.v, case.table_dev, lens, lens_dev) if case.paged
            else kv.bhsd_view(case.k, case.v, lens, lens_dev))
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, 0, max(lens)), dtype=torch.uint8, device="cuda")
    q = W.query(cfg, 0, "cpu")
    shape = (len(lens), cfg.n_q_heads, cfg.head_dim)
    out32 = torch.empty(shape, dtype=torch.float32, device="cuda")
    out16 = torch.empty(shape, dtype=cfg.torch_dtype, device="cuda")
    kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out32, kv.KV_OUT_F32, 0, ws)
    kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out16, kv.KV_OUT_SAME, 0, ws)
    torch.cuda.synchronize()
    K, V = case.k_cpu[0], case.v_cpu[0]
    want = o.attention(case.source(K), o.u16(K), o.u16(V), o.u16(q), cfg.dtype == W.BF16, lens, cfg.n_q_heads)
    _attn_check(out32, want)
    assert torch.equal(out16, out32.to(cfg.torch_dtype))
    if len(lens) > 1:
        assert not out32[1].any()


@pytest.mark.parametrize("B", [64, 65, 130])
@pytest.mark.parametrize("n_splits", [0, 5])
def test_decode_attention_many_ragged_sequences(B, n_splits):
    """Ragged batches at and beyond 64 sequences: up to 64 the grid holds only the splits with tokens (a lane of the
    lookup for each sequence).  Beyond that it does so where a table pays, with two sequences for each lane; otherwise, with a given
    split count and beyond 128, the full (split, head group, sequence) grid runs and the combine pass forms each
    sequence's own split count.  Some sequences are empty."""
    cfg = W.KVConfig(f"many{B}", 500 + B, 1, 2, 4, 64, B, W.F16, 512, 4, 2, W.PER_SEQ, W.BHSD, 0, len_range=(1, 900))
    lens = W.seq_lens(cfg)
    lens[3] = 0
    lens[B - 1] = 0
    lens[B // 2] = 900
    case = Case(cfg, "cuda", gen_device="cpu", lens=lens)
    view = case.make_view(case.k, case.v, lens)
    q = W.query(cfg, 0, "cpu")
    out = torch.full((B, cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
    torch.cuda.synchronize()
    K, V = case.k_cpu[0], case.v_cpu[0]
    want = o.attention(case.source(K), o.u16(K), o.u16(V), o.u16(q), False, lens, cfg.n_q_heads)
    _attn_check(out, want)
    assert not out[3].any() and not out[B - 1].any()


# 32 KV heads: 8 sequences are one workgroup for each compute unit of 256
@pytest.mark.parametrize("H,G,D,B,lo,hi,empty,layout", [
    (32, 1, 128, 9, 1, 1500, 0, W.BHSD),      # just over one workgroup per compute unit, longest first, cut more finely
    (32, 2, 64, 128, 1, 40, 0, W.PAGED),      # whole sequences, written without a second launch; too short for a table to pay
    (32, 2, 64, 129, 1, 40, 0, W.BHSD),       # one sequence more than the table holds
    (16, 3, 128, 100, 20, 700, 3, W.PAGED),   # beyond 64 sequences, some without tokens
    (32, 4, 256, 8, 1, 1200, 1, W.PAGED),
    (32, 1, 64, 31, 300, 1300, 0, W.BHSD),
    (5, 17, 128, 70, 5, 900, 2, W.BHSD),      # two parts of a KV head's query heads: the grid stays in the batch's order
    (8, 4, 128, 128, 20, 250, 0, W.PAGED),    # whole sequences in a table, its last entry, written without a second launch
    (32, 1, 64, 100, 400, 700, 0, W.BHSD),    # beyond 64, one split each, nearly equal: no table, lengths from the device
    (16, 4, 256, 66, 130, 300, 0, W.PAGED),   # the same at head_dim 256
    (1, 4, 64, 65, 513, 600, 0, W.BHSD),      # beyond 64, several splits each without a table, fewer workgroups than compute units
])
@pytest.mark.parametrize("n_splits", [0, 2])
def test_decode_attention_more_workgroups_than_compute_units(H, G, D, B, lo, hi, empty, layout, n_splits):
    """Ragged batches whose workgroups outnumber the compute units, or of more than 64 sequences.  Every sequence and head is checked, so that a split given to the
    wrong sequence, or to none, shows.  Bar: the file's."""
    cfg = W.KVConfig(f"crowd{B}", 1700 + B + D, 1, H, H * G, D, B, W.BF16 if G % 2 else W.F16, 512, 8, 2, W.PER_SEQ, layout, 0, len_range=(lo, hi))
    lens = W.seq_lens(cfg)
    for i in range(empty):
        lens[i * B // 4] = 0
    lens[B - 1] = hi
    case = Case(cfg, "cuda", gen_device="cpu", lens=lens)
    q = W.query(cfg, 0, "cpu")
    out = torch.full((B, H * G, D), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
    torch.cuda.synchronize()
    _attn_check(out, _reference_attention(case, case.k[0], case.v[0], q).float().numpy())


@pytest.mark.parametrize("wide", ["sequence", "head", "token"])
def test_decode_attention_strides_beyond_32_bits(wide):
    """One stride of 2^32 + 3 16-byte vectors, which reaches the kernel in more than 32 bits, the others small: K and V are two places of one
    allocation of 64 GiB.  With the upper bits lost the rows would be read from elsewhere in it, where other values lie."""
    B, H, G, D, S = 2, 2, 4, 128, 2
    far, apart = (1 << 35) + 24, 1 << 20   # elements
    sb, sh, ss = {"sequence": (far, 4 * D, 2 * D), "head": (4 * D, far, 2 * D), "token": (8 * D, 2 * D, far)}[wide]
    cfg = W.KVConfig("far", 77, 1, H, H * G, D, B, W.F16, 512, 4, 2, W.PER_SEQ, W.BHSD, 0, len_range=(S, S))
    plan = kv.kv_layout_plan(1, H, H * G, D, [S] * B, kv.KV_F16, 512, 4, kv.KV_PER_SEQ, 0, kv.KV_UNBOUNDED, 0, kv.KV_UNBOUNDED)
    buf = torch.empty(far + 2 * apart, dtype=torch.float16, device="cuda")
    buf[:2 * apart] = 7.0   # where rows whose stride lost its upper bits would come from
    k, v = (buf[i * apart:i * apart + far + apart].as_strided((B, H, S, D), (sb, sh, ss, 1)) for i in (0, 1))
    cpu = [W.normal_tensor((B, H, S, D), torch.float16, 900 + i) for i in (0, 1)]
    for dst, src in zip((k, v), cpu):
        for b in range(B):
            for h in range(H):
                for t in range(S):
                    dst[b, h, t].copy_(src[b, h, t])
    q = W.query(cfg, 0, "cpu")
    for lens, n_splits in (([S] * B, 0), ([S, 1], 0), ([S, 1], 2)):   # one length for all, lengths from the device, the table's grid
        view = kv.bhsd_view([k], [v], lens, torch.tensor(lens, dtype=torch.int32, device="cuda"))
        out = torch.full((B, H * G, D), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(kv.kv_decode_attn_workspace(plan, n_splits, S), dtype=torch.uint8, device="cuda")
        kv.kv_decode_attn(plan, view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
        torch.cuda.synchronize()
        for b in range(B):
            kd, vd = (x[b, :, :lens[b]].double().repeat_interleave(G, 0) for x in cpu)   # [Hq, S, D]
            p = torch.softmax((q[b].double()[:, None] * kd).sum(-1) / D ** 0.5, -1)
            _attn_check(out[b], (p[:, :, None] * vd).sum(1).numpy())
    del buf, k, v, dst
    torch.cuda.empty_cache()


@pytest.mark.parametrize("row_vecs", [(1 << 24) - 1, 1 << 24])
@pytest.mark.parametrize("D,G", [(64, 2), (128, 1), (128, 16), (256, 4)])
def test_decode_attention_rows_as_far_apart_as_32_bit_offsets_reach(D, G, row_vecs):
    """Token rows of 2^24 - 1 and of 2^24 16-byte vectors: the offsets of a tile's last rows fill 32 bits, and the first stride for which the kernel's loop
    has no offsets.  A whole tile and a tile of one row, the same tokens as in a dense cache.  Bar: the file's."""
    S = 17
    cfg = W.KVConfig("rows", 78, 1, 1, G, D, 1, W.BF16, 512, 8, 2, W.PER_SEQ, W.BHSD, 0, len_range=(S, S))
    plan = kv.kv_layout_plan(1, 1, G, D, [S], kv.KV_BF16, 512, 8, kv.KV_PER_SEQ, 0, kv.KV_UNBOUNDED, 0, kv.KV_UNBOUNDED)
    ss = 8 * row_vecs
    buf = torch.empty((S - 1) * ss + 2 * D, dtype=torch.bfloat16, device="cuda")
    k, v = (buf[i * D:i * D + (S - 1) * ss + D].as_strided((1, 1, S, D), (S * ss, S * ss, ss, 1)) for i in (0, 1))
    cpu = [W.normal_tensor((1, 1, S, D), torch.bfloat16, 950 + i) for i in (0, 1)]
    for dst, src in zip((k, v), cpu):
        for t in range(S):
            dst[0, 0, t].copy_(src[0, 0, t])
    q = W.query(cfg, 0, "cpu")
    view = kv.bhsd_view([k], [v], [S], torch.tensor([S], dtype=torch.int32, device="cuda"))
    out = torch.full((1, G, D), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(plan, 0, S), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(plan, view, 0, q.cuda(), out, kv.KV_OUT_F32, 0, ws)
    torch.cuda.synchronize()
    kd, vd = (x[0].double().repeat_interleave(G, 0) for x in cpu)   # [G, S, D]
    p = torch.softmax((q[0].double()[:, None] * kd).sum(-1) / D ** 0.5, -1)
    _attn_check(out[0], (p[:, :, None] * vd).sum(1).numpy())
    del buf, k, v, dst
    torch.cuda.empty_cache()


@pytest.mark.parametrize("row_vecs", [(1 << 24) - 1, 1 << 24, (1 << 24) + 2])
@pytest.mark.parametrize("D,G,dtype", [(64, 4, torch.float16), (128, 1, torch.bfloat16), (128, 16, torch.float16), (256, 3, torch.bfloat16)])
def test_decode_attention_of_far_rows_is_that_of_a_dense_cache(D, G, dtype, row_vecs):
    """The same tokens in the same steps: the last bits too are those of a dense cache, on both sides of the first stride that takes 64-bit row addresses, for
    one split and two, of whole tiles and of one that is a row short."""
    S, L2 = 95, 79
    plan = kv.kv_layout_plan(1, 1, G, D, [S, L2], kv.KV_F16 if dtype == torch.float16 else kv.KV_BF16, 512, 16, kv.KV_PER_SEQ, 0, kv.KV_UNBOUNDED, 0, kv.KV_UNBOUNDED)
    k, v = (W.normal_tensor((2, 1, S, D), dtype, 970 + i) for i in (0, 1))
    q = W.normal_tensor((2, G, D), dtype, 972).cuda()
    outs = []
    for far in (True, False):
        ss = 8 * row_vecs if far else 4 * D
        buf = torch.empty((S - 1) * ss + 4 * D, dtype=dtype, device="cuda")   # K and V of both sequences side by side in a row
        at = [[buf[(2 * b + i) * D:(2 * b + i) * D + (S - 1) * ss + D].as_strided((S, D), (ss, 1)) for b in (0, 1)] for i in (0, 1)]
        for i, src in enumerate((k, v)):
            for b in (0, 1):
                for t in range(S):
                    at[i][b][t].copy_(src[b, 0, t])
        kk, vv = (buf[i * D:i * D + (S - 1) * ss + 3 * D].as_strided((2, 1, S, D), (2 * D, S * ss, ss, 1)) for i in (0, 1))
        view = kv.bhsd_view([kk], [vv], [S, L2], torch.tensor([S, L2], dtype=torch.int32, device="cuda"))
        for n_splits in (1, 2):
            out = torch.full((2, G, D), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(plan, n_splits, S), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(plan, view, 0, q, out, kv.KV_OUT_F32, n_splits, ws)
            torch.cuda.synchronize()
            outs.append(out.cpu())
        del buf, at, kk, vv, view
        torch.cuda.empty_cache()
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[3])
    for b, n in enumerate((S, L2)):
        p = torch.softmax((q[b].cpu().double() @ k[b, 0, :n].double().T) / D ** 0.5, -1)
        _attn_check(outs[0][b], (p @ v[b, 0, :n].double()).numpy())


# tokens: as many as one workgroup's wavefronts have preassigned (two steps each; above that they claim steps from a counter), and one more
@pytest.mark.parametrize("D,tokens", [(64, 512), (128, 256), (256, 192)])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("odd", [0, 1])
def test_decode_attention_merge(D, tokens, G, odd):
    """The merge of a workgroup's states for every number of copies a query head has among the matrix columns (16, 4, 2, 1), to an aligned
    output and to one that is aligned to its elements only.  Bars: the file's; 16-bit results are the 32-bit ones rounded, up to the
    last place where a repetition of the same sums (in another order) falls to the other side of a rounding boundary."""
    cfg = W.KVConfig("merge", 2300 + D + G, 1, 2, 2 * G, D, 1, W.BF16 if odd else W.F16, 512, 8, 2, W.PER_SEQ, W.BHSD, 0)
    case = Case(cfg, "cuda", gen_device="cpu", lens=[tokens + odd])
    q = W.query(cfg, 0, "cpu")
    n = 2 * G * D
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, 1, tokens + odd), dtype=torch.uint8, device="cuda")
    buf = torch.full((n + 1,), float("nan"), dtype=torch.float32, device="cuda")
    half = torch.full((n + 1,), float("nan"), dtype=cfg.torch_dtype, device="cuda")
    out, out16 = buf[odd:n + odd].view(1, 2 * G, D), half[odd:n + odd].view(1, 2 * G, D)
    kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, 1, ws)
    kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out16, kv.KV_OUT_SAME, 1, ws)
    torch.cuda.synchronize()
    _attn_check(out, _reference_attention(case, case.k[0], case.v[0], q).float().numpy())
    eps = 2.0 ** -7 if odd else 2.0 ** -10   # one unit in the last place is at most this much of the value
    assert ((out16.float() - out).abs() <= eps * out.abs() + 1e-6).all()
    assert torch.isnan(buf[-1 if not odd else 0]) and torch.isnan(half[-1 if not odd else 0])   # nothing past the output


# a round of one wavefront, of two and of four, one split more than each, the weights' window of 64 and what needs several
@pytest.mark.parametrize("n_splits", [2, 8, 9, 16, 17, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("D,G", [(64, 2), (128, 1), (256, 2)])
@pytest.mark.parametrize("ragged", [False, True])
def test_decode_attention_combine_rounds(D, G, n_splits, ragged):
    """Every number of wavefronts and rounds of the combine kernel, with NaNs in the part of the workspace that no split writes (the second
    sequence of the ragged batch has a third of the splits).  Bar: the file's."""
    q_tok = 64 if D >= 128 else 128   # the shortest split
    lens = [n_splits * q_tok - 5, n_splits * q_tok // 3 + 1] if ragged else [n_splits * q_tok - 5]
    cfg = W.KVConfig("combine", 2700 + D + n_splits, 1, 1, G, D, len(lens), W.F16, 512, 8, 2, W.PER_SEQ, W.BHSD, 0)
    case = Case(cfg, "cuda", gen_device="cpu", lens=lens)
    q = W.query(cfg, 0, "cpu")
    out = torch.full((len(lens), G, D), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.full((kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)),), 0xff, dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
    torch.cuda.synchronize()
    _attn_check(out, _reference_attention(case, case.k[0], case.v[0], q).float().numpy())


# ------------------------------------------------------------------------------------------ pipeline
# (span_chunks, depth, copy_streams, d2h_mode, h2d_mode)
@pytest.mark.parametrize("D,G", [(64, 1), (64, 4), (128, 2), (128, 8), (256, 1), (256, 4)])
@pytest.mark.parametrize("paged", [False, True], ids=["bhsd", "paged"])
def test_decode_attention_long_splits_every_head_shape(D, G, paged):
    """Splits long enough that the wavefronts of a workgroup claim steps on demand (more than two rounds of eight),
    for every head width and query-group size the kernel is instantiated for, ragged (per-sequence split table)
    and uniform, automatic and given split counts."""
    H = 2
    for i, lens in enumerate(([5000, 37, 1201], [2100], [777, 777])):
        cfg = W.KVConfig(f"attn_D{D}_G{G}", 900 + 7 * i + D + G, 1, H, H * G, D, len(lens), W.BF16 if (D + G + i) % 2 else W.F16,
                         512, 8, 2, W.PER_SEQ, W.PAGED if paged else W.BHSD, 0, len_range=(1, 2))
        case = Case(cfg, "cuda", lens=list(lens))
        q = W.query(cfg, 0, "cpu")
        want = case.expected_attention(0, q)
        for n_splits in (0, 2):
            out = torch.full((len(lens), H * G, D), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
            torch.cuda.synchronize()
            _attn_check(out, want)


@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("G,bt", [(3, 16), (5, 12), (7, 0), (16, 32), (17, 0)])
def test_decode_attention_head_groups(D, G, bt):
    """Query-head groups that fill the MFMA columns partly, wholly and in two unequal parts, with sequence lengths at
    the edges of a tile, of a step and of a split, split and whole (results written by the partial kernel, to an output
    that is aligned to its elements only).  Bar: products of 16-bit numbers are exact in fp32, sums of up to n of them err by at
    most n 2^-24 of the sum of magnitudes; the usual bar of this file is far above that at these lengths."""
    H, lens = 2, [1, 15, 16, 17, 33, 64, 65, 129]
    cfg = W.KVConfig(f"groups_D{D}_G{G}", 1300 + D + G, 1, H, H * G, D, len(lens), W.BF16 if G % 3 else W.F16, 512, 8, 2, W.PER_SEQ,
                     W.PAGED if bt else W.BHSD, 0, len_range=(1, 2), block_tokens=max(bt, 1))
    case = Case(cfg, "cuda", lens=lens)
    q = W.query(cfg, 0, "cpu")
    want = case.expected_attention(0, q)
    for n_splits in (0, 1, 2):
        flat = torch.full((len(lens) * H * G * D + 1,), float("nan"), dtype=torch.float32, device="cuda")
        out = flat[1:].view(len(lens), H * G, D)
        ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
        kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
        torch.cuda.synchronize()
        _attn_check(out, want)


@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
@pytest.mark.parametrize("n_splits", [1, 3])
def test_decode_attention_infinite_values(dtype, n_splits):
    """An infinite element of V makes its column infinite for the heads of its KV head and leaves every other result as it
    is (a probability is multiplied in parts, some of which are zero); a NaN in V gives NaN in that column."""
    H, G, D, lens = 2, 4, 128, [100, 700]
    cfg = W.KVConfig("inf", 1400, 1, H, H * G, D, len(lens), dtype, 512, 8, 2, W.PER_SEQ, W.BHSD, 0, len_range=(1, 2))
    case = Case(cfg, "cuda", lens=lens)
    q = W.query(cfg, 0, "cpu")
    want = case.expected_attention(0, q)
    v = case.v[0].clone()
    v[0, 0, 7, 5] = float("inf")
    v[1, 1, 650, 70] = -float("inf")
    v[1, 0, 3, 127] = float("nan")
    view = case.make_view(case.k, [v])
    out = torch.zeros((len(lens), H * G, D), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    assert (got[0, :G, 5] == np.inf).all() and (got[1, G:, 70] == -np.inf).all() and np.isnan(got[1, :G, 127]).all()
    rest = np.ones(got.shape, dtype=bool)
    rest[0, :G, 5] = rest[1, G:, 70] = rest[1, :G, 127] = False
    assert np.isfinite(got[rest]).all() and np.abs(got - want)[rest].max() <= ATTN_ATOL


@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
@pytest.mark.parametrize("n_splits", [0, 1, 3])
def test_decode_attention_nan_scores(dtype, n_splits):
    """A NaN in K makes every result of its KV head's query heads NaN, a NaN in q those of its own head; the other heads and
    sequences keep their values.  An empty sequence still reads zeros."""
    H, G, D, lens = 2, 4, 128, [100, 700, 0, 300]
    cfg = W.KVConfig("nan", 1410, 1, H, H * G, D, len(lens), dtype, 512, 8, 2, W.PER_SEQ, W.BHSD, 0, len_range=(1, 2))
    case = Case(cfg, "cuda", lens=lens)
    q = W.query(cfg, 0, "cpu")
    want = case.expected_attention(0, q)
    k, q = case.k[0].clone(), q.clone()
    k[1, 0, 333, 17] = float("nan")
    q[3, 6, 100] = float("nan")
    out = torch.zeros((len(lens), H * G, D), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, case.make_view([k], case.v), 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    hit = np.zeros(got.shape[:2], dtype=bool)
    hit[1, :G] = hit[3, 6] = True
    assert np.isnan(got[hit]).all()
    assert np.isfinite(got[~hit]).all() and np.abs(got - want)[~hit].max() <= ATTN_ATOL and (got[2] == 0).all()


def _reference_attention(case, k, v, q, skip=(), p_bits=None):
    """Attention in float64 from the device tensors as they are (infinities and NaNs included); `skip` holds (sequence, block)
    pairs of a paged source whose tokens are not attended; p_bits keeps that many leading bits of a probability."""
    cfg, out = case.cfg, []
    for b, n in enumerate(case.lens):
        if case.paged:
            ids = case.table_dev[b, :-(-n // cfg.block_tokens)].long().clamp(0, case.n_pool - 1)
            K, V = (t[ids].transpose(0, 1).reshape(cfg.n_kv_heads, -1, cfg.head_dim)[:, :n].double().cpu() for t in (k, v))
        else:
            K, V = (t[b, :, :n].double().cpu() for t in (k, v))
        use = torch.tensor([(b, t // cfg.block_tokens) not in skip if case.paged else True for t in range(n)], dtype=torch.bool)
        K, V = K[:, use], V[:, use]
        qs = q[b].double().view(cfg.n_kv_heads, -1, cfg.head_dim)
        p = torch.softmax(torch.matmul(qs, K.transpose(1, 2).contiguous()) / cfg.head_dim ** 0.5, dim=-1)
        if p_bits is not None:
            mant, e = torch.frexp(p)
            p = torch.ldexp((mant * 2 ** p_bits).floor() / 2 ** p_bits, e)
        out.append(torch.matmul(p, V).reshape(cfg.n_q_heads, cfg.head_dim))
    return torch.stack(out)


@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
@pytest.mark.parametrize("bt", [0, 16, 12])
def test_decode_attention_keeps_32_bit_probabilities(D, dtype, bt):
    """The error against float64, head by head, is that of 32-bit arithmetic: every head width, type, layout, group size class
    (1 to 4, 5 to 8, 9 to 16 heads, two unequal parts), one split and several.  Bar, relative to a head's 2-norm: a score of up to 8 (in log2)
    is rounded to 2^-24 of itself in its sum and in the exponent, 11 units of 2^-24 in the probability, and the probability,
    its products and their sums add a few more; 20 units = 1.2e-6 (0.6e-6 measured), a single element 6 times that.  A probability that
    has lost its last part (kept to 16 bits in bf16, 11 in fp16) misses the bar: checked against the float64 reference."""
    H, lens, bar = 1, [1500, 333, 17], 20 * 2.0 ** -24
    for G in (1, 2, 3, 4, 5, 7, 16, 25):
        cfg = W.KVConfig("precise", 1500 + D + G + bt, 1, H, H * G, D, len(lens), dtype, 512, 8, 2, W.PER_SEQ, W.PAGED if bt else W.BHSD, 0,
                         len_range=(1, 2), block_tokens=max(bt, 1))
        case = Case(cfg, "cuda", lens=lens)
        q = W.query(cfg, 0, "cpu")
        want = _reference_attention(case, case.k[0], case.v[0], q)
        norm = want.norm(dim=-1)
        coarse = _reference_attention(case, case.k[0], case.v[0], q, p_bits=16 if dtype == W.BF16 else 11)
        assert ((coarse - want).norm(dim=-1) / norm).max() > 2 * bar
        for n_splits in (0, 1, 3):
            out = torch.zeros((len(lens), H * G, D), dtype=torch.float32, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
            torch.cuda.synchronize()
            err = out.double().cpu() - want
            assert (err.norm(dim=-1) / norm).max() <= bar, (G, n_splits)
            assert (err.abs().amax(dim=-1) * D ** 0.5 / norm).max() <= 6 * bar, (G, n_splits)


@pytest.mark.parametrize("D,G,dtype", [(64, 1, W.F16), (64, 5, W.BF16), (128, 1, W.BF16), (128, 4, W.F16), (128, 16, W.BF16), (256, 2, W.F16),
                                       (256, 9, W.BF16)])
@pytest.mark.parametrize("bt", [0, 16, 12])
def test_decode_attention_values_that_are_not_finite(D, G, dtype, bt):
    """Infinities and NaNs in V, K and q, at the edges of tiles, of splits and of sequences; a block id outside the pool whose
    stand-in (block 0) is infinite is still not attended.  Elements that are NaN or infinite in float64 are so here, and all others hold
    the file's bar (fp32) or one rounding to the output's type beside it."""
    H, lens = 2, [1, 100, 700, 65, 257]
    cfg = W.KVConfig("not_finite", 1430 + D + G + bt, 1, H, H * G, D, len(lens), dtype, 512, 8, 2, W.PER_SEQ, W.PAGED if bt else W.BHSD, 0,
                     len_range=(1, 2), block_tokens=max(bt, 1))
    case = Case(cfg, "cuda", lens=lens)
    k, v, q = case.k[0].clone(), case.v[0].clone(), W.query(cfg, 0, "cpu").clone()

    def put(t, b, h, tok, d, x):
        if bt:
            t[case.table_dev[b, tok // bt], h, tok % bt, d] = x
        else:
            t[b, h, tok, d] = x
    skip = set()
    if bt:
        bad = next(b for b in (2, 4) if 0 not in case.table_dev[b, 3:4].tolist())
        case.table_dev[bad, 3] = case.n_pool + 5
        skip = {(bad, 3)}
        if 0 not in case.table_dev[2:].flatten().tolist():
            v[0] = float("inf")                       # what an id outside the pool would read
    put(v, 0, 0, 0, 3, -float("inf"))
    put(v, 1, 1, 99, D - 1, float("inf"))
    put(v, 2, 0, 15, 0, float("nan"))
    put(v, 2, 1, 640, 40, float("inf"))
    put(k, 3, 0, 64, 7, float("nan"))
    q[4, 1, 5] = float("inf")                          # scores of either sign: NaN for this head alone
    want = _reference_attention(case, k, v, q, skip)
    view = case.make_view([k], [v])
    for out_mode, dt, rel in ((kv.KV_OUT_F32, torch.float32, 0.0), (kv.KV_OUT_SAME, k.dtype, 2.0 ** -8 if dtype == W.BF16 else 2.0 ** -11)):
        for n_splits in (0, 1, 3):
            out = torch.zeros((len(lens), H * G, D), dtype=dt, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out, out_mode, n_splits, ws)
            torch.cuda.synchronize()
            got = out.double().cpu()
            assert torch.equal(torch.isnan(got), torch.isnan(want)), n_splits
            assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
            fin = torch.isfinite(want)
            assert torch.isfinite(got[fin]).all()
            assert ((got - want).abs()[fin] <= ATTN_ATOL + rel * want.abs()[fin]).all()


@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
def test_decode_attention_scores_beyond_the_exact_range(D, dtype):
    """Scores of 2^30 and more, whose last place is far above 1: the largest score of a sequence takes all the weight, and the result is
    its row of V.  Every score is a whole multiple of a large power of two, exact in fp32, so no other token comes near."""
    H, G, lens = 1, 2, [40 + 13 * i for i in range(12)]
    cfg = W.KVConfig("steep", 1420 + D, 1, H, H * G, D, len(lens), dtype, 512, 8, 2, W.PER_SEQ, W.BHSD, 0, len_range=(1, 2))
    case = Case(cfg, "cuda", lens=lens)
    top = 2.0 ** (13 if dtype == W.F16 else 18)      # K = top (1 + j / 128): exact in both types
    k, q = case.k[0].clone(), W.query(cfg, 0, "cpu").clone()
    q[:] = torch.tensor([top, -top]).view(1, G, 1)   # the second head prefers the smallest key
    best = torch.empty((len(lens), G), dtype=torch.int64)
    for b, n in enumerate(lens):
        j = torch.randperm(n, generator=torch.Generator().manual_seed(b)) * 100 // n
        j[j == j.max()], j[j == j.min()] = 0, 1
        hi, lo = b % n, (7 * b + 5) % n
        j[hi], j[lo] = 101 + b, -1
        k[b, 0, :n] = (top * (1 + j.double() / 128)).to(k.dtype).cuda().view(n, 1)
        best[b] = torch.tensor([hi, lo])
    out = torch.zeros((len(lens), H * G, D), dtype=torch.float32, device="cuda")
    for n_splits in (0, 1, 3):
        ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
        kv.kv_decode_attn(case.plan, case.make_view([k], case.v), 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
        torch.cuda.synchronize()
        for b in range(len(lens)):
            for g in range(G):
                assert torch.equal(out[b, g].cpu(), case.v[0][b, 0, best[b, g]].float().cpu()), (n_splits, b, g)


@pytest.mark.parametrize("bt", [1, 2, 3, 5, 7, 8, 9, 10, 12, 13, 14, 15, 17, 20, 24, 31, 33, 100, 700])
@pytest.mark.parametrize("D,G,dtype", [(64, 4, torch.float16), (128, 1, torch.bfloat16), (128, 9, torch.float16), (256, 2, torch.bfloat16)])
def test_decode_attention_of_blocks_that_tiles_cross(D, G, dtype, bt):
    """Every place of a row in its block, blocks shorter and longer than a tile: the bits of the same tokens in blocks of whole tiles (up to 12 steps a split, which no
    wavefront takes out of turn)."""
    H, lens = 2, [190, 33, 161, 1, 16]
    plan = kv.kv_layout_plan(1, H, H * G, D, lens, kv.KV_F16 if dtype == torch.float16 else kv.KV_BF16, 512, 8, kv.KV_PER_SEQ, 0, kv.KV_UNBOUNDED, 0, kv.KV_UNBOUNDED)
    k, v = (W.normal_tensor((len(lens), H, max(lens), D), dtype, 980 + i) for i in (0, 1))
    q = W.normal_tensor((len(lens), H * G, D), dtype, 982).cuda()
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    outs = []
    for block in (bt, 16):
        per = [-(-n // block) for n in lens]
        ids = np.random.default_rng(5).permutation(sum(per))
        table = np.full((len(lens), max(per)), -1, dtype=np.int32)
        pools = [torch.zeros((sum(per), H, block, D), dtype=dtype) for _ in (0, 1)]
        at = 0
        for b, n in enumerate(lens):
            table[b, :per[b]] = ids[at:at + per[b]]
            at += per[b]
            for pool, src in zip(pools, (k, v)):
                for j in range(per[b]):
                    rows = src[b, :, j * block:min(n, (j + 1) * block)]
                    pool[table[b, j], :, :rows.shape[1]] = rows
        view = kv.paged_view([pools[0].cuda()], [pools[1].cuda()], torch.from_numpy(table).cuda(), lens, lens_dev)
        for n_splits in (1, 0):
            out = torch.full((len(lens), H * G, D), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.empty(kv.kv_decode_attn_workspace(plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
            kv.kv_decode_attn(plan, view, 0, q, out, kv.KV_OUT_F32, n_splits, ws)
            torch.cuda.synchronize()
            outs.append(out.cpu())
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[3])
    for b, n in enumerate(lens):
        kd, vd = (x[b, :, :n].double().repeat_interleave(G, 0) for x in (k, v))
        p = torch.softmax((q[b].cpu().double()[:, None] * kd).sum(-1) / D ** 0.5, -1)
        _attn_check(outs[0][b], (p[:, :, None] * vd).sum(1).numpy())


@pytest.mark.parametrize("bt", [1, 8, 12, 32, 48])
def test_paged_source_other_block_sizes(bt):
    """Paged pools whose blocks hold other than 16 token rows (a power of two below and above the 16-row tile, sizes
    that are not powers of two, one row per block): pack, unpack, decode attention and a pipeline round trip against
    the checker."""
    torch.cuda.set_device(0)
    H, G, D = 2, 4, 128
    lens = [700, 33, 257]
    cfg = W.KVConfig(f"paged_bt{bt}", 4200 + bt, 2, H, H * G, D, len(lens), W.F16 if bt % 2 else W.BF16, 512, 8, 2, W.PER_SEQ,
                     W.PAGED, 0, len_range=(1, 2), block_tokens=bt)
    case = Case(cfg, "cuda", lens=list(lens), raw=True)
    r = case.ref
    nbytes = r.n_blocks_tensor * r.lba_size
    for layer, kind in ((0, 0), (1, 1)):
        buf, dst = _guarded(nbytes)
        kv.kv_offload_pack(case.plan, layer, kind, case.view, kv.KV_SEQ_ALL, 0, 0, dst)
        torch.cuda.synchronize()
        assert np.array_equal(dst.cpu().numpy(), case.expected_extent(layer, kind)) and _guards_intact(buf, nbytes)
    region = pinned_bytes(r.region_bytes, 0x5A)
    arena = np.full(max(r.pageable_bytes, 1), 0x5A, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=2)
    want_region, _ = case.expected_host(fill=0x5A)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    k_new, v_new = case.blank_like_source()
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, cfg.n_layers, case.make_view(k_new, v_new), region, arena, depth=2)
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    # attention on values that are numbers (the raw bit patterns above include NaNs)
    case = Case(cfg, "cuda", lens=list(lens))
    q = W.query(cfg, 0, "cpu")
    want = case.expected_attention(0, q)
    for n_splits in (0, 3):
        out = torch.full((len(lens), H * G, D), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, n_splits, max(lens)), dtype=torch.uint8, device="cuda")
        kv.kv_decode_attn(case.plan, case.view, 0, q.cuda(), out, kv.KV_OUT_F32, n_splits, ws)
        torch.cuda.synchronize()
        _attn_check(out, want)


PIPE_VARIANTS = [(0, 3, 0, kv.KV_COPY_AUTO, kv.KV_COPY_AUTO),
                 (1, 2, 1, kv.KV_COPY_MEMCPY, kv.KV_COPY_MEMCPY),
                 (2, 4, 3, kv.KV_COPY_KERNEL, kv.KV_COPY_KERNEL),
                 (0, 1, 0, kv.KV_COPY_AUTO, kv.KV_COPY_AUTO),
                 (0, 8, 4, kv.KV_COPY_MEMCPY, kv.KV_COPY_KERNEL)]


@pytest.mark.parametrize("span_chunks,depth,copy_streams,d2h,h2d", PIPE_VARIANTS)
def test_pipeline_offload_reload(case, span_chunks, depth, copy_streams, d2h, h2d):
    cfg, r = case.cfg, case.ref
    FILL = 0xC3
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena,
                            depth=depth, span_chunks=span_chunks, copy_streams=copy_streams, d2h_mode=d2h, h2d_mode=h2d)
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    assert st.max_in_flight <= depth and st.n_chunks > 0
    assert st.bytes_direct == r.direct_blocks * r.lba_size and st.bytes_pagecache == r.pageable_bytes
    assert st.lba_seq_breaks == 0        # K then V, layers ascending: one ascending LBA run (Sec. IV-B placement)

    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, cfg.n_layers, view, region, arena,
                            depth=depth, span_chunks=span_chunks, copy_streams=copy_streams, d2h_mode=d2h, h2d_mode=h2d)
    assert st.max_in_flight <= depth
    _check_restored(case, k_new, v_new, range(cfg.n_layers))


@pytest.mark.parametrize("depth", [1, 3])
def test_pipeline_chunk_trace_shows_commands_and_depth_rule(case, depth):
    """The per-command record of a run: the commands are exactly those of Eq. 7-11 for every tensor (and sequence)
    in tensor-id order, as the checker computes them, and the queue-depth rule of Sec. IV-B "Data Flow" holds on the
    issuing thread's clock: command c is issued only after command c - depth was harvested."""
    from oracle import kv_oracle as o
    cfg, r = case.cfg, case.ref
    region = pinned_bytes(r.region_bytes, 0)
    arena = np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)
    nseq = len(case.lens) if r.per_seq else 1
    want = []
    for n in range(2 * cfg.n_layers):
        for b in range(nseq):
            rc, slba, req = o.token_range(r, n, b, 0, r.cap[b])
            assert rc == o.OK
            req = -(-req // r.lba_size) * r.lba_size           # the range reaches the extent tail: padded to a sector
            for c_slba, nlb, _ in o.chunk_cmds(slba, req, cfg.chunk_tokens * r.row_bytes, r.lba_size):
                want.append((n // 2, n % 2, int(r.path[n]), c_slba * r.lba_size, (nlb + 1) * r.lba_size))
    k_new, v_new = case.blank_like_source()
    for direction, view in ((kv.KV_DIR_OFFLOAD, case.view), (kv.KV_DIR_RELOAD, case.make_view(k_new, v_new))):
        st = kv.kv_pipeline_run(case.plan, direction, 0, cfg.n_layers, view, region, arena, depth=depth,
                                trace_cap=len(want) + 8)
        tr = st.trace
        assert st.n_traced == st.n_chunks == len(want)
        # the checker's path codes are 0 direct / 1 page-cache; the library's constants are compared by meaning
        got = [(t.layer, t.kind, 0 if t.path == kv.KV_PATH_DIRECT else 1, t.host_off, t.bytes) for t in tr]
        assert got == want
        for c, t in enumerate(tr):
            assert 0.0 <= t.t_issue_s <= t.t_done_s <= st.wall_s
            if c > 0:
                assert tr[c - 1].t_issue_s <= t.t_issue_s and tr[c - 1].t_done_s <= t.t_done_s   # harvested in issue order
            if c >= depth:
                assert tr[c - depth].t_done_s <= t.t_issue_s
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    # a record shorter than the run keeps the first entries only
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=2, trace_cap=3)
    assert st.n_traced == min(3, st.n_chunks) and [(t.host_off, t.bytes) for t in st.trace] == [w[3:] for w in want[:st.n_traced]]


def test_pipeline_without_issue_pacing(case):
    """KV_PIPE_NO_PACING: every command is queued as soon as the depth rule allows; same bytes either way."""
    cfg, r = case.cfg, case.ref
    FILL = 0x3C
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    want_region, want_arena = case.expected_host(fill=FILL)
    for pacing in (False, True):
        region.fill_(FILL)
        arena[:] = FILL
        st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=3, pacing=pacing)
        assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
        assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
        assert st.max_in_flight <= 3 and st.pace_GBps >= 0.0
        k_new, v_new = case.blank_like_source()
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, cfg.n_layers, case.make_view(k_new, v_new), region, arena,
                           depth=3, pacing=pacing)
        _check_restored(case, k_new, v_new, range(cfg.n_layers))


def test_pipeline_serialized_reference_run(case):
    """The no-overlap reference of the overlap fraction (every stage to completion before the next): same bytes,
    same reload, same attention, one command in flight."""
    cfg, r = case.cfg, case.ref
    FILL = 0x11
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=1, serialize=True)
    assert st.max_in_flight == 1
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    k_new, v_new = case.blank_like_source()
    qd = [W.query(cfg, l, "cpu").cuda() for l in range(cfg.n_layers)]
    outs = [torch.zeros((len(case.lens), cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda")
            for _ in range(cfg.n_layers)]
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, case.make_view(k_new, v_new), region, arena,
                            depth=1, serialize=True, q_layers=qd, out_layers=outs)
    assert st.max_in_flight == 1
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    _attn_check(outs[-1], case.expected_attention(cfg.n_layers - 1, qd[-1].cpu()))


@pytest.mark.parametrize("span_chunks", [0, 1])
def test_pipeline_reload_attention(case, span_chunks):
    cfg, r = case.cfg, case.ref
    region = pinned_bytes(r.region_bytes, 0)
    arena = np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=cfg.depth)
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    qs = [W.query(cfg, l, "cpu") for l in range(cfg.n_layers)]
    qd = [q.cuda() for q in qs]
    outs = [torch.full((len(case.lens), cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")
            for _ in range(cfg.n_layers)]
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, view, region, arena,
                            depth=cfg.depth, q_layers=qd, out_layers=outs, span_chunks=span_chunks, time_kernels=True)
    assert st.kernel_launches[kv.KV_KERNEL_ATTN_PARTIAL] == cfg.n_layers
    for l in range(cfg.n_layers):
        _attn_check(outs[l], case.expected_attention(l, qs[l]))
    _check_restored(case, k_new, v_new, range(cfg.n_layers))


def test_pipeline_reload_attention_from_extent(case):
    """Decode attention fed straight from the staged extent images (no unpack): same outputs, and the
    destination view is neither read nor written."""
    cfg, r = case.cfg, case.ref
    region = pinned_bytes(r.region_bytes, 0)
    arena = np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=cfg.depth)
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    qs = [W.query(cfg, l, "cpu") for l in range(cfg.n_layers)]
    qd = [q.cuda() for q in qs]
    outs = [torch.full((len(case.lens), cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")
            for _ in range(cfg.n_layers)]
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, view, region, arena,
                            depth=cfg.depth, q_layers=qd, out_layers=outs, attn_from_extent=True)
    assert st.kernel_launches[kv.KV_KERNEL_UNPACK] == 0
    assert st.kernel_launches[kv.KV_KERNEL_ATTN_PARTIAL] == cfg.n_layers
    for l in range(cfg.n_layers):
        _attn_check(outs[l], case.expected_attention(l, qs[l]))
        assert (bits(k_new[l]) == 0x7E7E).all() and (bits(v_new[l]) == 0x7E7E).all()
    with pytest.raises(kv.KVError):
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, view, region, arena, depth=cfg.depth,
                           q_layers=qd, out_layers=outs, attn_from_extent=True, span_chunks=1)


@pytest.mark.parametrize("span_chunks,order_pc,order_direct", [(0, kv.KV_ORDER_INTRA, kv.KV_ORDER_INTRA),
                                                              (2, kv.KV_ORDER_INTRA, kv.KV_ORDER_CROSS),
                                                              (0, kv.KV_ORDER_CROSS, kv.KV_ORDER_INTRA)])
def test_pipeline_overlap_orders(case, span_chunks, order_pc, order_direct):
    """Both overlap strategies (K then V, or K and V alternating) move the same bytes; the per-group
    clock runs for every path group that has layers."""
    cfg, r = case.cfg, case.ref
    FILL = 0x3C
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    kw = dict(depth=cfg.depth, span_chunks=span_chunks, order_pagecache=order_pc, order_direct=order_direct)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, **kw)
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    qd = [W.query(cfg, l, "cuda") for l in range(cfg.n_layers)]
    outs = [torch.zeros((len(case.lens), cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda")
            for _ in range(cfg.n_layers)]
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, view, region, arena,
                            q_layers=qd, out_layers=outs, **kw)
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    _attn_check(outs[0], case.expected_attention(0, qd[0].cpu()))
    assert (st.group_seconds[0] > 0) == (r.n1 > 0) and (st.group_seconds[1] > 0) == (r.n1 < r.L)
    assert st.max_in_flight <= cfg.depth
    # alternating K and V commands are two interleaved ascending streams: the single run is broken
    if order_direct == kv.KV_ORDER_INTRA and r.n1 < r.L:
        assert st.lba_seq_breaks > 0
    else:
        assert st.lba_seq_breaks == 0


def test_adaptive_strategy_over_decode_iterations(case):
    """Five decode iterations driven by the selector: orders follow warm-up / intra / cross / chosen, and
    every iteration reloads the same bytes."""
    cfg, r = case.cfg, case.ref
    region = pinned_bytes(r.region_bytes, 0)
    arena = np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=cfg.depth)
    a = kv.kv_adapt_init()
    seen = []
    for it in range(5):
        orders = (kv.kv_adapt_order(a, 0), kv.kv_adapt_order(a, 1))
        seen.append(orders)
        k_new, v_new = case.blank_like_source()
        st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, cfg.n_layers, case.make_view(k_new, v_new), region, arena,
                                depth=cfg.depth, order_pagecache=orders[0], order_direct=orders[1])
        _check_restored(case, k_new, v_new, [0, cfg.n_layers - 1])
        kv.kv_adapt_update(a, st)
    I, C_ = kv.KV_ORDER_INTRA, kv.KV_ORDER_CROSS
    assert seen[:3] == [(I, I), (I, I), (C_, C_)]
    assert seen[3] == seen[4] == (a.chosen[0], a.chosen[1])
    for g in (0, 1):
        want = C_ if a.gbps[g][C_] > a.gbps[g][I] else I
        assert a.chosen[g] == want


def test_pipeline_layer_subrange_and_other_chunk_size(case):
    """Only the requested layers move; a different (aligned) chunk size gives the same bytes."""
    cfg, r = case.cfg, case.ref
    if cfg.n_layers < 3:
        pytest.skip("needs 3 layers")
    FILL = 0x5A
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    sec_rows = max(1, r.lba_size // r.row_bytes)
    C = 3 * sec_rows * 8
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 1, 3, case.view, region, arena, chunk_tokens=C, depth=2)
    want_region, want_arena = case.expected_host(layers=[1, 2], fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    # a chunk larger than any (sub-)extent: one command per tensor (and sequence)
    region2 = pinned_bytes(r.region_bytes, FILL)
    arena2 = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 1, 3, case.view, region2, arena2, chunk_tokens=sec_rows * 100000,
                            depth=8)
    nseq = len(case.lens) if r.per_seq else 1
    assert st.n_chunks == 4 * nseq
    assert np.array_equal(region2.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena2[:r.pageable_bytes], want_arena[:r.pageable_bytes])


@pytest.mark.parametrize("span_chunks,limit_sectors", [(0, 1), (0, 3), (2, 5)])
def test_pipeline_transfer_size_limit(case, span_chunks, limit_sectors):
    """A command-size limit (Eq. 7 on a device's maximum transfer size) splits every chunk into commands of at
    most that many whole sectors: same bytes on the host and back, and the command count of Eq. 8 per chunk."""
    cfg, r = case.cfg, case.ref
    FILL = 0xA7
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    sec = r.lba_size
    limit = limit_sectors * sec + sec // 2          # not a sector multiple: aligned down
    kw = dict(depth=3, span_chunks=span_chunks, max_cmd_bytes=limit)
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, **kw)
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    nseq = len(case.lens) if r.per_seq else 1
    n_cmds = 0
    for layer in range(cfg.n_layers):
        for kind in (0, 1):
            for b in range(nseq):
                for c in kv.kv_plan_chunk_cmds(case.plan, layer, kind, b):
                    n_cmds += -(-(c.nlb + 1) // limit_sectors)
    assert st.n_chunks == n_cmds and st.max_in_flight <= 3
    k_new, v_new = case.blank_like_source()
    st = kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, cfg.n_layers, case.make_view(k_new, v_new), region, arena, **kw)
    assert st.n_chunks == n_cmds
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    with pytest.raises(kv.KVError) as e:
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=3,
                           max_cmd_bytes=sec - 1)
    assert e.value.code == kv.KV_EINVAL


def test_pipeline_argument_errors(case):
    cfg, r = case.cfg, case.ref
    region = pinned_bytes(r.region_bytes, 0)
    arena = np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)

    def code(**kw):
        a = dict(plan=case.plan, direction=kv.KV_DIR_OFFLOAD, layer_begin=0, layer_end=cfg.n_layers, view=case.view,
                 lba_region=region, pageable=arena, depth=2)
        a.update(kw)
        with pytest.raises(kv.KVError) as e:
            kv.kv_pipeline_run(**a)
        return e.value.code

    assert code(depth=0) == kv.KV_EINVAL
    assert code(depth=1025) == kv.KV_EINVAL
    assert code(chunk_tokens=-1) == kv.KV_EINVAL
    assert code(copy_streams=5) == kv.KV_EINVAL
    assert code(d2h_mode=7) == kv.KV_EINVAL and code(h2d_mode=-1) == kv.KV_EINVAL
    assert code(order_pagecache=3) == kv.KV_EINVAL and code(order_direct=-1) == kv.KV_EINVAL
    assert code(host_workers=65) == kv.KV_EINVAL
    assert code(span_chunks=-1) == kv.KV_EINVAL
    assert code(attn_from_extent=True) == kv.KV_EINVAL                      # only with KV_DIR_RELOAD_ATTN
    assert code(direction=9) == kv.KV_EINVAL
    assert code(layer_end=cfg.n_layers + 1) == kv.KV_ERANGE
    assert code(direction=kv.KV_DIR_RELOAD_ATTN) == kv.KV_EINVAL            # no attention arguments
    if r.n1 < r.L:
        assert code(lba_region=region[:r.region_bytes - 1]) == kv.KV_ENOSPC
        unpinned = torch.zeros(r.region_bytes, dtype=torch.uint8)
        assert code(lba_region=unpinned) == kv.KV_EINVAL                     # the LBA region must be pinned
    if r.n1 > 0:
        assert code(pageable=arena[:r.pageable_bytes - 1]) == kv.KV_ENOSPC
    if r.row_bytes % r.lba_size:
        assert code(chunk_tokens=1) == kv.KV_EALIGN


# ------------------------------------------------------------------------------------------ decode append
APPEND_CONFIGS = [
    SMALL[0],                                                    # 256 B rows in 512 B sectors: two rows per sector
    SMALL[5],                                                    # 1920 B rows in 512 B sectors: unaligned, 4-5 sectors
    W.shrink(SMALL[4], seq_len=100, pc_budget_bytes=2 * 103 * 32768),   # 32 KiB rows, 4 KiB sectors: aligned, no merge
    W.shrink(SMALL[3], len_range=(33, 200)),                     # ragged, paged, per-sequence extents, 2 KiB rows
    W.shrink(SMALL[2], seq_len=301, pc_budget_bytes=4 * 304 * 2048),    # both paths, odd length: first append merges
]


@pytest.mark.parametrize("D,H,B", [(64, 1, 1), (64, 3, 2), (128, 16, 1), (128, 17, 1), (256, 8, 1), (256, 9, 2), (128, 5, 7)])
@pytest.mark.parametrize("layout", [W.BHSD, W.PAGED])
@pytest.mark.parametrize("mode", [W.TOKEN_MAJOR, W.PER_SEQ])
def test_pack_unpack_at_the_edges_of_tiles(D, H, B, layout, mode):
    """Extent rows of up to 256 vectors and just above (the line between two launch shapes), rows that no power of two
    divides, lengths around a workgroup's tokens: whole extents of two layers out and back, byte for byte."""
    cfg = W.KVConfig("edges", 1600 + D + H + B, 2, H, H, D, B, W.F16, 512, 8, 2, mode, layout, 33,
                     len_range=(1, 35) if mode == W.PER_SEQ else None)
    case = Case(cfg, "cuda", raw=True, lens=[1, 15, 16, 17, 31, 32, 33][:B] if mode == W.PER_SEQ else [33] * B)
    nbytes = case.ref.n_blocks_tensor * case.ref.lba_size
    buf, dst = _guarded(2 * 2 * nbytes)
    kv.kv_offload_pack_layers(case.plan, 0, 2, case.view, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy().reshape(4, nbytes)
    for n in range(4):
        assert np.array_equal(got[n], case.expected_extent(n // 2, n % 2))
    assert _guards_intact(buf, 4 * nbytes)
    k_new, v_new = case.blank_like_source()
    kv.kv_reload_unpack_layers(case.plan, 0, 2, dst, case.make_view(k_new, v_new))
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, range(2))


# rows of one, two and three 4 KiB pieces, and rows that end inside their second or fourth
@pytest.mark.parametrize("D,H,B", [(128, 16, 3), (128, 32, 3), (64, 96, 2), (256, 24, 1), (64, 33, 4), (256, 25, 2), (128, 47, 1)])
@pytest.mark.parametrize("mode", [W.TOKEN_MAJOR, W.PER_SEQ])
def test_pack_unpack_of_wide_paged_rows(D, H, B, mode):
    """Byte for byte, like the test above: one token's row in pieces, a block id per piece, and whole rows where the pieces do not divide them."""
    test_pack_unpack_at_the_edges_of_tiles(D, H, B, W.PAGED, mode)


@pytest.mark.parametrize("D,H", [(64, 1), (128, 8), (128, 20), (256, 2), (256, 9)])
@pytest.mark.parametrize("layout", [W.BHSD, W.PAGED])
@pytest.mark.parametrize("n_long", [1, 6, 20])
def test_pack_unpack_of_a_batch_with_few_long_sequences(D, H, layout, n_long):
    """Sequences of very different lengths, more than one launch's runs: tiles looked up in one dense grid (1 and 6 long ones) or in
    the grid of the longest run (20).  Whole extents of two layers out and back, pads included, byte for byte."""
    lens = [(900 - 20 * i if i % 2 == 0 and i // 2 < n_long else 1 + i % 9) for i in range(40)]
    cfg = W.KVConfig("skewed", 1800 + D + H, 2, H, H, D, 40, W.F16, 512, 8, 2, W.PER_SEQ, layout, 900, len_range=(1, 2))
    case = Case(cfg, "cuda", raw=True, lens=lens, cap_extra=3)
    nbytes = case.ref.n_blocks_tensor * case.ref.lba_size
    buf, dst = _guarded(2 * 2 * nbytes)
    kv.kv_offload_pack_layers(case.plan, 0, 2, case.view, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy().reshape(4, nbytes)
    for n in range(4):
        assert np.array_equal(got[n], case.expected_extent(n // 2, n % 2))
    assert _guards_intact(buf, 4 * nbytes)
    k_new, v_new = case.blank_like_source()
    kv.kv_reload_unpack_layers(case.plan, 0, 2, dst, case.make_view(k_new, v_new))
    torch.cuda.synchronize()
    _check_restored(case, k_new, v_new, range(2))


@pytest.mark.parametrize("cfg", APPEND_CONFIGS, ids=lambda c: c.name)
def test_decode_append(cfg):
    """Offload len tokens, then append three tokens one by one; after each the host bytes must equal the
    checker's pack of the longer cache.  Only the first append after the offload may read a sector back."""
    EXTRA = 3
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=EXTRA)
    r = case.ref
    FILL = 0x99
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=2)
    lens = list(case.lens)
    row, sec = r.row_bytes, r.lba_size
    for step in range(EXTRA):
        lens = [n + 1 for n in lens]
        view = case.make_view(case.k, case.v, lens)
        st = kv.kv_append_tokens(case.plan, 0, cfg.n_layers, view, region, arena)
        want_region, want_arena = case.expected_host(fill=FILL, lens=lens)
        assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes]), step
        assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes]), step
        nseq = len(lens) if r.per_seq else 1
        assert st.n_cmds == 2 * cfg.n_layers * nseq
        starts_inside = sum(((n - 1) * row) % sec != 0 for n in lens[:nseq])
        assert st.n_rmw_reads == (2 * cfg.n_layers * starts_inside if step == 0 else 0)
    # attention over the longer cache includes the appended tokens
    q = W.query(cfg, 0, "cpu")
    out = torch.empty((len(lens), cfg.n_q_heads, cfg.head_dim), dtype=torch.float32, device="cuda")
    ws = torch.empty(kv.kv_decode_attn_workspace(case.plan, 0, max(lens)), dtype=torch.uint8, device="cuda")
    kv.kv_decode_attn(case.plan, view, 0, q.cuda(), out, kv.KV_OUT_F32, 0, ws)
    torch.cuda.synchronize()
    K, V = case.k_cpu[0], case.v_cpu[0]
    want = o.attention(case.source(K), o.u16(K), o.u16(V), o.u16(q), cfg.dtype == W.BF16, lens, cfg.n_q_heads)
    _attn_check(out, want)
    # the next decode step's reload (storage -> staged extent images -> attention) sees the appended rows too
    k_new, v_new = case.blank_like_source()
    qd = [W.query(cfg, l, "cpu").cuda() for l in range(cfg.n_layers)]
    outs = [torch.zeros_like(out) for _ in range(cfg.n_layers)]
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, case.make_view(k_new, v_new, lens), region, arena,
                       depth=2, q_layers=qd, out_layers=outs, attn_from_extent=True)
    _attn_check(outs[0], want)
    # capacity is a hard bound
    with pytest.raises(kv.KVError) as e:
        kv.kv_append_tokens(case.plan, 0, cfg.n_layers, case.make_view(case.k, case.v, [n + 1 for n in lens]), region, arena)
    assert e.value.code == kv.KV_ERANGE


@pytest.mark.parametrize("layers", [7, 8])
@pytest.mark.parametrize("behind_work", [False, True])
def test_append_merged_by_several_threads(layers, behind_work):
    """Rows of 252 KiB, which the calling thread merges alone, and of 288, which up to four threads merge (each call makes one more): odd lengths and even ones on both
    paths, the sector images of one append read by the next.  behind_work: the rows land after the threads that stood by have given up."""
    cfg = W.KVConfig("append_threads", 2100 + layers, layers, 8, 8, 128, 9, W.F16, 4096, 8, 2, W.PER_SEQ, W.PAGED, 0, len_range=(20, 31),
                     pc_budget_bytes=4 * 2 * 9 * 18 * 4096)
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=5)
    r = case.ref
    region = pinned_bytes(r.region_bytes, 0x77)
    arena = np.full(max(r.pageable_bytes, 1), 0x77, dtype=np.uint8)
    assert 0 < case.plan.info.n_pagecache_layers < layers
    want_region, want_arena = case.expected_host(fill=0x77)
    region.numpy()[:r.region_bytes] = want_region[:r.region_bytes]
    arena[:r.pageable_bytes] = want_arena[:r.pageable_bytes]
    lens = list(case.lens)
    for step in range(5):
        lens = [n + 1 for n in lens]
        if behind_work:
            torch.cuda._sleep(2_000_000)   # about a millisecond
        st = kv.kv_append_tokens(case.plan, 0, layers, case.make_view(case.k, case.v, lens), region, arena)
        want_region, want_arena = case.expected_host(fill=0x77, lens=lens)
        assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes]), step
        assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes]), step
        assert st.n_cmds == 2 * layers * 9 and st.n_rmw_reads == (2 * layers * sum(n % 2 == 0 for n in lens) if step == 0 else 0)


@pytest.mark.parametrize("host_workers", [1, 2, 8])
def test_append_and_pipeline_keep_their_threads(host_workers):
    """Calls in turn, as in a decode loop: after the first ones neither makes a thread or ends one, and the append has at most three, and no more than host_workers."""
    layers = 8
    cfg = W.KVConfig("threads", 2150, layers, 8, 8, 128, 9, W.F16, 4096, 8, 2, W.PER_SEQ, W.PAGED, 0, len_range=(20, 31), pc_budget_bytes=4 * 2 * 9 * 18 * 4096)
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=7)
    r = case.ref
    region, arena = pinned_bytes(r.region_bytes, 0x77), np.zeros(max(r.pageable_bytes, 1), dtype=np.uint8)
    assert 0 < case.plan.info.n_pagecache_layers < layers
    q, outs = [W.query(cfg, l, "cuda") for l in range(layers)], [torch.zeros((9, 8, 128), dtype=torch.float32, device="cuda") for _ in range(layers)]
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, layers, case.view, region, arena, depth=2, host_workers=host_workers)
    threads, lens = [], list(case.lens)
    for step in range(7):
        lens = [n + 1 for n in lens]
        view = case.make_view(case.k, case.v, lens)
        threads.append(set(os.listdir("/proc/self/task")))
        kv.kv_append_tokens(case.plan, 0, layers, view, region, arena)
        threads.append(set(os.listdir("/proc/self/task")))
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, layers, view, region, arena, depth=2, q_layers=q, out_layers=outs, host_workers=host_workers)
    want_region, want_arena = case.expected_host(fill=0x77, lens=lens)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    made = [b - a for a, b in zip(threads[::2], threads[1::2])]   # by each append
    assert sum(map(len, made)) <= min(3, host_workers) and not any(made[3:])
    assert all(t == threads[7] for t in threads[7:])


def test_append_of_a_thread_that_has_one_cpu():
    """No thread helps one that shares its only CPU with them."""
    cfg = W.KVConfig("one_cpu", 2160, 8, 8, 8, 128, 9, W.F16, 4096, 8, 2, W.PER_SEQ, W.PAGED, 0, len_range=(20, 31))
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=3)
    r = case.ref
    region, arena = pinned_bytes(r.region_bytes, 0x77), np.zeros(1, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, 8, case.view, region, arena, depth=2)
    lens, cpus = list(case.lens), os.sched_getaffinity(0)
    os.sched_setaffinity(0, {min(cpus)})
    try:
        for step in range(3):
            lens = [n + 1 for n in lens]
            view = case.make_view(case.k, case.v, lens)
            before = os.listdir("/proc/self/task")
            kv.kv_append_tokens(case.plan, 0, 8, view, region, arena)
            assert os.listdir("/proc/self/task") == before
    finally:
        os.sched_setaffinity(0, cpus)
    assert np.array_equal(region.numpy()[:r.region_bytes], case.expected_host(fill=0x77, lens=lens)[0][:r.region_bytes])


@pytest.mark.parametrize("layers,helped", [(8, False), (16, True)])
def test_append_of_few_wide_rows(layers, helped):
    """16 rows of 20 KiB, which one thread merges before another is awake, and 32."""
    cfg = W.KVConfig("wide_rows", 2170, layers, 8, 8, 64, 20, W.F16, 4096, 8, 2, W.TOKEN_MAJOR, W.PAGED, 30, pc_budget_bytes=0)
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=3)
    r = case.ref
    assert r.row_bytes == 20480
    region, arena = pinned_bytes(r.region_bytes, 0x77), np.zeros(1, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, layers, case.view, region, arena, depth=2)
    lens = list(case.lens)
    for step in range(3):
        lens = [n + 1 for n in lens]
        view = case.make_view(case.k, case.v, lens)
        before = set(os.listdir("/proc/self/task"))
        kv.kv_append_tokens(case.plan, 0, layers, view, region, arena)
        assert len(set(os.listdir("/proc/self/task")) - before) == int(helped)
    assert np.array_equal(region.numpy()[:r.region_bytes], case.expected_host(fill=0x77, lens=lens)[0][:r.region_bytes])


@pytest.mark.parametrize("H,D,layers", [(2, 128, 4), (3, 128, 4), (3, 64, 80)])
def test_append_of_a_length_that_moves_by_more_than_one(H, D, layers):
    """Rows of 512, 768 and 384 bytes in sectors of 4 KiB (one thread; 270 KiB of rows: several).  A length that skips rows of a sector, skips into the next one or goes
    back: rows of a kept sector that no append has written are zeros, whatever an earlier sector or a longer length had in their place; the rest is as for any append."""
    cfg = W.KVConfig("append_skips", 2200 + H + D, layers, H, H, D, 9, W.F16, 4096, 32, 2, W.PER_SEQ, W.PAGED, 0, len_range=(14, 30),
                     pc_budget_bytes=layers // 2 * 2 * 9 * 12 * 4096)
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=48)
    r, nseq, sec, rb = case.ref, 9, 4096, 2 * H * D
    region = pinned_bytes(r.region_bytes, 0x77)
    arena = np.full(max(r.pageable_bytes, 1), 0x77, dtype=np.uint8)
    host = [region.numpy().copy(), arena.copy()]   # direct path, page-cache path
    rows = [case.expected_extent(n // 2, n % 2, lens=case.caps) for n in range(2 * layers)]
    kept = {}
    lens = list(case.lens)
    for step, move in enumerate([1] * 9 + [2, 1, 3, 1, 1, 2, -1, 2, 1, -2, 1, 5, 9, 1, 2, 1]):
        lens = [n + move + (b % 3 == 1 and move > 1) for b, n in enumerate(lens)]
        st = kv.kv_append_tokens(case.plan, 0, layers, case.make_view(case.k, case.v, lens), region, arena)
        reads = 0
        for n in range(2 * layers):
            buf, base = host[int(r.path[n] != 0)], r.ext_byte_off(n)
            for b, ln in enumerate(lens):
                a = (ln - 1) * rb
                first, end = a // sec * sec, -(-(a + rb) // sec) * sec
                off, head = base + int(r.seq_base[b]) * sec, a % sec
                sector, img = kept.get((n, b), (-1, None))
                if head and sector == first:
                    buf[off + first:off + a] = img[:head]
                reads += bool(head and sector != first)
                buf[off + a:off + a + rb] = rows[n][int(r.seq_base[b]) * sec + a:][:rb]
                buf[off + a + rb:off + end] = 0
                kept[n, b] = (end - sec, buf[off + end - sec:off + end].copy()) if (a + rb) % sec else (-1, None)
        assert np.array_equal(region.numpy()[:r.region_bytes], host[0][:r.region_bytes]), (step, lens)
        assert np.array_equal(arena[:r.pageable_bytes], host[1][:r.pageable_bytes]), (step, lens)
        assert st.n_rmw_reads == reads, step


@pytest.mark.parametrize("layout,mode,B", [(W.PAGED, W.PER_SEQ, 130), (W.BHSD, W.PER_SEQ, 128), (W.BHSD, W.TOKEN_MAJOR, 40)])
def test_append_more_rows_than_one_launch_holds(layout, mode, B):
    """The rows of 33 layers and up to 130 sequences (a launch holds 32 layers and 128 sequences), and rows of all
    sequences together that are wider than a workgroup: offload without the newest row, append it, compare the extents."""
    cfg = W.KVConfig("append_many", 1500 + B, 33, 1, 1, 64, B, W.BF16, 512, 8, 2, mode, layout, 9,
                     len_range=(1, 9) if mode == W.PER_SEQ else None)
    case = Case(cfg, "cuda", raw=True)
    r = case.ref
    region = pinned_bytes(r.region_bytes, 0x5A)
    arena = np.full(max(r.pageable_bytes, 1), 0x5A, dtype=np.uint8)
    before = case.make_view(case.k, case.v, [n - 1 for n in case.lens])
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, before, region, arena, depth=2)
    st = kv.kv_append_tokens(case.plan, 0, cfg.n_layers, case.view, region, arena)
    assert st.n_cmds == cfg.n_layers * 2 * (B if mode == W.PER_SEQ else 1)
    want_region, _ = case.expected_host(fill=0x5A)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])


def test_append_after_trim_and_after_a_change_of_region():
    """The kept tail-sector image must not outlive the bytes it mirrors: after kv_plan_trim the sector reads zeros,
    and another region buffer holds whatever it holds.  offload, append, trim, append / append into a copy."""
    cfg = APPEND_CONFIGS[0]
    case = Case(cfg, "cuda", gen_device="cpu", cap_extra=2)
    r, L = case.ref, cfg.n_layers
    FILL = 0x99
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, L, case.view, region, arena, depth=2)
    lens1 = [n + 1 for n in case.lens]
    st = kv.kv_append_tokens(case.plan, 0, L, case.make_view(case.k, case.v, lens1), region, arena)
    assert (((lens1[0] - 1) * r.row_bytes) % r.lba_size != 0) == (st.n_rmw_reads > 0)
    # a second region with the same bytes: the images were taken from `region`, so the library reads this one back
    region2 = pinned_bytes(r.region_bytes, FILL)
    region2.copy_(region)
    arena2 = arena.copy()
    lens2 = [n + 1 for n in lens1]
    kv.kv_append_tokens(case.plan, 0, L, case.make_view(case.k, case.v, lens2), region2, arena2)
    want_region, want_arena = case.expected_host(fill=FILL, lens=lens2)
    assert np.array_equal(region2.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena2[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    # trim: every extent reads zeros; the next append merges with zeros, not with the rows written before
    kv.kv_plan_trim(case.plan, 0, L, region2, arena2)
    kv.kv_append_tokens(case.plan, 0, L, case.make_view(case.k, case.v, lens2), region2, arena2)
    got_region, got_arena = region2.numpy(), arena2
    row, sec = r.row_bytes, r.lba_size
    nseq = len(lens2) if r.per_seq else 1
    for n in range(2 * L):
        buf = got_region if r.path[n] == 0 else got_arena
        ext = buf[r.ext_byte_off(n):r.ext_byte_off(n) + r.n_blocks_tensor * sec]
        want = np.zeros_like(ext)
        full = case.expected_extent(n // 2, n % 2, lens=lens2)
        for b in range(nseq):                      # only the appended row of each (sub-)extent is non-zero
            base = int(r.seq_base[b]) * sec if r.per_seq else 0
            a = base + (lens2[b] - 1) * row
            want[a:a + row] = full[a:a + row]
        assert np.array_equal(ext, want), n


def test_pipeline_waits_for_the_callers_stream():
    """KV written by kernels on a side stream, offloaded without any device-wide synchronisation: the library's
    streams must be ordered after the caller's stream (kv_pipe_opts_t.caller_stream), so the host bytes are the
    checker's pack of the final values, not of what the buffers held before."""
    cfg = W.shrink(W.CONFIGS[1], n_layers=2, seq_len=2048)
    case = Case(cfg, "cuda", gen_device="cpu")
    r, L = case.ref, cfg.n_layers
    FILL = 0x42
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    final_k = [t.clone() for t in case.k]
    final_v = [t.clone() for t in case.v]
    for t in case.k + case.v:
        t.zero_()                                   # what a racing pack would pick up
    big = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(200):                        # tens of milliseconds of queued work ahead of the writes
            big.add_(1)
        for dst, src in zip(case.k + case.v, final_k + final_v):
            dst.copy_(src)
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, L, case.view, region, arena, depth=3)
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    # reload into buffers that a kernel on the side stream is still filling: the unpack must come after it
    k_new, v_new = case.blank_like_source()
    with torch.cuda.stream(side):
        for _ in range(200):
            big.add_(1)
        for t in k_new + v_new:
            t.fill_(1.0)
        kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, L, case.make_view(k_new, v_new), region, arena, depth=3)
    for l in range(L):
        assert np.array_equal(bits(k_new[l]), bits(case.k_cpu[l])) and np.array_equal(bits(v_new[l]), bits(case.v_cpu[l]))


def test_many_sequences_span_several_launches():
    """70 ragged per-sequence sub-extents per tensor: the pack / unpack segment table holds 32 runs, so one tensor
    takes several launches; the append packs 140 rows.  Host bytes, round trip and append against the checker."""
    B, EXTRA = 70, 1
    cfg = W.KVConfig("many_segments", 777, 1, 2, 4, 64, B, W.BF16, 512, 4, 3, W.PER_SEQ, W.BHSD, 0, len_range=(1, 300))
    lens = W.seq_lens(cfg)
    lens[5] = 0
    case = Case(cfg, "cuda", gen_device="cpu", lens=lens, cap_extra=EXTRA)
    r = case.ref
    FILL = 0x6D
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, 1, case.view, region, arena, depth=3)
    want_region, _ = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    k_new, v_new = case.blank_like_source()
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD, 0, 1, case.make_view(k_new, v_new), region, arena, depth=3)
    _check_restored(case, k_new, v_new, [0])
    # attention straight from the staged image: 70 per-sequence base offsets, ragged lengths (full grid: B > 64)
    q = W.query(cfg, 0, "cpu")
    out = [torch.full((B, cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")]
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, 1, case.make_view(k_new, v_new), region, arena, depth=3,
                       q_layers=[q.cuda()], out_layers=out, attn_from_extent=True)
    _attn_check(out[0], case.expected_attention(0, q))
    longer = [n + 1 for n in lens]
    st = kv.kv_append_tokens(case.plan, 0, 1, case.make_view(case.k, case.v, longer), region, arena)
    assert st.n_cmds == 2 * B
    want_region, _ = case.expected_host(fill=FILL, lens=longer)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])


# ------------------------------------------------------------------------------------------ random shapes
def _random_configs(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        D = int(rng.choice([64, 128, 256]))
        H = int(rng.integers(1, 7))
        G = int(rng.choice([1, 2, 3, 4, 8]))
        B = int(rng.integers(1, 5))
        sector = int(rng.choice([512, 4096]))
        per_seq = bool(rng.integers(0, 2))
        paged = bool(rng.integers(0, 2))
        row = (H if per_seq else B * H) * D * 2
        unit = sector // np.gcd(sector, row)                   # fewest rows that end on a sector boundary
        chunk = int(unit * rng.integers(1, 6))
        dtype = W.F16 if rng.integers(0, 2) else W.BF16
        if per_seq:
            lo = int(rng.integers(1, 40))
            cfg = W.KVConfig(f"rand{i}", 100 + i, 2, H, H * G, D, B, dtype, sector, chunk, int(rng.integers(1, 5)),
                             W.PER_SEQ, W.PAGED if paged else W.BHSD, 0, len_range=(lo, lo + int(rng.integers(0, 300))))
        else:
            cfg = W.KVConfig(f"rand{i}", 100 + i, 2, H, H * G, D, B, dtype, sector, chunk, int(rng.integers(1, 5)),
                             W.TOKEN_MAJOR, W.PAGED if paged else W.BHSD, int(rng.integers(1, 400)))
        # one of the two layers on the page-cache path in half of the cases
        if rng.integers(0, 2):
            lens = W.seq_lens(cfg)
            nb = o.tensor_blocks(per_seq, lens, H, D, 2, sector)[0]
            cfg = W.shrink(cfg, pc_budget_bytes=2 * nb * sector)
        out.append(cfg)
    return out


@pytest.mark.parametrize("cfg", _random_configs(24, 2024), ids=lambda c: c.name)
def test_random_shapes_end_to_end(cfg):
    """Seeded random shapes (head counts, group sizes, head dims, batch, sector, chunk, both extent modes,
    both layouts, mixed paths): offload bytes, round trip and attention against the checker."""
    case = Case(cfg, "cuda", gen_device="cpu", raw=False)
    r = case.ref
    FILL = 0x42
    region = pinned_bytes(r.region_bytes, FILL)
    arena = np.full(max(r.pageable_bytes, 1), FILL, dtype=np.uint8)
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_OFFLOAD, 0, cfg.n_layers, case.view, region, arena, depth=cfg.depth,
                       span_chunks=cfg.index % 3)
    want_region, want_arena = case.expected_host(fill=FILL)
    assert np.array_equal(region.numpy()[:r.region_bytes], want_region[:r.region_bytes])
    assert np.array_equal(arena[:r.pageable_bytes], want_arena[:r.pageable_bytes])
    k_new, v_new = case.blank_like_source()
    view = case.make_view(k_new, v_new)
    qs = [W.query(cfg, l, "cpu") for l in range(cfg.n_layers)]
    qd = [q.cuda() for q in qs]
    outs = [torch.full((len(case.lens), cfg.n_q_heads, cfg.head_dim), float("nan"), dtype=torch.float32, device="cuda")
            for _ in range(cfg.n_layers)]
    kv.kv_pipeline_run(case.plan, kv.KV_DIR_RELOAD_ATTN, 0, cfg.n_layers, view, region, arena, depth=cfg.depth,
                       q_layers=qd, out_layers=outs, span_chunks=(cfg.index + 1) % 3,
                       order_pagecache=cfg.index % 2, order_direct=(cfg.index // 2) % 2)
    _check_restored(case, k_new, v_new, range(cfg.n_layers))
    for l in range(cfg.n_layers):
        _attn_check(outs[l], case.expected_attention(l, qs[l]))
