"""The machine code made from the attention kernels (no GPU): no matrix product adds to the result of a product of another shape.
Such a pair has read part of the earlier result too early, and an error in a low-order term could pass for rounding."""
import os
import re
import subprocess

from paper_2604_26557_amd import build

MFMA = re.compile(r"v_mfma_f32_(16x16x\d+)\S*\s+(\S+), (\S+), (\S+), ([^\s;]+)")


def _regs(op):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", op) or re.fullmatch(r"([va])(\d+)", op)
    if not m:
        return []
    lo, hi = int(m[2]), int(m[m.lastindex])
    return [(m[1], r) for r in range(lo, hi + 1)]


def mixed_pairs(asm):
    """(kernel, earlier shape, later shape) of every product whose accumulator was last written, in program order, by a product of
    another shape; and how many products there are."""
    kernel, writer, found, n = None, {}, [], 0
    for line in asm.splitlines():
        label = re.match(r"(_Z\w+):", line)
        if label:
            kernel, writer = label[1], {}
        t = line.strip()
        m = MFMA.match(t)
        if m:
            n += 1
            found += [(kernel, writer[r], m[1]) for r in _regs(m[5])[:1] if writer.get(r, m[1]) != m[1]]
            writer.update((r, m[1]) for r in _regs(m[2]))
        elif re.match(r"(v_|global_load|ds_read|scratch_load)", t):
            for r in _regs(t.split()[1].rstrip(",")) if len(t.split()) > 1 else []:
                writer.pop(r, None)
    return found, n


def test_the_scan_finds_a_mixed_pair():
    a, b = "v_mfma_f32_16x16x16_bf16 v[0:3], v[8:9], v[10:11], 0\n", "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[0:3]\n"
    assert mixed_pairs("_Zk:\n" + a + "v_add_f32_e32 v20, v21, v22\n" + b)[0] == [("_Zk", "16x16x16", "16x16x32")]
    assert mixed_pairs("_Zk:\n" + a + "v_mov_b32_e32 v0, 0\n" + b)[0] == [] and mixed_pairs("_Zk:\n" + b + b.replace("v[0:3]", "v[4:7]"))[0] == []


def test_products_that_share_an_accumulator_are_of_one_shape(tmp_path):
    out = str(tmp_path / "attn.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.check_call([build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attn_kernels.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    with open(out) as f:
        found, n = mixed_pairs(f.read())
    assert n > 1000 and found == []
