"""A float64 matrix product's result may be read 19 wait states after its
``v_mfma_f64_16x16x4_f64`` (the count that the compiler keeps on gfx950 in
straight-line code); earlier reads return old values without an error.  The
compiler was seen to read one too early where a block ends in a branch, so the
float64 convolution waits by itself.

This test compiles the kernels to gfx950 assembly on the CPU and checks, with a
forward dataflow pass over the basic blocks of every instance, that no other
instruction touches a result earlier.  A product that accumulates onto the same
registers may follow at once.  Every instruction counts as one wait state and
``s_nop n`` as n + 1, as the compiler counts them.
"""
import re
import subprocess

import pytest

from paper_1905_05233_amd import build_native as B
from test_lds_waits import _blocks

WAIT = 19
INSTANCES = 3 * 2 * 3 * 2   # storage types, kernel heights, block shapes, load forms


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    B.generate_builtin_plans()
    out = tmp_path_factory.mktemp("f64") / "layer_ops.s"
    r = subprocess.run([B.HIPCC] + B.COMMON + B.DEVICE + ["--cuda-device-only", "-S", f"{B.CSRC}/layer_ops.hip", "-o",
                                                          str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def _regs(operands):
    regs = {(f, int(n)) for f, n in re.findall(r"\b([va])(\d+)\b", operands)}
    for f, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", operands):
        regs |= {(f, n) for n in range(int(lo), int(hi) + 1)}
    return regs


def _early(code):
    """Instructions of one kernel that touch a product's result too early."""
    blocks = _blocks(code)
    index = {label: k for k, (label, _) in enumerate(blocks)}
    entry = [{} for _ in blocks]   # register -> wait states still due
    work, hits = list(range(len(blocks))), set()
    while work:
        k = work.pop(0)
        due = dict(entry[k])
        last = ""
        for ins in blocks[k][1]:
            last = ins
            if ins.startswith("."):
                continue
            op, _, operands = ins.partition(" ")
            m = re.match(r"v_mfma_f64_16x16x4_f64 (\S+), (\S+), (\S+), (\S+)$", ins)
            if m:
                d, a, b, c = m.groups()
                used = _regs(f"{a} {b}") | (set() if c == d else _regs(f"{c} {d}"))
            else:
                used = _regs(operands)
            if any(due.get(r, 0) > 0 for r in used):
                hits.add(ins)
            n = int(operands) + 1 if op == "s_nop" else 1
            due = {r: v - n for r, v in due.items() if v > n}
            if m:
                due.update(dict.fromkeys(_regs(d), WAIT))
        succ = []
        m = re.match(r"^s_c?branch\w*\s+(\.LBB\w+)", last)
        if m:
            succ.append(index[m.group(1)])
        if not last.startswith(("s_branch", "s_endpgm", "s_setpc")) and k + 1 < len(blocks):
            succ.append(k + 1)
        for j in succ:
            new = {r: max(v, entry[j].get(r, 0)) for r, v in due.items()}
            if any(entry[j].get(r, 0) < v for r, v in new.items()):
                entry[j].update(new)
                work.append(j)
    return hits


def _kernels(asm):
    parts = re.split(r"\n(_Z\S+):[^\n]*\n", asm[:asm.index("amdhsa.kernels")])
    return {n: c for n, c in zip(parts[1::2], parts[2::2]) if "direct_f64_mfma_kernel" in n}


def test_every_instance_waits_for_its_products(asm):
    kernels = _kernels(asm)
    assert len(kernels) == INSTANCES
    assert all("v_mfma_f64_16x16x4_f64" in c for c in kernels.values())
    early = {n: sorted(h) for n, c in kernels.items() if (h := _early(c))}
    assert not early, early


def test_a_missing_wait_is_seen(asm):
    """With the nops taken out of the text the products' results are read too early."""
    code = next(iter(_kernels(asm).values()))
    assert not _early(code)
    assert _early(re.sub(r"\n\s*s_nop \d+", "", code))
