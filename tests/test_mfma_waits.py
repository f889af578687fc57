"""Every wait after a matrix instruction, read from the built library's own assembly.

The result of an MFMA is not interlocked against vector instructions: until it is written, a
read gives what the registers held before.  The compiler puts the waits in, and within straight
code it does so everywhere; where a product is used behind a branch it left some out (a walk
whose last block ended after three of four groups then added, in some runs, a stale group).
So the kernels keep a product and its first use on one side of every branch, and this test
follows all paths of all kernels.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2604_21026_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# Wait states from issue to the first use of the result: passes of four cycles, and four more
# (what the compiler inserts in straight code: s_nop 7 after a 16x16x32).
WAITS = {"16x16x32": 8, "32x32x16": 12}


def _registers(text):
    regs = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        regs |= {kind + str(r) for r in range(int(lo), int(hi) + 1)}
    return regs | {k + r for k, r in re.findall(r"\b([va])(\d+)\b", text)}


def early_uses(code):
    """code: list of (address, text, branch target or None).  Returns (address, register, states)
    of each use of an MFMA result too soon after it, over all paths; an MFMA that takes it as
    its accumulator is ordered by the hardware and the compiler's own rule and is not a use."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    parsed = []
    for _, text, target in code:
        op, _, args = text.partition(" ")
        shape = re.match(r"v_mfma_[a-z0-9]+_(\d+x\d+x\d+)", op)
        if shape:
            d, a, b = re.split(r",\s*(?![^\[]*\])", args)[:3]
            parsed.append((_registers(a) | _registers(b), _registers(d), WAITS[shape.group(1)], 1, op, target))
        else:
            used = set() if op.startswith("s_") else _registers(args)
            states = int(args.split()[0], 0) + 1 if op == "s_nop" else 1
            parsed.append((used, set(), 0, states, op, target))
    seen = [None] * len(code)  # per instruction: register -> wait states still missing
    found = {}
    work = [(0, {})]
    while work:
        i, missing = work.pop()
        while i < len(code):
            if seen[i] is not None:
                merged = dict(seen[i])
                for r, n in missing.items():
                    merged[r] = max(n, merged.get(r, 0))
                if merged == seen[i]:
                    break
                missing = merged
            seen[i] = missing
            used, written, wait, states, op, target = parsed[i]
            if missing:
                for r in used & missing.keys():
                    found[(code[i][0], r)] = missing[r]
                missing = {r: n - states for r, n in missing.items() if n > states}
            if written:
                missing = {**missing, **{r: wait for r in written}}
            if op == "s_endpgm":
                break
            if target is not None:
                if op == "s_branch":
                    i = at[target]
                    continue
                work.append((at[target], missing))
            i += 1
    return [(a, r, n) for (a, r), n in sorted(found.items())]


def kernels(lib, folder):
    """(name, code) of every kernel of the library that holds a matrix instruction."""
    shutil.copy(lib, os.path.join(folder, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=folder, check=True, capture_output=True)
    for f in sorted(os.listdir(folder)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", f], cwd=folder, check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            name = re.match(r"[0-9a-f]+ <(.*)>:", part)
            if not name or "v_mfma" not in part:
                continue
            code = []
            for line in part.splitlines()[1:]:
                m = re.match(r"\s+([a-z]\S*.*?)\s*// ([0-9A-F]+): ([0-9A-F]+)", line)
                if not m:
                    continue
                addr, target = int(m.group(2), 16), None
                if re.match(r"s_c?branch", m.group(1)):
                    off = int(m.group(3), 16) & 0xFFFF
                    target = addr + 4 + 4 * (off - 0x10000 if off & 0x8000 else off)
                code.append((addr, m.group(1), target))
            yield name.group(1), code


def test_a_missing_wait_is_found():
    product = "v_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[8:11], v[4:7]"
    straight = [(0, product, None), (8, "s_nop 7", None), (12, "v_add_f32_e32 v4, v4, v4", None), (16, "s_endpgm", None)]
    assert early_uses(straight) == []
    short = [(0, product, None), (8, "s_nop 6", None), (12, "v_add_f32_e32 v4, v4, v4", None), (16, "s_endpgm", None)]
    assert early_uses(short) == [(12, "v4", 1)]
    # the way round the wait: by the branch only one wait state lies between
    branch = [(0, product, None), (8, "s_cbranch_scc1 2", 20), (12, "s_nop 7", None),
              (16, "s_nop 0", None), (20, "v_add_f32_e32 v4, v4, v7", None), (24, "s_endpgm", None)]
    assert early_uses(branch) == [(20, "v4", 7), (20, "v7", 7)]
    # a loop back to a use that stands before the product
    loop = [(0, "v_add_f32_e32 v9, v9, v5", None), (4, product, None), (12, "s_cbranch_scc1 65532", 0), (16, "s_endpgm", None)]
    assert early_uses(loop) == [(0, "v5", 7)]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_kernel_uses_a_product_before_it_is_written(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    names, bad = [], []
    for name, code in kernels(build.LIB, str(tmp_path)):
        names.append(name)
        uses = early_uses(code)
        if uses:
            bad.append("%s: %d, first at %x: %s, %d states short" % ((name, len(uses)) + uses[0]))
    for kernel in ("gemv_slice", "gemv_rows", "gemv_mfma_ring", "gemm_w4a16"):
        assert any(kernel in n for n in names), kernel
    assert not bad, "\n".join(bad)
