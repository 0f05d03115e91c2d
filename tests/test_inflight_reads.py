"""LDS reads issued in inline asm, in the built code: none is outstanding where
control flow branches or joins.  The compiler takes an asm block's output as
written at once and may copy or reuse the register there, before the data has
arrived; the tiled GEMM and the prefill attention wait for their reads first.
Only the main loops are looked at (up to a kernel's last matrix instruction):
the epilogues' reads are the compiler's own.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_13076_amd import spade

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(r"^[0-9a-f]+ <(.*(?:gemm_tile_kernel|attn_prefill_kernel).*)>:$")
LABEL = re.compile(r"^[0-9a-f]+ <L\d+>:$")
WAIT = re.compile(r"lgkmcnt\((\d+)\)")


def _crossings(lines):
    """(line, reads outstanding) at each branch or join of one kernel."""
    last = max((i for i, l in enumerate(lines) if "v_mfma" in l), default=-1)
    reads, found = 0, []
    for i, l in enumerate(lines[:last + 1]):
        op = l.split(None, 1)[0] if l.strip() else ""
        if op == "ds_read_b128":
            reads += 1
        elif op == "s_waitcnt":
            w = WAIT.search(l)
            reads = min(reads, int(w.group(1))) if w else reads
        elif reads and (op.startswith(("s_cbranch", "s_branch")) or LABEL.match(l)):
            found.append((i, l.strip(), reads))
    return found


def test_walk_sees_an_outstanding_read():
    loop = ["ds_read_b128 v[0:3], v9", "000000 <L1>:", "s_waitcnt lgkmcnt(0)", "v_mfma_f32_16x16x32_bf16 a"]
    assert _crossings(loop) == [(1, "000000 <L1>:", 1)]
    assert _crossings([loop[0], loop[2], loop[1], loop[3]]) == []


def test_no_read_in_flight_at_a_branch_or_join(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(spade.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    kernels = {}
    for f in sorted(tmp_path.glob("lib.so.*amdgcn*")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(f)], check=True,
                              capture_output=True, text=True).stdout
        cur = None
        for l in text.splitlines():
            k = KERNEL.match(l)
            if k:
                cur = kernels.setdefault(k.group(1), [])
            elif re.match(r"^[0-9a-f]+ <(?!L\d+>)", l):
                cur = None
            elif cur is not None:
                cur.append(l.strip())
    tile = [k for k in kernels if "gemm_tile_kernel" in k]
    assert len(tile) >= 100 and any("attn_prefill" in k for k in kernels), len(tile)
    assert all(any("ds_read_b128" in l for l in ls) for ls in kernels.values())
    bad = {k: _crossings(ls) for k, ls in kernels.items()}
    bad = {k: v for k, v in bad.items() if v}
    assert not bad, (len(bad), next(iter(bad.items())))
