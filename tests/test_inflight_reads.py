"""LDS reads issued in inline asm, in the built code: none is outstanding where
control flow branches or joins, and no instruction touches a read's registers
before a wait that covers it.  The compiler takes an asm block's output as
written at once and may copy or reuse the register before the data has arrived;
the wide-row and tiled GEMMs and the prefill attention wait for their reads
first.  Only the main loops are looked at (up to a kernel's last matrix
instruction): the epilogues' reads are the compiler's own.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_13076_amd import spade

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(r"^[0-9a-f]+ <(.*(?:gemm_wide_kernel|gemm_tile_kernel|attn_prefill_kernel).*)>:$")
LABEL = re.compile(r"^[0-9a-f]+ <L\d+>:$")
WAIT = re.compile(r"lgkmcnt\((\d+)\)")
REG = re.compile(r"\bv(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for one, lo, hi in REG.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def _crossings(lines):
    """Lines of one kernel at which a 16-byte LDS read is outstanding that must not be."""
    last = max((i for i, l in enumerate(lines) if "v_mfma" in l), default=-1)
    flying, found = [], []  # registers of the LDS operations in flight, oldest first (None: not a 16-byte read)
    for i, l in enumerate(lines[:last + 1]):
        l = l.split("//")[0].strip()
        op, _, args = l.partition(" ")
        if op == "s_waitcnt":
            w = WAIT.search(args)
            if w:
                flying = flying[max(0, len(flying) - int(w.group(1))):]
            continue
        busy = [r for r in flying if r]
        if busy and (op.startswith(("s_cbranch", "s_branch")) or LABEL.match(l)):
            found.append((i, l))
        elif busy and any(r & _regs(args) for r in busy):
            found.append((i, l))
        if op.startswith("ds_"):
            flying.append(_regs(args.split(",")[0]) if op == "ds_read_b128" else None)
    return found


def test_walk_sees_an_outstanding_read():
    read, wait, mfma = "ds_read_b128 v[0:3], v9", "s_waitcnt lgkmcnt(0)", "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0"
    assert _crossings([read, "000000 <L1>:", wait, mfma]) == [(1, "000000 <L1>:")]
    assert _crossings([read, "v_mov_b32_e32 v8, v3", wait, mfma]) == [(1, "v_mov_b32_e32 v8, v3")]
    assert len(_crossings([read, "ds_read_b128 v[4:7], v9 offset:1024", "s_waitcnt lgkmcnt(1)", mfma])) == 1
    assert _crossings([read, wait, "000000 <L1>:", mfma]) == []


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
    assert len(tile) >= 100 and all(any(n in k for k in kernels) for n in ("attn_prefill", "gemm_wide")), len(tile)
    assert all(any("ds_read_b128" in l for l in ls) for ls in kernels.values())
    bad = {k: _crossings(ls) for k, ls in kernels.items()}
    bad = {k: v for k, v in bad.items() if v}
    assert not bad, (len(bad), next(iter(bad.items())))
