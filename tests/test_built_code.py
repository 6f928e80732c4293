"""The built gfx950 code, which is the library's own, built from this repository's sources.

It keeps the wait states that the hardware does not supply itself (CDNA ISA,
manually inserted wait states) around the direct loads into LDS and the 128-bit stores, which the
kernels issue from inline assembly where the compiler's hazard pass does not look:

  a scalar write of M0, then a load into LDS:                       1
  a vector instruction's write of an SGPR, then a memory
  instruction that reads it (descriptors, scalar offsets):           5
  a store of more than 64 bits, then a vector write of its data:    2

Each instruction between counts one, s_nop n counts n + 1.

And the large kernels hold their state in registers: the spills the compiler reports stay within what
was measured to cost nothing."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_23264_amd", "libxstage.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of the library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        n = struct.unpack_from("<Q", data, at + len(MAGIC))[0]
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if size and b"gfx950" in name:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def registers(operand):
    out = set()
    for kind, lo, hi, one in re.findall(r"\b([sv])\[(\d+):(\d+)\]|\b([sv]\d+|m0|vcc)\b", operand):
        out |= {f"{kind}{i}" for i in range(int(lo), int(hi) + 1)} if kind else {one}
    return out


def hazards(lines):
    """(kernel, hazard, instruction) of every pair that is too close; lines as llvm-objdump prints them."""
    found, kernel, recent = [], "", []
    for line in lines:
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            kernel, recent = m[1], []
            continue
        text = line.split("//")[0].strip()
        m = re.match(r"([a-z]\w+)(?:\s+(.*))?$", text)
        if not m or not line.startswith("\t"):
            continue
        op, operands = m[1], (m[2] or "").split(", ")
        vector = op.startswith("v_")
        memory = op.startswith(("buffer_", "global_", "flat_", "scratch_"))
        to_lds = memory and ("lds" in operands[-1].split() or "_lds_" in op)
        reads = registers(m[2] or "") if memory else set()
        writes = set()
        if op.startswith(("v_", "s_")) and not op.startswith(("s_waitcnt", "s_nop", "s_barrier", "s_cbranch", "s_cmp")):
            writes = registers(operands[0])
            if re.match(r"v_(swap|permlane\d+_swap|(add|sub|subrev|addc|subb|subbrev)_co|div_scale)", op):
                writes |= registers(operands[1])
        away = 0
        for w, by_vector, data, states in reversed(recent):
            if to_lds and away < 1 and "m0" in w:
                found.append((kernel, "M0 write, load into LDS", text))
            if by_vector and away < 5 and {r for r in w & reads if r[0] == "s"}:
                found.append((kernel, "SGPR written by a vector instruction, memory instruction", text))
            if vector and away < 2 and data & writes:
                found.append((kernel, "wide store, its data written", text))
            away += states
        data = set()
        if re.match(r"(global|flat|scratch|buffer)_store_dwordx[34]", op):
            data = registers(operands[0 if op.startswith("buffer") else 1])
        recent = recent[-7:] + [(writes, vector, data, int(operands[0], 0) + 1 if op == "s_nop" else 1)]
    return found


def test_the_scan_finds_each_hazard():
    ok = ["0000 <k>:", "\ts_mov_b32 m0, s4", "\ts_nop 0", "\tbuffer_load_dwordx4 v1, s[8:11], 0 offen lds",
          "\tv_readfirstlane_b32 s9, v3", "\ts_nop 4", "\tbuffer_load_dword v2, v1, s[8:11], 0 offen",
          "\tglobal_store_dwordx4 v[0:1], v[4:7], off sc1", "\ts_nop 1", "\tv_mov_b32_e32 v5, 0"]
    assert hazards(ok) == []
    assert [h[1] for h in hazards([ok[0]] + [x for x in ok if "s_nop" not in x])] == [
        "M0 write, load into LDS", "SGPR written by a vector instruction, memory instruction",
        "wide store, its data written"]
    assert hazards(["0000 <k>:", "\ts_add_i32 m0, s4, 8", "\tglobal_load_lds_dwordx4 v[2:3], off"])


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """Paths of the library's code objects."""
    if not (shutil.which(OBJDUMP) and shutil.which(READELF)):
        pytest.skip("needs ROCm's llvm-objdump and llvm-readelf")
    if not os.path.exists(LIB):
        from paper_2607_23264_amd.build import build
        build(verbose=False)
    out = []
    with open(LIB, "rb") as f:
        for i, obj in enumerate(code_objects(f.read())):
            out.append(tmp_path_factory.mktemp("objects") / f"{i}.o")
            out[-1].write_bytes(obj)
    assert out
    return out


def test_built_code_keeps_the_wait_states(objects):
    loads, found = 0, []
    for path in objects:
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True)
        lines = r.stdout.splitlines()
        loads += sum(" lds" in x.split("//")[0] for x in lines)
        found += hazards(lines)
    assert loads > 100            # the scan sees the direct loads
    assert not found, f"{len(found)} hazards, first {found[:5]}"


# (kernel, spilled VGPRs). The bf16 FFN's two are a constant of its error reports.
@pytest.mark.parametrize("kernel,vgprs", [("ep_ffn_kernelILi1E", 0), ("ep_ffn_kernelILi2E", 0), ("ep_ffn_kernelILi3E", 2),
                                          ("ep_ffn_mx_kernel", 24), ("ep_ffn_w4a8_kernel", 28)])
def test_expert_ffn_kernels_stay_in_registers(objects, kernel, vgprs):
    spills = {}
    for path in objects:
        r = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True)
        names = re.findall(r"^\s+\.name:\s+(_Z\w+)$", r.stdout, flags=re.M)
        counts = re.findall(r"^\s+\.vgpr_spill_count:\s+(\d+)$", r.stdout, flags=re.M)
        assert len(names) == len(counts)
        spills.update(zip(names, map(int, counts)))
    found = [n for name, n in spills.items() if kernel in name]
    assert len(found) == 1 and found[0] <= vgprs
