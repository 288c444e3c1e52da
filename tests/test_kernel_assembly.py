"""The gfx950 code of the built library, searched for vector instructions behind a
loop whose lanes have all left (EXEC is empty there until the next instruction
that sets it): the register allocator has placed copies of split live ranges
there, whose values are then lost.  Only instructions that ignore EXEC (scalar
ones, lane reads and writes) may stand between the loop's last branch and the
instruction that sets EXEC again."""
import os
import re
import struct
import subprocess

import pytest

from paper_2011_07209_amd import exx

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 code objects of a library's offload bundles."""
    data = open(lib, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode("ascii", "replace")
            p += 24 + idlen
            if name.endswith("gfx950") and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 24)


def _lost_writes(lines):
    """(function, instruction) of each vector instruction that runs with the EXEC of a finished loop."""
    found, exits, fn, prev, inside = [], 0, "", "", False
    for line in lines:
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            fn, prev, inside = m.group(1), "", False
            continue
        ins = line.split("//")[0].strip()
        if not ins or not line.startswith(("\t", " ")):
            continue
        op = ins.split()[0]
        if inside:
            if re.match(r"s_\w+ exec\b", ins) or "saveexec" in op or op.startswith(("s_branch", "s_cbranch", "s_endpgm", "s_setpc")):
                inside = False
            elif op.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_")) and \
                    not op.startswith(("v_readlane", "v_writelane", "v_readfirstlane")):
                found.append((fn, ins))
        if op == "s_cbranch_execnz" and re.match(r"s_andn2_b64 exec, exec", prev):
            exits += 1
            inside = True
        prev = ins
    return found, exits


def test_the_search_itself():
    loop = ["0 <k>:", "\ts_andn2_b64 exec, exec, s[0:1]", "\ts_cbranch_execnz 65000"]
    ok = loop + ["\tv_readlane_b32 s2, v9, 1", "\ts_or_b64 exec, exec, s[0:1]", "\tv_mov_b32_e32 v1, v2"]
    bad = loop + ["\tv_mov_b32_e32 v1, v2", "\ts_or_b64 exec, exec, s[0:1]"]
    assert _lost_writes(ok) == ([], 1)
    assert _lost_writes(bad) == ([("k", "v_mov_b32_e32 v1, v2")], 1)


def test_no_vector_write_behind_a_finished_loop(tmp_path):
    if not os.path.exists(exx.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("no built library, or no disassembler")
    exits = kernels = 0
    for i, obj in enumerate(_code_objects(exx.LIB_PATH)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(obj)
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True)
        lines = r.stdout.splitlines()
        found, n = _lost_writes(lines)
        assert not found, found[:8]
        exits += n
        kernels += sum("k_pcg" in l or "k_solve" in l for l in lines if l.endswith(">:"))
    print(f"kernels of the CG {kernels}, loops with an exit of all lanes {exits}")
    assert kernels > 300 and exits > 1000
