"""Wait states around the kernels' direct LDS loads, read from the disassembly of the
built library: the compiler adds none inside or around inline assembly.  gfx950 wants

  - one instruction or s_nop between a write of M0 and a *_lds_* load that uses it;
  - five wait states between a vector instruction that writes an SGPR and a vector
    memory instruction that reads it (none once a scalar instruction has rewritten it:
    the scalar unit waits for the vector write by itself).

Both hold for every load, the compiler's own included."""
import os
import re
import shutil
import subprocess

import pytest

seer = pytest.importorskip("paper_2410_13276_amd")
if not os.path.exists(seer.LIB_PATH):
    pytest.skip("libseer.so not built", allow_module_level=True)
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
if not os.path.exists(OBJDUMP):
    pytest.skip("no llvm-objdump", allow_module_level=True)

MEMORY = ("global_", "buffer_", "scratch_", "flat_")
SGPR = re.compile(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]")


def sgprs(text):
    out = set()
    for m in SGPR.finditer(text):
        lo = int(m.group(1) or m.group(2))
        out |= set(range(lo, int(m.group(3) or lo) + 1))
    return out


def violations(lines):
    """(kernel, instruction, rule) of every breach, and the number of direct LDS loads."""
    found, loads, kernel = [], 0, ""
    since = {}      # SGPR -> wait states since the vector instruction that wrote it last
    m0_written = False
    for line in lines:
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if m:
            kernel, since, m0_written = m.group(1), {}, False
            continue
        m = re.match(r"^\s+(\w+)\s*(.*?)\s*//", line)
        if not m:
            continue
        op, args = m.groups()
        if op.startswith(MEMORY):
            if "_lds_" in op:
                loads += 1
                if m0_written:
                    found.append((kernel, f"{op} {args}", "M0"))
            if any(since.get(r, 5) < 5 for r in sgprs(args)):
                found.append((kernel, f"{op} {args}", "SGPR"))
        if op in ("s_endpgm", "s_branch", "s_setpc_b64"):  # nothing falls through to the next line
            since, m0_written = {}, False
            continue
        states = int(args, 0) + 1 if op == "s_nop" else 1
        since = {r: n + states for r, n in since.items() if n + states < 5}
        operands = args.split(",")
        m0_written = op.startswith("s_") and operands[0] == "m0"
        if op.startswith("s_"):
            for r in sgprs(operands[0]):
                since.pop(r, None)
        elif op.startswith("v_"):
            # (a carry or scale flag is the second operand)
            for r in sgprs(operands[0]) | (sgprs(operands[1]) if "_co_" in op or "div_scale" in op else set()):
                since[r] = 0
    return found, loads


def disassemble(path, tmp):
    shutil.copy(path, tmp / "lib")
    subprocess.run([OBJDUMP, "--offloading", "lib"], cwd=tmp, check=True, capture_output=True)
    for f in sorted(tmp.glob("lib*gfx950")):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--mcpu=gfx950", str(f)], check=True,
                           capture_output=True, text=True)
        yield from r.stdout.splitlines()


def test_direct_loads_have_their_wait_states(tmp_path):
    found, loads = violations(disassemble(seer.LIB_PATH, tmp_path))
    assert loads > 500
    assert not found, (len(found), found[:4])


@pytest.mark.parametrize("text,rule", [
    (" s_mov_b32 m0, s1 //\n global_load_lds_dwordx4 v1, s[2:3] //", "M0"),
    (" s_mov_b32 m0, s1 //\n s_nop 0 //\n global_load_lds_dwordx4 v1, s[2:3] //", None),
    (" v_readlane_b32 s3, v9, 4 //\n s_nop 3 //\n global_load_lds_dwordx4 v1, s[2:3] //", "SGPR"),
    (" v_readlane_b32 s3, v9, 4 //\n s_nop 4 //\n global_load_lds_dwordx4 v1, s[2:3] //", None),
    (" v_readlane_b32 s3, v9, 4 //\n s_mov_b64 s[2:3], s[2:3] //\n global_load_dword v1, s[2:3] //", None),
    (" v_add_co_u32_e64 v1, s[4:5], v2, v3 //\n global_store_dword v1, v2, s[4:5] //", "SGPR"),
])
def test_the_reading_itself(text, rule):
    found, _ = violations(text.splitlines())
    assert [f[2] for f in found] == ([rule] if rule else [])
