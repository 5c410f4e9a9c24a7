"""Wait states in the library's machine code.  On gfx950 a scalar register (VCC among them) that a vector instruction has
written may be read by a vector instruction two wait states later at the earliest, as a lane number four and by a memory
instruction five.  The compiler keeps to that in what it writes itself, and does not look inside an asm string."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2007_14152_amd import build as hip_build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def scalars(operands):
    """The scalar registers an operand list names."""
    found = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\bvcc\b", operands):
        if m[1]:
            found.update(range(int(m[1]), int(m[2]) + 1))
        else:
            found.add(int(m[3]) if m[3] else "vcc")
    return found


def too_early(listing):
    """(kernel, line, what it follows) for every instruction that reads a scalar register before its wait is over."""
    kernel, behind, hits = "", [], []  # behind: (wait states, scalars a vector instruction wrote, text), oldest first
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            kernel, behind = m[1], []
            continue
        text = line.split("//")[0].strip()
        op, _, operands = text.partition(" ")
        vector = op.startswith("v_")
        memory = op.startswith(("buffer_", "global_", "flat_", "scratch_"))
        first, _, rest = operands.partition(",")
        written = scalars(first) if vector else set()
        if vector and re.search(r"_co_|^v_div_scale|^v_mad_[ui]64", op):  # the carry is the second operand
            second, _, rest = rest.partition(",")
            written = scalars(second)
        read = scalars(rest) if vector else scalars(operands) if memory else set()
        number = scalars(operands.rpartition(",")[2]) if op.startswith(("v_readlane", "v_writelane")) else set()  # of a lane
        since = 0
        for states, were_written, earlier in reversed(behind):
            if since < (5 if memory else 2) and were_written & read or since < 4 and were_written & number:
                hits.append((kernel, text, earlier))
                break
            since += states
        behind = behind[-5:] + [(int(operands, 0) + 1 if op == "s_nop" else 1, written, text)]
    return hits


def test_the_check_itself():
    at = "0 <k>:\n"
    assert too_early(at + "v_cmp_gt_u32_e32 vcc, v1, v2\nv_cndmask_b32_e32 v3, v4, v5, vcc")
    assert too_early(at + "v_cmp_gt_u32_e64 s[2:3], v1, v2\ns_nop 0\nv_cndmask_b32_e64 v3, v4, v5, s[2:3]")
    assert too_early(at + "v_readfirstlane_b32 s5, v2\ns_nop 3\nbuffer_load_dword v3, v4, s[4:7], 0 offen")
    assert too_early(at + "v_readfirstlane_b32 s5, v2\ns_nop 2\nv_readlane_b32 s6, v3, s5")
    assert not too_early(at + "v_readfirstlane_b32 s5, v2\ns_nop 2\nv_writelane_b32 v3, s5, 7")
    assert not too_early(at + "v_cmp_gt_u32_e32 vcc, v1, v2\ns_nop 1\nv_cndmask_b32_e32 v3, v4, v5, vcc")
    assert not too_early(at + "v_readfirstlane_b32 s5, v2\ns_nop 4\nbuffer_load_dword v3, v4, s[4:7], 0 offen")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_scalar_register_is_read_too_early(tmp_path):
    """Of what was built here, every kernel."""
    shutil.copy(hip_build.LIB, tmp_path)
    lib = os.path.basename(hip_build.LIB)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    objects = [f for f in os.listdir(tmp_path) if f.startswith(lib + ".") and "gfx950" in f]
    assert objects
    for f in objects:
        listing = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, stdout=subprocess.PIPE, text=True).stdout
        assert listing.count(">:") > 20 and listing.count("v_cndmask") > 100
        hits = too_early(listing)
        assert not hits, (len(hits), hits[:3])
