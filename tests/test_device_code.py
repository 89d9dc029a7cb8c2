"""What has to hold of the device code as it was compiled: it is read back from the built library."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2102_04782_amd import binding as daq

LLVM = next((os.path.dirname(p) for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump") or "") if p and os.path.exists(p)), None)
pytestmark = pytest.mark.skipif(LLVM is None, reason="no llvm-objdump")


def _tool(name, *args, cwd=None):
    res = subprocess.run([os.path.join(LLVM, name), *args], capture_output=True, text=True, timeout=300, cwd=cwd)
    assert res.returncode == 0, res.stderr[-2000:]
    return res.stdout


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    daq.lib()   # (loads it: a test run may be the first to build it)
    there = tmp_path_factory.mktemp("code")
    shutil.copy(daq.LIB_PATH, there / "lib.so")
    _tool("llvm-objdump", "--offloading", "lib.so", cwd=there)
    found = sorted(glob.glob(str(there / "*gfx950")))
    assert found
    return found


def _registers(operand):
    """'v7' -> {v7}, 'a[2:5]' -> {a2 .. a5}, anything else -> nothing."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    first, last = (m[2], m[2]) if m[2] else (m[3], m[4])
    return {f"{m[1]}{i}" for i in range(int(first), int(last) + 1)}


def test_matrix_instructions_wait_for_what_vector_instructions_wrote(code_objects):
    """A matrix instruction reads a register two wait states after a vector instruction wrote it, at the earliest.  The hardware does not wait
    and the compiler does so only for instructions that it knows, not for those inside inline assembly."""
    seen, bad = 0, []
    for path in code_objects:
        kernel, recent = "", []   # (wait states from its issue on, registers written), newest last
        for line in _tool("llvm-objdump", "-d", "--mcpu=gfx950", path).splitlines():
            if line.endswith(">:"):
                kernel, recent = line, []
                continue
            m = re.match(r"\t([a-z]\w+)\s*(.*?)\s*(?://.*)?$", line)
            if not m:
                continue
            op, args = m[1], re.split(r",\s*(?![^\[]*\])", m[2])
            if op.startswith("v_mfma") or op.startswith("v_smfma"):
                seen += 1
                reads = set().union(*(_registers(a) for a in args[1:4]))
                between = 0
                for states, written in reversed(recent):
                    if between >= 2:
                        break
                    if written & reads:
                        bad.append((kernel, line.strip(), sorted(written & reads)))
                    between += states
                recent.append((1, set()))
            else:
                written = _registers(args[0].split()[0]) if op.startswith("v_") and args[0] else set()
                recent.append((int(args[0], 0) + 1 if op == "s_nop" else 1, written))
            del recent[:-4]
    assert seen > 1000
    assert not bad, (len(bad), bad[:5])


def test_kernels_of_products_keep_their_registers(code_objects):
    """No kernel that multiplies matrices keeps vector registers in memory: forms and launch bounds are chosen so that they fit."""
    kernels, bad = 0, []
    for path in code_objects:
        for block in _tool("llvm-readelf", "--notes", path).split(".agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block)[1]
            spilled = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", block)[1])
            if re.search("k_conv_|k_dw|k_dx_|k_bwd_both|k_nhwc", name):
                kernels += 1
                if spilled:
                    bad.append((name, spilled))
    assert kernels > 50 and not bad, bad
