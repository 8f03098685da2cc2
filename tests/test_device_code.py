"""What the device code's own tests cannot show because it depends on the compiler's choices: wait states that it does not supply inside
inline assembly, looked for in the built library, and values that are read before they are set, looked for in a compilation that
gives these a pattern."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2512_23858_amd as ygg

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every function of the library's gfx950 code objects."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    where = tmp_path_factory.mktemp("device_code")
    shutil.copy(ygg.lib_path(), where / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=where, check=True, capture_output=True)
    functions = {}
    for obj in sorted(where.glob("*gfx950*")):
        code = []
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout.splitlines():
            if m := re.match(r"[0-9a-f]+ <(.*)>:$", line):
                code = functions[m[1]] = []
            elif line.startswith("\t"):
                code.append(line.split("//")[0].strip())
    return functions


def _states(instruction):
    m = re.match(r"s_nop (\d+)", instruction)
    return int(m[1]) + 1 if m else 1


def _too_close(code, load, writes, states):
    """Loads with fewer than `states` wait states between them and a write that `writes(write, load)` names."""
    found = []
    for i, instruction in enumerate(code):
        if not re.match(load, instruction):
            continue
        seen, j = 0, i - 1
        while j >= 0 and seen < states:
            if writes(code[j], instruction):
                found.append((code[j], instruction))
            seen += _states(code[j])
            j -= 1
    return found


DIRECT_TO_LDS = r"(global|buffer|scratch)_load_\S*lds|buffer_load_.* lds\b"


def test_direct_to_lds_loads_keep_their_distance_from_m0(kernels):
    loads = sum(bool(re.match(DIRECT_TO_LDS, x)) for code in kernels.values() for x in code)
    assert loads > 1000     # (the tile fills)
    for name, code in kernels.items():
        assert not _too_close(code, DIRECT_TO_LDS, lambda w, _: re.match(r"s_\S+ m0,", w), 1), name


def _scalars(operands):
    out = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        out |= set(range(int(lo), int(hi) + 1)) if lo else {int(one)}
    return out


def test_loads_keep_their_distance_from_scalars_that_the_vector_unit_writes(kernels):
    def writes(w, load):
        m = re.match(r"v_(?:readfirstlane|readlane|cmp\S*)\s+([^,]+),", w)
        return m and _scalars(m[1]) & _scalars(load)
    for name, code in kernels.items():
        assert not _too_close(code, DIRECT_TO_LDS, writes, 5), name


def test_no_count_or_index_is_read_before_it_is_set(tmp_path):
    """Local variables start as 0xAA bytes here; where these survive optimisation in whole numbers, a path reads them.  (The operand
    registers of wavefronts without rows, which nothing reads, are vectors of floats and of 16-bit halves.)"""
    from paper_2512_23858_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    flags = [x for x in build.FLAGS if x not in ("-O3", "-Wall", "-fPIC")]
    ir = tmp_path / "attention.ll"
    subprocess.run([build.HIPCC, *flags, "-w", "-O1", "--cuda-device-only", "-S", "-emit-llvm", "-ftrivial-auto-var-init=pattern",
                    os.path.join(os.path.dirname(build.__file__), "csrc", "attn_mfma.hip"), "-o", str(ir)], check=True)
    text = ir.read_text()
    assert text.count("define ") >= 20
    found = [line.strip()[:200] for line in text.splitlines() if "-1431655766" in line or "-6148914691236517206" in line]
    assert not found, found[:5]
