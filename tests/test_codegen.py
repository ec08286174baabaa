"""Waits in the generated code of the pipelined kernels (CPU: the built
library is disassembled).

The direct global->LDS loads of these kernels are waited for by counts that the
source writes next to its barriers.  A load into registers between them, or a
wait that the compiler adds for one, breaks what those counts stand for: it
drains the loads in flight, or it is not covered by the count at all.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_23159_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every kernel of the library, by mangled name."""
    d = str(tmp_path_factory.mktemp("code"))
    lib = os.path.join(d, "lib.so")
    shutil.copy(B.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    code = {}
    for obj in glob.glob(os.path.join(d, "*gfx950*")):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        name = None
        for line in out.splitlines():
            m = re.match(r"^[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
                code[name] = []
            elif name and line.startswith("\t"):
                code[name].append(line.split("//")[0].strip())
    return code


def _named(kernels, part):
    found = {n: c for n, c in kernels.items() if part in n and not n.endswith(".kd")}
    assert found, part
    return found


def _is_mfma(i):
    return i.startswith("v_mfma")


def _is_register_load(i):
    return re.match(r"(global|buffer|flat)_load", i) and not re.search(r"\blds\b", i)


def _waits_for_loads(i):
    return i.startswith("s_waitcnt") and "vmcnt" in i


def test_ring_gemm_waits_only_at_its_barriers(kernels):
    # up to the last product (after it come the epilogue's own loads)
    for name, code in _named(kernels, "k_gemm_ring").items():
        end = max(i for i, x in enumerate(code) if _is_mfma(x))
        loads = [x for x in code[:end] if _is_register_load(x)]
        assert not loads, (name, loads)
        extra = [(i, x) for i, x in enumerate(code[:end]) if _waits_for_loads(x) and code[i + 1] != "s_barrier"]
        assert not extra, (name, extra)


@pytest.mark.parametrize("kernel", ["k_flash_pad", "k_flash_dl"])
def test_attention_requests_all_of_q_before_waiting(kernels, kernel):
    for name, code in _named(kernels, kernel).items():
        first = min(i for i, x in enumerate(code) if _is_mfma(x))
        loads = [i for i, x in enumerate(code[:first]) if _is_register_load(x)]
        # head_dim / 16 fragments of 16 bytes per lane
        assert len(loads) >= int(re.search(r"ILi(\d+)E", name).group(1)) // 16, name
        waits = [x for x in code[loads[0]:loads[-1]] if _waits_for_loads(x)]
        assert not waits, (name, waits)
