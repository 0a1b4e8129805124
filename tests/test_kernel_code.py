"""What the compiled kernels have to hold whatever the compiler makes of the source: read from the disassembly of the
built library's own gfx950 code (no GPU needed)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> instructions, in the order of the code."""
    from paper_2506_03887_amd.binding import LIB_PATH
    at = tmp_path_factory.mktemp("code")
    shutil.copy(LIB_PATH, at / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(at / "lib.so")], check=True, capture_output=True)
    out = {}
    for f in glob.glob(str(at / "lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m.group(1)
                out[name] = []
            elif name and line.strip():
                out[name].append(line.split("//")[0].strip())
    assert out
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_a_block_of_the_spread_step_counts_itself_in_when_its_loads_have_returned(kernels):
    """The blocks of a row read its stack, count themselves in, and the last to do so overwrites the stack: between the
    last load before the count (the first atomic that returns a value) and the count, the wave has to wait for all loads."""
    found = {n: code for n, code in kernels.items() if "step_spread_kernel" in n}
    assert len(found) == 4
    for name, code in found.items():
        count = next(i for i, x in enumerate(code) if re.match(r"global_atomic_add\b.*\bsc0\b", x))
        loads = [i for i, x in enumerate(code[:count]) if re.match(r"(global|flat|buffer|scratch)_load", x)]
        waits = [i for i, x in enumerate(code[:count]) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", x)]
        assert waits and waits[-1] > loads[-1], name
        between = [x for x in code[waits[-1]: count] if re.match(r"s_cbranch|s_branch", x)]
        assert all(x.startswith("s_cbranch_execz") for x in between), (name, between)     # straight code, lanes switched off at most


def test_inputs_that_a_launch_overwrites_are_kept_where_they_are_read():
    """Loads through the constant address space may be moved behind a store or repeated after it, and no fence or wait orders
    them: every place that reads tokens, states or len that way in a kernel that writes them keeps the value at once."""
    src = open(os.path.join(os.path.dirname(__file__), "..", "paper_2506_03887_amd", "csrc", "advance_kernels.hip")).read()
    plan_only = src[src.index("void plan_only_scalar"):]
    src = src.replace(plan_only[: plan_only.index("\n}\n")], "")          # mask + masking: writes none of them
    reads = re.findall(r"table<true>\((?:tokens|len|states), b\)", src)
    places = re.findall(r"int ((?:\w+ = table<true>\((?:tokens|len|states), b\)(?:, )?)+);((?:\n *keep_input\(\w+\);)*)", src)
    for read, kept in places:
        assert re.findall(r"(\w+) = table", read) == re.findall(r"keep_input\((\w+)\)", kept), read
    assert sum(kept.count("keep_input") for _, kept in places) == len(reads) == 5
