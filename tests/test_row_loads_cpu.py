"""The built row kernels ask for a row's slots one behind the other: no load of a whole row waits for the one before it.  The compiler
puts such waits in where a register that it computes an address in may still be the target of an earlier row's load; results
are the same, a row then takes as many memory latencies as it has slots."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def rows_kernels(tmp_path):
    """(name, instructions) of every row kernel in the built library."""
    shutil.copy(os.path.join(ROOT, "paper_2505_07291_amd", "libgrpo.so"), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", "libgrpo.so"], cwd=tmp_path, check=True, capture_output=True)
    for name in sorted(os.listdir(tmp_path)):
        if not name.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-leading-addr", name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=<)", text):
            head = re.match(r"<(\S*grpo_rows_(?:cached|streamed)\S*)>:\n", part)
            if head:
                yield head.group(1), [line.split("//")[0].strip() for line in part.split("\n")[1:]]


def waits_between_loads(instructions):
    """16-byte loads that stand behind another one with nothing but address arithmetic and a wait for it in between."""
    found, last = 0, ""
    for x in instructions:
        if x.startswith(("global_load_dwordx4", "buffer_load_dwordx4")):
            found += last == "wait"
            last = "load"
        elif last == "load" and re.match(r"s_waitcnt\b.*vmcnt\(0\)", x):
            last = "wait"
        elif x.startswith(("s_barrier", "v_exp", "v_max3", "global_store")):  # a pass over the row, or its gradient
            last = ""
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_loads_of_a_row_do_not_wait_for_each_other(tmp_path):
    kernels = dict(rows_kernels(tmp_path))
    assert len(kernels) > 100
    slow = {name: n for name, n in ((k, waits_between_loads(v)) for k, v in kernels.items()) if n}
    assert not slow, slow
