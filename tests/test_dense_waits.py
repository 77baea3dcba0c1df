"""The dense-layer kernel's counted waits, read from the built library: a wait for a weight stage may leave outstanding no more than was
really issued behind that stage.  (A load whose registers nothing reads is taken out by the compiler; a count that has it waits too little.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2003_10688_amd import sol

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernels(tmp):
    """Template arguments and instructions of every conv_dense_kernel in the library."""
    shutil.copy(sol.LIB_PATH, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f], cwd=tmp, check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=\S*<\S+>:)", text):
            m = re.search(r"conv_dense_kernelI((?:Li\d+E)+)E", part.split("\n", 1)[0])
            if m:
                yield [int(v) for v in re.findall(r"\d+", m[1])], [l.split("//")[0].strip() for l in part.split("\n")[1:]]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_waits_count_what_was_issued(tmp_path):
    seen = 0
    for (pa, ca, wpa, ksb, dx, nsw, dw), ins in kernels(str(tmp_path)):
        events, allowed = [], []          # "D" weights, "X" pixels, "W" wait and barrier; what each W leaves outstanding
        for i, l in enumerate(ins):
            if l.startswith("buffer_load_dwordx4"):
                events.append("D" if l.endswith("lds") else "X")
            elif l.startswith("s_barrier"):
                before = next((b for b in reversed(ins[max(0, i - 3):i]) if "vmcnt" in b), None)
                if before:
                    events.append("W")
                    allowed.append(int(re.search(r"vmcnt\((\d+)\)", before)[1]))
        at = [i for i, e in enumerate(events) if e == "W"]
        steps = 2 * dx                    # one turn of the loop, the steps behind it, the last chunk's: as they lie in memory they are one path
        assert len(at) >= steps
        at.append(len(events))
        for k in range(steps):
            inside = events[at[k]:at[k + 1]]
            assert inside.count("D") >= 2 and ("X" in inside) == (k < dx), (pa, k, inside)
        for k in range(dw, steps):        # stage k: the first two D of step k - dw
            first = at[k - dw]
            second = [i for i in range(first, at[k]) if events[i] == "D"][1]
            behind = sum(e in "DX" for e in events[second + 1:at[k]])
            assert allowed[k] <= behind, (pa, ca, k, allowed[k], behind)
        seen += 1
    assert seen == 6
