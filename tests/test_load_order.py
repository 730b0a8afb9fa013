"""The fused attention kernel's explicit waits count the loads in flight: for the first keys of a
16-key tile two later keys' copies into LDS (four loads each) and the tile's k and v (eight loads),
for the last one the copies alone. The counts hold only while the loads are issued in the order they
were written for. This compiles the kernel for gfx950 (CPU only) and reads that order off the assembly:
as it is built, and under two other instruction schedulers of the compiler, which move whatever the
source leaves free to move."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_05439_amd", "csrc")


def loads_and_waits(tmp_path, scheduler):
    """The kernel's vector-memory operations in order: Z a copy into LDS, K a buffer load into
    registers, a number the count of an explicit wait (before the LDS reads of a key)."""
    from paper_2607_05439_amd import build
    asm = str(tmp_path / "fast.s")
    extra = ["-mllvm", f"-amdgpu-sched-strategy={scheduler}"] if scheduler else []
    subprocess.run(["hipcc", *build.FLAGS, *extra, "-S", "--cuda-device-only", os.path.join(CSRC, "fast.hip"), "-o", asm],
                   check=True, capture_output=True)
    body = re.search(r"^\w*11attn_kernel\w*:[^\n]*\n(.*?)^\s*s_endpgm", open(asm).read(), re.S | re.M).group(1)
    ops, in_asm = [], False
    for line in body.split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
        line = line.split(";")[0].strip()
        wait = re.match(r"s_waitcnt vmcnt\((\d+)\)$", line)
        if line.startswith("buffer_load_"):
            ops.append("Z" if line.endswith(" lds") else "K")
        elif line.startswith(("scratch_", "buffer_store", "global_store")):
            ops.append("S")
        elif wait and in_asm:
            ops.append(wait.group(1))
    return ops


@pytest.mark.parametrize("scheduler", [None, "max-ilp", "iterative-minreg"])
def test_attention_loads_are_issued_in_the_order_their_waits_count_on(tmp_path, scheduler):
    ops = loads_and_waits(tmp_path, scheduler)
    end = ops.index("0") if "0" in ops else len(ops)  # the wait for everything, after the loop
    prologue = ["Z"] * 12 + ["K"] * 8
    tile = (["16"] + ["Z"] * 4) * 3 + ["8"] + ["Z"] * 4 + ["K"] * 8
    assert ops[:end] == prologue + tile
