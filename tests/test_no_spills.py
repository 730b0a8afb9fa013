"""No kernel spills registers to scratch memory: each is sized to hold its working set (CPU only; the
figures the compiler writes beside every kernel of the library, as it is built)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2607_05439_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")


def test_no_kernel_spills_registers(tmp_path):
    def kernels(src):
        asm = str(tmp_path / (src + ".s"))
        subprocess.run(["hipcc", *build.FLAGS, *build.EXTRA.get(src, []), "-S", "--cuda-device-only",
                        os.path.join(CSRC, src), "-o", asm], check=True, capture_output=True)
        return re.findall(r"^    \.name: +(\w+)\n.*?^    \.vgpr_spill_count: (\d+)$", open(asm).read(), re.S | re.M)

    with ThreadPoolExecutor(max_workers=8) as ex:
        found = [k for ks in ex.map(kernels, build.SOURCES) for k in ks]
    assert len(found) > 50
    assert [name for name, spilled in found if spilled != "0"] == []
