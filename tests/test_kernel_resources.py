"""CPU check of what the compiler gives the decode kernels: registers and LDS
only.  A spill to scratch memory costs a launch the allocation of scratch and
its waves the memory traffic, and no output shows it."""
import os
import re
import subprocess

import pytest

from paper_2606_15789_amd import build


@pytest.mark.parametrize("source", ["wc_decode.hip", "wc_decode_wide.hip"])
def test_decode_kernels_spill_nothing(source, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    asm = tmp_path / "kernels.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-lpthread")]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", str(asm)],
                   check=True, capture_output=True, text=True, timeout=600)
    # the code object's metadata: one entry a kernel, its fields in alphabetical order
    kernels = re.findall(r"^    \.name: +(\S*wc_decode\w*)\n(.*?)\.wavefront_size:", asm.read_text(),
                         re.M | re.S)
    assert kernels
    for name, meta in kernels:
        fields = dict(re.findall(r"\.(\w+): +(\d+)", meta))
        got = {k: int(fields[k]) for k in ("private_segment_fixed_size", "sgpr_spill_count",
                                           "vgpr_spill_count")}
        assert not any(got.values()), (name, got)
