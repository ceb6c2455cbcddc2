"""A read batch's time stamp is taken when the wave's answers are stored: the
compiled stamp waits for the stores before it reads the clock."""
import re
import shutil
import subprocess

import pytest

from paper_2604_16725_amd import build_lib

SRC = """
#include "%s/flix_drain.hpp"
__global__ void k_probe(unsigned* out, unsigned long long* at) {
  out[threadIdx.x] = threadIdx.x;
  flix::stamp_stored(at);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_stamp_waits_for_the_stores(tmp_path):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(SRC % build_lib.CSRC)
    subprocess.run(["hipcc", *build_lib.HIPCC_FLAGS, "--offload-device-only", "-S", "-o", str(asm),
                    str(src)], check=True, capture_output=True)
    body = re.search(r"^_Z7k_probe\w*:(.*?)s_endpgm", asm.read_text(), re.S | re.M).group(1)
    ops = [l.split(";")[0].split() for l in body.splitlines() if l.startswith("\t")]
    name = [o[0] for o in ops if o]
    store = max(i for i, x in enumerate(name) if x.startswith("global_store"))
    clock = name.index("s_memrealtime")
    assert store < clock
    waits = [o for o in ops if o][store + 1: clock]
    assert any(o[0] == "s_waitcnt" and "vmcnt(0)" in " ".join(o) for o in waits), body
