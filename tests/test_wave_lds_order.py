"""Kernels that write their wave's LDS anew in a loop: a wave barrier (which keeps the
compiler from moving one lane's write above the reads other lanes' data comes from)
stands before the write as well as between the write and the reads.  Read off the
device code as the front end emits it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_01728_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# functions (with every template instance) that restage LDS in a loop
LOOPS = {"hblocks.hip": ["k_units_grp", "k_strips_grp"], "block.hip": ["rows32", "rows64"]}


@pytest.mark.parametrize("source", sorted(LOOPS))
def test_barrier_before_and_after_restaging(source, tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "d.ll"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-device-only", "-O1", "-std=c++17",
                    "-Xclang", "-disable-llvm-passes", "-S", "-emit-llvm",
                    "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, source),
                    "-o", str(out)], check=True, capture_output=True)
    text = out.read_text()
    bodies = {m.group(1): m.group(2) for m in
              re.finditer(r"^define [^\n]*@(\S+?)\(.*?\{\n(.*?)^\}", text, re.M | re.S)}

    def barriers(body):
        n = body.count("call void @llvm.amdgcn.wave.barrier()")
        return n + sum(body.count(f"@{f}(") for f in bodies if "wave_lds_fence" in f)

    for name in LOOPS[source]:
        found = [f for f in bodies if re.match(rf"_ZN3dpg\S*\d{name}I", f)]
        assert found, name
        for f in found:
            assert barriers(bodies[f]) >= 2, f
