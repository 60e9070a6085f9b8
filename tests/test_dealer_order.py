"""How the waves of a workgroup hand over what one of them asked the dispenser
for (WaveDealer, in the persistent escape-time kernel): the record of the tiles
and the cursor are ordinary LDS data, so the word that announces them is stored
with release and taken with acquire order, and a wave's report that it has read
the record is stored with release and read with acquire order. Seen in the LLVM
IR that the compiler makes of the kernel (CPU only)."""
import os
import re
import subprocess

import pytest

from test_kernel_isa import CSRC, HIPCC


def test_records_are_handed_over_in_order(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.ll"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S", "-emit-llvm", "-o",
                    str(out), os.path.join(CSRC, "kernels.hip")], check=True, capture_output=True)
    body = re.search(r"define[^\n]*@_ZN2ce12k_persistentINS_10EscapeTile.*?^}", out.read_text(), flags=re.S | re.M).group(0)
    lines = [x for x in body.splitlines() if "addrspace(3)" in x and 'syncscope("workgroup")' in x]
    order = {
        "state taken": [x for x in lines if "atomicrmw add" in x and ", i64 1 " in x],
        "state stored": [x for x in lines if "store atomic i64" in x],
        "read reported": [x for x in lines if "atomicrmw add" in x and ", i32 1 " in x],
        "read seen": [x for x in lines if "load atomic i32" in x],
    }
    want = {"state taken": " acquire,", "state stored": " release,", "read reported": " release,", "read seen": " acquire,"}
    for what, found in order.items():
        assert found, what
        for x in found:
            assert want[what] in x or " acq_rel," in x or " seq_cst," in x, (what, x)
