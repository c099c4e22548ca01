"""The attention kernels run from registers: the built code objects' own
metadata says how many bytes of scratch memory (spilled registers) a lane of
each kernel takes.  No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2606_27748_amd import build as B

LLVM = "/opt/rocm/llvm/bin"

# Three variants of the bf16 d = m = 64 kernels sit at the 256 registers of two
# workgroups per CU and spill a few: the adding dK/dV and dQ sweeps (m = 144 to
# 192) and the padded dK/dV sweep (m < 64), nonstationary causal.
ALLOWED = {
    "k_bwd_dkvIDF16bLi64ELi16ELi4ELb1ELb1ELb1ELb0E": 28,
    "k_bwd_dkvIDF16bLi64ELi16ELi4ELb1ELb1ELb0ELb1E": 8,
    "k_bwd_dqIDF16bLi64ELi16ELi4ELb1ELb1ELb1ELb1ELb0E": 8,
}


def scratch_bytes(obj, tmp):
    """{kernel symbol: scratch bytes per lane} of one built object file."""
    fat, co = os.path.join(tmp, "fat"), os.path.join(tmp, "co")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, os.devnull], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={fat}", f"--output={co}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
    names = re.findall(r"^\s+\.name:\s+(_ZN4flex\S+)$", notes, flags=re.M)
    sizes = re.findall(r"^\s+\.private_segment_fixed_size:\s+(\d+)$", notes, flags=re.M)
    assert len(names) == len(sizes) > 0
    return dict(zip(names, map(int, sizes)))


@pytest.mark.parametrize("source", ["flex_fwd.hip", "flex_bwd.hip", "flex_bwd_dq.hip"])
def test_no_spilled_registers(source, tmp_path):
    obj = os.path.join(B.BUILD, source.replace(".hip", ".o"))
    if not (os.path.exists(obj) and os.path.exists(f"{LLVM}/clang-offload-bundler")):
        pytest.skip("needs the built objects and the LLVM tools")
    over = {}
    for name, size in scratch_bytes(obj, str(tmp_path)).items():
        limit = max([v for k, v in ALLOWED.items() if k in name], default=0)
        if size > limit:
            over[name] = size
    assert not over
