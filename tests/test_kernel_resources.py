"""What the compiler says the interpreter's kernels use: registers kept in
memory are read back once per scheduling round of a wave whose latency is the
step's time."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"


def kernels(obj, tmp_path):
    fat, code = tmp_path / "fat", tmp_path / "code"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", obj, str(tmp_path / "rest")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={code}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(code)], capture_output=True, text=True, check=True).stdout
    out = {}
    for part in notes.split("- .agpr_count")[1:]:
        get = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s*$", part, re.M)}
        out[re.search(r"\.name:\s+(\S+)", part).group(1)] = get
    return out


def test_no_vector_register_is_spilled(tmp_path):
    """k_interp<lanes, cartridge bytes, who scans, no-ops>: without collision
    latches, and with them scanned by the helper waves (batches up to 256 tiles)."""
    obj = os.path.join(ROOT, "_build", "interp.o")
    if not os.path.exists(obj):
        pytest.skip("the library was not built here")
    seen = 0
    for name, k in kernels(obj, tmp_path).items():
        m = re.search(r"k_interpILi(\d+)ELi(\d+)EL[ib](\d)ELb(\d)E", name)
        if m and m.group(3) in "02":
            seen += 1
            assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0, (name, k)
            assert k["vgpr_count"] <= 256, (name, k)      # two waves per SIMD
    assert seen == 16
