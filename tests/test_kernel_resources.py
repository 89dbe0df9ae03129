"""Registers of the built GEMM kernels of the deeper nets (deep.hip), read from the
object the build left: code shared with the 128 x 128 tiles once cost the 64 x 64 pair
two more spilled registers, the smaller tiles four to eight registers, and the step
about 1 %."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJ = os.path.join(ROOT, "paper_2606_30497_amd", "_build", "deep.hip.o")
BIN = "/opt/rocm/llvm/bin"


def _kernels(tmp_path):
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev")
    subprocess.check_call(["objcopy", "--dump-section", ".hip_fatbin=" + fat, OBJ, str(tmp_path / "copy")])
    subprocess.check_call([os.path.join(BIN, "clang-offload-bundler"), "--unbundle", "--type=o",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + dev])
    notes = subprocess.check_output([os.path.join(BIN, "llvm-readelf"), "--notes", dev], text=True)
    out = {}
    for block in notes.split(".agpr_count:")[1:]:
        name = re.search(r"^\s+\.name:\s+(_Z\S+)", block, re.M).group(1)
        name = subprocess.check_output(["c++filt", name], text=True).strip().replace("mlp::", "")
        out[re.sub(r"^void |\(.*", "", name)] = {
            k: int(re.search(r"\.%s:\s+(\d+)" % k, block).group(1))
            for k in ("vgpr_count", "vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size")}
    return out


@pytest.mark.skipif(not os.path.exists(OBJ) or not os.path.exists(BIN), reason="nothing built, or no ROCm tools")
def test_gemm_tiles_keep_their_registers(tmp_path):
    k = _kernels(tmp_path)
    for ep in (2, 3):   # the pair of a weight gradient and a masked back-propagation
        pair = k["k_gemm_pair<1, 0, 64, 64, 2, %d, 64, 64, true>" % ep]
        assert pair["vgpr_spill_count"] <= 1 and pair["private_segment_fixed_size"] <= 8, pair
    most = {"k_gemm<0, 1, 32, 32, false>": 68,
            "k_gemm_pair<1, 0, 32, 64, 2, 2, 32, 64, false>": 108,
            "k_gemm_pair<1, 0, 32, 64, 2, 2, 64, 64, false>": 136,
            "k_gemm_pair<1, 0, 32, 64, 2, 3, 32, 64, false>": 112,
            "k_gemm_pair<1, 0, 32, 64, 2, 3, 64, 64, false>": 140}
    for name, n in most.items():
        assert k[name]["vgpr_count"] <= n, (name, k[name])
    for name, r in k.items():
        if "64, 64, true" not in name:
            assert r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, (name, r)
    assert k["k_deep_apply"]["sgpr_spill_count"] == 0
