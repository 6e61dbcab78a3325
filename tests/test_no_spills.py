"""What the compiler says of the built kernels: no call of rs_route_plus runs on a kernel that spills vector registers (at widths above
5120 such spills cost up to half of a call), and neither do the row norms, which hold all of a row's partial sums at once (120 of the 128 registers
that a thread of their workgroups has, above 8192 values a row)."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


def spills(tmp_path):
    import paper_2507_17307_amd as P
    fat, obj = tmp_path / "fat.bin", tmp_path / "gfx950.o"
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", P.library_path(), str(tmp_path / "rest.so")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--input={fat}", f"--output={obj}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
    return dict(zip(re.findall(r"\.name:\s+(_Z\S+)", notes), map(int, re.findall(r"\.vgpr_spill_count:\s+(\d+)", notes))))


needs_tools = pytest.mark.skipif(not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="needs the ROCm LLVM tools")


@needs_tools
def test_router_kernels_do_not_spill(tmp_path):
    router = {n: s for n, s in spills(tmp_path).items() if "router_plus" in n}
    assert len(router) == 5 and not any(router.values()), router


@needs_tools
def test_row_norms_do_not_spill(tmp_path):
    norms = {n: s for n, s in spills(tmp_path).items() if "k_rmsnorm_rows" in n}
    assert len(norms) == 3 and not any(norms.values()), norms
