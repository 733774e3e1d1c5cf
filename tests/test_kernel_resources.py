"""What the built kernels ask of a compute unit, read from the metadata of the library's own code objects: a tile whose LDS is sized for two
workgroups of eight waves per compute unit must need at most 128 registers a lane, whatever rides in its launch, and none of it in scratch
memory."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2305_11624_amd import build

LLVM = "/opt/rocm/llvm/bin"

# (kernels whose two workgroups share a compute unit: 74 and 66 KB of LDS)
SHARED = [r"conv_win_kernelILi128ELi64ELi3E", r"conv_ks_kernelILi32ELi32E"]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    tools = [os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("no LLVM tools")
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(build.LIB, d)
    subprocess.run([tools[0], "--offloading", lib], check=True, cwd=d, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        notes = subprocess.run([tools[1], "--notes", os.path.join(d, f)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.name: +(_Z\S+)", k).group(1)
            found[name] = {w: int(re.search(r"\.%s: +(\d+)" % w, k).group(1))
                           for w in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    return found


@pytest.mark.parametrize("pattern", SHARED)
def test_two_workgroups_share_a_compute_unit(kernels, pattern):
    mine = {n: r for n, r in kernels.items() if re.search(pattern, n)}
    assert len(mine) >= 3   # nothing, a fold-back or a transposed block's on the side
    for n, r in mine.items():
        assert r["vgpr_count"] <= 128 and r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, (n, r)
