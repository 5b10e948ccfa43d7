"""What the compiler can say of the sources without building them."""
import glob
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_1510_06706_amd import build


def test_no_value_is_changed_and_read_without_an_order():
    """An expression that changes a variable beside another use of it has no defined value."""
    sources = sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))
    assert sources

    def check(source):
        cmd = [build.HIPCC] + build.FLAGS + ["-Werror=unsequenced", "--offload-host-only", "-fsyntax-only", source]
        return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)

    with ThreadPoolExecutor(max_workers=8) as pool:
        for source, r in zip(sources, pool.map(check, sources)):
            assert r.returncode == 0, (source, r.stdout[-2000:])


# Vector registers that an instance of the split direct kernel may keep in memory: 256 are all there are, and 5 x 2 tiles take two more.
SPILLED = {(1, 8): 0, (2, 2): 0, (2, 8): 0, (3, 6): 0, (4, 3): 0, (5, 1): 0, (5, 2): 2}


def test_the_largest_tiles_keep_their_registers(tmp_path):
    """The direct forward and backward kernel, two waves on a SIMD: what its tiles leave of the registers has to hold the rest."""
    source = tmp_path / "instances.hip"
    source.write_text('#include "direct_split_impl.h"\n' + "".join(
        "template __global__ void znn::split::k_conv_split<%d, %d, 4>(znn::split::SplitTile);\n" % tiles for tiles in SPILLED))
    cmd = [build.HIPCC] + build.FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", str(source), "-o", str(tmp_path / "instances.o")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    spilled = {}
    for line in r.stdout.splitlines():
        name = re.search(r"Function Name: \S*k_conv_splitILi(\d+)ELi(\d+)ELi4E", line)
        if name:
            tiles = (int(name[1]), int(name[2]))
        count = re.search(r"VGPRs Spill: (\d+)", line)
        if count:
            spilled[tiles] = int(count[1])
    assert spilled.keys() == SPILLED.keys()
    assert all(spilled[tiles] <= SPILLED[tiles] for tiles in SPILLED), spilled
