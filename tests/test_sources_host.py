"""What the compiler can say of the sources without building them."""
import glob
import os
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
