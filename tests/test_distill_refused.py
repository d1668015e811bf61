"""The fine-tuning loss's calls refuse sizes that the matrix-core path cannot address before they launch anything.  A process of its
own, in which the library finds tests/launch_count.c's function instead of the runtime's."""
import os
import subprocess
import sys

import pytest

from paper_2410_17765_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CALLS = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2410_17765_amd import binding as b
ds = b.make_desc(*map(int, sys.argv[2:7]), b.BF16, int(sys.argv[7]))
p, enough = 1 << 20, 1 << 62                    # addresses that nothing follows
launches = ctypes.c_int.in_dll(shim, "launches")
rc = [b.lib().cp_head_distill_loss_fwd(ctypes.byref(ds), p, p, p, p, p, p, 0.5, 1.0, p, p, p, enough, None)]
rc.append(launches.value)
rc.append(b.lib().cp_head_distill_loss_bwd(ctypes.byref(ds), p, p, p, p, p, p, None, 1.0, p, p, None, None, None, p, enough, None))
rc.append(launches.value)
print(*rc)
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        from paper_2410_17765_amd import build
        build.build(verbose=False)
    path = str(tmp_path_factory.mktemp("launch_count") / "liblaunch_count.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(ROOT, "tests", "launch_count.c"), "-o", path], check=True)
    return path


def calls(shim, *args):
    out = subprocess.run([sys.executable, "-c", CALLS, shim, *map(str, args)], cwd=ROOT, check=True, capture_output=True, text=True).stdout
    return tuple(map(int, out.split()))


# T, d, V, n, r: a vocabulary and positions past the 32-bit offsets of a tile
@pytest.mark.parametrize("flags", [0, binding.MIN_WORKSPACE, binding.KEEP_LOGITS])
@pytest.mark.parametrize("shape", [(1, 64, 1 << 23, 1, 8), (1 << 23, 64, 64, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_refused_before_any_launch(shim, shape, flags):
    assert calls(shim, *shape, flags) == (-2, 0, -2, 0)


def test_launches_are_counted(shim):
    rc = calls(shim, 4, 64, 96, 2, 2, 0)
    assert rc[1] > 0 and rc[3] > rc[1]
