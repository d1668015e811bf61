"""The fine-tuning loss's calls refuse sizes that the matrix-core path cannot address, and workspaces that are too small, before they
launch anything.  A process of its own, in which the library finds tests/launch_count.c's function instead of the runtime's."""
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
p, enough = 1 << 20, int(sys.argv[8])                    # addresses that nothing follows
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


def calls(shim, *args, size=1 << 62):
    out = subprocess.run([sys.executable, "-c", CALLS, shim, *map(str, args), str(size)], cwd=ROOT, check=True, capture_output=True, text=True).stdout
    return tuple(map(int, out.split()))


# T, d, V, n, r: a vocabulary and positions past the 32-bit offsets of a tile
@pytest.mark.parametrize("flags", [0, binding.MIN_WORKSPACE, binding.KEEP_LOGITS])
@pytest.mark.parametrize("shape", [(1, 64, 1 << 23, 1, 8), (1 << 23, 64, 64, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_refused_before_any_launch(shim, shape, flags):
    assert calls(shim, *shape, flags) == (-2, 0, -2, 0)


def test_launches_are_counted(shim):
    rc = calls(shim, 4, 64, 96, 2, 2, 0)
    assert rc[1] > 0 and rc[3] > rc[1]


def second_product_bytes(T, d, V, n, r):
    """Room for a second product of U and y instead of a chunk of fp32 logits: what every call took before logits were stored."""
    def up(x):
        return (x + 255) // 256 * 256
    M, parts = T * n * r, (V + 255) // 256 * 2
    return (up(binding.cp_head_workspace_bytes(binding.make_desc(T, d, V, n, r, binding.BF16), binding.OP_LOSS_FWD))
            + up(M * 4) + up(T * n * 4) + up(M * 8) + up(M * parts * 8))


# the last: so many rows that the chunk of logits, 3 GiB, is less than their statistics
@pytest.mark.parametrize("shape", [(4, 64, 96, 2, 2), (4096, 512, 32000, 4, 8), (16384, 64, 128256, 4, 8)], ids=lambda s: "x".join(map(str, s)))
def test_workspace_without_room_for_logits(shim, shape):
    flags = [0, binding.MIN_WORKSPACE, binding.KEEP_LOGITS]
    query = [binding.cp_head_workspace_bytes(binding.make_desc(*shape, binding.BF16, f), binding.OP_DISTILL_FWD) for f in flags]
    least = [min(query[0], second_product_bytes(*shape)), query[1], query[2]]
    for f, size in zip(flags, least):
        assert calls(shim, *shape, f, size=size - 1)[:2] == (-3, 0)
        rc = calls(shim, *shape, f, size=size)
        assert rc[0] != -3 and rc[1] > 0
