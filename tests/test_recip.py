"""The kernels' division of an item index by the segments per chain, through the host's
reciprocal, against Python's: every divisor's quotient boundaries at the ends of its range."""
import ctypes
import os
import random

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_15240_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def div(tmp_path_factory):
    import subprocess
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    so = str(tmp_path_factory.mktemp("recip") / "librecip_host.so")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                        "-I", CSRC, os.path.join(ROOT, "tests", "recip", "recip_host.hip"), "-o", so],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    f = ctypes.CDLL(so).recip_div
    f.argtypes = [ctypes.c_uint32, ctypes.c_uint32]
    f.restype = ctypes.c_uint32
    return f


def test_division_by_the_reciprocal_is_exact(div):
    rng = random.Random(3)
    top = (1 << 32) - 1
    ds = list(range(1, 600)) + [(1 << k) + e for k in range(9, 32) for e in (-1, 0, 1)] + [top, top - 1]
    ds += [rng.randrange(1, top) for _ in range(500)]
    for d in ds:
        qmax = top // d
        qs = {0, 1, 2, qmax, max(qmax - 1, 0), qmax // 2} | {rng.randrange(qmax + 1) for _ in range(4)}
        for n in {min(max(q * d + e, 0), top) for q in qs for e in (-1, 0, 1)} | {top}:
            assert div(n, d) == n // d, (n, d)
