"""The library's host code on the CPU, over a stand-in for the HIP runtime
(tests/hostrt/hostrt.cpp): the order of the work that it queues on streams, what it
keeps between calls, what it does on a capturing stream, and its plans."""
import os
import shutil
import subprocess

import pytest

from test_gpu_layouts import LAYOUTS
from test_plan import SHAPES, segments

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers not found")
    out = str(tmp_path_factory.mktemp("hostrt") / "hostrt")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__",
                        "-isystem", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2410_15240_amd", "csrc"),
                        os.path.join(ROOT, "tests", "hostrt", "hostrt.cpp"), "-o", out],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    return out


def run(exe, *args, stdin=None):
    r = subprocess.run([exe, *args], input=stdin, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    return r.returncode, r.stdout


@pytest.mark.parametrize("what", ["capture_ragged", "per_thread", "scratch_area", "tag_lanes", "ragged_plan", "ring"])
def test_host_state(exe, what):
    rc, out = run(exe, what)
    assert rc == 0 and ": 0 failures, 0 races" in out, out[-4000:]


MODES = ("decrypt + verify", "CTR", "verify", "keystream", "keystream-apply")


def plans(exe, mode, shapes, cus=256):
    rc, out = run(exe, "plans", stdin="".join("%d %d %d %d\n" % (mode, l, c, cus) for l, c in shapes))
    assert rc == 0
    keys = ("lanes_log2", "seg_log2", "segs_full", "segs_last", "items")
    return [dict(zip(keys, (int(v) for v in line.split()))) for line in out.splitlines()]


@pytest.mark.parametrize("cus", [256, 80, 1])
@pytest.mark.parametrize("mode", range(5), ids=MODES)
def test_every_modes_segments_partition_the_chains(exe, mode, cus):
    """test_plan.py's checks of decrypt + verify, for the plans of every mode."""
    for (length, chain), p in zip(SHAPES, plans(exe, mode, SHAPES, cus)):
        n, qc = -(-length // chain), chain // 16
        q_last = -(-(length - (n - 1) * chain) // 16)
        g = 1 << p["seg_log2"]
        assert p["lanes_log2"] in (4, 5, 6)
        assert p["segs_full"] == -(-qc // g) and p["segs_last"] == -(-q_last // g)
        assert p["items"] == (n - 1) * p["segs_full"] + p["segs_last"] < 1 << 32
        assert p["items"] == n or p["items"] + n <= 230240   # the partial slots of a cut launch
        for q, S in ((qc, p["segs_full"]), (q_last, p["segs_last"])):
            if S > 1 << 16:
                continue
            segs = segments(p, q, S)
            assert segs[0][0] == 0 and segs[-1][1] == q
            assert all(a[1] == b[0] for a, b in zip(segs, segs[1:]))
            assert all(0 <= b < e <= q and e - b <= g for b, e in segs)
            assert all(e - b == g for b, e in segs[1:])


@pytest.mark.parametrize("mode", range(5), ids=MODES)
def test_the_gpu_layouts_reach_every_kernel(exe, mode):
    """The layouts that the GPU tests compare with the oracle take each mode through every
    lane count, with whole chains and with segments."""
    shapes = [(l, c) for l, c, _, _ in LAYOUTS]
    got = plans(exe, mode, shapes)
    reached = {(p["lanes_log2"], p["items"] > -(-l // c)) for (l, c), p in zip(shapes, got)}
    assert reached == {(ll, cut) for ll in (4, 5, 6) for cut in (False, True)}
    if mode == 0:
        for (l, c, _, want), p in zip(LAYOUTS, got):
            wave_items = -(-p["items"] // (64 >> p["lanes_log2"]))
            assert (p["lanes_log2"], p["items"] > -(-l // c), wave_items > 4096) == want
