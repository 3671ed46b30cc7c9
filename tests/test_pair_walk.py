"""The lists of (sequence, tile) pairs that a per-sequence bf16 launch's workgroups walk, on the host: the kernel's own walk over
the launch's own plan meets every pair once, for tile counts of every remainder of eight, few and many sequences (more than are
sorted by length), lengths that are equal, ragged, empty and dominated by one, and grids that keep a budget of compute units."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_23353_amd import build as libbuild

TESTS = os.path.dirname(os.path.abspath(__file__))
SAN = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
       "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]


def test_every_pair_is_met_once(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    objs = []
    for src in (os.path.join(libbuild.CSRC, "contraction_plan.cpp"), os.path.join(TESTS, "pair_walk_driver.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        r = subprocess.run(["hipcc", *[f for f in libbuild.FLAGS if f != "-O3"], "-O1", "-g", *SAN, "-x", "hip", "-c", src, "-o", objs[-1]],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
    exe = str(tmp_path / "pair_walk_driver")
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-fsanitize=address", "-fsanitize=undefined", "-fno-gpu-sanitize", "-o", exe,
                        *objs], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0 and "FAIL" not in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
    done = re.search(r"done failures=0 dealt=(\d+) ranges=(\d+) single=(\d+) alone=(\d+)", r.stdout)
    assert done and all(int(g) >= 10 for g in done.groups()), r.stdout[-300:]     # every arrangement was walked
