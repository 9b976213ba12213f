"""The choice of descriptor slots, walked on the CPU with made-up streams, events and captures (tests/sanitize/ring_walk.cpp says what is checked of every call)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ring") / "ring_walk")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-o", exe,
                           os.path.join(ROOT, "tests", "sanitize", "ring_walk.cpp")])
    return exe


@pytest.mark.parametrize("scenario", ["one_stream", "streams", "per_thread", "recycled", "capture", "idle", "gone", "failing_calls"])
def test_walk(walk, scenario):
    r = subprocess.run([walk, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and f"{scenario} fails=0" in r.stdout, (r.stdout, r.stderr[-2000:])
