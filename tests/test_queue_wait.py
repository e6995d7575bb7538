"""The waits of a compression launch's scanning workgroup, on the host:
tests/pins/queue_wait_check.cpp runs csrc/queue_wait.hpp, which the kernel uses.
While other launches hold the chip, so that no working workgroup has come, the
wait goes on; a taken chunk's size has a limit, and every wait ends."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_waits_of_the_scanning_workgroup(tmp_path):
    out = str(tmp_path / "queue_wait_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", os.path.join(HERE, "pins", "queue_wait_check.cpp"), "-o", out],
                   check=True)
    r = subprocess.run([out], capture_output=True, text=True, check=True).stdout
    f = dict(line.split() for line in r.strip().splitlines())
    assert f["absent-minute"] == "0" and f["wrong"] == "0", r
