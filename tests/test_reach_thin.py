"""No sample that the renderer's evaluation of a thin, near edge-on surfel takes lies in a tile or quadrant that the
reach test leaves out (the test's own source, compiled for the host)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2411_00771_amd", "csrc")


def test_thin_surfels_keep_their_samples(tmp_path):
    exe = str(tmp_path / "reach_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                           os.path.join(HERE, "reach_check.cpp"), "-o", exe])
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=100).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 18
    for ratio, tilt, taken, missed in rows:
        assert int(taken) > 20_000, (ratio, tilt)
        assert int(missed) == 0, (ratio, tilt, taken, missed)
