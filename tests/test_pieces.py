"""How a launch's workgroups find their columns, checked on the CPU: the table of cells against the
binary search against the run list, over a few hundred layouts; and the pooling jobs of the
replica-spread pass."""
import os
import subprocess

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2506_10911_amd", "csrc")


def test_every_owned_column_is_handed_out_once(tmp_path):
    exe = tmp_path / "piece_driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "piece_driver.cpp"),
                    os.path.join(CSRC, "launch_plan.cpp"), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300,
                         env=dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0"))
    assert run.returncode == 0 and "piece driver: ok" in run.stdout, run.stdout + run.stderr
