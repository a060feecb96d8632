"""The staged new electrons of the DSMC step are all written out, whichever
thread of the workgroup runs first: a host build of the staging code, its
threads stepped one after another between barriers."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2508_06771_amd", "csrc")


def test_every_staged_electron_is_written(tmp_path):
    exe = str(tmp_path / "dsmc_flush")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "host", "dsmc_flush_driver.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert "dsmc flush ok" in r.stdout
