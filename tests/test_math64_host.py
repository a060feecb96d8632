"""The binary64 pair rotation of the kernels, built for the host, against
extended precision: scattering strengths from zero to infinity at relative
speeds over two hundred orders of magnitude."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2508_06771_amd", "csrc")


def test_half_change_against_extended_precision(tmp_path):
    exe = str(tmp_path / "math64")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas", "-I", CSRC,
                    os.path.join(HERE, "host", "math64_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert "math64 ok" in r.stdout
