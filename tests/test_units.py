"""Feature rows read in 16-byte units (csrc/nlb_units.h), on the CPU: every
unit inside its row, every column used once and with its own weight, for
every width of 4 to 512 values."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_units_cover_every_width(tmp_path):
    exe = tmp_path / "units_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-Wno-unknown-pragmas",
                    "-I", os.path.join(ROOT, "paper_2402_01964_amd", "csrc"),
                    "-o", str(exe), os.path.join(ROOT, "tests", "units_check.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout + out.stderr
