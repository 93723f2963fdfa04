"""The scalar arithmetic of the tile lookup (csrc/hp_tile.hpp, the kernels' own code) against its plain form, and which launches are
paced, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lookup_arithmetic_is_exact(tmp_path):
    exe, csrc = tmp_path / "walk_lookup", os.path.join(ROOT, "paper_2605_27678_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-Wall",
                        "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "walk_lookup.cpp"), os.path.join(csrc, "hp_plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe), "7"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
