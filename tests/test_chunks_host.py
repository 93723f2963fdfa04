"""The lane chunks of every tile, walked on the CPU with the kernels' own index code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walker(tmp_path_factory):
    exe = tmp_path_factory.mktemp("walk") / "walk_chunks"
    csrc = os.path.join(ROOT, "paper_2605_27678_amd", "csrc")

    def build(sanitizers):
        r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", *sanitizers, "-fno-sanitize-recover=all", "-Wall",
                            "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                            os.path.join(ROOT, "tests", "walk_chunks.cpp"), os.path.join(csrc, "hp_plan.cpp"),
                            "-o", str(exe)], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr

    build(["-fsanitize=address,undefined", "-static-libasan"])
    first = subprocess.run([str(exe), "5", "2"], capture_output=True, text=True, timeout=300)
    if first.returncode != 0 and "ASan runtime does not come first" in first.stderr:
        build(["-fsanitize=undefined"])
    return str(exe)


@pytest.mark.parametrize("seed", [3, 4])
def test_every_chunk_of_every_tile_covers_its_bytes_once(walker, seed):
    r = subprocess.run([walker, str(seed), "60"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip() == "plans 60"
