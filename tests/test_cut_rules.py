"""The rules by which launches of row-strided plans ([S,B,H] order) are cut and shaped, on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe, csrc = tmp_path_factory.mktemp("rules") / "walk_rules", os.path.join(ROOT, "paper_2605_27678_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-Wall",
                        "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "walk_rules.cpp"), os.path.join(csrc, "hp_plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr

    def run(check, seed=11, plans=60):
        r = subprocess.run([str(exe), check, str(seed), str(plans)], capture_output=True, text=True, timeout=600)
        assert r.returncode == 0 and r.stdout.strip() == f"plans {plans}", r.stdout + r.stderr
    return run


def test_rules_of_a_launch_do_not_read_the_segments(walk):
    walk("once")


def test_tables_of_cut_rows_are_made_in_place(walk):
    walk("made_in_place")


def test_shapes_follow_what_is_launched(walk):
    walk("shapes", plans=1)


def test_launches_that_lose_by_it_are_not_cut(walk):
    walk("cuts", plans=1)


def test_grids_of_the_largest_launches_of_lines_stay_below_2_to_the_32_work_items(walk):
    walk("grids", plans=1)


def test_text_gradients_of_images_that_lie_alike_take_bands(walk):
    walk("alike", plans=1)
