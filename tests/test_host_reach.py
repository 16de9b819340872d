"""The bound behind the render kernel's key windows (csrc/reach.h, plain arithmetic that the kernel shares) on the CPU:
no pixel that a body's vertices can reach lies outside it, over random cameras, poses, shapes of either sign, collapsed and
stretched rotations and units of length from 2^-125 to 2^124."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_vertex_reaches_a_pixel_outside_the_bound(tmp_path):
    exe = str(tmp_path / "reach_check")
    csrc = os.path.join(ROOT, "paper_2502_00021_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(csrc, "scene.cpp"), os.path.join(ROOT, "tests", "reach_check_main.cpp"), "-o", exe])
    r = subprocess.run([exe, "30000"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    total, seen, outside, near = (int(x) for x in r.stdout.split()[1:])
    assert total == 120000 and seen > 20000 and outside > 10000 and near > 5000, r.stdout
