"""CPU check of the boxes that the adjoint's second pass stages in LDS: every element a thread reads, those
outside the grid included, lies inside its box, and for threads inside the grid it is the element that a lane
loaded from the stencil's point. For bricks away from the seam of an odd width, for those whose 24-wide rows
reach it, and for those whose 16-wide rows do (whose last column is then outside the grid)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = ("x", "y", "z", "xy", "xz", "yz", "k")


@pytest.fixture(scope="module")
def H(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("harness") / "gather_boxes.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2606_02053_amd", "csrc"), "-o", out,
                    os.path.join(ROOT, "tests", "harness", "gather_boxes.hip")], check=True, capture_output=True)
    return ctypes.CDLL(out)


def taps(place):
    """(shape, element, offset of its point) of every element the thread reads."""
    d2 = (-2, -1, 1, 2)
    for o in (-2, -1, 0, 1, 2):
        yield 0, place[0] + o, (o, 0, 0)
        yield 1, place[1] + 16 * o, (0, o, 0)
        yield 2, place[2] + 64 * o, (0, 0, o)
    for p in d2:
        for q in d2:
            yield 3, place[3] + p + 24 * q, (p, q, 0)
            yield 4, place[4] + p + 96 * q, (p, 0, q)
            yield 5, place[5] + 16 * p + 128 * q, (0, p, q)
    for o in range(-3, 4):
        yield 6, place[0] + o, (o, 0, 0)
    for m, o in enumerate((-3, -2, -1, 1, 2, 3)):
        yield 6, place[6 + m], (0, o, 0)
        yield 6, place[12 + m], (0, 0, o)


@pytest.mark.parametrize("shift24,shift16", [(0, 0), (1, 0), (1, 1)])
def test_reads_stay_in_their_boxes_and_meet_what_was_loaded(H, shift24, shift16):
    loaded = []
    for s in range(7):
        box = {}
        for e in range(64 * H.harness_chunks(s)):
            p = (ctypes.c_int * 3)()
            H.harness_box_point(s, e, -4 + shift24, -shift16, p)
            box[2 * e], box[2 * e + 1] = (p[0], p[1], p[2]), (p[0] + 1, p[1], p[2])
        loaded.append(box)
    for t in range(256):
        tx, ty, tz = t % 16, t // 16 % 4, t // 64
        place = (ctypes.c_int * 18)()
        H.harness_place(tx, ty, tz, shift24, shift16, place)
        for s, element, (dx, dy, dz) in taps(place):
            assert element in loaded[s], (SHAPES[s], (tx, ty, tz), element)
            if not (shift16 and tx == 15):
                assert loaded[s][element] == (tx + dx, ty + dy, tz + dz), (SHAPES[s], (tx, ty, tz), element)
