"""The rule for the update kernel that walks whole 128-byte lines (csrc/walk_lines.h), on the CPU: lists and launches that measured
slower with it keep the ordinary kernel, and the lists that the GPU tests of the kernel run are on its side of the rule."""
import os
import shutil
import subprocess

import pytest

from paper_2502_11034_amd import binding as B
import test_gpu_layouts as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ADAMW, LION, MUON = B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION, B.ADAGC_OPT_MUON
MI = 1 << 20
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("walk_lines") / "walk_lines_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2502_11034_amd", "csrc"),
                    os.path.join(ROOT, "tests", "walk_lines_check.cpp"), "-o", exe], check=True)

    def ask(*numbers):
        out = subprocess.run([exe], input=" ".join(str(int(x)) for x in numbers) + "\n", capture_output=True, text=True, check=True, timeout=60)
        return out.stdout.strip() == "1"
    return ask


# optimizer, bf16 gradients, copy, the least elements, the least workgroups of a limited launch (None: never)
@pytest.mark.parametrize("opt,bf16,copy,elems,workgroups", [
    (ADAMW, 0, 1, 3 * MI, 256), (ADAMW, 1, 1, 3 * MI, 256), (ADAMW, 1, 0, 4 * MI, 320), (ADAMW, 0, 0, 6 * MI, 320), (LION, 1, 1, 8 * MI, 640),
    (LION, 0, 1, None, None), (LION, 1, 0, None, None), (LION, 0, 0, None, None), (MUON, 1, 1, None, None)])
def test_limits(rule, opt, bf16, copy, elems, workgroups):
    if elems is None:
        assert not rule(opt, bf16, copy, 10, 1 << 30, 1 << 30, 1 << 20, 1 << 20)
        return
    items = elems // 2048
    assert rule(opt, bf16, copy, 10, elems, elems, items, items)
    assert rule(opt, bf16, copy, 10, elems, elems, workgroups, items)
    assert rule(opt, bf16, copy, 10, elems, elems, 100, 100)                              # a workgroup for each of few, large items
    assert not rule(opt, bf16, copy, 10, elems - 1, elems - 1, items, items)              # too small a list
    assert not rule(opt, bf16, copy, 10, elems, elems, workgroups - 1, items)             # too few workgroups
    assert not rule(opt, bf16, copy, 10, elems, elems // 2, items, items)                 # half of it starts on a line
    n = elems // 16384
    assert rule(opt, bf16, copy, n, elems, elems, items, items)
    assert not rule(opt, bf16, copy, n + 1, elems, elems, items, items)                   # too short tensors


def test_lists_of_the_gpu_tests_are_walked_in_lines(rule):
    for opt, grad, copy, entry, mode, kw, leads in L.LINE_RUNS:
        for lead in leads:
            starts = [lead]
            for n in L.LINES:
                starts.append(starts[-1] + n)
            off = sum(n for a, n in zip(starts, L.LINES) if a % 32)                       # the buffers start on a line
            items = 500                                                                   # or more; only that a limited launch has fewer counts
            assert rule(opt, grad == B.ADAGC_GRAD_BF16, copy, len(L.LINES), sum(L.LINES), off, kw.get("grid_blocks", items), items), \
                (opt, grad, copy, entry, kw, lead)
