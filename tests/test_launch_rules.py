"""The host's rules for launches (csrc/adagc_internal.h) on the CPU, compiled into small drivers with the HIP runtime's headers but without
the runtime."""
import os
import shutil
import subprocess

import pytest

from paper_2502_11034_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="needs g++ and the HIP headers")


def _driver(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2502_11034_amd", "csrc"), "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe], check=True)
    return exe


def test_a_stream_that_cannot_be_asked_leaves_no_error_behind(tmp_path):
    """The NULL stream while another stream is captured: the question fails, the step's launches must not report that."""
    res = subprocess.run([_driver(tmp_path, "issues_now_check")], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout


ADAMW, LION = B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION
LAYER = [128, 128, 49152, 16384, 65536, 65536]
# list, and whether a single launch is the quicker step with AdamW and Lion on f32 and bf16 gradients, on 256 compute units
ONE_LAUNCH = {
    "one element": ([1], True, True, True, True), "tensors of one item": ([2048] * 288, True, True, True, True),
    "one more of them": ([2048] * 289, False, False, False, False), "tiny tensors": ([500] * 1152, True, True, True, True),
    "short chunks": ([3693] * 46, True, True, True, True), "a workgroup to a compute unit": ([2049] * 128, True, True, True, True),
    "one more": ([2049] * 128 + [600], False, False, False, False),
    "a two-layer transformer": ([131072] + LAYER * 2 + [128], True, False, False, False), "whole chunks": ([16384] * 32, True, False, False, False),
    "ends of chunks": ([14500] * 27, True, True, False, False), "half of them whole": ([16384, 14500] * 8, True, True, False, False),
    "more than half": ([16384, 14500] * 8 + [16384], True, False, False, False),
    "a compute unit for all but ten": ([28200] * 17, False, False, False, False),
    "16 chunks": ([16 * 16384], True, False, False, False), "17 chunks": ([16 * 16384 + 1], False, False, False, False)}


@pytest.fixture(scope="module")
def one_launch(tmp_path_factory):
    exe = _driver(tmp_path_factory.mktemp("one_launch"), "one_launch_check")

    def ask(optimizer, bf16, compute_units, numels):
        line = " ".join(str(x) for x in [optimizer, bf16, compute_units, len(numels)] + numels)
        return subprocess.run([exe], input=line, capture_output=True, text=True, check=True, timeout=60).stdout.strip() == "1"
    return ask


@pytest.mark.parametrize("name", ONE_LAUNCH)
def test_a_single_launch_where_the_gpu_is_done_sooner(one_launch, name):
    numels, *pays = ONE_LAUNCH[name]
    assert [one_launch(o, b, 256, numels) for o in (ADAMW, LION) for b in (0, 1)] == pays


def test_a_single_launch_that_the_device_holds_at_once(one_launch):
    """A part of a GPU has fewer compute units: workgroups that are not running keep those that are waiting for them."""
    assert one_launch(ADAMW, 0, 64, [2048] * 72) and not one_launch(ADAMW, 0, 64, [2048] * 73)
    assert one_launch(ADAMW, 0, 64, [16384] * 8) and not one_launch(ADAMW, 0, 64, [16384] * 9) and not one_launch(ADAMW, 0, 32, [16384])
    assert not one_launch(ADAMW, 0, 0, [1])


def test_whole_lines_with_the_vectors_in_flight_that_a_library_ever_chose(tmp_path):
    """1, 2 and 4 vectors: a caller who sets the number that has been the library's own keeps the whole lines."""
    out = subprocess.run([_driver(tmp_path, "lines_unroll_check")], capture_output=True, text=True, check=True, timeout=60).stdout
    assert out.split("\n")[:2] == ["0 1 1", "0 1 0"]


# optimizer, unroll, update_split, grid_blocks: vectors in flight, work items of a chunk
UPDATE_ITEMS = [(ADAMW, 0, 0, 0, 2, 8), (ADAMW, 0, 1, 0, 4, 1), (ADAMW, 0, 2, 0, 4, 2), (ADAMW, 0, 4, 0, 4, 4), (ADAMW, 4, 0, 0, 4, 4),
                (ADAMW, 2, 0, 0, 2, 8), (ADAMW, 1, 0, 0, 1, 8), (ADAMW, 2, 4, 0, 2, 4), (ADAMW, 1, 16, 0, 1, 16), (ADAMW, 0, 0, 320, 4, 4),
                (ADAMW, 2, 0, 320, 2, 8), (ADAMW, 0, 2, 320, 4, 2), (LION, 0, 0, 0, 2, 8), (LION, 0, 4, 0, 2, 4), (LION, 0, 1, 0, 2, 1),
                (LION, 4, 0, 0, 4, 4), (LION, 1, 16, 0, 1, 16), (LION, 0, 0, 320, 2, 8)]


def _update_items(tmp_path, asked):
    """Per line (optimizer, unroll, update_split, grid_blocks, elements): vectors in flight, work items of a chunk, and the most elements in
    full items of a list whose rule is in the update kernel."""
    out = subprocess.run([_driver(tmp_path, "update_items_check")], input="\n".join("%d %d %d %d %d" % x for x in asked) + "\n",
                         capture_output=True, text=True, check=True, timeout=60).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_a_chosen_split_or_grid_has_the_vectors_in_flight_that_suit_it(tmp_path):
    got = _update_items(tmp_path, [x[:4] + (1 << 20,) for x in UPDATE_ITEMS])
    assert [x[:2] for x in got] == [x[4:] for x in UPDATE_ITEMS]
    # at the same list whatever the items; 1024 items where a workgroup walks many, one after the other
    assert [x[2] for x in got] == [1024 * 16384 // x[5] if x[3] else (16 if x[0] == LION else 32) << 20 for x in UPDATE_ITEMS]


def test_the_largest_launches_have_larger_items(tmp_path):
    """From 200 Mi elements AdamW has 4 vectors in flight and items of 4096 elements, unless the caller chooses."""
    at = 200 << 20
    asked = [(ADAMW, 0, 0, 0, at - 1, 2, 8), (ADAMW, 0, 0, 0, at, 4, 4), (ADAMW, 0, 0, 0, 1 << 34, 4, 4), (ADAMW, 2, 0, 0, at, 2, 8),
             (ADAMW, 0, 2, 0, at, 4, 2), (ADAMW, 1, 0, 0, at, 1, 8), (LION, 0, 0, 0, 1 << 34, 2, 8)]
    assert [x[:2] for x in _update_items(tmp_path, [x[:5] for x in asked])] == [x[5:] for x in asked]


MIB = 1 << 20
GROUP = 64 * MIB              # elements of a full group, f32
# list, sizes of its groups in tensors
GROUPS = [([1], [1]), ([GROUP, 1], [2]), ([1, GROUP], [2]), ([GROUP // 2] * 4 + [1], [2, 2, 1]), ([GROUP // 2 + 1] * 3, [1, 1, 1]),
          ([GROUP + 7, 4096] * 3, [2, 2, 2]), ([4096, 4096, 2 * GROUP, 4096, GROUP + 7, 4096], [4, 2]), ([9 * GROUP] + [1000] * 7, [8]),
          ([GROUP, GROUP // 16], [2]), ([GROUP, GROUP // 16 + 1], [1, 1]), ([GROUP // 16, GROUP], [2]), ([GROUP // 16 + 1, GROUP], [1, 1]),
          ([GROUP] + [GROUP // 32] * 3, [3, 1]), ([GROUP * 15 // 16, GROUP // 16, 1], [2, 1]), ([MIB] * 130, [64, 64, 2])]


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    exe = _driver(tmp_path_factory.mktemp("groups"), "groups_check")

    def ask(numels):
        line = " ".join(str(x) for x in [GROUP, len(numels)] + numels)
        ends = [int(x) for x in subprocess.run([exe], input=line, capture_output=True, text=True, check=True, timeout=60).stdout.split()]
        assert ends[-1] == len(numels)
        return [b - a for a, b in zip([0] + ends, ends)]
    return ask


@pytest.mark.parametrize("numels, sizes", GROUPS, ids=range(len(GROUPS)))
def test_small_tensors_beside_a_large_one_are_no_group_of_their_own(groups, numels, sizes):
    assert groups(numels) == sizes
