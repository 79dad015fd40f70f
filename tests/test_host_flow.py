"""The launch sequence of the library's calls, followed on the host (CPU only): tests/fake_hip.cpp stands in for the
HIP runtime, so a case can bring about totals, sizes and refused allocations that no frame here reaches, and look at
what a call launched, allocated and left in flight."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    import paper_2501_12581_amd as P
    P.lib()
    out = str(tmp_path_factory.mktemp("flow") / "fake_hip")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-rdynamic",
                           os.path.join(ROOT, "tests", "fake_hip.cpp"), "-ldl", "-o", out])
    return out, P.LIB_PATH


def _run(program, case, *args):
    res = subprocess.run([program[0], program[1], case] + [str(a) for a in args], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0, (case, args, res.returncode, res.stdout[-2000:], res.stderr[-2000:])
    return res.stdout


@pytest.mark.parametrize("case", ["refused_noalloc", "refused_overflow", "counted_pairs"])
def test_a_call_that_renders_nothing_leaves_nothing_in_flight(program, case):
    """A refused frame and a count of pairs return after the bins' fill pass, which starts before the totals are
    known, has ended: the next call may use the same buffers on any stream."""
    _run(program, case)


def test_pair_numbers_that_are_gone_are_made_again(program):
    """A larger frame frees the pair numbers and cannot have its own: the smaller frame, repeated, does not trust
    the new buffer's contents."""
    _run(program, "lost_numbers")


def test_a_frame_without_room_for_its_pairs_goes_per_tile(program):
    """No frame is refused for a buffer that only one of stage one's two forms needs."""
    _run(program, "refused_pair_buffers")


@pytest.mark.parametrize("case", ["large_images", "large_pair_lists", "thin_images"])
def test_launches_fit_however_large_the_output(program, case):
    """No launch of 2^32 threads in one dimension, which the runtime refuses."""
    _run(program, case)


@pytest.mark.parametrize("w,h,n_sub,tets_each,form", [
    (384, 384, 1, 1, "tiles"), (392, 384, 1, 1, "pairs"), (768, 768, 1, 1, "pairs"), (776, 768, 1, 1, "tiles"),
    (8, 8, 1, 1, "tiles"), (8, 8, 2, 1, "pairs"), (768, 768, 2, 1, "pairs"), (776, 768, 3, 9000, "tiles"),
    (776, 768, 4, 1, "tiles"), (776, 768, 4, 9311, "tiles"), (776, 768, 4, 9312, "pairs"),
    (776, 768, 8, 1, "pairs"), (1024, 1024, 8, 1, "pairs"), (1032, 1024, 8, 9000, "tiles"),
])
def test_stage_one_takes_pairs_where_the_rule_says(program, w, h, n_sub, tets_each, form):
    """The form on both sides of every line of the rule, for the global sum and for per-subdomain images."""
    assert _run(program, "route", w, h, n_sub, tets_each).split() == [form, form]


def test_the_scan_of_very_many_bins_has_two_levels(program):
    """The work of the bins' scan grows with the bins, not with their square."""
    _run(program, "many_bins")


def test_the_buffer_of_the_pairs_moments_is_bounded(program):
    """256 MiB at most, slack included, and room for a view with more pairs."""
    _run(program, "moments_buffer")


def test_kept_pieces_are_not_taken_for_another_mesh_at_the_same_address(program):
    """A mesh freed and another loaded where it was: stage two walks the new one."""
    _run(program, "kept_mesh")


def test_a_stream_under_the_callers_capture_reads_nothing_back(program):
    """Refused where totals are needed, and kernels only where the bins are at hand."""
    _run(program, "users_capture")
