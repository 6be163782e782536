"""Checks of the kernels' integer logic that need no GPU: the headers that hold it are compiled into small host programs."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_02470_amd", "csrc")


def _build(tmp_path, name):
    exe = str(tmp_path / name)
    b = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, name + ".cc"), "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    return exe


def _run(*cmd):
    return subprocess.run(cmd, capture_output=True, text=True, timeout=120)


def test_reduction_protocol_overwrites_nothing_that_is_still_to_be_read(tmp_path):
    """tri_plan_check.cc at every number of rows; and the check itself: it must refuse the protocol in which work-groups with
    nothing left to publish go on reading."""
    exe = _build(tmp_path, "tri_plan_check")
    r = _run(exe)
    assert r.returncode == 0 and "tri_plan_check ok" in r.stdout, r.stdout
    assert _run(exe, "planted").returncode == 1


def test_placement_on_xcds(tmp_path):
    """xcd_check.cc: which placements of work-groups on XCDs are taken for regular; and a launch that leaves one XCD alone does
    every unit of its work once, by the numbers of its work-groups alone, wherever they run."""
    r = _run(_build(tmp_path, "xcd_check"))
    assert r.returncode == 0 and "xcd_check ok" in r.stdout, r.stdout


def test_slots_of_the_reduction_are_emptied_in_time(tmp_path):
    """tri_slot_check.cc; and the check itself: it must refuse slots that are emptied a step early."""
    exe = _build(tmp_path, "tri_slot_check")
    r = _run(exe)
    assert r.returncode == 0 and "tri_slot_check ok" in r.stdout, r.stdout
    assert _run(exe, "planted").returncode == 1


def test_deferred_shrinks_leave_no_rows_behind(tmp_path):
    """defer_check.cc; and the check itself: it must refuse blocks that are not written when there is room for no more, and
    coefficients in two buffers, of which the side stream reads one while the eigensolve beside it writes it, and halves that move
    on after a captured call, whose replays find them where they were."""
    exe = _build(tmp_path, "defer_check")
    r = _run(exe)
    assert r.returncode == 0 and "defer_check ok" in r.stdout, r.stdout
    assert _run(exe, "planted").returncode == 1
    r = _run(exe, "two")
    assert r.returncode == 1 and "W is not that of the shrinks before the last" in r.stdout, r.stdout
    r = _run(exe, "forgets")
    assert r.returncode == 1 and "another half than the captured one" in r.stdout, r.stdout


def test_a_reduction_that_leaves_64_rows_has_all_it_stores(tmp_path):
    """tri_tail_check.cc; and the check itself: it must refuse a plan where nobody waits for the last step."""
    exe = _build(tmp_path, "tri_tail_check")
    r = _run(exe)
    assert r.returncode == 0 and "tri_tail_check ok" in r.stdout, r.stdout
    assert _run(exe, "planted").returncode == 1


def test_work_space_of_the_selection(tmp_path):
    """select_plan_check.cc; and the check itself: it must refuse a work space for the longest call alone."""
    exe = _build(tmp_path, "select_plan_check")
    r = _run(exe)
    assert r.returncode == 0 and "select_plan_check ok" in r.stdout, r.stdout
    assert _run(exe, "planted").returncode == 1


def test_kept_histograms_are_zero_when_a_run_begins(tmp_path):
    """topm_kept_check.cc; and the check itself: it must refuse a clearing launch that is taken for done when it is only captured, and
    graphs without one."""
    exe = _build(tmp_path, "topm_kept_check")
    r = _run(exe)
    assert r.returncode == 0 and "topm_kept_check ok" in r.stdout, r.stdout
    r = _run(exe, "enqueued")
    assert r.returncode == 1 and "eager: histogram" in r.stdout, r.stdout
    r = _run(exe, "bare")
    assert r.returncode == 1 and "replay: histogram" in r.stdout, r.stdout


def test_events_that_order_streams_release_what_they_order():
    """No run shows a missing release reliably, so the flag is looked for: hipEventDisableSystemFence takes the release away that
    lets a stream see what was written, on another XCD, before the event."""
    made = [(name, line) for name in sorted(os.listdir(CSRC)) if name.endswith((".hip", ".h"))
            for line in open(os.path.join(CSRC, name)) if "hipEventCreateWithFlags" in line or "hipEventRecordWithFlags" in line]
    assert made and not [m for m in made if "DisableSystemFence" in m[1]]
