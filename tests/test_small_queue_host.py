"""The queue of a launch that holds whole sweeps, modelled on the host with the
rule of the library (small_team in layout.h): however many blocks come from
the XCD that works, no link is loaded before the sweep before has written it,
and every item is done (CPU)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0904_0642_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "small_queue_host.cpp")


def test_no_link_is_loaded_before_it_was_written(tmp_path):
    exe = str(tmp_path / "small_queue_host")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, SRC, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0
    rows = [tuple(map(int, re.findall(r"\d+", line))) for line in out.stdout.splitlines()]
    assert len(rows) == 36
    for D, groups, blocks, stale, undone, all_stale, all_undone in rows:
        assert stale == undone == all_undone == 0, (D, groups, blocks)
        if blocks == groups:  # eight XCDs: the rule turns nobody away
            assert all_stale == 0
    # the model sees the fault where every block is let in: eight times as many
    # blocks as groups, four slices between two writes
    assert any(D == 2 and blocks == 8 * groups and bad > 0 for D, groups, blocks, _, _, bad, _ in rows)


def test_the_kernel_uses_the_rule():
    src = open(os.path.join(CSRC, "update_split.hip")).read()
    assert "const uint32_t team = small_team(xcc_id(), blockIdx.x);" in src
    assert "s_mine = old == 0u || old == team;" in src and "dim3 grid(8u * s.u.total_blocks)" in src
