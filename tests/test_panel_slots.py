"""The LDS slots of the pivoting panel (d > 256), on the CPU: a model of one
step, in which the wave owning the pivot's column runs as far ahead of the
others as the barriers let it, reads the slots by the rule the kernel is
compiled with.  The model is shown to catch a reused slot on a rule of its own
(as many slots as half a panel has entries)."""

import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2105_11004_amd" / "csrc"

DUMP = r"""
#include <cstdio>
#include "panel_slots.h"
int main() {
  for (int sh = lev::kPanelHalf; sh <= lev::kPanel; sh += lev::kPanel - lev::kPanelHalf)
    for (int j = 0; j < lev::kPanel; ++j)
      std::printf("%d %d %d %d %d\n", sh, j, lev::panel_stride(sh), lev::panel_slot(sh, j),
                  (int)lev::panel_posted(sh, j));
}
"""


def spoiled_steps(slots, posted, half):
    """Steps whose straight slot reads can miss an entry: entry t is to be
    found in slots[t] just before and just after the step's own write."""
    bad = []
    column = {}
    for j in range(len(slots)):
        ahead = {**column, slots[j]: j}  # the owner has written entry j already
        wanted = range(half if posted[j] else 0, j)
        if any(m.get(slots[t]) != t for m in (column, ahead) for t in wanted):
            bad.append(j)
        column = ahead
    return bad


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "dump.cpp").write_text(DUMP)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(d / "dump.cpp"), "-o", str(d / "dump")], check=True)
    rows = [tuple(map(int, line.split())) for line in subprocess.run([str(d / "dump")], check=True, capture_output=True,
                                                                     text=True).stdout.splitlines()]
    return {sh: [r for r in rows if r[0] == sh] for sh in (16, 32)}


@pytest.mark.parametrize("sh", [16, 32])
def test_no_step_reads_a_slot_written_without_a_barrier(rule, sh):
    rows = rule[sh]
    assert [r[1] for r in rows] == list(range(32))
    assert all(0 <= r[3] < r[2] for r in rows)  # inside the column's room
    assert spoiled_steps([r[3] for r in rows], [r[4] for r in rows], 16) == []


def test_model_catches_a_slot_reused_one_step_early():
    assert spoiled_steps([j % 16 for j in range(32)], [j > 16 for j in range(32)], 16) == [16]
