"""What the compiler makes of code whose speed or order hangs on it, from the listing of this library's own source."""
import os
import re
import subprocess

import pytest

from paper_2203_10983_amd.build import CSRC, FLAGS, HIPCC


@pytest.fixture(scope="module")
def aggregates(tmp_path_factory):
    """Per instance of spmm_kernel that counts segments, (pieces to a lane, its listing from the count on)."""
    out = tmp_path_factory.mktemp("listing") / "spmm.s"
    subprocess.run([HIPCC, *FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, "spmm.hip"), "-o", str(out)], check=True, capture_output=True)
    found = {}
    for body in re.split(r"\n(?=_ZN3bns\w+:)", out.read_text())[1:]:
        name, body = body.split(":", 1)
        lines = [x.split(";")[0].strip() for x in body.split(".Lfunc_end")[0].splitlines()]
        counts = [i for i, x in enumerate(lines) if x.startswith("global_atomic_add ")]
        if "11spmm_kernel" in name and counts:
            found[name] = int(re.search(r"ILi\d+ELi(\d+)E", name)[1]), lines, counts
    return found


def test_partial_sums_of_a_long_row_are_fetched_together(aggregates):
    """Eight at a time (rows of more than one piece to a lane: four), none waited for before the last of them is asked for; behind the
    count, at the agent's scope (sc1), and the segment's own stores before it, at that scope and waited for."""
    assert len(aggregates) >= 30
    for name, (pieces, lines, counts) in aggregates.items():
        assert len(counts) == 1, name
        loads = [i for i, x in enumerate(lines) if x.startswith("buffer_load_dword") and x.endswith(" sc1")]
        stores = [i for i, x in enumerate(lines) if x.startswith("buffer_store_dword") and x.endswith(" sc1")]
        waits = [i for i, x in enumerate(lines) if x.startswith("s_waitcnt") and "vmcnt" in x]
        assert len(loads) == (8 if pieces == 1 else 4 * pieces) and not any(loads[0] < i < loads[-1] for i in waits), name
        assert stores and stores[-1] < counts[0] < loads[0], name
        assert any(stores[-1] < i < counts[0] and "vmcnt(0)" in lines[i] for i in waits), name
