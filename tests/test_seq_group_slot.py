"""The sequence kernels' groups in the listing: thread 0 writes the number of a workgroup's next group to one word of LDS, the wavefronts read it
behind a barrier, and the next write is behind another one, whatever the group in between held -- one-step runs have no barrier of their own
in the backward kernel.  So every way from the write back to it passes at least two barriers."""
import os
import re
import shutil
import subprocess
from collections import deque

import pytest

from paper_2107_01460_amd import build


def barriers_between_slot_writes(listing):
    """{kernel: the fewest barriers on a way from the write of the group's number back to it}, over the kernels that take groups."""
    found = {}
    for m in re.finditer(r"^(_ZN4marl\S*gru_seq\S+):\s", listing, re.M):
        body = listing[m.end() : listing.index(".Lfunc_end", m.end())]
        lines = [re.sub(r"\s*;.*", "", x.strip()) for x in body.split("\n")]
        lines = [x for x in lines if x and (not x.startswith(".") or re.match(r"\.L\w+:", x))]
        label = {x.rstrip(":"): i for i, x in enumerate(lines) if x.endswith(":")}
        taken = [i for i, x in enumerate(lines) if x.startswith("global_atomic_add ")]
        if not taken:
            continue
        write = next(i for i in range(taken[0], len(lines)) if lines[i].startswith("ds_write"))

        def following(i):
            op = lines[i].split()[0]
            if op == "s_endpgm":
                return []
            if op == "s_branch":
                return [label[lines[i].split()[1]]]
            return [i + 1] + ([label[lines[i].split()[1]]] if op.startswith("s_cbranch") else [])

        fewest, todo = {}, deque((j, 0) for j in following(write))
        while todo:  # ways without a barrier before those with one
            i, n = todo.popleft()
            if fewest.get(i, n + 1) <= n:
                continue
            fewest[i] = n
            if i == write:
                continue
            for j in following(i):
                if lines[i].split()[0] == "s_barrier":
                    todo.append((j, n + 1))
                else:
                    todo.appendleft((j, n))
        found[m.group(1)] = fewest[write]
    return found


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_the_slot_is_read_before_it_is_written_again(tmp_path):
    out = str(tmp_path / "recurrent.s")
    subprocess.check_call(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "recurrent_kernels.hip"), "-o", out])
    with open(out) as f:
        found = barriers_between_slot_writes(f.read())
    assert len(found) == 24 and sum("gru_seq_bwd" in k for k in found) == 16  # eight widths: forward, backward of either network
    assert {k: n for k, n in found.items() if n < 2} == {}
