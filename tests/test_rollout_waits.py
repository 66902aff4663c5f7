"""The step loops of the rollout kernels in the listing: no wavefront meets a barrier with a write to LDS still on its way.

The env wavefront writes the windows of step t + 1 at the end of the loop and the others read them after the barrier at its
head.  The compiler once left the wait for those writes out on the back edge; a run then now and then used an old window."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2107_01460_amd import build


def pending_writes_at_barriers(listing):
    """{kernel: [instruction index of each s_barrier that some path reaches with an LDS write not waited for]}."""
    found = {}
    for m in re.finditer(r"^(_ZN4marl\S*rollout\S+):\s", listing, re.M):
        body = listing[m.end() : listing.index(".Lfunc_end", m.end())]
        lines = [re.sub(r"\s*;.*", "", x.strip()) for x in body.split("\n")]
        lines = [x for x in lines if x and (not x.startswith(".") or re.match(r"\.L\w+:", x))]
        label = {x.rstrip(":"): i for i, x in enumerate(lines) if x.endswith(":")}
        # state: the LDS (and scalar) accesses issued after the oldest pending write kind, or None if no write is pending
        state, todo, bad = {0: None}, [0], set()
        while todo:
            i = todo.pop()
            op, s = lines[i].split()[0], state[i]
            if op == "s_barrier" and s is not None:
                bad.add(i)
            if op.startswith("ds_write"):
                s = 0
            elif s is not None and (op.startswith("ds_") or op.startswith("s_load")):
                s = min(s + 1, 63)
            elif s is not None and op == "s_waitcnt":
                w = re.search(r"lgkmcnt\((\d+)\)", lines[i])
                if w and int(w.group(1)) <= s:
                    s = None
            to = [] if op == "s_endpgm" else [i + 1]
            if op == "s_branch":
                to = [label[lines[i].split()[1]]]
            elif op.startswith("s_cbranch"):
                to.append(label[lines[i].split()[1]])
            for j in (j for j in to if j < len(lines)):
                new = s
                if j in state:
                    new = state[j] if s is None else s if state[j] is None else min(s, state[j])
                if j not in state or new != state[j]:
                    state[j] = new
                    todo.append(j)
        found[m.group(1)] = sorted(bad)
    return found


def test_dataflow_sees_a_missing_wait():
    loop = "_ZN4marl9rollout_k: ; @k\n\ts_waitcnt vmcnt(0)\n.LBB0_1:\n%s\ts_barrier\n\tds_write_b32 v0, v1\n\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n.Lfunc_end0:\n"
    assert pending_writes_at_barriers(loop % "")["_ZN4marl9rollout_k"] == [2]
    assert pending_writes_at_barriers(loop % "\ts_waitcnt lgkmcnt(0)\n")["_ZN4marl9rollout_k"] == []


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_no_lds_write_is_pending_at_a_barrier(tmp_path):
    out = str(tmp_path / "rollout.s")
    subprocess.check_call(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "rollout_v3.hip"), "-o", out])
    with open(out) as f:
        found = pending_writes_at_barriers(f.read())
    assert any("rollout_train" in k for k in found) and any("rollout_eval" in k for k in found)
    assert {k: v for k, v in found.items() if v} == {}
