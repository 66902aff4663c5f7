"""The kernels' barriers in the listing: no wavefront meets one with a write to LDS still on its way.

The rollouts' env wavefront writes the windows of step t + 1 at the end of the loop and the others read them after the barrier at its
head.  The compiler once left the wait for those writes out on the back edge; a run then now and then used an old window.  The
sequence kernels hand their states over in loops too, and take their next group behind a barrier at a loop's head."""
import re

import pytest

from paper_2107_01460_amd import build


def pending_writes_at_barriers(listing):
    """{kernel: [instruction index of each s_barrier that some path reaches with an LDS write not waited for]}."""
    found = {}
    kernels = set(re.findall(r"^\s*\.amdhsa_kernel (\S+)", listing, re.M))
    for m in re.finditer(r"^(_Z\S+):\s", listing, re.M):
        if m.group(1) not in kernels:
            continue
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
    loop = "_ZN4marl9rollout_k: ; @k\n\ts_waitcnt vmcnt(0)\n.LBB0_1:\n%s\ts_barrier\n\tds_write_b32 v0, v1\n\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n.Lfunc_end0:\n\t.amdhsa_kernel _ZN4marl9rollout_k\n"
    assert pending_writes_at_barriers(loop % "")["_ZN4marl9rollout_k"] == [2]
    assert pending_writes_at_barriers(loop % "\ts_waitcnt lgkmcnt(0)\n")["_ZN4marl9rollout_k"] == []


# what each translation unit's loops with barriers are in
KERNELS = {"api.hip": [], "env_kernels.hip": ["env_step"], "gae_kernels.hip": [], "policy_kernels.hip": ["fused_forward_small", "split_net", "bf16_net_pair"],
           "ppo_kernels.hip": ["fused_train_pair", "split_net", "bf16_net", "bf16_wgrad", "gemm_split", "reduce_partials"],
           "recurrent_kernels.hip": ["gru_seq_fwd", "gru_seq_bwd", "gru_actor_step", "seq_runs", "gemm_split"],
           **{f"rollout_v{v}.hip": ["rollout_train", "rollout_eval"] for v in (3, 5, 7)}}


@pytest.mark.parametrize("src", build.SOURCES)
def test_no_lds_write_is_pending_at_a_barrier(listings, src):
    found = pending_writes_at_barriers(listings[src])
    for name in KERNELS[src]:
        assert any(name in k for k in found), name
    assert {k: v for k, v in found.items() if v} == {}
