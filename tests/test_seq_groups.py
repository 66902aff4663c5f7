"""The sequence kernels' groups of runs in the listing.  With resident weights they are dealt out by arithmetic: a counter in memory would serve them one
after the other.  With streamed weights thread 0 takes the number of a workgroup's next group from a counter and writes it to one word of LDS, the
wavefronts read it behind a barrier, and the next write is behind another one, whatever the group in between held -- one-step runs have no barrier
of their own in the backward kernel.  So every way from the write back to it passes at least two barriers."""
import re
from collections import deque


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
        assert len(taken) == 1, m.group(1)
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


def test_groups_of_runs(listings):
    text = listings["recurrent_kernels.hip"]
    kernels = set(re.findall(r"^\s*\.amdhsa_kernel (_ZN4marl\S*gru_seq\S+)", text, re.M))
    assert sum("gru_seq_fwd" in k for k in kernels) == 24 and sum("gru_seq_bwd" in k for k in kernels) == 46
    found = barriers_between_slot_writes(text)
    # forward and the backward kernels of either network of the four streamed widths, in runs: <units / 32, 1, false, true ...>
    assert len(found) == 12 and all(re.search(r"gru_seq_(fwd|bwd)_kernelILi[5-8]ELi1ELb0ELb1E", k) for k in found), sorted(found)
    assert {k: n for k, n in found.items() if n < 2} == {}
    for k in kernels - set(found):
        at = text.index("\n" + k + ":")
        assert "atomic" not in text[at : text.index(".Lfunc_end", at)], k
