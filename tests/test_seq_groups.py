"""The sequence kernels' groups of runs are dealt out by arithmetic: none of these kernels takes its work from a counter in memory, which
would serve them one after the other, and their workgroups share no word that the next group's number is handed over in."""
import re


def test_sequence_kernels_have_no_counter(listings):
    text = listings["recurrent_kernels.hip"]
    found = {}
    for m in re.finditer(r"^(_ZN4marl\S*gru_seq\S+):\s", text, re.M):
        found[m.group(1)] = "atomic" in text[m.end() : text.index(".Lfunc_end", m.end())]
    assert sum("gru_seq_fwd" in k for k in found) == 24 and sum("gru_seq_bwd" in k for k in found) == 46
    assert not any(found.values())
