"""The colour table's flush: two neighbouring lanes read one slot (with packed
sums the same word) and one of them clears it.  Between the reads and the clear
stands a wavefront barrier, so that their order does not rest on how the compiler
happens to place them.  Shown on the source text."""
import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_07526_amd", "csrc",
                   "pcr_render.hip")


def test_slot_is_read_by_both_lanes_before_it_is_cleared():
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    body = text[text.index("void flush_sum_pairs("):]
    body = body[:body.index("\n}")]
    reads = [body.index("L.tag[h];"), body.index("L.val[h].words()")]
    clears = [body.index("L.val[h].clear()"), body.index("L.tag[h] = kEmptyPid")]
    assert max(reads) < body.index("Team<true>::barrier();") < min(clears)
