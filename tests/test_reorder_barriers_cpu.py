"""The reorder's gather by the top bits reads a word that other workgroups set
while it runs.  Its workgroups go through barriers afterwards, so all threads
of one have to come to the same decision: one thread reads the word.  Shown on
the source text (a barrier that only some wavefronts reach is not run)."""
import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_07526_amd", "csrc",
                   "pcr_reorder.hip")


def body(text, name):
    at = text.index("{", text.index(f"void {name}("))
    depth = 0
    for k in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[k], 0)
        if depth == 0:
            return text[at:k + 1]
    raise AssertionError(name)


def test_one_thread_reads_the_word_that_changes():
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    gather = " ".join(body(text, "k_gather").split())
    loads = [m.start() for m in re.finditer(r"__hip_atomic_load\(bb \+ kWhole", gather)]
    assert len(loads) == 1
    # thread 0 alone, into LDS, a barrier, then the decision from LDS
    m = re.search(r"if \(threadIdx\.x == 0\) (\w+) = __hip_atomic_load\(bb \+ kWhole[^;]*; __syncthreads\(\); "
                  r"if \(\1\) return;", gather)
    assert m
    assert f"__shared__ uint32_t {m.group(1)};" in gather
    # no thread reads the word in any other way
    assert not re.search(r"bb\[kWhole\](?! = 1;)", gather)
