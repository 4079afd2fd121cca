"""What the first wavefront of a k_history workgroup decides for the others goes through words of LDS.  It runs on after the
barrier behind which they are read, so a word that a later decision also uses can change before a slower wavefront
has read it: with one word for all of them, a workgroup whose tile was the last and whose solver had given way could take part
of its tile through the transform twice.  Held here in the source: a word per decision, one store each, and a barrier
between the store and the reads."""
import os
import re

import pytest

from paper_2410_16029_amd import build as ngbuild

WORDS = ("tile_cmd", "solver_cmd", "taken")


def _source():
    with open(os.path.join(ngbuild.CSRC, "k_history.hip")) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def test_decisions_are_the_listed_words():
    shared = re.search(r"struct HistShared \{(.*?)\};", _source(), re.S).group(1)
    ints = re.findall(r"\bint ([^;]*);", shared)
    assert [w.strip() for line in ints for w in line.split(",")] == list(WORDS)


@pytest.mark.parametrize("word", WORDS)
def test_a_decision_is_stored_once_and_read_behind_a_barrier(word):
    src = _source()
    stores = [m.end() for m in re.finditer(r"\bsh\.%s = " % word, src)]
    reads = [m.start() for m in re.finditer(r"readfirstlane\(sh\.%s\)" % word, src)]
    assert len(stores) == 1 and len(reads) == 1
    assert len(re.findall(r"\bsh\.%s\b" % word, src)) == 2
    assert stores[0] < reads[0] and "__syncthreads();" in src[stores[0]:reads[0]]
