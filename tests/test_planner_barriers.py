"""Order of the planner's accesses to words of LDS that its waves share, read off its source: which way a wave goes must not hang
on a word that another wave may already have set back.  (A missing barrier shows on a device only when a wave is late.)"""
import os
import re

import pytest

from conftest import ROOT

SOURCE = os.path.join(ROOT, "paper_2605_06046_amd", "csrc", "fea_planner.hip")


def _plan_kernel():
    """The kernel's body without comments, and without the statements that only run where the planner finds the runs itself."""
    with open(SOURCE) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    text = text[text.index("void plan_kernel("):]
    text = text[:text.index("\n}\n")]
    while (m := re.search(r"if \(!a\.pre\) \{", text)):
        depth, end = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[end], 0)
            end += 1
        text = text[:m.start()] + text[end:]
    return text


@pytest.mark.parametrize("before,after", [
    (r"s_nflw == 0", r"s_nflw = 0; s_nest"),                                  # whether anything is shared, and the word taken for the next count
    (r"\n    reset_groups\(0\);", r"atomicMin\(&u\.c\.run\[lead1"),           # the groups' words, and the counts in them
])
def test_a_barrier_stands_between(before, after):
    text = _plan_kernel()
    first = re.search(before, text)
    assert first, before
    then = re.search(after, text[first.end():])
    assert then, after
    between = text[first.end():first.end() + then.start()]
    # (the whole-history branch has barriers of its own, which the waves that do not take it do not pass)
    branch = between.find("return;") if "s_nflw" in before else -1
    between = between[branch + 1:]
    assert re.search(r"\n    (if \(a\.pre\) )?__syncthreads\(\);", between), f"no barrier between {before!r} and {after!r}"
