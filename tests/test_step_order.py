"""A tracking step that cannot have its pinned words fails before it has
changed anything."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_09214_amd", "csrc")


def body(text, head):
    """The definition that starts with head, up to its closing brace in column 0."""
    at = re.search(re.escape(head) + r"[^;{]*\{", text)
    return text[at.end():text.index("\n}\n", at.end())]


def test_pinned_words_before_the_first_launch():
    """Where the failure cannot be forced the order of the source stands for
    it: the allocation precedes every launch and copy of the step, and the
    compaction at its end makes none but workspace."""
    text = open(os.path.join(CSRC, "track.hip")).read()
    step, end = body(text, 'extern "C" obem_status track_step('), body(text, "static obem_status compact_step(")
    first = min(step.index(w) for w in ("hipLaunchKernelGGL", "hipMemcpyAsync", "bem_solve("))
    assert 0 <= step.find("hipHostMalloc") < first
    assert "hipHostMalloc" not in end and "hipMalloc" not in end
