"""The framed build's tile indices in LDS: the words that every wave reads
ahead of the tile loop are none that a wave writes inside it, because no
barrier that all launches run lies between (one wave may be through its first
tile's staging before another has read its first index)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1412_3387_amd", "csrc")


def test_first_indices_are_not_overwritten_by_the_loop():
    with open(os.path.join(CSRC, "nlist.hip")) as f:
        body = f.read().split("void k_build_fast(", 1)[1]
    ahead, loop = body.split("for (;;) {", 1)
    reads = list(re.finditer(r"uni\(sh\.grab\[(\w+)\]\)", ahead))
    writes = re.findall(r"sh\.grab\[(\w+)\] = ", loop)
    assert reads and writes
    # a barrier of every launch behind the reads would order them as well; the
    # one that is there belongs to bonded contexts
    tail = re.sub(r"if constexpr \(EXCL\) \{[^{}]*\}", "", ahead[reads[-1].end():])
    assert "lds_barrier();" in tail or not {m.group(1) for m in reads} & set(writes)
