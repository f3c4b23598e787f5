"""Host-side: which instructions the sources write by hand.  The compiler
counts the wait states between a vector instruction that writes a scalar
register and the instructions that use it (two for a vector use, five for a
memory instruction, four for a lane select), but does not look into inline
assembly: such instructions come from its builtins."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1412_3387_amd", "csrc")
SCALAR_WRITERS = re.compile(r"v_readfirstlane|v_readlane|v_cmpx?_")


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        txt = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm\b[^;]*;", txt):
            yield os.path.basename(path), m.group(0)


def test_the_sources_hold_inline_assembly():
    assert len(list(statements())) >= 5


def test_no_vector_result_in_a_scalar_register():
    for name, text in statements():
        assert not SCALAR_WRITERS.search(text), (name, text)


def test_the_unused_carry_of_the_wide_product():
    """The one statement with a scalar output beside its result: the carry of
    a 64-bit product, which nothing reads."""
    outs = [(n, t) for n, t in statements() if re.search(r'"=s"', t)]
    assert [n for n, _ in outs] == ["device.h"] and "v_mad_u64_u32" in outs[0][1]
    txt = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "device.h")).read())
    body = re.search(r"uint64_t mul_wide\(.*?\n\}", txt, flags=re.S).group(0)
    assert len(re.findall(r"\bcarry\b", body)) == 2  # declared, and named as the output
