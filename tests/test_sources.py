"""Properties of the device sources that no run can show."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1608_04904_amd", "csrc")


def _code(name):
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*", "", text)


def test_streaming_decides_by_what_the_chain_does_not_write():
    """The streaming and the MD chain of one interval run at once.  The chain
    rewrites the records of the list's members, so who is a member is read from
    the list bits, which the chain does not touch."""
    stream, chain = _code("rmp_stream.h"), _code("rmp_chain.h")
    decisions = re.findall(r"\bgo\[u\] = ([^;]*);", stream)
    assert len(decisions) == 1
    assert "members[u]" in decisions[0] and "st[u]" not in decisions[0]
    assert re.search(r"members\[u\] = [^;]*\blbits\[", stream)
    assert not re.search(r"lbits|list_bits", chain)
