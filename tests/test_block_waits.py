"""Which kernels wait for another block.

A bounded wait that gives up leaves wrong values behind, so it needs a flag that the
host reads before anyone uses them.  Only the radix sort's look-back has one (the next
build's first read-back), and its flag's message names the sort: no other kernel
polls memory, and the partner search hands its state from launch to launch."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_24688_amd", "csrc")


def _code(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def test_only_the_sort_waits_for_other_blocks():
    waiting = [n for n in sorted(os.listdir(CSRC)) if re.search(r"s_sleep|SpinMax|atomicOr\(a\.err", _code(n))]
    assert waiting == ["dmb_sort.h"]


def test_the_flag_is_the_sorts():
    api = _code("dmb_api.hip")
    assert re.findall(r"\.err = c->os_err", api) == [".err = c->os_err"]
    assert '"radix sort: a look-back wait gave up"' in api
