"""What the compiler made of the kernels, read from the metadata of the library that was built from this tree: no kernel spills
vector registers or has a stack (a stack needs memory that the runtime provides at dispatch, and reloads wait for
every load in flight), and all keep to the registers that their workgroups per CU leave."""
import os
import re

import paper_1901_10008_amd as sk

LIB = os.path.join(os.path.dirname(sk.__file__), "libsuperkernel.so")


def _uint(b, at):
    """The MessagePack unsigned integer at `at`."""
    if b[at] < 0x80:
        return b[at]
    n = {0xCC: 1, 0xCD: 2, 0xCE: 4}[b[at]]
    return int.from_bytes(b[at + 1:at + 1 + n], "big")


def _all(blob, key):
    return [_uint(blob, m.end()) for m in re.finditer(re.escape(key), blob)]


def test_no_kernel_spills_or_has_a_stack():
    with open(LIB, "rb") as f:
        blob = f.read()
    vgprs = _all(blob, b".vgpr_count")
    assert len(vgprs) == 12  # eleven instantiations of the superkernel and the one that arms the start stamp
    assert _all(blob, b".vgpr_spill_count") == [0] * 12
    assert _all(blob, b".private_segment_fixed_size") == [0] * 12
    assert max(vgprs) <= 256  # two workgroups per CU
    assert sum(v <= 168 for v in vgprs) >= 4  # the three narrow ones (three workgroups per CU) and the small one
