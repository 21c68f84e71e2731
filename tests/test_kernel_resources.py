"""What the compiler says of the kernels in the built library: none of them keeps registers in memory."""
import re

from paper_2002_01119_amd import psgd


def _counts(blob, key):
    """The values of one key in the kernels' metadata (MessagePack: the key's text, then a small integer)."""
    at = [m.end() for m in re.finditer(re.escape(key) + rb"(?![a-z_])", blob)]
    wide = {0xCC: 1, 0xCD: 2, 0xCE: 4}
    return [blob[i] if blob[i] < 0x80 else int.from_bytes(blob[i + 1:i + 1 + wide[blob[i]]], "big") for i in at]


def test_no_kernel_spills_vector_registers():
    psgd.load()
    with open(psgd._LIB_PATH, "rb") as f:
        blob = f.read()
    spilled, scratch = _counts(blob, b".vgpr_spill_count"), _counts(blob, b".private_segment_fixed_size")
    assert len(spilled) == len(scratch) >= 100
    assert not any(spilled) and not any(scratch), (sum(v > 0 for v in spilled), max(spilled), max(scratch))
