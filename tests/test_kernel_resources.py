"""What the compiler made of the kernels, read from the metadata that it writes into the library: no kernel
keeps anything in scratch memory. The outer step promises to need no device memory beyond the arena, and
the register kernels are built around their rows staying in registers."""
import re

import pytest

import paper_2506_10911_amd as nl


def kernel_fields(data, field):
    """The unsigned msgpack integers that follow a field's name, one per kernel."""
    values = []
    for m in re.finditer(re.escape(b"." + field), data):
        kind, rest = data[m.end()], data[m.end() + 1:m.end() + 9]
        width = {0xCC: 1, 0xCD: 2, 0xCE: 4, 0xCF: 8}.get(kind, 0)
        assert kind < 0x80 or width, f"{field}: not an unsigned integer"
        values.append(int.from_bytes(rest[:width], "big") if width else kind)
    return values


@pytest.mark.parametrize("field", [b"private_segment_fixed_size", b"vgpr_spill_count"])
def test_no_kernel_uses_scratch(field):
    with open(nl.library_path(), "rb") as f:
        values = kernel_fields(f.read(), field)
    assert len(values) > 100                       # the step's kernels alone are more than that
    assert [v for v in values if v] == []
