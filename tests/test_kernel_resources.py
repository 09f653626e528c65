"""What the compiler made of the kernels, read from the metadata that it writes into the library: no kernel
keeps anything in scratch memory. The outer step promises to need no device memory beyond the arena, and
the register kernels are built around their rows staying in registers."""
import os
import re
import subprocess

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


def test_scalar_registers_that_move_to_vector_lanes():
    """A scalar register that the compiler spills goes to a lane of a vector register (not to scratch) and costs an
    instruction each way. Only the kernels of 17 to 56 members that hold phi and delta have such: their members' ids and
    addresses are more than the scalar registers take. Reading the ids anew instead was slower."""
    with open(nl.library_path(), "rb") as f:
        data = f.read()
    moved = {}
    for m in re.finditer(rb"\.sgpr_spill_count(?:([\x00-\x7f])|\xcc(.)|\xcd..|\xce....)\xa7\.symbol(?:\xd9(.)|\xda(..))", data, re.S):
        length = int.from_bytes(m[3] or m[4], "big")
        symbol = data[m.end():m.end() + length].decode()
        moved[symbol] = int.from_bytes(m[1] or m[2] or b"\xff\xff", "big")
    assert len(moved) == len(kernel_fields(data, b"sgpr_spill_count")) > 100
    assert {symbol: count for symbol, count in moved.items() if count > (80 if "outer_step_held" in symbol else 0)} == {}


def device_code(path):
    """The GPU's ELF image inside the library."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        machine = int.from_bytes(data[at + 18:at + 20], "little")
        if machine == 224:                         # AMDGPU
            table, entry, count = (int.from_bytes(data[at + a:at + b], "little") for a, b in ((40, 48), (58, 60), (60, 62)))
            return data[at:at + table + entry * count]
        at = data.find(b"\x7fELF", at + 4)
    raise AssertionError("no GPU code in the library")


def kernel_bodies(tmp_path, name):
    """(symbol, instructions) of every kernel of the library whose symbol contains `name`."""
    image = tmp_path / "gfx950.elf"
    image.write_bytes(device_code(nl.library_path()))
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(image)], check=True, capture_output=True, text=True).stdout
    return [(symbol, body.splitlines()) for symbol, body in re.findall(r"<([^>]*%s[^>]*)>:\n(.*?)\n\n" % name, text + "\n\n", re.S)]


def loads_behind_a_wait(body):
    """Vector loads that come after a wait for other ones."""
    waited, late = False, 0
    for line in body:
        late += waited and re.search(r"\b(buffer|global)_load", line) is not None
        waited = waited or "vmcnt(" in line
    return late


def test_step_asks_for_all_members_at_once(tmp_path):
    """No load of the register kernels (groups of up to 16) waits for another: one that does costs the wave a second
    round trip to HBM."""
    bodies = kernel_bodies(tmp_path, "outer_step_fixed")
    assert len(bodies) >= 16 * 2 * 3               # group sizes, storage types, ways of launching
    assert [symbol for symbol, body in bodies if loads_behind_a_wait(body)] == []


def test_hyper_parameters_are_one_load(tmp_path):
    """What an in-order launch of the register kernels needs beyond its rows (the hyper-parameters, how to store) is asked
    for in one scalar load or two: pairs of many small tensors took 0.5 to 1.5 % longer with three."""
    bodies = kernel_bodies(tmp_path, "outer_step_fixed[^>]*InOrderArgs")
    assert len(bodies) == 16 * 2 * 2               # group sizes, storage types, lengths of the member table
    late = {}
    for symbol, body in bodies:
        first = next(i for i, line in enumerate(body) if "buffer_load" in line)
        late[symbol] = sum("s_load" in line for line in body[first:])
    assert [symbol for symbol, loads in late.items() if loads > 2] == []


def test_spread_asks_for_its_rows_at_once(tmp_path):
    """No load of the replica-spread kernels that hold bf16 rows or more than 16, or take four steps, waits for another."""
    held = []
    for symbol, body in kernel_bodies(tmp_path, "replica_spread_tiles"):
        rows, steps, tag = re.search(r"tilesILi(\d+)ELi\d+ELi(\d+)E(f|N)", symbol).groups()
        if int(rows) > 16 or int(steps) > 1 or (tag == "N" and int(rows) > 0):
            held.append((symbol, body))
    assert len(held) >= 27 + 11                    # bf16, float
    assert [symbol for symbol, body in held if loads_behind_a_wait(body)] == []


def test_knobs_store_as_the_header_says(tmp_path):
    """Under launch-shape knobs stores are non-temporal or ordinary: none is written through the L2 (sc1)."""
    bodies = kernel_bodies(tmp_path, "outer_step[^>]*StepArgs")
    assert len(bodies) >= 16 * 2 * 2
    assert [symbol for symbol, body in bodies if any("_store" in line and "sc1" in line for line in body)] == []


def test_pooling_waits_for_its_sums_before_the_ticket(tmp_path):
    """The workgroup that draws the last ticket reads the sums that the others stored. The ticket's release waits
    for the stores of the wave that draws it; every other wave has to wait for its own before the barrier
    in front of the ticket."""
    image = tmp_path / "gfx950.elf"
    image.write_bytes(device_code(nl.library_path()))
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(image)], check=True, capture_output=True, text=True).stdout
    body = re.search(r"<[^>]*replica_spread_pool[^>]*>:\n(.*?)\n\n", text, re.S).group(1).splitlines()
    ticket = next(i for i, line in enumerate(body) if "global_atomic_add" in line)
    barrier = max(i for i in range(ticket) if "s_barrier" in body[i])
    assert any("buffer_wbl2" in line for line in body[barrier:ticket])
    last_store = max(i for i in range(barrier) if "global_store" in body[i])
    assert any(re.search(r"s_waitcnt vmcnt\(0\)\s*(//|$)", line) for line in body[barrier - 3:barrier]) and last_store < barrier - 3
