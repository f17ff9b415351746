"""What the compiler made of the kernels (no GPU): the library's device code as assembly for gfx950."""
import os
import re
import subprocess

import pytest


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    from paper_1803_00933_amd import build
    out = str(tmp_path_factory.mktemp("assembly") / "device.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-w", "-I", os.path.join(build.ROOT, "include"),
                           "-I", os.path.join(build.HERE, "csrc"), "-o", out] + build.SOURCES)
    with open(out) as f:
        return f.read().splitlines()


def registers(operand):
    """Vector registers that an operand names."""
    m = re.fullmatch(r"v(\d+)|v\[(\d+):(\d+)\]", operand)
    if not m:
        return []
    return [int(m.group(1))] if m.group(1) else list(range(int(m.group(2)), int(m.group(3)) + 1))


def test_wait_states_between_vector_instructions(assembly):
    """Two wait states, which the compiler keeps on this target and which assembly has to bring itself, from a vector
    instruction that writes vcc to one that reads it (carries and selections), and from one that writes a register to one
    that reads it through a DPP control."""
    carries = dpps = states = 0
    vcc, written, too_soon = -9, {}, []
    for number, line in enumerate(assembly, 1):
        text = line.split(";")[0].strip()
        if text.endswith(":"):       # reached from elsewhere too
            vcc, written = -9, {}
            continue
        if not text or text.startswith("."):
            continue
        op, _, rest = text.partition(" ")
        operands = [x.strip() for x in rest.split(",")]
        operands[-1] = operands[-1].split(" ")[0]
        if op == "s_nop":
            states += int(operands[0], 0) + 1
            continue
        if op.startswith("v_"):
            with_carry = "_co_" in op
            if "vcc" in operands[2 if with_carry else 1:] and not op.startswith("v_cmp"):
                carries += 1
                if states - vcc < 2:
                    too_soon.append((number, text))
            if "_dpp" in op:
                dpps += 1
                for r in registers(operands[2 if with_carry else 1].strip("-|")):
                    if states - written.get(r, -9) < 2:
                        too_soon.append((number, text))
        states += 1
        if op.startswith("v_"):
            if operands[0] == "vcc" or ("_co_" in op and operands[1] == "vcc"):
                vcc = states
            for r in registers(operands[0]):
                written[r] = states
    assert carries > 1000 and dpps > 1000, (carries, dpps)   # the parsing finds them
    assert not too_soon, (len(too_soon), too_soon[:5])


def test_two_workgroups_of_a_prioritized_add_fit_a_compute_unit(assembly):
    """Workgroups of 1024 threads: 8 waves per SIMD for two of them, which have 64 of its 512 vector registers each."""
    held = {}
    for line in assembly:
        if line.strip().startswith("- .a"):      # the next kernel's entry in the metadata
            name = None
        m = re.match(r"\s+\.(name|vgpr_count):\s+(\S+)", line)
        if m and m.group(1) == "name" and m.group(2).startswith("_Z"):
            name = m.group(2)
        elif m and m.group(1) == "vgpr_count" and "pe_add_rows_kernel" in (name or ""):
            held[name] = int(m.group(2))
    assert len(held) == 4 and max(held.values()) <= 64, held
