"""The built library's own device code.  Loads that go straight to LDS, marks of selected columns and bounds of tiles are written
as instructions, so the compiler keeps no distance in front of them: every one has to bring it along."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs a disassembler")
def test_loads_to_lds_keep_their_distance(tmp_path):
    from paper_2310_01777_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    shutil.copy(build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    loads = 0
    for obj in glob.glob(str(tmp_path / "*gfx950")):
        dump = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True, capture_output=True, text=True)
        before = []  # the run of such loads and of what belongs to them, up to here
        for line in dump.stdout.splitlines():
            ins = " ".join(line.split("//")[0].split())
            if re.match(r"buffer_load_dword(x4)? .* lds$", ins):
                loads += 1
                # scalars from vector instructions are read five wait states later, m0 from the scalar unit one
                waits = [int(w[1]) + 1 if (w := re.match(r"s_nop (\d+)$", x)) else 1 for x in before]
                assert sum(waits) >= 5 and re.match(r"s_nop \d+$", before[-1]) and before[-2].startswith("s_mov_b32 m0, "), (obj, before, ins)
                before.append(ins)
            elif ins.startswith("s_mov_b32 m0, ") or re.match(r"s_nop \d+$", ins):
                before.append(ins)
            elif ins:
                before = []
    assert loads > 0


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The device code objects of the built library, as files."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs a disassembler")
    from paper_2310_01777_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("objects")
    shutil.copy(build.LIB, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    return sorted(glob.glob(str(d / "*gfx950")))


# Registers a kernel may use so that the waves it is written for stay resident together (512 a SIMD, in eights): the key
# kernel of columns of any width, bidirectional, whose launches are a few rounds of blocks.
@pytest.mark.parametrize("kernel,registers", [("key_columns_kernelILi4ELb0E", 80), ("key_columns_kernelILi2ELb0E", 64)])
def test_registers_leave_room(objects, kernel, registers):
    used = []
    for obj in objects:
        notes = subprocess.run([READELF, "--notes", obj], check=True, capture_output=True, text=True).stdout
        for entry in notes.split("  - .agpr_count")[1:]:
            if kernel in re.search(r"\.name: +(\S+)", entry)[1]:
                used.append(int(re.search(r"\.vgpr_count: +(\d+)", entry)[1]))
    assert used and max(used) <= registers


@pytest.fixture(scope="module")
def kernels(objects):
    """Instructions of every kernel and function, by name."""
    out = {}
    for obj in objects:
        dump = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"^(?:[0-9a-f]+ )?<", dump, flags=re.M)[1:]:
            name, _, body = part.partition(">:")
            out[name] = [" ".join(line.split("//")[0].split()) for line in body.splitlines()[1:] if line.split("//")[0].strip()]
    return out


# The kernel for one column per row that writes the scores too takes each product once: four for 32 features of the projection,
# m / 16 for 32 of the contraction's 128 columns.
@pytest.mark.parametrize("m", [64, 128])
def test_scores_of_one_column_rows_take_one_pass(kernels, m):
    found = [ins for name, ins in kernels.items() if f"estimate_rows_bidir_kernelILi{m // 32}ELi8ELb1E" in name]
    assert len(found) == 1
    assert sum(i.startswith("v_mfma_f32_32x32x16_bf16") for i in found[0]) == 4 * (m // 32) + 4 * (m // 16)


def _registers(operand):
    """The scalar and vector registers an operand names."""
    operand = operand.strip().lstrip("-").strip("|")
    if m := re.fullmatch(r"([sv])\[(\d+):(\d+)\]", operand):
        return {m[1] + str(i) for i in range(int(m[2]), int(m[3]) + 1)}
    return {operand} if operand == "vcc" or re.fullmatch(r"[sv]\d+", operand) else set()


def _distances(instructions):
    """(writer, wait states between, reader) for scalars that vector instructions write and vector instructions read, and for
    results of matrix instructions that other vector instructions read; straight-line code, a branch counted as one state."""
    written = {}  # register: [its writer, wait states since]
    for ins in instructions:
        op, _, rest = ins.partition(" ")
        ops = [o.split()[0] if o.split() else "" for o in re.split(r",\s*(?![^\[]*\])", rest)] if rest else []
        outputs = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", op) else 1
        vector, matrix = op.startswith("v_"), "mfma" in op
        if vector and not matrix:
            for r in set().union(*map(_registers, ops[outputs:])) & set(written):
                yield written[r][0], written[r][1], ins
        states = int(ops[0]) + 1 if op == "s_nop" else 1
        for r in list(written):
            written[r][1] += states
            if written[r][1] > 40:
                del written[r]
        for r in set().union(*map(_registers, ops[: outputs if vector else 1])):
            if vector and (matrix or r[0] == "s" or r == "vcc"):
                written[r] = [op, 0]
            else:
                written.pop(r, None)
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            written = {}


# Wait states that gfx950 wants, which the compiler keeps for its own instructions only: the marks of selected columns and the
# bounds of tiles are written as instructions, and some of them read what matrix instructions wrote.
WAIT_STATES = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x16_bf16": 12, "v_mfma_i32_16x16x64_i8": 8}


def _too_close(instructions):
    return [d for d in _distances(instructions) if d[1] < (WAIT_STATES.get(d[0], 0) if "mfma" in d[0] else 2)]


def test_vector_instructions_keep_their_distance(kernels):
    assert any("v_addc_co_u32_e64" in i for ins in kernels.values() for i in ins)  # (marks)
    assert {name: d for name, ins in kernels.items() if (d := _too_close(ins))} == {}


def test_distances_are_seen():
    marks = ["v_cmp_ge_u32_e64 s[4:5], v1, v9", "v_cmp_ge_u32_e64 s[6:7], v2, v9", "v_addc_co_u32_e64 v0, vcc, v0, v0, s[4:5]"]
    assert _too_close(marks)
    assert not _too_close(marks[:2] + ["s_nop 0"] + marks[2:])
    assert _too_close(["v_cmp_lt_f32_e32 vcc, v1, v2", "v_cndmask_b32_e32 v3, v4, v5, vcc"])
    product = ["v_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[8:11], v[4:7]", "s_nop 6", "v_add_f32_e32 v1, v2, v6"]
    assert _too_close(product)
    assert not _too_close(product[:1] + ["s_nop 7"] + product[2:])
    assert not _too_close(product[:1] + ["v_mov_b32_e32 v6, 0"] + product[2:])


def test_outputs_of_several_instructions_are_early():
    """An output that is written before all inputs are read must not share a register with one of them: `&`."""
    from paper_2310_01777_amd import build
    several = 0
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        # an asm statement, or a macro that is a part of one
        for part in re.findall(r"\basm(?: volatile)?\s*\((?:[^;]|;(?!\n))*;|#define \w+_OPERANDS(?:.*\\\n)*.*", text):
            code, _, operands = part.partition(":" if part.startswith("asm") else "OPERANDS")
            if "\\n" in code or part.startswith("#define"):
                several += 1
                assert not re.findall(r'"[=+](?!&)[vs]"', operands), (path, part)
    assert several >= 5
