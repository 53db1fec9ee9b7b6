"""What the correctness of kernels rests on below the level of the source, read from the assembly that the
compiler makes of this repository's own files (CPU: hipcc cross-compiles for gfx950).

* A matrix instruction may read a vector instruction's result only two wait states after it.  The compiler
  counts them for the instructions that it makes itself, not for those inside an asm block.
* A load may read a scalar register that a vector instruction wrote only five wait states after it; again the compiler
  counts them for its own loads only.  And a load from memory into the LDS takes its place there from m0, which an asm
  block writes without the compiler's help.
* A buffer load is in range where its vector offset lies below num_records less its scalar offset: a load
  that relies on reading zeros past the end keeps the scalar offset within num_records.
"""
import re
import subprocess

import pytest

from paper_2402_09398_amd import build as hip_build

WAIT_STATES = 2


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    made = {}

    def get(name):
        if name not in made:
            out = tmp_path_factory.mktemp("asm") / (name + ".s")
            flags = [f for f in hip_build.FLAGS if f != "-shared"]
            subprocess.run([hip_build.HIPCC, *flags, "-w", "-S", "--cuda-device-only", "-o", str(out),
                            str(hip_build.CSRC / name)], check=True)
            made[name] = out.read_text().splitlines()
        return made[name]

    return get


def registers(operand):
    """Vector registers an operand names: v7, -v7, |v7|, v[4:7], a[0:3]."""
    m = re.fullmatch(r"[-|]*([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return set()
    lo, hi = (m.group(2), m.group(2)) if m.group(2) else (m.group(3), m.group(4))
    return {(m.group(1), i) for i in range(int(lo), int(hi) + 1)}


def early_matrix_reads(lines):
    """(line number, matrix instruction, the vector instruction too close before it) in straight-line order."""
    found, recent = [], []                    # recent: (wait states since, registers written, text)
    for n, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            if text.endswith(":"):
                recent = []                   # a label: another way in
            continue
        op, _, rest = text.partition(" ")
        operands = [x for x in re.split(r",\s*(?![^\[]*\])", rest.split(" op_sel")[0])]
        if op.startswith("v_mfma"):
            reads = set().union(*(registers(x.split(" ")[0]) for x in operands[1:4]))
            found += [(n, text, t) for waited, regs, t in recent if waited < WAIT_STATES and regs & reads]
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        recent = [(waited + states, regs, t) for waited, regs, t in recent if waited + states < WAIT_STATES]
        if op.startswith("v_") and not op.startswith("v_mfma"):
            recent.append((0, registers(operands[0].split(" ")[0]), text))
    return found


def test_the_reader_of_wait_states():
    near = ["v_fma_mixhi_f16 v5, -v1, 1.0, v2", "s_nop 0", "v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]"]
    far = [near[0], "s_nop 1", near[2]]
    assert len(early_matrix_reads(near)) == 1 and not early_matrix_reads(far)
    assert early_matrix_reads([near[0], near[2]]) and not early_matrix_reads(["v_mov_b32_e32 v12, 0", near[2]])


def scalars(operand):
    """Scalar registers an operand names: s7, s[4:7], m0."""
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return {operand} if operand == "m0" else set()
    lo, hi = (m.group(1), m.group(1)) if m.group(1) else (m.group(2), m.group(3))
    return set(range(int(lo), int(hi) + 1))


SCALAR_WAIT_STATES = 5


def scalar_hazards(lines):
    """Loads and stores that read a scalar register too soon after a vector instruction wrote it, and instructions other than
    an asm block's own that touch m0: (line number, text, cause)."""
    found, recent, in_asm = [], [], False     # recent: (wait states since, registers written, text)
    for n, line in enumerate(lines, 1):
        in_asm = (in_asm or "#ASMSTART" in line) and "#ASMEND" not in line
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue                          # (a label: what fell through to it counts on)
        op, _, rest = text.partition(" ")
        operands = [x.strip().split(" ")[0] for x in re.split(r",\s*(?![^\[]*\])", rest)]
        if not in_asm and "m0" in operands:
            found.append((n, text, "m0"))
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            reads = set().union(*(scalars(x) for x in operands))
            found += [(n, text, t) for waited, regs, t in recent if waited < SCALAR_WAIT_STATES and regs & reads]
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        recent = [(waited + states, regs, t) for waited, regs, t in recent if waited + states < SCALAR_WAIT_STATES]
        if op.startswith("v_") and scalars(operands[0]):
            recent.append((0, scalars(operands[0]), text))
    return found


def test_the_reader_of_scalar_hazards():
    load = "buffer_load_dwordx4 v3, s[12:15], 0 offen lds"
    assert scalar_hazards(["v_readfirstlane_b32 s13, v1", "s_nop 3", load])
    assert not scalar_hazards(["v_readfirstlane_b32 s13, v1", "s_nop 4", load]) and not scalar_hazards(["s_mov_b32 s13, s1", load])
    assert scalar_hazards(["v_readlane_b32 s7, v9, 3", ";;#ASMSTART", "s_mov_b32 m0, s7", "s_nop 0", load, ";;#ASMEND"]) == []
    assert scalar_hazards(["s_mov_b32 m0, s7"]) and scalar_hazards(["v_cmp_lt_i32_e64 s[14:15], v0, v1", load])


@pytest.mark.parametrize("name", [s for s in hip_build.SOURCES if "lessdec_lds.h" in (hip_build.CSRC / s).read_text()])
def test_loads_into_the_lds_read_settled_scalars(assembly, name):
    lines = assembly(name)
    assert any("lds" in x.split(";")[0] for x in lines) and scalar_hazards(lines) == []


@pytest.mark.parametrize("name", [s for s in hip_build.SOURCES
                                  if "mfma" in (hip_build.CSRC / s).read_text() or "lessdec_mlp.h" in (hip_build.CSRC / s).read_text()])
def test_matrix_instructions_wait_for_vector_results(assembly, name):
    assert early_matrix_reads(assembly(name)) == []


def test_prompt_rows_past_the_end_are_in_the_range_check(assembly):
    """The row pass reads a tile through a buffer of a whole tile, rows past the prompt clamped to the last one by the vector
    offset; scalar offsets are constants below a row of 64 halves, or clamped themselves."""
    written, loads = {}, 0
    for line in assembly("lessdec_rows.hip"):
        op, _, rest = line.split(";")[0].strip().partition(" ")
        operands = [x.strip() for x in rest.split(",")]
        if op.startswith("buffer_load"):
            soffset = operands[2].split(" ")[0] if "[" not in operands[2] else operands[3].split(" ")[0]
            loads += 1
            assert soffset.isdigit() and int(soffset) <= 64 or written.get(soffset, "").startswith("s_min_"), line
        elif op.startswith("s_") and operands[0].startswith("s"):
            written[operands[0]] = op
    assert loads


def resident_waves(lines):
    """kernel -> (waves a SIMD holds of it, scratch bytes): vector registers by the compiler's own count; a SIMD's 800 scalar registers
    are given out in sixteens, with sixteen more to every wave."""
    found, name, scalar, scratch = {}, None, 0, 0
    for line in lines:
        word = line.split()
        if len(word) == 2 and word[0] == ".amdhsa_kernel":
            name = word[1]
        elif line.startswith("; TotalNumSgprs:"):
            scalar = int(word[-1])
        elif line.startswith("; ScratchSize:"):
            scratch = int(word[-1])
        elif line.startswith("; Occupancy:"):
            found[name] = (min(int(word[-1]), 800 // ((scalar + 15) // 16 * 16 + 16)), scratch)
    return found


def test_the_step_that_finishes_the_maps_keeps_its_waves(assembly):
    """The any-shape step with the maps' last activation in it has as many waves a SIMD as without, and no scratch memory."""
    waves = {k: v for k, v in resident_waves(assembly("lessdec_step.hip")).items() if "11step_kernel" in k}
    compared = 0
    for kernel, (n, scratch) in waves.items():
        m = re.search(r"step_kernelI(f|6__half)Li(\d+)ELi(\d+)ELi(\d+)ELb1E", kernel)
        if not m:
            continue
        storage, d, turns, w = m.group(1), *map(int, m.groups()[1:])
        without, spilled = waves[kernel.replace("ELb1E", "ELb0E")]
        assert scratch <= spilled, kernel
        if storage == "f" or turns != 7:              # (fp16, seven turns: see step_waves_per_simd)
            assert n >= without, (kernel, n, without)
            compared += 1
    assert compared >= 20
