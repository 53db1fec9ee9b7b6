"""What the correctness of kernels rests on below the level of the source, read from the assembly that the
compiler makes of this repository's own files (CPU: hipcc cross-compiles for gfx950).

* A matrix instruction may read a vector instruction's result only two wait states after it.  The compiler
  counts them for the instructions that it makes itself, not for those inside an asm block.
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


@pytest.mark.parametrize("name", [s for s in hip_build.SOURCES
                                  if "mfma" in (hip_build.CSRC / s).read_text() or "lessdec_mlp.h" in (hip_build.CSRC / s).read_text()])
def test_matrix_instructions_wait_for_vector_results(assembly, name):
    assert early_matrix_reads(assembly(name)) == []


def test_prompt_rows_past_the_end_are_in_the_range_check(assembly):
    """The row pass reads a tile through a buffer of the rows that the prompt still has, one at least: constant
    scalar offsets stay below a row of 64 halves, the others are clamped to the buffer's size."""
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
