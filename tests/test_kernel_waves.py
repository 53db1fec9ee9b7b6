"""Waves a SIMD holds of the decode kernels whose speed rests on them, read from the assembly (CPU; how: tests/test_kernel_asm.py)."""
import re

from tests.test_kernel_asm import assembly, resident_waves  # noqa: F401  (a fixture)


def test_query_heads_that_share_a_unit(assembly):  # noqa: F811
    """Two launches, rank up to 8: three waves for 129 to 256 rows, as many as a wave per head and row had; four for fewer rows and two heads a
    wave, so that the blocks of 1024 units are there at once."""
    seen = set()
    for kernel, (n, scratch) in resident_waves(assembly("lessdec_gqs.hip")).items():
        m = re.search(r"gqs_step_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELi(\d+)ELb0E", kernel)
        if not m:
            continue
        d, rows, rank, heads = map(int, m.groups())
        if rank == 8 and (rows == 4 or (rows == 2 and heads == 2)):
            assert n >= (3 if rows == 4 else 4) and scratch == 0, (kernel, n, scratch)
            seen.add((d, rows, heads))
    assert len(seen) == 6
