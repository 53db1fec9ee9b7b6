"""Waves a SIMD holds of the decode kernels whose speed rests on them, read from the assembly (CPU; how: tests/test_kernel_asm.py)."""
import re

from tests.test_kernel_asm import assembly, resident_waves  # noqa: F401  (a fixture)


def test_query_heads_that_share_a_unit(assembly):  # noqa: F811
    """Two launches; rank up to 8, and any rank at D = 64 with two heads a wave and up to 128 rows: three waves for 129 to 256 rows, as many as a wave per head and row had; four for fewer rows and two heads a
    wave, so that the blocks of 1024 units are there at once."""
    seen = set()
    for kernel, (n, scratch) in resident_waves(assembly("lessdec_gqs.hip")).items():
        m = re.search(r"gqs_step_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELi(\d+)ELb0E", kernel)
        if not m:
            continue
        d, rows, rank, heads = map(int, m.groups())
        if (rank == 8 and (rows == 4 or (rows == 2 and heads == 2))) or (d, rows, heads) == (64, 2, 2):
            assert n >= (3 if rows == 4 else 4) and scratch == 0, (kernel, n, scratch)
            seen.add((d, rows, heads, rank))
    assert len(seen) == 7


def test_a_wave_waits_for_its_entries_as_long_at_any_interval(assembly):  # noqa: F811
    """Every loop that asks for feature-map entries of its own launch sleeps 2^14 x 32 x 64 cycles before the wave gives up, give or take two
    polls, and is bounded; no sleep is longer than 256 cycles, which is what a wave may come too late by."""
    loops = 0
    for source in ("lessdec_wpu.hip", "lessdec_gqs.hip"):
        lines = assembly(source)
        for at, line in enumerate(lines):
            if (sleep := re.match(r"\s*s_sleep (\d+)", line)) is None:
                continue
            end = next(i for i in range(at, len(lines)) if "s_cbranch" in lines[i])
            bound = [int(m.group(1), 0) for x in lines[at:end] if (m := re.match(r"\s*s_cmpk?_gt_u32 s\d+, (\w+)", x))]
            assert len(bound) == 1, (source, at)
            assert int(sleep.group(1)) <= 4, (source, at)
            cycles = 64 * int(sleep.group(1)) * bound[0]
            assert abs(cycles - 2 ** 25) <= 2 * 64 * int(sleep.group(1)), (source, at, cycles)
            loops += 1
    assert loops >= 8


def test_every_form_of_the_streaming_step_can_be_launched(assembly):  # noqa: F811
    """A wave per unit with the maps in the launch: no more than 256 rows, head_dim 128."""
    forms = {tuple(map(int, m.groups())) for x in assembly("lessdec_wpu.hip")
             if (m := re.search(r"\.amdhsa_kernel \S*wpu_step_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELb(\d)ELb(\d)E", x))}
    assert {(d, rows) for d, rows, _, split, fused in forms if fused and not split} == {(128, 2), (128, 4)}
    assert {rows for _, rows, _, split, fused in forms if not fused} == {2, 4, 8}
