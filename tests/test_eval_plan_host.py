"""How evaluation is cut into launches, on the host: whole images where a launch a block takes several times as long, strips of
rows where a few images would leave most compute units idle, and the pitch that was measured to be the shorter one."""
import pytest

from tests.eval_plan import DOWN, IDENT, STEM, launches

# (blocks, height = width): what the wider pitch alone would cut into a launch a block
NARROW = [([(IDENT, 32, 1)] * 9, 27), ([(IDENT, 32, 1)] * 9, 28), ([(IDENT, 32, 1)] * 9, 29), ([(IDENT, 64, 1)] * 9, 17),
          ([(IDENT, 64, 1)] * 9, 18), ([(DOWN, 32, 2)] + [(IDENT, 64, 1)] * 8, 23), ([(DOWN, 32, 2)] + [(IDENT, 64, 1)] * 8, 24)]


@pytest.mark.parametrize("blocks,hw", NARROW)
def test_images_that_only_the_narrow_pitch_fits_are_one_launch(blocks, hw):
    assert [l[:2] for l in launches(blocks, 256, hw)] == [(9, 1)]


@pytest.mark.parametrize("c,hw,gap", [(32, 16, 32), (64, 8, 32), (64, 16, 32), (32, 24, 16), (32, 38, 16), (64, 24, 16), (64, 20, 32)])
def test_pitch_by_measured_time(c, hw, gap):
    assert {l[2] for l in launches([(IDENT, c, 1)] * 3, 256, hw)} == {gap}


# (blocks of 16 channels, height = width, images, whole images)
@pytest.mark.parametrize("blocks,hw,n,whole", [(1, 40, 1, False), (1, 44, 37, False), (3, 48, 8, False), (5, 48, 8, False), (3, 48, 256, True), (9, 40, 100, True)])
def test_a_few_large_images_are_spread_over_the_compute_units(blocks, hw, n, whole):
    plan = launches([(IDENT, 16, 1)] * blocks, n, hw)
    assert [l[0] for l in plan] == ([blocks] if whole else [1] * blocks)
    assert all((l[1] == 1) == whole for l in plan)


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("n", [1, 37, 256])
def test_every_launch_fits(n, bf16):
    for hw in range(6, 57, 1 if n == 37 else 5):
        for blocks in ([(STEM, 3, 1), (IDENT, 16, 1), (DOWN, 16, 2), (IDENT, 32, 1), (DOWN, 32, 2), (IDENT, 64, 1)], [(STEM, 3, 2), (IDENT, 16, 1)],
                       [(IDENT, 64, 1)]):
            plan = launches(blocks, n, hw, bf16)
            assert sum(l[0] for l in plan) == len(blocks)
            for count, strips, gap, lds in plan:
                assert lds <= 160 * 1024 and (strips == 1 or count == 1) and gap in ((16, 32) if bf16 else (16,))
