"""The plans of the three convolutions in one kernel, compiled for the CPU: which form a call takes, and that LDS holds what it puts there."""
import pytest


@pytest.mark.parametrize("hw,s3,passes,two", [
    ((84, 84), 1, 1023, False), ((84, 84), 1, 1024, True), ((84, 84), 1, 6144, True), ((52, 100), 2, 1024, True),
    ((37, 68), 1, 900, False), ((37, 68), 1, 1200, True),
    ((88, 84), 1, 6144, False)])                                # two outputs of the first layer do not fit
def test_two_images_from_four_passes_per_unit_on(tower_plan, hw, s3, passes, two):
    assert tower_plan.tower_two_images(*hw, 4, s3, passes, 256) == two


def test_pieces_of_lds_lie_apart(tower_plan):
    for s, s3 in ((4, 1), (4, 2), (8, 1)):
        for H in range(36, 129):
            for W in range(36, 129, 4):
                if s == 8 and min(H, W) < 64:
                    continue                                    # no second or third layer
                assert tower_plan.tower_overlap(H, W, s, s3) == 0, (H, W, s, s3)
