"""The plan of a stage that runs as two chains: every image once, no round longer than the workspace is sized for.  CPU only."""
import pytest

import stage_plan


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384])
@pytest.mark.parametrize("nW", [4, 24, 96, 126, 192, 361, 575, 1392, 2500, 4096])
def test_every_image_is_taken_once_and_fits_its_part_of_the_workspace(nW, C):
    for B in range(2, 80):
        L, n = stage_plan.lib, stage_plan.lib.rounds(B, nW, C)
        assert 1 <= n <= B // 2
        taken = []
        for chain in (0, 1):
            for r in range(n):
                first, images = L.part_first(B, nW, C, chain, r), L.part_images(B, nW, C, chain, r)
                assert 1 <= images <= L.round_images(B, nW, C, chain)
                taken += range(first, first + images)
        assert taken == list(range(B))


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384])
def test_a_round_is_a_share_of_the_map_of_about_the_same_size_at_every_width(C):
    """Where the images are small enough to choose, a chain's round holds 0.75 to 1.5 times the 53 MB a map that the rule names."""
    for B in range(8, 400):
        n = stage_plan.lib.rounds(B, 96, C)
        if n > 1:
            assert 0.75 * 2800 * 96 <= B * 96 * C / 2 / n <= 1.5 * 2800 * 96, (B, n)


@pytest.mark.parametrize("C,most", [(96, 128), (128, 128), (192, 128), (256, 160), (384, 128)])
def test_maps_of_few_windows_stay_on_one_chain_however_many_blocks(C, most):
    assert not stage_plan.lib.pays(2, most // 2, C, 1000) and stage_plan.lib.pays(2, most // 2 + 1, C, 1000)
