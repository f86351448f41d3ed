"""The plan of a stage that runs as two chains: every image once, no round longer than the workspace is sized for.  CPU only."""
import pytest

import stage_plan


@pytest.mark.parametrize("nW", [4, 24, 96, 126, 192, 361, 575, 1392, 2500, 4096])
def test_every_image_is_taken_once_and_fits_its_part_of_the_workspace(nW):
    for B in range(2, 80):
        L, n = stage_plan.lib, stage_plan.lib.rounds(B, nW)
        assert 1 <= n <= B // 2
        taken = []
        for chain in (0, 1):
            for r in range(n):
                first, images = L.part_first(B, nW, chain, r), L.part_images(B, nW, chain, r)
                assert 1 <= images <= L.round_images(B, nW, chain)
                taken += range(first, first + images)
        assert taken == list(range(B))
