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


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384, 512, 768, 1024])
def test_long_stages_near_two_windows_a_cu_take_two_chains(C):
    """One chain of blocks in one kernel: up to a window a CU at any length; beyond, while the stage is short."""
    L = stage_plan.lib
    for windows in range(0, 1100):
        whole = [L.whole_stage(C, windows, windows, n) for n in range(1, 30)]
        if windows <= 256 or not L.whole_block(C, windows, windows, 0):
            assert len(set(whole)) == 1 and whole[0] == L.whole_block(C, windows, windows, 0)
        else:
            assert all(whole[:6]) and not any(whole[12:]) and sorted(whole, reverse=True) == whole, windows


@pytest.mark.parametrize("C,computed,most", [(96, 352, 8), (96, 383, 8), (96, 384, 12), (96, 512, 12), (128, 400, 6), (128, 447, 6), (128, 448, 8),
                                             (128, 512, 8)])
def test_lengths_of_a_stage_on_one_chain(C, computed, most):
    for windows in (computed, 512):                                   # with pruned windows and without
        assert stage_plan.lib.whole_stage(C, windows, computed, most) and not stage_plan.lib.whole_stage(C, windows, computed, most + 1)
