"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element."""
import numpy as np
import pytest
import torch

import product_plan
import wide_sums
from paper_2507_19131_amd import synth

pytestmark = pytest.mark.gpu

gh = pytest.importorskip("gpu_harness") if torch.cuda.is_available() else None
if torch.cuda.is_available():
    from paper_2507_19131_amd import binding as M

def _case(B, H, W, C, heads, shift, keep, seed, blobs=False, outliers=False, bits=(8, 4), wbits=8, ranges=None, mode=0,
          mlp_ratio=4, **block_kw):
    spec = synth.BlockSpec(B, H, W, C, heads, shift=shift, act_bits_high=bits[0], act_bits_low=bits[1],
                           weight_bits=wbits, score_mode=mode, mlp_ratio=mlp_ratio)
    inp = synth.make_block_inputs(spec, seed, ranges=ranges, **block_kw)
    x = synth.make_feature_map(spec, seed, blobs=blobs, outlier_channels=outliers)
    return spec, inp, x, M.mixaq_keep_count(spec.nW, keep)


SMALL = [
    # B, H, W, C, heads, shift, keep, seed, kwargs
    (1, 56, 56, 96, 3, 0, 0.5, 1001, {}),                                             # config 1
    (2, 26, 33, 96, 3, 3, 0.4, 11, dict(blobs=True)),                                 # padded + shifted + batch
    (2, 20, 27, 128, 4, 3, 0.4, 12, dict(outliers=True, ranges={"a_qkv_in": (-12.0, 13.5), "a_fc1_in": (-11.0, 10.0)})),
    (1, 14, 21, 192, 6, 3, 0.5, 13, dict(mode=1)),
    (2, 20, 28, 256, 8, 0, 0.3, 14, {}),
    (2, 50, 84, 384, 12, 3, 0.25, 1003, {}),                                          # config 3 block
    (1, 25, 42, 768, 24, 3, 0.5, 1004, dict(bits=(4, 2), wbits=4)),                   # config 4 stage 4
    (1, 30, 30, 96, 3, 3, 0.0, 15, {}),                                               # everything low
    (1, 30, 30, 96, 3, 3, 1.0, 16, {}),                                               # everything high
    (3, 15, 16, 96, 3, 0, 0.11, 17, dict(blobs=True)),                                # one high window per image
    (1, 28, 35, 96, 3, 3, 0.5, 18, dict(bits=(6, 3))),                                # odd bit widths
    (2, 21, 21, 128, 4, 3, 0.6, 19, dict(bits=(5, 2), wbits=4)),                      # 2-bit low branch, 4-bit weights
    (1, 7, 7, 96, 3, 0, 1.0, 20, {}),                                                 # a single window
    (1, 5, 6, 96, 3, 0, 0.0, 24, {}),                                                 # a map smaller than one window
    (2, 3, 20, 128, 4, 0, 0.5, 25, {}),                                               # one row of windows, mostly padding
    (3, 98, 98, 192, 6, 3, 0.5, 26, {}),                                              # 588 windows at six heads: one wave per head
    (2, 84, 91, 128, 4, 3, 0.5, 28, dict(bits=(8, 2))),                               # 312 windows at four heads: one wave per head, codes four per byte
    (2, 21, 28, 512, 16, 3, 0.4, 29, dict(bits=(7, 3))),                              # sixteen heads (FC2 with K = 2048), seven kernels
    (1, 14, 21, 1024, 32, 3, 0.5, 27, {}),                                            # the widest supported block (FC2 with K = 4096)
]


# both implementations: the two fused kernels (C <= 384) and the seven-kernel path; the default path of the wider blocks is in
# WIDE_CASES
BLOCK_CASES = [case + (fused,) for case in SMALL for fused in (True, False) if not (fused and case[3] > 384)]


@pytest.mark.parametrize("B,H,W,C,heads,shift,keep,seed,kw,fused", BLOCK_CASES)
def test_block_matches_oracle(B, H, W, C, heads, shift, keep, seed, kw, fused):
    """fused: the window and token kernels (C <= 384); otherwise the seven-kernel path."""
    spec, inp, x, k = _case(B, H, W, C, heads, shift, keep, seed, **kw)
    print("case", B, H, W, C, heads, shift, keep, seed, kw, "fused", fused, flush=True)
    res = gh.compare_block(inp, x, k, fused=fused)
    print(res, flush=True)
    gh.assert_parity(res)


BIAS_CASES = [(C, heads, bits, wbits, shift, fused)
              for (C, heads, bits, wbits) in [(96, 3, (8, 4), 8), (384, 12, (8, 4), 8), (768, 24, (4, 2), 4)]
              for shift in (0, 3) for fused in (True, False) if not (fused and C > 384)]


@pytest.mark.parametrize("C,heads,bits,wbits,shift,fused", BIAS_CASES)
def test_independent_biases_per_branch(C, heads, bits, wbits, shift, fused):
    """PTQ variant (Sec. 4.3, PTQ setup): the low branch has biases of its own, visibly different from the
    high branch's; every tap must follow the bias of the row's branch (both implementations up to C = 384, the
    seven-kernel path at C = 768)."""
    spec, inp, x, k = _case(2, 20, 27, C, heads, shift, 0.4, 51, blobs=True, bits=bits, wbits=wbits,
                            per_branch_bias=True, bias_std=0.1)
    for n in ("b_qkv", "b_proj", "b_fc1", "b_fc2"):
        assert not np.array_equal(getattr(inp.branches[0], n), getattr(inp.branches[1], n))
    print("independent biases", C, shift, "fused", fused, flush=True)
    res = gh.compare_block(inp, x, k, fused=fused)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("C,heads,mlp_ratio", [(96, 3, 3), (96, 3, 1), (192, 6, 3), (128, 4, 2), (96, 3, 8), (768, 24, 7)])
def test_other_mlp_ratios(C, heads, mlp_ratio):
    """FFN widths other than 4C run the separate kernels: hidden sizes that are not a whole number of ring turns of the tile
    kernel (9 or 3 slabs of 32), K = 768 with an N = 96 that the ring kernel does not take, and K = 5376, 42 stages of that one."""
    spec, inp, x, k = _case(2, 20, 27, C, heads, 3, 0.5, 52, blobs=True, mlp_ratio=mlp_ratio)
    print("mlp_ratio", mlp_ratio, "C", C, flush=True)
    res = gh.compare_block(inp, x, k)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("C,heads,H,W,shift,bits,hidden", [
    (96, 3, 26, 33, 3, (8, 4), (-0.07, 0.35)),               # the high branch has no table of steps: both take the cubic
    (128, 4, 20, 27, 0, (8, 4), (-0.07, 0.35)), (192, 6, 14, 21, 3, (8, 4), (-0.07, 0.35)), (256, 8, 20, 28, 0, (8, 4), (-0.07, 0.35)),
    (384, 12, 20, 27, 3, (8, 4), (-0.07, 0.35)), (384, 12, 50, 84, 0, (8, 4), (-0.07, 0.35)),        # 32 and 64 rows
    (96, 3, 26, 33, 3, (8, 8), (-0.17, 0.45)), (384, 12, 50, 84, 0, (8, 7), (-0.17, 0.45)),          # tables of 1500 entries
    (96, 3, 26, 33, 3, (2, 2), (-0.17, 4.0)), (256, 8, 20, 28, 0, (8, 3), (-0.17, 40.0)), (192, 6, 20, 28, 0, (5, 6), (-0.6, 0.6))])
def test_gelu_codes_by_steps_and_by_the_cubic(C, heads, H, W, shift, bits, hidden):
    spec, inp, x, k = _case(2, H, W, C, heads, shift, 0.5, 57, blobs=True, bits=bits, ranges={"a_fc2_in": hidden})
    print("gelu", C, H, W, bits, hidden, flush=True)
    res = gh.compare_block(inp, x, k)
    print(res, flush=True)
    gh.assert_parity(res)


AT, OVER, FAR = wide_sums.WIDEST, wide_sums.WIDEST + 1, 20480           # widths of rows: 8-bit sums of 2^22 less 64, 2^22 and 191, 1.25 * 2^22


@pytest.mark.parametrize("C,H,W,widths,sign,bits", [                    # widths of the rows of w_qkv, w_proj and w_fc1
    (96, 26, 33, (12288,) * 3, 1, (8, 8)), (128, 20, 27, (16384,) * 3, 1, (8, 4)),   # the widest rows of these widths: never beyond
    (192, 20, 27, (AT,) * 3, 1, (8, 4)), (192, 20, 27, (AT,) * 3, -1, (8, 8)), (192, 20, 27, (OVER,) * 3, 1, (8, 4)), (192, 20, 27, (OVER,) * 3, -1, (8, 4)),
    (192, 20, 27, (FAR, AT, AT), 1, (8, 4)), (192, 20, 27, (AT, FAR, AT), 1, (8, 4)), (192, 20, 27, (AT, AT, FAR), 1, (8, 4)),
    (192, 20, 27, (FAR, AT, AT), -1, (8, 4)), (192, 20, 27, (AT, FAR, AT), -1, (8, 4)), (192, 20, 27, (AT, AT, FAR), -1, (4, 8)),
    (256, 20, 28, (AT,) * 3, 1, (8, 4)), (256, 20, 28, (FAR,) * 3, 1, (8, 4)),
    (384, 20, 27, (AT,) * 3, 1, (8, 4)), (384, 50, 84, (AT,) * 3, -1, (8, 4)), (384, 50, 84, (FAR,) * 3, 1, (8, 4)),     # 32 and 64 rows
    (512, 21, 28, (AT,) * 3, 1, (8, 4)), (512, 21, 28, (FAR,) * 3, -1, (8, 4)), (512, 49, 56, (AT, FAR, FAR), 1, (8, 4)), (512, 49, 56, (FAR,) * 3, 1, (8, 4)),
    (768, 42, 49, (AT,) * 3, 1, (8, 4)), (768, 42, 49, (FAR, AT, AT), -1, (8, 4)), (1024, 21, 56, (AT,) * 3, 1, (8, 4)), (1024, 35, 49, (FAR,) * 3, 1, (8, 4))])
def test_sums_at_and_beyond_what_a_binary32_holds(C, H, W, widths, sign, bits):
    """Sums of q, k, v, the projection and FC1 that the kernels take as binary32 without a conversion, up to the bound of that form, and
    blocks beyond it, which convert (tests/test_wide_sums.py: the sums reach these sizes, and taking them for their own bits would show)."""
    spec = synth.BlockSpec(2 if C <= 512 else 1, H, W, C, C // 32, shift=3, act_bits_high=bits[0], act_bits_low=bits[1])
    inp, x = wide_sums.make_inputs(spec, widths, sign), synth.make_feature_map(spec, 58, blobs=True)
    print("sums", C, H, W, widths, sign, bits, flush=True)
    res = gh.compare_block(inp, x, spec.nW // 2)
    print(res, flush=True)
    gh.assert_parity(res)
    assert res["y_bit_identical"] and res["h_maxabs"] == 0, res


FEW, RING64, RING128, TILE = "few", "ring64", "ring128", "tile"


@pytest.mark.parametrize("B,H,W,C,keep,kw,forms", [                     # forms: of the projection, FC1 and FC2
    # C = 512: the projection and FC2 on 256 and 320 tiles of 32 x 32; FC1 on 256 and 272 tiles of 128 x 128; FC2 on 256 and 260; the projection on
    # 384 and 388
    (1, 14, 35, 512, 1.0, {}, (FEW, RING64, FEW)), (1, 7, 91, 512, 1.0, {}, (RING64, RING64, RING64)),
    (1, 35, 56, 512, 0.5, {}, (RING64, RING64, RING64)), (1, 28, 77, 512, 1.0, {}, (RING64, RING128, RING64)),
    (1, 7, 1169, 512, 1.0, {}, (RING64, RING128, RING64)), (1, 84, 98, 512, 1.0, {}, (RING64, RING128, RING128)),
    (1, 70, 175, 512, 1.0, {}, (RING64, RING128, RING128)), (1, 77, 161, 512, 1.0, {}, (RING128, RING128, RING128)),
    (1, 42, 49, 512, 0.5, {}, (RING64, RING128, RING64)), (1, 43, 49, 512, 0.4, {}, (RING64, RING128, RING64)),
    (1, 21, 28, 512, 0.5, {}, (RING64, RING64, RING64)), (1, 21, 35, 512, 1.0, {}, (RING64, RING64, RING64)),
    (2, 63, 105, 512, 0.4, {}, (RING128, RING128, RING128)),            # 420, 1680 and 420 tiles: several a workgroup, both branches
    # C = 768: the projection on 192 and 288 tiles of 32 x 32; FC2 on 480 and 576; FC1 on 240 and 264 of 128 x 128
    (1, 7, 35, 768, 1.0, {}, (FEW, RING64, FEW)), (1, 7, 49, 768, 0.0, {}, (RING64, RING64, FEW)),
    (1, 14, 35, 768, 0.4, {}, (RING64, RING64, FEW)), (1, 14, 42, 768, 0.0, {}, (RING64, RING64, FEW)), (1, 14, 49, 768, 1.0, {}, (RING64, RING64, RING64)),
    (1, 14, 91, 768, 1.0, {}, (RING64, RING64, RING64)), (1, 28, 49, 768, 1.0, {}, (RING64, RING128, RING64)),
    (2, 84, 84, 768, 0.0, dict(bits=(4, 2), wbits=4), (RING128, RING128, RING128)),   # the other branch; rows of the pad
    # C = 1024: the projection on 256 and 384 tiles of 32 x 32; FC2 on 512 and 640; FC1 on 256 and 288 of 128 x 128
    (1, 14, 14, 1024, 0.5, {}, (FEW, RING64, FEW)), (1, 7, 49, 1024, 1.0, {}, (RING64, RING64, FEW)),
    (1, 14, 28, 1024, 0.4, dict(bits=(4, 2), wbits=4), (RING64, RING64, FEW)), (1, 7, 91, 1024, 1.0, {}, (RING64, RING64, RING64)),
    (1, 28, 35, 1024, 0.5, {}, (RING64, RING64, RING64)), (1, 7, 161, 1024, 0.0, {}, (RING64, RING128, RING64)),
    # the cubic on both kinds of tiles
    (1, 43, 49, 512, 0.4, dict(ranges={"a_fc2_in": (-0.07, 0.35)}), (RING64, RING128, RING64)),
    (1, 14, 14, 768, 0.25, dict(ranges={"a_fc2_in": (-0.07, 0.35)}), (RING64, RING64, FEW)),
    (1, 14, 14, 512, 0.25, dict(ranges={"a_fc2_in": (-0.07, 0.35)}), (FEW, RING64, FEW)),
    # other hidden widths: K that the few-rows kernel has not, N = 512 and 256 on both sides of its line, and K that the ring has not
    (2, 14, 21, 768, 0.5, dict(mlp_ratio=1), (RING64, RING64, RING64)), (1, 28, 35, 768, 0.5, dict(mlp_ratio=3), (RING64, RING64, RING64)),
    (1, 14, 35, 512, 1.0, dict(mlp_ratio=6), (FEW, RING64, FEW)), (1, 7, 91, 512, 1.0, dict(mlp_ratio=6), (RING64, RING64, RING64)),
    (1, 28, 35, 256, 0.5, dict(mlp_ratio=8), (TILE, TILE, FEW)), (1, 35, 35, 256, 0.5, dict(mlp_ratio=8), (TILE, TILE, RING64)),
    (1, 14, 14, 1024, 0.5, dict(mlp_ratio=2), (FEW, RING64, FEW)),
    # N = 128: FC2 on 256 and 260, and on 1364 and 1368 tiles of 64 x 64, and on 384 and 385 of 128 x 128
    (1, 7, 1169, 128, 1.0, dict(mlp_ratio=6), (TILE, TILE, RING64)), (1, 84, 98, 128, 1.0, dict(mlp_ratio=5), (TILE, TILE, TILE)),
    (1, 70, 623, 128, 1.0, dict(mlp_ratio=8), (TILE, TILE, TILE)), (1, 189, 231, 128, 1.0, dict(mlp_ratio=6), (TILE, TILE, RING64)),
    (1, 119, 413, 128, 1.0, dict(mlp_ratio=8), (TILE, TILE, RING64)), (1, 28, 1757, 128, 1.0, dict(mlp_ratio=7), (TILE, TILE, RING128)),
    (2, 35, 35, 192, 0.5, dict(mlp_ratio=7), (TILE, TILE, TILE)), (2, 70, 84, 192, 0.5, dict(mlp_ratio=5), (TILE, TILE, TILE)),
    (1, 35, 35, 96, 0.5, dict(mlp_ratio=7), (TILE, TILE, TILE))])
def test_products_of_the_separate_kernels_at_their_lines(B, H, W, C, keep, kw, forms):
    """The kernels of the linear layers on both sides of the lines between them; which one a case takes is asked of the library's own rule."""
    spec, inp, x, k = _case(B, H, W, C, C // 32, 3 if H > 7 else 0, keep, 60, blobs=True, **kw)
    assert product_plan.forms(spec, k) == forms
    print("products", B, H, W, C, keep, kw, flush=True)
    res = gh.compare_block(inp, x, k, taps=("acc_proj", "h", "a_fc1_in", "a_fc2_in", "acc_fc2"))
    print(res, flush=True)
    gh.assert_parity(res)


def test_long_k_on_a_few_hundred_row_tiles():
    """FC2 with K = 3072 behind a projection and an FC1 of the tile kernel: 112 x 6 tiles of 64 x 64, 24 stages of the ring kernel."""
    spec, inp, x, k = _case(2, 50, 60, 384, 12, 3, 0.5, 54, blobs=True, mlp_ratio=8)
    assert product_plan.rows(spec, k) == 112 * 64 and product_plan.forms(spec, k) == (TILE, TILE, RING64)
    print("long K on many tiles", flush=True)
    res = gh.compare_block(inp, x, k)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("score_mode,value", [(0, float("nan")), (1, float("inf"))])
def test_window_whose_score_is_not_a_number(score_mode, value, fused):
    """A NaN in the map (or an Inf under the scoring LayerNorm) gives a NaN score: that window is ranked last,
    the list stays a permutation, every kernel exits normally and all other windows match the oracle."""
    import oracle_api as O
    spec, inp, x, k = _case(2, 28, 35, 96, 3, 0, 0.5, 53, blobs=True, mode=score_mode)
    x = x.copy()
    x[1, 9, 16, 5] = value                                 # window (1, 2) of image 1
    bad_w = 1 * 5 + 2
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    print("NaN score case", score_mode, value, "fused", fused, flush=True)
    with gh.GpuBlock(inp, fused=fused) as gb:
        scores, perm = gb.score_select(xt, k)
        y = gb.forward(xt, perm, k)
        y2 = gb.forward(xt, None, k)                       # selection inside the call
        torch.cuda.synchronize()
    o_scores = O.score_windows(inp, x)
    assert np.isnan(o_scores[1, bad_w]) and np.isnan(o_scores).sum() == 1
    g_scores = scores.cpu().numpy()
    assert np.array_equal(np.isnan(g_scores), np.isnan(o_scores))
    o_perm = O.select_windows(o_scores, k)
    assert np.array_equal(perm.cpu().numpy(), o_perm) and o_perm[1, -1] == bad_w
    oy, _ = O.block_forward(inp, x, o_perm, k)
    yn = y.cpu().numpy()
    other = np.ones(yn.shape, dtype=bool)
    other[1, 7:14, 14:21] = False
    assert np.array_equal(yn[other], oy[other])
    assert np.array_equal(np.isnan(yn), np.isnan(oy))
    fin = ~np.isnan(oy)
    assert np.array_equal(yn[fin], oy[fin])
    assert np.array_equal(np.isnan(y2.cpu().numpy()), np.isnan(oy)) and torch.equal(torch.nan_to_num(y), torch.nan_to_num(y2))


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("shift", [0, 3])
def test_config2_full_size(shift, fused):
    """Swin-T stage 1 at detection scale, the size the benchmark times."""
    spec, inp, x, k = _case(1, 200, 336, 96, 3, shift, 0.5, 1002, blobs=True)
    print("config 2 shift", shift, "fused", fused, flush=True)
    res = gh.compare_block(inp, x, k, fused=fused)
    print(res, flush=True)
    gh.assert_parity(res)


def test_maximum_window_count():
    """4096 windows per image is the most the selection handles (448x448 map, shifted); more is refused."""
    spec, inp, x, k = _case(1, 448, 448, 96, 3, 3, 0.5, 23, blobs=True)
    assert spec.nW == 4096
    print("maximum window count", flush=True)
    res = gh.compare_block(inp, x, k, taps=("a_proj_in", "a_fc2_in"))
    print(res, flush=True)
    gh.assert_parity(res)
    sh, br = M.to_device(inp)
    with pytest.raises(M.MixaqError) as e:
        M.mixaq_block_create(M.make_desc(synth.BlockSpec(1, 455, 448, 96, 3)), sh, br)
    assert e.value.code == -2


def test_order_invariance_and_reverse_selection():
    spec, inp, x, k = _case(2, 26, 33, 96, 3, 3, 0.4, 21, blobs=True)
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    import oracle_api as O
    with gh.GpuBlock(inp) as gb:
        scores, perm = gb.score_select(xt, k)
        y0 = gb.forward(xt, perm, k)
        rng = np.random.default_rng(0)
        p2 = perm.cpu().numpy().copy()
        for b in range(2):
            p2[b, :k] = rng.permutation(p2[b, :k])
            p2[b, k:] = rng.permutation(p2[b, k:])
        y1 = gb.forward(xt, torch.from_numpy(p2).to(dev), k)
        torch.cuda.synchronize()
        assert torch.equal(y0, y1)
        _, rperm = gb.score_select(xt, k, reverse=1)
        assert np.array_equal(rperm.cpu().numpy(), O.select_windows(scores.cpu().numpy(), k, 1))


def test_error_paths_do_not_launch():
    spec, inp, x, k = _case(1, 14, 14, 96, 3, 0, 0.5, 22)
    sh, br = M.to_device(inp)
    d = M.make_desc(spec)
    d.act_bits_low = 9
    with pytest.raises(M.MixaqError) as e:
        M.mixaq_block_create(d, sh, br)
    assert e.value.code == -3
    d = M.make_desc(spec)
    d.C = 100
    with pytest.raises(M.MixaqError) as e:
        M.mixaq_block_create(d, sh, br)
    assert e.value.code == -2
    d = M.make_desc(spec, shift=3)
    d.H = 7
    with pytest.raises(M.MixaqError):
        M.mixaq_block_create(d, sh, br)
    with gh.GpuBlock(inp) as gb:
        xt = torch.from_numpy(x).cuda()
        y = torch.empty_like(xt)
        small = torch.empty(1024, dtype=torch.uint8, device="cuda")
        with pytest.raises(M.MixaqError) as e:
            M.mixaq_block_forward(gb.blk, xt, None, k, y, small)
        assert e.value.code == -4
        with pytest.raises(M.MixaqError) as e:
            M.mixaq_block_forward(gb.blk, xt, None, 99, y, gb.ws)
        assert e.value.code == -2
        with pytest.raises(M.MixaqError) as e:
            M.mixaq_block_forward(gb.blk, xt, None, k, xt, gb.ws)
        assert e.value.code == -2
        # the stage call: x, y and tmp must be three separate maps; blocks of another shape are refused
        scores = torch.empty((1, spec.nW), dtype=torch.float64, device="cuda")
        perm = torch.empty((1, spec.nW), dtype=torch.int32, device="cuda")
        tmp = torch.empty_like(xt)
        for bad in ((xt, xt, tmp), (xt, y, y), (xt, y, xt)):
            with pytest.raises(M.MixaqError) as e:
                M.mixaq_stage_forward([gb.blk, gb.blk], bad[0], [k], None, bad[1], bad[2], scores, perm, gb.ws)
            assert e.value.code == -2
        with pytest.raises(M.MixaqError) as e:
            M.mixaq_stage_forward([gb.blk, gb.blk], xt, [spec.nW + 1], None, y, tmp, scores, perm, gb.ws)
        assert e.value.code == -2
        M.mixaq_stage_forward([gb.blk, gb.blk], xt, [k], None, y, tmp, scores, perm, gb.ws)      # and the good call still runs
        torch.cuda.synchronize()


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("shift,kh_frac,kl_frac", [(0, 0.3, 0.4), (3, 0.25, 0.5), (3, 0.0, 0.0), (0, 0.5, 0.0)])
def test_activation_pruning_matches_oracle(shift, kh_frac, kl_frac, fused):
    """Three-way split (Sec. 3.4): high, low, pruned windows; pruned features are forwarded."""
    import oracle_api as O
    spec, inp, x, _ = _case(2, 26, 33, 96, 3, shift, 0.5, 31, blobs=True)
    nW = spec.nW
    kh, kl = int(kh_frac * nW), int(kl_frac * nW)
    print("pruning case shift", shift, "k_high", kh, "k_low", kl, "fused", fused, flush=True)
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    with gh.GpuBlock(inp, fused=fused) as gb:
        scores = torch.empty((2, nW), dtype=torch.float64, device=dev)
        perm = torch.empty((2, nW), dtype=torch.int32, device=dev)
        M.mixaq_score_windows(gb.blk, xt, scores)
        M.mixaq_select_windows3(scores, 2, nW, kh, kl, 0, perm)
        y = torch.full_like(xt, float("nan"))
        M.mixaq_block_forward_pruned(gb.blk, xt, perm, kh, kl, y, gb.ws)
        y2 = torch.full_like(xt, float("nan"))
        M.mixaq_block_forward_pruned(gb.blk, xt, None, kh, kl, y2, gb.ws)          # internal three-way selection
        torch.cuda.synchronize()
    o_perm = O.select_windows(O.score_windows(inp, x), kh, k_low=kl)
    assert np.array_equal(perm.cpu().numpy(), o_perm)
    oy, _ = O.block_forward(inp, x, o_perm, kh, k_low=kl)
    assert np.array_equal(y.cpu().numpy(), oy)
    assert torch.equal(y, y2)


@pytest.mark.parametrize("C,heads", [(96, 3), (128, 4), (384, 12), (768, 24)])
@pytest.mark.parametrize("shift,kh_frac,kl_frac", [(0, 0.5, -1), (3, 0.25, 0.5), (3, 0.0, 0.0)])
def test_forward_from_scores_matches_oracle(C, heads, shift, kh_frac, kl_frac):
    """The selection taken inside the first kernel from the stage's scores gives the oracle's block output."""
    import oracle_api as O
    spec, inp, x, _ = _case(2, 26, 33, C, heads, shift, 0.5, 41, blobs=True)
    nW = spec.nW
    kh = int(kh_frac * nW)
    kl = -1 if kl_frac < 0 else int(kl_frac * nW)
    print("scored case", C, shift, kh, kl, flush=True)
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    with gh.GpuBlock(inp) as gb:
        scores = torch.empty((2, nW), dtype=torch.float64, device=dev)
        M.mixaq_score_windows(gb.blk, xt, scores)
        y = torch.full_like(xt, float("nan"))
        perm_out = torch.full((2, nW), -1, dtype=torch.int32, device=dev)
        M.mixaq_block_forward_scored(gb.blk, xt, scores, kh, kl, y, gb.ws, perm_out=perm_out)
        torch.cuda.synchronize()
    o_perm = O.select_windows(O.score_windows(inp, x), kh, k_low=None if kl < 0 else kl)
    assert np.array_equal(perm_out.cpu().numpy(), o_perm)
    oy, _ = O.block_forward(inp, x, o_perm, kh, k_low=None if kl < 0 else kl)
    assert np.array_equal(y.cpu().numpy(), oy)


@pytest.mark.parametrize("B,H,W,C,heads", [(1, 84, 84, 384, 12), (1, 161, 165, 192, 6), (3, 50, 57, 256, 8)])
def test_forward_from_scores_past_the_small_map_forms(B, H, W, C, heads):
    """The in-kernel selection in the kernel forms of larger maps: one twelve-head workgroup per window (more than
    128 windows at C = 384), one wave per head at C = 192 (more than 512 windows), eight heads; shifted block, pruning."""
    import oracle_api as O
    spec, inp, x, _ = _case(B, H, W, C, heads, 3, 0.5, 43, blobs=True)
    nW = spec.nW
    kh, kl = int(0.4 * nW), int(0.45 * nW)
    print("scored case", C, B * nW, "windows", flush=True)
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    with gh.GpuBlock(inp) as gb:
        scores = torch.empty((B, nW), dtype=torch.float64, device=dev)
        M.mixaq_score_windows(gb.blk, xt, scores)
        y = torch.full_like(xt, float("nan"))
        perm_out = torch.full((B, nW), -1, dtype=torch.int32, device=dev)
        M.mixaq_block_forward_scored(gb.blk, xt, scores, kh, kl, y, gb.ws, perm_out=perm_out)
        torch.cuda.synchronize()
    o_perm = O.select_windows(O.score_windows(inp, x), kh, k_low=kl)
    assert np.array_equal(perm_out.cpu().numpy(), o_perm)
    oy, _ = O.block_forward(inp, x, o_perm, kh, k_low=kl, threads=16)
    assert np.array_equal(y.cpu().numpy(), oy)


# the FC2 input's range: None, or one too narrow for a table of steps.  Blocks with a table are one kernel on some of these numbers of windows; those
# without take the window kernel's forms there.
NO_STEPS = {"a_fc2_in": (-0.07, 0.35)}


@pytest.mark.parametrize("C,rows,cols,hidden", [
    *((*m, None) for m in [(96, 16, 32), (96, 19, 27), (128, 8, 16), (128, 3, 43), (128, 16, 16), (128, 6, 43), (128, 16, 24), (128, 11, 35),
                           (128, 16, 32), (128, 19, 27), (192, 16, 16), (192, 6, 43), (192, 16, 32), (192, 19, 27),
                           (384, 8, 16), (384, 3, 43), (384, 11, 15), (384, 12, 15), (384, 15, 22), (384, 17, 21), (384, 20, 26)]),
    *((*m, NO_STEPS) for m in [(96, 16, 32), (128, 16, 16), (128, 16, 32), (192, 16, 16)])])
def test_forms_of_the_fused_kernels_on_both_sides_of_their_lines(C, rows, cols, hidden):
    """One block on the largest and next larger number of windows of every form of the window kernel, and of 32 and 64 rows of the token
    kernel, given a list, given scores and with pruned windows: the oracle's bits."""
    import oracle_api as O
    dev = torch.device("cuda:0")
    spec, inp, x_np, k = _case(1, 7 * rows - 3, 7 * cols - 2, C, C // 32, 3, 0.4, 700 + cols, blobs=True, ranges=hidden)
    assert spec.nW == rows * cols
    print("forms", C, spec.nW, flush=True)
    sc = O.score_windows(inp, x_np)
    x = torch.from_numpy(x_np).to(dev)
    with gh.GpuBlock(inp) as gb:
        for k_low in (spec.nW - k, spec.nW // 3):
            perm_o = O.select_windows(sc, k, k_low=k_low)
            want, _ = O.block_forward(inp, x_np, perm_o, k, 3, threads=16, k_low=k_low)
            scores, perm = gb.score_select(x, k)
            y = gb.forward_pruned(x, perm, k, k_low)
            y2, p2 = torch.full_like(x, float("nan")), torch.full_like(perm, -1)
            M.mixaq_block_forward_scored(gb.blk, x, scores, k, k_low, y2, gb.ws, perm_out=p2)
            torch.cuda.synchronize()
            assert np.array_equal(perm.cpu().numpy(), perm_o) and torch.equal(p2, perm)
            assert np.array_equal(y.cpu().numpy(), want) and torch.equal(y, y2)


def test_equal_scores_are_ordered_by_window_index():
    """Windows with exactly equal scores (here: windows that are zero everywhere, and two copies of one
    window) must be ranked by their index on both sides; the block output follows."""
    spec, inp, x, _ = _case(2, 35, 42, 96, 3, 3, 0.5, 61, blobs=True)
    x = x.copy()
    x[:, 7:21, 14:35, :] = 0.0                       # six whole windows of the un-shifted grid, score 0
    x[:, 28:35, 0:7, :] = x[:, 0:7, 0:7, :]          # window 20 repeats window 0
    for k in (3, 12, 26):                            # the cut falls before, inside and after the tied windows
        print("tie case k_high", k, flush=True)
        res = gh.compare_block(inp, x, k, taps=("a_proj_in",))
        print(res, flush=True)
        gh.assert_parity(res)
        assert res["y_internal_select_equal"]


@pytest.mark.parametrize("case", range(8))
def test_random_shapes_and_precisions(case):
    """Seeded random draws of batch, map size (padding in both directions), width, shift, keep ratio and bit
    widths: every tap and the output against the oracle."""
    rng = np.random.default_rng(9000 + case)
    C, heads = [(96, 3), (128, 4), (192, 6), (256, 8)][int(rng.integers(0, 4))]
    B = int(rng.integers(1, 4))
    H, W = int(rng.integers(14, 40)), int(rng.integers(14, 40))
    shift = int(rng.integers(0, 2)) * 3
    keep = float(rng.choice([0.0, 0.2, 0.5, 0.8, 1.0]))
    hi = int(rng.integers(4, 9))
    lo = int(rng.integers(2, hi + 1))
    wbits = int(rng.choice([4, 8]))
    spec, inp, x, k = _case(B, H, W, C, heads, shift, keep, 9100 + case, blobs=bool(rng.integers(0, 2)), bits=(hi, lo), wbits=wbits,
                            mode=int(rng.integers(0, 2)))
    print("random case", case, B, H, W, C, shift, keep, hi, lo, wbits, flush=True)
    res = gh.compare_block(inp, x, k)
    print(res, flush=True)
    gh.assert_parity(res)


def test_random_sweep_of_small_blocks():
    """Forty more seeded draws in one test, wider than the cases above: maps from 7x7 up, C = 384 too, either
    implementation, shared or independent biases, outlier channels.  (A one-off run of 1800 such draws during
    development found no mismatch.)"""
    for case in range(40):
        rng = np.random.default_rng(31000 + case)
        C, heads = [(96, 3), (128, 4), (192, 6), (256, 8), (384, 12)][int(rng.choice([0, 0, 1, 2, 3, 4]))]
        B = int(rng.integers(1, 4))
        H, W = int(rng.integers(7, 46)), int(rng.integers(7, 46))
        shift = int(rng.integers(0, 2)) * 3
        if (H + 6) // 7 * 7 < 14 or (W + 6) // 7 * 7 < 14:
            shift = 0                                  # a shifted block needs a padded map of at least 14x14
        keep = float(rng.choice([0.0, 0.2, 0.5, 0.8, 1.0]))
        hi = int(rng.integers(4, 9))
        lo = int(rng.integers(2, hi + 1))
        fused = bool(rng.integers(0, 4) != 0)
        spec, inp, x, k = _case(B, H, W, C, heads, shift, keep, 31100 + case, blobs=bool(rng.integers(0, 2)),
                                outliers=bool(rng.integers(0, 3) == 0), bits=(hi, lo), wbits=int(rng.choice([4, 8])),
                                mode=int(rng.integers(0, 2)), per_branch_bias=bool(rng.integers(0, 2)))
        print("sweep case", case, B, H, W, C, shift, keep, hi, lo, "fused", fused, flush=True)
        res = gh.compare_block(inp, x, k, fused=fused)
        gh.assert_parity(res)


@pytest.mark.parametrize("kind", ["zeros", "constant_tokens", "huge", "denormal", "one_hot"])
def test_degenerate_inputs(kind):
    """Inputs at the edges of the float arithmetic: zero variance (rstd = 1/sqrt(eps)), saturated quantizers,
    binary32 denormals, a single non-zero channel."""
    spec, inp, x, k = _case(1, 21, 30, 96, 3, 3, 0.5, 71)
    rng = np.random.default_rng(72)
    if kind == "zeros":
        x = np.zeros_like(x)
    elif kind == "constant_tokens":
        x = np.repeat(rng.standard_normal(x.shape[:3] + (1,)).astype(np.float32), 96, axis=3)
    elif kind == "huge":
        x = (x * np.float32(3e4)).astype(np.float32)
    elif kind == "denormal":
        x = (x.astype(np.float64) * 1e-39).astype(np.float32)
        assert np.any((x != 0) & (np.abs(x) < 1.1754944e-38))
    else:
        x = np.zeros_like(x)
        x[..., 5] = rng.standard_normal(x.shape[:3]).astype(np.float32) * 10
    print("degenerate input", kind, flush=True)
    res = gh.compare_block(inp, np.ascontiguousarray(x), k)
    print(res, flush=True)
    assert res["perm_mismatch"] == 0 and res["y_nan"] == 0
    for n in gh.INT_TAPS:
        assert res[n] == 0, (n, res)
    assert res["y_bit_identical"], res


@pytest.mark.parametrize("kind", ["plus_inf", "minus_inf", "nan", "overflow", "huge", "products", "tiny_step"])
@pytest.mark.parametrize("C,heads,fused", [(96, 3, True), (96, 3, False), (384, 12, True), (768, 24, None)])
def test_logits_that_are_no_ordinary_numbers(C, heads, fused, kind):
    """Infinities, NaN and overflowing values in the relative position bias, products of q and k that overflow the logits, and
    probability steps below 2^-100: the softmax's exponents are held at their floor, as the definition says, and every tap is
    the oracle's."""
    spec, inp, x, k = _case(2, 14, 21, C, heads, 3, 0.5, 81, blobs=True)
    rng = np.random.default_rng(82)
    rpb = inp.shared.rel_pos_bias.copy()
    some = rng.random(rpb.shape) < 0.02
    if kind == "plus_inf":
        rpb[some] = np.inf                       # some rows with one or two of them, some with none
    elif kind == "minus_inf":
        rpb[some] = -np.inf
        rpb[0, 3, :] = -np.inf                   # a row that shuts every key out
    elif kind == "nan":
        rpb[some] = np.nan
    elif kind == "overflow":
        rpb[some] = 3e38                         # finite, infinite times log2(e)
    elif kind == "huge":
        rpb[some] = 2e38
        rpb[rng.random(rpb.shape) < 0.02] = -2e38
    elif kind == "products":                     # q and k in steps of about 1e17: the largest products overflow, the others do not
        inp.shared.s_qkv = inp.shared.s_qkv.copy()
        inp.shared.s_qkv[:2 * C] *= np.float32(1e19)
        for br in inp.branches:
            for n in ("a_q", "a_k"):
                br.q[n] = (br.q[n][0] * 1e19, 0)
    else:
        for br in inp.branches:
            br.q["a_p"] = (2.0 ** -101, 0)       # every probability but 2^-100 and less saturates
    inp.shared.rel_pos_bias = rpb
    print("logits", kind, "C", C, "fused", fused, flush=True)
    res = gh.compare_block(inp, x, k, fused=fused)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("span,kind", [(32.5, "bias"), (33.5, "bias"), (35.0, "bias"), (94.0, "plain"), (101.0, "plain"), (400.0, "plain"), (30.0, "made_up")])
@pytest.mark.parametrize("C,heads,fused,bits", [(96, 3, True, (8, 4)), (96, 3, False, (8, 4)), (384, 12, True, (4, 2))])
def test_exponents_around_the_lines_of_their_floor(C, heads, fused, bits, span, kind):
    """Products of q and k that span `span` exponents with saturated codes, on both sides of the lines from which windows with
    masked pairs (33) and all windows (99 with the bias) hold their exponents at the floor, and a bias that makes up for the mask
    of some pairs.  Every tap is the oracle's."""
    spec, inp, x, k = _case(2, 14, 21, C, heads, 3, 0.5, 83, blobs=True, bits=bits)
    rng = np.random.default_rng(84)
    steps = []
    for br, b in zip(inp.branches, bits):        # span = 2 * 32 * 2^(2 b - 2) * s_q * s_k * log2(e) / sqrt(32)
        s = float(np.sqrt(span * np.sqrt(32.0) / (1.442695 * 64 * 4.0 ** (b - 1))))
        steps.append(s / br.q["a_q"][0])
        br.q["a_q"], br.q["a_k"] = (s * 1.0625, 0), (s / 1.0625, 0)
    inp.shared.s_qkv = inp.shared.s_qkv.copy()
    inp.shared.s_qkv[:2 * C] *= np.float32(3.0 * max(steps))
    rpb = inp.shared.rel_pos_bias.copy()
    if kind == "bias":
        rpb *= np.float32(4.0)
    elif kind == "plain":
        rpb *= np.float32(0.25)
    else:
        rpb[rng.random(rpb.shape) < 0.05] += np.float32(130.0)
    inp.shared.rel_pos_bias = rpb
    print("floor lines", span, kind, "C", C, "fused", fused, "bits", bits, flush=True)
    res = gh.compare_block(inp, x, k, fused=fused)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("B,H,W,C,mode", [(9, 56, 63, 768, 1), (10, 56, 63, 768, 1), (10, 56, 63, 768, 0), (4, 130, 140, 384, 1), (5, 82, 91, 1024, 1)])
def test_scores_of_wide_maps_on_both_sides_of_the_workgroup_size(B, H, W, C, mode):
    """Wide maps are scored by 1024 threads per window, large ones with the scoring LayerNorm by 256."""
    import oracle_api as O
    spec, inp, x, k = _case(B, H, W, C, C // 32, 0, 0.5, 45, blobs=True, mode=mode)
    print("scores", B, H, W, C, "mode", mode, "windows times channels", B * spec.nW * C, flush=True)
    with gh.GpuBlock(inp) as gb:
        scores, perm = gb.score_select(torch.from_numpy(x).cuda(), k)
        torch.cuda.synchronize()
    want = O.score_windows(inp, x)
    assert np.max(np.abs(scores.cpu().numpy() - want) / want) <= 1e-12
    assert np.array_equal(perm.cpu().numpy(), O.select_windows(want, k))


WIDE_CASES = [
    # B, H, W, C, shift, keep, bits, kwargs: the default path of the wide blocks (LN1, then a window's heads over several workgroups)
    (2, 21, 28, 512, 3, 0.4, (7, 3), {}),
    (1, 7, 7, 512, 0, 1.0, (8, 4), {}),                               # a single window
    (3, 33, 40, 512, 3, 0.0, (4, 2), dict(wbits=4)),                  # 90 windows, everything low
    (1, 14, 21, 1024, 3, 0.5, (8, 4), {}),
    (2, 20, 27, 1024, 0, 0.3, (4, 2), dict(wbits=4, per_branch_bias=True)),
    (2, 20, 27, 768, 3, 1.0, (6, 3), dict(mode=1)),
    (1, 20, 27, 512, 3, 0.5, (8, 4), dict(mlp_ratio=3)),
    # both sides of 256 workgroups of four heads each
    (1, 56, 56, 512, 3, 0.5, (8, 4), {}), (1, 35, 91, 512, 0, 0.4, (8, 4), {}),        # 64 and 65 windows
    (1, 42, 49, 768, 3, 0.5, (8, 4), {}), (1, 7, 301, 768, 0, 0.4, (8, 4), {}),        # 42 and 43
    (1, 28, 56, 1024, 3, 0.5, (8, 4), {}), (1, 21, 77, 1024, 3, 0.4, (8, 4), {}),      # 32 and 33
]


@pytest.mark.parametrize("B,H,W,C,shift,keep,bits,kw", WIDE_CASES)
def test_wide_blocks_on_their_default_path(B, H, W, C, shift, keep, bits, kw):
    spec, inp, x, k = _case(B, H, W, C, C // 32, shift, keep, 46, bits=bits, blobs=True, **kw)
    print("wide block", B, H, W, C, shift, keep, bits, kw, flush=True)
    res = gh.compare_block(inp, x, k)
    print(res, flush=True)
    gh.assert_parity(res)


@pytest.mark.parametrize("C,heads", [(512, 16), (1024, 32)])
@pytest.mark.parametrize("shift,kh_frac,kl_frac", [(0, 0.5, -1), (3, 0.25, 0.5), (3, 0.0, 0.0)])
def test_wide_blocks_from_scores_and_lists_with_pruning(C, heads, shift, kh_frac, kl_frac):
    """Selection inside the call and from a list, pruned windows forwarded, at the widths the case above does not cover."""
    import oracle_api as O
    spec, inp, x, _ = _case(2, 26, 33, C, heads, shift, 0.5, 47, blobs=True)
    nW = spec.nW
    kh = int(kh_frac * nW)
    kl = nW - kh if kl_frac < 0 else int(kl_frac * nW)
    print("wide block, scores", C, shift, kh, kl, flush=True)
    dev = torch.device("cuda:0")
    xt = torch.from_numpy(x).to(dev)
    with gh.GpuBlock(inp) as gb:
        scores = torch.empty((2, nW), dtype=torch.float64, device=dev)
        M.mixaq_score_windows(gb.blk, xt, scores)
        y = torch.full_like(xt, float("nan"))
        perm = torch.full((2, nW), -1, dtype=torch.int32, device=dev)
        M.mixaq_block_forward_scored(gb.blk, xt, scores, kh, kl, y, gb.ws, perm_out=perm)
        y_list = gb.forward_pruned(xt, perm, kh, kl)
        torch.cuda.synchronize()
    o_perm = O.select_windows(O.score_windows(inp, x), kh, k_low=kl)
    assert np.array_equal(perm.cpu().numpy(), o_perm)
    oy, _ = O.block_forward(inp, x, o_perm, kh, k_low=kl, threads=16)
    assert np.array_equal(y.cpu().numpy(), oy)
    assert torch.equal(y, y_list)


@pytest.mark.parametrize("C,heads,mlp_ratio", [(96, 3, 4), (384, 12, 3), (768, 24, 4)])
def test_switching_between_the_implementations_and_back(C, heads, mlp_ratio):
    """mixaq_block_set_fused is accepted in both directions at every width and gives the same bits; 1 is the default again."""
    spec, inp, x, k = _case(2, 20, 27, C, heads, 3, 0.5, 48, blobs=True, mlp_ratio=mlp_ratio)
    xt = torch.from_numpy(x).cuda()
    print("switching", C, mlp_ratio, flush=True)
    with gh.GpuBlock(inp) as gb:
        outs, names = [], []
        for enable in (None, 0, 1):
            if enable is not None:
                M.mixaq_block_set_fused(gb.blk, enable)
            outs.append(gb.forward(xt, None, k))
            y = torch.empty_like(xt)
            ms = M.mixaq_block_forward_profile(gb.blk, xt, None, k, y, gb.ws, repeats=1)
            names.append({n for n, v in ms.items() if v > 0})
        torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert names[0] == names[2] and "window_ln1_qkv_attention" in names[0]
    assert "window_ln1_qkv_attention" not in names[1] and "qkv_gemm" in names[1]
