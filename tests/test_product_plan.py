"""Which kernel takes a linear layer: both sides of every line of the rule, at the sizes that the GPU tests run.  CPU only."""
import pytest

import product_plan as P

R = 128                                                   # rows come in whole 128s


@pytest.mark.parametrize("C,few", [(512, 512), (768, 256), (1024, 256)])
def test_projection(C, few):
    """32 x 32 tiles up to one a CU; 128 x 128 tiles from one and a half a CU."""
    assert P.form(P.PROJ, few, C, C) == "few" and P.form(P.PROJ, few + R, C, C) == "ring64"
    most = 384 * 128 // C * 128
    assert P.form(P.PROJ, most, C, C) == "ring64" and P.form(P.PROJ, most + R, C, C) == "ring128"


@pytest.mark.parametrize("C,most", [(512, 2048), (768, 1280), (1024, 1024)])
def test_fc1(C, most):
    assert P.form(P.FC1, R, 4 * C, C) == "ring64"
    assert P.form(P.FC1, most, 4 * C, C) == "ring64" and P.form(P.FC1, most + R, 4 * C, C) == "ring128"


@pytest.mark.parametrize("N,K,few", [(512, 2048, 512), (512, 3072, 512), (512, 4096, 512), (256, 2048, 1024), (768, 3072, 640), (1024, 2048, 512),
                                     (1024, 3072, 512), (1024, 4096, 512)])
def test_fc2(N, K, few):
    """32 x 32 tiles up to one a CU, up to two where a row's tiles are 24 or more; 128 x 128 tiles beyond one a CU."""
    assert P.form(P.FC2, few, N, K) == "few" and P.form(P.FC2, few + R, N, K) == "ring64"
    most = 256 * 128 // N * 128 // R * R
    assert P.form(P.FC2, most, N, K) == "ring64" and P.form(P.FC2, most + R, N, K) == "ring128"


@pytest.mark.parametrize("K", [640, 768, 896, 1024])
def test_fc2_of_128_channels(K):
    """64 x 64 tiles up to one a CU and from five and a third, row tiles of all channels between; 128 x 128 tiles from one and a half a CU."""
    few, many, most = 256 * 64 * 64 // 128, 341 * 128, 384 * 128
    assert P.form(P.FC2, R, 128, K) == P.form(P.FC2, few, 128, K) == "ring64"
    assert P.form(P.FC2, few + R, 128, K) == P.form(P.FC2, many, 128, K) == "tile"
    assert P.form(P.FC2, many + R, 128, K) == P.form(P.FC2, most, 128, K) == "ring64"
    assert P.form(P.FC2, most + R, 128, K) == "ring128"


@pytest.mark.parametrize("epi,N,K,want", [
    (P.QKV, 1536, 512, "ring64"), (P.QKV, 1152, 384, "tile"),
    (P.FC2, 96, 768, "tile"), (P.FC2, 192, 1344, "tile"), (P.FC2, 192, 1536, "ring64"), (P.FC2, 192, 960, "tile"), (P.FC2, 128, 512, "ring64"),
    (P.FC2, 128, 384, "tile"), (P.FC2, 768, 768, "ring64"), (P.FC2, 384, 3072, "ring64"), (P.FC1, 96, 96, "tile")])
def test_kinds_of_sizes(epi, N, K, want):
    """The ring takes K from 512 in whole 128s and N in whole 64s, the few-rows kernel N in whole 256s; tiles take the rest."""
    assert P.form(epi, 256, N, K) == want
