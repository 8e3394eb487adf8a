"""Split products that gain nothing from cutting tiles along k run whole, one
workgroup per tile (also where that is many rounds of 256), and those that do
are cut; results against numpy within the bars of the tile tests."""
import pytest

from test_gpu_split_products import CODES, lib, run  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,M,N,K,cut", [
    ("bf16x3", 540, 3160, 3160, False), ("bf16x2", 540, 3160, 3160, False), ("fp32", 540, 3160, 3160, False),
    ("bf16x3", 704, 704, 704, False), ("bf16x2", 704, 704, 704, False), ("fp32", 704, 704, 704, True),
    ("bf16x3", 45, 3160, 3160, True), ("bf16x2", 45, 3160, 3160, True)])
def test_cut_where_it_pays(lib, prec, M, N, K, cut):  # noqa: F811
    run(lib, prec, 0, 256, M, N, K, 0, cut)


@pytest.mark.parametrize("prec", list(CODES))
@pytest.mark.parametrize("bm", [64, 96, 128])
# 256 tiles and one, and 2300 to 4600 of them: several rounds of workgroups, none cut
@pytest.mark.parametrize("M,N,K", [(130, 11000, 40), (4600, 8000, 70)])
def test_many_whole_tiles(lib, prec, bm, M, N, K):  # noqa: F811
    run(lib, prec, bm, 0, M, N, K, 1, False)
