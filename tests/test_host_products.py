"""How products are cut into tiles (pie_product_plan), without a GPU."""
import pytest

from paper_2510_24051_amd import PieError, product_plan

WS = 256 * 28672 * 8  # the 8B-shaped layer's workspace
LM_HEAD = [(128256, 4096), (32000, 2048), (128256, 8192)]


@pytest.mark.parametrize("n_out,k", LM_HEAD + [(28672, 4096), (4096, 14336), (6144, 4096), (1184, 320), (96, 64)])
@pytest.mark.parametrize("rows", [65, 97, 129, 192, 257, 384, 512, 1024, 4100])
def test_the_row_tiles_of_a_column_meet_in_one_l2(rows, n_out, k):
    """However many tiles there are (128256 columns are 501 tiles, 32000 are 125), a column tile of the weights is fetched by
    one XCD, and by two where an XCD's range begins."""
    p = product_plan(rows, n_out, k, WS)
    tiles_n = (n_out + 255) // 256
    tiles_m = -(-(p["whole_rows"] or rows) // p["tile_rows"])
    bands = -(-tiles_m // 8)  # rows of tiles are taken eight at a time
    assert p["column_fetches"] <= p["splits"] * (bands * tiles_n + 8), p


def test_product_plan_arguments():
    assert product_plan(64, 4096, 4096, WS)["tile_rows"] == 0    # weight-streaming
    assert product_plan(300, 4096, 4096 + 32, WS)["tile_rows"] == 0  # contraction not a multiple of 64
    assert product_plan(300, 4096, 14336, 0)["splits"] == 1      # no room for partial sums
    for bad in ((0, 32, 64, 0), (1, 0, 64, 0), (1, 32, 0, 0), (1, 32, 63, 0), (1, 32, 64, -1)):
        with pytest.raises(PieError):
            product_plan(*bad)
    with pytest.raises(PieError):
        product_plan(1, 32, 64, 0, n_cus=0)
