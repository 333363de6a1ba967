"""How products are cut into tiles (pie_product_plan), without a GPU."""
import numpy as np
import pytest

from paper_2510_24051_amd import PieError, product_plan, product_stream

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


# (rows, n_out, k, {(rows of a tile, parts of K): us}): the faster forms as measured on the device, weights from HBM
MEASURED = [
    (160, 28672, 4096, {(96, 1): 61, (128, 1): 67, (96, 2): 74, (128, 2): 75, (256, 2): 74, (256, 1): 96}),
    (900, 28672, 4096, {(96, 1): 219, (128, 1): 204, (256, 1): 198, (256, 2): 263}),
    (1024, 28672, 4096, {(96, 1): 231, (128, 1): 210, (256, 1): 202, (256, 2): 277}),
    (3072, 28672, 4096, {(96, 1): 642, (128, 1): 570, (256, 1): 578}),
    (448, 57344, 8192, {(96, 1): 464, (128, 1): 414, (256, 1): 410, (256, 2): 475}),
    (768, 57344, 8192, {(96, 1): 670, (128, 1): 618, (256, 1): 610, (256, 2): 720}),
    (1536, 57344, 8192, {(96, 1): 1264, (128, 1): 1165, (256, 1): 1162}),
    (3072, 10240, 8192, {(96, 1): 446, (128, 1): 397, (256, 1): 388, (256, 2): 490}),
    (5000, 6144, 4096, {(96, 1): 212, (128, 1): 204, (256, 1): 201}),
    (6144, 6144, 4096, {(96, 1): 281, (128, 1): 248, (256, 1): 269}),
    (1792, 16384, 2048, {(96, 1): 118, (128, 1): 115, (256, 1): 108}),
    (129, 128256, 4096, {(96, 1): 244, (128, 1): 264, (256, 1): 244, (256, 2): 303}),
    (192, 128256, 8192, {(96, 1): 493, (128, 1): 520, (256, 1): 520, (256, 2): 592}),
    (333, 4096, 14336, {(96, 4): 57, (128, 4): 60, (128, 5): 54, (96, 8): 64, (256, 7): 63, (96, 5): 80, (128, 6): 77}),
    (333, 4096, 4096, {(96, 4): 26, (128, 4): 26, (96, 3): 28, (128, 3): 29, (96, 5): 35, (256, 6): 32}),
    (1152, 4096, 14336, {(96, 4): 158, (128, 3): 147, (128, 5): 153, (256, 3): 136, (96, 1): 168, (256, 2): 170}),
    (2304, 4096, 14336, {(96, 1): 261, (96, 2): 260, (128, 3): 270, (256, 3): 273, (256, 1): 317}),
]


@pytest.mark.parametrize("rows,n_out,k,us", MEASURED, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_plan_picks_a_form_near_the_fastest_measured(rows, n_out, k, us):
    """Within 5%: two runs of one form differ by 2 to 3%."""
    p = product_plan(rows, n_out, k, 256 * max(28672, 2 * k, n_out if n_out <= 57344 else 0) * 8)
    assert p["whole_rows"] == 0
    assert us[p["tile_rows"], p["splits"]] <= 1.05 * min(us.values())


@pytest.mark.parametrize("rows", [1, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 256, 257, 320, 321, 384, 450, 640])
@pytest.mark.parametrize("n_out,k", LM_HEAD + [(28672, 4096), (4096, 14336), (6144, 4096), (4096, 4096), (16384, 2048), (2048, 8192),
                                               (10240, 8192), (8192, 28672), (24608, 1088), (4160, 4160), (3072, 2048), (2048, 2048), (1536, 1024), (96, 256)])
@pytest.mark.parametrize("ws", [0, 3 * 4096 * 100, WS])
def test_streamed_products_fit_their_form(rows, n_out, k, ws):
    """At most eight row tiles, parts of K that every slice of every workgroup gets at least a full ring of steps of, and room
    for the partial sums."""
    p = product_stream(rows, n_out, k, ws)
    if p["tile_rows"] == 0:
        return
    assert p["tile_rows"] in (64, 96, 128, 160, 192) and -(-rows // p["tile_rows"]) <= 8
    steps, parts, slices = k // 64, p["splits"], p["k_slices"]
    assert steps % slices == 0
    per = -(-(steps // slices) // parts)       # k steps of a slice, and what is left for the last part
    assert -(-(steps // slices) // per) == parts and steps // slices - (parts - 1) * per >= 4
    assert parts == 1 or parts * rows * ((n_out + 31) // 32 * 32) <= ws


def test_what_is_not_streamed():
    assert product_stream(641, 4096, 4096, WS)["tile_rows"] == 0          # more rows than it takes
    assert product_stream(100, 28672, 4096 + 32, WS)["tile_rows"] == 0    # contraction not a multiple of 64
    assert product_stream(100, 2048, 2048, WS)["tile_rows"] == 0          # 8 MiB of weights
    assert product_stream(16, 128256, 4096, WS)["tile_rows"] == 0         # the widest outputs at few rows
    for bad in ((0, 32, 64, 0), (1, 0, 64, 0), (1, 32, 0, 0), (1, 32, 63, 0), (1, 32, 64, -1)):
        with pytest.raises(PieError):
            product_stream(*bad)


# (rows, n_out, k, us on the streaming kernel's best form, us on the tiled kernels): weights from HBM, kernel plus epilogue;
# pairs whose difference is not what a split product's following kernel saves
STREAMED = [
    (200, 3072, 2048, 10.4, 15.9), (600, 3072, 2048, 16.5, 21.6), (324, 2048, 2048, 10.7, 14.9), (200, 2048, 2048, 10.7, 9.0),
    (600, 8192, 8192, 87.1, 96.4),
    (300, 28672, 4096, 78.2, 99.6), (450, 28672, 4096, 119.1, 104.9), (324, 16384, 2048, 33.6, 31.9), (520, 8192, 28672, 260.4, 286.7),
    (140, 8192, 1024, 11.0, 16.7), (520, 8192, 1024, 17.9, 17.4), (324, 1536, 1024, 7.5, 12.5), (384, 1024, 4096, 15.7, 13.3),
]


@pytest.mark.parametrize("rows,n_out,k,streamed,tiled", STREAMED)
def test_the_faster_kernel_takes_the_product(rows, n_out, k, streamed, tiled):
    p = product_stream(rows, n_out, k, 256 * max(28672, n_out) * 8)
    assert (p["tile_rows"] > 0) == (streamed < tiled)


def test_whole_products_that_end_in_the_residual_have_narrow_row_tiles():
    """Output and down projections (at most 8192 columns) are never streamed whole in row tiles of 160 or 192 by 256 columns, which
    are not built for them: over every hidden size, and as many contractions, 65 to 640 rows, with and without a workspace."""
    rng = np.random.default_rng(1)
    for hidden in range(32, 8193, 32):
        for rows in (65, 160, 192, 333, 512, 640, *rng.integers(65, 641, 6)):
            for k in (64 * int(rng.integers(4, 129)), 64 * int(rng.integers(4, 600))):
                for ws in (0, min(int(rows), 256) * max(hidden, 2 * k) * 8):
                    p = product_stream(int(rows), hidden, k, ws)
                    assert p["splits"] != 1 or p["k_slices"] > 1 or p["tile_rows"] < 160, (rows, hidden, k, ws, p)
