"""QKV projections of window rows that rotate q and k and write the key-contiguous values in their epilogue (65-128 rows on 128 x 64
tiles, fewer on 64 x 64, above 384 rows the tiles of whole canvases; windows of whole 16-key groups) and the rotary pass beside them
(windows that are not; 129-384 rows, which split K): rounds against the oracle with several canvases in a tile, tiles that end
inside a canvas, canvases of whole and of ragged key tiles, windows cut by the canvas end."""
import pytest

from tests import test_gpu_window_shapes as shapes
from tests.test_gpu_window_shapes import models  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G,K,bl,pl,gl,k", [(2048, 1, 0, 32, 64, 64, 1), (2048, 3, 0, 16, 32, 96, 3), (2048, 1, 4, 16, 48, 80, 4),
                                              (3072, 1, 0, 64, 64, 128, 0), (3072, 1, 2, 16, 48, 96, 2),
                                              (2048, 1, 3, 64, 77, 192, 1), (2048, 1, 3, 64, 64, 192, 1), (2048, 1, 3, 64, 53, 192, 2),
                                              (2048, 1, 4, 40, 61, 160, 2), (512, 2, 4, 36, 45, 144, 1), (512, 1, 8, 48, 96, 144, 2)])
def test_round(models, d, G, K, bl, pl, gl, k):  # noqa: F811
    shapes.test_cached_round_with_drafts(models, d, G, K, bl, pl, gl, k)


# every tile shape of whole canvases above 384 rows (the tests above and beside this one take 128 x 128): waves of 64, 96 and 128
# rows, windows that begin inside a pass of 32 rows and inside a group of 64 keys, tiles that end inside a canvas
@pytest.mark.parametrize("d,G,K,bl,pl,gl,k", [(3072, 2, 3, 80, 48, 80, 0),           # 128 x 256, 640 rows
                                              (3072, 1, 6, 48, 64, 144, 2),          # 256 x 128, 672 rows, windows cut by the end
                                              (3072, 2, 4, 48, 32, 144, 1),          # 192 x 256, 960 rows
                                              (3072, 3, 2, 80, 64, 240, 1)])         # 256 x 256, 1440 rows
def test_round_on_large_tiles(models, d, G, K, bl, pl, gl, k):  # noqa: F811
    shapes.test_cached_round_with_drafts(models, d, G, K, bl, pl, gl, k)
