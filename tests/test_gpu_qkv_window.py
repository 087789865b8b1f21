"""QKV projections of window rows that rotate q and k and write the key-contiguous values in their epilogue (65-128 rows on 128 x 64
tiles, fewer on 64 x 64, above 384 rows the tiles of whole canvases; windows of whole 16-key groups) and launches of those rows whose
windows are not: rounds against the oracle with several canvases in a tile, tiles that end inside a canvas, canvases of whole and
of ragged key tiles, windows cut by the canvas end."""
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
