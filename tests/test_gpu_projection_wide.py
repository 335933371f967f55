"""Mixed rows over large streamed weights: up to 64 rows in 64 x 256 tiles, though their weights are one round of 128 x 256 tiles (or one column tile
less), and up to 256 rows in 256 x 128 tiles.  Bounds are those of test_gpu_projection_tiles."""
import pytest

import test_gpu_projection_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,vocab,hidden,tile", [(1, 65536, 3072, 2), (33, 65536, 3072, 2), (64, 65472, 3072, 2), (64, 63744, 3072, 2), (60, 57344, 3072, 2),
                                                 (130, 65536, 4096, 4), (256, 65536, 4096, 4), (255, 61440, 3072, 4)])
def test_tiles_of_mixed_rows(n, vocab, hidden, tile):
    tiles._check(n, vocab, hidden, "mixed", True, tiles=(tile, tile))
