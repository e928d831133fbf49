"""Products of odd K of few rows (CPU): 16 x 16 blocks, or tiles of 64 x 64 where K is long and the blocks would be more than one per compute
unit; on shapes measured both ways."""
import pytest

import paper_2006_03031_amd as nb


@pytest.mark.parametrize("M,N,K,tile", [
    # tiles would take 5 to 32 % longer
    (52, 1397, 261, 16), (712, 131, 267, 16), (28, 2593, 335, 16), (226, 413, 499, 16), (50, 1079, 523, 16), (68, 961, 553, 16),
    # blocks would take 3 to 100 % longer
    (760, 112, 583, 64), (82, 1265, 635, 64), (114, 1024, 979, 64), (191, 381, 1663, 64),
    # either side of the line
    (80, 1001, 575, 16), (80, 1001, 577, 64),
    # one block per compute unit; K even; more than two per compute unit
    (64, 1001, 1003, 16), (128, 1001, 1002, 16), (129, 1001, 261, 64), (16, 9001, 1003, 16)])
def test_blocks_and_tiles(M, N, K, tile):
    for out in (nb.BF16, nb.F32):
        p = nb.dense_plan(M, N, K, out_dtype=out)
        assert p.name == "generic" and p.bm == p.bn == tile, p
