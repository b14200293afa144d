"""GMRES of one system on both sides of the row limits of the small-system
kernels: from restart 16 on 160 blocks of 64 rows (32x20x16 nodes are 10,240
rows, 32x20x17 10,880), below 96 (32x16x12 are 6,144, 33x16x12 6,336 in 6,400)."""
import pytest

import test_gpu_tensor as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,restart", [((31, 19, 15), 16), ((31, 19, 15), 56), ((31, 19, 16), 16), ((31, 19, 16), 56),
                                          ((31, 15, 11), 15), ((32, 15, 11), 15)])
def test_gmres_at_the_row_limit(monkeypatch, size, restart):
    import paper_2112_00087_amd as P
    T.test_gmres_of_small_boxes(P, monkeypatch, size, restart)
