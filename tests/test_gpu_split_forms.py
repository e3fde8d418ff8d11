"""The forms of weights the float32 split path packs itself: attention vectors
folded into tiles with few or many folded columns."""
import numpy as np
import pytest

from test_gpu_split_gemm import test_attention_vectors_folded_into_the_weights as check_folded

pytestmark = pytest.mark.gpu


# folded columns of a tile: 2 (one head), 4 + 2, 4, 10, 12, 4 + 10, 6
@pytest.mark.parametrize("Fi,heads,D,mean", [(5, 1, 64, False), (130, 1, 16, True), (7, 3, 4, False), (40, 2, 32, False),
                                             (9, 5, 4, False), (129, 6, 8, False), (33, 7, 4, False), (20, 3, 8, False)])
def test_folded_columns_of_a_tile(Fi, heads, D, mean):
    check_folded(Fi, heads, D, mean)
