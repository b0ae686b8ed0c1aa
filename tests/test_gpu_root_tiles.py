"""Root products of both sides in one launch: k of one segment is below the lengths at which the tile changes, that of all six segments
above.  Numbers of matrices on either side of one block per CU (128 x 128 tiles in eight stages) and of half a round (256 x 128 tiles).
Against the same rounds in 64 bits, and a matrix among others has the bits that it has alone (64 x 64 tiles)."""
import pytest

from tests.test_gpu_shampoo_terms import _check, _step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,cols,bf16", [
    (21, 250, 256, True), (22, 256, 200, False),      # 252 and 264 blocks of 128 x 128, k 6 x 256
    (7, 512, 500, True), (21, 500, 512, False), (22, 512, 512, True),   # 140 blocks; 126 and 132 tiles of 256 x 256
    (4, 1024, 1000, True),                            # 80 tiles, k 6 x 1024
    (3, 1537, 1025, False),                           # 129 tiles, two lengths of k
    (2, 1537, 1025, True),                            # 86 tiles
])
def test_among_others_as_alone(canz, n, rows, cols, bf16):
    import torch
    dtype, eps = torch.bfloat16 if bf16 else torch.float32, 1e-3
    step = _step(torch, canz, rows, cols, n, 22, dtype, eps)
    _check(torch, rows, cols, n, 22, eps, *step)
    alone = _step(torch, canz, rows, cols, 1, 22, dtype, eps)
    for together, one in zip(step, alone):
        assert torch.equal(together[0], one[0])
