"""Batch-norm passes that take the rows by eighths, one per XCD: at the lines of that route (4.1 MB; 26 MB backward, above which a launch of its
own finishes the sums), with row counts that neither eight nor a block divides."""
import pytest

import test_gpu_bn_chunks as chunks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,N,H,W,C", [
    ("bf16", 33, 31, 33, 64), ("bf16", 34, 31, 33, 64),           # 4.1 and 4.25 MiB
    ("f32", 257, 32, 32, 4), ("f32", 9, 11, 11, 1024),            # one vector a row; eight blocks a chunk
    ("bf16", 23, 7, 7, 2048),                                     # sixteen chunks
    ("bf16", 27, 57, 67, 128), ("bf16", 27, 58, 69, 128),         # 25.2 and 26.4 MiB
])
def test_lines_of_the_route(dtype, N, H, W, C):
    chunks.test_both_directions(N, H, W, C, dtype)
