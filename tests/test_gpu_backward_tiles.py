"""bfloat16 dK, dV where the 16-key tiles and 32-row chunks of the kernel end: blocks of 1 to 32 pooled keys packed to a workgroup
(up to 32 blocks, 32 or 64 keys), chunks of fewer than 32 rows, query blocks of a number of chunks that is no power of two.

Against the oracle with the bar of the other edge tests."""
import pytest

from tests import test_gpu_backward_edges as edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,N,d,bq,bk,levels,causal,keep", [
    (1, 1, 203, 128, 24, 8, 3, False, 0.5),       # pooled blocks of 8, 4 and 2 keys: 32 blocks a workgroup
    (2, 1, 700, 64, 64, 16, 5, True, 0.5),        # ... of 16 down to 1 key
    (1, 1, 1300, 64, 8, 8, 2, False, 0.05),       # chunks of 8 rows, columns of 163 query blocks
    (48, 48, 520, 128, 128, 64, 4, False, 0.5),   # 64 keys a workgroup
    (48, 6, 461, 64, 96, 32, 4, True, 0.7),       # ... three chunks a query block, grouped heads
    (1, 1, 9000, 64, 8, 32, 3, False, 0.03),      # packed blocks over two lists of query blocks
    (24, 24, 2100, 128, 32, 32, 3, False, 0.2),   # workgroups started by length
    (28, 4, 4200, 64, 32, 64, 4, True, 0.2),
    (192, 192, 264, 128, 32, 16, 3, False, 0.4),  # workgroups of two wavefronts: packed blocks only, a ragged last query block
    (140, 14, 461, 64, 96, 32, 4, True, 0.7),     # ... three chunks a query block, grouped heads
    (128, 128, 900, 128, 24, 64, 4, False, 0.2),  # ... chunks of 24 rows
    (96, 12, 524, 128, 128, 128, 2, True, 0.6),    # ... 128-key blocks in two parts
    (3, 1, 22000, 128, 128, 128, 4, False, 0.04),  # 128-key blocks in two parts
])
def test_backward_tile_edges(Hq, Hkv, N, d, bq, bk, levels, causal, keep):
    edges.test_backward_edges(Hq, Hkv, N, d, bq, bk, levels, causal, keep, False)
