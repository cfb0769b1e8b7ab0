"""GPU parity at the sizes where a kernel's own partition of the work ends: remainders of its steps, the shortest and
the longest lists, tile shapes off the beaten track.  Against the oracle, with the tolerances of the parity tests."""
import numpy as np
import pytest

from paper_2407_08330_amd import inputs
from test_gpu_bwd import run_bwd_case
from test_gpu_fwd import run_fwd_case
from gpu_common import say

pytestmark = pytest.mark.gpu


def _padded(docs, n):
    level = np.stack([np.concatenate([l, np.full(n - l.shape[0], -1, np.int32)]) for l, _ in docs])
    parent = np.stack([np.concatenate([p, np.full(n - p.shape[0], -1, np.int32)]) for _, p in docs])
    return level, parent


@pytest.mark.parametrize("tile,D,windowed", [((96, 96), 64, False), ((32, 32), 128, False), ((128, 128), 64, True),
                                             ((64, 96), 128, True)])
def test_fp32_rows_lists_and_tile_shapes(oracle, tile, D, windowed):
    # the fp32 kernels take a wave per row, four rows per workgroup, 256 key slots per round and 16 keys per step: an odd
    # number of rows, groups of 1, 15, 16, 17, 255-257 siblings, and one of 700 that needs several rounds
    docs = [inputs.document_from_sections([[1, 14, 15], [16, 17], [254, 255, 256]], 850),
            inputs.document_from_sections([[700, 3], [1]], 721)]
    level, parent = _padded(docs, 851)
    say(f"[fp32 edges] tile {tile} d={D} windowed={windowed}")
    run_fwd_case(oracle, level, parent, 3, D, "f32", 31, tile=tile, windowed=windowed)
    run_bwd_case(oracle, level, parent, 3, D, "f32", 32, tile=tile, windowed=windowed)
    run_bwd_case(oracle, level, parent, 1, D, "f32", 33, tile=tile, windowed=windowed, edges=6)
