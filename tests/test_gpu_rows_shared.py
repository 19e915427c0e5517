"""Encode variants of small batches, whose tiles are shared by the four waves of
a workgroup, on both sides of the rule that chooses them: up to 512 tiles of
1 KiB, and no more 64-row steps than tiles. Rows from a few to thousands of
16-byte groups, so runs are written together and one by one."""
import numpy as np
import pytest

import paper_2601_05531_amd as dt
from test_gpu_rows import _check, _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,k,variant", [(dt.SINGLE, 1, 1), (dt.KMER, 2, 1), (dt.KMER, 6, 2), (dt.KMER, 9, 3)])
@pytest.mark.parametrize("shape", ["one", "reads", "many_groups", "at_the_limit", "past_it", "rows_limit", "rows_past"])
def test_shared_tiles(kind, k, variant, shape):
    rng = np.random.default_rng(k + len(shape))
    lens = {"one": [1023], "reads": rng.integers(50, 100, 300), "many_groups": rng.integers(250, 400, 90),
            "at_the_limit": [130000] * 4, "past_it": [131073] * 4, "rows_limit": [6] * 1000 + [1024] * 12,
            "rows_past": [2] * 3000}[shape]
    data, offs = _rows(len(shape), lens)
    _check([(kind, k)], data, offs, True, dt.PACKED, variant=variant, shift=1)
    for side in (dt.PAD_RIGHT, dt.PAD_LEFT):
        _check([(kind, k)], data, offs, side == dt.PAD_LEFT, dt.PADDED, side, variant, 3, 5 * side)
