"""BPE with offsets that go back, so that rows overlap and hold more 64-base
chunks together than the input has room for: the flag, nothing written past the
capacity, and the next call on the stream right."""
import numpy as np
import pytest

import paper_2601_05531_amd as dt
from test_bpe_wave_model import load, tandem
from test_gpu_bpe import _packed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("motif", [b"TAT", b"ACGTTGCATC"])
@pytest.mark.parametrize("rows", [3, 9, 64])
def test_overlapping_rows(motif, rows):
    import torch
    merges = load()
    v = dt.Vocab(dt.BPE, merges=merges)
    data = tandem(motif, 20000)
    offs = np.array([0, 20000] * ((rows + 1) // 2) + [0] * ((rows + 1) % 2), np.int64)
    print("overlapping", motif, rows, flush=True)
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda()
    ids = torch.full((30064,), -7, dtype=torch.int32, device="cuda")
    out = torch.empty(len(offs), dtype=torch.int64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    dt.dnatok_encode(v.handle, d.data_ptr(), len(data), o.data_ptr(), len(offs) - 1, ids.data_ptr(), 30000,
                     out.data_ptr(), None, dt.make_opts(False), stream)
    assert dt.sync_status() & dt.DERR_OFFSETS
    assert (ids[30000:] == -7).all()
    _packed(v, merges, data, np.array([0, 4100, 4100, 20000], np.int64), cls=True)
    v.close()
