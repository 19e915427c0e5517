"""Row scans on both sides of the rows at which a launch of its own changes from
independent to chained units, one call after another on one stream and under
capture: the chained form's state must be clear for each next launch."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
from test_gpu_rows import _check, _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12287, 12288, 12289, 16385, 40000])
def test_around_the_rule(n):
    rng = np.random.default_rng(n)
    data, offs = _rows(n, rng.integers(0, 9, n))
    for layout in (dt.PACKED, dt.PADDED):
        _check([(dt.SINGLE, 1)], data, offs, True, layout)
        _check([(dt.KMER, 2), (dt.KMER, 5)], data, offs, False, layout)
        _check([(dt.KMER, 3)], data, offs, True, layout, variant=dt.VARIANT_OVERLAP)


def test_replays():
    import torch
    data, offs = _rows(3, np.random.default_rng(3).integers(0, 9, 20000))
    v = dt.Vocab(dt.KMER, k=3)
    w_ids, w_off = oracle.encode(oracle.KMER, data, offs, k=3)
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda()
    ids = torch.empty(len(w_ids), dtype=torch.int32, device="cuda")
    oo = torch.empty(len(offs), dtype=torch.int64, device="cuda")

    def call():
        dt.dnatok_encode(v.handle, d.data_ptr(), d.numel(), o.data_ptr(), len(offs) - 1, ids.data_ptr(), ids.numel(),
                         oo.data_ptr(), None, dt.make_opts(False), torch.cuda.current_stream().cuda_stream)

    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call()
    for rep in range(5):
        ids.fill_(-7)
        oo.fill_(-7)
        torch.cuda.synchronize()
        if rep == 3:
            with torch.cuda.stream(s):
                call()  # an eager call between replays
            torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), w_ids) and np.array_equal(oo.cpu().numpy(), w_off)
    v.close()
