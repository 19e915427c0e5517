"""A stream's first decode under graph capture: accepted where an earlier call
gave the stream a scratch, as a BPE encode does, whatever the decode's size."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,k,n_ids", [(dt.SINGLE, 1, 2000000), (dt.KMER, 6, 700000), (dt.KMER, 13, 300000)])
def test_first_decode_is_captured(kind, k, n_ids):
    import torch
    merges = np.array([(5, 6), (7, 8), (10, 11)], np.int32)
    bpe, v = dt.Vocab(dt.BPE, merges=merges), dt.Vocab(kind, k=k)
    rng = np.random.default_rng(k)
    print("first decode under capture", kind, k, n_ids, flush=True)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        text = torch.from_numpy(np.frombuffer(b"ACGTACGG", np.uint8).copy()).cuda()
        dt.encode(bpe, text, torch.tensor([0, 8], dtype=torch.int64).cuda(), h_offsets=np.array([0, 8]), stream=s)
    torch.cuda.synchronize()
    offs = synth.offsets_from_lengths([n_ids // 2, n_ids - n_ids // 2])
    ids = torch.from_numpy(rng.integers(0, 60, n_ids).astype(np.int32)).cuda()
    o = torch.from_numpy(offs).cuda()
    out = torch.zeros(n_ids * k, dtype=torch.uint8, device="cuda")
    oo = torch.zeros(3, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        dt.dnatok_decode(v.handle, ids.data_ptr(), n_ids, o.data_ptr(), 2, out.data_ptr(), out.numel(), oo.data_ptr(),
                         torch.cuda.current_stream().cuda_stream)
    for rep in range(4):
        new = rng.integers(0, 60, n_ids).astype(np.int32)
        ids.copy_(torch.from_numpy(new))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        want, want_off = oracle.decode(kind, new, offs, k=k)
        assert np.array_equal(oo.cpu().numpy(), want_off) and np.array_equal(out.cpu().numpy()[:len(want)], want)
    bpe.close()
    v.close()
