"""Decode of tiles in which more rows start than a workgroup has threads: empty
rows at the front, in the middle and at the end, rows of one id, all empty."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,k", [(dt.SINGLE, 1), (dt.KMER, 5), (dt.BPE, 1)])
@pytest.mark.parametrize("shape", ["empty", "front", "middle", "end", "ones", "mixed"])
def test_many_rows_in_a_tile(kind, k, shape):
    import torch
    rng = np.random.default_rng(len(shape) + k)
    none, some = np.zeros(1300, np.int64), rng.integers(1, 40, 90)
    lens = {"empty": none, "front": np.r_[none, some], "middle": np.r_[some, none, some], "end": np.r_[some, none],
            "ones": np.ones(2700, np.int64), "mixed": rng.integers(0, 2, 5000)}[shape]
    merges = np.array([(5, 6), (7, 8), (10, 11), (12, 12)], np.int32)
    v = dt.Vocab(kind, merges=merges) if kind == dt.BPE else dt.Vocab(kind, k=k)
    offs = synth.offsets_from_lengths(lens)
    ids = rng.integers(0, min(v.vocab_size, 3000) + 3, size=int(offs[-1])).astype(np.int32)
    print(kind, shape, len(ids), flush=True)
    want, want_off = oracle.decode(kind, ids, offs, k=k, merges=merges if kind == dt.BPE else None)
    out, out_off = dt.decode(v, torch.from_numpy(ids).cuda(), torch.from_numpy(offs).cuda())
    assert dt.sync_status() == 0
    assert np.array_equal(out_off.cpu().numpy(), want_off)
    assert np.array_equal(out.cpu().numpy()[:len(want)], want)
    v.close()
