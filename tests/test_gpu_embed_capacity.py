"""PACKED embedding lookups into buffers of more rows than there are tokens, and
over more rows than one look around a tile's place finds: rows of equal and of
very unequal length, empty rows, tiles with more rows than a wave has lanes."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth

pytestmark = pytest.mark.gpu


def _lengths(kind, n, rng):
    if kind == "equal":
        return np.full(n, 7)
    if kind == "sparse":  # mostly empty rows
        return np.where(rng.random(n) < 0.02, rng.integers(1, 90, n), 0)
    lens = rng.integers(0, 4, n)  # short rows at one end, long ones at the other
    lens[-n // 50:] = rng.integers(200, 400, n // 50 + 1)[-len(lens[-n // 50:]):]
    return lens


@pytest.mark.parametrize("kind", ["equal", "sparse", "skewed"])
@pytest.mark.parametrize("n,dim", [(1, 128), (4096, 128), (4097, 128), (30000, 64), (30000, 8), (70001, 3)])
def test_rows_and_capacity(kind, n, dim):
    import torch
    rng = np.random.default_rng(n + dim)
    lens = _lengths(kind, n, rng)
    offs = synth.offsets_from_lengths(lens)
    data = rng.choice(np.frombuffer(b"ACGTNacgt", np.uint8), size=max(1, int(offs[-1])))
    for vocab, k, cls in ((dt.SINGLE, 1, False), (dt.KMER, 3, True), (dt.KMER, 3, False)):
        print(kind, n, dim, k, cls, flush=True)
        v = dt.Vocab(vocab, k=k)
        table = torch.randint(-30000, 30000, (v.vocab_size, dim), dtype=torch.int16)
        want_ids, want_off = oracle.encode(vocab, data, offs, k=k, add_cls_sep=cls)
        want = oracle.embed(table.numpy(), want_ids)
        for times in (1, 5):
            out = torch.full((times * len(want_ids) + 3, dim), 77, dtype=torch.int16, device="cuda")
            emb, out_off, ids, _ = dt.embed(v, torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda(), table.cuda(),
                                            h_offsets=offs, add_cls_sep=cls, want_ids=True, out=out)
            assert dt.sync_status() == 0
            assert np.array_equal(out_off.cpu().numpy(), want_off)
            assert np.array_equal(ids.cpu().numpy(), want_ids) and np.array_equal(emb.cpu().numpy(), want)
            assert (out[len(want_ids):] == 77).all()
        v.close()
