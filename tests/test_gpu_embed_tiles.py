"""GPU parity of the embedding lookup at the sizes where its tiles can go
wrong: table rows of 1 byte (1,024 cells a tile) to 36 KB (4 cells), rows that
end inside tiles, counts around a tile, and the row scan's units inside and
outside the launch."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth

pytestmark = pytest.mark.gpu


def _check(v, k, lens, row_bytes, layout, side=dt.PAD_RIGHT):
    import torch
    rng = np.random.default_rng(row_bytes + len(lens))
    offs = synth.offsets_from_lengths(np.array(lens, np.int64))
    data = np.frombuffer(b"ACGTN", np.uint8)[rng.integers(0, 5, int(offs[-1]))].copy()
    table = rng.integers(0, 256, (v.vocab_size, row_bytes), dtype=np.uint8)
    print("embed k=%d rows=%d row_bytes=%d layout=%d side=%d" % (k, len(lens), row_bytes, layout, side), flush=True)
    w_ids, w_off = oracle.encode(v.kind, data, offs, k=k, add_cls_sep=True)
    if layout == dt.PADDED:
        w_ids, _ = oracle.pad(w_ids, w_off, int(np.diff(w_off).max()), side)
    emb, oo, ids, _ = dt.embed(v, torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda(),
                               torch.from_numpy(table).cuda(), h_offsets=offs, add_cls_sep=True, layout=layout,
                               pad_side=side, want_ids=True)
    assert dt.sync_status() == 0
    assert np.array_equal(oo.cpu().numpy(), w_off)
    assert np.array_equal(ids.cpu().numpy().ravel(), w_ids.ravel())
    assert np.array_equal(emb.cpu().numpy().reshape(-1, row_bytes), table[w_ids.ravel()])
    flat = torch.from_numpy(w_ids.ravel().copy()).cuda()
    assert torch.equal(dt.embed_ids(flat, torch.from_numpy(table).cuda()).view(-1), emb.reshape(-1))
    assert dt.sync_status() == 0


@pytest.mark.parametrize("row_bytes", [1, 2, 7, 12, 32, 100, 256, 400, 1000, 4096, 8192, 8194, 12288, 36000])
@pytest.mark.parametrize("kind,k", [(dt.SINGLE, 1), (dt.KMER, 4)])
def test_tile_sizes(kind, k, row_bytes):
    v = dt.Vocab(kind, k=k)
    cells = min(1024, max(4, 32768 // row_bytes // 4 * 4))
    lens = [0, 1, cells * k, (cells - 2) * k, (cells - 3) * k, 0, 2 * cells * k + 1] + [5] * 30
    for layout, side in ((dt.PACKED, 0), (dt.PADDED, dt.PAD_RIGHT), (dt.PADDED, dt.PAD_LEFT)):
        _check(v, k, lens, row_bytes, layout, side)
    v.close()


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 65536, 65537])
def test_row_scan_units(n):
    v = dt.Vocab(dt.KMER, k=3)
    lens = np.random.default_rng(n).integers(0, 12, n)
    for layout in (dt.PACKED, dt.PADDED):
        _check(v, 3, lens, 32, layout)
    v.close()
