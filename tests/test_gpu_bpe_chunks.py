"""GPU parity of the chunked BPE encode at the sizes where it can go wrong:
rows around its 64-base chunks, its 127-base reach and the 62 chunks a wave
owns, many rows in one wave, rows of no bases, barriers at chunk edges, and
tandem repeats in which neighbouring chunks do not meet (the walk)."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth
from test_bpe_chunk_rule import ACGT, short_token_table
from test_gpu_bpe import _packed, _padded

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 94, 96, 126, 127, 128, 129, 190, 191, 192, 193, 61 * 64, 62 * 64 - 1, 62 * 64,
         62 * 64 + 1, 63 * 64 + 1, 64 * 64, 124 * 64 + 5]


def _rows(kind, lens, rng):
    rows = []
    for L in lens:
        if kind == "random":
            row = ACGT[rng.integers(0, 4, size=L)]
        elif kind == "repeat":
            row = np.tile(ACGT[rng.integers(0, 4, size=int(rng.integers(1, 6)))], L + 1)[:L]
        else:  # repeats of 1 to 400 bases, one after another
            parts = [ACGT[:0]]
            while sum(map(len, parts)) < L:
                motif = ACGT[rng.integers(0, 4, size=int(rng.integers(1, 6)))]
                parts.append(np.tile(motif, 400)[:int(rng.integers(1, 400))])
            row = np.concatenate(parts)[:L]
        rows.append(row.copy())
    return rows


@pytest.mark.parametrize("kind", ["random", "repeat", "mixed"])
@pytest.mark.parametrize("R,p_chain,longest", [(0, 0.0, 1), (5, 0.6, 8), (60, 0.3, 64), (700, 0.05, 24)])
def test_chunk_edges(kind, R, p_chain, longest):
    rng = np.random.default_rng(R + len(kind))
    merges = short_token_table(7 + R, R, p_chain, longest)
    v = dt.Vocab(dt.BPE, merges=merges)
    lens = list(EDGES) + list(rng.integers(0, 200, 150)) + [20000]
    rng.shuffle(lens)
    rows = _rows(kind, lens, rng)
    for row in rows[::3]:  # barriers: single ones, runs, soft-masked bases
        if len(row):
            at = rng.integers(0, len(row), size=1 + len(row) // 300)
            row[at] = rng.choice(np.frombuffer(b"Nnxacgt", np.uint8), size=len(at))
    data, offs = np.concatenate(rows), synth.offsets_from_lengths(lens)
    _packed(v, merges, data, offs, cls=True)
    _padded(v, merges, data, offs, cls=bool(R), side=R % 2)
    v.close()


def test_misaligned_bytes_capacity_and_width():
    import torch
    merges = short_token_table(3, 200, 0.1, 16)
    v = dt.Vocab(dt.BPE, merges=merges)
    rng = np.random.default_rng(8)
    lens = [700, 0, 33, 5000, 64]
    data, offs = np.concatenate(_rows("mixed", lens, rng)), synth.offsets_from_lengths(lens)
    want, want_off = oracle.encode(oracle.BPE, data, offs, merges=merges, add_cls_sep=True)
    d_offs = torch.from_numpy(offs).cuda()
    for shift in (1, 2, 3):
        buf = torch.full((len(data) + 8,), ord("A"), dtype=torch.uint8, device="cuda")
        buf[shift:shift + len(data)] = torch.from_numpy(data).cuda()
        ids, out_off, _ = dt.encode(v, buf[shift:shift + len(data)], d_offs, h_offsets=offs, add_cls_sep=True)
        assert dt.sync_status() == 0
        assert np.array_equal(ids.cpu().numpy(), want) and np.array_equal(out_off.cpu().numpy(), want_off)
    # a short buffer: the flag, true offsets, nothing past the capacity
    d = torch.from_numpy(data).cuda()
    out = torch.full((len(want) + 64,), -7, dtype=torch.int32, device="cuda")
    oo = torch.empty(len(offs), dtype=torch.int64, device="cuda")
    cap = len(want) - 10
    stream = torch.cuda.current_stream().cuda_stream
    dt.dnatok_encode(v.handle, d.data_ptr(), len(data), d_offs.data_ptr(), len(lens), out.data_ptr(), cap,
                     oo.data_ptr(), None, dt.make_opts(True), stream)
    assert dt.sync_status() == dt.DERR_CAPACITY
    got = out.cpu().numpy()
    assert np.array_equal(got[:cap], want[:cap]) and (got[cap:] == -7).all()
    assert np.array_equal(oo.cpu().numpy(), want_off)
    # a row wider than pad_to: the flag, that row left alone
    W = int(np.diff(want_off)[0]) + 1
    ids = torch.full((len(lens), W), -7, dtype=torch.int32, device="cuda")
    mask = torch.full((len(lens), W), 9, dtype=torch.int8, device="cuda")
    dt.dnatok_encode(v.handle, d.data_ptr(), len(data), d_offs.data_ptr(), len(lens), ids.data_ptr(), ids.numel(),
                     oo.data_ptr(), mask.data_ptr(), dt.make_opts(True, dt.PADDED, dt.PAD_LEFT, W), stream)
    assert dt.sync_status() == dt.DERR_ROW_WIDTH
    got = ids.cpu().numpy()
    assert (got[3] == -7).all() and np.array_equal(got[0][1:], want[:W - 1]) and got[0][0] == 0
    v.close()
