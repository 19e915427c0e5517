"""GPU parity of the decode (single letters, k-mers, BPE) where its tiles
can go wrong: every number of slices per wave, slices with and without
silent ids, groups of 64 and supers of 4,096 tiles, ids outside the rows,
misaligned ids and outputs, many rows in one tile, launches of different sizes
one after another, the words of very long decodes, and captured launches."""
import numpy as np
import pytest

import oracle
import paper_2601_05531_amd as dt
import synth

pytestmark = pytest.mark.gpu


def _ids(rng, kind, k, n):
    vs = 10 if kind == dt.SINGLE else 5 + 4 ** k
    ids = rng.integers(5, vs, n).astype(np.int32)
    for _ in range(max(1, n // 5000)):  # silent and unknown ids in patches, whole slices without
        if n:
            at = int(rng.integers(0, n))
            m = len(ids[at:at + 40])
            ids[at:at + m] = rng.integers(-2, 8, m)
    return ids


def _check(v, k, ids, offs, shift=0, slack=16):
    import torch
    print("decode kind=%d k=%d ids=%d rows=%d shift=%d" % (v.kind, k, len(ids), len(offs) - 1, shift), flush=True)
    want, want_off = oracle.decode(v.kind, ids, offs, k=k)
    d = torch.zeros(len(ids) + shift + 4, dtype=torch.int32, device="cuda")
    d[shift:shift + len(ids)] = torch.from_numpy(ids).cuda()
    cap = int(want_off[-1])
    out = torch.full((cap + shift + slack,), 7, dtype=torch.uint8, device="cuda")
    oo = torch.full((len(offs) + 1,), -7, dtype=torch.int64, device="cuda")
    dt.dnatok_decode(v.handle, d.data_ptr() + 4 * shift, len(ids), torch.from_numpy(offs).cuda().data_ptr(),
                     len(offs) - 1, out.data_ptr() + shift, cap, oo.data_ptr(), None)
    assert dt.sync_status() == 0
    got = out.cpu().numpy()
    assert np.array_equal(oo.cpu().numpy(), np.append(want_off, -7))
    assert np.array_equal(got[shift:shift + cap], want)
    assert np.all(got[:shift] == 7) and np.all(got[shift + cap:] == 7)


@pytest.mark.parametrize("kind,k", [(dt.SINGLE, 1)] + [(dt.KMER, k) for k in (1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 13, 15)])
def test_every_tile_size(kind, k):
    rng = np.random.default_rng(k)
    v = dt.Vocab(kind, k=k)
    for n_ids in (1, 255, 256, 1023, 1024, 1025, 65 * 1024 + 3, 1_400_000, 3_000_000, 6_000_000, 12_000_000):
        if n_ids * k > 30_000_000:
            continue
        ids = _ids(rng, kind, k, n_ids)
        offs = np.unique(np.concatenate([[0], rng.integers(0, n_ids + 1, 1 + n_ids // 3000), [n_ids]])).astype(np.int64)
        if n_ids % 2 and len(offs) > 2:  # ids before the first and after the last row
            offs = offs + 0
            offs[0], offs[-1] = min(3, offs[1]), max(n_ids - 5, offs[-2])
        _check(v, k, ids, offs, shift=n_ids % 4)
    v.close()


def test_many_rows_in_a_tile_and_launch_sizes():
    rng = np.random.default_rng(5)
    v = dt.Vocab(dt.KMER, k=3)
    for lens in ([0] * 70_000 + [5], [5] + [0] * 3000 + [2000], list(rng.integers(0, 3, 40_000)), [0], [1] * 300,
                 [9_000_000], [4000], [0] * 5000 + [9_000_000] + [0] * 5000, []):
        offs = synth.offsets_from_lengths(np.array(lens, np.int64))
        _check(v, 3, _ids(rng, dt.KMER, 3, int(offs[-1])), offs)
    v.close()


def test_more_tiles_than_the_workspace_holds():
    import torch
    k, block = 15, 1000
    rng = np.random.default_rng(6)
    v = dt.Vocab(dt.KMER, k=k)
    ids = _ids(rng, dt.KMER, k, block)
    want, want_off = oracle.decode(dt.KMER, ids, np.array([0, block], np.int64), k=k)
    reps = 2048 * 16384 // block + 9
    d = torch.from_numpy(ids).cuda().repeat(reps)
    offs = torch.arange(reps + 1, dtype=torch.int64, device="cuda") * block
    print("decode of %d ids in %d rows" % (d.numel(), reps), flush=True)
    for _ in range(2):
        out, oo = dt.decode(v, d, offs, out_capacity=reps * len(want))
        assert dt.sync_status() == 0
        assert bool((out.view(reps, -1) == torch.from_numpy(want).cuda()).all())
        assert bool((oo == torch.arange(reps + 1, dtype=torch.int64, device="cuda") * len(want)).all())
        _check(v, k, ids, np.array([0, 10, block], np.int64))
    v.close()


def test_bad_offsets_are_flagged_wherever_they_are():
    import torch
    v = dt.Vocab(dt.SINGLE)
    ids = torch.full((5000,), 5, dtype=torch.int32, device="cuda")
    for n in (3, 200, 9000):  # rows looked at by a tile, by several, by workgroups after the tiles
        good = np.linspace(0, 5000, n + 1).astype(np.int64)
        for at in sorted({1, n // 2, n - 1}):
            bad = good.copy()
            bad[at] = 5001
            dt.decode(v, ids, torch.from_numpy(bad).cuda())
            assert dt.sync_status() & dt.DERR_OFFSETS, (n, at)
        dt.decode(v, ids, torch.from_numpy(good).cuda())
        assert dt.sync_status() == 0
    v.close()


def test_capture_and_replay():
    import torch
    rng = np.random.default_rng(9)
    v = dt.Vocab(dt.KMER, k=4)
    n_ids = 300_000
    offs = synth.offsets_from_lengths(np.full(100, n_ids // 100, np.int64))
    ids = _ids(rng, dt.KMER, 4, n_ids)
    d, d_offs = torch.from_numpy(ids).cuda(), torch.from_numpy(offs).cuda()
    out = torch.zeros(4 * n_ids, dtype=torch.uint8, device="cuda")
    oo = torch.zeros(len(offs), dtype=torch.int64, device="cuda")

    def call(x, xo):
        dt.dnatok_decode(v.handle, x.data_ptr(), x.numel(), xo.data_ptr(), xo.numel() - 1, out.data_ptr(), out.numel(),
                         oo.data_ptr(), torch.cuda.current_stream().cuda_stream)

    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call(d, d_offs)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call(d, d_offs)
        for rep in range(5):  # eager decodes of other sizes between the replays, on the same stream
            ids = _ids(rng, dt.KMER, 4, n_ids)
            d.copy_(torch.from_numpy(ids))
            call(d[:(1000, 280_000, 7)[rep % 3]], d_offs[:1])
            g.replay()
            torch.cuda.synchronize()
            want, want_off = oracle.decode(dt.KMER, ids, offs, k=4)
            assert np.array_equal(oo.cpu().numpy(), want_off)
            assert np.array_equal(out.cpu().numpy()[:len(want)], want)
    assert dt.sync_status(s) == 0
    v.close()


@pytest.mark.parametrize("longest", [2, 15, 16, 17, 48, 4096])
def test_bpe_tokens_of_every_length(longest):
    """Tokens around the 16 bases read at once; 4,096 bases: tiles whose
    output exceeds the stage; both tile sizes, edges of a thread's ids."""
    import torch
    merges, at = [(5, 6)], {2: 10}  # AC, then each token one base longer, or twice as long
    n = 2
    while n < longest:
        step = n if longest > 64 else 1
        merges.append((at[n], at[n] if step == n and longest > 64 else 5 + n % 4))
        n += step
        at[n] = 10 + len(merges) - 1
    merges = np.array(merges, np.int32)
    v = dt.Vocab(dt.BPE, merges=merges)
    rng = np.random.default_rng(longest)
    for n_ids in (0, 1, 15, 16, 1023, 1024, 1025, 4097, 60_000) + ((2_100_000,) if longest < 48 else ()):
        ids = rng.integers(5, 10 + len(merges), n_ids).astype(np.int32)
        odd = rng.random(n_ids) < 0.02
        ids[odd] = rng.integers(-2, 14 + len(merges), int(odd.sum()))
        offs = np.sort(np.concatenate([[0], rng.integers(0, n_ids + 1, 1 + n_ids // 700), [n_ids]])).astype(np.int64)
        if n_ids % 2:
            offs[0], offs[-1] = min(2, offs[1]), max(n_ids - 3, offs[-2])
        print("bpe decode longest=%d ids=%d rows=%d" % (longest, n_ids, len(offs) - 1), flush=True)
        want, want_off = oracle.decode(oracle.BPE, ids, offs, merges=merges)
        cap = int(want_off[-1])
        for short in (0, 5):
            room = max(cap - short, 0)
            out = torch.full((cap + 32,), 7, dtype=torch.uint8, device="cuda")
            oo = torch.empty(len(offs), dtype=torch.int64, device="cuda")
            d = torch.from_numpy(np.append(ids, np.int32(0))).cuda()
            dt.dnatok_decode(v.handle, d.data_ptr(), n_ids, torch.from_numpy(offs).cuda().data_ptr(), len(offs) - 1,
                             out.data_ptr() + 3, room, oo.data_ptr(), None)
            assert dt.sync_status() == (dt.DERR_CAPACITY if short and cap else 0)
            got = out.cpu().numpy()
            assert np.array_equal(got[3:3 + room], want[:room]) and np.all(got[3 + room:] == 7)
            assert np.array_equal(oo.cpu().numpy(), want_off)
    v.close()
