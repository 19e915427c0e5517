"""GPU parity of the chunked BPE encode on tandem repeats with the committed
4,096-merge table: repeats that cover the edge between two waves (62 chunks of
64 bases, 3,968 bases of a row that starts a wave), where the waves' own
tokens of the shared chunk may differ."""
import numpy as np
import pytest

import paper_2601_05531_amd as dt
import synth
from test_bpe_chunk_rule import ACGT, short_token_table
from test_bpe_wave_model import edge_repeats, load, tandem
from test_gpu_bpe import _packed, _padded

pytestmark = pytest.mark.gpu


def _check(v, merges, rows):
    data, offs = np.concatenate(rows), synth.offsets_from_lengths([len(r) for r in rows])
    _packed(v, merges, data, offs, cls=False)
    _padded(v, merges, data, offs, cls=True, side=1)


@pytest.fixture(scope="module")
def table():
    merges = load()
    v = dt.Vocab(dt.BPE, merges=merges)
    yield v, merges
    v.close()


@pytest.mark.parametrize("motif,bases", [(b"TAT", 4032), (b"TAT", 4033), (b"TAT", 4300), (b"TAT", 8000), (b"TAT", 20000),
                                         (b"TCA", 4033), (b"TCA", 20000), (b"CAG", 20000), (b"AAT", 20000)])
def test_repeat_from_the_row_start(table, motif, bases):
    _check(*table, [tandem(motif, bases)])


@pytest.mark.parametrize("motif", [b"T", b"TGA", b"TAT", b"AC", b"GATA"])
def test_repeats_across_the_wave_edge(table, motif):
    g = np.random.default_rng(len(motif))
    rows = []
    for at, bases in ((3840, 400), (3900, 200), (3923, 145), (3967, 2), (3700, 9000)):
        row = ACGT[g.integers(0, 4, 14000)]
        row[at:at + bases] = tandem(motif, bases)
        _check(*table, [row])
        rows.append(row)
    # the same rows behind one another, so the edges fall elsewhere, with empty and short rows between
    _check(*table, [rows[0], rows[1][:0], rows[2], rows[3][:77], rows[4], rows[1]])


def test_random_repeats_across_the_wave_edge(table):
    v, merges = table
    rows = edge_repeats(np.random.default_rng(8), 300)
    for row in rows[:100]:  # each the first row of its batch: the edge lies at base 3,968
        _packed(v, merges, row, np.array([0, len(row)], np.int64), cls=False)
    _check(v, merges, rows)


@pytest.mark.parametrize("motif", [b"T", b"AC", b"CAG", b"AAT", b"GATA", b"TTAGGG"])
def test_long_repeats_out_of_phase(table, motif):
    """What precedes a long repeat is out of phase with the chunks inside it
    for most lengths: its tokens go on to the repeat's end."""
    g = np.random.default_rng(len(motif))
    rows = []
    for n in range(24):
        tail = ACGT[g.integers(0, 4, int(g.integers(0, 200)))]
        rows.append(np.concatenate([ACGT[g.integers(0, 4, n)], tandem(motif, int(g.integers(300, 6000))), tail]))
    rows.append(np.concatenate([rows[5], rows[9], tandem(b"N", 3), rows[11], rows[2]]))
    soft = np.concatenate([rows[7], tandem(motif, 9000)])
    soft[::3] |= 0x20
    rows.append(soft)
    rows.append(np.concatenate([ACGT[g.integers(0, 4, 77)], tandem(motif, 150000), ACGT[g.integers(0, 4, 77)]]))
    _check(*table, rows)


@pytest.mark.parametrize("seed,R,p_chain,longest", [(1, 6, 0.6, 8), (2, 40, 0.3, 12), (4, 30, 0.6, 32), (5, 60, 0.3, 64)])
def test_random_tables_long_repeats(seed, R, p_chain, longest):
    merges = short_token_table(seed, R, p_chain, longest)
    v = dt.Vocab(dt.BPE, merges=merges)
    g = np.random.default_rng(seed)
    rows = []
    for n in range(60):
        motif = ACGT[g.integers(0, 4, int(g.integers(1, 40)))].tobytes()
        lead = ACGT[g.integers(0, 4, int(g.integers(0, 70)))]
        rows.append(np.concatenate([lead, tandem(motif, int(g.integers(100, 9000))), lead[::-1]]))
    data, offs = np.concatenate(rows), synth.offsets_from_lengths([len(r) for r in rows])
    _packed(v, merges, data, offs, cls=False)
    v.close()


def test_small_table_across_the_wave_edge():
    merges = np.array([(5, 6), (10, 10), (11, 11)], np.int32)
    v = dt.Vocab(dt.BPE, merges=merges)
    for start in (3840, 3899, 3957, 3966):
        for bases in (100, 120, 231, 400):
            row = np.concatenate([tandem(b"G", start), tandem(b"AC", bases), tandem(b"G", 64)])
            _packed(v, merges, row, np.array([0, len(row)], np.int64), cls=False)
    v.close()
