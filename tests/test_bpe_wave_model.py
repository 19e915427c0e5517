"""The chunked BPE encode's waves on the CPU (bpe_wave_model.cpp: lanes in
lockstep, the chunks that a wave repeats of its neighbours, the edge words,
the walk) against the oracle, over tandem repeats laid across the edge between
two waves. A wave's last lane ends at its chunk's last base and the next
wave's lanes do not, so the two may hold different tokens at the edge."""
import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import oracle
import synth
from test_bpe_chunk_rule import ACGT, short_token_table

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "golden"))
from make_bpe4096 import load  # noqa: E402


def tandem(motif, bases):
    return np.tile(np.frombuffer(motif, np.uint8), bases // len(motif) + 1)[:bases].copy()


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    so = str(tmp_path_factory.mktemp("model") / "model.so")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-fPIC", "-shared", "-o", so,
                        os.path.join(HERE, "bpe_wave_model.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(so)
    lib.model_new.restype = ctypes.c_void_p
    lib.model_new.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    lib.model_free.argtypes = [ctypes.c_void_p]
    lib.model_encode.restype = ctypes.c_int64
    lib.model_encode.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 3 + [ctypes.c_void_p] * 3
    return lib


class Model:
    def __init__(self, lib, merges):
        self.lib, self.merges = lib, np.ascontiguousarray(merges, np.int32)
        self.h = lib.model_new(self.merges.ctypes.data, len(self.merges))

    def __call__(self, rows, lanes=64, edge_rule=True):
        data, offs = np.concatenate(rows), synth.offsets_from_lengths([len(r) for r in rows])
        ids, out = np.empty(len(data) + 1, np.int32), np.empty(len(offs), np.int64)
        stats = np.zeros(3, np.int64)
        total = self.lib.model_encode(self.h, data.ctypes.data, offs.ctypes.data, len(rows), lanes, int(edge_rule),
                                      ids.ctypes.data, out.ctypes.data, stats.ctypes.data)
        return ids[:total], out, stats

    def check(self, rows, lanes=64):
        ids, out, stats = self(rows, lanes)
        data, offs = np.concatenate(rows), synth.offsets_from_lengths([len(r) for r in rows])
        want, want_off = oracle.encode(oracle.BPE, data, offs, merges=self.merges)
        assert np.array_equal(out, want_off) and np.array_equal(ids, want)
        return stats

    def close(self):
        self.lib.model_free(self.h)


def test_repeats_over_the_wave_edge(lib):
    m = Model(lib, load())
    for L in (4032, 4033, 4300, 8000):
        m.check([tandem(b"TAT", L)])
    m.check([tandem(b"TCA", 8000)])
    g = np.random.default_rng(1)
    poly = ACGT[g.integers(0, 4, 6000)]
    poly[3900:4100] = ord("T")
    m.check([poly])
    # 145 bases of TGA, and ordinary rows before the edge
    tga = ACGT[g.integers(0, 4, 6000)]
    tga[3923:3923 + 145] = tandem(b"TGA", 145)
    m.check([tga])
    m.check([poly[:700], tandem(b"TAT", 5000), poly[:0], tandem(b"CAG", 9000)])
    # repeats out of phase with the chunks inside them are walked to their end
    for motif in (b"T", b"AC", b"CAG", b"GATA"):
        rows = [np.concatenate([ACGT[g.integers(0, 4, lead)], tandem(motif, 3000), ACGT[g.integers(0, 4, 50)]])
                for lead in range(0, 36, 3)]
        at_once = [m.check([row])[2] for row in rows]
        assert max(at_once) > 2500 or motif == b"GATA"
    m.close()


def edge_repeats(g, rows):
    """Rows of random bases with a repeat of 1 to 6 bases across base 3,968."""
    out = []
    for _ in range(rows):
        row = ACGT[g.integers(0, 4, int(g.integers(4300, 5000)))]
        at, bases = int(g.integers(3840, 3969)), int(g.integers(100, 401))
        repeat = tandem(ACGT[g.integers(0, 4, int(g.integers(1, 7)))].tobytes(), bases)
        row[at:at + bases] = repeat[:len(row) - at]
        out.append(row)
    return out


def test_random_repeats_over_the_wave_edge(lib):
    m = Model(lib, load())
    unmet = [m.check([row])[0] for row in edge_repeats(np.random.default_rng(7), 160)]
    assert sum(x > 0 for x in unmet) > 10
    m.close()


def test_small_table_over_the_wave_edge(lib):
    m = Model(lib, np.array([(5, 6), (10, 10), (11, 11)], np.int32))
    row = np.concatenate([tandem(b"G", 3957), tandem(b"AC", 120), tandem(b"G", 64)])
    m.check([row])
    # the case needs the rule: a wave that did not meet its second lane must say so at the edge
    want = oracle.encode(oracle.BPE, row, np.array([0, len(row)]), merges=m.merges)[0]
    assert len(m([row], edge_rule=False)[0]) != len(want)
    for start in range(3840, 3970, 7):
        for bases in (100, 131, 222, 400):
            m.check([np.concatenate([tandem(b"G", start), tandem(b"AC", bases), tandem(b"G", 64)])])
    m.close()


@pytest.mark.parametrize("seed,R,p_chain,longest", [(1, 6, 0.6, 8), (2, 40, 0.3, 12), (3, 120, 0.05, 16),
                                                    (4, 30, 0.6, 32), (5, 60, 0.3, 64), (6, 0, 0.0, 1)])
@pytest.mark.parametrize("lanes", [8, 64])
def test_random_tables(lib, seed, R, p_chain, longest, lanes):
    m = Model(lib, short_token_table(seed, R, p_chain, longest))
    g = np.random.default_rng(seed)
    unmet = 0
    for _ in range(60 if lanes == 8 else 12):
        rows = []
        for _ in range(int(g.integers(1, 4))):
            L, parts = int(g.integers(0, 100 * lanes)), [ACGT[:0]]
            while sum(map(len, parts)) < L:
                some = ACGT[g.integers(0, 4, int(g.integers(1, 7)))]
                parts.append(np.tile(some, 400)[:int(g.integers(1, 400))] if g.random() < 0.7 else
                             ACGT[g.integers(0, 4, int(g.integers(1, 200)))])
            rows.append(np.concatenate(parts)[:L])
        rows.append(ACGT[:1])
        unmet += m.check(rows, lanes)[0]
    assert unmet > 0 or R == 0
    m.close()
