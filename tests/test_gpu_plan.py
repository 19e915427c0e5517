"""Host sizing of an encode (dnatok_encode_plan) against exact arithmetic:
row counts around its blocks of 1,024 rows, blocks of more than 2^31 bases,
every k, stride-1 windows, and the row named when offsets decrease. Marked gpu
because a vocabulary needs a device."""
import numpy as np
import pytest

import paper_2601_05531_amd as dt

pytestmark = pytest.mark.gpu


def _want(offs, k, cls, overlap):
    tokens = []
    for L in np.diff(offs).tolist():
        body = (L - k + 1 if L >= k else int(L > 0)) if overlap else -(-L // k)
        tokens.append(body + 2 * cls)
    return sum(tokens), max(tokens, default=0)


@pytest.mark.parametrize("k", range(1, 16))
def test_plan_is_exact(k):
    rng = np.random.default_rng(k)
    v = dt.Vocab(dt.KMER, k=k)
    for n in (0, 1, 1023, 1024, 1025, 3000):
        for hi in (1, 20, 4000, 1 << 31, 1 << 40):
            offs = np.concatenate([[7], 7 + np.cumsum(rng.integers(0, hi + 1, n))]).astype(np.int64)
            for cls in (False, True):
                assert dt.plan(v, offs, cls) == _want(offs, k, cls, False)
                assert dt.plan(v, offs, cls, dt.VARIANT_OVERLAP) == _want(offs, k, cls, True)
            if n > 1 and hi > 1:
                at = int(rng.integers(1, n))
                offs[at] = offs[at - 1] - 1
                with pytest.raises(dt.DnatokError) as e:
                    dt.plan(v, offs)
                assert e.value.code == dt.EINVAL and str(e.value).endswith("row %d" % (at - 1))
    v.close()
