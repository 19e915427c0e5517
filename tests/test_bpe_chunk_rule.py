"""The rule behind the chunked BPE encode, on the CPU against the oracle: two
tokens may be neighbours when undoing their merges, the later one first,
never meets a boundary pair that ranks before the merge that ended it; a
search over such neighbours is the segmentation; and the segmentations of
overlapping texts join at a token that both have."""
import numpy as np
import pytest

import oracle

NO = 1 << 30
ACGT = np.frombuffer(b"ACGT", np.uint8)


def short_token_table(seed, R, p_chain, longest):
    """A random well-formed table whose tokens have at most `longest` bases."""
    rng = np.random.default_rng(seed)
    merges, length, seen = [], {5: 1, 6: 1, 7: 1, 8: 1}, set()
    for _ in range(50 * R):
        ids = [5, 6, 7, 8] + [10 + r for r in range(len(merges))]
        a = int(rng.choice(ids))
        b = a if rng.random() < p_chain else int(rng.choice(ids))
        if len(merges) < R and (a, b) not in seen and length[a] + length[b] <= longest:
            seen.add((a, b))
            length[10 + len(merges)] = length[a] + length[b]
            merges.append((a, b))
    return np.array(merges, np.int32).reshape(-1, 2)


class Rule:
    def __init__(self, merges):
        self.m = [tuple(int(x) for x in p) for p in merges]
        self.rank = {p: r for r, p in enumerate(self.m)}
        text = {5 + i: (i,) for i in range(4)}
        self.tok = {(i,): 5 + i for i in range(4)}
        valid = set(text)
        for r, (a, b) in enumerate(self.m):
            text[10 + r] = text[a] + text[b]
            if a in valid and b in valid and self.holds(a, b, r):
                valid.add(10 + r)
                self.tok[text[10 + r]] = 10 + r
        self.longest = max(len(t) for t in self.tok)

    def holds(self, x, y, limit=NO):
        while True:
            if self.rank.get((x, y), NO) < limit:
                return False
            rx, ry = x - 10 if x >= 10 else -1, y - 10 if y >= 10 else -1
            if rx < 0 and ry < 0:
                return True
            if rx > ry:
                limit, x = rx, self.m[rx][1]
            else:
                limit, y = ry + 1, self.m[ry][0]

    def search(self, digits):
        """[(start, token)] of the text, longest tokens first, back where nothing fits."""
        n, out, dead, p, size = len(digits), [], set(), 0, self.longest
        while p < n:
            while size:
                t = self.tok.get(tuple(digits[p:p + size])) if p + size <= n else None
                if t and p + size not in dead and (not out or self.holds(out[-1][1], t)):
                    break
                size -= 1
            if size:
                out.append((p, t))
                p, size = p + size, self.longest
            else:
                dead.add(p)
                at, _ = out.pop()
                size, p = p - at - 1, at
        return out


@pytest.mark.parametrize("seed,R,p_chain,longest", [(1, 6, 0.6, 8), (2, 40, 0.3, 12), (3, 120, 0.05, 16),
                                                    (4, 30, 0.6, 32), (5, 0, 0.0, 1)])
def test_search_and_joins_equal_the_oracle(seed, R, p_chain, longest):
    merges = short_token_table(seed, R, p_chain, longest)
    rule = Rule(merges)
    rng = np.random.default_rng(100 + seed)
    joined = 0
    for case in range(30):
        L = int(rng.integers(1, 160))
        kind = case % 3
        if kind == 0:
            d = rng.integers(0, 4, size=L)
        elif kind == 1:
            d = np.tile(rng.integers(0, 4, size=int(rng.integers(1, 5))), L)[:L]
        else:
            d = np.repeat(rng.integers(0, 4, size=L), rng.integers(1, 9, size=L))[:L]
        d = [int(x) for x in d]
        want, _ = oracle.encode(oracle.BPE, ACGT[d], np.array([0, L], np.int64), merges=merges)
        whole = rule.search(d)
        assert [t for _, t in whole] == list(want)
        # a cut, both sides read on and joined at the first token they share
        cut = int(rng.integers(0, L))
        left = rule.search(d[:min(L, cut + 64)])
        right = [(p + cut, t) for p, t in rule.search(d[cut:])]
        both = sorted(set(left) & set(right))
        if both:
            at = both[0][0]
            joined += 1
            assert [x for x in left if x[0] < at] + [x for x in right if x[0] >= at] == whole
    assert joined >= 10
