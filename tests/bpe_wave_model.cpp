// CPU model of the chunked BPE encode: the waves of k_bpe_chunks with their
// lanes in lockstep, the two chunks that a wave repeats of its neighbours, the
// edge words, and the walk over what did not meet. It keeps the kernel's
// decisions (what ends a lane's search, what counts as met, what an edge word
// holds) and none of its code; tables come from the merges by brute force.
#include <algorithm>
#include <cstdint>
#include <map>
#include <unordered_map>
#include <vector>

namespace {

constexpr int kChunk = 64;
constexpr uint32_t kReach = 127, kNoRank = 0xFFFFu, kUnk = 1, kN = 9;

struct Node {
    uint32_t kid[4] = {0, 0, 0, 0}, tok = 0;
};

struct Table {
    std::vector<std::pair<uint32_t, uint32_t>> m;
    std::unordered_map<uint32_t, uint32_t> ranks;
    std::vector<std::vector<uint8_t>> text;
    std::vector<uint32_t> link;  // next shorter token that begins it
    std::vector<Node> trie;
    std::vector<int8_t> memo;    // may b follow a: -1 unknown
    uint32_t V = 0;

    uint32_t rank(uint32_t a, uint32_t b) const {
        auto it = ranks.find(a | (b << 16));
        return it == ranks.end() ? kNoRank : it->second;
    }
    bool holds(uint32_t x, uint32_t y, uint32_t limit) const {
        for (;;) {
            if (rank(x, y) < limit) return false;
            const int rx = x >= 10 ? (int)x - 10 : -1, ry = y >= 10 ? (int)y - 10 : -1;
            if (rx < 0 && ry < 0) return true;
            if (rx > ry) limit = (uint32_t)rx, x = m[rx].second;
            else limit = (uint32_t)ry + 1, y = m[ry].first;
        }
    }
    bool follows(uint32_t a, uint32_t b) {
        if (!b) return false;
        int8_t &x = memo[(size_t)a * V + b];
        if (x < 0) x = holds(a, b, kNoRank);
        return x;
    }
    uint32_t bases(uint32_t t) const { return t >= 5 && t != kN ? (uint32_t)text[t].size() : 1u; }
    uint32_t longest_bases() const {
        size_t n = 1;
        for (const auto &x : text) n = std::max(n, x.size());
        return (uint32_t)n;
    }
    // longest token that the len bases at d begin with
    uint32_t longest(const uint8_t *d, int64_t len) const {
        if (d[0] > 3) return d[0] == 4 ? kN : kUnk;
        uint32_t at = 0, tok = 0;
        for (int64_t i = 0; i < len && d[i] < 4; ++i) {
            at = trie[at].kid[d[i]];
            if (!at) break;
            if (trie[at].tok) tok = trie[at].tok;
        }
        return tok;
    }
    Table(const int32_t *merges, int32_t R) : text(10 + R), link(10 + R, 0), trie(1), V(10 + (uint32_t)R) {
        for (int32_t r = 0; r < R; ++r) {
            m.push_back({(uint32_t)merges[2 * r], (uint32_t)merges[2 * r + 1]});
            ranks[m[r].first | (m[r].second << 16)] = (uint32_t)r;
        }
        memo.assign((size_t)V * V, -1);
        std::vector<char> valid(V, 0);
        for (uint32_t b = 0; b < 4; ++b) text[5 + b] = {(uint8_t)b}, valid[5 + b] = 1;
        for (uint32_t id = 5; id < V; ++id) {
            if (id >= 10) {
                const auto [a, b] = m[id - 10];
                text[id] = text[a];
                text[id].insert(text[id].end(), text[b].begin(), text[b].end());
                valid[id] = valid[a] && valid[b] && holds(a, b, id - 10);
            }
            if (!valid[id]) continue;
            uint32_t at = 0;
            for (uint8_t c : text[id]) {
                if (!trie[at].kid[c]) {
                    trie[at].kid[c] = (uint32_t)trie.size();
                    trie.emplace_back();
                }
                at = trie[at].kid[c];
            }
            trie[at].tok = id;
        }
        for (uint32_t id = 10; id < V; ++id) {
            uint32_t at = 0;
            for (size_t j = 0; valid[id] && j + 1 < text[id].size(); ++j) {
                at = trie[at].kid[text[id][j]];
                if (trie[at].tok) link[id] = trie[at].tok;
            }
        }
    }
};

typedef unsigned __int128 Bits;
uint32_t lowest(uint64_t x) { return (uint32_t)__builtin_ctzll(x); }
uint32_t highest(Bits b) {
    const uint64_t hi = (uint64_t)(b >> 64);
    return hi ? 127u - (uint32_t)__builtin_clzll(hi) : 63u - (uint32_t)__builtin_clzll((uint64_t)b);
}

struct Chunk {
    int32_t row;
    int64_t at;    // first base in the row
    int64_t left;  // bases of the row from there on
    bool failed = false;
    uint64_t mask = 0;
};

struct Model {
    Table t;
    std::vector<Chunk> chunks;
    std::vector<uint32_t> edge;  // two per wave
    std::vector<std::vector<uint8_t>> rows;
    std::vector<std::vector<uint32_t>> sym;  // token that starts at a base
    int lanes = 64;

    Model(const int32_t *merges, int32_t R) : t(merges, R) {}
    int own() const { return lanes - 2; }

    struct Lane {
        bool valid = false, prev_same = false, next_same = false;
        int64_t left = 0;
        uint32_t end = 0, p = 0, prev = 0, cand = 0, meet = 0;
        Bits starts = 1, closed = 0;
        std::vector<uint32_t> toks;  // tokens before p, in order
    };

    void wave(int64_t task, bool edge_rule) {
        const int64_t total = (int64_t)chunks.size(), first = task * own() - 1;
        std::vector<Lane> w(lanes);
        auto best = [&](int lane, uint32_t x) -> uint32_t {
            const int64_t c = first + lane + (x >> 6);
            if (lane + (int)(x >> 6) >= lanes || c >= total || (int64_t)(x & 63) >= chunks[c].left) return 0;
            return t.longest(rows[chunks[c].row].data() + chunks[c].at + (x & 63), chunks[c].left - (x & 63));
        };
        for (int l = 0; l < lanes; ++l) {
            Lane &a = w[l];
            const int64_t c = first + l;
            a.valid = c >= 0 && c < total;
            if (!a.valid) continue;
            a.left = chunks[c].left;
            a.end = (uint32_t)std::min<int64_t>(a.left, l == lanes - 1 ? kChunk : kReach);
            a.prev_same = l > 0 && chunks[c].at > 0;
            a.next_same = l < lanes - 1 && c + 1 < total && chunks[c + 1].at > 0;
            a.cand = best(l, 0);
        }
        for (uint32_t step = 0;; ++step) {
            if (step % 4 == 0) {
                bool any_need = false;
                for (int l = 0; l < lanes; ++l) {
                    Lane &a = w[l];
                    // the end of the first token that this lane and the next both hold
                    a.meet = 0;
                    const uint64_t mine = (uint64_t)(a.starts >> 64), next = l + 1 < lanes ? (uint64_t)w[l + 1].starts : 0;
                    bool common = false;
                    for (int x = 0; a.next_same && x < 64 && !a.meet; ++x) {
                        const bool i = (mine >> x) & 1, j = (next >> x) & 1;
                        if (i && j && common) a.meet = (uint32_t)x;
                        if (i || j) common = i && j;
                    }
                    if (a.next_same && a.p == a.end && a.left == (int64_t)a.end) a.meet = a.end - kChunk;
                    any_need = any_need || (a.valid && a.p != a.end && (l == lanes - 1 ? a.prev_same : a.meet == 0));
                }
                if (!any_need) break;
            }
            // (a lane that is done waits for the others' next look)
            std::vector<char> go(lanes);
            for (int l = 0; l < lanes; ++l)
                go[l] = w[l].valid && w[l].p != w[l].end && (l == lanes - 1 ? w[l].prev_same : w[l].meet == 0);
            for (int l = 0; l < lanes; ++l) {
                if (!go[l]) continue;
                Lane &a = w[l];
                // the candidate and the two next shorter ones
                uint32_t c = a.cand, took = 0;
                for (int i = 0; i < 3 && c && !took; ++i, c = took ? c : t.link[c]) {
                    const uint32_t q = a.p + t.bases(c);
                    if (q <= a.end && !((a.closed >> q) & 1) && t.follows(a.prev, c)) took = c;
                }
                if (took) {
                    a.toks.push_back(took);
                    a.prev = took;
                    a.p += t.bases(took);
                    a.starts |= (Bits)1 << a.p;
                    a.cand = best(l, a.p);
                } else if (c) {
                    a.cand = c;
                } else {
                    a.closed |= (Bits)1 << a.p;
                    a.starts &= ~((Bits)1 << a.p);
                    a.cand = a.prev;  // its end is closed now, so a shorter one follows
                    a.p -= t.bases(a.prev);
                    a.toks.pop_back();
                    a.prev = a.toks.empty() ? 0 : a.toks.back();
                }
            }
        }
        for (int l = 0; l < lanes; ++l) {
            const Lane &a = w[l];
            const int64_t c = first + l;
            const uint64_t below = a.prev_same ? (1ull << w[l - 1].meet) - 1 : 0;
            const uint64_t lo = ((uint64_t)a.starts & ~below) | (l ? (uint64_t)(w[l - 1].starts >> 64) & below : 0);
            const uint64_t hi = (uint64_t)(a.starts >> 64);
            if (l == 0 || l == lanes - 2) {
                const uint32_t side = l ? 1 : 0;
                uint32_t token = 0;
                if (a.next_same) {
                    token = 0x20000u + side;
                    if (lo && hi && (side || a.meet || !edge_rule))
                        token = 0x10000u | ((63u - (uint32_t)__builtin_clzll(lo)) << 8) | lowest(hi);
                }
                edge[2 * task + side] = token;
            }
            if (l == 0 || l == lanes - 1 || !a.valid) continue;
            chunks[c].failed = a.next_same && !a.meet;
            chunks[c].mask = a.left >= kChunk ? lo : lo & ((1ull << a.left) - 1);
        }
    }

    bool fails(int64_t c) const {
        if (chunks[c].failed) return true;
        const int64_t w = c / own();
        return c == w * own() + own() - 1 && 2 * w + 2 < (int64_t)edge.size() && edge[2 * w + 1] != edge[2 * w + 2];
    }

    // Row r's chunks cb.. from the first that does not go on: the search with
    // the row's own starts as its stack. Where the tokens taken repeat (looked
    // for every eight, among the last 64), those of all repetitions that the
    // text goes on with are taken at once.
    void walk(int64_t cb, int64_t ce, int64_t *walked, int64_t *at_once) {
        const int32_t r = chunks[cb].row;
        const std::vector<uint8_t> &d = rows[r];
        const int64_t L = (int64_t)d.size();
        std::vector<char> start(L + 1, 0), dead(L + 1, 0);
        auto load = [&](int64_t c) {
            for (int x = 0; x < kChunk && chunks[c].at + x < L; ++x) start[chunks[c].at + x] = (chunks[c].mask >> x) & 1;
        };
        for (int64_t c = cb; c < ce; ++c) load(c);
        auto before = [&](int64_t p) {
            while (!start[--p]) {}
            return p;
        };
        auto token_at = [&](int64_t p, int64_t q) {
            uint32_t tok = t.longest(d.data() + p, L - p);
            while (tok && (int64_t)t.bases(tok) != q - p) tok = t.link[tok];
            return tok;
        };
        auto next_failed = [&](int64_t c) {
            while (c < ce && !fails(c)) ++c;
            return c;
        };
        for (int64_t f = next_failed(cb); f < ce;) {
            const int64_t f_end = (f - cb + 1) * kChunk;
            int64_t p = before(std::min(f_end, L)), from = p;
            std::vector<char> old = start;
            for (int64_t x = f_end; x < L; ++x) start[x] = 0;
            std::fill(dead.begin(), dead.end(), 0);
            uint32_t prev = p ? token_at(before(p), p) : 0, cand = t.longest(d.data() + p, L - p);
            int64_t resume = -1;
            std::vector<std::pair<int64_t, uint32_t>> taken;  // since the last that the search did not take
            int until = 8;
            for (;;) {
                if (!cand) {
                    if (!taken.empty()) taken.pop_back();
                    dead[p] = 1;
                    start[p] = 0;
                    p = before(p);
                    prev = p ? token_at(before(p), p) : 0;
                    cand = t.longest(d.data() + p, L - p);
                    continue;
                }
                const int64_t q = p + t.bases(cand);
                if (q > L || dead[q] || !t.follows(prev, cand)) {
                    cand = t.link[cand];
                    continue;
                }
                if (q == L) {
                    resume = L;
                    break;
                }
                start[q] = 1;
                if (p >= f_end && old[p] && old[q]) {
                    bool met = true;
                    for (int64_t x = p + 1; x < q; ++x) met = met && !old[x];
                    for (int64_t c = p / kChunk; c < q / kChunk; ++c) met = met && !fails(cb + c);
                    if (met) {
                        resume = q;
                        break;
                    }
                }
                taken.push_back({p, cand});
                prev = cand;
                p = q;
                if (--until == 0) {
                    until = 8;
                    const size_t n = taken.size();
                    for (size_t j = 1; 2 * j <= std::min<size_t>(n, 64); ++j) {
                        bool again = true;
                        for (size_t i = 1; again && i <= j; ++i) again = taken[n - i].second == taken[n - i - j].second;
                        if (!again) continue;
                        const int64_t bases = p - taken[n - j].first;
                        int64_t end = p;
                        while (end < L && d[end] == d[end - bases]) ++end;
                        const int64_t room = std::max<int64_t>(0, end - 2 * (int64_t)t.longest_bases() - p);
                        const int64_t past = p + room / bases * bases;
                        if (past - p >= 96) {
                            for (int64_t x = p + 1; x <= past; ++x) start[x] = start[x - bases];
                            *at_once += past - p;
                            p = past;
                            taken.clear();
                        }
                        break;
                    }
                }
                cand = t.longest(d.data() + p, L - p);
            }
            *walked += resume - from;
            for (int64_t x = resume; x < L; ++x) start[x] = old[x];
            f = resume == L ? ce : next_failed(cb + resume / kChunk);
        }
        for (int64_t c = cb; c < ce; ++c) {
            chunks[c].mask = 0;
            for (int x = 0; x < kChunk && chunks[c].at + x < L; ++x)
                chunks[c].mask |= (uint64_t)start[chunks[c].at + x] << x;
        }
    }

    int64_t encode(const uint8_t *bytes, const int64_t *offs, int32_t n, int wave_lanes, bool edge_rule, int32_t *ids,
                   int64_t *out_offs, int64_t *stats) {
        lanes = wave_lanes;
        rows.clear();
        chunks.clear();
        std::vector<int64_t> first;
        for (int32_t r = 0; r < n; ++r) {
            std::vector<uint8_t> d;
            for (int64_t i = offs[r]; i < offs[r + 1]; ++i) {
                const char f = (char)(bytes[i] | 0x20);
                d.push_back(f == 'a' ? 0 : f == 'c' ? 1 : f == 'g' ? 2 : f == 't' ? 3 : f == 'n' ? 4 : 5);
            }
            rows.push_back(d);
            first.push_back((int64_t)chunks.size());
            const int64_t L = (int64_t)d.size();
            for (int64_t at = 0; at == 0 || at < L; at += kChunk) chunks.push_back(Chunk{r, at, L - at});
        }
        first.push_back((int64_t)chunks.size());
        const int64_t tasks = ((int64_t)chunks.size() + own() - 1) / own();
        edge.assign(2 * tasks, 0);
        for (int64_t k = 0; k < tasks; ++k) wave(k, edge_rule);
        std::fill(stats, stats + 3, 0);  // chunks that did not go on, bases walked, of them at once
        for (int64_t c = 0; c < (int64_t)chunks.size(); ++c) stats[0] += fails(c);
        int64_t out = 0;
        for (int32_t r = 0; r < n; ++r) {
            out_offs[r] = out;
            walk(first[r], first[r + 1], &stats[1], &stats[2]);
            const int64_t L = (int64_t)rows[r].size();
            std::vector<int64_t> at;
            for (int64_t c = first[r]; c < first[r + 1]; ++c)
                for (uint64_t y = chunks[c].mask; y; y &= y - 1) at.push_back(chunks[c].at + lowest(y));
            at.push_back(L);
            for (size_t i = 0; i + 1 < at.size(); ++i) {
                uint32_t tok = t.longest(rows[r].data() + at[i], L - at[i]);
                while (tok && (int64_t)t.bases(tok) > at[i + 1] - at[i]) tok = t.link[tok];
                ids[out++] = (int32_t)tok;
            }
        }
        out_offs[n] = out;
        return out;
    }
};

}  // namespace

extern "C" {
void *model_new(const int32_t *merges, int32_t R) { return new Model(merges, R); }
void model_free(void *m) { delete static_cast<Model *>(m); }
int64_t model_encode(void *m, const uint8_t *bytes, const int64_t *offs, int32_t n, int32_t lanes, int32_t edge_rule,
                     int32_t *ids, int64_t *out_offs, int64_t *stats) {
    return static_cast<Model *>(m)->encode(bytes, offs, n, lanes, edge_rule != 0, ids, out_offs, stats);
}
}
