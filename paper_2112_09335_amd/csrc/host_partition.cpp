// Deterministic multilevel partitioner: size-capped synchronous label propagation until it rests, contraction of
// the clusters to the nodes of the next level, greedy merging on the last level along the heaviest connection,
// and propagation on the finest graph at the end until it rests again.
// The paper leaves the partition to METIS (Section 2); this is the library's own stand-in, every tie broken
// by node or cluster number so that the result depends on nothing but the input.
#include "host_partition.h"

#include <algorithm>
#include <atomic>
#include <map>
#include <queue>
#include <tuple>
#include <vector>

#include "host_pool.h"

namespace cadmm {

namespace {

// Weighted graph of one level: neighbours of a node ascending, no repeats, no self.
// A row is [ptr[i], end[i]).  Without ew every edge weighs one, without nw every node.
struct Level {
    int64_t n = 0;
    HVec<int64_t> ptr;             // [n]
    HVec<int64_t> end;             // [n]
    HVec<int32_t> col;
    std::vector<int64_t> ew;       // edge weights, parallel to col
    std::vector<int64_t> nw;       // [n] node weights
    int64_t weight(int64_t v) const { return nw.empty() ? 1 : nw[(size_t)v]; }
};

Level finest_level(HostPool& pool, int64_t N, int64_t n_edges, const int32_t* src, const int32_t* dst) {
    Level g;
    g.n = N;
    HVec<int32_t> len;
    distinct_neighbours(pool, N, n_edges, src, dst, [](int32_t x) { return x; }, g.ptr, g.col, len);
    g.end.resize((size_t)N);
    pool.run(N, 65536, [&](int64_t lo, int64_t hi, int) {
        for (int64_t i = lo; i < hi; ++i) g.end[(size_t)i] = g.ptr[(size_t)i] + len[(size_t)i];
    });
    return g;
}

inline bool takes_part(uint64_t v, uint64_t r) {
    return (((v * 2654435761ull + r * 40503ull) >> 16) & 1ull) == 0;     // arithmetic modulo 2^64
}

// Weights by label for one node's neighbours: an open hash table of at least twice their number that remembers which
// slots it has used.
class LabelWeights {
public:
    void begin(int64_t n) {
        for (const uint32_t s : used_) slot_[s].label = -1;
        used_.clear();
        int bits = 4;
        while ((int64_t)1 << bits < 2 * n) ++bits;
        if (bits > bits_) {
            bits_ = bits;
            slot_.assign((size_t)1 << bits, Slot{-1, 0});
        }
        shift_ = 32 - bits;
    }
    void add(int32_t label, int64_t w) {
        uint32_t s = ((uint32_t)label * 2654435769u) >> shift_;
        const uint32_t mask = (1u << (32 - shift_)) - 1;
        while (slot_[s].label != label) {
            if (slot_[s].label < 0) { slot_[s] = Slot{label, 0}; used_.push_back(s); break; }
            s = (s + 1) & mask;
        }
        slot_[s].w += w;
    }
    template <class F>
    void each(F f) const {
        for (const uint32_t s : used_) f(slot_[s].label, slot_[s].w);
    }

private:
    struct Slot { int32_t label; int64_t w; };
    std::vector<Slot> slot_;
    std::vector<uint32_t> used_;
    int bits_ = 0, shift_ = 28;
};

// What the rounds of one level keep between them.  A node that wants no move wants none until its own label or a
// neighbour's changes, so only the nodes marked `dirty` are looked at: those around the last moves, and those whose wish was
// refused for lack of room.  Late rounds, in which little moves, then cost what moves and not a pass over the graph.
struct Propagation {
    std::vector<int32_t> label;    // [n]
    std::vector<int64_t> size;     // weight of the nodes with a label
    std::vector<int64_t> granted;  // weight let into a label this round; zero between rounds
    HVec<uint8_t> dirty;           // [n]
    HVec<int32_t> want;            // [n] the label a node listed in `movers` wants
    std::vector<std::vector<int32_t>> movers;    // per block of nodes, ascending
    Propagation(HostPool& pool, int64_t n) {
        dirty.resize((size_t)n);
        want.resize((size_t)n);
        pool.run(n, 65536, [&](int64_t lo, int64_t hi, int) { std::fill(dirty.begin() + lo, dirty.begin() + hi, (uint8_t)1); });
    }
};

constexpr int64_t kRoundBlock = 256;       // nodes per block of a round

// One synchronous round.  label[v] in [0, size.size()); size[c] = weight of the nodes with label c.
// Returns the number of moves.
int64_t propagation_round(HostPool& pool, const Level& g, Propagation& p, int64_t cap, int r) {
    const int64_t n = g.n;
    const int64_t nb = (n + kRoundBlock - 1) / kRoundBlock;
    p.movers.resize((size_t)nb);
    std::vector<int32_t>& label = p.label;
    pool.run(nb, 1, [&](int64_t b0, int64_t b1, int) {
        LabelWeights seen;
        for (int64_t blk = b0; blk < b1; ++blk) {
            std::vector<int32_t>& out = p.movers[(size_t)blk];
            out.clear();
            for (int64_t v = blk * kRoundBlock; v < std::min(n, (blk + 1) * kRoundBlock); ++v) {
                if (!p.dirty[(size_t)v]) continue;
                const int64_t b = g.ptr[(size_t)v], e = g.end[(size_t)v];
                if (b == e) { p.dirty[(size_t)v] = 0; continue; }
                if (!takes_part((uint64_t)v, (uint64_t)r)) continue;
                const int32_t own = label[(size_t)v];
                seen.begin(e - b);
                for (int64_t k = b; k < e; ++k) seen.add(label[(size_t)g.col[(size_t)k]], g.ew.empty() ? 1 : g.ew[(size_t)k]);
                int32_t best = -1;
                int64_t best_w = 0, own_w = 0;
                seen.each([&](int32_t lab, int64_t w) {                  // the heaviest; of equal ones the smallest label
                    if (w > best_w || (w == best_w && lab < best)) { best_w = w; best = lab; }
                    if (lab == own) own_w = w;
                });
                if (best_w > own_w) { p.want[(size_t)v] = best; out.push_back((int32_t)v); }
                else p.dirty[(size_t)v] = 0;
            }
        }
    });
    // Room is given out in node order; size[] still holds the weights at the start of the round.  Who is refused stays
    // dirty and leaves the list.
    int64_t moves = 0;
    for (auto& out : p.movers) {
        size_t kept = 0;
        for (const int32_t v : out) {
            const int32_t c = p.want[(size_t)v];
            if (g.weight(v) <= cap - p.size[(size_t)c] - p.granted[(size_t)c]) { p.granted[(size_t)c] += g.weight(v); out[kept++] = v; }
        }
        out.resize(kept);
        moves += (int64_t)kept;
    }
    // The moves.  Labels of different nodes are different words; the weights are sums of whole numbers, in any order; a
    // mark is only written where there is none (several threads may mark the same node, and a line that is only read
    // does not bounce between cores).
    auto mark = [&](int64_t v) {
        uint8_t* d = &p.dirty[(size_t)v];
        if (!__atomic_load_n(d, __ATOMIC_RELAXED)) __atomic_store_n(d, (uint8_t)1, __ATOMIC_RELAXED);
    };
    if (moves > 0)
        pool.run(nb, 1, [&](int64_t b0, int64_t b1, int) {
            for (int64_t blk = b0; blk < b1; ++blk)
                for (const int32_t v : p.movers[(size_t)blk]) {
                    const int32_t from = label[(size_t)v], to = p.want[(size_t)v];
                    __atomic_fetch_sub(&p.size[(size_t)from], g.weight(v), __ATOMIC_RELAXED);
                    __atomic_fetch_add(&p.size[(size_t)to], g.weight(v), __ATOMIC_RELAXED);
                    __atomic_store_n(&p.granted[(size_t)to], (int64_t)0, __ATOMIC_RELAXED);
                    label[(size_t)v] = to;
                    mark(v);
                    for (int64_t k = g.ptr[(size_t)v]; k < g.end[(size_t)v]; ++k) mark(g.col[(size_t)k]);
                }
        });
    return moves;
}

// Rounds until two in a row move nothing (a round asks about half of the nodes), at most kPartitionMaxRounds.
void propagate(HostPool& pool, const Level& g, Propagation& p, int64_t cap) {
    int quiet = 0;
    for (int r = 0; r < kPartitionMaxRounds && quiet < 2; ++r) quiet = propagation_round(pool, g, p, cap, r) == 0 ? quiet + 1 : 0;
}

// Clusters numbered in increasing order of their label become the nodes of the next level.
Level contract(HostPool& pool, const Level& g, const std::vector<int32_t>& label, std::vector<int32_t>& member_of) {
    const int64_t n = g.n;
    std::vector<int32_t> number((size_t)n, -1);
    for (int64_t v = 0; v < n; ++v) number[(size_t)label[(size_t)v]] = 0;
    int32_t K = 0;
    for (int64_t c = 0; c < n; ++c)
        if (number[(size_t)c] == 0) number[(size_t)c] = K++;
    member_of.resize((size_t)n);
    Level h;
    h.n = K;
    h.nw.assign((size_t)K, 0);
    for (int64_t v = 0; v < n; ++v) {
        member_of[(size_t)v] = number[(size_t)label[(size_t)v]];
        h.nw[(size_t)member_of[(size_t)v]] += g.weight(v);
    }
    // members of every cluster; then, cluster by cluster, the clusters its edges lead to, sorted, equal ones added up
    HVec<int64_t> start;
    HVec<int32_t> member((size_t)n);
    stable_counting_sort(pool, n, K, start, [&](int64_t v) { return (int64_t)member_of[(size_t)v]; },
                         [&](int64_t v, int64_t at) { member[(size_t)at] = (int32_t)v; });
    std::vector<std::vector<std::pair<int32_t, int64_t>>> rows((size_t)K);
    // few clusters: a weight per possible target instead of a sort of all edges
    const bool dense = K <= 8192;
    pool.run(K, std::max<int64_t>(1, K / (8 * pool.size())), [&](int64_t a0, int64_t a1, int) {
        std::vector<int64_t> w(dense ? (size_t)K : 0, 0);
        std::vector<std::pair<int32_t, int64_t>> out;
        for (int64_t a = a0; a < a1; ++a) {
            out.clear();
            for (int64_t m = start[(size_t)a]; m < start[(size_t)a + 1]; ++m) {
                const int64_t v = member[(size_t)m];
                for (int64_t k = g.ptr[(size_t)v]; k < g.end[(size_t)v]; ++k) {
                    const int32_t b = member_of[(size_t)g.col[(size_t)k]];
                    if (b == a) continue;
                    const int64_t ew = g.ew.empty() ? 1 : g.ew[(size_t)k];
                    if (!dense) { out.emplace_back(b, ew); continue; }
                    if (w[(size_t)b] == 0) out.emplace_back(b, 0);       // (edge weights are positive)
                    w[(size_t)b] += ew;
                }
            }
            std::sort(out.begin(), out.end());
            if (dense) {
                for (auto& o : out) { o.second = w[(size_t)o.first]; w[(size_t)o.first] = 0; }
            } else {
                size_t kept = 0;
                for (size_t i = 0; i < out.size(); ++i) {
                    if (kept && out[kept - 1].first == out[i].first) out[kept - 1].second += out[i].second;
                    else out[kept++] = out[i];
                }
                out.resize(kept);
            }
            rows[(size_t)a] = out;
        }
    });
    h.ptr.resize((size_t)K);
    h.end.resize((size_t)K);
    int64_t at = 0;
    for (int32_t a = 0; a < K; ++a) {
        h.ptr[(size_t)a] = at;
        at += (int64_t)rows[(size_t)a].size();
        h.end[(size_t)a] = at;
    }
    h.col.resize((size_t)at);
    h.ew.resize((size_t)at);
    for (int32_t a = 0; a < K; ++a) {
        int64_t o = h.ptr[(size_t)a];
        for (const auto& e : rows[(size_t)a]) { h.col[(size_t)o] = e.first; h.ew[(size_t)o++] = e.second; }
    }
    return h;
}

// Community of every node of the last level: merge along the heaviest admissible connection, then the lightest
// nodes regardless of the cap, until at most M are left.
std::vector<int32_t> merge_down_to(const Level& g, int32_t M, int64_t cap) {
    const int32_t K = (int32_t)g.n;
    std::vector<std::map<int32_t, int64_t>> adj(K);
    using Entry = std::tuple<int64_t, int32_t, int32_t>;        // (-weight, a, b): the smallest entry is the wanted pair
    std::priority_queue<Entry, std::vector<Entry>, std::greater<Entry>> heap;
    for (int32_t a = 0; a < K; ++a)
        for (int64_t k = g.ptr[a]; k < g.end[a]; ++k) {
            const int64_t ew = g.ew.empty() ? 1 : g.ew[(size_t)k];
            adj[a][g.col[(size_t)k]] = ew;
            if (a < g.col[(size_t)k]) heap.emplace(-ew, a, g.col[(size_t)k]);
        }
    std::vector<int64_t> weight((size_t)K);
    for (int32_t c = 0; c < K; ++c) weight[c] = g.weight(c);
    std::vector<char> alive(K, 1);
    std::vector<int32_t> into(K);
    for (int32_t c = 0; c < K; ++c) into[c] = c;
    int32_t n_alive = K;
    auto absorb = [&](int32_t a, int32_t b) {                   // b disappears into a (a < b)
        weight[a] += weight[b];
        weight[b] = 0;
        alive[b] = 0;
        into[b] = a;
        --n_alive;
    };
    // Weights of a pair only change by a merge, which pushes the new value; weights of nodes only grow, so a pair
    // that once did not fit never fits later.  An entry is current if both ends live and the weight is the stored one.
    while (n_alive > M && !heap.empty()) {
        const Entry top = heap.top();
        heap.pop();
        const int32_t a = std::get<1>(top), b = std::get<2>(top);
        if (!alive[a] || !alive[b]) continue;
        auto it = adj[a].find(b);
        if (it == adj[a].end() || it->second != -std::get<0>(top)) continue;
        if (weight[a] + weight[b] > cap) continue;
        for (const auto& kv : adj[b]) {
            const int32_t x = kv.first;
            if (x == a) continue;
            const int64_t w = (adj[a][x] += kv.second);
            adj[x].erase(b);
            adj[x][a] = w;
            heap.emplace(-w, std::min(a, x), std::max(a, x));
        }
        adj[a].erase(b);
        adj[b].clear();
        absorb(a, b);
    }
    while (n_alive > M) {
        int32_t s0 = -1, s1 = -1;                               // lightest and second lightest by (weight, number)
        for (int32_t c = 0; c < K; ++c) {
            if (!alive[c]) continue;
            if (s0 < 0 || weight[c] < weight[s0]) { s1 = s0; s0 = c; }
            else if (s1 < 0 || weight[c] < weight[s1]) s1 = c;
        }
        absorb(std::min(s0, s1), std::max(s0, s1));
    }
    std::vector<int32_t> community(K, -1);
    int32_t n_comm = 0;
    for (int32_t c = 0; c < K; ++c)
        if (alive[c]) community[c] = n_comm++;
    std::vector<int32_t> out(K);
    for (int32_t c = 0; c < K; ++c) {
        int32_t r = c;
        while (into[r] != r) r = into[r];
        out[c] = community[r];
    }
    return out;
}

}  // namespace

std::string partition_graph(int64_t N, int64_t n_edges, const int32_t* src, const int32_t* dst, int32_t M,
                            int32_t* comm) {
    if (N < 1 || N > INT32_MAX) return "N must be in [1, 2^31)";
    if (M < 1) return "M must be positive";
    if (n_edges < 0) return "n_edges must be non-negative";
    if (n_edges > 0 && (!src || !dst)) return "src/dst are null";
    if (!comm) return "comm is null";
    HostPool pool(4 * n_edges + 8 * N);
    std::atomic<bool> bad{false};
    pool.run(n_edges, 65536, [&](int64_t lo, int64_t hi, int) {
        bool b = false;
        for (int64_t e = lo; e < hi; ++e) b |= src[e] < 0 || src[e] >= N || dst[e] < 0 || dst[e] >= N;
        if (b) bad = true;
    });
    if (bad) return "edge endpoint out of range";
    const Level finest = finest_level(pool, N, n_edges, src, dst);
    const int64_t cap = (N + M - 1) / M + (N / M) / 20 + 1;

    // levels: propagate until at rest, contract
    std::vector<std::vector<int32_t>> chain;      // chain[i][v] = node of level i+1 that node v of level i went into
    Level coarse;                                 // the current level once it is no longer the finest
    const Level* g = &finest;
    while (g->n > M) {
        const int64_t n = g->n;
        Propagation p(pool, n);
        p.label.resize((size_t)n);
        p.size.resize((size_t)n);
        p.granted.assign((size_t)n, 0);
        for (int64_t v = 0; v < n; ++v) { p.label[(size_t)v] = (int32_t)v; p.size[(size_t)v] = g->weight(v); }
        propagate(pool, *g, p, cap);
        chain.emplace_back();
        Level next = contract(pool, *g, p.label, chain.back());
        const bool stalled = 20 * next.n > 19 * n;
        coarse = std::move(next);
        g = &coarse;
        if (stalled) break;
    }
    const std::vector<int32_t> top = merge_down_to(*g, M, cap);

    // back to the finest graph, then polish the borders
    Propagation p(pool, N);
    p.label.resize((size_t)N);
    pool.run(N, 16384, [&](int64_t lo, int64_t hi, int) {
        for (int64_t v = lo; v < hi; ++v) {
            int32_t c = (int32_t)v;
            for (const auto& member_of : chain) c = member_of[(size_t)c];
            p.label[(size_t)v] = top[(size_t)c];
        }
    });
    p.size.assign((size_t)M, 0);
    p.granted.assign((size_t)M, 0);
    for (int64_t v = 0; v < N; ++v) p.size[(size_t)p.label[(size_t)v]]++;
    propagate(pool, finest, p, cap);
    std::copy(p.label.begin(), p.label.end(), comm);
    return std::string();
}

}  // namespace cadmm
