// Graph construction on the host: symmetric simple graph -> community-contiguous numbering ->
// CSR of the normalised adjacency -> per-row community segments (paper, Section 2).
#include "host_graph.h"

#include <algorithm>
#include <cmath>

namespace cadmm {

namespace {

// Stored class of a row with len entries (see RowSchedule): -1 = split.
int stored_class(int64_t len) {
    if (len > kSplitThreshold) return -1;
    int k = 0;
    while (k < kLengthClasses - 1 && (int64_t)(4 << k) < len) ++k;     // smallest k with 4 * 2^k >= len, at most 7
    return kLengthClasses - 1 - k;
}

// Row r of the list has the entries [lo(r), hi(r)) of col / val, belongs to group grp(r) (n_groups groups) and goes
// to output row out(r).
template <class Lo, class Hi, class Out, class Grp>
void make_schedule(HostPool& pool, RowSchedule& rs, int64_t nrows, Lo lo, Hi hi, Out out, Grp grp, int32_t n_groups,
                   const int32_t* col, const float* val) {
    rs = RowSchedule();
    // counting sort on (group, class); the rows to be split are picked out in order
    const int64_t nkeys = (int64_t)n_groups * kLengthClasses;
    HVec<int32_t> src((size_t)nrows);                          // list row of scheduled row i
    HVec<int64_t> start;
    stable_counting_sort(
        pool, nrows, nkeys, start,
        [&](int64_t r) {
            const int j = stored_class(hi(r) - lo(r));
            return j < 0 ? (int64_t)-1 : (int64_t)grp(r) * kLengthClasses + j;
        },
        [&](int64_t r, int64_t at) { src[(size_t)at] = (int32_t)r; });
    const int64_t n_sched = start[(size_t)nkeys];
    for (int64_t k = 0; k < nkeys; ++k)
        if (start[(size_t)k + 1] > start[(size_t)k])
            rs.runs.push_back({start[(size_t)k], start[(size_t)k + 1], (int32_t)(k % kLengthClasses), (int32_t)(k / kLengthClasses)});
    rs.n_sched = n_sched;
    std::vector<int64_t> long_src;
    if (n_sched < nrows)
        for (int64_t r = 0; r < nrows; ++r)
            if (stored_class(hi(r) - lo(r)) < 0) long_src.push_back(r);
    // records and chunk ranges: chunk 0 is the padding chunk, then the scheduled rows, then the parts of split rows
    auto chunks_of = [](int64_t len) { return (len + kChunkEntries - 1) / kChunkEntries; };
    HVec<int64_t> chunk0;
    prefix_sum(pool, n_sched, 1, chunk0, [&](int64_t i) {
        const int64_t r = src[(size_t)i];
        return chunks_of(hi(r) - lo(r));
    });
    std::vector<int64_t> part_lo, part_hi;                     // entry ranges of the parts in col / val
    std::vector<RowRecord> part_rec;
    int64_t at = chunk0[(size_t)n_sched];
    rs.long_part_ptr.push_back(0);
    for (int64_t r : long_src) {
        for (int64_t p = lo(r); p < hi(r); p += kSplitPart) {
            const int64_t p1 = p + kSplitPart < hi(r) ? p + kSplitPart : hi(r);
            const int64_t nc = chunks_of(p1 - p);
            part_rec.push_back({(int32_t)at, (int32_t)(at + nc), (int32_t)part_lo.size(), 0});
            part_lo.push_back(p);
            part_hi.push_back(p1);
            at += nc;
        }
        rs.long_row.push_back(out(r));
        rs.long_part_ptr.push_back((int32_t)part_lo.size());
    }
    const int64_t n_parts = (int64_t)part_lo.size();
    rs.rec.resize((size_t)(n_sched + n_parts));
    rs.ent.resize((size_t)at * kChunkEntries);
    for (int k = 0; k < kChunkEntries; ++k) rs.ent[(size_t)k] = EntryPair{0, 0.f};
    auto fill = [&](const RowRecord& rec, int64_t p0, int64_t p1) {
        EntryPair* e = rs.ent.data() + (size_t)rec.chunk0 * kChunkEntries;
        const int64_t n = p1 - p0, padded = (int64_t)(rec.chunk1 - rec.chunk0) * kChunkEntries;
        for (int64_t k = 0; k < n; ++k) e[k] = {col[p0 + k], val[p0 + k]};
        for (int64_t k = n; k < padded; ++k) e[k] = {n > 0 ? col[p0] : 0, 0.f};
    };
    pool.run(n_sched, 1024, [&](int64_t i0, int64_t i1, int) {
        for (int64_t i = i0; i < i1; ++i) {
            const int64_t r = src[(size_t)i];
            RowRecord& rec = rs.rec[(size_t)i];
            rec = {(int32_t)chunk0[(size_t)i], (int32_t)chunk0[(size_t)i + 1], out(r), 0};
            fill(rec, lo(r), hi(r));
        }
    });
    pool.run(n_parts, 64, [&](int64_t k0, int64_t k1, int) {
        for (int64_t k = k0; k < k1; ++k) {
            rs.rec[(size_t)(n_sched + k)] = part_rec[(size_t)k];
            fill(part_rec[(size_t)k], part_lo[(size_t)k], part_hi[(size_t)k]);
        }
    });
}

// What the aggregation kernels rely on: every record names an in-range, non-empty chunk range past the padding chunk,
// the chunk ranges tile the entry array in order, the runs tile the scheduled rows and a row sits in a run whose
// class bounds its length, a part is no longer than kSplitPart, output rows are in range, every column is in range.
bool schedule_ok(HostPool& pool, const RowSchedule& rs, int64_t n_out, int64_t n_cols) {
    const int64_t n = rs.n_rows(), np = rs.n_parts(), nchunks = rs.n_chunks();
    if (n < 0 || np < 0 || nchunks < 1 || nchunks > INT32_MAX || rs.ent.size() % kChunkEntries != 0) return false;
    std::atomic<bool> bad{false};
    pool.run(n + np, 16384, [&](int64_t i0, int64_t i1, int) {
        bool b = false;
        for (int64_t i = i0; i < i1; ++i) {
            const RowRecord& r = rs.rec[(size_t)i];
            b |= r.chunk0 != (i ? rs.rec[(size_t)i - 1].chunk1 : 1) || r.chunk1 <= r.chunk0 || r.chunk1 > nchunks;
            b |= r.out < 0 || r.out >= (i < n ? n_out : np);
            b |= i >= n && (int64_t)(r.chunk1 - r.chunk0) * kChunkEntries > kSplitPart;
        }
        if (b) bad = true;
    });
    if ((n + np ? rs.rec[(size_t)(n + np) - 1].chunk1 : 1) != nchunks) return false;
    pool.run((int64_t)rs.ent.size(), 65536, [&](int64_t i0, int64_t i1, int) {
        bool b = false;
        for (int64_t i = i0; i < i1; ++i) b |= rs.ent[(size_t)i].col < 0 || rs.ent[(size_t)i].col >= n_cols;
        if (b) bad = true;
    });
    int64_t row = 0;
    for (const ScheduleRun& run : rs.runs) {
        if (run.row0 != row || run.row1 <= run.row0 || run.cls < 0 || run.cls >= kLengthClasses) return false;
        row = run.row1;
    }
    if (row != n) return false;
    pool.run((int64_t)rs.runs.size(), 8, [&](int64_t k0, int64_t k1, int) {
        bool b = false;
        for (int64_t k = k0; k < k1; ++k) {
            const ScheduleRun& run = rs.runs[(size_t)k];
            const int64_t cap = run.cls == 0 ? kSplitThreshold : (int64_t)(4 << (kLengthClasses - 1 - run.cls));
            const int64_t cap_chunks = (cap + kChunkEntries - 1) / kChunkEntries;
            for (int64_t i = run.row0; i < run.row1; ++i) b |= rs.rec[(size_t)i].chunk1 - rs.rec[(size_t)i].chunk0 > cap_chunks;
        }
        if (b) bad = true;
    });
    if (bad) return false;
    if (rs.long_part_ptr.size() != rs.long_row.size() + 1) return false;
    for (size_t i = 0; i < rs.long_row.size(); ++i)
        if (rs.long_row[i] < 0 || rs.long_row[i] >= n_out || rs.long_part_ptr[i] >= rs.long_part_ptr[i + 1] ||
            rs.long_part_ptr[i + 1] > (int32_t)np) return false;
    if (!rs.long_part_ptr.empty() && rs.long_part_ptr.back() != (int32_t)np) return false;
    return true;
}

// lane groups per row (log2) for the rows of stored class cls when a gathered row takes 2^lpr_log2 lanes
int groups_log2(int cls, int lpr_log2) {
    const int g_max = 6 - lpr_log2;
    if (cls == 0) return g_max;
    int g = 0;
    while (g < g_max && (kChunkEntries << g) < (4 << (kLengthClasses - 1 - cls))) ++g;
    return g;
}

}  // namespace

int64_t count_blocks(const RowSchedule& rs, int lpr_log2) {
    int64_t n = (rs.n_parts() + 3) / 4;                 // a part takes a whole wavefront, four per workgroup
    for (const ScheduleRun& run : rs.runs) {
        const int64_t per = 4LL << (6 - lpr_log2 - groups_log2(run.cls, lpr_log2));
        n += (run.row1 - run.row0 + per - 1) / per;
    }
    return n;
}

void build_block_table(const RowSchedule& rs, int lpr_log2, BlockTable& out) {
    const int64_t n_rows = rs.n_rows(), n_parts = rs.n_parts();
    const int g_max = 6 - lpr_log2;
    auto chunks = [&](int64_t i) { return (int64_t)(rs.rec[(size_t)i].chunk1 - rs.rec[(size_t)i].chunk0); };
    auto trips_for = [](int64_t longest_chunks, int g) { return (int32_t)std::max<int64_t>(1, (longest_chunks + (1LL << g) - 1) >> g); };
    auto block_of = [&](int64_t r, int64_t r1, int g, double& cost) {
        int64_t longest = 0, total = 0;
        for (int64_t i = r; i < r1; ++i) { longest = std::max(longest, chunks(i)); total += chunks(i); }
        cost = (double)(total * kChunkEntries) + 8.0 * (double)(r1 - r);     // its entries, plus a fixed share per row
        return BlockRows{(int32_t)r, (int32_t)r1, g, trips_for(longest, g)};
    };
    // the parts of split rows, dealt round-robin to the XCDs; they come first in every slice, so that the longest
    // pieces of work do not form the tail of a launch
    std::vector<BlockRows> parts[8];
    double part_cost[8] = {}, total = 0.0, c = 0.0;
    for (int64_t p = 0, b = 0; p < n_parts; p += 4, ++b) {
        parts[b & 7].push_back(block_of(n_rows + p, n_rows + std::min(p + 4, n_parts), g_max, c));
        part_cost[b & 7] += c;
        total += c;
    }
    // the scheduled rows in run order
    std::vector<BlockRows> rows;
    std::vector<double> cost;
    rows.reserve((size_t)count_blocks(rs, lpr_log2));
    cost.reserve(rows.capacity());
    for (const ScheduleRun& run : rs.runs) {
        const int g = groups_log2(run.cls, lpr_log2);
        const int64_t per = 4LL << (6 - lpr_log2 - g);
        for (int64_t r = run.row0; r < run.row1; r += per) {
            rows.push_back(block_of(r, std::min(r + per, run.row1), g, c));
            cost.push_back(c);
            total += c;
        }
    }
    // slice k: its parts, then consecutive row workgroups until it holds an eighth of the work
    out.blocks.clear();
    out.blocks.reserve(rows.size() + (size_t)((n_parts + 3) / 4));
    const int64_t nb = (int64_t)rows.size();
    int64_t b = 0;
    double done = 0.0;                    // work handed out so far, parts included
    for (int k = 0; k < 8; ++k) {
        out.xcd_start[k] = (int64_t)out.blocks.size();
        out.blocks.insert(out.blocks.end(), parts[k].begin(), parts[k].end());
        done += part_cost[k];
        const double want = total * (k + 1) / 8.0;
        while (b < nb && (k == 7 || done + 0.5 * cost[(size_t)b] < want)) {
            out.blocks.push_back(rows[(size_t)b]);
            done += cost[(size_t)b++];
        }
    }
    out.xcd_start[8] = (int64_t)out.blocks.size();
}

// What the kernels' row mapping relies on: every scheduled row and every part is in exactly one workgroup, no
// workgroup mixes the two or holds more rows than four wavefronts cover with its lane groups, its trip count covers
// its longest row, and the XCD slices tile the table.
bool block_table_ok(const RowSchedule& rs, int lpr_log2, const BlockTable& bt) {
    const int64_t n_rows = rs.n_rows(), n_parts = rs.n_parts();
    if (n_rows + n_parts > INT32_MAX) return false;
    int64_t next = 0;                              // the workgroups of scheduled rows come in row order
    std::vector<char> part_seen((size_t)n_parts, 0);
    int64_t parts_listed = 0;
    for (const BlockRows& b : bt.blocks) {
        if (b.row1 <= b.row0 || b.row0 < 0 || b.row1 > n_rows + n_parts || b.g < 0 || lpr_log2 + b.g > 6 || b.trips < 1) return false;
        if ((int64_t)b.row1 - b.row0 > (4LL << (6 - lpr_log2 - b.g))) return false;
        if (b.row0 < n_rows) {
            if (b.row0 != next || b.row1 > n_rows) return false;
            next = b.row1;
        } else {
            for (int64_t i = b.row0; i < b.row1; ++i) {
                if (part_seen[(size_t)(i - n_rows)]) return false;
                part_seen[(size_t)(i - n_rows)] = 1;
                ++parts_listed;
            }
        }
        for (int64_t i = b.row0; i < b.row1; ++i)
            if ((int64_t)(rs.rec[(size_t)i].chunk1 - rs.rec[(size_t)i].chunk0) > ((int64_t)b.trips << b.g)) return false;
    }
    if (next != n_rows || parts_listed != n_parts) return false;
    if (bt.xcd_start[0] != 0 || bt.xcd_start[8] != (int64_t)bt.blocks.size()) return false;
    for (int k = 0; k < 8; ++k)
        if (bt.xcd_start[k] > bt.xcd_start[k + 1]) return false;
    return true;
}

void build_chunks(const HostGraph& g, int64_t rows, int64_t segs, std::vector<Chunk>& chunks, std::vector<int32_t>& unit_ptr) {
    chunks.clear();
    chunks.reserve((size_t)count_chunks(g, rows, segs));
    unit_ptr.assign(g.M + 1, 0);
    auto cut = [&](int32_t m, int32_t kind, int64_t begin, int64_t end, int64_t per) {
        for (int64_t b = begin; b < end; b += per) chunks.push_back({m, kind, (int32_t)b, (int32_t)std::min(b + per, end)});
    };
    for (int32_t m = 0; m < g.M; ++m) {
        cut(m, 0, g.comm_row_ptr[m], g.comm_row_ptr[m + 1], rows);
        if (segs > 0) cut(m, 1, g.segc_comm_ptr[m], g.segc_comm_ptr[m + 1], segs);
        unit_ptr[m + 1] = (int32_t)chunks.size();
    }
}

int64_t count_chunks(const HostGraph& g, int64_t rows, int64_t segs) {
    int64_t n = 0;
    for (int32_t m = 0; m < g.M; ++m) {
        n += (g.comm_row_ptr[m + 1] - g.comm_row_ptr[m] + rows - 1) / rows;
        if (segs > 0) n += (g.segc_comm_ptr[m + 1] - g.segc_comm_ptr[m] + segs - 1) / segs;
    }
    return n;
}

std::string build_host_graph(HostGraph& g, int64_t N, int64_t n_edges, const int32_t* src,
                             const int32_t* dst, int32_t M, const int32_t* comm) {
    if (N < 1 || N > INT32_MAX) return "N must be in [1, 2^31)";
    if (M < 1) return "M must be positive";
    if (n_edges < 0) return "n_edges must be non-negative";
    if (n_edges > 0 && (!src || !dst)) return "src/dst are null";
    g = HostGraph();
    g.N = N;
    g.M = M;
    HostPool pool(4 * n_edges + 8 * N);
    std::atomic<bool> bad{false};
    pool.run(n_edges, 65536, [&](int64_t lo, int64_t hi, int) {
        bool b = false;
        for (int64_t e = lo; e < hi; ++e) b |= src[e] < 0 || src[e] >= N || dst[e] < 0 || dst[e] >= N;
        if (b) bad = true;
    });
    if (bad) return "edge endpoint out of range";
    const int64_t chunk = (N + M - 1) / M;
    if (comm)
        pool.run(N, 65536, [&](int64_t lo, int64_t hi, int) {
            bool b = false;
            for (int64_t i = lo; i < hi; ++i) b |= comm[i] < 0 || comm[i] >= M;
            if (b) bad = true;
        });
    if (bad) return "community id out of range";

    // stable counting sort by community: internal numbering
    g.perm.resize((size_t)N);
    g.inv_perm.resize((size_t)N);
    g.row_comm.resize((size_t)N);
    auto comm_of = [&](int64_t i) { return comm ? comm[i] : (int32_t)(i / chunk); };
    stable_counting_sort(pool, N, M, g.comm_row_ptr, [&](int64_t i) { return (int64_t)comm_of(i); },
                         [&](int64_t i, int64_t r) {
                             g.perm[(size_t)r] = (int32_t)i;
                             g.inv_perm[(size_t)i] = (int32_t)r;
                             g.row_comm[(size_t)r] = comm_of(i);
                         });

    for (int32_t m = 0; m < M; ++m) {
        const double n = (double)(g.comm_row_ptr[(size_t)m + 1] - g.comm_row_ptr[(size_t)m]);
        g.group_rows += n * n / (double)N;
    }

    // both orientations of every edge by row, sorted, repeats dropped
    HVec<int64_t> raw_ptr;
    HVec<int32_t> raw, deg;
    distinct_neighbours(pool, N, n_edges, src, dst, [&](int32_t x) { return g.inv_perm[(size_t)x]; }, raw_ptr, raw, deg);
    prefix_sum(pool, N, 0, g.row_ptr, [&](int64_t i) { return (int64_t)deg[(size_t)i] + 1; });      // + self loop
    g.nnz = g.row_ptr[(size_t)N];
    g.E = (g.nnz - N) / 2;
    g.col.resize((size_t)g.nnz);
    g.val.resize((size_t)g.nnz);
    HVec<int32_t> seg_cnt((size_t)N);
    std::atomic<int64_t> n_halo{0};
    pool.run(N, 1024, [&](int64_t lo, int64_t hi, int) {
        int64_t n_h = 0;
        for (int64_t i = lo; i < hi; ++i) {
            const int32_t* b = raw.data() + raw_ptr[(size_t)i];
            const int32_t own = g.row_comm[(size_t)i], d = deg[(size_t)i];
            int64_t o = g.row_ptr[(size_t)i];
            const double di = (double)(d + 1);
            int32_t prev = -1, segs = 0;
            bool halo = false, self_done = false;
            auto put = [&](int32_t j) {
                const double dj = (double)(deg[(size_t)j] + 1);
                g.col[(size_t)o] = j;
                g.val[(size_t)o++] = (float)(1.0 / std::sqrt(di * dj));
                const int32_t cc = g.row_comm[(size_t)j];
                if (cc != prev) { ++segs; prev = cc; }
                halo |= cc != own;
            };
            for (int32_t k = 0; k < d; ++k) {
                if (!self_done && b[k] > i) { put((int32_t)i); self_done = true; }
                put(b[k]);
            }
            if (!self_done) put((int32_t)i);
            seg_cnt[(size_t)i] = segs;
            n_h += halo;
        }
        n_halo += n_h;
    });
    g.n_halo_rows = n_halo;
    HVec<int32_t>().swap(raw);
    HVec<int64_t>().swap(raw_ptr);

    // segments in (row, community) order
    g.neighbour.assign((size_t)M * M, 0);
    prefix_sum(pool, N, 0, g.row_seg_ptr, [&](int64_t i) { return (int64_t)seg_cnt[(size_t)i]; });
    g.n_seg = g.row_seg_ptr[(size_t)N];
    if (g.n_seg > INT32_MAX) return "too many (row, community) segments";
    g.seg_ptr.resize((size_t)g.n_seg + 1);
    g.seg_row.resize((size_t)g.n_seg);
    g.seg_comm.resize((size_t)g.n_seg);
    pool.run(N, 1024, [&](int64_t lo, int64_t hi, int) {
        for (int64_t i = lo; i < hi; ++i) {
            const int32_t own = g.row_comm[(size_t)i];
            int32_t prev = -1;
            int64_t s = g.row_seg_ptr[(size_t)i] - 1;
            for (int64_t p = g.row_ptr[(size_t)i]; p < g.row_ptr[(size_t)i + 1]; ++p) {
                const int32_t cc = g.row_comm[(size_t)g.col[(size_t)p]];
                if (cc == prev) continue;
                ++s;
                g.seg_ptr[(size_t)s] = p;
                g.seg_row[(size_t)s] = (int32_t)i;
                g.seg_comm[(size_t)s] = cc;
                prev = cc;
                if (cc != own) {
                    uint8_t* nb = &g.neighbour[(size_t)own * M + cc];        // several threads may set it, all to 1
                    if (!__atomic_load_n(nb, __ATOMIC_RELAXED)) __atomic_store_n(nb, (uint8_t)1, __ATOMIC_RELAXED);
                }
            }
        }
    });
    g.seg_ptr[(size_t)g.n_seg] = g.nnz;

    // segments in (community, row) order: stable counting sort on the community
    g.segc_order.resize((size_t)g.n_seg);
    g.segc_row.resize((size_t)g.n_seg);
    g.seg_pos.resize((size_t)g.n_seg);
    stable_counting_sort(pool, g.n_seg, M, g.segc_comm_ptr, [&](int64_t s) { return (int64_t)g.seg_comm[(size_t)s]; },
                         [&](int64_t s, int64_t j) {
                             g.segc_order[(size_t)j] = s;
                             g.segc_row[(size_t)j] = g.seg_row[(size_t)s];
                             g.seg_pos[(size_t)s] = (int32_t)j;
                         });

    make_schedule(pool, g.row_sched, N, [&](int64_t r) { return g.row_ptr[(size_t)r]; }, [&](int64_t r) { return g.row_ptr[(size_t)r + 1]; },
                  [](int64_t r) { return (int32_t)r; }, [&](int64_t r) { return g.row_comm[(size_t)r]; }, M, g.col.data(), g.val.data());
    {
        // by length: key 0 = one entry (scaled copies of a row), key 1 = several (aggregated like rows), both in the
        // (community, row) order
        HVec<int64_t> start;
        auto len_of = [&](int64_t j) {
            const int64_t s = g.segc_order[(size_t)j];
            return g.seg_ptr[(size_t)s + 1] - g.seg_ptr[(size_t)s];
        };
        HVec<int32_t> by_len((size_t)g.n_seg);
        stable_counting_sort(pool, g.n_seg, 2, start, [&](int64_t j) { return (int64_t)(len_of(j) > 1); },
                             [&](int64_t j, int64_t at) { by_len[(size_t)at] = (int32_t)j; });
        const int64_t n1 = start[1];
        g.seg1_pos.resize((size_t)n1);
        g.seg1_col.resize((size_t)n1);
        g.seg1_val.resize((size_t)n1);
        pool.run(n1, 16384, [&](int64_t lo, int64_t hi, int) {
            for (int64_t k = lo; k < hi; ++k) {
                const int32_t j = by_len[(size_t)k];
                const int64_t p = g.seg_ptr[(size_t)g.segc_order[(size_t)j]];
                g.seg1_pos[(size_t)k] = j;
                g.seg1_col[(size_t)k] = g.col[(size_t)p];
                g.seg1_val[(size_t)k] = g.val[(size_t)p];
            }
        });
        const int32_t* m = by_len.data() + n1;
        auto seg_of = [&](int64_t r) { return (size_t)g.segc_order[(size_t)m[r]]; };
        make_schedule(pool, g.seg_sched, g.n_seg - n1, [&](int64_t r) { return g.seg_ptr[seg_of(r)]; },
                      [&](int64_t r) { return g.seg_ptr[seg_of(r) + 1]; }, [&](int64_t r) { return m[r]; },
                      [&](int64_t r) { return g.seg_comm[seg_of(r)]; }, M, g.col.data(), g.val.data());
    }

    if (!schedule_ok(pool, g.row_sched, N, N) || !schedule_ok(pool, g.seg_sched, g.n_seg, N)) return "internal error: row schedule";
    pool.run(14, 1, [&](int64_t t0, int64_t t1, int) {
        for (int64_t t = t0; t < t1; ++t) {
            const RowSchedule& rs = t < 7 ? g.row_sched : g.seg_sched;
            const int l = (int)(t % 7);
            BlockTable& bt = t < 7 ? g.row_tables[l] : g.seg_tables[l];
            build_block_table(rs, l, bt);
            if (!block_table_ok(rs, l, bt)) bad = true;
        }
    });
    if (bad) return "internal error: workgroup table of the aggregation";
    return "";
}

}  // namespace cadmm
