// Worker threads for the host-side graph work: one pool per call of the library, joined before the call returns.
#pragma once
#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <memory>
#include <mutex>
#include <thread>
#include <type_traits>
#include <utility>
#include <vector>

namespace cadmm {

// std::vector whose resize leaves new elements uninitialised: a large array is then first touched by the threads that
// fill it (the page faults of a serial zero fill are most of the cost of a big std::vector).
template <class T>
struct NoInitAlloc : std::allocator<T> {
    template <class U> struct rebind { using other = NoInitAlloc<U>; };
    NoInitAlloc() = default;
    template <class U> NoInitAlloc(const NoInitAlloc<U>&) noexcept {}
    template <class U> void construct(U* p) noexcept(std::is_nothrow_default_constructible<U>::value) { ::new (static_cast<void*>(p)) U; }
    template <class U, class... A> void construct(U* p, A&&... a) { ::new (static_cast<void*>(p)) U(std::forward<A>(a)...); }
};
template <class T> using HVec = std::vector<T, NoInitAlloc<T>>;

// Threads are started once per pool (a parallel region that starts its own costs more than most of the regions here) and
// spin briefly between regions before they sleep.  `work`: number of elementary steps of the whole call; a pool takes one
// thread per 16384 of them, at most 16 and at most what the machine has, so that a small call stays on its caller's thread.
// Where the system gives no more threads the pool works with those it has: the calls here are C entries, nothing may throw.
class HostPool {
public:
    explicit HostPool(int64_t work) {
        const int64_t hw = std::max(1u, std::thread::hardware_concurrency());
        const int n = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(hw, 16), work / 16384));
        try {
            threads_.reserve((size_t)n - 1);
            for (int w = 1; w < n; ++w) threads_.emplace_back([this, w] { loop(w); });
        } catch (const std::exception&) {   // std::system_error, std::bad_alloc
        }
    }
    ~HostPool() {
        {
            std::lock_guard<std::mutex> lock(m_);
            stop_ = true;
            epoch_.fetch_add(1, std::memory_order_release);
        }
        cv_.notify_all();
        for (auto& t : threads_) t.join();
    }
    HostPool(const HostPool&) = delete;
    HostPool& operator=(const HostPool&) = delete;

    int size() const { return (int)threads_.size() + 1; }

    // f(lo, hi, worker) over [0, n) in pieces of `grain`, handed out in order to whichever worker is free.
    template <class F>
    void run(int64_t n, int64_t grain, F f) {
        if (n <= 0) return;
        if (threads_.empty() || n <= grain) { f((int64_t)0, n, 0); return; }
        next_.store(0, std::memory_order_relaxed);
        n_ = n;
        grain_ = grain;
        call_ = [](void* ctx, int64_t lo, int64_t hi, int w) { (*static_cast<F*>(ctx))(lo, hi, w); };
        ctx_ = &f;
        busy_.store((int)threads_.size(), std::memory_order_relaxed);
        {
            std::lock_guard<std::mutex> lock(m_);
            epoch_.fetch_add(1, std::memory_order_release);
        }
        cv_.notify_all();
        work(0);
        for (int k = 0; busy_.load(std::memory_order_acquire) != 0; ++k)
            if (k > 256) std::this_thread::yield();
    }

    // f(block, lo, hi) for size() blocks of nearly equal length, for algorithms that need to know who owns what.
    template <class F>
    void blocks(int n_blocks, int64_t n, F f) {
        run(n_blocks, 1, [&](int64_t b0, int64_t b1, int) {
            for (int64_t b = b0; b < b1; ++b) f((int)b, n * b / n_blocks, n * (b + 1) / n_blocks);
        });
    }

private:
    void work(int w) {
        for (;;) {
            const int64_t lo = next_.fetch_add(grain_, std::memory_order_relaxed);
            if (lo >= n_) return;
            call_(ctx_, lo, std::min(n_, lo + grain_), w);
        }
    }
    void loop(int w) {
        uint64_t seen = 0;
        for (;;) {
            for (int k = 0; k < 2000 && epoch_.load(std::memory_order_acquire) == seen; ++k)
                if (k > 200) std::this_thread::yield();
            if (epoch_.load(std::memory_order_acquire) == seen) {
                std::unique_lock<std::mutex> lock(m_);
                cv_.wait(lock, [&] { return epoch_.load(std::memory_order_acquire) != seen; });
            }
            seen = epoch_.load(std::memory_order_acquire);
            if (stop_) return;
            work(w);
            busy_.fetch_sub(1, std::memory_order_release);
        }
    }

    std::vector<std::thread> threads_;
    std::mutex m_;
    std::condition_variable cv_;
    std::atomic<uint64_t> epoch_{0};
    std::atomic<int64_t> next_{0};
    std::atomic<int> busy_{0};
    int64_t n_ = 0, grain_ = 1;
    void (*call_)(void*, int64_t, int64_t, int) = nullptr;
    void* ctx_ = nullptr;
    bool stop_ = false;
};

// A stable counting sort cut into blocks of consecutive items: key(i) in [0, n_keys) for i < n (or -1: not listed);
// place(i, position) is called for every listed item, positions ordered by (key, i).  start [n_keys + 1] gets the first
// position of every key.
template <class Key, class Place>
void stable_counting_sort(HostPool& pool, int64_t n, int64_t n_keys, HVec<int64_t>& start, Key key, Place place) {
    // every block has a counter per key: as many blocks as keep those small against the items
    int nb = pool.size() == 1 ? 1 : 2 * pool.size();
    while (nb > 1 && n_keys * nb > n / 2) nb /= 2;
    std::vector<int64_t> count((size_t)(n_keys * nb), 0);
    pool.blocks(nb, n, [&](int b, int64_t lo, int64_t hi) {
        int64_t* c = count.data() + (size_t)b * n_keys;
        for (int64_t i = lo; i < hi; ++i) {
            const int64_t k = key(i);
            if (k >= 0) ++c[k];
        }
    });
    start.resize((size_t)n_keys + 1);
    int64_t at = 0;
    for (int64_t k = 0; k < n_keys; ++k) {
        start[(size_t)k] = at;
        for (int b = 0; b < nb; ++b) {
            int64_t& c = count[(size_t)b * n_keys + k];
            const int64_t here = c;
            c = at;
            at += here;
        }
    }
    start[(size_t)n_keys] = at;
    pool.blocks(nb, n, [&](int b, int64_t lo, int64_t hi) {
        int64_t* c = count.data() + (size_t)b * n_keys;
        for (int64_t i = lo; i < hi; ++i) {
            const int64_t k = key(i);
            if (k >= 0) place(i, c[k]++);
        }
    });
}

// out[i] = first + sum of len(j) over j < i for i <= n.
template <class Len>
void prefix_sum(HostPool& pool, int64_t n, int64_t first, HVec<int64_t>& out, Len len) {
    out.resize((size_t)n + 1);
    const int nb = pool.size();
    std::vector<int64_t> total((size_t)nb + 1, 0);
    pool.blocks(nb, n, [&](int b, int64_t lo, int64_t hi) {
        int64_t t = 0;
        for (int64_t i = lo; i < hi; ++i) t += len(i);
        total[(size_t)b + 1] = t;
    });
    total[0] = first;
    for (int b = 0; b < nb; ++b) total[(size_t)b + 1] += total[(size_t)b];
    pool.blocks(nb, n, [&](int b, int64_t lo, int64_t hi) {
        int64_t t = total[(size_t)b];
        for (int64_t i = lo; i < hi; ++i) { out[(size_t)i] = t; t += len(i); }
    });
    out[(size_t)n] = total[(size_t)nb];
}

// The undirected edges of a list as rows of neighbours: nb[start[i] .. start[i] + len[i]) = the distinct neighbours of row i,
// ascending; row(x) maps an endpoint to its row.  Self pairs are dropped; start[i + 1] - start[i] leaves room for repeats.
// Both orientations of the edges go into buckets of consecutive rows first (each thread into its own stretch of every
// bucket), then one thread sorts out a bucket in its cache: counters that several threads bump would bounce between cores
// (measured: two thirds of the time of the whole step).
template <class Row>
void distinct_neighbours(HostPool& pool, int64_t n_rows, int64_t n_edges, const int32_t* src, const int32_t* dst, Row row,
                         HVec<int64_t>& start, HVec<int32_t>& nb, HVec<int32_t>& len) {
    struct Pair { int32_t row, other; };
    int shift = 0;
    while ((n_rows >> shift) > 512) ++shift;
    const int64_t n_buckets = ((n_rows - 1) >> shift) + 1;
    const int n_blocks = pool.size();
    std::vector<int64_t> at((size_t)(n_blocks * n_buckets), 0);
    pool.blocks(n_blocks, n_edges, [&](int b, int64_t lo, int64_t hi) {
        int64_t* c = at.data() + (size_t)b * n_buckets;
        for (int64_t e = lo; e < hi; ++e)
            if (src[e] != dst[e]) { ++c[row(src[e]) >> shift]; ++c[row(dst[e]) >> shift]; }
    });
    std::vector<int64_t> bucket((size_t)n_buckets + 1);
    int64_t total = 0;
    for (int64_t k = 0; k < n_buckets; ++k) {
        bucket[(size_t)k] = total;
        for (int b = 0; b < n_blocks; ++b) {
            int64_t& c = at[(size_t)b * n_buckets + k];
            const int64_t here = c;
            c = total;
            total += here;
        }
    }
    bucket[(size_t)n_buckets] = total;
    HVec<Pair> pairs((size_t)total);
    pool.blocks(n_blocks, n_edges, [&](int b, int64_t lo, int64_t hi) {
        int64_t* c = at.data() + (size_t)b * n_buckets;
        for (int64_t e = lo; e < hi; ++e)
            if (src[e] != dst[e]) {
                const int32_t x = row(src[e]), y = row(dst[e]);
                pairs[(size_t)c[x >> shift]++] = {x, y};
                pairs[(size_t)c[y >> shift]++] = {y, x};
            }
    });
    start.resize((size_t)n_rows + 1);
    start[(size_t)n_rows] = total;
    nb.resize((size_t)total);
    len.resize((size_t)n_rows);
    pool.run(n_buckets, 1, [&](int64_t k0, int64_t k1, int) {
        for (int64_t k = k0; k < k1; ++k) {
            const int64_t r0 = k << shift, r1 = std::min(n_rows, (k + 1) << shift);
            std::fill(len.begin() + r0, len.begin() + r1, 0);
            for (int64_t p = bucket[(size_t)k]; p < bucket[(size_t)k + 1]; ++p) ++len[(size_t)pairs[(size_t)p].row];
            int64_t o = bucket[(size_t)k];
            for (int64_t r = r0; r < r1; ++r) { start[(size_t)r] = o; o += len[(size_t)r]; len[(size_t)r] = 0; }
            for (int64_t p = bucket[(size_t)k]; p < bucket[(size_t)k + 1]; ++p) {
                const Pair q = pairs[(size_t)p];
                nb[(size_t)(start[(size_t)q.row] + len[(size_t)q.row]++)] = q.other;
            }
            for (int64_t r = r0; r < r1; ++r) {
                int32_t* b = nb.data() + start[(size_t)r];
                int32_t* e = b + len[(size_t)r];
                std::sort(b, e);
                len[(size_t)r] = (int32_t)(std::unique(b, e) - b);
            }
        }
    });
}

}  // namespace cadmm
