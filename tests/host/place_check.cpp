// Host check of place_row and schedule_rows (csrc/cx_schedule.hpp): the row order and the schedule made with a thread for
// every row, run by that many real threads and compared with the peer table itself, whatever order the cycles come in.
#include <pthread.h>

#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "cx_schedule.hpp"

struct ThreadGroup {
    pthread_barrier_t *barrier;
    void sync() const { pthread_barrier_wait(barrier); }
    int add(int *p, int v) const { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
    void claim(int *p, int v) const { __atomic_store_n(p, v, __ATOMIC_RELAXED); }
};

// nullptr, or what is wrong with the schedule in `work`
static const char *wrong(const std::vector<int> &work, const std::vector<int> &as_table, int n)
{
    std::vector<int> indeg(n, 0), seen(n, 0);
    bool permutation = true;
    for (int v : as_table) {
        if (v < 0 || v >= n) permutation = false;
        else ++indeg[v];
    }
    for (int v : indeg) permutation = permutation && v == 1;
    for (int i = 0; i < n; ++i)
        if (work[i] != (permutation ? as_table[i] : i)) return "the table as used";
    int first = -1;
    for (int k = 0; k < n; ++k) {
        const int e = work[n + k], row = e & kRowMask;
        if (row >= n || seen[row]++) return "a row twice, or none";
        if (first < 0) first = row;
        const int next = (e & kLastBit) ? first : k + 1 < n ? work[n + k + 1] & kRowMask : -1;
        if (next != work[row]) return "not in cycle order";
        if (e & kLastBit) first = -1;
    }
    return first < 0 ? nullptr : "a cycle left open";
}

int main(int argc, char **argv)
{
    const int min_n = std::atoi(argv[1]), max_n = std::atoi(argv[2]), spare = std::atoi(argv[3]);   // threads beyond the rows
    unsigned rng = 4242u;
    auto next = [&rng]() { rng = rng * 1664525u + 1013904223u; return rng >> 8; };
    long cases = 0;
    for (int n = min_n; n <= max_n; n = n < 20 ? n + 1 : n < 1024 && 2 * n - 7 > 1024 ? 1024 : 2 * n - 7) {
        for (int rep = 0; rep < 7; ++rep) {
            const int S = 2, seg = rep & 1, nthreads = n + spare > 2 ? n + spare : 2;
            std::vector<int32_t> peers(static_cast<size_t>(S) * n, 0);
            int32_t *t = peers.data() + static_cast<size_t>(seg) * n;
            for (int i = 0; i < n; ++i) t[i] = i;
            int shift = 0;
            if (rep < 3 || rep == 5)                          // a permutation; one of them with an entry out of range
                for (int i = n - 1; i > 0; --i) std::swap(t[i], t[next() % (i + 1)]);
            if (rep == 3) for (int i = 0; i < n; ++i) t[i] = static_cast<int32_t>(next() % n);       // rows twice or never
            if (rep == 4) shift = n > 1 ? 1 + static_cast<int>(next() % (n - 1)) : 0;
            if (rep == 5) t[next() % n] = next() % 2 ? n + 3 : -1;
            const bool table = rep != 4 && rep != 6;          // 6: no table at all
            std::vector<int> as_table(n), partner(n, -1), work(kScheduleWords(n), -77);
            for (int i = 0; i < n; ++i) as_table[i] = shift > 0 ? ((i - shift) % n + n) % n : table ? t[i] : i;
            pthread_barrier_t barrier;
            pthread_barrier_init(&barrier, nullptr, nthreads);
            std::vector<std::thread> pool;
            for (int tid = 0; tid < nthreads; ++tid)
                pool.emplace_back([&, tid]() {
                    const ThreadGroup group{&barrier};
                    const int32_t *source = table ? peers.data() : nullptr;
                    const Place p = place_row(work.data(), n, tid, source, seg, shift, group);
                    if (tid < n) partner[tid] = p.partner;
                    group.sync();
                    schedule_rows(work.data(), n, tid, nthreads, source, seg, shift, group);
                });
            for (auto &th : pool) th.join();
            pthread_barrier_destroy(&barrier);
            const char *fault = wrong(work, as_table, n);
            for (int i = 0; i < n && !fault; ++i)
                if (partner[i] != (as_table[i] >= 0 && as_table[i] < n ? as_table[i] : i)) fault = "partner";
            if (fault) {
                std::printf("n=%d rep=%d: %s\n", n, rep, fault);
                return 1;
            }
            ++cases;
        }
    }
    std::printf("ok %ld tables\n", cases);
    return 0;
}
