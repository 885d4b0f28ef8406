// Host check of schedule_part (csrc/cx_schedule.hpp): a segment's rows mixed in place by parts, one after the other in
// several orders, each part reading its two rows ahead of all stores, against the averages taken from a copy.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "cx_schedule.hpp"

struct Alone {
    void sync() const {}
    void add(int *p, int v) const { *p += v; }
};

int main()
{
    unsigned rng = 777u;
    auto next = [&rng]() { rng = rng * 1664525u + 1013904223u; return rng >> 8; };
    long cases = 0;
    for (int n = 1; n <= 1024; n = n < 40 ? n + 1 : 2 * n - 11) {
        for (int rep = 0; rep < 12; ++rep) {
            std::vector<int32_t> peers(n);
            for (int i = 0; i < n; ++i) peers[i] = i;
            if (rep % 4 < 2) {                             // a random permutation
                for (int i = n - 1; i > 0; --i) std::swap(peers[i], peers[next() % (i + 1)]);
            } else if (rep % 4 == 2) {                     // pairs
                for (int i = 0; i + 1 < n; i += 2) std::swap(peers[i], peers[i + 1]);
            }
            const int shift = rep % 4 == 3 && n > 1 ? 1 + static_cast<int>(next() % (n - 1)) : 0;
            std::vector<int> work(kScheduleWords(n));
            build_schedule(work.data(), n, 0, 1, peers.data(), 0, shift, Alone{});
            std::vector<double> x(n), want(n);
            for (double &v : x) v = next();
            for (int i = 0; i < n; ++i) want[i] = (x[i] + x[work[i]]) * 0.5;
            for (int parts = 1; parts <= 16; parts *= 2) {
                std::vector<SchedulePart> part(parts);
                std::vector<double> head(parts, -1), tail(parts, -1), y = x;
                std::vector<int> order(parts);
                int covered = 0;
                for (int q = 0; q < parts; ++q) {
                    part[q] = schedule_part(work.data(), n, q, parts, 0, 1, [](bool c) { return c ? 1u : 0u; });
                    if (part[q].begin != covered) return std::printf("gap: n %d parts %d\n", n, parts), 1;
                    covered = part[q].end;
                    order[q] = q;
                    if (part[q].begin < part[q].end) tail[q] = y[part[q].tail];
                    if (part[q].head >= 0) head[q] = y[part[q].head];
                }
                if (covered != n) return std::printf("rows left over: n %d parts %d\n", n, parts), 1;
                if (rep & 1) std::reverse(order.begin(), order.end());
                const int *sched = work.data() + n;
                for (int q : order) {                      // the walk of one part, as in walk()
                    const SchedulePart &p = part[q];
                    if (p.begin == p.end) continue;
                    double cur = y[sched[p.begin] & kRowMask], first = p.head >= 0 ? head[q] : cur;
                    for (int k = p.begin; k < p.end; ++k) {
                        const bool end = k + 1 == p.end, last = (sched[k] & kLastBit) != 0;
                        const double nx = end ? tail[q] : y[sched[k + 1] & kRowMask];
                        if (end) first = tail[q];
                        y[sched[k] & kRowMask] = (cur + (last ? first : nx)) * 0.5;
                        if (last) first = nx;
                        cur = nx;
                    }
                }
                if (y != want) return std::printf("wrong rows: n %d parts %d rep %d\n", n, parts, rep), 1;
                ++cases;
            }
        }
    }
    std::printf("ok (%ld cases)\n", cases);
    return 0;
}
