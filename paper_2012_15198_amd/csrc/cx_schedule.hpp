// Cycle schedule of a peer table: the order in which the mixing kernels visit the rows.
// Plain C++ with no device intrinsics, so that the same text runs inside the kernels (the
// including file defines CX_SCHED_FN as __device__ __forceinline__) and in a host test.
#ifndef CX_SCHEDULE_HPP
#define CX_SCHEDULE_HPP
#include <cstddef>
#include <cstdint>

#ifndef CX_SCHED_FN
#define CX_SCHED_FN inline
#endif

constexpr int kLastBit = 1 << 30;          // schedule entry flag: last row of its cycle
constexpr int kRowMask = kLastBit - 1;

// ---------------------------------------------------------------------------------
// Cycle schedule of one segment, built in LDS by a group of threads (one wavefront in its
// private region, or a whole workgroup): `work` holds kScheduleWords(n) ints,
//   work[0..n)   : the table as used (a table that is not a permutation -> the identity)
//   work[n..2n)  : the schedule: rows in cycle order, cycles by ascending smallest row, each
//                  starting at its smallest row; kLastBit marks the last row of a cycle
// Source of the table: shift > 0 -> row i receives from (i - shift) mod n;
// peers == null -> identity; else peers[seg*n + i].
// No serial walk: every row finds the smallest row of its cycle and its distance to it by
// pointer doubling (log2 n rounds over words that pack successor, minimum and distance), a
// prefix sum over the cycle lengths places the cycles, and every row writes its own entry.
// `group.sync()` orders the group's traffic on `work`; `group.add(p, v)` is an atomic *p += v.
// ---------------------------------------------------------------------------------
constexpr int kRowBits = 10;                          // CX_MAX_ROWS == 1 << kRowBits
constexpr int kRowField = (1 << kRowBits) - 1;
constexpr size_t kScheduleWords(int n) { return 4 * static_cast<size_t>(n) + 4; }

template <class Group>
CX_SCHED_FN void build_schedule(int *work, int n, int tid, int nthreads, const int32_t *peers, int seg,
                                int shift, Group group)
{
    int *tab = work, *sched = work + n, *a = work + 2 * n, *b = work + 3 * n;
    int *bad = work + 4 * n;
    if (tid == 0) *bad = 0;
    bool ok = true;
    for (int i = tid; i < n; i += nthreads) {
        int v = i;
        if (shift > 0) v = i >= shift ? i - shift : i - shift + n;
        else if (peers) v = peers[static_cast<int64_t>(seg) * n + i];
        if (static_cast<unsigned>(v) >= static_cast<unsigned>(n)) { ok = false; v = i; }
        tab[i] = v;
        sched[i] = 0;
    }
    group.sync();
    for (int i = tid; i < n; i += nthreads) group.add(&sched[tab[i]], 1);   // in-degree
    group.sync();
    for (int i = tid; i < n; i += nthreads) ok = ok && (sched[i] == 1);
    if (!ok) group.add(bad, 1);
    group.sync();
    const bool valid = *bad == 0;
    // word i: successor after `span` steps | smallest row among the next `span` rows of the
    // cycle, i included | distance from i to that row
    for (int i = tid; i < n; i += nthreads) {
        if (!valid) tab[i] = i;
        a[i] = (valid ? tab[i] : i) | (i << kRowBits);
    }
    group.sync();
    for (int span = 1; span < n; span <<= 1) {
        for (int i = tid; i < n; i += nthreads) {
            const int w = a[i];
            const int wj = a[w & kRowField];
            int mn = (w >> kRowBits) & kRowField, d = w >> (2 * kRowBits);
            const int mj = (wj >> kRowBits) & kRowField;
            if (mj < mn) { mn = mj; d = span + (wj >> (2 * kRowBits)); }
            b[i] = (wj & kRowField) | (mn << kRowBits) | (d << (2 * kRowBits));
        }
        group.sync();
        int *t = a; a = b; b = t;
    }
    // a[i] now names the smallest row of i's cycle and i's distance to it.  Cycle lengths at
    // the smallest rows, then an inclusive prefix sum that ends in `b`.
    int rounds = 0;
    for (int span = 1; span < n; span <<= 1) ++rounds;
    int *p = (rounds & 1) ? sched : b, *q = (rounds & 1) ? b : sched;
    for (int i = tid; i < n; i += nthreads) {
        const bool leader = ((a[i] >> kRowBits) & kRowField) == i;
        p[i] = leader ? (a[tab[i]] >> (2 * kRowBits)) + 1 : 0;
    }
    group.sync();
    for (int span = 1; span < n; span <<= 1) {
        for (int i = tid; i < n; i += nthreads) q[i] = p[i] + (i >= span ? p[i - span] : 0);
        group.sync();
        int *t = p; p = q; q = t;
    }
    // p == b: cycles end at p[smallest row]; place every row
    for (int i = tid; i < n; i += nthreads) {
        const int w = a[i];
        const int mn = (w >> kRowBits) & kRowField, d = w >> (2 * kRowBits);
        const int len = (a[tab[mn]] >> (2 * kRowBits)) + 1;
        const int pos = d == 0 ? 0 : len - d;
        sched[p[mn] - len + pos] = i | (pos == len - 1 ? kLastBit : 0);
    }
    group.sync();
}

// ---------------------------------------------------------------------------------
// The row that gossiping row `row` averages with in segment s (Algorithm 1: receive_from):
// the fixed shift of the push-sum schedule, or the peer table's entry; an entry outside
// [0, n) means the row itself.
CX_SCHED_FN int partner_of(const int32_t *__restrict__ peers, int shift, int n, int s, int row)
{
    int peer = row;
    if (shift > 0) peer = row >= shift ? row - shift : row - shift + n;
    else if (peers) peer = peers[static_cast<int64_t>(s) * n + row];
    if (static_cast<unsigned>(peer) >= static_cast<unsigned>(n)) peer = row;
    return peer;
}

// The place of row `i` in the cycle order of segment s, the cycles in any order, for a group with a thread for every row
// (threads without one come along for the syncs).  `work` holds kScheduleWords(n) ints, of which the first n stay as they are.
//
// build_schedule orders the cycles as well and serves fewer threads than rows: with a thread for each row the row's own word
// stays in a register, one write and one read tell whether the table is a permutation, and an atomic places a cycle where
// a prefix sum did: 12 syncs instead of 24 at 512 rows.  Beside more than 64 rows several wavefronts race for the places, so the
// workgroups of one launch may walk the cycles in different orders; that costs nothing (in place, 28 shapes of 65 to 1,000 rows and
// 100,003 to 25,557,032 columns 0.97 to 1.001 of the time with build_schedule, whose order is one for all).  `group.add` returns what was there, `group.claim(p, v)` is *p = v
// where several threads may write the same word.
struct Place {
    int partner;                           // as the table has it, entries outside [0, n) the row itself
    int at;                                // a table that is not a permutation: every row a cycle of its own
    bool last, permutation;                // last of its cycle
};
template <class Group>
CX_SCHED_FN Place place_row(int *work, int n, int i, const int32_t *__restrict__ peers, int s, int shift, Group group)
{
    int *claimed = work + n, *a = work + 2 * n, *b = work + 3 * n, *state = work + 4 * n;   // state: not a permutation, rows placed
    const bool mine = i < n;
    if (i < 2) state[i] = 0;
    int to = i, w = 0;
    bool in_range = true;
    if (mine) {
        to = partner_of(peers, shift, n, s, i);
        in_range = shift > 0 || !peers || peers[static_cast<int64_t>(s) * n + i] == to;
        group.claim(&claimed[to], i);             // one of a row's claimants stays
        // successor after `span` steps | smallest row among the next `span` rows of the cycle, i included | distance to it
        w = to | (i << kRowBits);
        a[i] = w;
    }
    group.sync();
    if (mine && !(in_range && claimed[to] == i)) group.add(&state[0], 1);
    group.sync();
    if (state[0] != 0) return Place{to, i, true, false};   // the group's threads together
    for (int span = 1; span < n; span <<= 1) {
        if (mine) {
            const int ahead = a[w & kRowField];
            int least = (w >> kRowBits) & kRowField, d = w >> (2 * kRowBits);
            const int other = (ahead >> kRowBits) & kRowField;
            if (other < least) { least = other; d = span + (ahead >> (2 * kRowBits)); }
            w = (ahead & kRowField) | (least << kRowBits) | (d << (2 * kRowBits));
            b[i] = w;
        }
        group.sync();
        int *t = a; a = b; b = t;
    }
    const int least = (w >> kRowBits) & kRowField, d = w >> (2 * kRowBits);
    if (mine && least == i) {                              // its successor is as far from it as the cycle is long, less one
        const int length = (a[to] >> (2 * kRowBits)) + 1;
        b[i] = group.add(&state[1], length) | (length << kRowBits);
    }
    group.sync();
    const int cycle = mine ? b[least] : 0, first = cycle & kRowField, length = cycle >> kRowBits;
    return Place{to, d == 0 ? first : first + length - d, to == least, true};
}

// The schedule of segment s in `work`, as build_schedule lays it out: by place_row where the group has a thread for every
// row.  In place, us, build_schedule / this: fp32 gossip on 512 x 3,001 25.5 / 23.3, 256 x 30,011 21.6 / 20.0, 12 x 400,007
// 11.5 / 10.6, 300 x 100,003 56.8 / 54.8; bf16 gossip on 355 x 50,356 27.4 / 25.4, on 32 x 25,557,032 596 / 591.
// Up to 64 rows of up to 6 GB (240 drawn calls of all operators in place) 0.990 of the time, 0.90 to 1.04; long fp32 rows of groups lie on
// both sides: mean of groups of 4 on 40 x 9,000,001 542 / 550, of 6 on 24 x 6,544,953 239 / 243, gradient step of groups of 2 0.93 to 1.04.
template <class Group>
CX_SCHED_FN void schedule_rows(int *work, int n, int tid, int nthreads, const int32_t *__restrict__ peers, int s,
                                              int shift, Group group)
{
    if (n > nthreads) {
        build_schedule(work, n, tid, nthreads, peers, s, shift, group);
        return;
    }
    const Place p = place_row(work, n, tid, peers, s, shift, group);
    if (tid < n) {
        work[tid] = p.permutation ? p.partner : tid;
        work[n + p.at] = tid | (p.last ? kLastBit : 0);
    }
    group.sync();
}

// ---------------------------------------------------------------------------------
// A schedule walked in parts, each by a wavefront of its own and all of them at once: part q of Q takes the positions
// [n*q/Q, n*(q+1)/Q).  In place, a part's walk needs two rows that another part overwrites, and reads them before any
// part stores:
//   tail  the row that the last position averages with (the next part's first row, or where a cycle closes there its
//         first row, which may lie in an earlier part);
//   head  the first row of the cycle that was open when the part began, where that cycle closes inside the part before
//         the last position; -1 otherwise.  Every cycle that opens inside the part finds its first row in registers.
// `ballot(c)` collects one bit a lane of the `lanes` that call together.
// ---------------------------------------------------------------------------------
struct SchedulePart {
    int begin, end, head, tail;
};

template <class Ballot>
CX_SCHED_FN SchedulePart schedule_part(const int *work, int n, int part, int parts, int lane, int lanes, Ballot ballot)
{
    const int *tab = work, *sched = work + n;
    SchedulePart p{n * part / parts, n * (part + 1) / parts, -1, -1};
    if (p.begin == p.end) return p;
    p.tail = tab[sched[p.end - 1] & kRowMask];
    if (p.begin == 0 || (sched[p.begin - 1] & kLastBit)) return p;
    for (int k = p.begin; k < p.end - 1; k += lanes) {
        const uint64_t closes = ballot(k + lane < p.end - 1 && (sched[k + lane] & kLastBit));
        if (closes) {
            p.head = tab[sched[k + __builtin_ctzll(closes)] & kRowMask];
            break;
        }
    }
    return p;
}

#endif  // CX_SCHEDULE_HPP
