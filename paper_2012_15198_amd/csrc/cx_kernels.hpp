// Device half of the gossip-mixing library for gfx950 (MI355X): the mixing kernels behind
// cx_gossip_mix / cx_hier_mix / cx_pushsum_mix / cx_sgd_fused_mix / cx_hier_sgd_fused_mix and
// their 16-bit variants.  Internal header; the pieces: cx_tile.hpp (slices, tiles, fp32 row
// accesses), cx_ops.hpp and cx_ops16.hpp (the row operators), this file (the three mixing kernels and the
// two that write the row order), cx_launch.hpp (launch shapes, the row-order table's slots, argument checks;
// the header each cx_api_*.hip includes).  Everything has internal linkage.
//
// Mixing is independent per column and every element has to be read once and written once
// (8 B per worker-parameter; 20 B with the fused optimizer), so the whole path is bound by
// HBM bandwidth.  A lane always handles 16-byte column slices (4 fp32 or 8 bfloat16), a
// wavefront 1 KB of contiguous columns per memory instruction.  Three kernels serve the same
// arithmetic:
//
//  gather_kernel (output buffer != input buffer) -- the fast one.
//   * One short-lived workgroup per (gossiping row, column chunk): it loads the row's chunk
//     and its partner's chunk, averages, stores to the other buffer.  Every chunk is
//     fetched twice from L2 but once from HBM: blocks are ordered so that both fetches meet
//     in the L2 of one XCD (block b runs on XCD b mod 8; an XCD walks a cluster of
//     neighbouring chunks row after row; rows follow the cycles of the peer permutation,
//     so a block's partner is the next block's own row).
//   * Rows that begin inside a line of 128 bytes: each row's tiles start on the row's own lines (OnLines), for the operators
//     that gain by it.
//   * Long contiguous row visits per XCD keep the DRAM row buffers busy, which a kernel
//     whose waves each wander over all rows cannot do as well.
//   * segment_order_kernel, a few microseconds ahead of it, derives the row order from the
//     device-resident peer table into library-owned device memory (no allocation): one word
//     per (segment, position) with the row and its partner, and one per tile with its segment and
//     a "one segment covers this tile" bit, so almost every workgroup starts its loads after two
//     scalar loads; or order_kernel, where clusters are many beside the segments' edges: one word
//     per (cluster, position) with the row, its partner and that bit, and one scalar load.
//     Workgroups are many and small (one slice per lane for plain gossip): their count of
//     instructions, not only their bytes, decides the rate.
//
//  mix_kernel (in place capable) -- the column-owner cycle walk.
//   * A wavefront owns a tile of 64*U slices (256*U fp32 columns) and visits every row of it.  The peer table
//     of a segment is a permutation, so the rows split into cycles i -> peers[i] -> ...
//     Walking a cycle, the lane keeps the current and the next row's slice in registers,
//     writes (cur + next) * 0.5f to the current row and moves on; the cycle's first slice
//     is kept for its last row.  A row is overwritten only after its two readers have it
//     in registers, so x_out may be x_in.  Loads run D rows ahead of the stores.
//   * The cycle order of a segment is built per wavefront (or once per workgroup in the
//     lock-step variant) in LDS from the peer table; a table that is not a permutation is
//     replaced by the identity, so no row index can leave [0, n).
//
//  parts_kernel (in place, few tiles) -- the same walk, with the rows of a tile split over the wavefronts of a workgroup.
//
//  All: tiles wholly inside one segment take the 16-byte vector path.  In the at most S tiles of a row (S+1 with tiles on the row's
//  own lines) that a segment boundary or an end of the row crosses, every piece between two boundaries loads the slices it
//  meets and stores under a mask of elements: piece after piece by the tile's wavefront in gather_kernel, one
//  wavefront for each piece in mix_kernel.  Columns [P, ld) are neither read nor written.  Row operators
//  (MeanOp / FusedOp / HierFusedOp / PushOp / Row16Op ...) say what loading and storing a "gossiping row" means:
//  the mean of a group of G rows summed in fp64, the momentum-SGD update applied on the way in (to the row or
//  to a group leader fed with the group's mean gradient), the push-sum de-biasing, or the
//  unpacking and rounding of 16-bit rows (bfloat16, binary16).  Each operator also names its
//  measured launch shapes (kGather, kWalk).
#ifndef CX_KERNELS_HPP
#define CX_KERNELS_HPP
#include "cx_ops.hpp"
#include "cx_ops16.hpp"

#pragma clang fp contract(off)

namespace {

// The two groups that build schedules: one wavefront in its private LDS region, or a workgroup.
struct WaveSync {
    __device__ __forceinline__ void sync() const { wave_sync(); }
    __device__ __forceinline__ int add(int *p, int v) const { return atomicAdd(p, v); }
    __device__ __forceinline__ void claim(int *p, int v) const { *p = v; }
};
struct BlockSync {
    __device__ __forceinline__ void sync() const { __syncthreads(); }
    __device__ __forceinline__ int add(int *p, int v) const { return atomicAdd(p, v); }
    __device__ __forceinline__ void claim(int *p, int v) const { *p = v; }
};

// One lane's walk over all cycles of the schedule.  Rows are fetched in schedule order, each exactly
// once, into a ring of D register slots (statically indexed: the step loop is unrolled by D), up to D
// rows ahead of the step that averages and stores.
//
// The steps run in two loops.  As long as every step of a turn has a row to fetch, a turn holds no branch
// around a load, so the compiler knows how many accesses follow the one it waits for.  What it makes of that
// depends on finish() (waits read from the assembly): where finish() consumes the slot by arithmetic and a store
// (FusedOp with one slice, HierFusedOp, Fused16Op), every step waits for its own row and the others stay in
// flight; where finish() only copies, widens or sums the slot (gossip, group means, push-sum, 16-bit rows), the
// compiler gathers that at the head of the turn, or issues the first turn's loads in another order, whose last row then
// bounds the wait of every turn: it waits there for all rows in flight and the last stores, and the ring is a batch of D rows
// a turn, not a pipeline.  The batch is the better of the two: with the order pinned (sched_barrier between the loads and
// steps, the first turn peeled) every step waits for its own row only, and in place, batch / pipeline, us, bf16 gossip on
// 32 x 25,557,032 takes 597 / 602, on 512 x 1,000,003 514 / 558, the binary16 mean of groups of 4 on 64 x 11,689,511 594 / 638,
// fp32 gossip and steps as long either way: DRAM serves reads and writes that come in turns better than mixed ones.  (A branch around each load made it wait for all but the last
// access of the wavefront at every step: gossip on 256 x 8,303 fp32, in place, 8 segments: 230 -> 86 us together
// with the boundary pieces below; fused step 256 x 300,007: 806 -> 573 us.)  The schedule's words are read from
// LDS one step ahead and kept until their row arrives.  The last turns, up to 2 * D steps, decide step by step;
// walks of at most 2 * D rows consist of them.
struct NoEnds {
    static constexpr bool kPart = false, kAhead = false;
    __device__ __forceinline__ bool has_head() const { return false; }
};
template <class Op, int U, int D, TileMode MODE, bool NT, class Ends = NoEnds, bool SYNC = false>
__device__ __forceinline__ void walk(const Op &op, const int *sched, int n, bool skip_mix,
                                     int64_t off, const unsigned (&mask)[U], const Ends &ends = Ends{})
{
    constexpr bool PART = Ends::kPart;
    using WorkT = typename Op::template Work<U>;
    typename Op::template Raw<U> slot[D];
    WorkT cur, first, tail;
    int e = 0, base = 0;
    if constexpr (PART && Ends::kAhead) ends.template load<MODE, NT>(mask, first, tail);
    // Without the steady loop: the mean of groups of 16, whose registers would spill, and the shape that few long rows of
    // plain gossip take (MeanOp::walk).
    constexpr bool kSteady = !std::is_same_v<Op, MeanOp<16>> && !(std::is_same_v<Op, MeanOp<1>> && U == 1 && D == 2);
    auto step = [&](const WorkT &nx, int e1) {            // average row k, open the next cycle where one closes
        const bool last = (e & kLastBit) != 0;
        WorkT out;
#pragma unroll
        for (int u = 0; u < WorkT::kN; ++u) out.v[u] = average(cur.v[u], last ? first.v[u] : nx.v[u]);
        op.template store<U, MODE, NT>(e & kRowMask, off, mask, out);
        if (last) first = nx;
        cur = nx;
        e = e1;
    };
    if (kSteady && n > 2 * D) {
        int word[D];                                      // schedule words of the rows in flight
#pragma unroll
        for (int j = 0; j < D; ++j) {
            word[j] = uniform(sched[j]);
            op.template issue<U, MODE, NT>(word[j] & kRowMask, off, mask, slot[j]);
        }
        int ahead = sched[D];
        if constexpr (PART && !Ends::kAhead) ends.template load<MODE, NT>(mask, first, tail);
        e = word[0];
        op.template finish<U, MODE, NT>(e & kRowMask, off, mask, slot[0], cur);
        word[0] = uniform(ahead);
        op.template issue<U, MODE, NT>(word[0] & kRowMask, off, mask, slot[0]);
        ahead = sched[D + 1];
        if (!ends.has_head()) first = cur;
        for (; base + 2 * D < n; base += D) {
            static_for<0, D>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                constexpr int kNextSlot = (j + 1) % D;
                const int k = base + j;
                if constexpr (SYNC) __builtin_amdgcn_s_barrier();   // the workgroup visits each row together
                WorkT nx;
                const int e1 = word[kNextSlot];           // row of step k+1 arrives; its slot is refilled at once
                op.template finish<U, MODE, NT>(e1 & kRowMask, off, mask, slot[kNextSlot], nx);
                word[kNextSlot] = uniform(ahead);
                op.template issue<U, MODE, NT>(word[kNextSlot] & kRowMask, off, mask, slot[kNextSlot]);
                ahead = sched[k + 2 + D < n ? k + 2 + D : n - 1];
                step(nx, e1);
            });
        }
    } else {
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (j < n) op.template issue<U, MODE, NT>(uniform(sched[j]) & kRowMask, off, mask, slot[j]);
        if constexpr (PART && !Ends::kAhead) ends.template load<MODE, NT>(mask, first, tail);
        e = uniform(sched[0]);
        op.template finish<U, MODE, NT>(e & kRowMask, off, mask, slot[0], cur);
        if (D < n) op.template issue<U, MODE, NT>(uniform(sched[D]) & kRowMask, off, mask, slot[0]);
        if (skip_mix) {                   // a single gossiping row: nothing to average with
            op.template store<U, MODE, NT>(e & kRowMask, off, mask, cur);
            return;
        }
        if (!ends.has_head()) first = cur;
    }
    for (; base < n; base += D) {
        static_for<0, D>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            constexpr int kNextSlot = (j + 1) % D;
            const int k = base + j;
            if (k < n) {
                if constexpr (SYNC) __builtin_amdgcn_s_barrier();
                WorkT nx;
                int e1 = 0;
                if (k + 1 < n) {
                    e1 = uniform(sched[k + 1]);
                    op.template finish<U, MODE, NT>(e1 & kRowMask, off, mask, slot[kNextSlot], nx);
                    if (k + 1 + D < n)
                        op.template issue<U, MODE, NT>(uniform(sched[k + 1 + D]) & kRowMask, off, mask,
                                                       slot[kNextSlot]);
                } else if constexpr (PART) {
                    nx = first = tail;
                }
                step(nx, e1);
            }
        });
    }
}

// SHORT: rows shorter than one slice.
template <class Op, int U, int D, bool NT, bool SHORT = false>
__global__ __launch_bounds__(kWave *kMaxWavesPerBlock) void mix_kernel(
    Op op, int n, int64_t P, int S, const int64_t *__restrict__ seg_off,
    const int32_t *__restrict__ peers, int shift, int skip_mix, int64_t ntiles, int lockstep, unsigned piece_blocks)
{
    // The first piece_blocks workgroups serve the pieces that begin at a segment boundary inside a tile, one
    // wavefront each; the others serve the tiles, from a tile's first column to its end or to the first
    // boundary in it.  (One wavefront per tile walked all rows again for every segment that meets the tile, one
    // walk after the other: the longest part of every launch with few tiles.)
    extern __shared__ int lds[];
    OncePerLaunch<Op>::run(op);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int nwaves = blockDim.x >> 6;
    const bool is_piece = blockIdx.x < piece_blocks;
    const int64_t block = static_cast<int64_t>(blockIdx.x) - piece_blocks;
    constexpr int kSliceCols = Op::kElems;            // columns in one 16-byte slice
    constexpr int kTileCols = kWave * kSliceCols * U;

    if (!SHORT && lockstep && !is_piece) {
        // Workgroup-uniform fast path: the whole super-tile of the workgroup lies inside one
        // segment, so its waves share one schedule and walk the rows in lock-step.
        const int64_t g0 = block * nwaves * kTileCols;
        const int64_t g1 = g0 + static_cast<int64_t>(nwaves) * kTileCols;
        int lo = 1, hi = S;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_off[mid] <= g0) lo = mid + 1; else hi = mid;
        }
        const int s = lo - 1;
        const int64_t b = (s == 0) ? 0 : seg_off[s];
        const int64_t e = (s == S - 1) ? P : seg_off[s + 1];
        if (g1 <= P && b <= g0 && e >= g1) {
            const int *sched = lds + n;
            if (n > kWave) {
                schedule_rows(lds, n, static_cast<int>(threadIdx.x), static_cast<int>(blockDim.x), peers, s, shift, BlockSync{});
            } else {
                if (wave == 0) schedule_rows(lds, n, lane, kWave, peers, s, shift, WaveSync{});
                __syncthreads();
            }
            unsigned mask[U];
#pragma unroll
            for (int u = 0; u < U; ++u) mask[u] = (1u << kSliceCols) - 1u;
            const int64_t first = g0 + static_cast<int64_t>(wave) * kTileCols;
            walk<Op, U, D, kFull, NT, NoEnds, true>(op, sched, n, skip_mix != 0, column_of<Op>(first, lane, 0, 0), mask);
            return;
        }
    }
    // from here on waves are independent: no block barrier
    int *work = lds + wave * kScheduleWords(n);
    const int *sched = work + n;
    auto bound = [&](int s) -> int64_t {                   // where segment s begins, inside [0, P]
        if (s <= 0) return 0;
        if (s >= S) return P;
        const int64_t b = seg_off[s];
        return b < 0 ? 0 : (b > P ? P : b);
    };
    int s;
    int64_t b, c0;
    if (is_piece) {
        const int64_t piece = static_cast<int64_t>(blockIdx.x) * nwaves + wave + 1;
        if (piece >= S) return;
        s = static_cast<int>(piece);
        b = bound(s);
        c0 = b / kTileCols * kTileCols;
        if (b == c0) return;                               // begins with a tile: the tile's own wavefront
    } else {
        const int64_t tile = block * nwaves + wave;
        if (tile >= ntiles) return;
        b = c0 = tile * kTileCols;
        int lo = 1, hi = S;                                // segment of c0: number of interior boundaries <= c0
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_off[mid] <= c0) lo = mid + 1; else hi = mid;
        }
        s = lo - 1;
    }
    int64_t e = bound(s + 1);
    if (e > c0 + kTileCols) e = c0 + kTileCols;
    if (b >= e) return;
    const int64_t place = column_of<Op>(c0, lane, 0, 0);
    // this lane's first column
    const int64_t off = place - (SHORT ? 0 : row_end_slide(P, c0, place, U, kTileCols, kSliceCols));
    schedule_rows(work, n, lane, kWave, peers, s, shift, WaveSync{});
    unsigned mask[U];
    if (e - b == kTileCols) {
#pragma unroll
        for (int u = 0; u < U; ++u) mask[u] = (1u << kSliceCols) - 1u;
        walk<Op, U, D, kFull, NT>(op, sched, n, skip_mix != 0, off, mask);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
            mask[u] = slice_mask(off + u * (kWave * kSliceCols), kSliceCols, wanted_from(b, place, U), e);
        walk<Op, U, D, SHORT ? kShortRow : kBoundary, NT>(op, sched, n, skip_mix != 0, off, mask);
    }
}

// ---------------------------------------------------------------------------------
// In place, the rows of a tile split over wavefronts.  A wavefront that visits every row of its tile one after the
// other makes a launch last as long as one walk, whatever the tile's width: 1,024 rows eight at a time are 128 memory
// latencies.  Here `parts` wavefronts of a workgroup share a tile and its schedule, which they build together, and
// take a part of the rows each (schedule_part); `tiles` adjacent tiles make up the workgroup.  The rows of a part that
// other parts overwrite are read ahead (PartEnds), and no wavefront stores before all of the workgroup have theirs.
// In place, us, mix_kernel / this: fp32 gossip on 512 x 3,001 118 / 21, on 256 x 30,011 61 / 20; bf16 gossip on
// 355 x 50,356 123 / 31; binary16 optimizer step on 256 x 30,011 232 / 50; push-sum with the copy on 826 x 79,896 628 / 249.
// The first `pieces` workgroups serve the pieces that begin at a segment boundary inside a workgroup's columns.
// ---------------------------------------------------------------------------------
template <class Op, int U>
struct PartEnds {
    static constexpr bool kPart = true;
    // operators with many registers behind a row turn the two rows into tiles one after the other, before the ring
    static constexpr bool kAhead = Op::kRawPerSlice * U >= 6;
    using WorkT = typename Op::template Work<U>;
    const Op &op;
    int64_t off;
    int head_row, tail_row;                    // head_row -1: none
    __device__ __forceinline__ bool has_head() const { return head_row >= 0; }
    // COMMIT is false throughout: what an operator writes on arrival (v') is the owner's to write
    template <TileMode MODE, bool NT>
    __device__ __forceinline__ void load(const unsigned (&mask)[U], WorkT &head, WorkT &tail) const
    {
        typename Op::template Raw<U> raw;
        op.template issue<U, MODE, false>(tail_row, off, mask, raw);
        if constexpr (kAhead) {
            op.template finish<U, MODE, NT, false>(tail_row, off, mask, raw, tail);
            if (head_row >= 0) {
                op.template issue<U, MODE, false>(head_row, off, mask, raw);
                op.template finish<U, MODE, NT, false>(head_row, off, mask, raw, head);
            }
        } else {
            typename Op::template Raw<U> other;
            if (head_row >= 0) op.template issue<U, MODE, false>(head_row, off, mask, other);
            op.template finish<U, MODE, NT, false>(tail_row, off, mask, raw, tail);
            if (head_row >= 0) op.template finish<U, MODE, NT, false>(head_row, off, mask, other, head);
        }
        // the loads themselves have to be back, not only ordered: other wavefronts store to these rows next
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
};

// Most wavefronts of a workgroup: sixteen leave each 128 registers.
template <class Op, int U, int D>
constexpr int kPartWaves = (Op::kRawPerSlice * U * (PartEnds<Op, U>::kAhead ? D + 1 : D + 2) * 4 +
                            5 * Op::template Work<U>::kN * Op::template Work<U>::kRegs) <= 100 ? 16 : kMaxWavesPerBlock;

template <class Op, int U, int D>
__global__ __launch_bounds__((kWave * kPartWaves<Op, U, D>)) void parts_kernel(
    Op op, int n, int64_t P, int S, const int64_t *__restrict__ seg_off,
    const int32_t *__restrict__ peers, int shift, int parts, unsigned pieces)
{
    extern __shared__ int lds[];
    OncePerLaunch<Op>::run(op);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const int tiles = static_cast<int>(blockDim.x >> 6) / parts;
    constexpr int kSliceCols = Op::kElems;
    constexpr int kTileCols = kWave * kSliceCols * U;
    const int64_t block_cols = static_cast<int64_t>(kTileCols) * tiles;
    auto bound = [&](int s) -> int64_t {                   // where segment s begins, inside [0, P]
        if (s <= 0) return 0;
        if (s >= S) return P;
        const int64_t b = seg_off[s];
        return b < 0 ? 0 : (b > P ? P : b);
    };
    // the columns [b, e) of one segment that this workgroup serves: the returns are its waves' all together
    int s;
    int64_t b, c0;
    if (blockIdx.x < pieces) {
        s = static_cast<int>(blockIdx.x) + 1;
        b = bound(s);
        c0 = b / block_cols * block_cols;
        if (b == c0) return;                               // begins with a workgroup's columns: that one's
    } else {
        b = c0 = (static_cast<int64_t>(blockIdx.x) - pieces) * block_cols;
        int lo = 1, hi = S;                                // segment of c0: number of interior boundaries <= c0
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_off[mid] <= c0) lo = mid + 1; else hi = mid;
        }
        s = lo - 1;
    }
    int64_t e = bound(s + 1);
    if (e > c0 + block_cols) e = c0 + block_cols;
    if (b >= e) return;
    schedule_rows(lds, n, static_cast<int>(threadIdx.x), static_cast<int>(blockDim.x), peers, s, shift, BlockSync{});
    const SchedulePart part = schedule_part(lds, n, wave / tiles, parts, lane, kWave,
                                            [](bool c) { return __builtin_amdgcn_ballot_w64(c); });
    c0 += static_cast<int64_t>(wave % tiles) * kTileCols;
    if (b < c0) b = c0;
    if (e > c0 + kTileCols) e = c0 + kTileCols;
    const int first = uniform(part.begin), rows = uniform(part.end) - first;
    if (rows == 0 || b >= e) {
        __syncthreads();                                   // PartEnds::load of the others
        return;
    }
    const int64_t place = column_of<Op>(c0, lane, 0, 0);
    const int64_t off = place - row_end_slide(P, c0, place, U, kTileCols, kSliceCols);
    const PartEnds<Op, U> ends{op, off, uniform(part.head), uniform(part.tail)};
    const int *sched = lds + n + first;
    unsigned mask[U];
    if (e - b == kTileCols) {
#pragma unroll
        for (int u = 0; u < U; ++u) mask[u] = (1u << kSliceCols) - 1u;
        walk<Op, U, D, kFull, true>(op, sched, rows, false, off, mask, ends);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
            mask[u] = slice_mask(off + u * (kWave * kSliceCols), kSliceCols, wanted_from(b, place, U), e);
        walk<Op, U, D, kBoundary, true>(op, sched, rows, false, off, mask, ends);
    }
}

// ---------------------------------------------------------------------------------
// Row order of the out-of-place path: a table of 32-bit words in device memory that the
// library owns (no allocation at run time), written by order_kernel or segment_order_kernel and read by gather_kernel
// through a pointer both receive as an argument.
//
// Two layouts, by the tile (segment_order_kernel) and by the cluster (order_kernel).  By the cluster,
// entry (cluster, k): the k-th row the cluster's workgroups visit, that row's partner in the
// segment of the cluster's first column, and a flag saying that this segment covers every
// column of the cluster (so a whole tile of the cluster needs no segment lookup at all), also where its tiles start up to
// `slack` columns earlier (OnLines).
//
// The ordinary entry points keep kOrderSlots tables of kOrderEntries words per GPU and entry
// point (g_order).  A slot serves ONE stream at a time: calls on a stream run in stream order,
// so a table is never rewritten while an earlier call still reads it.  A stream keeps its slot
// while it has work in flight; a slot whose stream has drained (or has been destroyed) can be
// taken over by another stream.  Streams that find no free slot run without a table (natural
// row order: same results, slower).
// ---------------------------------------------------------------------------------
constexpr int kOrderSlots = 4;
constexpr int kOrderEntries = 1 << 18;
constexpr int kOrderRowBits = kRowBits;
constexpr unsigned kOrderRowField = (1u << kOrderRowBits) - 1u;
constexpr unsigned kOrderOneSegment = 1u << (2 * kOrderRowBits);
constexpr unsigned kLineBytes = 128;
__device__ __align__(256) unsigned g_order[kOrderSlots][kOrderEntries];

__device__ __forceinline__ unsigned order_word(const Place &p, int row)
{
    return static_cast<unsigned>(row) | (static_cast<unsigned>(p.partner) << kOrderRowBits);
}

// One workgroup per segment: builds the segment's row order and writes it for every cluster whose first
// column lies in that segment.  With build_schedule and the partners read again / now, us: 32 rows in 8 segments 6.7 / 5.8;
// segment_order_kernel below, 512 rows in 16 segments 6.4 / 4.8; the call on 512 x 100,003 fp32 93.4 / 91.6, on 512 x 50,003
// 52.9 / 50.9, on 900 x 50,003 bf16 48.4 / 45.1.
__global__ __launch_bounds__(1024) void order_kernel(int n, int64_t P, int S,
                                                    const int64_t *__restrict__ seg_off,
                                                    const int32_t *__restrict__ peers, int shift,
                                                    int64_t cluster_cols, int nclusters, int slack,
                                                    unsigned *__restrict__ order)
{
    extern __shared__ int lds[];
    const int s = blockIdx.x;
    int64_t sb = (s == 0) ? 0 : seg_off[s];
    int64_t se = (s == S - 1) ? P : seg_off[s + 1];
    sb = sb < 0 ? 0 : (sb > P ? P : sb);
    se = se < 0 ? 0 : (se > P ? P : se);
    const int row = static_cast<int>(threadIdx.x);         // a thread for every row: order_threads
    const Place p = place_row(lds, n, row, peers, s, shift, BlockSync{});
    unsigned *words = reinterpret_cast<unsigned *>(lds);
    if (row < n) words[p.at] = order_word(p, row);
    __syncthreads();
    const int64_t c_lo = (sb + cluster_cols - 1) / cluster_cols;
    int64_t c_hi = (se + (s == S - 1 ? slack : 0) + cluster_cols - 1) / cluster_cols;
    if (c_hi > nclusters) c_hi = nclusters;
    const unsigned un = static_cast<unsigned>(n);
    const unsigned total = static_cast<unsigned>(c_hi > c_lo ? c_hi - c_lo : 0) * un;   // fits: the table does
    for (unsigned idx = threadIdx.x; idx < total; idx += blockDim.x) {
        const unsigned k = idx % un;
        const int64_t c = c_lo + idx / un;
        const int64_t first_col = c * cluster_cols - slack > 0 ? c * cluster_cols - slack : 0;
        const int64_t last_col = (c + 1) * cluster_cols < P ? (c + 1) * cluster_cols : P;
        unsigned e = words[k];
        if (first_col >= sb && last_col <= se) e |= kOrderOneSegment;
        order[c * n + k] = e;
    }
}

// The order by the tile: n words for each segment, its row order, and behind all S of them one word for each tile, the
// segment of its first column and whether that one covers the tile (one segment: n words).  A cluster that several
// segments meet walks every tile in its own segment's order; in the order of the cluster's first column the partners of
// the others miss L2 and their tiles look the segment up.  Against order_kernel's, us: fp32 gossip on 512 x 100,003,
// 16 ragged segments 111 / 98, on 512 x 312,501 302 / 253, on 128 x 2,500,001 499 / 449; fp32 optimizer step on
// 512 x 312,501 813 / 650; bf16 gossip on 512 x 625,001 347 / 271.
constexpr unsigned kTileOneSegment = 1u << 31;

__global__ __launch_bounds__(1024) void segment_order_kernel(int n, int64_t P, int S, const int64_t *__restrict__ seg_off,
                                                            const int32_t *__restrict__ peers, int shift, int tile_shift,
                                                            int slack, unsigned *__restrict__ order)
{
    extern __shared__ int lds[];
    const int s = blockIdx.x;
    int64_t sb = (s == 0) ? 0 : seg_off[s];
    int64_t se = (s == S - 1) ? P : seg_off[s + 1];
    sb = sb < 0 ? 0 : (sb > P ? P : sb);
    se = se < 0 ? 0 : (se > P ? P : se);
    const int row = static_cast<int>(threadIdx.x);
    const Place p = place_row(lds, n, row, peers, s, shift, BlockSync{});
    if (row < n) order[static_cast<unsigned>(s) * n + p.at] = order_word(p, row);
    if (S == 1) return;
    unsigned *tiles = order + static_cast<unsigned>(S) * n;
    const int64_t tile_cols = static_cast<int64_t>(1) << tile_shift;
    const int64_t end = se + (s == S - 1 ? slack : 0);
    for (int64_t t = ((sb + tile_cols - 1) >> tile_shift) + threadIdx.x; (t << tile_shift) < end; t += blockDim.x) {
        const int64_t first_col = (t << tile_shift) - slack > 0 ? (t << tile_shift) - slack : 0;
        tiles[t] = static_cast<unsigned>(s) | (first_col >= sb && (t + 1) << tile_shift <= se ? kTileOneSegment : 0u);
    }
}

// ---------------------------------------------------------------------------------
// Rows that begin inside lines of 128 bytes.  In the column grid every access of a wavefront to its own row then meets
// nine lines instead of eight, and the lines at its ends are written in two parts by two wavefronts, which reach memory
// apart as often as not.  With an operator marked OnLines a row's tiles start on the row's own lines, up to kLineSlack columns
// earlier, so that only the partner's loads, which L2 serves, are shifted against lines; the first tile of a row hangs
// over its beginning and is a boundary tile.  A tile or cluster counts as inside one segment if it is, wherever its row
// begins.  In the column grid / on lines, us: fp32 gossip on 512 x 100,003 96.3 / 94.4, on 32 x 25,557,032 1,131 / 1,112;
// push-sum of bf16 rows with the copy on 128 x 11,689,513 1,595 / 1,568; optimizer step on 64 x 5,000,001 fp32 1,168 / 1,144, on
// 128 x 3,000,003 bf16 961 / 939; which operators take it: starts_on_lines in cx_launch.hpp.  (With the shift as an argument instead
// of a kernel of its own, rows on lines paid 0.5 to 1.5 % for it.)
// ---------------------------------------------------------------------------------
template <class Op>
struct OnLines : Op {};
template <class Op> constexpr bool kOnLines = false;
template <class Op> constexpr bool kOnLines<OnLines<Op>> = true;
template <class Op>
constexpr int kLineSlack = 7 * Op::kElems;             // rows are aligned to 16 bytes, one slice
// Columns by which an output row begins past a line.
template <class Op>
__device__ __forceinline__ int columns_past_line(const Op &op, int row)
{
    constexpr unsigned kBytes = 16 / Op::kElems;
    const unsigned at = static_cast<unsigned>(reinterpret_cast<uintptr_t>(op.xout)) +
                        static_cast<unsigned>(row) * (static_cast<unsigned>(op.ld) * kBytes);
    return static_cast<int>((at & (kLineBytes - 1)) / kBytes);
}

// The same column, but not known to the compiler as such: what is computed from it is computed again instead of
// being kept in registers.
__device__ __forceinline__ int64_t fresh_column(int64_t column)
{
    asm volatile("" : "+v"(column));
    return column;
}

// ---------------------------------------------------------------------------------
// Out-of-place path: one short-lived workgroup per (gossiping row, column chunk).  It loads
// the row's chunk and its partner's chunk, averages, and stores to the other buffer.  Each
// chunk is fetched twice (once as "own", once as somebody's partner); the block order makes
// the two fetches meet in one XCD's L2, so HBM still sees every element once:
//   * workgroups go to the XCDs round-robin by block id, so block b belongs to XCD b % nxcd;
//   * an XCD works through clusters of CL neighbouring chunks, row after row (CL chunks of one
//     row, then CL chunks of the next).  Rows are taken in the order of the segment's
//     permutation cycles (order_kernel), so the partner chunk a block fetches is the own
//     chunk of the block that follows it: only two row visits have to stay in L2;
//   * the XCDs hold neighbouring clusters at the same time, which keeps the stream of every
//     row dense in DRAM.
// Needs x_out != x_in (and v_out != v_in): a partner's input may be read after its owner
// has stored.  Any table with entries in [0, n) is served, permutation or not.
// ---------------------------------------------------------------------------------
// SHORT: rows shorter than one slice.
template <class Op, int U, bool NT, bool SHORT = false>
__global__ __launch_bounds__(kWave *kMaxWavesPerBlock) void gather_kernel(
    Op op, int n, int64_t P, int S, const int64_t *__restrict__ seg_off,
    const int32_t *__restrict__ peers, int shift, int skip_mix, unsigned nchunks, unsigned CL,
    unsigned nwaves, int xcd_shift, const unsigned *__restrict__ order, int by_tile)
{
    // grid: x = (chunk within cluster, xcd) with the xcd in the low bits, y = gossiping row,
    // z = cluster.  Blocks are dispatched x-fastest, so an XCD sees, for one cluster, row 0's
    // CL chunks, then row 1's, ... and no integer division is needed to decode the block.
    // Chunk and tile numbers fit 32 bits (checked by the host), so the block is decoded with
    // a handful of scalar instructions, and the two ways out of the grid's padding share one
    // branch: the kernel's arguments are fetched once, ahead of it.
    constexpr bool LINES = kOnLines<Op>;
    OncePerLaunch<Op>::run(op);
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned wave = uniform(threadIdx.x >> 6);
    const unsigned xcd = blockIdx.x & ((1u << xcd_shift) - 1u);
    const unsigned t = blockIdx.x >> xcd_shift;
    const unsigned cluster = (blockIdx.z << xcd_shift) + xcd;
    const unsigned chunk = cluster * CL + t;
    constexpr int kSliceCols = Op::kElems;
    constexpr int kTileCols = kWave * kSliceCols * U;
    int64_t c0 = static_cast<int64_t>(chunk * nwaves + wave) * kTileCols;
    if (chunk >= nchunks || c0 >= P + (LINES ? kLineSlack<Op> : 0)) return;
    int64_t c1 = (c0 + kTileCols < P) ? c0 + kTileCols : P;
    int64_t off = column_of<Op>(c0, lane, 0, 0);           // this lane's first column
    unsigned full_mask[U];
#pragma unroll
    for (int u = 0; u < U; ++u) full_mask[u] = (1u << kSliceCols) - 1u;

    // `mine` holds (or will hold) this row's data; average it with the partner's and store.
    // Operators with many rows behind a gossiping row (hierarchical groups) reduce their
    // own rows before the partner's are requested, which halves the registers in flight.  Boundary tiles always
    // do, and form the rows' addresses anew for each phase: they are few, but the kernel is given the registers of
    // its hungriest path, and with fewer wavefronts per SIMD every tile runs slower.  Against both rows at once, with
    // their addresses kept: mean of groups of 2 85 -> 72 registers, gradient step of groups of 3 171 -> 118.
    int row = blockIdx.y;
    typename Op::template Raw<U> mine;
    auto mix_and_store = [&](auto mode_c, int64_t at, const unsigned (&m)[U], int peer) {
        constexpr TileMode MODE = decltype(mode_c)::value;
        using WorkT = typename Op::template Work<U>;
        constexpr bool kOneAtATime = Op::kRawPerSlice * WorkT::kN >= 16 ||            // 16-byte registers per phase
                                     (WorkT::kRegs == 8 && Op::kRawPerSlice * U >= 6);  // fp64 chains take more
        typename Op::template Work<U> a, out;
        if (skip_mix) {
            op.template finish<U, MODE, NT, true>(row, at, m, mine, a);
            out = a;
        } else {
            typename Op::template Work<U> c;
            if constexpr (kOneAtATime || MODE != kFull) {
                op.template finish<U, MODE, NT, true>(row, at, m, mine, a);
                if constexpr (MODE != kFull) at = fresh_column(at);
                op.template issue<U, MODE, false>(peer, at, m, mine);
                op.template finish<U, MODE, NT, false>(peer, at, m, mine, c);
            } else {
                typename Op::template Raw<U> theirs;
                op.template issue<U, MODE, false>(peer, at, m, theirs);
                op.template finish<U, MODE, NT, true>(row, at, m, mine, a);
                op.template finish<U, MODE, NT, false>(peer, at, m, theirs, c);
            }
#pragma unroll
            for (int u = 0; u < Op::template Work<U>::kN; ++u) out.v[u] = average(a.v[u], c.v[u]);
        }
        if constexpr (MODE != kFull) at = fresh_column(at);
        op.template store<U, MODE, NT>(row, at, m, out);
    };

    // y is the position in the cluster's row order: with the order kernel's table, rows follow
    // the permutation cycles, so this block's partner is the next block's own row (fresh in L2).
    // Fast path, almost every tile: the table entry also names the partner and it or the tile's word says
    // that one segment covers the tile, so a tile that does not hang over the row end starts all its
    // loads after one or two scalar loads.  Whatever the table holds, no access leaves the
    // matrix: rows are checked against n and the tile against P.
    auto to_line = [&] {                                   // once the row is known
        if constexpr (LINES) {
            const int past = columns_past_line(op, row);
            c0 -= past;
            off -= past;
            c1 = (c0 + kTileCols < P) ? c0 + kTileCols : P;
        }
    };
    if (!SHORT && order) {
        unsigned at = cluster, one_segment = 0;
        if (by_tile) {
            const unsigned w = S > 1 ? order[static_cast<unsigned>(S * n) + chunk * nwaves + wave] : kTileOneSegment;
            at = w & ~kTileOneSegment;
            one_segment = w & kTileOneSegment ? kOrderOneSegment : 0u;
            if (at >= static_cast<unsigned>(S)) at = 0;
        }
        const unsigned e = order[at * static_cast<unsigned>(n) + blockIdx.y] | one_segment;
        const int r = static_cast<int>(e & kOrderRowField);
        const int q = static_cast<int>((e >> kOrderRowBits) & kOrderRowField);
        if (r < n) row = r;
        to_line();
        if constexpr (LdsStaged<Op>::value) {
            // the whole chunk of this workgroup inside one segment and inside the row: every wavefront
            // of the workgroup takes this branch together (the table entry and the chunk are shared)
            const int64_t chunk_c0 = static_cast<int64_t>(chunk) * nwaves * kTileCols;
            if ((e & kOrderOneSegment) != 0 && r < n && q < n && !skip_mix && U == 1 &&
                nwaves * kWave == blockDim.x && static_cast<size_t>(nwaves) * nwaves * kWave * sizeof(f4) == LdsStaged<Op>::bytes &&
                chunk_c0 + static_cast<int64_t>(nwaves) * kTileCols <= P) {
                extern __shared__ f4 staging[];
                op.template lds_mix<NT>(row, q, chunk_c0, lane, static_cast<int>(wave), staging);
                return;
            }
        }
        if ((e & kOrderOneSegment) != 0 && r < n && q < n && (!LINES || c0 >= 0) && c0 + kTileCols <= P) {
            op.template issue<U, kFull, false>(row, off, full_mask, mine);
            mix_and_store(std::integral_constant<TileMode, kFull>{}, off, full_mask, q);
            return;
        }
    } else {
        to_line();
    }
    if (LINES && c0 >= P) return;

    // General path: tiles of clusters that a segment boundary or the row end crosses, and every
    // tile when there is no order table.  With up to 63 segments one vector load brings the
    // whole offset table and this row's partner in every segment into lanes 0..S at once (a
    // single memory latency); the segment of c0 is then a ballot + popcount and the table
    // entries are read across lanes.  Longer tables fall back to a scalar binary search.
    // The row's own data does not depend on the segment: a tile that does not hang over the
    // row end puts its loads in flight before the lookup.
    const bool whole = (!LINES || c0 >= 0) && c0 + kTileCols <= P;
    if (whole) op.template issue<U, kFull, false>(row, off, full_mask, mine);
    const bool in_lanes = S <= 63;
    int64_t lane_off = 0;
    int lane_peer = row;
    int first_seg;
    if (in_lanes) {
        if (lane <= S && S > 1) lane_off = seg_off[lane];
        if (lane < S) lane_peer = partner_of(peers, shift, n, lane, row);
        const bool below = lane >= 1 && lane < S && lane_off <= c0;
        first_seg = __builtin_popcountll(__builtin_amdgcn_ballot_w64(below));
    } else {
        int lo = 1, hi = S;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_off[mid] <= c0) lo = mid + 1; else hi = mid;
        }
        first_seg = lo - 1;
    }
    auto offset_at = [&](int k) -> int64_t {
        if (!in_lanes) return seg_off[k];
        const unsigned lo32 = __builtin_amdgcn_readlane(static_cast<int>(lane_off), k);
        const unsigned hi32 = __builtin_amdgcn_readlane(static_cast<int>(lane_off >> 32), k);
        return static_cast<int64_t>((static_cast<uint64_t>(hi32) << 32) | lo32);
    };
    constexpr TileMode kCut = SHORT ? kShortRow : kBoundary;
    const int64_t at = off - (SHORT ? 0 : row_end_slide(P, c0, off, U, kTileCols, kSliceCols));
    for (int s = first_seg; s < S; ++s) {
        int64_t sb = (s == 0) ? 0 : offset_at(s);
        int64_t se = (s == S - 1) ? P : offset_at(s + 1);
        sb = sb < 0 ? 0 : (sb > P ? P : sb);
        se = se < 0 ? 0 : (se > P ? P : se);
        if (sb >= c1) break;
        if (sb < c0) sb = c0;
        if (se > c1) se = c1;
        if (sb >= se) continue;
        const int peer = in_lanes ? __builtin_amdgcn_readlane(lane_peer, s) : partner_of(peers, shift, n, s, row);
        if (whole && sb == c0 && se == c0 + kTileCols) {  // one segment covers the whole tile
            mix_and_store(std::integral_constant<TileMode, kFull>{}, off, full_mask, peer);
            return;
        }
        // boundary tile: per-element predication, once per overlapped segment
        unsigned mask[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            mask[u] = slice_mask(at + u * (kWave * kSliceCols), kSliceCols, wanted_from(sb, off, U), se);
        const int64_t here = fresh_column(at);
        op.template issue<U, kCut, false>(row, here, mask, mine);
        mix_and_store(std::integral_constant<TileMode, kCut>{}, here, mask, peer);
    }
}

}  // namespace

#endif  // CX_KERNELS_HPP
