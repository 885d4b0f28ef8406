// Host side of the device half (internal header): launch shapes, the row-order table's slots, the two
// launchers and the argument checks shared by the entry points.  Each cx_api_*.hip includes this header and
// defines its entry points, so the operators compile in parallel; everything has internal linkage (each
// translation unit carries its own row-order table).
#ifndef CX_LAUNCH_HPP
#define CX_LAUNCH_HPP
#include "cx_kernels.hpp"

namespace {

// ---------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------
struct Launch {
    int U, D, waves, nt, lockstep, wgs_per_cu;
};

Launch pick_launch(const WalkShape &dflt)
{
    Launch l;
    l.U = cx_get_tuning(0);
    if (l.U != 1 && l.U != 2 && l.U != 4) l.U = dflt.U;
    l.lockstep = cx_get_tuning(4) == 0 ? 0 : 1;
    l.waves = cx_get_tuning(1);
    if (l.waves < 1 || l.waves > kMaxWavesPerBlock) l.waves = dflt.waves;
    l.nt = cx_get_tuning(2);
    if (l.nt != 0 && l.nt != 1) l.nt = 1;
    l.D = cx_get_tuning(3);
    if (l.D != 2 && l.D != 4 && l.D != 8) l.D = dflt.D;
    l.wgs_per_cu = cx_get_tuning(9);
    if (l.wgs_per_cu < 0 || l.wgs_per_cu > 16) l.wgs_per_cu = dflt.wgs_per_cu;
    return l;
}

[[maybe_unused]] bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// true if the byte ranges [a, a+bytes) and [b, b+bytes) overlap without being identical
[[maybe_unused]] bool partial_overlap(const void *a, const void *b, uint64_t bytes)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    if (x == y) return false;
    return x < y ? (y - x) < bytes : (x - y) < bytes;
}
[[maybe_unused]] bool any_overlap(const void *a, const void *b, uint64_t bytes)
{
    return a == b || partial_overlap(a, b, bytes);
}

struct MixArgs {
    int n;
    int64_t P;
    int S;
    const int64_t *seg_off;
    const int32_t *peers;
    int shift, skip_mix;
    hipStream_t stream;
    bool out_of_place;          // every output buffer is distinct from its input buffer
    int rows_per_gossip_row;    // G: matrix rows behind one gossiping row (cluster footprint)
    // Row-order table supplied by the entry point instead of one of the library's per-stream
    // slots: its capacity in words and where to get its device address once the workload is known
    // to fit (the call fails with CX_ERR_SHAPE rather than run without a table when it does not).
    unsigned *(*order_provider)() = nullptr;
    int64_t order_entries = 0;
};

// Dynamic LDS a workgroup reserves so that at most `wgs_per_cu` of them are resident on a CU
// (0 = no cap).  Fewer resident workgroups keep fewer bytes in flight per CU, which this
// memory system rewards for the row-wandering walk (+3 to +8 %) and for the fused gather
// (+2 %).  A CU has 160 KB of LDS; a workgroup may take up to 64 KB.
[[maybe_unused]] size_t lds_reservation(int wgs_per_cu)
{
    if (wgs_per_cu <= 0) return 0;
    const size_t reserve = (160u << 10) / static_cast<unsigned>(wgs_per_cu);
    return reserve > (64u << 10) ? (64u << 10) : reserve;
}

// A (slices, depth) pair is built for an operator only if its ring of in-flight rows stays
// within the register file without spilling (at least two waves per SIMD stay resident).
template <class Op, class = void>
struct MaxSlices {
    static constexpr int value = 4;
};
template <class Op>
struct MaxSlices<Op, std::void_t<decltype(Op::kMaxU)>> {
    static constexpr int value = Op::kMaxU;                // an operator may build fewer shapes
};

// Shapes within the estimate below for which the compiler still put registers into scratch (an operator names its own).
template <class Op, int U, int D, class = void>
struct Spills {
    static constexpr bool value = false;
};
template <class Op, int U, int D>
struct Spills<Op, U, D, std::void_t<decltype(Op::template kSpills<U, D>)>> {
    static constexpr bool value = Op::template kSpills<U, D>;
};

template <class Op, int U, int D>
constexpr bool fits()
{
    // registers of the ring of rows in flight plus the four working tiles of the walk: a
    // workgroup of eight waves leaves each wave 256 registers
    return U <= MaxSlices<Op>::value && !Spills<Op, U, D>::value &&
           Op::kRawPerSlice * U * D * 4 + 4 * Op::template Work<U>::kN * Op::template Work<U>::kRegs <= 224 &&
           Op::kRawPerSlice * U * D * 4 <= 144 && !(U == 4 && Op::kRawPerSlice * D >= 8);
}

// The waves of an in-place workgroup whose schedules, one per wave, stay within 48 KB of LDS.
template <class Op>
constexpr int waves_with_schedules(int n, int waves)
{
    while (waves > 1 && (sizeof(int) * kScheduleWords(n) + StageBytes<Op>::value) * waves > 48 * 1024) --waves;
    return waves;
}

// In-place walk on short rows: a wavefront walks all rows of its tile one after the other, so a launch lasts as
// long as one walk and the bytes in flight come from narrow tiles (more walks) and a deep ring (more rows of each).
// Below kShortTiles tiles (8 wavefronts per CU; three times as many where a lane would take two slices) a lane takes
// one slice and the deepest ring that stays within kShortRing 16-byte registers; workgroups are halved until there
// are kShortBlocks of them, one for every second CU (fewer, larger ones lose to idle CUs, more lose the lock-step of
// the waves: bf16 gradient step on 256 x 400,007 in groups of 8, one segment: 102 us with 4 waves, 149 with eight, 138 with
// two, 161 with one).  fp32 optimizer step on 64 x 300,007, one segment: 131 -> 82 us with one slice, eight rows; bf16
// gossip on 256 x 800,007: 273 -> 194.  (Calls that part_shape splits do not come here.)
//
// The cap on resident workgroups is a cap on wavefronts: where a workgroup has fewer than the operator's, because rows
// are short or because many rows' schedules fill the LDS, more of them may be resident.  1,024 x 600,003 fp32 in place,
// workgroups of two waves, two of them against eight per CU: gossip 1,274 -> 1,196 us, optimizer step 2,796 -> 2,793,
// push-sum with the de-biased copy 3,063 -> 2,274.
//
// Operators on plain rows that take one slice instead of two there, with tiles enough, take eight rows in flight beside
// many rows only: push-sum of 16-bit rows with the copy on 64 x 2,000,003 193 us with eight, 155 with four; bf16 gossip
// on 32 x 3,200,013 97 us with eight, 83 with four; push-sum of 16-bit rows on 256 x 3,000,001 606 and 599.
constexpr int64_t kShortTiles = 2048, kShortBlocks = 128;
constexpr int kShortRing = 32;
template <class Op, class = void>
struct LongWalk {
    static constexpr WalkShape of(const Op &, int, int64_t, bool) { return Op::kWalk; }
};
template <class Op>
struct LongWalk<Op, std::void_t<decltype(std::declval<const Op &>().walk(0, 0, false))>> {
    static constexpr WalkShape of(const Op &op, int n, int64_t P, bool whole_lines) { return op.walk(n, P, whole_lines); }
};
template <class Op>
constexpr WalkShape walk_shape(const Op &op, int n, int64_t P)
{
    const bool whole_lines = op.ld * (16 / Op::kElems) % 128 == 0;
    WalkShape shape = LongWalk<Op>::of(op, n, P, whole_lines);
    const auto tiles = [&] {
        const int64_t cols = static_cast<int64_t>(kWave) * Op::kElems * shape.U;
        return (P + cols - 1) / cols;
    };
    if (tiles() < (shape.U > 1 ? 3 : 1) * kShortTiles) {
        shape.U = 1;
        shape.waves = Op::kWalk.waves;
        shape.wgs_per_cu = Op::kWalk.wgs_per_cu;
        shape.D = fits<Op, 1, 8>() && Op::kRawPerSlice * 8 <= kShortRing   ? 8
                  : fits<Op, 1, 4>() && Op::kRawPerSlice * 4 <= kShortRing ? 4
                                                                          : 2;
        if (Op::kRawPerSlice == 1 && tiles() >= kShortTiles && shape.D > ring_for(n)) shape.D = ring_for(n);
    }
    const int full_waves = shape.waves;
    while (shape.waves > 1 && tiles() <= (kShortBlocks - 1) * shape.waves) shape.waves /= 2;
    shape.waves = waves_with_schedules<Op>(n, shape.waves);
    shape.wgs_per_cu = shape.wgs_per_cu * full_waves / shape.waves;
    return shape;
}

template <class Op, int U, int D>
bool try_launch(const Op &op, const Launch &l, const MixArgs &a)
{
    if (l.U != U || l.D != D) return false;
    if constexpr (!fits<Op, U, D>()) {
        return false;
    } else {
        const int64_t tile_cols = static_cast<int64_t>(kWave) * Op::kElems * U;
        const int64_t ntiles = (a.P + tile_cols - 1) / tile_cols;
        const int waves = waves_with_schedules<Op>(a.n, l.waves);
        const int64_t nblocks = (ntiles + waves - 1) / waves;
        // one wavefront for each inner segment boundary, ahead of the tiles (boundaries that fall on a tile's edge
        // leave theirs at once)
        const unsigned pieces = a.S > 1 ? (static_cast<unsigned>(a.S) - 1 + waves - 1) / waves : 0;
        const dim3 grid(static_cast<unsigned>(nblocks) + pieces), block(kWave * waves);
        const size_t schedules = (sizeof(int) * kScheduleWords(a.n) * waves + 15) / 16 * 16;
        size_t lds = schedules + static_cast<size_t>(StageBytes<Op>::value) * waves;
        if (lds < lds_reservation(l.wgs_per_cu)) lds = lds_reservation(l.wgs_per_cu);
        const Op staged = with_stage_base(op, schedules);
        const auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, lds, a.stream, staged, a.n, a.P, a.S, a.seg_off, a.peers, a.shift,
                               a.skip_mix, ntiles, l.lockstep, pieces);
        };
        if constexpr (U == 1 && D == 2)
            if (a.P < Op::kElems) { launch(mix_kernel<Op, U, D, false, true>); return true; }
        if (l.nt) launch(mix_kernel<Op, U, D, true>);
        else launch(mix_kernel<Op, U, D, false>);
        return true;
    }
}

// Device address of this translation unit's g_order on the current device.  In host code the
// array's name is only a handle: the address comes from hipGetSymbolAddress, once per device.
constexpr int kMaxDevices = 64;
unsigned *order_tables_base(int *device_out)
{
    static std::mutex mu;
    static unsigned *base[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    *device_out = dev;
    std::lock_guard<std::mutex> lock(mu);
    if (!base[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_order)) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        base[dev] = static_cast<unsigned *>(p);
    }
    return base[dev];
}

// Serialises "order_kernel, then gather_kernel" of one call against other host threads, so
// that two threads enqueueing on one stream cannot interleave their pairs.
std::mutex &enqueue_mutex()
{
    static std::mutex mu;
    return mu;
}

// The order table `stream` may write on the current device, or nullptr (run without one).
// A stream keeps the slot it used last.  When every slot belongs to another stream, a slot
// whose owner has no work in flight (or no longer exists) changes hands.  Calls recorded under
// stream capture get a slot of their own, apart from the one the same stream uses for eager
// calls, and keep it for good: the captured graph names it, and may be replayed on any stream
// while eager calls go on.  (Graphs captured on ONE stream share that slot: replay them in
// one stream's order.)
unsigned *order_table_for(hipStream_t stream)
{
    struct Slot {
        hipStream_t owner;
        bool used, for_capture;
    };
    static Slot slots[kMaxDevices][kOrderSlots];
    int dev = 0;
    unsigned *base = order_tables_base(&dev);
    if (!base) return nullptr;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    const bool capturing = hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
    Slot *mine = slots[dev];
    int slot = -1;
    for (int i = 0; i < kOrderSlots && slot < 0; ++i)
        if (mine[i].used && mine[i].owner == stream && mine[i].for_capture == capturing) slot = i;
    for (int i = 0; i < kOrderSlots && slot < 0; ++i)
        if (!mine[i].used) slot = i;
    // (no questions about other streams while this one records: a capture forbids them)
    for (int i = 0; i < kOrderSlots && slot < 0 && !capturing; ++i) {
        if (mine[i].for_capture) continue;                                        // a graph names it
        hipStreamCaptureStatus ocs = hipStreamCaptureStatusNone;
        const hipError_t q = hipStreamIsCapturing(mine[i].owner, &ocs);
        if (q == hipSuccess && ocs != hipStreamCaptureStatusNone) continue;       // recording: leave it
        const hipError_t busy = q == hipSuccess ? hipStreamQuery(mine[i].owner) : q;
        if (busy == hipErrorNotReady) continue;                                   // work in flight
        if (busy != hipSuccess) (void)hipGetLastError();                          // the stream is gone
        slot = i;
    }
    if (slot < 0) return nullptr;
    mine[slot] = Slot{stream, true, capturing};
    return base + static_cast<int64_t>(slot) * kOrderEntries;
}

// Out-of-place launch: one workgroup per (gossiping row, chunk of waves * 64 * U slices).
//
// Short rows: a workgroup of the operator's full size would leave too few chunks to deal out evenly to eight
// XCDs, so the workgroup is halved until there are kMinChunks of them (or it is one wavefront): 13 or more
// chunks per XCD keep the uneven last one below 8 %.  512 rows x 100,003 fp32 columns: 98 chunks of 4 waves.
// An operator staged through LDS keeps its waves: the staging is laid out for one shape, and other workgroups of it
// take the path in registers.
constexpr int64_t kMinChunks = 104;
// A thread for every row, as place_row needs (512 rows with 256 threads and build_schedule 9.5 us, with 512 7.4, with
// place_row 4.8).
constexpr int order_threads(int n) { return n <= 256 ? 256 : n <= 512 ? 512 : 1024; }
constexpr int64_t kCachedBytes = 64LL << 20;              // a matrix that the last-level cache holds, and its copy
constexpr int kTileOrder = 16;                            // see by_tile in try_gather
template <class Op, int U>
constexpr int gather_waves(int64_t P, int waves)
{
    const int64_t wave_cols = static_cast<int64_t>(kWave) * Op::kElems * U;
    while (!LdsStaged<Op>::value && waves > 1 && P <= (kMinChunks - 1) * wave_cols * waves) waves /= 2;
    return waves;
}
enum class Push { kNo, kPlain, kWithCopy };
template <class Op> constexpr Push push_kind(const Op &) { return Push::kNo; }
constexpr Push push_kind(const PushOp &op) { return op.zout ? Push::kWithCopy : Push::kPlain; }
template <bool H> constexpr Push push_kind(const Push16Op<H> &op) { return op.zout ? Push::kWithCopy : Push::kPlain; }
template <class Op, class = void>
struct HasMomentum : std::false_type {};
template <class Op>
struct HasMomentum<Op, std::void_t<decltype(std::declval<const Op &>().vin)>> : std::true_type {};

// Operators whose tiles start on the rows' own lines (OnLines) where rows begin inside lines.  Time on lines over that in the column
// grid, geometric mean (largest): fp32 gossip, its stores written through on lines, 0.982 (1.029) of 84 shapes, fp32 optimizer step
// 0.989 (1.015) of 49, 16-bit 0.981 (1.000) of 93, push-sum with the copy 0.987 (1.000) of 19 and 0.981 (0.994) of 23, fp32 without
// it 0.989 (1.008) of 13.  16-bit rows that are only averaged gain nothing: gossip 1.004 (1.094) of 170, 200 rows and more of
// 300,000 to 3,000,000 columns 1.02, push-sum without the copy 1.004 (1.096) of 19.
template <class Op>
constexpr bool kMayStartOnLines = Op::kRows == 1 && !std::is_same_v<Op, Bf16Op> && !std::is_same_v<Op, Fp16Op>;
template <class Op>
constexpr bool starts_on_lines(const Op &op)
{
    return kMayStartOnLines<Op> && !(Op::kElems == 8 && push_kind(op) == Push::kPlain);
}
template <class Op>
constexpr bool staged_shape(int waves)
{
    return LdsStaged<Op>::value && static_cast<size_t>(waves) * waves * kWave * sizeof(f4) == LdsStaged<Op>::bytes;
}

template <class Op, int U>
bool try_gather(const Op &op, int want_u, int waves, bool waves_fixed, int nt, int cl_req, int xcd_aware,
                const MixArgs &a, int *status)
{
    if (want_u != U) return false;
    if constexpr (U > MaxSlices<Op>::value || (U > 1 && Op::kRawPerSlice * U > 8)) {   // launch_mix asks for no such U
        return false;
    } else {
    const int full_waves = waves;
    if (!waves_fixed && xcd_aware) waves = gather_waves<Op, U>(a.P, waves);
    const int64_t chunk_cols = static_cast<int64_t>(kWave) * Op::kElems * U * waves;
    const int64_t matrix_bytes = static_cast<int64_t>(a.n) * a.rows_per_gossip_row * a.P * (16 / Op::kElems);
    // Rows in cycle order pay when the partner's fetch has to be kept out of HBM; a matrix that
    // the last-level cache holds whole gains nothing from the extra launch.
    const bool own_table = a.order_provider != nullptr;
    bool ordered = a.n > 1 && a.S <= 4096 &&
                   (own_table || cx_get_tuning(8) == 1 || (cx_get_tuning(8) != 0 && matrix_bytes > kCachedBytes));
    // Rows that begin inside a line keep to their lines where the operator gains by it and they are in cycle order too: what the
    // cache holds whole loses by the one chunk more that a row may need (fp32 gossip on 700 x 3,003 9.1 / 9.4 us, on
    // 8 x 1,000,001 13.0 / 13.5).  A tile must not reach over both ends of a row, a group's rows begin on different columns of a
    // line, and a table of the caller's holds what it was sized for.
    const bool on_lines = ((reinterpret_cast<uintptr_t>(op.xout) | static_cast<uint64_t>(op.ld) * (16 / Op::kElems)) & (kLineBytes - 1)) == 0;
    const bool lines = starts_on_lines(op) && !on_lines && ordered && !own_table && a.P >= 2 * kWave * Op::kElems * U;
    const int slack = lines ? kLineSlack<Op> : 0;
    const int64_t nchunks = (a.P + slack + chunk_cols - 1) / chunk_cols;
    if (nchunks < 8) xcd_aware = 0;               // fewer chunks than XCDs: rows go round the XCDs instead
    const int nxcd = xcd_aware ? 8 : 1;
    if (own_table && !ordered) { *status = CX_ERR_SHAPE; return true; }
    std::lock_guard<std::mutex> enqueue_lock(enqueue_mutex());
    unsigned *order = nullptr;
    const int64_t order_entries = own_table ? a.order_entries : kOrderEntries;
    if (ordered && !own_table) {
        order = order_table_for(a.stream);
        if (!order) ordered = false;
    }
    int64_t cl = cl_req, least_cl = 1;
    if (cl < 1) {
        // ordered rows: the operator's visit length per XCD (shorter visits lose DRAM row
        // locality, longer ones push the previous visit out of L2);
        // natural row order: the whole cluster (all rows) should fit one XCD's 4 MB L2
        const int64_t row_bytes = chunk_cols * (16 / Op::kElems) * a.rows_per_gossip_row;
        cl = ordered ? (static_cast<int64_t>(VisitKb<Op>::of(a.n, a.P, a.S)) << 10) / row_bytes : (4 << 20) / (row_bytes * a.n);
        if (cl < 1) cl = 1;
    }
    if (ordered) {                                // the order table must fit its slot
        const int64_t max_clusters = order_entries / a.n - nxcd;
        if (max_clusters < 1) { if (own_table) { *status = CX_ERR_SHAPE; return true; } ordered = false; }
        else {
            const int64_t min_cl = (nchunks + max_clusters - 1) / max_clusters;
            if (cl < min_cl) {
                if (own_table) { *status = CX_ERR_SHAPE; return true; }       // beyond the stated maximum
                cl = min_cl;
            }
            least_cl = min_cl;
        }
    }
    if (cl_req < 1) {
        // An XCD works through every nxcd-th cluster.  Clusters are shortened until the last round of clusters
        // is as full as the others: 512 rows x 100,003 fp32 columns are 98 chunks, and clusters of the full 64
        // would put them all on two of the eight XCDs (439 us a call; dealt out evenly 89 us).
        const int64_t rounds = (nchunks + cl * nxcd - 1) / (cl * nxcd);
        cl = (nchunks + rounds * nxcd - 1) / (rounds * nxcd);
        if (cl < least_cl) cl = least_cl;
    }
    if (cl > 4096) cl = 4096;
    int64_t clusters = (nchunks + cl * nxcd - 1) / (cl * nxcd);
    if (clusters > 65535) {                       // grid.z limit: widen the clusters
        cl = (nchunks + 65535LL * nxcd - 1) / (65535LL * nxcd);
        clusters = (nchunks + cl * nxcd - 1) / (cl * nxcd);
    }
    if (cl * nxcd > 0x7fffffffLL || clusters > 65535 || a.n > 65535) { *status = CX_ERR_SHAPE; return true; }
    // the kernel numbers chunks and tiles, the grid's padding included, in 32 bits
    if ((clusters * nxcd * cl + 1) * waves > 0x7fffffffLL) { *status = CX_ERR_SHAPE; return true; }
    if (ordered && clusters * nxcd * a.n > order_entries) {        // table too large: natural row order
        if (own_table) { *status = CX_ERR_SHAPE; return true; }
        ordered = false;
    }
    // The order by the tile where the table holds it and about every kTileOrder-th cluster or more holds the edge of a
    // segment; one segment needs no words of tiles.  On long rows a tile's word is read from memory for few rows, ahead
    // of all loads (4 x 23,403,072 fp32 in 3 segments: by the cluster 137 us, by the tile 151), and clusters with an edge
    // are few.  The mean staged through LDS needs one row for a whole workgroup, which the order by the cluster gives.
    const bool edges = !LdsStaged<Op>::value && a.n >= kFewRows && static_cast<int64_t>(a.S - 1) * kTileOrder >= clusters * nxcd;
    const bool by_tile = ordered && (a.S == 1 || edges) &&
                         static_cast<int64_t>(a.S) * a.n + (a.S > 1 ? (nchunks + 1) * waves : 0) <= order_entries;
    const dim3 grid(static_cast<unsigned>(cl * nxcd), static_cast<unsigned>(a.n),
                    static_cast<unsigned>(clusters));
    const dim3 block(kWave * waves);
    const int xcd_shift = xcd_aware ? 3 : 0;
    if (!ordered) order = nullptr;
    if (ordered && own_table) {
        order = a.order_provider();
        if (!order) { *status = CX_ERR_HIP; return true; }
    }
    if (by_tile) {
        hipLaunchKernelGGL(segment_order_kernel, dim3(a.S), dim3(order_threads(a.n)), sizeof(int) * kScheduleWords(a.n), a.stream, a.n, a.P, a.S,
                           a.seg_off, a.peers, a.shift, __builtin_ctz(kWave * Op::kElems * U), slack, order);
        if (hipGetLastError() != hipSuccess) { *status = CX_ERR_HIP; return true; }
    } else if (ordered) {
        const int64_t nclusters = clusters * nxcd;
        hipLaunchKernelGGL(order_kernel, dim3(a.S), dim3(order_threads(a.n)), sizeof(int) * kScheduleWords(a.n), a.stream, a.n,
                           a.P, a.S, a.seg_off, a.peers, a.shift, cl * chunk_cols, static_cast<int>(nclusters),
                           slack, order);
        if (hipGetLastError() != hipSuccess) { *status = CX_ERR_HIP; return true; }
    }
    int cap = cx_get_tuning(9);
    if (cap < 0 || cap > 16) cap = GatherWgs<Op>::of(op) * full_waves / waves;   // the same waves per CU
    size_t glds = lds_reservation(cap);
    if (U == 1 && staged_shape<Op>(waves) && glds < LdsStaged<Op>::bytes) glds = LdsStaged<Op>::bytes;
    if (glds < static_cast<size_t>(StageBytes<Op>::value) * waves) glds = static_cast<size_t>(StageBytes<Op>::value) * waves;
    const Op staged = with_stage_base(op, 0);
    const auto launch = [&](auto kernel, const auto &rows) {
        hipLaunchKernelGGL(kernel, grid, block, glds, a.stream, rows, a.n, a.P, a.S, a.seg_off, a.peers, a.shift,
                           a.skip_mix, static_cast<unsigned>(nchunks), static_cast<unsigned>(cl),
                           static_cast<unsigned>(waves), xcd_shift, order,
                           by_tile ? 1 : 0);
    };
    if (a.P < Op::kElems) {
        if constexpr (U == 1) launch(gather_kernel<Op, U, false, true>, staged);
    } else if (std::is_same_v<Op, MeanOp<1>> && nt && ordered && (lines || (on_lines && matrix_bytes > kCachedBytes))) {
        if constexpr (std::is_same_v<Op, MeanOp<1>>) {
            if (lines) launch(gather_kernel<OnLines<ThroughOp>, U, true>, OnLines<ThroughOp>{{staged}});
            else launch(gather_kernel<ThroughOp, U, true>, ThroughOp{staged});
        }
    } else if (lines) {
        if constexpr (kMayStartOnLines<Op>) {
            if (nt) launch(gather_kernel<OnLines<Op>, U, true>, OnLines<Op>{staged});
            else launch(gather_kernel<OnLines<Op>, U, false>, OnLines<Op>{staged});
        }
    } else if (nt) launch(gather_kernel<Op, U, true>, staged);
    else launch(gather_kernel<Op, U, false>, staged);
    *status = hipGetLastError() == hipSuccess ? CX_OK : CX_ERR_HIP;
    return true;
    }
}

// ---------------------------------------------------------------------------------
// In place with the rows of a tile split over wavefronts (parts_kernel), or parts == 0: mix_kernel.  (What even_shape below
// takes does not come here.)
//
// Lengths are counted in tiles of one slice per lane and in rounds of mix_kernel, kRound tiles: one workgroup of eight
// waves on every CU, each wavefront with a tile and all rows of it.  Two parts need twice the wavefronts for half the
// rows each, so that tiles up to the middle of mix_kernel's last round take the split an odd number of half rounds where
// mix_kernel pays for a whole one, and beyond the middle both take the same and the split has its two extra rows on top.
// Time of the split over mix_kernel's, in place, several matrices in turn, on 16 to 350 rows: geometric
// mean (largest), 7,000 shapes in all:
//   tiles                    512-1,023    1,024-2,047  2,049-3,072  3,073-4,096  4,097-5,120  5,121-6,144
//   fp32 gossip              0.87 (1.00)  0.96 (1.04)  0.90 (1.01)  1.04 (1.09)  0.93 (1.00)  1.04 (1.12)
//   fp32 push-sum, copy      0.56 (0.71)  0.79 (0.98)  0.92 (0.99)  1.05 (1.11)  0.91 (0.95)  0.96 (1.05)
//   bf16 gossip              0.78 (0.95)  0.97 (1.12)  0.92 (1.03)  1.04 (1.18)  0.94 (1.05)  1.00 (1.16)
//   fp32 optimizer step      0.95 (1.10)  1.01 (1.14)  0.91 (1.02)  1.02 (1.12)  0.92 (0.97)  0.99 (1.04)
//   fp32 groups, up to four registers a row and slice
//                            0.96 (1.11)  1.05 (1.30)  0.91 (1.06)  1.04 (1.16)  0.95 (1.05)  0.99 (1.14)
//   16-bit steps and groups  0.91 (1.18)  0.99 (1.37)  0.90 (1.21)  1.03 (1.24)  0.93 (1.05)  1.03 (1.18)
// later_round() follows that.  In the first round what counts is how soon mix_kernel's wavefronts have enough loads in
// flight, and whether all its workgroups walk in lock-step, as they do in one segment (first_round()):
//   fp32 plain rows    three quarters of the round, with the copy of push-sum all of it; half below 16 rows and in push-sum
//               without the copy;
//   16-bit plain rows  all of the round with the copy and below 32 rows (beyond three quarters 0.92), three quarters, half
//               from 256 rows on (beyond half: fewer rows 0.95, more 1.01, up to 1.21);
//   fp32 steps, and groups of up to four registers  a quarter of the round from 16 rows on (400-512 tiles: 0.85), half of it
//               from 32 rows in several segments (0.90; in one 0.98, up to 1.09), the step on plain rows three quarters from
//               64 rows in several segments;
//   fp32 groups of more  half of the round in several segments (0.89), a quarter in one (up to there 0.95, to half of the
//               round 1.04, up to 1.24), less for gradient steps and below eight rows;
//   16-bit steps and groups  three quarters in several segments (0.88); in one half of it to a quarter (512-640 tiles of
//               groups 0.89, 768-1,536 0.99, up to 1.23);
//   fewer than eight rows otherwise, and fewer than 16 of fp32 steps and groups  short rows (kPartLong).
// Of 5,930 shapes drawn afterwards (60 to 9,000 tiles, 3 to 1,024 rows) 16 took more than 1.03 of mix_kernel's time, up to 1.11
// (bf16 gossip on 237 x 708,400 in one segment 167 / 150 us); a rule by length and row count alone had 130, up to 1.39.
// ---------------------------------------------------------------------------------
struct PartShape {
    int U, D, parts, tiles;
};
template <class Op>
struct PartRing {                       // the two rings that are built: short rows, long rows
    static constexpr bool kBuilt = !LdsStaged<Op>::value && Op::kRawPerSlice < 16;          // groups of 16 keep mix_kernel
    // (two slices of groups of 5 would keep registers in scratch)
    static constexpr int kLongU = fits<Op, 2, 2>() && Op::kRawPerSlice <= 4 ? 2 : 1, kLongD = std::is_same_v<Op, FusedOp> ? 4 : 2;
    static constexpr int kShortD = Op::kRawPerSlice == 1 ? 4 : 2;
};

constexpr int64_t kPartJobs = 1024, kCUs = 256;           // wavefronts
constexpr int64_t kPartLong = 400;                        // tiles of one slice per lane
constexpr int64_t kRound = kCUs * kMaxWavesPerBlock;

// Most tiles in mix_kernel's first round that are split.
template <class Op>
constexpr int64_t first_round(const Op &op, int n, bool one_segment)
{
    constexpr int kRaw = Op::kRawPerSlice;
    constexpr bool kWideRows = Op::kElems == 4, kStep = HasMomentum<Op>::value, kPlainStep = std::is_same_v<Op, FusedOp>;
    constexpr int64_t kShort = kPartLong - 1;
    const Push push = push_kind(op);
    if (kWideRows && kRaw > 1) {
        if (n < 8) return kStep && kRaw > 6 ? kRound / 16 : kRaw > 4 || (one_segment && !kPlainStep) ? kRound / 8 : kShort;
        if (n < 16) return kRaw <= 6 || !one_segment ? kShort : kRound / 8;
        if (one_segment) return kStep && kRaw > 5 ? kRound * 5 / 32 : kRound / 4;
        if (kRaw > 4) return n >= 32 ? kRound / 2 : kRound * 3 / 8;
        return kPlainStep && n >= 64 ? kRound * 3 / 4 : n >= 32 ? kRound / 2 : kRound / 4;
    }
    if (n < 8) return kShort;
    if (kRaw == 1) {
        if (kWideRows) return n < 16 || push == Push::kPlain ? kRound / 2 : push == Push::kWithCopy ? kRound : kRound * 3 / 4;
        return push == Push::kWithCopy || n < 32 ? kRound : n < 256 ? kRound * 3 / 4 : kRound / 2;
    }
    if (!one_segment) return kRound * 3 / 4;
    return kRaw <= 2 ? kRound / 2 : kRaw <= 4 ? kRound * 3 / 8 : kStep ? kRound / 4 : kRound * 5 / 16;
}

// In the first half of a later round?  Up to the round from which the walk's own time hides the difference.
template <class Op>
constexpr bool later_round(const Op &op, int n, int64_t tiles)
{
    constexpr int kRaw = Op::kRawPerSlice;
    constexpr bool kWideRows = Op::kElems == 4;
    const Push push = push_kind(op);
    const int last = !kWideRows                                     ? (kRaw == 1 || kRaw > 5 ? 3 : kRaw > 3 ? 2 : 1)
                     : std::is_same_v<Op, FusedOp>                  ? 4
                     : kRaw > 4 || (kRaw == 1 && push == Push::kPlain) ? 1
                                                                    : 3;
    if (n < (kWideRows ? 16 : 8)) return false;
    const int64_t round = kCUs * waves_with_schedules<Op>(n, kMaxWavesPerBlock), before = (tiles - 1) / round;
    return before >= 1 && before < last && 2 * (tiles - before * round) <= round;
}

template <class Op>
constexpr PartShape part_shape(const Op &op, int n, int64_t P, int S)
{
    using Ring = PartRing<Op>;
    constexpr PartShape kNone{0, 0, 0, 0};
    constexpr bool kWideRows = Op::kElems == 4, kPlainRows = Op::kRawPerSlice == 1;
    constexpr bool kGroups = kWideRows && !kPlainRows && !std::is_same_v<Op, FusedOp>;
    if (!Ring::kBuilt || n < 4 || P < Op::kElems) return kNone;
    const int64_t tiles = (P + kWave * Op::kElems - 1) / (kWave * Op::kElems);
    // up to 8 very long fp32 rows, which mix_kernel's two waves serve badly: gossip where they begin inside lines
    // (0.75 to 0.98 between 4 and 8 rows of 4.2 to 21 million columns), push-sum without the copy (0.74 to 0.90)
    const bool whole_lines = op.ld * (16 / Op::kElems) % 128 == 0;
    const Push push = push_kind(op);
    const bool few = kWideRows && kPlainRows && n <= 8 && tiles >= 8 * kRound &&
                     (push == Push::kNo ? !whole_lines : push == Push::kPlain);
    if (!few && tiles > first_round(op, n, S == 1) && !later_round(op, n, tiles)) return kNone;
    const bool long_rows = tiles >= kPartLong;
    PartShape s{long_rows ? Ring::kLongU : 1, long_rows ? Ring::kLongD : Ring::kShortD, 2, 1};
    const int limit = long_rows ? kPartWaves<Op, Ring::kLongU, Ring::kLongD> : kPartWaves<Op, 1, Ring::kShortD>;
    const int64_t jobs = (tiles + s.U - 1) / s.U;
    // As many parts as give kPartJobs wavefronts; longer rows gain from two parts, since the two rows that a part reads
    // ahead come all at once.
    while (s.parts * jobs < kPartJobs && s.parts < limit && 2 * s.parts <= n) s.parts *= 2;
    // As many adjacent tiles a workgroup as leave the last round of workgroups, one a CU, nearly as full as the others
    // (fp32 means of groups of 2 to 4 on 700 to 800 tiles: 0.95 of mix_kernel's time, with 2 parts x 4 tiles 1.40).  Beside
    // 64 rows and more one round of the widest is best whatever it leaves idle (measured on the fp32 optimizer step on
    // 256 x 300,007, 154 workgroups of 4 tiles 340 us, 593 of one tile 362; from kEvenRows rows on even_shape serves that better).  Two slices per lane of groups on longer rows: one tile each (on 2,049
    // to 3,072 tiles 0.94 with one, 0.95 with two, 1.03 with four).
    int most_full = 0;
    const int widest = s.parts >= kMaxWavesPerBlock || (kGroups && tiles > kRound) ? 1 : (n < 8 ? 4 : kMaxWavesPerBlock) / s.parts;
    for (int t = widest; t >= 1 && most_full < 90; t /= 2) {
        const int64_t blocks = (jobs + t - 1) / t + S - 1, rounds = (blocks + kCUs - 1) / kCUs;
        const int full = n >= 64 && long_rows && rounds == 1 ? 100 : static_cast<int>(100 * blocks / (rounds * kCUs));
        if (full > most_full) {
            s.tiles = t;
            most_full = full;
        }
    }
    // mix_kernel where few rows leave the split's rounds of workgroups badly filled (the workgroups of the segments' pieces
    // count: fp32 gradient step without groups on 20 x 119,800 in 32 segments, 257 workgroups, 1.32)
    const bool idle = long_rows && kWideRows && !kPlainRows && Op::kRawPerSlice <= 4 && n < 64 && most_full < 70;
    return idle ? kNone : s;
}

template <class Op>
bool launch_parts(const Op &op, const PartShape &s, const MixArgs &a)
{
    if constexpr (!PartRing<Op>::kBuilt) {
        return false;
    } else {
        const int64_t block_cols = static_cast<int64_t>(kWave) * Op::kElems * s.U * s.tiles;
        const int64_t blocks = (a.P + block_cols - 1) / block_cols + a.S - 1;
        if (blocks > 0x7fffffffLL) return false;
        const int waves = s.parts * s.tiles;
        const size_t schedule = (sizeof(int) * kScheduleWords(a.n) + 15) / 16 * 16;
        const size_t lds = schedule + static_cast<size_t>(StageBytes<Op>::value) * waves;
        const Op staged = with_stage_base(op, schedule);
        const auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kWave * waves), lds, a.stream, staged, a.n, a.P,
                               a.S, a.seg_off, a.peers, a.shift, s.parts, static_cast<unsigned>(a.S - 1));
        };
        using Ring = PartRing<Op>;
        if (s.U == Ring::kLongU && s.D == Ring::kLongD) launch(parts_kernel<Op, Ring::kLongU, Ring::kLongD>);
        else launch(parts_kernel<Op, 1, Ring::kShortD>);
        return true;
    }
}

// ---------------------------------------------------------------------------------
// In place, many plain rows of medium length: mix_kernel with as many waves a workgroup as deal the tiles out evenly.  A launch
// lasts as long as the CU with the most slices: ceil(workgroups / CUs) * waves * slices per lane.  Eight waves, or five where
// many rows' schedules fill the LDS, leave CUs idle (fp32, 300,007 columns: 1,172 tiles are 147 workgroups of eight waves, of
// the split's four tiles as well, 235 of five), so waves and slices are chosen for the least of that, and of equals the one with
// fewer, wider workgroups.  From kEvenLoad slices a CU on, below which a CU has too few wavefronts and the split or mix_kernel's
// short shapes serve, where the other shape is more than kEvenGain per cent off (at 8 slices for 7 the step on 117 x 398,433
// took 171 us for 166).  The lines for plain 16-bit rows and for long rows were drawn with two workgroups a CU whatever their size
// (831 x 943,628 899 us, 738 before; bf16 gossip on 30 x 3,322,532 94, 86 before).  With the present cap the even walk would take 0.91
// of the time beyond kEvenRows16 (0.79 to 1.06, 53 shapes); beyond kEvenMost its workgroups of three waves 0.95 to 1.09, of five
// 0.91 to 1.08, two slices 0.91 to 0.96 (77 shapes).
// The cap on resident workgroups is one on wavefronts, as in walk_shape: three waves, two / five workgroups a CU, us: fp32 gossip
// on 24 x 523,592 in 16 segments 29.1 / 24.0, bf16 gossip on 105 x 1,045,250 in 24 117 / 101, fp32 push-sum on 439 x 543,169
// 418 / 392; four to six waves and two slices are as long either way.  Steps on 16-bit rows keep two workgroups of four waves and
// more: three waves took 0.96 to 1.04 of the time of eight, five workgroups of them 0.96 to 1.07 (32 shapes of 6,423 to 6,897 slices).
// Before / now, us: fp32 optimizer step on 256 x 300,007 342 / 314; fp32 gossip on 265 x 278,339 136 / 117, on 611 x 512,664
// 525 / 474; fp32 push-sum on 171 x 1,202,009 321 / 294, on 34 x 598,370 38 / 30; bf16 gossip on 118 x 626,350 75 / 60; bf16
// optimizer step on 158 x 3,248,642 1,553 / 1,351, on 75 x 2,115,692 506 / 413.
// It takes 65 to 94 % of the lengths up to 1,535 slices (of 16-bit steps 24 %) and few of the longer ones, up to 4 %, except of fp32
// push-sum without the copy (57 % up to 3,071, 29 % up to 6,143) and 16-bit steps (28 % from 3,072 on, 10 % from 6,144 on): elsewhere
// the other shapes' CUs count as full, the split's two-wave workgroups too, though they are slower than that (fp32 optimizer step on
// 263 x 589,905 722 split, 616 in workgroups of five waves).  Time over the other shapes' on 153 shapes drawn from those it takes:
// geometric mean 0.89, 0.72 to 1.012.
// ---------------------------------------------------------------------------------
constexpr int kEvenRows = 24, kEvenRows16 = 500, kEvenLoad = 5, kEvenMost = 24, kEvenMostStep = 32, kEvenGain = 15;

// Slices on the CU with the most, workgroups of `tiles` tiles of U slices.  The workgroups of the segments' pieces count: fp32
// optimizer step on 66 x 650,762 in 20 segments, 255 workgroups and four of pieces 196 us, 171 with workgroups of eight waves.
template <class Op>
constexpr int64_t cu_load(int64_t P, int U, int tiles, int pieces)
{
    const int64_t cols = static_cast<int64_t>(kWave) * Op::kElems * U * tiles, blocks = (P + cols - 1) / cols + pieces;
    return (blocks + kCUs - 1) / kCUs * tiles * U;
}

template <class Op>
constexpr WalkShape even_shape(const Op &op, int n, int64_t P, int S)
{
    constexpr WalkShape kNone{0, 0, 0, 0};
    constexpr bool kStep = HasMomentum<Op>::value, kHalf = Op::kElems == 8;
    if (Op::kRows != 1 || n < kEvenRows || (kHalf && !kStep && n > kEvenRows16) || push_kind(op) == Push::kWithCopy) return kNone;
    const int64_t slices = (P + kWave * Op::kElems - 1) / (kWave * Op::kElems);
    if (slices <= (kEvenLoad - 1) * kCUs || slices > (kStep ? kEvenMostStep : kEvenMost) * kCUs) return kNone;
    WalkShape best = kNone;
    int64_t least = 0;
    for (int U = 1; U <= Op::kWalk.U; ++U)
        for (int waves = kHalf && kStep ? 4 : 3; waves <= waves_with_schedules<Op>(n, kMaxWavesPerBlock); ++waves) {
            const int64_t load = cu_load<Op>(P, U, waves, (S - 1 + waves - 1) / waves);
            if (best.U && (load > least || (load == least && waves * U <= best.waves * best.U))) continue;
            least = load;
            best = WalkShape{U, 0, waves, kHalf && kStep ? 2 : 2 * kMaxWavesPerBlock / waves};
        }
    if (!best.U) return kNone;
    // where the split serves, few waves of a narrow tile each do not replace it (fp32 gossip and optimizer step, three waves 1.02 of
    // the split's time, 0.93 to 1.07, four 0.99; plain 16-bit rows would gain, 0.91, 0.85 to 0.95: 26 shapes)
    const PartShape split = part_shape(op, n, P, S);
    if (split.parts && (kHalf ? best.waves : best.waves * best.U) < kEvenLoad) return kNone;
    // The first workgroup of pieces does not count for the walk as it is otherwise: beside a full round of tiles it makes no round
    // of its own, since few of its wavefronts have a piece.  That walk, 256 workgroups and one / three or four waves, us: bf16 gossip
    // on 115 x 1,047,248 in two segments 94 / 121, fp32 optimizer step on 119 x 522,620 in 8 243 / 268; of 83 such shapes of gossip
    // and steps three or four waves took 0.92 to 1.29 of its time, beside more workgroups of pieces 0.74 to 1.0.
    const WalkShape whole = walk_shape(op, n, P);
    const int pieces = (S - 1 + whole.waves - 1) / whole.waves;
    const int64_t usual = split.parts ? cu_load<Op>(P, split.U, split.tiles, S - 1)
                                      : cu_load<Op>(P, whole.U, whole.waves, pieces > 1 ? pieces - 1 : 0);
    if (100 * usual <= (100 + kEvenGain) * least) return kNone;
    best.D = kStep ? (kHalf ? 2 : 4) : push_kind(op) == Push::kPlain && best.U == 2 ? 2 : kHalf ? 4 : 8;
    return best;
}

// What serves a call in place: the split (parts.parts > 0), or mix_kernel in `walk`, which `even` says is even_shape's.
struct InPlaceShape {
    PartShape parts;
    WalkShape walk;
    bool even;
};
template <class Op>
constexpr InPlaceShape in_place_shape(const Op &op, int n, int64_t P, int S)
{
    const WalkShape even = even_shape(op, n, P, S);
    if (even.U) return InPlaceShape{{0, 0, 0, 0}, even, true};
    return InPlaceShape{part_shape(op, n, P, S), walk_shape(op, n, P), false};
}

template <class Op>
int launch_mix(const Op &op, const MixArgs &a)
{
    constexpr int U0 = Op::kWalk.U, D0 = Op::kWalk.D;
    static_assert(fits<Op, U0, D0>(), "default launch shape must fit");
    static_assert(fits<Op, 1, 2>(), "the shape of rows shorter than a tile must fit");
    if ((a.P + 255) / 256 > 0x7fffffffLL) return CX_ERR_SHAPE;
    constexpr int64_t kSliceLanes = static_cast<int64_t>(kWave) * Op::kElems;   // a tile of one slice per lane
    // Rows shorter than a tile take one slice per lane, rows shorter than a slice the short-row kernels (in
    // place: shape 1/2): the tile at the row end has nothing to slide over otherwise (cx_columns.hpp).
    if (a.out_of_place && cx_get_tuning(5) != 1) {
        int u = cx_get_tuning(0);
        if (u != 1 && u != 2 && u != 4) u = Op::kGather.U;
        while (u > 1 && Op::kRawPerSlice * u > 8) u >>= 1;   // the rows in flight must fit the registers
        if (Op::kRawPerSlice >= 8 || u > MaxSlices<Op>::value || a.P < kSliceLanes * u) u = 1;
        int waves = cx_get_tuning(1);
        const bool waves_fixed = waves >= 1 && waves <= kMaxWavesPerBlock;
        if (!waves_fixed) waves = Op::kGather.waves;
        const int nt = cx_get_tuning(2) == 0 ? 0 : 1;
        const int cl = cx_get_tuning(6);
        const int xcd_aware = cx_get_tuning(7) == 0 ? 0 : 1;
        int status = CX_OK;
        if (try_gather<Op, 1>(op, u, waves, waves_fixed, nt, cl, xcd_aware, a, &status) ||
            try_gather<Op, 2>(op, u, waves, waves_fixed, nt, cl, xcd_aware, a, &status) ||
            try_gather<Op, 4>(op, u, waves, waves_fixed, nt, cl, xcd_aware, a, &status))
            return status;
    }
    bool as_tuned = a.skip_mix != 0;                       // launch parameters of the in-place kernel ask for mix_kernel's shapes
    for (const int key : {0, 1, 2, 3, 4, 9}) as_tuned = as_tuned || cx_get_tuning(key) != -1;
    const InPlaceShape shape = as_tuned ? InPlaceShape{{0, 0, 0, 0}, walk_shape(op, a.n, a.P), false} : in_place_shape(op, a.n, a.P, a.S);
    if (shape.parts.parts && launch_parts<Op>(op, shape.parts, a)) return hipGetLastError() == hipSuccess ? CX_OK : CX_ERR_HIP;
    Launch l = pick_launch(shape.walk);
    if (a.P < kSliceLanes * l.U) l.U = 1;
    if (a.P < Op::kElems) l.D = 2;
    const bool done =
        try_launch<Op, 1, 2>(op, l, a) || try_launch<Op, 1, 4>(op, l, a) || try_launch<Op, 1, 8>(op, l, a) ||
        try_launch<Op, 2, 2>(op, l, a) || try_launch<Op, 2, 4>(op, l, a) || try_launch<Op, 2, 8>(op, l, a) ||
        try_launch<Op, 4, 2>(op, l, a) || try_launch<Op, 4, 4>(op, l, a) || try_launch<Op, 4, 8>(op, l, a);
    if (!done) {                     // requested shape not built for this operator
        const bool narrow = a.P < kSliceLanes * U0;
        l.U = narrow ? 1 : U0;
        l.D = narrow ? 2 : D0;
        if (!try_launch<Op, U0, D0>(op, l, a)) try_launch<Op, 1, 2>(op, l, a);
    }
    return hipGetLastError() == hipSuccess ? CX_OK : CX_ERR_HIP;
}

[[maybe_unused]] int check_matrix_args(const void *x_in, const void *x_out, int64_t ld, int64_t rows,
                                       int64_t P, int32_t S, uint32_t flags, int elem_bytes = 4)
{
    if (!x_in || !x_out) return CX_ERR_NULL;
    if (S < 1 || P < 1 || ld < P || rows < 1) return CX_ERR_SHAPE;
    if (rows > (INT64_MAX / 4) / ld) return CX_ERR_SHAPE;
    if (ld % (16 / elem_bytes) != 0 || misaligned(x_in) || misaligned(x_out)) return CX_ERR_ALIGN;
    if (partial_overlap(x_in, x_out, static_cast<uint64_t>(rows) * ld * elem_bytes)) return CX_ERR_ALIAS;
    if (flags != 0) return CX_ERR_UNSUPPORTED;
    return CX_OK;
}

}  // namespace

#endif  // CX_LAUNCH_HPP
