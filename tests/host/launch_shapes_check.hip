// Launch shapes that the entry points choose, checked at compile time (host half only; nothing here runs).
#include "cx_launch.hpp"

namespace {

// The mean staged through LDS is laid out for workgroups of eight waves: it keeps them on every row length, the
// lengths of the tests that run it (6,007 and 150,001 columns) among them, while the sum in registers takes fewer.
static_assert(gather_waves<MeanLdsOp<8>, 1>(6007, MeanLdsOp<8>::kGather.waves) == 8);
static_assert(gather_waves<MeanLdsOp<8>, 1>(150001, MeanLdsOp<8>::kGather.waves) == 8);
static_assert(staged_shape<MeanLdsOp<8>>(MeanLdsOp<8>::kGather.waves) && !staged_shape<MeanLdsOp<8>>(4));
static_assert(gather_waves<MeanOp<8>, 1>(150001, MeanOp<8>::kGather.waves) == 4 && !staged_shape<MeanOp<8>>(8));

// In place, as many wavefronts per CU whatever the workgroup's size: two workgroups of eight, or eight of two where
// rows are short or 1,024 rows' schedules leave no room for more.
template <class Op>
constexpr WalkShape shape(int n, int64_t P, int64_t ld, Op op = Op{})
{
    op.ld = ld;
    return walk_shape(op, n, P);
}
constexpr bool is(const WalkShape &s, int U, int D, int waves, int wgs_per_cu)
{
    return s.U == U && s.D == D && s.waves == waves && s.wgs_per_cu == wgs_per_cu;
}
static_assert(is(shape<MeanOp<1>>(1024, 600003, 600032), 1, 8, 2, 8) && is(shape<MeanOp<1>>(1024, 600003, 600008), 1, 8, 2, 8));
static_assert(is(shape<PushOp>(1024, 11689511, 11689512), 2, 8, 2, 8) && is(shape<FusedOp>(12, 110003, 110004), 1, 8, 2, 8));

// Long rows: two waves where rows begin on 128-byte lines (11,689,536 fp32 columns: a multiple of 32) and there are
// few of them, eight where they begin inside lines.
static_assert(is(shape<MeanOp<1>>(64, 11689511, 11689536), 2, 2, 2, 2) && is(shape<MeanOp<1>>(64, 11689511, 11689512), 2, 8, 8, 2));
static_assert(is(shape<MeanOp<1>>(32, 25557032, 25557056), 1, 2, 2, 8) && is(shape<MeanOp<1>>(32, 25557032, 25557032), 2, 4, 2, 2) &&
              is(shape<MeanOp<1>>(32, 2000003, 2000032), 1, 4, 8, 2));
static_assert(is(shape<MeanOp<4>>(16, 11689511, 11689536), 1, 4, 2, 2) && is(shape<MeanOp<4>>(16, 11689511, 11689512), 2, 2, 8, 2));
static_assert(is(shape<MeanOp<4>>(8, 11689511, 11689512), 1, 2, 2, 2) && is(shape<MeanOp<4>>(64, 11689511, 11689536), 2, 2, 8, 2));
static_assert(is(shape<HierFusedOp<8>>(8, 11689511, 11689536), 1, 2, 2, 2) && is(shape<HierFusedOp<8>>(8, 11689511, 11689512), 1, 2, 8, 2));
static_assert(is(shape<MeanOp<8>>(4, 900001, 900032), 1, 4, 8, 2) && is(shape<FusedOp>(32, 900001, 900032), 1, 8, 8, 2));
static_assert(is(shape<PushOp>(64, 25557032, 25557056), 2, 2, 2, 2) && is(shape<PushOp>(128, 25557032, 25557056), 2, 8, 8, 2));
static_assert(is(shape<MeanOp<16>>(4, 11689511, 11689536), 1, 2, 8, 2) && is(shape<Row16Op<false, 4>>(16, 11689511, 11689536), 1, 2, 8, 2));

// Plain rows: eight rows in flight beside many rows, or where tiles are few.
static_assert(is(shape<Row16Op<false>>(256, 3000003, 3000008), 1, 8, 8, 2) && is(shape<Row16Op<false>>(64, 3000003, 3000008), 1, 4, 8, 2) &&
              is(shape<Row16Op<false>>(16, 3000003, 3000008), 1, 4, 8, 2) && is(shape<Row16Op<false>>(3, 100003, 100008), 1, 8, 1, 16) &&
              is(shape<MeanOp<1>>(3, 100003, 100032), 1, 8, 2, 8));

// In place with a tile's rows split over wavefronts: as many parts as make kPartJobs wavefronts and the rows and the
// registers allow, as many tiles a workgroup as fill the last round of workgroups; mix_kernel elsewhere.
template <class Op>
constexpr bool parts_are(int n, int64_t P, int S, int U, int D, int parts, int tiles, int64_t ld = 0, Op op = Op{})
{
    op.ld = ld ? ld : P + 4;
    const PartShape s = part_shape(op, n, P, S);
    return s.parts == parts && (parts == 0 || (s.U == U && s.D == D && s.tiles == tiles));
}
template <class Op>
constexpr bool no_parts(int n, int64_t P, int S, int64_t ld = 0)
{
    return parts_are<Op>(n, P, S, 0, 0, 0, 0, ld);
}
static_assert(parts_are<MeanOp<1>>(512, 3001, 4, 1, 4, 16, 1) && parts_are<MeanOp<1>>(9, 3001, 4, 1, 4, 8, 1) &&
              parts_are<FusedOp>(4, 2000, 4, 1, 2, 4, 1) && no_parts<FusedOp>(3, 2000, 4));
static_assert(parts_are<MeanOp<1>>(16, 256 * 399, 1, 1, 4, 4, 2) && parts_are<MeanOp<1>>(16, 256 * 399 + 1, 1, 2, 2, 8, 1) &&
              no_parts<MeanOp<1>>(7, 256 * 399 + 1, 1) && no_parts<FusedOp>(15, 256 * 399 + 1, 1));
static_assert(parts_are<FusedOp>(256, 300007, 8, 2, 4, 2, 4) && no_parts<MeanOp<1>>(33, 800003, 7) &&
              parts_are<MeanOp<4>>(33, 1100003, 7, 2, 2, 2, 1));
static_assert(parts_are<MeanOp<1>>(8, 6000011, 7, 2, 2, 2, 4) && no_parts<MeanOp<1>>(8, 6000011, 7, 6000032) && no_parts<MeanOp<1>>(9, 6000011, 7));
static_assert(parts_are<Row16Op<true, 4>>(16, 400009, 7, 1, 2, 2, 4) && no_parts<Row16Op<true, 4>>(16, 4000009, 7) &&
              parts_are<Row16Op<true, 8>>(16, 2100003, 7, 1, 2, 2, 1) && no_parts<Row16Op<false>>(32, 25557032, 8));
static_assert(no_parts<MeanOp<16>>(32, 3001, 4) && kPartWaves<MeanOp<1>, 1, 4> == 16 && kPartWaves<FusedOp, 2, 4> == 8);

float a_copy;
constexpr PushOp with_copy()
{
    PushOp op{};
    op.zout = &a_copy;
    return op;
}
static_assert(parts_are<PushOp>(64, 256 * 2048, 1, 2, 2, 2, 4, 0, with_copy()) && parts_are<PushOp>(9, 256 * 1025, 1, 0, 0, 0, 0, 0, with_copy()));

// The short shapes of mix_kernel above are those of calls that are not split.
static_assert(no_parts<MeanOp<1>>(1024, 600003, 8) && no_parts<FusedOp>(12, 110003, 8) && no_parts<Row16Op<false>>(3, 100003, 8) &&
              no_parts<MeanOp<1>>(3, 100003, 8) && no_parts<MeanOp<8>>(4, 900001, 8) && no_parts<FusedOp>(32, 900001, 1) &&
              no_parts<Row16Op<false>>(64, 3000003, 8) && no_parts<MeanOp<1>>(32, 2000003, 8));

// Shapes that the split slowed by 5 to 32 per cent stay whole.
static_assert(no_parts<Row16Op<false>>(500, 650003, 8) && no_parts<Row16Op<false>>(500, 1500003, 8) && no_parts<HierFusedOp<8>>(5, 60007, 4) &&
              no_parts<HierFused16Op<true, 8>>(64, 828274, 1) && no_parts<Row16Op<false, 4>>(10, 884531, 1) &&
              parts_are<PushOp>(200, 840693, 1, 0, 0, 0, 0, 0, with_copy()) && no_parts<HierFusedOp<8>>(33, 139500, 1) && no_parts<HierFusedOp<1>>(20, 119800, 32));

// Every length of a stretch takes one answer: in the first half of mix_kernel's second and third round the split, one tile a
// workgroup for groups, in the second halves mix_kernel; many rows, whose schedules leave a workgroup fewer waves, have
// shorter rounds.
template <class Op>
constexpr bool all_lengths(int n, int S, int64_t from, int64_t to, bool split, int tiles_a_workgroup = 0)
{
    for (int64_t tiles = from; tiles <= to; tiles += 7) {
        Op op{};
        op.ld = tiles * kWave * Op::kElems + 8;
        const PartShape s = part_shape(op, n, tiles * kWave * Op::kElems, S);
        if ((s.parts != 0) != split || (split && tiles_a_workgroup && s.tiles != tiles_a_workgroup)) return false;
    }
    return true;
}
static_assert(all_lengths<MeanOp<4>>(33, 7, 2049, 3072, true, 1) && all_lengths<MeanOp<4>>(33, 7, 3073, 4096, false) &&
              all_lengths<MeanOp<4>>(33, 7, 4097, 5120, true, 1) && all_lengths<MeanOp<4>>(33, 7, 5121, 20000, false) &&
              all_lengths<MeanOp<4>>(33, 7, 1025, 2048, false) && all_lengths<MeanOp<4>>(64, 7, 400, 1024, true));
static_assert(all_lengths<MeanOp<1>>(64, 8, 20, 1536, true) && all_lengths<MeanOp<1>>(64, 8, 1537, 2048, false) &&
              all_lengths<MeanOp<1>>(64, 8, 2049, 3072, true) && all_lengths<MeanOp<1>>(64, 8, 3073, 4096, false) &&
              all_lengths<HierFusedOp<8>>(33, 1, 321, 20000, false) && all_lengths<Row16Op<true, 2>>(33, 8, 1537, 20000, false));
static_assert(all_lengths<MeanOp<1>>(500, 1, 1537, 2304, true) && all_lengths<MeanOp<1>>(500, 1, 2305, 3072, false));
static_assert(all_lengths<FusedOp>(64, 8, 6145, 7168, true) && all_lengths<FusedOp>(64, 8, 7169, 20000, false) &&
              all_lengths<FusedOp>(15, 8, 400, 20000, false) && all_lengths<PushOp>(64, 1, 1025, 20000, false));

// Visits of the out-of-place kernel, KB: longer ones of operators on groups only where they gain.  Seven rows in segments shorter
// than `cols` and of that length, seven rows in one segment, eight and nine rows in many.
template <class Op>
constexpr bool visits(int cut, int whole, int eight, int nine, int64_t cols = 655360)
{
    using Kb = VisitKb<Op>;
    return Kb::of(7, cols * 5 - 1, 5) == cut && Kb::of(7, cols * 5, 5) == whole && Kb::of(7, 1000, 1) == whole &&
           Kb::of(8, cols, 5) == eight && Kb::of(9, cols, 5) == nine;
}
static_assert(visits<Row16Op<false, 8>>(384, 384, 384, 1024) && visits<Row16Op<true, 7>>(384, 384, 384, 896) && visits<Row16Op<true, 6>>(384, 768, 768, 768) &&
              visits<Row16Op<false, 5>>(384, 384, 384, 384) && visits<Row16Op<true, 4>>(256, 512, 512, 512) && visits<Row16Op<true, 3>>(256, 256, 256, 256) &&
              visits<Row16Op<false, 1>>(96, 96, 96, 96) && visits<Push16Op<true>>(192, 192, 192, 192));
static_assert(visits<HierFused16Op<false, 8>>(384, 384, 384, 384, 655359) && visits<HierFused16Op<true, 8>>(384, 384, 384, 384, 599999) &&
              VisitKb<HierFused16Op<false, 8>>::of(8, 5 * 655360, 5) == 512 && VisitKb<HierFused16Op<true, 8>>::of(8, 5 * 655360 - 1, 5) == 384 &&
              VisitKb<HierFused16Op<true, 8>>::of(40, 3000000, 1) == 512 && VisitKb<HierFused16Op<true, 8>>::of(40, 2999999, 1) == 384 &&
              VisitKb<HierFused16Op<true, 8>>::of(7, 9000000, 1) == 384 &&
              visits<HierFused16Op<true, 7>>(384, 384, 384, 384) &&
              visits<HierFused16Op<true, 5>>(384, 384, 384, 384) && visits<HierFused16Op<false, 3>>(256, 256, 256, 256));
static_assert(visits<HierFusedOp<8>>(256, 1024, 1024, 1024, 131072) && visits<HierFusedOp<7>>(768, 768, 768, 768) && visits<HierFusedOp<5>>(768, 768, 768, 768) &&
              visits<HierFusedOp<16>>(256, 256, 256, 768) && visits<MeanOp<8>>(256, 512, 512, 768, 65536) && visits<MeanOp<16>>(256, 256, 256, 768) &&
              visits<MeanLdsOp<8>>(256, 512, 512, 768, 65536) && visits<MeanOp<1>>(256, 256, 256, 256));

// Tiles on the rows' own lines: not plain 16-bit gossip and push-sum, which they slow; no operator on groups.
uint16_t a_copy16;
constexpr Push16Op<true> with_copy16()
{
    Push16Op<true> op{};
    op.zout = &a_copy16;
    return op;
}
static_assert(starts_on_lines(MeanOp<1>{}) && starts_on_lines(FusedOp{}) && starts_on_lines(Fused16Op<false>{}) && starts_on_lines(PushOp{}) &&
              starts_on_lines(with_copy()) && starts_on_lines(with_copy16()) && starts_on_lines(HierFusedOp<1>{}));
static_assert(!starts_on_lines(Row16Op<false>{}) && !starts_on_lines(Row16Op<true>{}) && !starts_on_lines(Push16Op<true>{}) &&
              !starts_on_lines(MeanOp<2>{}) && !starts_on_lines(HierFused16Op<false, 8>{}));

// What serves a call in place: the split, mix_kernel with the tiles dealt out evenly, or mix_kernel in walk_shape above.  (The checks
// above are of part_shape by itself, which the launch asks where even_shape takes nothing.)
template <class Op>
constexpr InPlaceShape in_place(int n, int64_t P, int S, int64_t ld = 0, Op op = Op{})
{
    op.ld = ld ? ld : P + 4;
    return in_place_shape(op, n, P, S);
}
template <class Op>
constexpr bool split_is(int n, int64_t P, int S, int U, int D, int parts, int tiles, int64_t ld = 0, Op op = Op{})
{
    const PartShape s = in_place(n, P, S, ld, op).parts;
    return s.parts == parts && s.U == U && s.D == D && s.tiles == tiles;
}
template <class Op>
constexpr bool even_is(int n, int64_t P, int S, int U, int D, int waves, int wgs_per_cu, Op op = Op{})
{
    const InPlaceShape s = in_place(n, P, S, 0, op);
    return s.even && s.parts.parts == 0 && is(s.walk, U, D, waves, wgs_per_cu);
}
template <class Op>
constexpr bool walks(int n, int64_t P, int S, int64_t ld = 0, Op op = Op{})
{
    const InPlaceShape s = in_place(n, P, S, ld, op);
    return s.parts.parts == 0 && !s.even;
}
template <class Op>
constexpr bool not_split(int n, int64_t P, int S, Op op = Op{})
{
    return in_place(n, P, S, 0, op).parts.parts == 0;
}

// The split: as many parts as make kPartJobs wavefronts and the rows and the registers allow, as many tiles a workgroup as
// fill the last round of workgroups.
static_assert(split_is<MeanOp<1>>(512, 3001, 4, 1, 4, 16, 1) && split_is<MeanOp<1>>(9, 3001, 4, 1, 4, 8, 1) &&
              split_is<FusedOp>(4, 2000, 4, 1, 2, 4, 1) && walks<FusedOp>(3, 2000, 4));
static_assert(split_is<MeanOp<1>>(16, 256 * 399, 1, 1, 4, 4, 2) && split_is<MeanOp<1>>(16, 256 * 399 + 1, 1, 2, 2, 8, 1) &&
              walks<MeanOp<1>>(7, 256 * 399 + 1, 1) && walks<FusedOp>(15, 256 * 399 + 1, 1));
static_assert(split_is<FusedOp>(64, 256 * 1024, 8, 2, 4, 2, 4) && walks<MeanOp<1>>(33, 800003, 7) &&
              split_is<MeanOp<4>>(33, 1100003, 7, 2, 2, 2, 1));
static_assert(split_is<MeanOp<1>>(8, 6000011, 7, 2, 2, 2, 4) && walks<MeanOp<1>>(8, 6000011, 7, 6000032) && walks<MeanOp<1>>(9, 6000011, 7));
static_assert(split_is<Row16Op<true, 4>>(16, 400009, 7, 1, 2, 2, 4) && walks<Row16Op<true, 4>>(16, 4000009, 7) &&
              split_is<Row16Op<true, 8>>(16, 2100003, 7, 1, 2, 2, 1) && walks<Row16Op<false>>(32, 25557032, 8));
static_assert(walks<MeanOp<16>>(32, 3001, 4) && kPartWaves<MeanOp<1>, 1, 4> == 16 && kPartWaves<FusedOp, 2, 4> == 8);

static_assert(split_is<PushOp>(64, 256 * 2048, 1, 2, 2, 2, 4, 0, with_copy()) && walks<PushOp>(9, 256 * 1025, 1, 0, with_copy()));

// The short shapes of mix_kernel above are those of calls that are not split.
static_assert(walks<MeanOp<1>>(1024, 600003, 8) && walks<FusedOp>(12, 110003, 8) && walks<Row16Op<false>>(3, 100003, 8) &&
              walks<MeanOp<1>>(3, 100003, 8) && walks<MeanOp<8>>(4, 900001, 8) && walks<FusedOp>(32, 900001, 1) &&
              walks<Row16Op<false>>(64, 3000003, 8) && walks<MeanOp<1>>(32, 2000003, 8));

// Shapes that the split slowed by 5 to 32 per cent are not split.
static_assert(not_split<Row16Op<false>>(500, 650003, 8) && walks<Row16Op<false>>(500, 1500003, 8) && walks<HierFusedOp<8>>(5, 60007, 4) &&
              walks<HierFused16Op<true, 8>>(64, 828274, 1) && walks<Row16Op<false, 4>>(10, 884531, 1) &&
              walks<PushOp>(200, 840693, 1, 0, with_copy()) && walks<HierFusedOp<8>>(33, 139500, 1) && walks<HierFusedOp<1>>(20, 119800, 32));

// Every length of a stretch takes one answer, those aside that the even walk takes: in the first half of mix_kernel's second and third round the split, one tile a
// workgroup for groups, in the second halves mix_kernel; many rows, whose schedules leave a workgroup fewer waves, have
// shorter rounds.
template <class Op>
constexpr bool all_calls(int n, int S, int64_t from, int64_t to, bool split, int tiles_a_workgroup = 0)
{
    for (int64_t tiles = from; tiles <= to; tiles += 7) {
        Op op{};
        op.ld = tiles * kWave * Op::kElems + 8;
        const InPlaceShape shape = in_place_shape(op, n, tiles * kWave * Op::kElems, S);
        if (shape.even) continue;
        const PartShape s = shape.parts;
        if ((s.parts != 0) != split || (split && tiles_a_workgroup && s.tiles != tiles_a_workgroup)) return false;
    }
    return true;
}
static_assert(all_calls<MeanOp<4>>(33, 7, 2049, 3072, true, 1) && all_calls<MeanOp<4>>(33, 7, 3073, 4096, false) &&
              all_calls<MeanOp<4>>(33, 7, 4097, 5120, true, 1) && all_calls<MeanOp<4>>(33, 7, 5121, 20000, false) &&
              all_calls<MeanOp<4>>(33, 7, 1025, 2048, false) && all_calls<MeanOp<4>>(64, 7, 400, 1024, true));
static_assert(all_calls<MeanOp<1>>(64, 8, 20, 1536, true) && all_calls<MeanOp<1>>(64, 8, 1537, 2048, false) &&
              all_calls<MeanOp<1>>(64, 8, 2049, 3072, true) && all_calls<MeanOp<1>>(64, 8, 3073, 4096, false) &&
              all_calls<HierFusedOp<8>>(33, 1, 321, 20000, false) && all_calls<Row16Op<true, 2>>(33, 8, 1537, 20000, false));
static_assert(all_calls<MeanOp<1>>(500, 1, 1537, 2304, true) && all_calls<MeanOp<1>>(500, 1, 2305, 3072, false));
static_assert(all_calls<FusedOp>(64, 8, 6145, 7168, true) && all_calls<FusedOp>(64, 8, 7169, 20000, false) &&
              all_calls<FusedOp>(15, 8, 400, 20000, false) && all_calls<PushOp>(64, 1, 1025, 20000, false));

// The even walk: from 24 plain rows on, at 1,025 slices of 256 or 512 columns and more; mix_kernel with the waves that leave
// the busiest CU the fewest slices, and as many wavefronts on a CU whatever the workgroup's size.
static_assert(even_is<FusedOp>(256, 300007, 8, 1, 4, 5, 3) && even_is<MeanOp<1>>(265, 278339, 4, 1, 8, 5, 3) &&
              even_is<MeanOp<1>>(24, 256 * 1025, 3, 1, 8, 5, 3) && !in_place<MeanOp<1>>(23, 256 * 1025, 3).even &&
              !in_place<MeanOp<1>>(24, 256 * 1024, 3).even && !in_place<MeanOp<2>>(256, 300007, 8).even &&
              !in_place<PushOp>(256, 300007, 1, 0, with_copy()).even);
static_assert(even_is<Row16Op<false>>(500, 512 * 1025, 1, 1, 4, 5, 3) && !in_place<Row16Op<false>>(501, 512 * 1025, 1).even &&
              even_is<Fused16Op<true>>(24, 512 * 1025, 1, 1, 2, 5, 2));
// One workgroup of the segments' pieces beside a full round of tiles does not make a second round; several do.
static_assert(walks<Row16Op<false>>(115, 1047248, 2) && walks<FusedOp>(119, 522620, 8) && walks<MeanOp<1>>(29, 523264, 8) &&
              walks<MeanOp<1>>(30, 1047296, 3) && even_is<MeanOp<1>>(163, 522496, 16, 1, 8, 3, 5) &&
              even_is<FusedOp>(98, 523520, 16, 1, 4, 3, 5) && !even_is<FusedOp>(66, 650762, 20, 2, 4, 5, 3));
// Every count of waves and slices that the rule chooses: the calls of test_gpu_even_walk.py that are there for it.
static_assert(even_is<MeanOp<1>>(24, 522735, 17, 1, 8, 3, 5) && even_is<MeanOp<1>>(512, 323055, 17, 2, 8, 3, 5) && even_is<MeanOp<1>>(400, 455919, 17, 2, 8, 4, 4) &&
              even_is<MeanOp<1>>(400, 688623, 1, 2, 8, 6, 2));
static_assert(even_is<Row16Op<false>>(33, 1045487, 17, 1, 4, 3, 5) && even_is<Row16Op<true>>(24, 1033199, 17, 1, 4, 8, 2) &&
              even_is<Row16Op<false>>(400, 911855, 17, 2, 4, 4, 4));
static_assert(even_is<FusedOp>(24, 390639, 8, 1, 4, 3, 5) && even_is<FusedOp>(512, 323055, 17, 2, 4, 3, 5) && even_is<FusedOp>(400, 455919, 17, 2, 4, 4, 4));
static_assert(even_is<Fused16Op<true>>(24, 2612207, 17, 1, 2, 4, 2) && even_is<Fused16Op<false>>(24, 656879, 1, 1, 2, 6, 2) &&
              even_is<Fused16Op<true>>(24, 524783, 1, 1, 2, 5, 2));
static_assert(even_is<PushOp>(24, 525039, 1, 1, 8, 3, 5) && even_is<PushOp>(24, 590319, 1, 2, 2, 5, 3) && even_is<PushOp>(24, 655599, 1, 2, 2, 6, 2) &&
              even_is<PushOp>(400, 458991, 1, 2, 2, 4, 4) && even_is<Push16Op<false>>(64, 656879, 1, 1, 4, 6, 2));
// That test's calls at both ends of the rule: whole slices, columns beyond them, segments (push-sum has one).
template <class Op>
constexpr bool even_at(int n, int slices, int beyond, int S)
{
    return in_place<Op>(n, static_cast<int64_t>(slices) * kWave * Op::kElems + beyond, S).even;
}
static_assert(even_at<MeanOp<1>>(24, 1024, 1, 3) && even_at<MeanOp<1>>(120, 1172, -25, 8) && even_at<MeanOp<1>>(101, 1172, 3, 40) && even_at<MeanOp<1>>(513, 1030, 9, 5) &&
              even_at<FusedOp>(24, 1024, 1, 3) && even_at<FusedOp>(120, 1172, -25, 8) && even_at<FusedOp>(25, 1279, 77, 30) && even_at<FusedOp>(513, 1030, 9, 5) &&
              even_at<PushOp>(24, 1024, 1, 1) && even_at<PushOp>(25, 1279, 77, 1) && even_at<Row16Op<true>>(24, 1024, 1, 3) && even_at<Row16Op<true>>(101, 1172, 3, 40) &&
              even_at<Push16Op<true>>(24, 1024, 1, 1) && even_at<Push16Op<true>>(25, 1279, 77, 1));
static_assert(!even_at<MeanOp<1>>(23, 1024, 1, 3) && !even_at<MeanOp<1>>(25, 1279, 77, 30) && !even_at<MeanOp<1>>(26, 6143, 5, 2) &&
              !even_at<FusedOp>(23, 1024, 1, 3) && !even_at<Row16Op<true>>(513, 1030, 9, 5) && !even_at<Fused16Op<true>>(24, 1024, 1, 3));
// Its last lengths: 6,144 slices, steps 8,192.
static_assert(even_at<MeanOp<1>>(480, 6144, 0, 24) && !even_at<MeanOp<1>>(480, 6144, 1, 24) && even_at<PushOp>(400, 6144, 0, 1) && !even_at<PushOp>(400, 6144, 1, 1) &&
              even_at<FusedOp>(200, 8192, 0, 24) && !even_at<FusedOp>(200, 8192, 1, 24));

// Steps on 16-bit rows: no workgroups of three waves.
static_assert(walks<Fused16Op<false>>(61, 3505152, 2));

}  // namespace
