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
static_assert(is(shape<MeanOp<1>>(1024, 300007, 300032), 1, 8, 2, 8) && is(shape<MeanOp<1>>(1024, 300007, 300008), 1, 8, 2, 8));
static_assert(is(shape<PushOp>(1024, 11689511, 11689512), 2, 8, 2, 8) && is(shape<FusedOp>(256, 100003, 100004), 1, 8, 2, 8));

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
              is(shape<Row16Op<false>>(16, 3000003, 3000008), 1, 4, 8, 2) && is(shape<Row16Op<false>>(16, 100003, 100008), 1, 8, 1, 16) &&
              is(shape<MeanOp<1>>(16, 100003, 100032), 1, 8, 2, 8));

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
static_assert(parts_are<FusedOp>(256, 300007, 8, 2, 4, 2, 4) && no_parts<MeanOp<4>>(33, 515003, 7) && no_parts<MeanOp<1>>(33, 800003, 7) &&
              parts_are<MeanOp<4>>(33, 1100003, 7, 2, 2, 2, 1) && parts_are<MeanOp<1>>(33, 515003, 7, 2, 2, 2, 2));
static_assert(parts_are<MeanOp<1>>(8, 6000011, 7, 2, 2, 2, 4) && no_parts<MeanOp<1>>(8, 6000011, 7, 6000032) && no_parts<MeanOp<1>>(9, 6000011, 7));
static_assert(parts_are<Row16Op<true, 4>>(16, 400009, 7, 1, 2, 2, 4) && no_parts<Row16Op<true, 4>>(16, 4000009, 7) &&
              parts_are<Row16Op<true, 8>>(16, 2100003, 7, 1, 2, 2, 1) && no_parts<Row16Op<false>>(32, 25557032, 8));
static_assert(no_parts<MeanOp<16>>(32, 3001, 4) && kPartWaves<MeanOp<1>, 1, 4> == 16 && kPartWaves<FusedOp, 2, 4> == 8);

}  // namespace
