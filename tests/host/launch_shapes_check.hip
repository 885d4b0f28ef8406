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

}  // namespace
