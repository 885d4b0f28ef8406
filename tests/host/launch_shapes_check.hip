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
// 1,024 rows' schedules leave no room for more.
constexpr bool same_waves_per_cu(const WalkShape &s) { return s.wgs_per_cu * s.waves == 16; }
static_assert(walk_shape<MeanOp<1>>(256, 11689511).waves == 8 && same_waves_per_cu(walk_shape<MeanOp<1>>(256, 11689511)));
static_assert(walk_shape<MeanOp<1>>(1024, 300007).waves == 2 && same_waves_per_cu(walk_shape<MeanOp<1>>(1024, 300007)));
static_assert(walk_shape<PushOp>(1024, 11689511).waves == 2 && same_waves_per_cu(walk_shape<PushOp>(1024, 11689511)));
static_assert(walk_shape<FusedOp>(256, 100003).waves == 2 && same_waves_per_cu(walk_shape<FusedOp>(256, 100003)));

}  // namespace
