// Row operators on fp32 rows (internal header): the plain and the hierarchical mean (Section 3.3), the
// momentum-SGD step fused in front of the mix (Section 3.1), its gradient-reducing hierarchical form, and the
// push-sum comparison (Sections 2.1, 3); with the traits through which the kernels ask an operator for its
// launch shapes and LDS needs.
#ifndef CX_OPS_HPP
#define CX_OPS_HPP
#include "cx_tile.hpp"

#pragma clang fp contract(off)

namespace {

// ---------------------------------------------------------------------------------
// Row operators: what "load gossiping row r" and "store gossiping row r" mean.
// ---------------------------------------------------------------------------------
// Each operator splits "load gossiping row r" into issue() -- put the row's global loads in
// flight into a Raw slot -- and finish() -- turn the arrived data into the tile that takes
// part in the pairwise average.  kRawPerSlice = 16-byte registers per slice and slot.
// kGather = the operator's default launch shape in the out-of-place kernel, kWalk = in the
// in-place kernel (measured optima on MI355X).
struct GatherShape {
    int U, waves, visit_kb, wgs_per_cu;   // slices per lane, waves per workgroup, KB of one row visit
};                                        // per XCD, resident workgroups per CU (0 = as many as fit)
struct WalkShape {
    int U, D, waves, wgs_per_cu;       // slices per lane, rows in flight, waves per workgroup,
};                                     // resident workgroups per CU (0 = as many as fit)
// Long rows in place: kWalk, eight waves in lock-step, unless the operator's walk(n, P, whole_lines) names another shape
// (whole_lines: the row stride is a multiple of 128 bytes, so that rows begin on lines where the allocation does).
// Short rows: see walk_shape in cx_launch.hpp.
//
// Rows that begin inside a line: neighbouring tiles share lines, and eight waves in lock-step touch them together.
// Rows that begin on a line, and few rows in general, are better off with workgroups of two waves: no lines to share,
// and the last of few rounds of large workgroups leaves CUs idle.  Two waves against eight, in place, us:
//                                    64 x 11,689,511 on lines   inside lines   32 x 25,000,003 on lines   inside lines
//     fp32 gossip                    1,089 / 1,126              1,185 / 1,151  1,155 / 1,194              1,208 / 1,217
//     fp32 mean of groups of 4       1,103 / 1,130              1,221 / 1,195  1,095 / 1,247              1,234 / 1,281
//     fp32 mean of groups of 8       1,117 / 1,155              1,266 / 1,258  1,140 / 1,201              1,310 / 1,275
//     fp32 gradient step, groups of 6  1,298 / 1,371            1,453 / 1,476  1,371 / 1,454
// 256 rows on lines take eight again: mean of groups of 4 on 256 x 3,000,001 1,238 / 1,195.  16-bit groups gain
// nothing from two waves on long rows (binary16 mean of groups of 4 on 64 x 11,689,511: 581 / 558).
// Neither do rows below two million columns (32 x 900,001, groups of 8: 50 / 45).
constexpr bool two_waves(int G, int rows, int64_t P, bool whole_lines)
{
    return P >= (2 << 20) && ((rows <= 32 && G <= 5) || (rows <= 64 && whole_lines));
}

// Rows in flight of an operator whose finish() only copies or widens (see walk() in cx_kernels.hpp): eight beside
// many rows only, since the last 2 * D steps of a walk are slower ones.
constexpr int ring_for(int n) { return n >= 128 ? 8 : 4; }

// For the visit of the out-of-place kernel (VisitKb): gossiping rows that are few, columns of long rows, and whether a longer visit seldom meets the edge of
// a segment (they are `cols` columns and more) or does not suffer by it (rows that may be ordered by the tile, see try_gather).
constexpr int kFewRows = 8;
constexpr int64_t kLongRows = 3000000;
constexpr bool inside_segments(int n, int64_t P, int S, int64_t cols) { return n >= kFewRows || S == 1 || P >= cols * S; }

// Plain gossip (G == 1) and hierarchical mode (a gossiping row = a group of G rows).
// G == 1 is Algorithm 1's averaging line in fp32, as written.  For G > 1 the group sum (rows in
// order, from zero), the division by G and the average between leaders run in fp64 registers and
// the result is rounded ONCE to fp32: the correctly rounded value of the plain definition, whatever
// cancels inside the group -- an fp32 sum of values that cancel cannot promise an error relative to
// the result.  The kernel is bound by HBM bandwidth; the fp64 rate is not what limits it.
template <int G>
struct MeanOp {
    static constexpr int kRows = G;                       // matrix rows behind a gossiping row
    static constexpr int kElems = 4;                       // fp32 columns per 16-byte slice
    template <int U> using Work = std::conditional_t<G == 1, Tile<U>, WideTile<U>>;
    static constexpr int kRawPerSlice = G;
    // out-of-place launch: slices per lane, waves per workgroup, KB of one visit to a gossiping row
    // (all G rows behind it) per XCD -- measured optima on MI355X (see VisitKb)
    static constexpr GatherShape kGather =
        G == 1 ? GatherShape{1, 4, 256, 0} : G <= 4 ? GatherShape{1, 8, 512, 0} : GatherShape{1, 8, 768, 0};
    static constexpr int visit_kb(int n, int64_t P, int S)
    {
        return G < 8 || n > kFewRows ? 0 : G == 8 && inside_segments(n, P, S, 65536) ? 512 : 256;
    }
    static constexpr WalkShape kWalk =
        G == 1 ? WalkShape{2, 8, 8, 2} : G == 2 ? WalkShape{2, 4, 8, 2} : G <= 5 ? WalkShape{2, 2, 8, 2}
        : G <= 8 ? WalkShape{1, 4, 8, 2} : WalkShape{1, 2, 8, 2};
    template <int U, int D> static constexpr bool kSpills = U > 1 && (G >= 6 || (G == 3 && U * D >= 8));
    constexpr WalkShape walk(int n, int64_t P, bool whole_lines) const
    {
        const bool few = n * G <= 32;
        if constexpr (G == 1) {
            // few long rows on lines: one slice of two rows, many small workgroups, no steady loop (32 x 25,000,003:
            // 1,109 us, with the steady loop 1,192, with two slices of two to eight rows 1,144 to 1,194; the length is
            // that from which two slices count as long)
            if (few) return whole_lines && P >= (3 << 20) ? WalkShape{1, 2, 2, 8} : WalkShape{2, 4, 2, 2};
            return n <= 64 && whole_lines ? WalkShape{2, 2, 2, 2} : kWalk;
        } else {
            if (G > 8 || !two_waves(G, n * G, P, whole_lines)) return kWalk;
            if (G == 2) return few ? WalkShape{2, 4, 2, 2} : kWalk;
            if (G == 3) return few ? WalkShape{2, 2, 2, 2} : WalkShape{1, 4, 2, 2};
            return WalkShape{1, G == 4 && !few ? 4 : 2, 2, 2};
        }
    }
    template <int U> struct Raw { Tile<U> r[G]; };
    const float *xin;
    float *xout;
    int64_t ld;

    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void issue(int row, int64_t off, const unsigned (&mask)[U], Raw<U> &raw) const
    {
        const float *p = xin + static_cast<int64_t>(row) * G * ld + off;
#pragma unroll
        for (int j = 0; j < G; ++j) tile_load<U, MODE, NT>(p + j * ld, mask, raw.r[j]);
    }
    template <int U, TileMode MODE, bool NT, bool COMMIT = true>
    __device__ __forceinline__ void finish(int row, int64_t off, const unsigned (&mask)[U], const Raw<U> &raw, Work<U> &t) const
    {
        if constexpr (G == 1) {
            t = raw.r[0];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int j = 0; j < G; ++j) sum = sum + widen(raw.r[j].v[u]);
                t.v[u] = sum / static_cast<double>(G);
            }
        }
    }
    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void store(int row, int64_t off, const unsigned (&mask)[U], const Work<U> &t) const
    {
        Tile<U> out;
        if constexpr (G == 1) {
            out = t;
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) out.v[u] = narrow(t.v[u]);
        }
        float *p = xout + static_cast<int64_t>(row) * G * ld + off;
#pragma unroll
        for (int j = 0; j < G; ++j) tile_store<U, MODE, NT>(p + j * ld, mask, out);
    }
};

// Plain gossip out of place whose wavefronts store whole lines, to matrices that the last-level cache does not hold: the lines
// go to memory in the order in which they are made, not in that in which L2 gives them up, which DRAM serves faster.
// Non-temporal / written through, us: 32 x 25,557,032 1,088 / 1,067; 4 x 25,557,032 inside lines 154 / 141; 64 x 11,689,512
// 997 / 983; 1,024 x 1,200,003 1,671 / 1,655; 100 x 200,003 31.1 / 30.7; 512 x 100,003 94.3 / 94.1.  What L2 would have
// merged must not go out by itself (8 x 1,000,001 inside lines, wavefronts in the column grid, 13.0 / 15.1; in-place walks 1 to
// 12 % slower), and other operators gain nothing: optimizer step on 64 x 5,000,001 1,144 / 1,165, push-sum on
// 128 x 1,689,513 291 / 296, bf16 gossip on 32 x 25,557,032 551 / 554, mean of groups of 8 on 64 x 11,689,512 1,057 / 1,056.
struct ThroughOp : MeanOp<1> {
    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void store(int row, int64_t off, const unsigned (&mask)[U], const Tile<U> &t) const
    {
        float *p = xout + static_cast<int64_t>(row) * ld + off;
        if constexpr (MODE == kFull && NT) {
#pragma unroll
            for (int u = 0; u < U; ++u) store_through(reinterpret_cast<f4 *>(p + u * 256), t.v[u]);
        } else {
            tile_store<U, MODE, NT>(p, mask, t);
        }
    }
};

// The hierarchical mean staged through LDS, kept for measurement next to the sum in registers (launch
// parameter 10).  A workgroup is G wavefronts and owns G tiles of 256 columns; wavefront j fetches
// row j of its group and of the partner group (G contiguous 1-KB loads each), the rows meet in
// LDS (G x G KB), wavefront w reduces tile w over the G rows in the same order and precision, and
// the result travels back through LDS so that wavefront j stores row j.  Same arithmetic in the
// same order as MeanOp<G>, hence the same bits; five barriers per workgroup.  Chunks that a
// segment boundary or the row end crosses take MeanOp<G>'s register path.
template <int G>
struct MeanLdsOp : MeanOp<G> {
    static constexpr bool kLdsStaged = true;
    static constexpr size_t kLdsBytes = static_cast<size_t>(G) * G * kWave * sizeof(f4);

    template <bool NT>
    __device__ __forceinline__ void lds_mix(int row, int peer, int64_t chunk_c0, int lane, int wave, f4 *lds) const
    {
        const int64_t col = chunk_c0 + 4 * lane;
        const float *own = this->xin + (static_cast<int64_t>(row) * G + wave) * this->ld + col;
        const float *oth = this->xin + (static_cast<int64_t>(peer) * G + wave) * this->ld + col;
        f4 mine[G], theirs[G];
#pragma unroll
        for (int t = 0; t < G; ++t) mine[t] = *reinterpret_cast<const f4 *>(own + t * 256);
#pragma unroll
        for (int t = 0; t < G; ++t) theirs[t] = *reinterpret_cast<const f4 *>(oth + t * 256);
#pragma unroll
        for (int t = 0; t < G; ++t) lds[(wave * G + t) * kWave + lane] = mine[t];        // [row][tile][lane]
        __syncthreads();
        d4 a = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < G; ++j) a = a + widen(lds[(j * G + wave) * kWave + lane]);
        a = a / static_cast<double>(G);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < G; ++t) lds[(wave * G + t) * kWave + lane] = theirs[t];
        __syncthreads();
        d4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < G; ++j) c = c + widen(lds[(j * G + wave) * kWave + lane]);
        c = c / static_cast<double>(G);
        __syncthreads();
        lds[wave * kWave + lane] = narrow(average(a, c));                                        // result tile `wave`
        __syncthreads();
        float *dst = this->xout + (static_cast<int64_t>(row) * G + wave) * this->ld + col;
#pragma unroll
        for (int t = 0; t < G; ++t) {
            f4 *q = reinterpret_cast<f4 *>(dst + t * 256);
            const f4 v = lds[t * kWave + lane];
            if (NT) __builtin_nontemporal_store(v, q); else *q = v;
        }
    }
};

// Operators that change between memory order and lane order through LDS say how much each wavefront
// needs and are told where their areas start.
template <class Op, class = void>
struct StageBytes {
    static constexpr int value = 0;
};
template <class Op>
struct StageBytes<Op, std::void_t<decltype(Op::kStageBytes)>> {
    static constexpr int value = Op::kStageBytes;
};
template <class Op>
Op with_stage_base(const Op &op, size_t base)
{
    Op copy = op;
    if constexpr (StageBytes<Op>::value > 0) copy.stage_base = static_cast<int>(base);
    return copy;
}

// Visit length of the out-of-place kernel: kGather.visit_kb, unless the operator's visit_kb(rows, P, S) names another one (0: it does not).
//
// Operators on groups, in chunks of 8 KB of every matrix row (before the clusters are shortened to fill their last round).  Eight or
// sixteen chunks, with which the XCDs' visits of a row together begin and end on multiples of 512 KB, gain on matrices as torch
// allocates them for some operators and group sizes.  Time over that with the visit otherwise taken, shapes of 250,000 to
// 25,000,000 columns, 2 to 40 gossiping rows and 1 to 32 segments, several matrices in turn, geometric mean (range):
//   fp32 mean             groups of 8, up to 8 rows    8 for 4              90 shapes   0.995 (0.97 to 1.025)
//   16-bit mean           groups of 4, 6              16 for 8             160          0.97 (0.86 to 1.03)
//                         groups of 7, 8, beyond 8    16 for 6              70          0.97 (0.88 to 1.02)
//   fp32 gradient step    groups of 8                 16 for 12 (few: 4)   120          0.98 (0.93 to 1.02)
//   16-bit gradient step  groups of 8, see below       8 for 6             100          0.994 (0.97 to 1.04)
// Not where fewer rows than kFewRows, which are ordered by the cluster, are cut into segments shorter than four visits, of 16-bit rows
// ten: every cluster with an edge takes the general path, and longer clusters have more of them.  Longer / shorter visit, us: fp32
// gradient step on 24 x 852,780 in 29 segments 47.0 / 41.9, 16-bit mean of groups of 4 on 20 x 2,549,454 in 20 46.7 / 44.1, of groups
// of 6 on 30 x 5,699,719 in 11 142.9 / 134.3, fp32 mean on 56 x 407,136 in 24 43.4 / 42.2.
// Not taken, since they gained nothing or lost: 16-bit mean of groups of 3, 16 for 10 chunks (40 shapes) 0.994, up to 1.12, of 5, 8 for 9, 1.00,
// of 7 and 8 with up to 8 rows 1.00, up to 1.06; fp32 gradient step of groups of 5 and 7, 16 for 19 and 13, 1.00, up to 1.05; 16-bit
// gradient step of groups of 3, 8 for 10 (40) 0.993, up to 1.066, of 5 and 7 1.01, up to 1.14, of 8, 8 for 6, with fewer than kFewRows
// rows 1.00, up to 1.068, on rows below kLongRows up to 1.04, in segments below ten visits of 16 chunks up to 1.066 (70 shapes).
// On matrices spread over the physical memory what is taken gains less or loses: fp32 mean 0.980 to 1.010, 16-bit mean 0.97 to
// 1.013, fp32 gradient step 0.983 to 1.030.
// With groups of 16, at most kFewRows gossiping rows visit 256 KB: their longest cycle's visits then fit one XCD's 4 MB L2.
template <class Op, class = void>
struct VisitKb {
    static constexpr int of(int, int64_t, int) { return Op::kGather.visit_kb; }
};
template <class Op>
struct VisitKb<Op, std::void_t<decltype(Op::visit_kb(0, 0, 1))>> {
    static constexpr int of(int n, int64_t P, int S) { return Op::visit_kb(n, P, S) ? Op::visit_kb(n, P, S) : Op::kGather.visit_kb; }
};

template <class Op, class = void>
struct LdsStaged {
    static constexpr bool value = false;
    static constexpr size_t bytes = 0;
};
template <class Op>
struct LdsStaged<Op, std::void_t<decltype(Op::kLdsStaged)>> {
    static constexpr bool value = Op::kLdsStaged;
    static constexpr size_t bytes = Op::kLdsBytes;
};

// Resident workgroups per CU out of place: kGather's, unless the operator names them by what it is asked to write.
template <class Op, class = void>
struct GatherWgs {
    static constexpr int of(const Op &) { return Op::kGather.wgs_per_cu; }
};
template <class Op>
struct GatherWgs<Op, std::void_t<decltype(std::declval<const Op &>().gather_wgs_per_cu())>> {
    static constexpr int of(const Op &op) { return op.gather_wgs_per_cu(); }
};

// Momentum-SGD applied as the row arrives; the mix then averages the updated rows.
// The whole chain runs in fp64 registers, in the order the formula is written:
//     t = g + wd*x ;  v' = mu*v + t ;  h = x - lr*v' ;  x' = (h_i + h_peer) * 0.5
// (every input widened exactly, the hyper-parameters as the doubles of their fp32 values, no
// fused multiply-add), and v' and x' are each rounded ONCE to fp32 when they are stored.  An
// fp32 chain would round six times against intermediates larger than the result and misses a
// 1e-6 relative bound once the momentum has grown; the kernel is bound by HBM bandwidth, so
// the fp64 rate is not what limits it.

struct SgdStep {
    double lr, mu, wd;
    // one optimizer step on a vector of columns: returns h, leaves v' in `v`
    __device__ __forceinline__ d4 apply(const d4 &x, d4 &v, const d4 &g) const
    {
        const d4 decayed = g + x * wd;
        v = v * mu + decayed;
        return x - v * lr;
    }
};

struct FusedOp {
    static constexpr int kRows = 1;                       // matrix rows behind a gossiping row
    static constexpr int kElems = 4;                       // fp32 columns per 16-byte slice
    template <int U> using Work = WideTile<U>;             // the updated row, in fp64
    static constexpr int kRawPerSlice = 3;
    static constexpr GatherShape kGather{1, 8, 128, 3};
    static constexpr WalkShape kWalk{2, 4, 8, 2};
    static constexpr int kMaxU = 2;                        // fp64 rows: two slices per lane fill the registers
    constexpr WalkShape walk(int n, int64_t P, bool whole_lines) const
    {
        // in place, rows on lines, two waves against eight: 32 x 3,200,013 384 / 442 us, 64 x 11,689,511 2,917 / 2,862,
        // 32 x 900,001 119 / 114
        return n <= 32 && P >= (2 << 20) && whole_lines ? WalkShape{1, 4, 2, 2} : kWalk;
    }
    template <int U> struct Raw { Tile<U> x, v, g; };
    const float *xin;
    float *xout;
    const float *vin;
    float *vout;
    const float *g;
    int64_t ld;
    SgdStep sgd;

    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void issue(int row, int64_t off, const unsigned (&mask)[U], Raw<U> &raw) const
    {
        const int64_t o = static_cast<int64_t>(row) * ld + off;
        tile_load<U, MODE, NT>(xin + o, mask, raw.x);
        tile_load<U, MODE, NT>(vin + o, mask, raw.v);
        tile_load<U, MODE, NT>(g + o, mask, raw.g);
    }
    // COMMIT: also write v' of this row (false when the row is only recomputed as a partner)
    template <int U, TileMode MODE, bool NT, bool COMMIT = true>
    __device__ __forceinline__ void finish(int row, int64_t off, const unsigned (&mask)[U], const Raw<U> &raw, Work<U> &t) const
    {
        Tile<U> v32;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            d4 v = widen(raw.v.v[u]);
            t.v[u] = sgd.apply(widen(raw.x.v[u]), v, widen(raw.g.v[u]));
            v32.v[u] = narrow(v);
        }
        if constexpr (COMMIT) tile_store<U, MODE, NT>(vout + static_cast<int64_t>(row) * ld + off, mask, v32);
    }
    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void store(int row, int64_t off, const unsigned (&mask)[U], const Work<U> &t) const
    {
        Tile<U> out;
#pragma unroll
        for (int u = 0; u < U; ++u) out.v[u] = narrow(t.v[u]);
        tile_store<U, MODE, NT>(xout + static_cast<int64_t>(row) * ld + off, mask, out);
    }
};

// Hierarchical step with gradients: a gossiping row is a group; loading it reduces the G
// gradient rows, applies the momentum-SGD step to the LEADER's parameters and momentum, and
// hands the updated leader parameters to the mix; storing broadcasts.  fp64 registers as in
// FusedOp: the gradients are summed in row order starting from zero and divided by G.
template <int G>
struct HierFusedOp {
    static constexpr int kRows = G;                       // matrix rows behind a gossiping row
    static constexpr int kElems = 4;                       // fp32 columns per 16-byte slice
    template <int U> using Work = WideTile<U>;             // the updated leader row, in fp64
    static constexpr int kRawPerSlice = G + 2;
    // out-of-place launch: slices, waves, group visit KB per XCD
    static constexpr GatherShape kGather =
        G == 1 ? GatherShape{1, 8, 256, 0} : G <= 4 ? GatherShape{1, 8, 512, 0}
        : GatherShape{1, 8, 768, 0};
    static constexpr int visit_kb(int n, int64_t P, int S)                          // see VisitKb
    {
        return G == 8 && inside_segments(n, P, S, 131072) ? 1024 : G >= 8 && n <= kFewRows ? 256 : 0;
    }
    static constexpr WalkShape kWalk = G <= 4 ? WalkShape{1, 4, 8, 2} : WalkShape{1, 2, 8, 2};
    static constexpr int kMaxU = G <= 2 ? 2 : 1;
    template <int U, int D> static constexpr bool kSpills = G == 5 && D == 4;
    constexpr WalkShape walk(int n, int64_t P, bool whole_lines) const
    {
        return G <= 8 && two_waves(G, n * G, P, whole_lines) ? WalkShape{1, G == 1 ? 4 : 2, 2, 2} : kWalk;
    }
    template <int U> struct Raw { Tile<U> g[G], x, v; };
    const float *xin;
    float *xout;
    const float *vin;     // [L][ld]
    float *vout;          // [L][ld]
    const float *g;       // [W][ld]
    int64_t ld;
    SgdStep sgd;

    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void issue(int row, int64_t off, const unsigned (&mask)[U], Raw<U> &raw) const
    {
        const int64_t lead = static_cast<int64_t>(row) * G * ld + off;
#pragma unroll
        for (int j = 0; j < G; ++j) tile_load<U, MODE, NT>(g + lead + j * ld, mask, raw.g[j]);
        tile_load<U, MODE, NT>(xin + lead, mask, raw.x);
        tile_load<U, MODE, NT>(vin + static_cast<int64_t>(row) * ld + off, mask, raw.v);
    }
    template <int U, TileMode MODE, bool NT, bool COMMIT = true>
    __device__ __forceinline__ void finish(int row, int64_t off, const unsigned (&mask)[U], const Raw<U> &raw, Work<U> &t) const
    {
        Tile<U> v32;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            d4 gsum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int j = 0; j < G; ++j) gsum = gsum + widen(raw.g[j].v[u]);
            const d4 gbar = gsum / static_cast<double>(G);
            d4 v = widen(raw.v.v[u]);
            t.v[u] = sgd.apply(widen(raw.x.v[u]), v, gbar);
            v32.v[u] = narrow(v);
        }
        if constexpr (COMMIT) tile_store<U, MODE, NT>(vout + static_cast<int64_t>(row) * ld + off, mask, v32);
    }
    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void store(int row, int64_t off, const unsigned (&mask)[U], const Work<U> &t) const
    {
        Tile<U> out;
#pragma unroll
        for (int u = 0; u < U; ++u) out.v[u] = narrow(t.v[u]);
        float *p = xout + static_cast<int64_t>(row) * G * ld + off;
#pragma unroll
        for (int j = 0; j < G; ++j) tile_store<U, MODE, NT>(p + j * ld, mask, out);
    }
};

// The weights of push-sum, w_out[i] = (w_in[i] + w_in[(i - hop) mod n]) * 0.5f.  The de-biasing of a row divides by its new
// weight; the first workgroup of the launch also writes them (a launch of its own in front of the mix cost as much as
// the mix on small matrices: 8 x 20,011 fp32 15.3 / 8.3 us.  Written beside the row's column 0 instead, in store(), the
// branch cost the in-place walk its rows in flight: 64 x 300,007 fp32 without the copy 37 / 55).
struct PushWeights {
    const float *in;
    float *out;
    int n, hop;
    __device__ __forceinline__ float of(int row) const
    {
        const int from = row >= hop ? row - hop : row - hop + n;
        return (in[row] + in[from]) * 0.5f;
    }
    __device__ __forceinline__ void write_all() const
    {
        for (int i = threadIdx.x; i < n; i += blockDim.x) out[i] = of(i);
    }
};

// What an operator has done once a launch, by its first workgroup.
template <class Op, class = void>
struct OncePerLaunch {
    static __device__ __forceinline__ void run(const Op &) {}
};
template <class Op>
struct OncePerLaunch<Op, std::void_t<decltype(std::declval<const Op &>().weights)>> {
    static __device__ __forceinline__ void run(const Op &op)
    {
        if ((blockIdx.x | blockIdx.y | blockIdx.z) == 0) op.weights.write_all();
    }
};

// Push-sum: plain rows, optional de-biased copy z = x' / w'.
struct PushOp {
    static constexpr int kRows = 1;                       // matrix rows behind a gossiping row
    static constexpr int kElems = 4;                       // fp32 columns per 16-byte slice
    template <int U> using Work = Tile<U>;                 // fp32 values a lane works on
    static constexpr int kRawPerSlice = 1;
    static constexpr GatherShape kGather{2, 4, 512, 0};
    // Out of place with the copy, five workgroups on a CU instead of as many as fit (six): 1 to 5 % on every shape of seven,
    // most on many rows (500 x 300,007 347 -> 331 us, 128 x 1,500,013 407 -> 396, 16 x 25,557,032 859 -> 843, 128 x 11,689,513
    // 3,080 -> 3,049).  Without it no cap of four or more moves a shape by more than 3 %, either way.
    constexpr int gather_wgs_per_cu() const { return zout ? 5 : kGather.wgs_per_cu; }
    static constexpr WalkShape kWalk{2, 8, 8, 2};
    template <int U> struct Raw { Tile<U> x; };
    // The weights that the de-biased copy loads make every row wait for all before it: one slice and a
    // short ring.  Against eight rows of two slices and eight waves, rows on lines: 64 x 11,689,511 with the copy
    // 1,791 -> 1,713 us, without 1,127 -> 1,070; 128 x 25,557,032 without 4,247 -> 4,346, so many rows keep them.
    constexpr WalkShape walk(int n, int64_t, bool) const
    {
        if (zout) return WalkShape{1, ring_for(n), 8, 2};
        return n <= 64 ? WalkShape{2, n <= 32 ? 4 : 2, 2, 2} : kWalk;
    }
    const float *xin;
    float *xout;
    float *zout;          // may be null
    int64_t ld;
    PushWeights weights;

    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void issue(int row, int64_t off, const unsigned (&mask)[U], Raw<U> &raw) const
    {
        tile_load<U, MODE, NT>(xin + static_cast<int64_t>(row) * ld + off, mask, raw.x);
    }
    template <int U, TileMode MODE, bool NT, bool COMMIT = true>
    __device__ __forceinline__ void finish(int row, int64_t off, const unsigned (&mask)[U], const Raw<U> &raw, Tile<U> &t) const
    {
        t = raw.x;
    }
    template <int U, TileMode MODE, bool NT>
    __device__ __forceinline__ void store(int row, int64_t off, const unsigned (&mask)[U], const Tile<U> &t) const
    {
        const int64_t o = static_cast<int64_t>(row) * ld + off;
        tile_store<U, MODE, NT>(xout + o, mask, t);
        if (zout) {
            const float wn = weights.of(row);
            Tile<U> z;
#pragma unroll
            for (int u = 0; u < U; ++u) z.v[u] = t.v[u] / wn;
            tile_store<U, MODE, NT>(zout + o, mask, z);
        }
    }
};

}  // namespace

#endif  // CX_OPS_HPP
