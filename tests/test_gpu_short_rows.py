"""Short rows out of place: where the launch halves its workgroups and shortens its clusters so that every XCD
gets its share of the column chunks, and where there are too few chunks for that.  Row lengths on both sides of
each edge of the rule (fewer than eight chunks, kMinChunks chunks of 1, 2, 4 and 8 waves), natural and cycle order."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import Tuning, dev, host, in_place_equals_the_oracle, once, same_bits

pytestmark = pytest.mark.gpu

TILE = 256                                                     # columns of one wavefront on fp32 rows
EDGES = [TILE * 7, TILE * 8, TILE * 103, TILE * 206, TILE * 412, TILE * 824]


@pytest.mark.parametrize("ordered", [-1, 1])
@pytest.mark.parametrize("P", sorted(e + d for e in EDGES for d in (0, 1)))
@pytest.mark.parametrize("kind", ["gossip", "hier", "fused", "bf16"])
def test_short_rows(kind, P, ordered):
    W, G, S = 6, 3, 3
    ld = (P + 7) // 8 * 8
    so = np.array([0, P // 3 + 1, P - 2, P], dtype=np.int64)
    x = WL.gen_matrix(W, P, 0.05, seed=P, ld=ld)
    print(kind, P, ordered, flush=True)
    with Tuning(ordered=ordered):
        if kind == "bf16":
            pe = O.topology(P, W, S, 0, 1)[0]
            xb = O.f32_to_bf16(x)
            a = dev(xb.view(np.int16))
            b = torch.zeros_like(a)
            cx.cx_gossip_mix_bf16(a, b, P, dev(so), dev(pe))
            assert (host(b).view(np.uint16)[:, :P] == O.gossip_mix_bf16(xb, P, so, pe)[:, :P]).all()
            return
        a, b = dev(x), torch.full((W, ld), float("nan"), device="cuda:0")
        if kind == "gossip":
            pe = O.topology(P, W, S, 0, 1)[0]
            cx.cx_gossip_mix(a, b, P, dev(so), dev(pe))
            want = O.gossip_mix(x, P, so, pe)
        elif kind == "hier":
            pe = O.topology(P, W // G, S, 0, 1)[0]
            cx.cx_hier_mix(a, b, P, G, dev(so), dev(pe))
            want = once(O.hier_mix_f64(x, P, G, so, pe))
        else:
            pe = O.topology(P, W, S, 0, 1)[0]
            v, g = (WL.gen_matrix(W, P, s, seed=P, ld=ld, stream=k) for s, k in ((0.02, 1), (0.01, 2)))
            vo = torch.zeros_like(a)
            cx.cx_sgd_fused_mix(a, b, dev(v), vo, dev(g), 0.1, 0.9, 1e-4, P, dev(so), dev(pe))
            want, wv = (once(t) for t in O.sgd_fused_mix_f64(x, v, g, 0.1, 0.9, 1e-4, P, so, pe))
            assert same_bits(host(vo)[:, :P], wv[:, :P])
        assert same_bits(host(b)[:, :P], want[:, :P])


@pytest.mark.parametrize("W", [2, 257, 1024])
def test_rows_of_one_column_to_one_chunk(W):
    for P in (1, 3, 255, 257, 1000):
        ld = (P + 3) // 4 * 4
        x = WL.gen_matrix(W, P, 0.05, seed=P, ld=ld)
        pe = O.topology(P, W, 1, 0, 1)[0]
        so = np.array([0, P], dtype=np.int64)
        a = dev(x)
        for call in (cx.cx_gossip_mix, cx.cx_gossip_mix_noalloc):
            b = torch.full((W, ld), float("nan"), device="cuda:0")
            call(a, b, P, dev(so), dev(pe))
            assert same_bits(host(b)[:, :P], O.gossip_mix(x, P, so, pe)[:, :P])


@pytest.mark.parametrize("P", [1, 5, 255, 259, 515, 1030])
@pytest.mark.parametrize("in_place", [False, True])
def test_boundary_tiles_keep_to_their_columns(P, in_place):
    """Boundary tiles load whole 16-byte slices: what lies in the padding (NaN here) or in the other segment of a
    slice reaches no result, and neither does the padding change.  Segments of 1 to 7 columns cut every slice."""
    W, rng = 5, np.random.default_rng(P)
    ld = (P + 7) // 8 * 8 + 8
    so = np.unique(np.concatenate([[0], np.cumsum(rng.integers(1, 8, size=P)), [P]]).clip(0, P)).astype(np.int64)
    pe = O.topology(P, W, len(so) - 1, 0, 1)[0]
    x, v, g = (WL.gen_matrix(W, P, s, seed=P, ld=ld, stream=k) for k, s in enumerate((0.05, 0.02, 0.01)))
    for a in (x, v, g):
        a[:, P:] = np.nan
    sod, ped = dev(so), dev(pe)
    a = dev(x)
    b = a if in_place else dev(x)
    cx.cx_gossip_mix(a, b, P, sod, ped)
    assert same_bits(host(b)[:, :P], O.gossip_mix(x, P, so, pe)[:, :P]) and np.isnan(host(b)[:, P:]).all()
    a, av = dev(x), dev(v)
    b, bv = (a, av) if in_place else (dev(x), dev(v))
    cx.cx_sgd_fused_mix(a, b, av, bv, dev(g), 0.1, 0.9, 1e-4, P, sod, ped)
    wx, wv = (once(t) for t in O.sgd_fused_mix_f64(x, v, g, 0.1, 0.9, 1e-4, P, so, pe))
    for got, want in ((b, wx), (bv, wv)):
        assert same_bits(host(got)[:, :P], want[:, :P]) and np.isnan(host(got)[:, P:]).all()
    for fmt, narrow in (("bf16", O.f32_to_bf16), ("f16", O.f32_to_f16)):
        xb, gb = narrow(x), narrow(g)
        a, av = dev(xb.view(np.int16)), dev(v)
        b, bv = (a, av) if in_place else (dev(xb.view(np.int16)), dev(v))
        getattr(cx, f"cx_sgd_fused_mix_{fmt}")(a, b, av, bv, dev(gb.view(np.int16)), 0.1, 0.9, 1e-4, P, sod, ped)
        wx, wv = O.sgd_fused_mix16(fmt, xb, v, gb, 0.1, 0.9, 1e-4, P, so, pe)
        assert (host(b).view(np.uint16)[:, :P] == wx[:, :P]).all() and same_bits(host(bv)[:, :P], wv[:, :P])
        assert (host(b).view(np.uint16)[:, P:] == xb[:, P:]).all() and np.isnan(host(bv)[:, P:]).all()


# in place: the edges where workgroups are halved (127 * 1, 2, 4, 8 tiles) and full ones of one slice per lane, for rings
# that the steady loop turns never, once and many times (n <= 2 D, n just above, n = 37).  Most of these calls split their
# rows over wavefronts by default; the lock-step parameter at its default value asks for mix_kernel and leaves it its shape.
@pytest.mark.parametrize("lockstep", [-1, 1])
@pytest.mark.parametrize("W", [3, 5, 17, 37])
@pytest.mark.parametrize("P", [TILE * 127 + 1, TILE * 254, TILE * 1016 + 3, 2 * TILE * 2047, 2 * TILE * 2047 + 1])
@pytest.mark.parametrize("kind", ["gossip", "fused", "bf16"])
def test_in_place_walk_shapes(kind, W, P, lockstep):
    ld = (P + 7) // 8 * 8
    so = np.array([0, P // 3 + 1, P // 3 + 1, P - 2, P], dtype=np.int64)
    pe = O.topology(P, W, len(so) - 1, 0, 1)[0]
    x = WL.gen_matrix(W, P, 0.05, seed=P, ld=ld)
    print(kind, W, P, lockstep, flush=True)
    if kind == "bf16":
        xb = O.f32_to_bf16(x)
        a = dev(xb.view(np.int16))
        with Tuning(lockstep=lockstep):
            cx.cx_gossip_mix_bf16(a, a, P, dev(so), dev(pe))
        assert (host(a).view(np.uint16)[:, :P] == O.gossip_mix_bf16(xb, P, so, pe)[:, :P]).all()
        return
    a = dev(x)
    if kind == "gossip":
        with Tuning(lockstep=lockstep):
            cx.cx_gossip_mix(a, a, P, dev(so), dev(pe))
        want = O.gossip_mix(x, P, so, pe)
    else:
        v, g = (WL.gen_matrix(W, P, s, seed=P, ld=ld, stream=k) for s, k in ((0.02, 1), (0.01, 2)))
        vd = dev(v)
        with Tuning(lockstep=lockstep):
            cx.cx_sgd_fused_mix(a, a, vd, vd, dev(g), 0.1, 0.9, 1e-4, P, dev(so), dev(pe))
        want, wv = (once(t) for t in O.sgd_fused_mix_f64(x, v, g, 0.1, 0.9, 1e-4, P, so, pe))
        assert same_bits(host(vd)[:, :P], wv[:, :P])
    assert same_bits(host(a)[:, :P], want[:, :P])


@pytest.mark.parametrize("slices", [-1, 2, 4])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 7, 9, 259, 515, 1030, 2061])
@pytest.mark.parametrize("in_place", [False, True])
def test_the_last_rows_storage_may_end_at_its_last_column(P, in_place, slices):
    """Columns [P, ld) are the caller's own: a matrix may stop at the last row's column P (what follows here belongs
    to somebody else and stays as it is).  Row lengths below a slice, below a tile and just above, slices per lane
    1, 2 and 4: no slice at the row end ends with the row."""
    W, G, S = 6, 3, 3
    ld = (P + 7) // 8 * 8 + 8
    so = np.array([0, P // 3, max(P - 2, P // 3), P], dtype=np.int64)
    pe, pl = O.topology(P, W, S, 0, 1)[0], O.topology(P, W // G, S, 0, 1)[0]
    x, v, g = (WL.gen_matrix(W, P, s, seed=P, ld=ld, stream=k) for k, s in enumerate((0.05, 0.02, 0.01)))
    sod, ped, pld = dev(so), dev(pe), dev(pl)
    print(P, in_place, slices, flush=True)

    def tight(a):                                          # rows of a in storage that ends at the last row's column P
        a = np.ascontiguousarray(a)
        n = (a.shape[0] - 1) * ld + P
        buf = dev(np.concatenate([a.reshape(-1)[:n], np.full(16, 77, a.dtype)]))
        return buf, buf[:n].as_strided((a.shape[0], P), (ld, 1))

    def check(call, a, want, wide=(), keep=()):
        """call(x_in, x_out, *other buffers) with a's rows; want: the oracle's matrices, one for each written buffer."""
        bufs = [tight(m) for m in (a, *wide)]
        outs = bufs if in_place else [tight(m) for m in (a, *wide)]
        kept = [tight(m)[1] for m in keep]
        call(*[t for pair in zip(bufs, outs) for t in (pair[0][1], pair[1][1])], *kept)
        for (buf, out), w in zip(outs, want):
            got = host(out)
            if got.dtype == np.int16:
                assert (got.view(np.uint16) == w[:, :P]).all()
            else:
                assert same_bits(got, w[:, :P])
            assert (host(buf)[-16:] == 77).all()

    with Tuning(slices=slices):
        check(lambda a, b: cx.cx_gossip_mix(a, b, P, sod, ped), x, [O.gossip_mix(x, P, so, pe)])
        check(lambda a, b: cx.cx_hier_mix(a, b, P, G, sod, pld), x, [once(O.hier_mix_f64(x, P, G, so, pl))])
        want = [once(t) for t in O.sgd_fused_mix_f64(x, v, g, 0.1, 0.9, 1e-4, P, so, pe)]
        check(lambda a, b, c, d, e: cx.cx_sgd_fused_mix(a, b, c, d, e, 0.1, 0.9, 1e-4, P, sod, ped), x, want, [v], [g])
        for fmt, narrow in (("bf16", O.f32_to_bf16), ("f16", O.f32_to_f16)):
            xb, gb = narrow(x), narrow(g)
            mix, step = getattr(cx, f"cx_gossip_mix_{fmt}"), getattr(cx, f"cx_sgd_fused_mix_{fmt}")
            check(lambda a, b: mix(a, b, P, sod, ped), xb.view(np.int16), [getattr(O, f"gossip_mix_{fmt}")(xb, P, so, pe)])
            check(lambda a, b, c, d, e: step(a, b, c, d, e, 0.1, 0.9, 1e-4, P, sod, ped), xb.view(np.int16),
                  O.sgd_fused_mix16(fmt, xb, v, gb, 0.1, 0.9, 1e-4, P, so, pe), [v], [gb.view(np.int16)])


# in place, both sides of the edges between shapes: 2,048 tiles of one slice per lane (256 fp32 or 512 16-bit columns), 3 *
# 2,048 of two where the long shape has two, the two or three million columns from which workgroups of two waves are taken;
# walks of just more than 2 D steps, so that the steady loop turns.
# (kind, rows per group, gossiping rows, columns of the last row below the edge, ld a multiple of)
LONG_EDGES = [("gossip", 1, 9, (3 << 20) - 1, 32), ("gossip", 1, 9, 512 * 6143, 8), ("gossip", 1, 33, 512 * 6143, 32),
              ("gossip", 1, 33, 512 * 6143, 8), ("hier", 2, 9, 512 * 6143, 8), ("hier", 3, 5, 512 * 6143, 8),
              ("hier", 3, 13, (2 << 20) - 1, 32), ("hier", 4, 5, (2 << 20) - 1, 8), ("hier", 4, 9, (2 << 20) - 1, 32),
              ("hier", 4, 9, 512 * 6143, 8), ("hier", 8, 5, (2 << 20) - 1, 32), ("hier", 8, 9, 256 * 2047, 8),
              ("hier", 16, 5, 256 * 2047, 32), ("fused", 1, 9, (2 << 20) - 1, 32), ("fused", 1, 9, 512 * 6143, 8),
              ("hiersgd", 1, 9, (2 << 20) - 1, 32), ("hiersgd", 4, 5, (2 << 20) - 1, 8), ("hiersgd", 5, 9, 256 * 2047, 8),
              ("hiersgd", 6, 5, (2 << 20) - 1, 32), ("pushsum", 1, 9, 512 * 6143, 8), ("debias", 1, 17, 256 * 2047, 32),
              ("gossip16", 1, 9, 1024 * 6143, 8), ("pushsum16", 1, 9, 1024 * 6143, 8), ("debias16", 1, 9, 512 * 2047, 64),
              ("hier16", 4, 5, 512 * 2047, 8), ("fused16", 1, 5, 512 * 2047, 8), ("hiersgd16", 3, 5, 512 * 2047, 64)]


@pytest.mark.parametrize("kind,G,n,short,ld_of", LONG_EDGES)
@pytest.mark.parametrize("beyond", [0, 1])
def test_in_place_edge_of_short_rows(kind, G, n, short, ld_of, beyond):
    P = short + beyond
    ld = (P + ld_of - 1) // ld_of * ld_of
    print(kind, G, n, P, ld, flush=True)
    in_place_equals_the_oracle(kind, G, n, P, ld, np.array([0, P // 3 + 1, P // 3 + 1, P - 2, P], dtype=np.int64))
