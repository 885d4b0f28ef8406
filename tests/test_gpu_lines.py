"""Out of place where rows begin inside lines of 128 bytes and every row's tiles start on its own lines: the oracle's bits
and nothing written beside the rows, at the shortest rows that take that kernel, at rows whose last tile exists for some
of them only, with segments that end inside the shift and with more of them than a wavefront has lanes, in both layouts of the row
order, from matrices that begin inside a line themselves.  (16-bit gossip, and 16-bit push-sum without the copy, stay in the column
grid: the same calls there.)"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import Tuning, dev, host, once, same_bits

pytestmark = pytest.mark.gpu

SGD = (0.1, 0.9, 1e-4)


def inside_lines(rows, ld, dtype, first, fill):
    """A matrix whose storage begins `first` slices of 16 bytes past a line, with a guard of one line on either side."""
    per_slice = 16 // torch.empty((), dtype=dtype).element_size()
    flat = torch.full((rows * ld + (16 + first) * per_slice,), fill, dtype=dtype, device="cuda:0")
    begin = (8 + first) * per_slice
    return flat, flat[begin:begin + rows * ld].view(rows, ld)


def offsets(P, S):
    if S > 63:                                                                 # the first ones inside the shift of some rows
        inner = np.random.default_rng(S).integers(0, P + 1, size=S - 6)
        return np.array([0, 3, 8, 8, 20, 50, *np.sort(inner[inner >= 50]), *[P] * int((inner < 50).sum()), P], dtype=np.int64)
    edges = [P // 3, P // 3 + 5, P // 2, P // 2, P - 3, P - 1][:S - 1]         # short, empty, and at the row end
    return np.array([0, *edges, P], dtype=np.int64)


# tiles of one slice: 256 fp32 or 512 16-bit columns
@pytest.mark.parametrize("slices", [-1, 2, 4])
@pytest.mark.parametrize("rows", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n,P,S,pad,first", [(2, 2048, 1, 0, 1), (5, 2049, 3, 1, 0), (9, 4096, 7, 3, 7), (16, 4093, 4, 5, 2),
                                             (33, 9001, 7, 1, 0), (3, 70_000, 2, 7, 3), (12, 30_720, 5, 1, 4),
                                             (40, 5001, 70, 3, 0), (300, 4097, 65, 1, 5)])
def test_gossip(rows, n, P, S, pad, first, slices):
    e = 4 if rows == "f32" else 8
    ld, so, pe = (P + e - 1) // e * e + pad * e, offsets(P, S), O.topology(S, n, S, 0, 1)[0]
    x = WL.gen_matrix(n, P, 0.05, seed=P + n, ld=ld)
    if rows == "f32":
        want, dtype, call = O.gossip_mix(x, P, so, pe), torch.float32, cx.cx_gossip_mix
    else:
        x = (O.f32_to_bf16 if rows == "bf16" else O.f32_to_f16)(x)
        want, dtype = getattr(O, "gossip_mix_" + rows)(x, P, so, pe), torch.int16
        call = getattr(cx, "cx_gossip_mix_" + rows)
    fill = 7.0 if rows == "f32" else 7
    for cluster in (-1, 1):
        _, xd = inside_lines(n, ld, dtype, 0, fill)
        xd.copy_(dev(x if rows == "f32" else x.view(np.int16)))
        flat, y = inside_lines(n, ld, dtype, first, fill)
        print(rows, n, P, S, pad, first, slices, cluster, flush=True)
        with Tuning(ordered=1, slices=slices, cluster=cluster):
            call(xd, y, P, dev(so), dev(pe))
        got = host(y)
        assert same_bits(got[:, :P], want[:, :P]) if rows == "f32" else (got.view(np.uint16)[:, :P] == want[:, :P]).all()
        y[:, :P] = fill
        assert (flat == fill).all()                            # nothing beside the rows


@pytest.mark.parametrize("rows", ["f32", "bf16"])
@pytest.mark.parametrize("n,P,S,pad", [(4, 2049, 3, 1), (17, 5000, 7, 3), (9, 40_001, 5, 1)])
def test_optimizer_step_and_push_sum(rows, n, P, S, pad):
    e = 4 if rows == "f32" else 8
    ld, so, pe = (P + e - 1) // e * e + pad * e, offsets(P, S), O.topology(S, n, S, 0, 1)[0]
    x, v, g = (WL.gen_matrix(n, P, s, seed=P + n, ld=ld, stream=k) for k, s in enumerate((0.05, 0.02, 0.01)))
    w = np.random.default_rng(n).uniform(0.5, 1.5, n).astype(np.float32)
    print(rows, n, P, S, pad, flush=True)
    if rows == "f32":
        step, push, put, raw = cx.cx_sgd_fused_mix, cx.cx_pushsum_mix, dev, host
        want_x, want_v = (once(t) for t in O.sgd_fused_mix_f64(x, v, g, *SGD, P, so, pe))
    else:
        step, push = cx.cx_sgd_fused_mix_bf16, cx.cx_pushsum_mix_bf16
        put, raw = lambda a: dev(a.view(np.int16)), lambda t: host(t).view(np.uint16)
        x, g = O.f32_to_bf16(x), O.f32_to_bf16(g)
        want_x, want_v = O.sgd_fused_mix16("bf16", x, v, g, *SGD, P, so, pe)
    xd, vd, gd = put(x), dev(v), put(g)
    y, vo, wo, z = torch.full_like(xd, 7), torch.full_like(vd, 7.0), torch.empty(n, device="cuda:0"), torch.full_like(xd, 7)
    with Tuning(ordered=1):
        step(xd, y, vd, vo, gd, *SGD, P, dev(so), dev(pe))
    same = (lambda a, b: same_bits(a, b)) if rows == "f32" else (lambda a, b: bool((a == b).all()))
    assert same(raw(y)[:, :P], want_x[:, :P]) and same_bits(host(vo)[:, :P], want_v[:, :P])
    assert (y[:, P:] == 7).all() and (vo[:, P:] == 7).all()
    results = []
    for ordered in (0, 1):                                     # against the natural order, which takes gather_kernel
        y.fill_(7)
        with Tuning(ordered=ordered):
            push(xd, y, dev(w), wo, z, P, n // 2)
        results.append((raw(y), raw(z), host(wo)))
    assert all((a.view(np.uint8) == b.view(np.uint8)).all() for a, b in zip(*results))
    assert (y[:, P:] == 7).all() and (z[:, P:] == 7).all()


@pytest.mark.parametrize("rows", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n,P,S,pad", [(4, 2049, 3, 1), (17, 5000, 7, 3), (9, 40_001, 5, 1), (150, 3001, 70, 1)])
def test_step_and_push_sum_have_the_bits_of_the_column_grid(rows, n, P, S, pad):
    e, dtype = (4, torch.float32) if rows == "f32" else (8, torch.bfloat16 if rows == "bf16" else torch.float16)
    ld, so, pe = (P + e - 1) // e * e + pad * e, dev(offsets(P, S)), dev(O.topology(S, n, S, 0, 1)[0])
    x, v, g = (dev(WL.gen_matrix(n, P, s, seed=P + n, ld=ld, stream=k)) for k, s in enumerate((0.05, 0.02, 0.01)))
    x, g, w = x.to(dtype), g.to(dtype), dev(np.random.default_rng(n).uniform(0.5, 1.5, n).astype(np.float32))
    suffix, results = "" if rows == "f32" else "_" + rows, []
    print(rows, n, P, S, pad, flush=True)
    for ordered in (0, 1):                                     # the natural order takes the column grid
        a, b, c, z = (torch.full_like(x, 7) for _ in range(4))
        vo, wb, wc = torch.full_like(v, 7), torch.empty_like(w), torch.empty_like(w)
        with Tuning(ordered=ordered):
            getattr(cx, "cx_sgd_fused_mix" + suffix)(x, a, v, vo, g, *SGD, P, so, pe)
            getattr(cx, "cx_pushsum_mix" + suffix)(x, b, w, wb, z, P, n // 2)
            getattr(cx, "cx_pushsum_mix" + suffix)(x, c, w, wc, None, P, n // 2)
        results.append([host(t.view(torch.uint8)) for t in (a, vo, b, wb, z, c, wc)])
        assert all((t[:, P:] == 7).all() for t in (a, vo, b, z, c))
    assert all((p == q).all() for p, q in zip(*results))
