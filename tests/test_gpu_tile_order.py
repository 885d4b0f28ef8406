"""Out of place with the row order looked up by the tile: the oracle's bits and those of the natural row order, where
segments begin and end inside tiles, are empty or shorter than a tile, where there is one, where the table is too small
for the order by the tile (that by the cluster takes over) and with a table that is no permutation."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import Tuning, dev, host, once, same_bits

pytestmark = pytest.mark.gpu

CALLS = {"f32": (torch.float32, 1), "bf16": (torch.bfloat16, 1), "groups": (torch.float32, 3), "groups16": (torch.float16, 4)}


def offsets(P, S, seed):
    inner = np.sort(np.random.default_rng(seed).integers(0, P + 1, size=S - 1))
    if S > 3:
        inner[1] = inner[0]                                    # an empty segment
    return np.concatenate([[0], inner, [P]]).astype(np.int64)


@pytest.mark.parametrize("kind", CALLS)
@pytest.mark.parametrize("n,P,S", [(2, 2049, 1), (5, 2048, 2), (33, 9000, 16), (7, 70_001, 40), (64, 30_011, 5), (1000, 2300, 3),
                                   (12, 40_000, 300), (700, 2500, 400), (1024, 2100, 257),
                                   (8, 70_001, 40), (9, 2048, 2)])      # (fewer than eight rows keep the order by the cluster)
def test_order_by_the_tile(kind, n, P, S):
    dtype, G = CALLS[kind]
    if n * G * P > 30_000_000:
        n = 30_000_000 // (G * P)
    ld, so = (P + 7) // 8 * 8, offsets(P, S, n + P)
    pe = O.topology(S, n, S, 0, 1)[0]
    if P == 30_011:
        pe = np.random.default_rng(3).integers(0, n, size=pe.shape, dtype=np.int32)          # rows chosen twice or never
    x = WL.gen_matrix_device(n * G, P, 0.05, 5, ld=ld, device="cuda:0", out=torch.zeros((n * G, ld), dtype=dtype, device="cuda:0"))
    suffix = {torch.float32: "", torch.bfloat16: "_bf16", torch.float16: "_f16"}[dtype]
    out = []
    print(kind, n, P, S, flush=True)
    for ordered in (0, 1, 1):
        y = torch.full_like(x, float("nan"))
        with Tuning(ordered=ordered):
            if G == 1:
                getattr(cx, "cx_gossip_mix" + suffix)(x, y, P, dev(so), dev(pe))
            else:
                getattr(cx, "cx_hier_mix" + suffix)(x, y, P, G, dev(so), dev(pe))
        out.append(y[:, :P].clone())
        assert torch.isnan(y[:, P:]).all()                     # padding never written
    bits = torch.int32 if dtype == torch.float32 else torch.int16
    assert torch.equal(out[1].view(bits), out[0].view(bits)) and torch.equal(out[2].view(bits), out[0].view(bits))
    if kind == "f32":
        assert same_bits(host(out[1]), O.gossip_mix(host(x), P, so, pe)[:, :P])


@pytest.mark.parametrize("rows", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n,P,S", [(8, 9000, 16), (9, 2049, 2), (33, 70_001, 40), (7, 70_001, 40), (64, 30_011, 5), (700, 2500, 400),
                                   (12, 40_000, 1)])
def test_optimizer_step_in_the_order_by_the_tile(rows, n, P, S):
    """The same for the step on plain rows, momentum included, against the oracle as well."""
    ld, so, sgd = (P + 7) // 8 * 8, offsets(P, S, n + P), (0.1, 0.9, 1e-4)
    pe = O.topology(S, n, S, 0, 1)[0]
    x, v, g = (WL.gen_matrix(n, P, s, seed=P + n, ld=ld, stream=k) for k, s in enumerate((0.05, 0.02, 0.01)))
    if rows == "f32":
        put, call = dev, cx.cx_sgd_fused_mix
        want = [once(t) for t in O.sgd_fused_mix_f64(x, v, g, *sgd, P, so, pe)]
    else:
        narrow = O.f32_to_bf16 if rows == "bf16" else O.f32_to_f16
        x, g = narrow(x), narrow(g)
        put, call = lambda a: dev(a.view(np.int16)), getattr(cx, "cx_sgd_fused_mix_" + rows)
        want = O.sgd_fused_mix16(rows, x, v, g, *sgd, P, so, pe)
    xd, vd, gd = put(x), dev(v), put(g)
    print(rows, n, P, S, flush=True)
    for ordered in (0, 1, 1):
        y, vo = torch.full_like(xd, 7), torch.full_like(vd, 7.0)
        with Tuning(ordered=ordered):
            call(xd, y, vd, vo, gd, *sgd, P, dev(so), dev(pe))
        got = host(y)
        assert same_bits(got[:, :P], want[0][:, :P]) if rows == "f32" else (got.view(np.uint16)[:, :P] == want[0][:, :P]).all()
        assert same_bits(host(vo)[:, :P], want[1][:, :P])
        assert (got[:, P:] == 7).all() and (host(vo)[:, P:] == 7).all()
