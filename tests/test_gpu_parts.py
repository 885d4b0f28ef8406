"""In place with the rows of a tile split over wavefronts: the rows' parts against the out-of-place kernel, bit for bit, at
the edges of the rule -- one row a part and less, the most parts, odd parts of cycles, rows that end inside a tile and a
slice, segment boundaries inside a workgroup's columns, both rings -- and the oracle on both sides of where the rule ends."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import dev, in_place_equals_the_oracle

pytestmark = pytest.mark.gpu

KINDS = {"gossip": ("f32", 1), "gossip16": ("bf16", 1), "fused": ("f32", 1), "fused16": ("f16", 1), "hier": ("f32", 3),
         "hier5": ("f32", 5), "hier16": ("bf16", 8), "hiersgd": ("f32", 2), "hiersgd16": ("f16", 4), "pushsum": ("f32", 1), "pushsum16": ("bf16", 1)}
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def mixed(kind, n, P, so, in_place, seed):
    rows, G = KINDS[kind]
    ld = (P + 7) // 8 * 8
    t = TYPES[rows]
    make = lambda count, dtype, k: WL.gen_matrix_device(count, P, 0.05, seed, ld=ld, stream=k, device="cuda:0",
                                                        out=torch.zeros((count, ld), dtype=dtype, device="cuda:0"))
    second = lambda a: a if in_place else torch.zeros_like(a)
    x = make(n * G, t, 0)
    y = second(x)
    call = getattr(cx, {"gossip": "cx_gossip_mix", "fused": "cx_sgd_fused_mix", "hier": "cx_hier_mix", "hiersgd":
                        "cx_hier_sgd_fused_mix", "pushsum": "cx_pushsum_mix"}[kind.rstrip("156")] + ("" if rows == "f32" else "_" + rows))
    if kind.startswith("pushsum"):
        w, w2, z = torch.rand(n, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(seed)) + 0.5, torch.zeros(n, device="cuda:0"), torch.zeros_like(x)
        call(x, y, w, w2, z, P, max(1, n // 3))
        return y, z, w2
    tables = dev(so), dev(O.topology(seed, n, len(so) - 1, 0, 1)[0])
    if kind.startswith("gossip"):
        call(x, y, P, *tables)
        return (y,)
    if kind.rstrip("156") == "hier":
        call(x, y, P, G, *tables)
        return (y,)
    v, g = make(n, torch.float32, 1), make(n * G, t, 2)
    v2 = second(v)
    call(x, y, v, v2, g, 0.1, 0.9, 1e-4, P, *((G,) if kind.startswith("hiersgd") else ()), *tables)
    return y, v2


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,P", [(4, 9), (5, 1000), (8, 256), (9, 513), (16, 2047), (17, 30_001), (33, 4099), (130, 1027), (1000, 301),
                                 (7, 102_401), (16, 102_145), (12, 204_809), (33, 261_003), (33, 270_003), (8, 1_048_577), (33, 1_048_331), (40, 2_097_163)])
def test_parts_equal_the_out_of_place_kernel(kind, n, P):
    G = KINDS[kind][1]
    if n * G * P > 100_000_000:
        n = max(4, 100_000_000 // (G * P))
    so = np.array([0, P // 5, P // 5, P // 2 + 1, P - 1, P], dtype=np.int64)
    print(kind, n, P, flush=True)
    for got, want in zip(mixed(kind, n, P, so, True, 7 + n), mixed(kind, n, P, so, False, 7 + n)):
        bits = torch.int32 if got.dtype == torch.float32 else torch.int16
        assert torch.equal(got.view(bits)[..., :P], want.view(bits)[..., :P])


# (kind, rows per group, gossiping rows, tiles below the edge, segments, whole lines): the short ring's and the long ring's
# lengths, ends of the first round, halves of the later rounds of 2,048 tiles and of the shorter ones beside 500 rows, up to
# eight very long rows
EDGES = [("gossip", 1, 9, 399, 4), ("gossip", 1, 16, 1536, 4), ("gossip", 1, 17, 2048, 4), ("gossip", 1, 16, 3072, 1),
         ("gossip", 1, 8, 16383, 4), ("gossip", 1, 5, 16383, 1), ("pushsum", 1, 5, 16383, 1), ("pushsum", 1, 8, 16383, 1),
         ("pushsum", 1, 9, 399, 1), ("pushsum", 1, 33, 1024, 1), ("debias", 1, 16, 2048, 1), ("debias", 1, 17, 3072, 1),
         ("fused", 1, 33, 1024, 4), ("fused", 1, 17, 512, 1), ("fused", 1, 16, 2048, 4), ("hier", 2, 33, 1024, 4), ("hier", 4, 16, 2048, 4),
         ("hier", 8, 33, 1024, 3), ("hier", 5, 6, 256, 1), ("hiersgd", 8, 5, 128, 3), ("hiersgd", 2, 16, 512, 1), ("hiersgd", 6, 33, 256, 1),
         ("gossip16", 1, 16, 1536, 4), ("gossip16", 1, 9, 3072, 4), ("gossip", 1, 500, 1536, 1), ("pushsum16", 1, 9, 1536, 1),
         ("debias16", 1, 16, 2048, 1), ("hier16", 2, 9, 1024, 1), ("hier16", 8, 9, 640, 1), ("fused16", 1, 9, 1536, 4), ("fused16", 1, 17, 768, 1),
         ("hiersgd16", 3, 9, 512, 1), ("hiersgd16", 2, 9, 1536, 4)]


@pytest.mark.parametrize("kind,G,n,tiles,S", EDGES)
@pytest.mark.parametrize("beyond", [0, 1])
def test_both_sides_of_the_rule_against_the_oracle(kind, G, n, tiles, S, beyond):
    P = tiles * (512 if kind.endswith("16") else 256) + beyond
    ld = P // 8 * 8 + 8
    if ld * (2 if kind.endswith("16") else 4) % 128 == 0:
        ld += 8                                                # rows begin inside lines
    so = np.array([0, P // 3 + 1, P // 3 + 1, P - 2, P], dtype=np.int64)[[0, *range(5 - S, 5)]]
    print(kind, G, n, P, S, flush=True)
    in_place_equals_the_oracle(kind, G, n, P, ld, so)


@pytest.mark.parametrize("apart", ["v", "x"])
@pytest.mark.parametrize("n,P", [(4, 1000), (17, 30_001), (33, 103_001)])
def test_only_one_of_parameters_and_momentum_in_place(n, P, apart):
    """The fp32 step on plain rows takes that, in the in-place kernels: what a row's owner writes, others still read."""
    print(n, P, apart, flush=True)
    in_place_equals_the_oracle("fused", 1, n, P, P // 8 * 8 + 8, np.array([0, P // 3 + 1, P], dtype=np.int64), apart)
