"""In place with the rows of a tile split over wavefronts: the rows' parts against the out-of-place kernel, bit for bit, at
the edges of the rule -- one row a part and less, the most parts, odd parts of cycles, rows that end inside a tile and a
slice, segment boundaries inside a workgroup's columns, both rings."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import dev

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
                                 (7, 102_401), (16, 102_145), (12, 204_809), (33, 270_003), (8, 1_048_577), (33, 1_048_331), (40, 2_097_163)])
def test_parts_equal_the_out_of_place_kernel(kind, n, P):
    G = KINDS[kind][1]
    if n * G * P > 100_000_000:
        n = max(4, 100_000_000 // (G * P))
    so = np.array([0, P // 5, P // 5, P // 2 + 1, P - 1, P], dtype=np.int64)
    print(kind, n, P, flush=True)
    for got, want in zip(mixed(kind, n, P, so, True, 7 + n), mixed(kind, n, P, so, False, 7 + n)):
        bits = torch.int32 if got.dtype == torch.float32 else torch.int16
        assert torch.equal(got.view(bits)[..., :P], want.view(bits)[..., :P])
