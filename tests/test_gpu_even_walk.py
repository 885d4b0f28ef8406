"""In place on many plain rows of medium length, where the waves of a workgroup are chosen to deal the tiles out evenly:
the bits of the out-of-place kernels at both ends of that rule's lengths and rows, where the split or the usual walk serves, and
at every count of waves and slices that the rule chooses.  Which call takes what is pinned in tests/host/launch_shapes_check.hip."""
import pytest
import torch

import oracle as O
from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as WL
from gpu_util import dev

pytestmark = pytest.mark.gpu

SGD = (0.1, 0.9, 1e-4)


@pytest.mark.parametrize("kind", ["gossip", "step", "push"])
@pytest.mark.parametrize("rows", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n,slices,beyond,S", [(24, 1024, 1, 3), (23, 1024, 1, 3), (120, 1172, -25, 8), (25, 1279, 77, 30), (26, 6143, 5, 2), (101, 1172, 3, 40), (513, 1030, 9, 5),
                                               (500, 1100, 0, 1)])
def test_even_walk_equals_the_out_of_place_kernel(kind, rows, n, slices, beyond, S):
    P = slices * (256 if rows == "f32" else 512) + beyond
    ld, dtype = (P + 7) // 8 * 8 + 8, {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[rows]
    suffix = "" if rows == "f32" else "_" + rows
    print(kind, rows, n, P, S, flush=True)

    def matrix(t, sigma, stream):
        out = WL.gen_matrix_device(n, P, sigma, 9, ld=ld, stream=stream, device="cuda:0", out=torch.empty((n, ld), dtype=t, device="cuda:0"))
        out[:, P:] = 7
        return out

    x, y = matrix(dtype, 0.05, 0), torch.full((n, ld), 7, dtype=dtype, device="cuda:0")
    so, pe = dev(WL.equal_seg_off(P, S)), dev(O.topology(S, n, S, 0, 1)[0])
    if kind == "gossip":
        call = getattr(cx, "cx_gossip_mix" + suffix)
        call(x, y, P, so, pe)
        call(x, x, P, so, pe)
    elif kind == "step":
        call, v, g = getattr(cx, "cx_sgd_fused_mix" + suffix), matrix(torch.float32, 0.02, 1), matrix(dtype, 0.01, 2)
        v2 = torch.full_like(v, 7)
        call(x, y, v, v2, g, *SGD, P, so, pe)
        call(x, x, v, v, g, *SGD, P, so, pe)
        assert torch.equal(v.view(torch.int32)[:, :P], v2.view(torch.int32)[:, :P]) and (v[:, P:] == 7).all()
    else:
        call, w = getattr(cx, "cx_pushsum_mix" + suffix), torch.rand(n, device="cuda:0") + 0.5
        w2, w3 = torch.empty_like(w), torch.empty_like(w)
        call(x, y, w, w2, None, P, 1 + n // 3)
        call(x, x, w, w3, None, P, 1 + n // 3)
        assert torch.equal(w2, w3)
    bits = torch.int32 if rows == "f32" else torch.int16
    assert torch.equal(x.view(bits)[:, :P], y.view(bits)[:, :P]) and (x[:, P:] == 7).all()


# one slice a lane: three, four, six and eight waves a workgroup; two slices: three to six
@pytest.mark.parametrize("kind,rows,n,P,S", [
    ("gossip", "f32", 24, 522_735, 17), ("gossip", "f32", 512, 323_055, 17), ("gossip", "f32", 400, 455_919, 17), ("gossip", "f32", 400, 688_623, 1),
    ("gossip", "bf16", 33, 1_045_487, 17), ("gossip", "f16", 24, 1_033_199, 17), ("gossip", "bf16", 400, 911_855, 17),
    ("step", "f32", 24, 390_639, 8), ("step", "f32", 512, 323_055, 17), ("step", "f32", 400, 455_919, 17),
    ("step", "f16", 24, 2_612_207, 17), ("step", "bf16", 24, 656_879, 1), ("step", "f16", 24, 524_783, 1),
    ("push", "f32", 24, 525_039, 1), ("push", "f32", 24, 590_319, 1), ("push", "f32", 24, 655_599, 1), ("push", "f32", 400, 458_991, 1),
    ("push", "bf16", 64, 656_879, 1)])
def test_every_shape_of_the_even_walk(kind, rows, n, P, S):
    test_even_walk_equals_the_out_of_place_kernel(kind, rows, n, 0, P, S)
