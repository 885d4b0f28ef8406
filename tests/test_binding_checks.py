"""CPU-only tests of the Python binding's argument checks.  The C ABI sees one leading dimension and
raw addresses, so a tensor of the wrong shape, stride, element type or device must be refused before
anything is launched: every case below raises ValueError on host tensors (the device check comes
last, so the other mismatches are reachable without a GPU), and the all-correct host case raises the
device error -- no call reaches the library."""
import pytest
import torch

from paper_2012_15198_amd import cxmix as cx

W, P, LD, S, G = 8, 60, 64, 3, 2


def mat(rows=W, ld=LD, dtype=torch.float32):
    return torch.zeros((rows, ld), dtype=dtype)


def tables(n=W, S=S):
    return torch.tensor([0, 20, 40, P], dtype=torch.int64)[:S + 1], torch.zeros((S, n), dtype=torch.int32)


def refuses(fn, *args, match):
    with pytest.raises(ValueError, match=match):
        fn(*args)


def test_correct_host_tensors_reach_only_the_device_check():
    so, pe = tables()
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so, pe, match="device tensors")
    refuses(cx.cx_sgd_fused_mix, mat(), mat(), mat(), mat(), mat(), 0.1, 0.9, 1e-4, P, so, pe, match="device tensors")
    so2, pe2 = tables(W // G)
    refuses(cx.cx_hier_mix, mat(), mat(), P, G, so2, pe2, match="device tensors")
    refuses(cx.cx_hier_sgd_fused_mix, mat(), mat(), mat(W // G), mat(W // G), mat(), 0.1, 0.9, 1e-4, P, G, so2, pe2,
            match="device tensors")
    refuses(cx.cx_pushsum_mix, mat(), mat(), torch.ones(W), torch.ones(W), None, P, 1, match="device tensors")
    refuses(cx.cx_gossip_mix_bf16, mat(dtype=torch.bfloat16), mat(dtype=torch.bfloat16), P, so, pe, match="device tensors")
    refuses(cx.cx_copy_baseline, torch.zeros(64), torch.zeros(64), match="device tensors")


@pytest.mark.parametrize("bad,match", [
    (lambda: mat(ld=P), "row stride"),                           # unpadded next to a padded x_in
    (lambda: mat(rows=W - 1), "rows"),
    (lambda: mat(dtype=torch.float64), "float32"),
    (lambda: mat(dtype=torch.bfloat16), "float32"),
    (lambda: mat(dtype=torch.int32), "float32"),
    (lambda: mat(ld=2 * LD)[:, ::2], "row-major"),               # strided columns
    (lambda: torch.zeros(W * LD), "row-major"),                  # not a matrix
])
def test_every_matrix_argument_is_checked_against_x_in(bad, match):
    so, pe = tables()
    refuses(cx.cx_gossip_mix, mat(), bad(), P, so, pe, match=match)
    refuses(cx.cx_gossip_mix, bad(), mat(), P, so, pe, match=".")          # x_in itself or the mismatch of x_out
    for slot in range(1, 5):                                               # x_out, v_in, v_out, g
        args = [mat(), mat(), mat(), mat(), mat()]
        args[slot] = bad()
        refuses(cx.cx_sgd_fused_mix, *args, 0.1, 0.9, 1e-4, P, so, pe, match=match)
    so2, pe2 = tables(W // G)
    refuses(cx.cx_hier_mix, mat(), bad(), P, G, so2, pe2, match=match)
    refuses(cx.cx_pushsum_mix, mat(), bad(), torch.ones(W), torch.ones(W), None, P, 1, match=match)
    refuses(cx.cx_pushsum_mix, mat(), mat(), torch.ones(W), torch.ones(W), bad(), P, 1, match=match)


@pytest.mark.parametrize("columns", [slice(0, P - 1), slice(LD // 2, LD), slice(4, P), slice(0, 0)])
def test_every_matrix_argument_holds_P_columns(columns):
    """A view with x_in's row stride and fewer than P columns: the kernels would write beyond it, for the last row beyond
    the allocation.  Exactly P columns are enough."""
    so, pe = tables()
    so2, pe2 = tables(W // G)
    w = lambda: torch.ones(W)
    b16 = lambda *a: mat(*a, dtype=torch.bfloat16)
    calls = [(cx.cx_gossip_mix, [mat, mat], (P, so, pe)), (cx.cx_gossip_mix_noalloc, [mat, mat], (P, so, pe)),
             (cx.cx_gossip_mix_bf16, [b16, b16], (P, so, pe)), (cx.cx_hier_mix, [mat, mat], (P, G, so2, pe2)),
             (cx.cx_hier_mix_f16, [b16, b16], (P, G, so2, pe2)),
             (cx.cx_sgd_fused_mix, [mat] * 5, (0.1, 0.9, 1e-4, P, so, pe)),
             (cx.cx_sgd_fused_mix_bf16, [b16, b16, mat, mat, b16], (0.1, 0.9, 1e-4, P, so, pe)),
             (cx.cx_hier_sgd_fused_mix, [mat, mat, lambda: mat(W // G), lambda: mat(W // G), mat], (0.1, 0.9, 1e-4, P, G, so2, pe2)),
             (cx.cx_hier_sgd_fused_mix_f16, [b16, b16, lambda: mat(W // G), lambda: mat(W // G), b16],
              (0.1, 0.9, 1e-4, P, G, so2, pe2)),
             (lambda x, y, z, *r: cx.cx_pushsum_mix(x, y, w(), w(), z, *r), [mat, mat, mat], (P, 1)),
             (lambda x, y, z, *r: cx.cx_pushsum_mix_bf16(x, y, w(), w(), z, *r), [b16, b16, b16], (P, 1))]
    for on_device in (False, True):
        view = lambda make, c: OnDevice(make()[:, c]) if on_device else make()[:, c]
        tail = lambda rest: [OnDevice(t) if on_device and torch.is_tensor(t) else t for t in rest]
        for call, makes, rest in calls[:9] if on_device else calls:
            for slot in range(1, len(makes)):
                refuses(call, *[view(m, columns if i == slot else slice(0, P)) for i, m in enumerate(makes)], *tail(rest),
                        match=f"columns, P is {P}")
    x = OnDevice(mat()[:, :P])
    assert cx._full_checks(x, 4, (("x_out", x, 1, 4),), P, 1, OnDevice(so), OnDevice(pe), ()) == (W, LD, S)
    assert cx._ready(x, 4, (("x_out", OnDevice(mat()[:, columns]), 1, 4),), P, 1, OnDevice(so), OnDevice(pe), ()) is None


def test_hierarchical_gradient_step_checks_the_leader_momentum_shape():
    so, pe = tables(W // G)
    L = W // G
    ok = lambda: [mat(), mat(), mat(L), mat(L), mat()]
    for slot, bad, match in [(2, mat(W), "rows"), (3, mat(L, ld=P), "row stride"), (4, mat(L), "rows"),
                             (1, mat(dtype=torch.float16), "float32")]:
        args = ok()
        args[slot] = bad
        refuses(cx.cx_hier_sgd_fused_mix, *args, 0.1, 0.9, 1e-4, P, G, so, pe, match=match)
    refuses(cx.cx_hier_sgd_fused_mix, *ok(), 0.1, 0.9, 1e-4, P, 3, so, pe, match="divide")


def test_16bit_entry_points_refuse_other_element_sizes():
    so, pe = tables()
    b = lambda: mat(dtype=torch.bfloat16)
    refuses(cx.cx_gossip_mix_bf16, mat(), b(), P, so, pe, match="16-bit")
    refuses(cx.cx_gossip_mix_f16, b(), mat(), P, so, pe, match="16-bit")
    refuses(cx.cx_gossip_mix_bf16, b(), mat(ld=P, dtype=torch.bfloat16), P, so, pe, match="row stride")
    so2, pe2 = tables(W // G)
    refuses(cx.cx_hier_mix_bf16, b(), mat(), P, G, so2, pe2, match="16-bit")
    refuses(cx.cx_gossip_mix, b(), b(), P, so, pe, match="float32")
    refuses(cx.cx_pushsum_mix_bf16, b(), mat(), torch.ones(W), torch.ones(W), None, P, 1, match="16-bit")
    refuses(cx.cx_pushsum_mix_f16, b(), b(), torch.ones(W), torch.ones(W), mat(), P, 1, match="16-bit")
    refuses(cx.cx_pushsum_mix_bf16, b(), b(), torch.ones(W - 1), torch.ones(W), None, P, 1, match="w_in")
    refuses(cx.cx_pushsum_mix, b(), b(), torch.ones(W), torch.ones(W), None, P, 1, match="float32")


def test_tables_and_vectors_are_checked():
    so, pe = tables()
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so.to(torch.int32), pe, match="seg_off_dev")
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so, pe.to(torch.int64), match="peers_dev")
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so, pe[:, :W - 1], match="peers_dev")
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so, torch.zeros((S, W + 1), dtype=torch.int32), match="peers_dev")
    refuses(cx.cx_gossip_mix, mat(), mat(), P, so[:1], pe, match="seg_off_dev")
    refuses(cx.cx_gossip_mix, mat(), mat(), LD + 1, so, pe, match="P must")
    refuses(cx.cx_hier_mix, mat(), mat(), P, G, so, pe, match="peers_dev")          # table for W rows, not W/G
    refuses(cx.cx_pushsum_mix, mat(), mat(), torch.ones(W - 1), torch.ones(W), None, P, 1, match="w_in")
    refuses(cx.cx_pushsum_mix, mat(), mat(), torch.ones(W), torch.ones(W, dtype=torch.float64), None, P, 1, match="w_out")
    refuses(cx.cx_copy_baseline, torch.zeros(64), torch.zeros(32), match="dst")


class OnDevice:
    """A host tensor that says it lives on a GPU: the argument checks ask a tensor for nothing but its properties."""
    is_cuda = True

    def __init__(self, tensor, device="cuda:0"):
        self.tensor, self.device = tensor, torch.device(device)

    def __getattr__(self, name):
        return getattr(self.tensor, name)


def vec(n=W, dtype=torch.float32):
    return torch.ones(n, dtype=dtype)


@pytest.mark.parametrize("kind", ["gossip", "hier", "fused", "hiersgd", "gossip16", "fused16", "pushsum"])
def test_the_short_way_through_the_checks_accepts_only_what_the_full_checks_accept(kind):
    """_ready() answers for the usual tensors: what it accepts the full checks accept with the same geometry, and of the
    correct call it is not silent; every call with one odd argument gets the full checks' answer."""
    cx.lib()
    size = 2 if kind.endswith("16") else 4
    x = lambda: mat(dtype=torch.bfloat16 if size == 2 else torch.float32)
    G_of = G if kind.startswith("hier") else 1
    mats = {"gossip": [x], "hier": [x], "gossip16": [x], "fused": [x, mat, mat, x], "fused16": [x, mat, mat, x],
            "hiersgd": [x, lambda: mat(W // G), lambda: mat(W // G), x], "pushsum": [x, x]}[kind]
    rows_of = [1, G_of, G_of, 1] if len(mats) == 4 else [1] * len(mats)
    sizes = [size, 4, 4, size] if len(mats) == 4 else [size] * len(mats)
    so, pe = tables(W // G_of)
    good = [x()] + [m() for m in mats] + ([vec(), vec()] if kind == "pushsum" else [so, pe])
    odd = [mat(), mat(ld=P), mat(rows=W - 1), mat(rows=1), mat(rows=W // G), mat(ld=LD + 1)[:, :LD], mat(ld=2 * LD)[:, ::2],
           mat(ld=LD + 8)[:, 8:], torch.zeros((W + 1) * LD).as_strided((W, LD + 1), (LD, 1)), torch.zeros(W, 2, LD),
           torch.zeros(W * LD), mat(dtype=torch.int32), mat(dtype=torch.float64), mat(dtype=torch.bfloat16),
           mat(dtype=torch.int16), vec(), vec(W + 3), vec(W - 1), vec(2 * W)[::2], vec(dtype=torch.float64),
           vec(dtype=torch.int32), so, so[:1], so.to(torch.int32), so.repeat(2)[::2], pe, pe[:, 1:], pe.to(torch.int64), pe.t(),
           pe.reshape(-1), pe.to(torch.float32), None]

    def ask(check, args, cols, groups, elsewhere=None):
        t = [a if a is None else OnDevice(a, "cuda:1" if i == elsewhere else "cuda:0") for i, a in enumerate(args)]
        m = tuple((f"m{i}", a, r, s) for i, (a, r, s) in enumerate(zip(t[1:], rows_of, sizes)))
        tail = t[1 + len(m):]
        try:
            if kind == "pushsum":
                return check(t[0], size, m, cols, groups, None, None, (("w_in", tail[0]), ("w_out", tail[1])))
            return check(t[0], size, m, cols, groups, tail[0], tail[1], ())
        except (ValueError, AttributeError):
            return "refused"

    assert ask(cx._ready, good, P, G_of) == ask(cx._full_checks, good, P, G_of) == (W, LD, 1 if kind == "pushsum" else S)
    calls = [(good, cols, groups, None) for cols in (0, 1, LD, LD + 1) for groups in (G_of, 0, -1, 3, W, 2 * W)]
    calls += [(good, P, G_of, i) for i in range(len(good))]
    calls += [(good[:i] + [bad] + good[i + 1:], P, G_of, None) for i in range(len(good)) for bad in odd]
    for args, cols, groups, elsewhere in calls:
        if args[0] is None or (groups != G_of and kind == "hiersgd" and groups < 1):
            continue
        short = ask(cx._ready, args, cols, groups, elsewhere)
        assert short in (None, "refused") or short == ask(cx._full_checks, args, cols, groups, elsewhere)
