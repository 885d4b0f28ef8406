"""Performance cases of the mixing library: the gossip rounds that a user's training loop has it do.

A case is one round of one entry point on one shape.  What a program keeps between rounds is prepared
beforehand: the worker matrices, the segment offsets and the peer tables of the next ROUNDS rounds, drawn and
uploaded in one go.  A pass is the one call that the loop makes per round.

    kind      gossip, hier, fused (momentum-SGD and mix), hiersgd (group gradients, SGD and mix), pushsum
    rows      f32, bf16 or f16: the type of the parameter (and gradient) rows
    W, P      workers and parameters per worker;  G: workers per group;  S: segments per vector
    layers    0: S equal segments; otherwise segments end on the edges of this many ragged layers
    ld_of     rows are padded to a multiple of this many columns
    in_place  the round updates its buffers instead of writing a second set
    debias    pushsum only: also writes the de-biased parameters that the next forward pass uses
"""
from __future__ import annotations

import math

import torch

from paper_2012_15198_amd import cxmix as cx
from paper_2012_15198_amd import workloads as wl

ROUNDS = 8                                   # peer tables at hand, used in turn
LR, MU, WD = 0.1, 0.9, 1e-4                  # the optimizer constants of the repository's workload C4
SIGMA_X, SIGMA_V, SIGMA_G = 0.05, 0.02, 0.01
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEVICE = "cuda:0"


def _case(name, kind, rows, W, P, S, G=1, layers=0, ld_of=1024, in_place=False, debias=False):
    case = {"kind": kind, "rows": rows, "W": W, "P": P, "S": S, "G": G, "layers": layers, "ld_of": ld_of,
            "in_place": in_place, "debias": debias}
    return {"name": name, **case} if name else case


def listed():
    """The repository's workloads C1 to C5 and shapes between and around them."""
    return [
        # a toy model on a handful of workers: a first run, a unit test, a parameter sweep of the method
        _case("toy-gossip", "gossip", "f32", 4, 20_011, 2, ld_of=4),
        # C1: eight workers, a model of a million parameters
        _case("c1-gossip", "gossip", "f32", 8, 1_000_000, 4),
        # hundreds of workers on a small ragged model: how the method scales with the number of workers
        _case("many-workers", "gossip", "f32", 512, 100_003, 16, layers=40, ld_of=4),
        # the same kind of study with the optimizer fused in, one set of buffers
        _case("many-workers-fused-inplace", "fused", "f32", 256, 300_007, 8, ld_of=4, in_place=True),
        # C2: the headline round of the benchmark
        _case("c2-gossip", "gossip", "f32", 32, 25_557_032, 8),
        # C2 on mixed-precision rows, one buffer, segments on layer edges
        _case("c2-bf16-inplace", "gossip", "bf16", 32, 25_557_032, 8, layers=161, in_place=True),
        # C3: eight groups of eight with their means
        _case("c3-hier", "hier", "f32", 64, 11_689_512, 16, G=8),
        # sixteen groups of four on binary16 rows of odd length, packed as tightly as the rows may be, in place
        _case("hier-f16-inplace", "hier", "f16", 64, 11_689_511, 16, G=4, layers=62, ld_of=8, in_place=True),
        # C3's shape with the group's gradients reduced at the leader, mixed precision: a training step
        _case("c3-hiersgd-bf16", "hiersgd", "bf16", 64, 11_689_512, 16, G=8),
        # C4: the largest state, optimizer and mix in one step
        _case("c4-fused", "fused", "f32", 128, 25_557_032, 8),
        # the push-sum comparison as its training loop runs it, de-biased parameters included
        _case("pushsum-bf16-debias", "pushsum", "bf16", 128, 11_689_513, 1, ld_of=8, debias=True),
        # C5: 32 groups of eight, segments on ragged layers
        _case("c5-hier", "hier", "f32", 256, 25_557_032, 32, G=8, layers=161),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any entry point on any row type: up to 1024 gossiping rows, 1,000 to 25.6 million parameters, up to 24 GB."""
    while True:
        kind = rng.choice(["gossip", "gossip", "hier", "fused", "hiersgd", "pushsum"])
        rows = rng.choice(["f32", "f32", "bf16", "f16"])
        G = rng.choice([2, 3, 4, 6, 8, 8]) if kind in ("hier", "hiersgd") else 1
        W = G * _log_uniform(rng, 1, 64) if G > 1 else _log_uniform(rng, 2, 1024)   # one group: the plain mean
        P = _log_uniform(rng, 1_000, 25_557_032)
        S = 1 if kind == "pushsum" else rng.randint(1, 32)
        layers = rng.randint(S, 5 * S) if S > 1 and rng.random() < 0.5 else 0
        case = _case(None, kind, rows, W, P, S, G, layers, rng.choice([8, 1024]), rng.random() < 0.4,
                     kind == "pushsum" and rng.random() < 0.5)
        if work(case)["bytes"] <= 24e9:
            return case


def _element_bytes(case):
    return 4 if case["rows"] == "f32" else 2


def work(case):
    """Each worker's parameters are read once and written once; the fused steps also read the gradients and read
    and write the momentum (of the leaders alone in the grouped one, which reads only the leaders' parameters);
    the de-biased copy is written once.  Operations: those of the formulas, per element."""
    W, P, G, e, kind = case["W"], case["P"], case["G"], _element_bytes(case), case["kind"]
    N, L = W * P, (W // G) * P
    if kind == "fused":
        traffic, flops = N * (3 * e + 8), 8 * N
    elif kind == "hiersgd":
        traffic, flops = N * 2 * e + L * (e + 8), N + 9 * L
    elif kind == "hier":
        traffic, flops = N * 2 * e, N + 3 * L
    else:
        traffic, flops = N * 2 * e + (N * e if case["debias"] else 0), (3 if case["debias"] else 2) * N
    return {"bytes": traffic + 4 * case["S"] * (W // G), "flops": flops}


def tolerance(case):
    """Every result is defined to the bit: the fp32 formula as written, or the fp64 formula rounded once."""
    return "exact"


def prepare(case, seed):
    W, P, S, G, kind = case["W"], case["P"], case["S"], case["G"], case["kind"]
    rows, n = TYPES[case["rows"]], W // G
    ld = -(-P // case["ld_of"]) * case["ld_of"]

    def matrix(count, dtype, sigma, stream):
        out = torch.empty((count, ld), dtype=dtype, device=DEVICE)
        return wl.gen_matrix_device(count, P, sigma, seed, ld=ld, stream=stream, device=DEVICE, out=out)

    def second(t):
        return t if case["in_place"] else torch.empty_like(t)

    state = {"case": case, "round": 0, "x": matrix(W, rows, SIGMA_X, 0)}
    state["y"] = second(state["x"])
    if kind in ("fused", "hiersgd"):
        state["v"] = matrix(W if kind == "fused" else n, torch.float32, SIGMA_V, 1)
        state["v2"] = second(state["v"])
        state["g"] = matrix(W, rows, SIGMA_G, 2)
    if kind == "pushsum":
        state["w"] = 0.5 + torch.rand(W, device=DEVICE, generator=torch.Generator(DEVICE).manual_seed(seed))
        state["w2"] = torch.empty_like(state["w"])
        state["z"] = torch.empty_like(state["x"]) if case["debias"] else None
        return state
    sizes = wl.layer_sizes(P, case["layers"], seed=5) if case["layers"] else None      # the model's, not the data's
    offsets = wl.equal_seg_off(P, S) if sizes is None else wl.layer_aligned_seg_off(sizes, S)
    cx.cx_check_segments(offsets, P)
    state["offsets"] = torch.from_numpy(offsets).to(DEVICE)
    if n == 1:                               # nobody to gossip with
        state["peers"] = [None] * ROUNDS
        return state
    tables = cx.cx_topology_gen(seed, n, S, 0, ROUNDS)
    for table in tables:
        cx.cx_check_peers(table)
    state["peers"] = list(torch.from_numpy(tables).to(DEVICE))
    return state


def run(state):
    """One round.  The fused steps carry parameters and momentum from round to round; a plain round starts from
    the parameters that the loop's own optimizer would just have written to x."""
    case, s = state["case"], state
    kind, P, r = case["kind"], case["P"], s["round"]
    call = getattr(cx, {"gossip": "cx_gossip_mix", "hier": "cx_hier_mix", "fused": "cx_sgd_fused_mix",
                        "hiersgd": "cx_hier_sgd_fused_mix", "pushsum": "cx_pushsum_mix"}[kind]
                   + ("" if case["rows"] == "f32" else "_" + case["rows"]))
    s["round"] = r + 1
    if kind == "pushsum":
        hop = 1 << (r % max(1, (case["W"] - 1).bit_length()))
        call(s["x"], s["y"], s["w"], s["w2"], s["z"], P, hop)
        return [t for t in (s["y"][:, :P], s["w2"], s["z"][:, :P] if case["debias"] else None) if t is not None]
    peers = s["peers"][r % ROUNDS]
    if kind == "gossip":
        call(s["x"], s["y"], P, s["offsets"], peers)
        return [s["y"][:, :P]]
    if kind == "hier":
        call(s["x"], s["y"], P, case["G"], s["offsets"], peers)
        return [s["y"][:, :P]]
    grouped = (case["G"],) if kind == "hiersgd" else ()
    call(s["x"], s["y"], s["v"], s["v2"], s["g"], LR, MU, WD, P, *grouped, s["offsets"], peers)
    s["x"], s["y"], s["v"], s["v2"] = s["y"], s["x"], s["v2"], s["v"]
    return [s["x"][:, :P], s["v"][:, :P]]
